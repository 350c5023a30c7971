"""A distribution value near the top of the FP32 range overflows in f^{n+1},
also at velocities whose wall adjoint is zero: the products 0 x inf of the wall
rows' position adjoint stay in it, so the loss shows in the gradient."""
import pytest
import torch

import paper_2408_02350_amd.adjoint as A
import paper_2408_02350_amd.bgk as B
from paper_2408_02350_amd.inputs import CavityConfig

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_overflowed_rows_reach_the_position_gradient_of_their_walls():
    cav = CavityConfig("big", 2, 9, 8, 4.0, 2.4, 0.8, 0.1, 1, 0)
    p = A.MovingCavity(cav, device=DEV, seed=1, precision="fp32")
    c, x = p.ctx, p.x0
    inner = torch.nonzero(p.wall_id == 0)[:, 0]
    f = p.rest_state()
    rho, U, T = B.bgk_moments(c, f)
    f[0, inner[len(inner) // 2], 3] = 1e38
    f1, U1 = torch.empty_like(f), U.clone()
    B.bgk_step(c, f, f1, x.clone(), U1, rho.clone(), T.clone())
    zero, zU, dlid = torch.zeros_like(f), torch.zeros_like(U), U.new_zeros(1)
    lx = torch.empty_like(U)
    B.bgk_adjoint_step_move(c, f, U, x, zero, zU, zU, None, None, torch.empty_like(f),
                            torch.empty_like(U), lx, dlid)
    cnt, idx, _, _ = (t.cpu() for t in B.bgk_wall_stencil(c, x))
    bad = ~torch.isfinite(f1).all(dim=2).all(dim=0).cpu()
    hit = [b for b in torch.nonzero(p.wall_id)[:, 0].tolist() if bad[idx[b, :cnt[b]].long()].any()]
    assert hit and torch.isnan(lx[:, hit]).all()


@pytest.mark.parametrize("component", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_edges_under_a_nan_velocity_take_no_part_in_2d(component, precision):
    # no projection of a NaN is negative: the particle keeps its row (the
    # forward step drops its upwind terms) and its edges have no adjoint
    cav = CavityConfig("nan", 2, 9, 8, 4.0, 2.4, 0.8, 0.1, 1, 0)
    p = A.MovingCavity(cav, device=DEV, seed=1, precision=precision)
    c, x = p.ctx, p.x0
    inner = torch.nonzero(p.wall_id == 0)[:, 0]
    f = p.rest_state()
    _, U, _ = B.bgk_moments(c, f)
    U[component, inner[len(inner) // 2]] = float("nan")
    f1, U1, rho, T = torch.empty_like(f), U.clone(), U.new_empty(c.N), U.new_empty(c.N)
    B.bgk_step(c, f, f1, x.clone(), U1, rho, T)
    assert torch.isfinite(f1).all()
    lam = torch.rand(f.shape, generator=torch.Generator().manual_seed(2)).to(f)
    zU, dlid = torch.zeros_like(U), U.new_zeros(1)
    lx = torch.empty_like(U)
    B.bgk_adjoint_step_move(c, f, U, x, lam, zU, zU, None, None, torch.empty_like(f),
                            torch.empty_like(U), lx, dlid)
    assert torch.isfinite(lx).all()
