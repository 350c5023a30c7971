"""The reverse step's interior patches at every lane width of their launch plan:
full and ragged velocity lines, tiles that are nearly empty, and both storage
types.  Checked as the transpose of the oracle's dual step along f^n and U^n,
and entry by entry: a single value of f^n moved must meet its own adjoint."""
import numpy as np
import pytest
import torch

import oracle
import paper_2408_02350_amd.bgk as bgk
from paper_2408_02350_amd.inputs import CavityConfig, make_cloud

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# FP64: the rounding of sums of ~1e6 terms, as the other dual-step checks.
# FP32 storage: f and the adjoint are rounded to 6e-8 at each of the step's
# stages, far below 1e-5 of the sum of absolute terms.
TOL = {"fp64": 1e-11, "fp32": 1e-5}


def t(a, dtype=torch.float64):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV, dtype)


@pytest.mark.parametrize("dim,n,nv,precision", [
    (2, 7, 2, "fp64"),     # 2 per lane, one lane in use
    (2, 8, 12, "fp64"),    # 3 per lane
    (2, 8, 14, "fp64"),    # 4 per lane, the last group of a line overlaps by 2
    (2, 7, 22, "fp64"),    # 3 per lane, overlaps by 2, a nearly empty tile
    (2, 6, 24, "fp64"),    # 3 per lane, full tiles
    (2, 6, 36, "fp32"),
    (3, 5, 6, "fp64"),     # 2 per lane
    (3, 5, 8, "fp64"),     # 4 per lane
    (3, 5, 10, "fp64"),    # 5 per lane
    (3, 5, 14, "fp64"),    # 7 per lane
    (3, 5, 18, "fp64"),    # 6 per lane
    (3, 4, 22, "fp64"),    # 6 per lane, overlaps by 2
    (3, 5, 10, "fp32"),
])
def test_adjoint_step_over_lane_widths(dim, n, nv, precision):
    cav = CavityConfig("sizes", dim, n, nv, 4.0, 2.2, 0.7, 0.2, 1, 0, wls_degree=1)
    c = oracle.config(cav)
    x, wid = make_cloud(dim, n, 2)
    ctx = bgk.bgk_init(bgk.config_from(cav, precision, flags=bgk.BGK_FLAG_ADJOINT),
                       t(wid, torch.int32))
    rng = np.random.default_rng(dim * 100 + nv)
    U = np.stack([0.2 * np.sin(np.pi * x[1]) * np.sin(np.pi * x[0])] +
                 [0.1 * np.cos(np.pi * x[a]) for a in range(1, dim)])
    f = oracle.maxwellian(c, 1.0 + 0.1 * x[0], U, 1.0 + 0.05 * x[dim - 1])
    f = f * rng.uniform(0.95, 1.05, f.shape)
    fd = torch.float64 if precision == "fp64" else torch.float32
    f = t(f, fd).double().cpu().numpy()
    lf = t(rng.normal(size=f.shape), fd).double().cpu().numpy()
    _, U, _ = oracle.moments(c, f)
    lU = rng.normal(size=U.shape)
    print(f"case {dim}D n={n} nv={nv} {precision}", flush=True)
    lam_f, lam_U = bgk.bgk_adjoint_step(ctx, t(f, fd), t(U), t(x), t(lf, fd), t(lU))[:2]
    bgk.bgk_check(ctx)
    lam_f, lam_U = lam_f.double().cpu().numpy(), lam_U.cpu().numpy()
    one = np.zeros_like(f)
    j = int(np.flatnonzero(wid == 0)[3])
    one[0, j].flat[-1] = f[0, j].flat[-1]  # the last velocity of the last line
    for name, kw, got in (("f", dict(f_dot=(df := f * rng.normal(size=f.shape))),
                           (lam_f * df).sum()),
                          ("one", dict(f_dot=one), (lam_f * one).sum()),
                          ("U", dict(U_dot=(dU := 0.1 * rng.normal(size=U.shape))),
                           (lam_U * dU).sum())):
        _, f1d, _, U1d = oracle.step_dual(c, wid, x, f, U, **kw)[:4]
        want = (lf * f1d).sum() + (lU * U1d).sum()
        scale = np.abs(lf * f1d).sum() + np.abs(lU * U1d).sum()
        print(f"  {name}: {got:.12e} against {want:.12e}, scale {scale:.3e}", flush=True)
        assert abs(got - want) <= TOL[precision] * scale, name
