"""FP32 and BF16 storage: a wider lane changes no bit.  A cloud with patches to
spare, which takes the widest lanes, against the part of it that its first
particles form, too small for them: where a particle's whole support is in the
part, its neighbours, operators and f rows are the same, and so is f-tilde.  (2D BF16
takes no wider lanes; its products pair the rows of a patch's union, so a
particle's sum there depends on its patch.)"""
import pytest
import torch

import paper_2408_02350_amd.bgk as bgk
from paper_2408_02350_amd.inputs import CavityConfig, make_cloud

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


CASES = [
    (3, 15, 8), (3, 15, 10), (3, 15, 12), (3, 15, 14), (3, 15, 16), (3, 15, 18),  # 549 patches
    (3, 19, 8), (3, 19, 10),                                                      # 1228
    (2, 93, 10), (2, 93, 12), (2, 93, 14), (2, 93, 16), (2, 93, 20), (2, 93, 24)]  # 2070


@pytest.mark.parametrize("dim,n,nv,precision",
                         [(*c, p) for p in ("fp32", "bf16") for c in CASES
                          if p == "fp32" or c[0] == 3])
def test_transport_of_a_part_of_the_cloud(dim, n, nv, precision):
    cav = CavityConfig("bits", dim, n, nv, 4.0, 2.5 if dim == 2 else 2.2, 1.0, 0.1, 1, 0)
    x, wid = make_cloud(dim, n, 2)
    x, wid = torch.from_numpy(x).to(DEV), torch.from_numpy(wid).to(DEV)
    U = torch.stack([0.2 * torch.sin(3.0 * x[1])] + [0.1 * torch.cos(3.0 * x[a])
                                                     for a in range(1, dim)])
    layer = n ** (dim - 1)  # the slowest axis is the last: layers of the lattice
    layers, deep = (5, 2) if dim == 3 else (12, 8)

    def transport(N):
        ctx = bgk.bgk_init(bgk.config_from(cav, precision, n_particles=N), wid[:N].contiguous())
        xs, Us = x[:, :N].contiguous(), U[:, :N].contiguous()
        f = bgk.bgk_maxwellian(ctx, 1.0 + 0.1 * xs[0], Us, 1.0 + 0.1 * xs[dim - 1])
        f = f * (1.0 + 0.05 * torch.sin(40.0 * xs[0])).to(f)[None, :, None]
        out = torch.zeros_like(f)
        bgk.bgk_geometry(ctx, xs)
        bgk.bgk_transport(ctx, f.contiguous(), out, Us)
        return out

    print(f"case {dim}D n={n} nv={nv} {precision}", flush=True)
    inner = torch.nonzero(wid[:deep * layer] == 0)[:, 0]
    whole, part = transport(x.shape[1]), transport(layers * layer)
    assert torch.equal(whole[:, inner], part[:, inner])
