"""Sums of a row against 80-bit sums, and what a non-finite value makes of them:
an infinite density stays infinite."""
import numpy as np
import pytest
import torch

import paper_2408_02350_amd.bgk as B
from paper_2408_02350_amd.inputs import CavityConfig, cloud_for

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def cavity(dim, n, nv, precision):
    cav = CavityConfig("sums", dim, n, nv, 4.0, 2.4, 0.8, 0.1, 1, 0, precision=precision)
    x, wid = cloud_for(cav, 1)
    c = B.bgk_init(B.config_from(cav, precision, move=0), torch.from_numpy(wid).to(DEV))
    rng = np.random.default_rng(5)
    rho = torch.from_numpy(1.0 + 0.1 * rng.uniform(-1, 1, c.N)).to(DEV)
    U = torch.from_numpy(0.2 * rng.uniform(-1, 1, (c.d, c.N))).to(DEV)
    T = torch.from_numpy(1.0 + 0.1 * rng.uniform(-1, 1, c.N)).to(DEV)
    return c, B.bgk_maxwellian(c, rho, U, T)


# the smallest row, ragged groups, a row of several groups per thread, and one
# that no thread keeps whole
@pytest.mark.parametrize("dim,n,nv", [(2, 6, 2), (2, 9, 18), (3, 5, 8), (3, 5, 14), (3, 5, 28)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_moments_of_rows(dim, n, nv, precision):
    c, f = cavity(dim, n, nv, precision)
    rho, U, _ = (t.cpu().numpy() for t in B.bgk_moments(c, f))
    F = f[0].cpu().numpy().astype(np.longdouble)
    v1 = np.longdouble(4.0) * (2 * np.arange(nv) - (nv - 1)) / np.longdouble(nv - 1)
    q = np.arange(nv ** dim)
    s0 = F.sum(axis=1)
    # each term rounds twice (node, product), and one partial sum per thread,
    # then per pair and quad, rounds as it grows: no more than this many times
    steps = 2 + -(-nv ** dim // 256) + 4
    for a in range(dim):
        v = v1[(q // nv ** a) % nv]
        bound = steps * 2.0 ** -53 * (F * abs(v)).sum(axis=1) / s0
        assert (abs(U[a] - (F * v).sum(axis=1) / s0) <= bound + 2.0 ** -52 * abs(U[a])).all()
    omega = (np.longdouble(8.0) / (nv - 1)) ** dim
    assert (abs(rho - omega * s0) <= (steps + 4) * 2.0 ** -53 * rho).all()


@pytest.mark.parametrize("dim,nv", [(2, 8), (3, 8)])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("at", [0, 37, -1])
def test_a_value_that_is_not_finite(dim, nv, value, at):
    c, f = cavity(dim, 6, nv, "fp64")
    f[0, 3, at] = value
    rho, U, T = B.bgk_moments(c, f)
    bad = torch.zeros(c.N, dtype=torch.bool, device=DEV)
    bad[3] = True
    assert torch.equal(~torch.isfinite(rho), bad)
    assert torch.equal(rho[3:4].cpu(), torch.tensor([value], dtype=torch.float64)) or value != value
    assert torch.isfinite(U[:, ~bad]).all() and not torch.isfinite(U[:, 3]).any()
