"""Particle management where its scans take several blocks (more than 8192
particles or lattice nodes) and where a new particle's row is shorter or
longer than its block, against the oracle."""
import pytest

from test_gpu_particles import cavity, compare
from paper_2408_02350_amd.inputs import disturbed_cloud

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n,nv", [(2, 90, 4), (2, 91, 4), (2, 129, 2), (3, 27, 4), (2, 30, 24)])
def test_management_over_scan_blocks(dim, n, nv):
    cav = cavity(dim, n, nv)
    x, wid = disturbed_cloud(dim, n, 4)
    compare(cav, x, wid, 0.25 * cav.dx, 0.45 * cav.h)
