"""The kernel that bench.py names in its roofline is the one that the library
launches (csrc/k_fused.hip: plan_fused, launch_fused)."""
import pytest

import bench


@pytest.mark.parametrize("nv,walks", [(8, False), (10, False), (12, False), (14, True), (16, False),
                                      (18, True), (20, True), (22, True), (24, True)])
def test_transport_kernel_of_3d_fp64_grids(nv, walks):
    assert bench.transport_kernel(3, nv, "fp64") == ("k_walk + k_collide" if walks else "k_fused")


@pytest.mark.parametrize("dim,nv,precision", [(2, 32, "fp64"), (2, 64, "fp64"), (3, 20, "fp32"),
                                              (3, 20, "bf16")])
def test_transport_kernel_of_the_others(dim, nv, precision):
    assert bench.transport_kernel(dim, nv, precision) == "k_fused"
