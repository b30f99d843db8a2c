"""Device memory of a handle: the plane-wise copies of the links are held only
where a kernel can read them."""

import pytest

pytestmark = pytest.mark.gpu
gu = pytest.importorskip("tests.gpu_util")
torch = gu.torch
B = gu.binding


def test_no_copies_for_domains_too_large_for_the_chip():
    """16^4 domains: neither a group of workgroups nor a hyperplane in LDS holds
    one.  A handle holds its links in three precisions and two orders (2016
    bytes a site), its tables and the allocator's rounding; the two plane-wise
    copies would be 896 bytes a site more."""
    dims, block = (32, 32, 32, 32), (16, 16, 16, 16)
    V = 32 ** 4
    U = torch.zeros((V, 4, 3, 3), dtype=torch.complex128, device="cuda")
    U[..., range(3), range(3)] = 1
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    h = B.mbbs_lattice_create(dims, block, U, 0.12, gu.PH_AP)
    try:
        torch.cuda.synchronize()
        held = free - torch.cuda.mem_get_info()[0]
        assert held <= 2016 * V + (64 << 20), held / V
    finally:
        B.mbbs_lattice_destroy(h)
