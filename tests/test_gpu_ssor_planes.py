"""SSOR sweeps through LDS (the wavefront kernel of lattices with few domains)
against the kernel that keeps the fields in global memory.

A batch of enough systems takes the latter, a single system the former; with
real boundary phases and no clover term both round alike, so a system of the
batch must equal the same system alone, bit for bit.  Shapes: hyperplanes of one
pass and of several, idle lanes, one and several columns per workgroup, odd
extents.
"""

import numpy as np
import pytest

from paper_1104_0737_amd import inputs

pytestmark = pytest.mark.gpu
gu = pytest.importorskip("tests.gpu_util")
torch = gu.torch
B = gu.binding


def _run(h, X, prec, ncy, nssor, omega):
    L = X.shape[1]
    ws = torch.empty(B.mbbs_ssor_workspace_size(h, L, prec), dtype=torch.uint8, device="cuda")
    Y, Z = torch.empty_like(X), torch.empty_like(X)
    B.mbbs_sap_apply_ssor(h, L, X, Y, ncy, nssor, omega, prec, ws)
    B.mbbs_apply_ssor_blocked(h, L, X, Z, nssor, omega, prec, ws)
    return gu.host(Y), gu.host(Z)


@pytest.mark.parametrize("dims,block,L,nsys,nssor", [
    ((4, 6, 4, 8), (2, 3, 2, 4), 5, 17, 1),
    ((8, 8, 4, 8), (4, 4, 2, 4), 12, 17, 0),
    ((16, 16, 16, 16), (4, 4, 4, 4), 12, 2, 1),      # columns up to the thread limit (FP32)
    ((16, 16, 16, 16), (8, 8, 8, 8), 1, 17, 1)])     # 344 sites in a hyperplane: two passes in FP64
@pytest.mark.parametrize("prec", [0, 1])
def test_system_of_a_large_batch_runs_as_alone(dims, block, L, nsys, nssor, prec):
    gu.flush(f"ssor through LDS {dims} L={L} prec={prec}")
    V = int(np.prod(dims))
    U = inputs.gauge_field(dims, 0.3, 660)
    ks = [0.112 + 0.0005 * k for k in range(nsys)]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(661)
    X = torch.view_as_complex(torch.randn((12 * V * nsys, L, 2), dtype=torch.float64, device="cuda", generator=gen))
    Ud = gu.dev(U)
    h = B.mbbs_lattice_create_batch(dims, block, [Ud] * nsys, ks, gu.PH_AP)
    try:
        Yb, Zb = _run(h, X, prec, 2, nssor, 1.26 if nssor else 1.0)
    finally:
        B.mbbs_lattice_destroy(h)
    for k in (0, nsys - 1):
        N = 12 * V
        with gu.Lattice(dims, block, U, ks[k]) as lat:
            Y, Z = _run(lat.h, X[k * N:(k + 1) * N].contiguous(), prec, 2, nssor, 1.26 if nssor else 1.0)
        assert Yb[k * N:(k + 1) * N].tobytes() == Y.tobytes(), k
        assert Zb[k * N:(k + 1) * N].tobytes() == Z.tobytes(), k
