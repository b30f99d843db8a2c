"""Which domains SAP solves on the chip: those that keep the lanes of their
workgroups busy, and not for fewer MR steps than pay for the exchange between
the workgroups of a large domain.  The others run as before that form was there,
bit for bit.  Near the line the on-chip form is compared with the oracle
(tolerances as for the other SAP kernels): idle lanes, odd extents, flat tiles."""

import numpy as np
import pytest

from oracle import sap
from paper_1104_0737_amd import inputs

pytestmark = pytest.mark.gpu
gu = pytest.importorskip("tests.gpu_util")
torch = gu.torch
B = gu.binding

PH_TWIST = ((np.cos(0.3), np.sin(0.3)), (1.0, 0.0), (np.cos(1.1), -np.sin(1.1)), (-1.0, 0.0))
SAP_TOL = {0: 1e-12, 1: 3e-5}


def _sap(lat, X, nmr, prec):
    ws = torch.empty(B.mbbs_sap_workspace_size(lat.h, X.shape[1], prec), dtype=torch.uint8, device="cuda")
    Y = torch.empty_like(X)
    B.mbbs_sap_apply(lat.h, X.shape[1], X, Y, 2, nmr, prec, ws)
    return gu.host(Y)


@pytest.mark.parametrize("dims,block,L,steps", [
    # steps: the fewest MR steps from which the chip serves (None: none)
    ((8, 8, 8, 8), (4, 4, 4, 4), 12, 1),            # one workgroup, every lane busy
    ((12, 12, 12, 12), (3, 3, 3, 3), 4, 2),         # one workgroup, 81 of 256
    ((16, 16, 16, 16), (8, 8, 8, 8), 12, 2),        # a group, every lane busy
    ((12, 12, 12, 12), (6, 6, 6, 6), 6, 3),         # a group, part of the lanes
    ((8, 8, 8, 8), (1, 1, 1, 1), 4, None),
    ((8, 8, 8, 8), (2, 2, 2, 2), 6, None),
    ((10, 10, 10, 10), (5, 5, 5, 5), 4, None),      # 125 of 512 lanes
    ((16, 16, 16, 4), (8, 8, 8, 1), 5, None)])
@pytest.mark.parametrize("prec", [0, 1])
def test_choice(dims, block, L, steps, prec):
    gu.flush(f"on-chip choice {dims} {block} L={L} prec={prec}")
    V, Vb = int(np.prod(dims)), int(np.prod(block))
    with gu.Lattice(dims, block, inputs.gauge_field(dims, 0.3, 700), 0.12) as lat:
        assert [B.mbbs_lattice_sap_on_chip(lat.h, L, prec, nmr) for nmr in (1, 2, 3, 4, 9)] == \
            [steps is not None and nmr >= steps for nmr in (1, 2, 3, 4, 9)]
        with pytest.raises(B.MbbsError) as e:
            B.mbbs_lattice_sap_on_chip(lat.h, L, prec, 0)
        assert e.value.code == B.EINVAL
        if steps != 1:
            X = gu.dev(inputs.gaussian_block(V, L, 701))
            nmr = 4 if steps is None else steps - 1
            Y = _sap(lat, X, nmr, prec)
            B.mbbs_lattice_tune(lat.h, B.TUNE_MR_FUSED, 1 if Vb * L <= 2048 else 0)
            assert _sap(lat, X, nmr, prec).tobytes() == Y.tobytes()


@pytest.mark.parametrize("dims,block,L", [
    ((6, 6, 6, 8), (3, 3, 3, 4), 5),          # 108 of 256 lanes
    ((12, 12, 12, 4), (6, 6, 6, 2), 3),       # flat tiles
    ((4, 8, 8, 6), (2, 4, 4, 3), 12)])        # 96 of 256 lanes
@pytest.mark.parametrize("prec", [0, 1])
def test_parity_near_the_line(dims, block, L, prec):
    gu.flush(f"on-chip parity {dims} {block} L={L} prec={prec}")
    V = int(np.prod(dims))
    U = inputs.gauge_field(dims, 0.3, 702)
    eta = inputs.gaussian_block(V, L, 703)
    with gu.Lattice(dims, block, U, 0.12, PH_TWIST) as lat:
        assert B.mbbs_lattice_sap_on_chip(lat.h, L, prec, 3)
        Y = _sap(lat, gu.dev(eta), 3, prec)
    ref = sap.sap(U, 0.12, PH_TWIST, sap.Domains(dims, block), eta, 2, 3).reshape(12 * V, L)
    assert np.all(gu.rel_col_err(Y, ref) <= SAP_TOL[prec])
    assert np.all(gu.max_elem_err(Y, ref) <= SAP_TOL[prec])
