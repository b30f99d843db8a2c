"""SAP with the domain solves kept on the chip (one launch per colour and
cycle), the default for FP64 and FP32 storage, against the oracle and against
the launches it stands for (one per part of an MR step).

Shapes: a domain in one workgroup, a domain cut into tiles that exchange their
faces, odd extents and odd L (one column per thread), several column chunks
and column groups, a clover term, twisted phases, several systems.  Tolerances:
the oracle's as for the other SAP kernels; between the two GPU forms only the
order of the domain sums and the contraction of products differ, so 64 units of
the last place for the at most 9 MR steps of these cases, whose errors the
contracting steps do not amplify.
"""

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
PAIR_TOL = {0: 64 * 2.0 ** -52, 1: 64 * 2.0 ** -23}


def _apply(h, X, ncy, nmr, prec, ws=None):
    if ws is None:
        ws = torch.empty(B.mbbs_sap_workspace_size(h, X.shape[1], prec), dtype=torch.uint8, device="cuda")
    Y = torch.empty_like(X)
    B.mbbs_sap_apply(h, X.shape[1], X, Y, ncy, nmr, prec, ws)
    return Y


@pytest.mark.parametrize("dims,block,L,ncy,nmr,csw", [
    ((8, 8, 8, 8), (4, 4, 4, 4), 4, 2, 4, 0.0),        # one workgroup, 256 sites
    ((4, 6, 4, 8), (2, 3, 2, 4), 5, 3, 3, 0.0),        # odd extent, odd L, part of a wave idle
    ((4, 4, 4, 8), (2, 2, 2, 4), 16, 2, 1, 0.0),       # several columns per site
    ((8, 8, 8, 8), (4, 4, 4, 4), 6, 2, 2, 1.0),        # clover term
    ((16, 8, 8, 8), (8, 4, 4, 4), 12, 2, 4, 0.0),      # tiles
    ((12, 12, 12, 12), (6, 6, 6, 6), 3, 1, 3, 0.0),    # tiles, odd extents
    ((16, 16, 8, 8), (8, 8, 4, 4), 2, 2, 2, 1.0)])     # tiles cut in two directions, clover term
@pytest.mark.parametrize("prec", [0, 1])
def test_parity(dims, block, L, ncy, nmr, csw, prec):
    gu.flush(f"sap on chip {dims} L={L} prec={prec}")
    V = int(np.prod(dims))
    U = inputs.gauge_field(dims, 0.3, 610)
    eta = inputs.gaussian_block(V, L, 611)
    with gu.Lattice(dims, block, U, 0.12, PH_TWIST) as lat:
        if csw:
            B.mbbs_lattice_set_clover(lat.h, csw)
        X = gu.dev(eta)
        Y = _apply(lat.h, X, ncy, nmr, prec)
        Y2 = _apply(lat.h, X, ncy, nmr, prec)
        B.mbbs_lattice_tune(lat.h, B.TUNE_MR_FUSED, 0)
        S = gu.host(_apply(lat.h, X, ncy, nmr, prec))
        Y, Y2 = gu.host(Y), gu.host(Y2)
    assert Y.tobytes() == Y2.tobytes()
    assert np.all(gu.rel_col_err(Y, S) <= PAIR_TOL[prec]), gu.rel_col_err(Y, S)
    if not csw and V <= 8192:   # (the larger shapes against the other form only)
        ref = sap.sap(U, 0.12, PH_TWIST, sap.Domains(dims, block), eta, ncy, nmr).reshape(12 * V, L)
        assert np.all(gu.rel_col_err(Y, ref) <= SAP_TOL[prec])
        assert np.all(gu.max_elem_err(Y, ref) <= SAP_TOL[prec])


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dims,block,L", [((8, 8, 4, 8), (4, 4, 2, 4), 4), ((16, 8, 8, 8), (8, 4, 4, 4), 6)])
def test_systems_of_a_batch_run_as_alone(dims, block, L, prec):
    V = int(np.prod(dims))
    Us = [inputs.gauge_field(dims, 0.3, 620 + k) for k in range(3)]
    ks = [0.112 + 0.004 * k for k in range(3)]
    etas = [inputs.gaussian_block(V, L, 630 + k) for k in range(3)]
    U_dev = [gu.dev(U) for U in Us]
    h = B.mbbs_lattice_create_batch(dims, block, U_dev, ks, gu.PH_AP)
    try:
        Y = gu.host(_apply(h, gu.dev(np.concatenate(etas)), 2, 3, prec))
    finally:
        B.mbbs_lattice_destroy(h)
    for k in range(3):
        with gu.Lattice(dims, block, Us[k], ks[k]) as lat:
            R = gu.host(_apply(lat.h, gu.dev(etas[k]), 2, 3, prec))
        assert Y[k * 12 * V:(k + 1) * 12 * V].tobytes() == R.tobytes(), k


def test_zero_and_nan_columns():
    """A zero column gives exactly zero (omega 0 / 0 is 0); a NaN stays in its column."""
    dims, block, L = (16, 8, 8, 8), (8, 4, 4, 4), 4
    V = int(np.prod(dims))
    eta = inputs.gaussian_block(V, L, 640)
    eta[..., 1] = 0
    eta.reshape(12 * V, L)[5, 3] = np.nan
    with gu.Lattice(dims, block, inputs.gauge_field(dims, 0.3, 641), 0.12) as lat:
        for prec in (0, 1):
            Y = gu.host(_apply(lat.h, gu.dev(eta), 2, 3, prec)).reshape(12 * V, L)
            assert not np.any(Y[:, 1])
            assert np.all(np.isfinite(Y[:, [0, 2]]))
            assert np.any(np.isnan(Y[:, 3]))


def test_two_streams_and_graph_replays():
    """Two streams with a workspace each, and replays of a captured graph with
    eager calls between them, give the eager bits."""
    dims, block, L = (16, 8, 8, 8), (8, 4, 4, 4), 12
    V = int(np.prod(dims))
    with gu.Lattice(dims, block, inputs.gauge_field(dims, 0.3, 650), 0.12) as lat:
        X = [gu.dev(inputs.gaussian_block(V, L, 651 + k)) for k in range(2)]
        ws = [torch.empty(B.mbbs_sap_workspace_size(lat.h, L, 1), dtype=torch.uint8, device="cuda") for _ in range(2)]
        ref = [gu.host(_apply(lat.h, x, 2, 3, 1)) for x in X]
        Y = [torch.zeros_like(x) for x in X]
        streams = [torch.cuda.Stream() for _ in range(2)]
        torch.cuda.synchronize()
        for _ in range(3):
            for k in range(2):
                B.mbbs_sap_apply(lat.h, L, X[k], Y[k], 2, 3, 1, ws[k], stream=streams[k])
        for k in range(2):
            assert gu.host(Y[k]).tobytes() == ref[k].tobytes(), k
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            B.mbbs_sap_apply(lat.h, L, X[0], Y[0], 2, 3, 1, ws[0])
        for _ in range(3):
            Y[0].fill_(0)
            g.replay()
            assert gu.host(Y[0]).tobytes() == ref[0].tobytes()
            assert gu.host(_apply(lat.h, X[1], 2, 3, 1, ws[0])).tobytes() == ref[1].tobytes()


@pytest.mark.parametrize("prec,L", [(0, 12), (1, 15)])
def test_omega_summed_in_the_update(prec, L):
    """The launches per MR step: few block partials of a domain are summed by the
    update, many (small blocks) by a launch of their own."""
    dims, block = (8, 8, 8, 8), (4, 4, 4, 4)
    with gu.Lattice(dims, block, inputs.gauge_field(dims, 0.3, 660), 0.12) as lat:
        X = gu.dev(inputs.gaussian_block(4096, L, 661))
        B.mbbs_lattice_tune(lat.h, B.TUNE_MR_FUSED, 0)
        Y = gu.host(_apply(lat.h, X, 2, 4, prec))
        B.mbbs_lattice_tune(lat.h, B.TUNE_BLOCK_THREADS, 32)
        S = gu.host(_apply(lat.h, X, 2, 4, prec))
    assert np.all(gu.rel_col_err(Y, S) <= PAIR_TOL[prec]), gu.rel_col_err(Y, S)
