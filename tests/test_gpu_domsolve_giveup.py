"""A wait between workgroups that gives up (here at once: its bound is set to no
polls) ends the call normally and shows everywhere: all of the result is NaN,
a solve reports a breakdown, and with the bound restored the same workspace
serves again."""

import numpy as np
import pytest

from paper_1104_0737_amd import inputs

pytestmark = pytest.mark.gpu
gu = pytest.importorskip("tests.gpu_util")
torch = gu.torch
B = gu.binding

DIMS, BLOCK, L = (16, 16, 8, 8), (8, 8, 4, 4), 4      # 1024 sites a domain: several workgroups each
V = int(np.prod(DIMS))


@pytest.mark.parametrize("prec", [0, 1])
def test_sap(prec):
    gu.flush(f"sap with waits that give up prec={prec}")
    X = gu.dev(inputs.gaussian_block(V, L, 690))
    with gu.Lattice(DIMS, BLOCK, inputs.gauge_field(DIMS, 0.3, 691), 0.12) as lat:
        ws = torch.zeros(B.mbbs_sap_workspace_size(lat.h, L, prec), dtype=torch.uint8, device="cuda")
        Y = torch.zeros_like(X)
        for ncy, nmr in ((1, 2), (2, 3)):
            assert B.mbbs_lattice_sap_on_chip(lat.h, L, prec, nmr)
            B.mbbs_lattice_sap_polls(lat.h, 1 << 24)
            B.mbbs_sap_apply(lat.h, L, X, Y, ncy, nmr, prec, ws)
            ref = gu.host(Y)
            assert np.all(np.isfinite(ref))
            B.mbbs_lattice_sap_polls(lat.h, 0)
            Y.zero_()
            B.mbbs_sap_apply(lat.h, L, X, Y, ncy, nmr, prec, ws)
            bad = gu.host(Y)
            assert np.all(np.isnan(bad.real)) and np.all(np.isnan(bad.imag))
            B.mbbs_lattice_sap_polls(lat.h, 1 << 24)
            B.mbbs_sap_apply(lat.h, L, X, Y, ncy, nmr, prec, ws)
            assert gu.host(Y).tobytes() == ref.tobytes()
        for polls in (-1, (1 << 30) + 1):
            with pytest.raises(B.MbbsError) as e:
                B.mbbs_lattice_sap_polls(lat.h, polls)
            assert e.value.code == B.EINVAL


@pytest.mark.parametrize("graph_iters", [1, 2])
def test_solve_reports_a_breakdown(graph_iters):
    X = gu.dev(inputs.gaussian_block(V, L, 692))
    with gu.Lattice(DIMS, BLOCK, inputs.gauge_field(DIMS, 0.3, 693), 0.12) as lat:
        p = B.mbbs_solve_params_default(tol=1e-8, sap_prec=B.FP32, graph_iters=graph_iters)
        ws = torch.empty(B.mbbs_solve_workspace_size(lat.h, L, p), dtype=torch.uint8, device="cuda")
        B.mbbs_lattice_sap_polls(lat.h, 0)
        with pytest.raises(B.MbbsError) as e:
            B.mbbs_solve(lat.h, L, X, torch.empty_like(X), p, ws)
        assert e.value.code == B.EBREAKDOWN
        B.mbbs_lattice_sap_polls(lat.h, 1 << 24)
        info = B.mbbs_solve(lat.h, L, X, torch.empty_like(X), p, ws)
        assert info["status"] == B.OK
