"""mbbs_cholqr waits for its verdict alone: the last product may still run when
the call returns, and what follows on its stream sees Q and gamma complete."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
gu = pytest.importorskip("tests.gpu_util")
torch = gu.torch
B = gu.binding


@pytest.mark.parametrize("passes", [1, 2])
@pytest.mark.parametrize("N,L", [(12, 1), (12 * 4096, 4), (12 * 65536, 16)])
def test_results_in_stream_order(N, L, passes):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(720 + L)
    P = torch.view_as_complex(torch.randn((N, L, 2), dtype=torch.float64, device="cuda", generator=gen))
    ws = torch.empty(B.mbbs_gram_workspace_size(N, L) + 5 * L * L * 16 + 256, dtype=torch.uint8, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        for _ in range(3):
            Q, gamma = torch.zeros_like(P), torch.zeros((L, L), dtype=torch.complex128, device="cuda")
            B.mbbs_cholqr(N, L, P, Q, gamma, passes, ws, stream=s)
            Qc, gc = Q.clone(), gamma.clone()          # on the same stream, at once
            Q.zero_()
            gamma.zero_()
        Qc, gc = gu.host(Qc), gu.host(gc)
    Ph = gu.host(P)
    # N (0, 1) columns: the Gram matrix's condition is at most (1 + sqrt(L / N))^2 /
    # (1 - sqrt(L / N))^2, below 4 here (L = 1: 1); sums of N products in FP64
    assert np.max(np.abs(Qc.conj().T @ Qc - np.eye(L))) <= 1e-13 * L
    assert np.max(np.abs(Qc @ gc - Ph)) <= 1e-13 * np.max(np.abs(Ph)) * L
    assert np.all(np.tril(gc, -1) == 0)
