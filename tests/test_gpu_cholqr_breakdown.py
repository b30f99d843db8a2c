"""A block that is not numerically of full rank leaves gamma, and the Q of the
failed pass, as they were: the launches behind the failed pivot have no effect."""

import pytest

pytestmark = pytest.mark.gpu
gu = pytest.importorskip("tests.gpu_util")
torch = gu.torch
B = gu.binding


@pytest.mark.parametrize("passes", [1, 2])
@pytest.mark.parametrize("N,L", [(12, 2), (12 * 4096, 4)])
def test_nothing_written_behind_a_failed_pivot(N, L, passes):
    P = torch.zeros((N, L), dtype=torch.complex128, device="cuda")
    P[:, 0] = 1.0                       # the other columns are exactly zero
    Q = torch.full_like(P, 7.0)
    gamma = torch.full((L, L), 5.0, dtype=torch.complex128, device="cuda")
    ws = torch.empty(B.mbbs_gram_workspace_size(N, L) + 5 * L * L * 16 + 256, dtype=torch.uint8, device="cuda")
    with pytest.raises(B.MbbsError) as e:
        B.mbbs_cholqr(N, L, P, Q, gamma, passes, ws)
    assert e.value.code == B.EBREAKDOWN
    assert torch.all(Q == 7.0) and torch.all(gamma == 5.0)
