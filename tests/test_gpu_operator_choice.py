"""The operator's choice of launch by lattice size against the plain launch
(no tiles, two columns per thread outside FP64, 256 threads), which a handle runs
once a knob is set.

FP64 and FP32 give the same bits.  FP16S may contract products differently with
another number of columns per thread: one unit of the last place of the stored
halves (2^-10 of the site's scale, which is at most the largest component).
"""

import numpy as np
import pytest

from paper_1104_0737_amd import inputs

pytestmark = pytest.mark.gpu
gu = pytest.importorskip("tests.gpu_util")
torch = gu.torch
B = gu.binding


def _field(V, L, prec, offset=0):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(670 + L)
    n = 12 * V * L * 2
    x = torch.randn(n + 2 * offset, dtype=torch.float64, device="cuda", generator=gen)
    if prec == 0:
        return torch.view_as_complex(x[2 * offset:].view(12 * V, L, 2)), None
    x = x.to(torch.float32 if prec == 1 else torch.float16)[2 * offset:].view(12 * V, L, 2)
    s = torch.rand((V, L), device="cuda", generator=gen) + 0.5 if prec == 2 else None
    return x, s


def _apply(lat, V, L, prec, X, Xs, offset=0):
    Y, Ys = _field(V, L, prec, offset)
    Y.zero_()
    B.mbbs_apply_dirac_raw(lat.h, L, prec, X, Xs, Y, Ys)
    return gu.host(Y), None if Ys is None else gu.host(Ys)


@pytest.mark.parametrize("dims,block,L", [
    ((4, 4, 4, 4), (2, 2, 2, 2), 1), ((8, 8, 8, 8), (4, 4, 4, 4), 4), ((8, 8, 8, 8), (4, 4, 4, 4), 6),
    ((12, 12, 12, 12), (6, 6, 6, 6), 5), ((12, 12, 12, 12), (6, 6, 6, 6), 8), ((12, 12, 12, 12), (6, 6, 6, 6), 12),
    ((16, 16, 16, 16), (8, 8, 8, 8), 1), ((16, 16, 16, 16), (8, 8, 8, 8), 7), ((4, 4, 4, 4), (2, 2, 2, 2), 64)])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_choice_matches_plain(dims, block, L, prec):
    gu.flush(f"operator choice {dims} L={L} prec={prec}")
    V = int(np.prod(dims))
    with gu.Lattice(dims, block, inputs.gauge_field(dims, 0.3, 671), 0.12) as lat:
        X, Xs = _field(V, L, prec)
        Y, Ys = _apply(lat, V, L, prec, X, Xs)
        B.mbbs_lattice_tune(lat.h, B.TUNE_TILE[prec], 0)
        P, Ps = _apply(lat, V, L, prec, X, Xs)
    if prec < 2:
        assert Y.tobytes() == P.tobytes()
    else:
        y = Y.astype(np.float32).reshape(V, 12, L, 2) * Ys.reshape(V, 1, L, 1)
        p = P.astype(np.float32).reshape(V, 12, L, 2) * Ps.reshape(V, 1, L, 1)
        assert np.all(np.abs(y - p) <= 2.0 ** -10 * Ps.reshape(V, 1, L, 1) * 1.001)


def test_fields_off_the_16_byte_grid():
    dims, block, L = (12, 12, 12, 12), (6, 6, 6, 6), 12
    V = int(np.prod(dims))
    with gu.Lattice(dims, block, inputs.gauge_field(dims, 0.3, 672), 0.12) as lat:
        X, _ = _field(V, L, 1, 1)
        Y, _ = _apply(lat, V, L, 1, X, None, 1)
        P, _ = _apply(lat, V, L, 1, X.clone(), None)
    assert Y.tobytes() == P.tobytes()
