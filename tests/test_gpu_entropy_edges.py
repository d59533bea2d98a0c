"""The per-sequence statistic at the edges of its flat sweeps: rows of whole 16-byte words of which the last may be partly valid,
one word a row, empty and full sequences, sequences of very different lengths, more histograms than the flat sweeps take, and NaN
or infinities in the padding (which must not be seen) or among the valid values (which must)."""
import numpy as np
import pytest

from paper_2604_10597_amd import workloads as wl
from test_gpu_entropy import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16, wl.F32])
@pytest.mark.parametrize("D,L,lens", [(3, 8, (8, 1, 0, 7)), (5, 16, (9, 16)), (130, 72, (72, 5, 64)), (700, 200, (200, 199, 8, 0, 33)),
                                      (1, 4096, (4096, 1)), (2500, 512, (512, 40)), (3, 24, tuple(range(24)) * 3)])
def test_padded_rows(D, L, lens, dtype):
    print(f"[case] padded rows D{D} L{L} {len(lens)} sequences {dtype}", flush=True)
    rng = np.random.default_rng(D + L)
    x = rng.standard_normal((len(lens), D, L)).astype(np.float32)
    for b, n in enumerate(lens):
        x[b, :, n:] = [np.nan, np.inf, -6e4][b % 3]
    store, val = wl.store(x, dtype)
    _check(store, val, dtype, 64, seqlens=np.array(lens, dtype=np.int32))
    for bad in (np.nan, -np.inf):                       # the last valid value of the first sequence
        x[0, -1, lens[0] - 1] = bad
        store, val = wl.store(x, dtype)
        _check(store, val, dtype, 64, seqlens=np.array(lens, dtype=np.int32))


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
def test_constant_rows(dtype):
    """A degenerate range: every valid value in bin 0, the words that end a row counted by their valid part only."""
    x = np.full((2, 9, 24), 1.5, dtype=np.float32)
    store, val = wl.store(x, dtype)
    _check(store, val, dtype, 32, seqlens=np.array([21, 24], dtype=np.int32))
