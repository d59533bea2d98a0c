"""The statistic of few values in one launch and of more in three, on either side of the line between them (40960 values a
histogram); the per-sequence statistic at the edges of both forms: rows of whole 16-byte words of which the last may be partly valid,
one word a row, empty and full sequences, sequences of very different lengths, more histograms than the flat sweeps take, and NaN
or infinities in the padding (which must not be seen) or among the valid values (which must)."""
import numpy as np
import pytest
import torch

import paper_2604_10597_amd as corey
from gpu_util import to_dev
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


def _first_long(count, lens, shortest):
    """`count` sequences: the given lengths, then short ones."""
    return lens + tuple(shortest + b % 13 for b in range(count - len(lens)))


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16, wl.F32])
@pytest.mark.parametrize("D,L,lens", [(70, 2056, _first_long(64, (2051, 2056, 2049, 1003), 1)),      # 64 histograms: 16 workgroups each
                                      (1400, 2056, (2051, 0, 2056)),                                  # 341, and 512 for one
                                      (2100, 2056, (2045,)),
                                      (21, 2056, _first_long(65, (2056, 2051, 2048, 0), 40)),         # one more: the general kernels, vectors
                                      (24, 2051, (2051, 2050, 7))])                                   # and rows off the 16-byte words
def test_padded_rows_beyond_one_launch(D, L, lens, dtype):
    """More than 40960 values a sequence: workgroups of the flat sweeps that take several turns and end in a partial one, over rows
    whose number of words is no power of two and whose last word is partly valid; and what the flat sweeps do not take."""
    print(f"[case] padded rows D{D} L{L} {len(lens)} sequences {dtype}", flush=True)
    rng = np.random.default_rng(D + len(lens))
    x = np.full((len(lens), D, L), np.nan, dtype=np.float32)
    for b, n in enumerate(lens):
        x[b, :, :n] = rng.laplace(0, 1 + b % 3, (D, n))
    store, val = wl.store(x, dtype)
    for K in (64, 2731):
        _check(store, val, dtype, K, seqlens=np.array(lens, dtype=np.int32))


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("D,L,lens", [(9, 24, (21, 24)), (25, 2048, (2045, 2048))])
def test_constant_rows(D, L, lens, dtype):
    """A degenerate range: every valid value in bin 0, the words that end a row counted by their valid part only."""
    x = np.full((2, D, L), 1.5, dtype=np.float32)
    store, val = wl.store(x, dtype)
    _check(store, val, dtype, 32, seqlens=np.array(lens, dtype=np.int32))
    _check(store, val, dtype, 32)


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16, wl.F32])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_non_finite_value_in_the_sweeps(bad, dtype):
    """More than 40960 values a histogram: the first sequence's last valid value spoils its statistic, and the whole tensor's."""
    x = np.random.default_rng(3).standard_normal((2, 25, 2048)).astype(np.float32)
    x[0, -1, 2044] = bad
    store, val = wl.store(x, dtype)
    out, _ = _check(store, val, dtype, 64)
    assert int(out["counts"].sum()) == 0
    out, _ = _check(store, val, dtype, 64, seqlens=np.array([2045, 2048], dtype=np.int32))
    assert int(out["counts"][0].sum()) == 0 and int(out["counts"][1].sum()) == 25 * 2048


@pytest.mark.parametrize("dtype,V", [(wl.BF16, 8), (wl.F16, 8), (wl.F32, 4)])
@pytest.mark.parametrize("values", [8, 8184, 8192, 8200, 40952, 40960, 40968])
@pytest.mark.parametrize("K", [2, 300, 4096])
def test_few_values(values, K, dtype, V):
    """One launch up to 40960 values: a lane's last word there or not, bins beyond the reducing lanes."""
    print(f"[case] few values {values} K{K} {dtype}", flush=True)
    rng = np.random.default_rng(values + K)
    store, val = wl.store(rng.standard_normal((1, values // V, V)).astype(np.float32), dtype)
    out, _ = _check(store, val, dtype, K)
    pol = corey.policy_default()
    xd = to_dev(store, dtype)
    routed = corey.corey_route_device(xd, K, pol)
    assert torch.equal(routed["counts"], out["counts"]) and routed["r"].item() == out["r"].item()
    assert routed["chunks"].item() == corey.corey_select_chunk(out["r"].item(), V, pol)
    route = corey.corey_route_device_deferred(xd, K, pol)          # the reduction of partial histograms adds the same numbers in the same order
    N = 4
    z = torch.zeros_like(xd)
    B, C = torch.zeros((1, N, V), dtype=xd.dtype, device="cuda"), torch.zeros((1, N, V), dtype=xd.dtype, device="cuda")
    A = -torch.ones((values // V, N), device="cuda")
    corey.selective_scan_fwd(xd, z, A, B, C, chunk=16, route=route["route"])
    assert route["r"].item() == out["r"].item() and route["H"].item() == out["H"].item()
    store, val = wl.store(np.full((1, values // V, V), -2.0, dtype=np.float32), dtype)
    _check(store, val, dtype, K)


@pytest.mark.parametrize("L,stride", [(L, s) for L in (8, 8184, 8192, 8200, 8192 * 3 + 16) for s in (1, 4)] + [(838880, 1), (3355536, 4)])
def test_producers_range(L, stride):
    """The count sweep on the producer's range.  A workgroup's turn is 1024 words and there are up to 512 workgroups: five words,
    a turn each but for a partial last one, whole turns, and (the two long rows) a second turn of which there are 12 words, or 15."""
    print(f"[case] producer's range L{L} stride {stride}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(L)
    x = torch.randn((1, 5, L), generator=g, device="cuda").to(torch.bfloat16)
    u, _, parts = corey.causal_conv1d_silu_fwd(x, torch.randn((5, 4), generator=g, device="cuda"), torch.zeros(5, device="cuda"))
    block = 8 if stride > 1 else 1
    out = corey.corey_entropy_hist(u, 64, stride=stride, block=block, range_parts=parts)
    lo, hi = (float(v) for v in out["range"].flatten().tolist())
    v = u.float().flatten().cpu().numpy()
    if stride > 1:
        v = v.reshape(-1, block)[::stride].ravel()
    scale = np.float32(64 / (hi - lo))
    k = np.clip((v - np.float32(lo)) * scale, 0.0, 63.0).astype(np.int64)      # of all values, sampled or not
    assert np.array_equal(out["counts"].cpu().numpy().ravel(), np.bincount(k, minlength=64))
