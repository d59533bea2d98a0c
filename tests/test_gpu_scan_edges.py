"""The scan at the edges of its dispatch: rows of any length (vectors that straddle a row's end, rows shorter than a lane's
run), launches on either side of the row counts where B and C are read directly and where long chunks are walked in parts of
512, padding that holds NaN."""
import numpy as np
import pytest
import torch

import paper_2604_10597_amd as corey
from gpu_util import assert_close, check_y, fp32_rtol, oracle_scan, upload, y_to_f64
from paper_2604_10597_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _scan(d, chunk, **kw):
    return corey.selective_scan_fwd(d["u"], d["delta"], d["A"], d["B"], d["C"], Dv=d["D"], z=d["z"], delta_bias=d["delta_bias"],
                                    h0=d.get("h0"), seqlens=d["seqlens"], chunk=chunk, **kw)


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16, wl.F32])
@pytest.mark.parametrize("B,D,N,L", [(1, 5, 16, 1), (2, 3, 16, 15), (2, 3, 16, 16), (1, 7, 16, 17), (2, 5, 8, 1031), (1, 3, 4, 1023),
                                     (2, 2, 16, 2049), (1, 6, 20, 527), (2, 3, 6, 77), (1, 4, 1, 1025)])
def test_rows_of_any_length(B, D, N, L, dtype):
    cfg = wl.Config("edges", B, D, N, L, dtype, 16, (), seed=4000 + L + N)
    w = wl.make(cfg, a_kind="random", with_h0=True)
    d = upload(w)
    y_ref, s_ref = oracle_scan(w)
    for chunk in (16, 64, 256, 512, 1024, 2048):
        for whole in (False, True):
            y, s = _scan(d, chunk, whole_rows=whole)
            check_y(y_to_f64(y), y_ref, cfg, f"y chunk {chunk}")
            assert_close(s.cpu().numpy(), s_ref, fp32_rtol(L), f"state chunk {chunk}")


@pytest.mark.parametrize("dtype,D", [(wl.BF16, 3), (wl.F32, 3), (wl.BF16, 1100)])
def test_padding_is_never_read_into_a_result(dtype, D):
    """Sequences shorter than L whose padded positions hold NaN in every input."""
    lens = (1, 29, 543, 1030)
    cfg = wl.Config("edges_nan", 4, D, 16, 1031, dtype, 16, (), seqlens=lens, seed=4100)
    w = wl.make(cfg, a_kind="random")
    d = upload(w)
    for b, n in enumerate(lens):
        for name in ("u", "delta", "z", "B", "C"):
            d[name][b, :, n:] = float("nan")
    rows = np.arange(3) if D > 3 else None
    y_ref, s_ref = oracle_scan(w, rows=rows)
    for chunk in (64, 512, 1024):
        y, s = _scan(d, chunk)
        assert torch.isfinite(y.float()).all() and torch.isfinite(s).all()
        check_y(y_to_f64(y)[:, :3], y_ref, cfg, f"y chunk {chunk}")
        assert_close(s.cpu().numpy()[:, :3], s_ref, fp32_rtol(cfg.L), f"state chunk {chunk}")


@pytest.mark.parametrize("B,D", [(1, 3072), (1, 3073), (1, 4096), (1, 4097), (3, 1366)])
def test_either_side_of_the_row_counts_the_launch_changes_at(B, D):
    """3072 rows read B and C directly, more are staged; beyond 4096 rows tiles are at most 512 steps, of two kinds of rows."""
    cfg = wl.Config("edges_rows", B, D, 16, 1100, wl.BF16, 16, (), seed=4200)
    w = wl.make(cfg, a_kind="random")
    d = upload(w)
    rows = np.unique(np.concatenate([[0, 1, D - 2, D - 1], np.random.default_rng(3).integers(0, D, 6)]))
    y_ref, s_ref = oracle_scan(w, rows=rows)
    routed = torch.full((B,), 1024, dtype=torch.int32, device="cuda")
    for chunk, dev in ((512, None), (1024, None), (2048, None), (512, routed)):
        y, s = _scan(d, chunk, chunks_dev=dev)
        check_y(y_to_f64(y)[:, rows], y_ref, cfg, f"y chunk {chunk}")
        assert_close(s.cpu().numpy()[:, rows], s_ref, fp32_rtol(cfg.L), f"state chunk {chunk}")


@pytest.mark.parametrize("a_kind", ["mamba", "random"])
@pytest.mark.parametrize("dtype,B,D", [(wl.F32, 1, 1024), (wl.F32, 1, 1025), (wl.F32, 2, 1024), (wl.F32, 1, 2049), (wl.F32, 1, 3072),
                                       (wl.F32, 1, 3073), (wl.F32, 1, 4096), (wl.F32, 3, 1400), (wl.F16, 1, 3072), (wl.F16, 1, 3073),
                                       (wl.F16, 1, 4200), (wl.F16, 3, 1400)])
def test_direct_and_staged_launches_of_the_other_storage_types(dtype, B, D, a_kind):
    """Which launches read B and C directly (they leave the workspace alone) and what either kind gives: static chunks, the chunk
    in device memory, sequences of unequal lengths; one kind of rows and two (beyond 4096 rows)."""
    L = 1100
    cfg = wl.Config("edges_kinds", B, D, 16, L, dtype, 16, (), seqlens=None if B == 1 else (L, 530, 1024)[:B], seed=4300 + D)
    w = wl.make(cfg, a_kind=a_kind)
    d = upload(w)
    rows = np.unique(np.concatenate([[0, 1, D - 2, D - 1], np.random.default_rng(5).integers(0, D, 4)]))
    y_ref, s_ref = oracle_scan(w, rows=rows)
    n = B * D
    ws = torch.empty(corey.selective_scan_fwd_workspace(B, 16, L), dtype=torch.uint8, device="cuda")
    for chunk in (256, 512, 1024):
        for routed in (False, True):
            if dtype != wl.F32 or n <= 1024 or n > 3072:
                direct = n <= 3072
            else:                                         # binary32: as long as the waves of the launch are resident together
                pairs = corey.selective_scan_fwd_plan_split(B, D, 16, chunk)
                direct = not routed and (chunk == 256 or (chunk == 512 and n * (1 + pairs) <= 2048))
            ws.fill_(0x5A)
            dev = torch.full((B,), chunk, dtype=torch.int32, device="cuda") if routed else None
            y, s = _scan(d, 512 if routed else chunk, chunks_dev=dev, workspace=ws)
            what = f"chunk {chunk} routed {routed}"
            assert bool((ws == 0x5A).all()) == direct, what
            check_y(y_to_f64(y)[:, rows], y_ref, cfg, "y " + what)
            assert_close(s.cpu().numpy()[:, rows], s_ref, fp32_rtol(L), "state " + what)


@pytest.mark.parametrize("dtype,B,D,N", [(wl.BF16, 1, 64, 16), (wl.F32, 2, 33, 4), (wl.F16, 1, 1536, 8), (wl.BF16, 1, 1537, 16)])
def test_the_longest_chunk_is_launched_as_the_tiles_it_is_walked_in(dtype, B, D, N):
    """Chunk 2048 on few rows takes the launch of chunk 1024, two rows per channel where that has them: the same bits, static and
    with the chunk in device memory."""
    cfg = wl.Config("edges_2048", B, D, N, 2500, dtype, 16, (), seed=4400 + D)
    d = upload(wl.make(cfg, a_kind="random", with_h0=True))
    want = _scan(d, 1024)
    for dev in (None, torch.full((B,), 2048, dtype=torch.int32, device="cuda")):
        got = _scan(d, 512 if dev is not None else 2048, chunks_dev=dev)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16, wl.F32])
@pytest.mark.parametrize("N", [4, 8, 12])
@pytest.mark.parametrize("gate", [True, False])
def test_tiles_requested_ahead(N, gate, dtype):
    """Direct launches ask for the gate and the next tile a group of states before the last: rows of one group, two and three, of one
    full tile, several and a partial one behind them, with and without a gate."""
    for L in (64, 128, 512, 1024, 1100):
        cfg = wl.Config("edges_ahead", 2, 5, N, L, dtype, 16, (), seed=4400 + L + N)
        w = wl.make(cfg, a_kind="random", with_h0=True)
        d = upload(w)
        if not gate:
            d["z"] = None
        y_ref, s_ref = oracle_scan(w, use_z=gate)
        for chunk in (16, 64, 128, 256, 512, 1024):
            for whole in (False, True):
                y, s = _scan(d, chunk, whole_rows=whole)
                check_y(y_to_f64(y), y_ref, cfg, f"y L {L} chunk {chunk}")
                assert_close(s.cpu().numpy(), s_ref, fp32_rtol(L), f"state L {L} chunk {chunk}")


@pytest.mark.parametrize("a_kind", ["mamba", "random"])
@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16, wl.F32])
@pytest.mark.parametrize("N", [4, 8, 12])
def test_tiles_requested_ahead_of_routed_and_padded_rows(N, dtype, a_kind):
    """The same loops with the chunk in device memory (one for all sequences, one each, neither the host's), with the structured A, and
    with sequences that end inside a tile behind full ones in the middle of their rows; the tensor's last row ends beside a lane's run."""
    for lens in ((1101, 530, 1024), (530, 1024, 1101), (67, 33, 64)):
        L = max(lens)
        cfg = wl.Config("edges_ahead_routed", 3, 5, N, L, dtype, 16, (), seqlens=lens, seed=4500 + L + N)
        w = wl.make(cfg, a_kind=a_kind, with_h0=True)
        d = upload(w)
        for b, n in enumerate(lens):                        # what lies behind a sequence's end is read into no result
            for name in ("u", "delta", "z", "B", "C"):
                d[name][b, :, n:] = float("nan")
        y_ref, s_ref = oracle_scan(w)
        routes = [(c, None) for c in (16, 64, 256, 512, 1024)]
        routes += [(512 if c != 512 else 64, (c,) * 3) for c in (16, 64, 256, 512, 1024, 2048)] + [(256, (64, 1024, 512)), (16, (2048, 16, 128))]
        for chunk, dev in routes:
            dev_t = None if dev is None else torch.tensor(dev, dtype=torch.int32, device="cuda")
            for whole in (False, True):
                y, s = _scan(d, chunk, chunks_dev=dev_t, whole_rows=whole)
                what = f"lens {lens} chunk {chunk} routed {dev} whole {whole}"
                check_y(y_to_f64(y), y_ref, cfg, "y " + what)
                assert_close(s.cpu().numpy(), s_ref, fp32_rtol(L), "state " + what)
