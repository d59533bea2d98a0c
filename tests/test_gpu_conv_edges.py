"""The convolution at the edges of its dispatch: one step by words of x (even D) or by rows, rows on either side of two vectors,
last vectors moved back by every remainder, waves that stay in one row, more vectors than one per lane, views at any element."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_10597_amd as corey
from gpu_util import to_dev
from paper_2604_10597_amd import workloads as wl
from test_gpu_conv import _parts_range, _tolerance, _widen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16, wl.F32])
@pytest.mark.parametrize("B,D,L", [(1, 1, 1), (3, 7, 1), (2, 514, 1), (300, 2500, 1), (7, 163840, 1), (2, 524300, 1),
                                   (51, 5120, 1), (52, 5120, 1), (102, 5120, 1), (103, 5120, 1), (700, 5120, 1),      # one sequence a lane, two, seven
                                   (2, 6, 7), (2, 3, 8), (2, 5, 15), (2, 3, 16), (1, 9, 17),
                                   (3, 2, 23), (1, 3, 511), (2, 3, 512), (1, 3, 513), (5, 1, 1024), (3, 1500, 1500), (2, 1100, 1024)])
def test_outputs_state_and_range(B, D, L, dtype):
    print(f"[case] conv edges {B} {D} {L} {dtype}", flush=True)
    cfg = wl.Config("conv_edges", B, D, 16, L, dtype, 16, (), seed=6000 + L)
    c = wl.make_conv(cfg, 4, with_state=True)
    val = c["val"]
    xd, sd = to_dev(c["dev"]["x"], dtype), to_dev(c["dev"]["state_in"], dtype)
    wd, bd = torch.from_numpy(c["dev"]["weight"]).cuda(), torch.from_numpy(c["dev"]["bias"]).cuda()
    u, so, parts = corey.causal_conv1d_silu_fwd(xd, wd, bd, sd, want_state=True)
    off = torch.zeros(xd.numel() + 1, dtype=xd.dtype, device="cuda")          # the same rows one element further on
    off[1:].copy_(xd.view(-1))
    u1, so1, parts1 = corey.causal_conv1d_silu_fwd(off[1:].view(B, D, L), wd, bd, sd, want_state=True)
    torch.cuda.synchronize()
    ref_u, ref_so = oracle.causal_conv1d_silu(val["x"], val["weight"], val["bias"], val["state_in"])
    got = _widen(u).astype(np.float64)
    assert (np.abs(got - ref_u) <= _tolerance(ref_u, val, 4, dtype)).all()
    assert np.array_equal(_widen(so), ref_so)
    assert np.array_equal(_widen(u1), _widen(u)) and np.array_equal(_widen(so1), ref_so)
    for p in (parts, parts1):
        assert _parts_range(p) == (_widen(u).min(), _widen(u).max(), False)
    if dtype != wl.F32:                                                        # and with the bit-pattern table filled on the way
        table = torch.empty(corey.corey_pattern_table_workspace(), dtype=torch.uint8, device="cuda")
        u2, so2, _ = corey.causal_conv1d_silu_fwd(xd, wd, bd, sd, want_state=True, pattern_table=table)
        got = corey.corey_entropy_hist_from_table(table, u2.dtype, L, 64)
        want = corey.corey_entropy_hist(u, 64)
        torch.cuda.synchronize()
        assert np.array_equal(_widen(u2), _widen(u)) and np.array_equal(_widen(so2), ref_so)
        assert torch.equal(got["counts"], want["counts"])
