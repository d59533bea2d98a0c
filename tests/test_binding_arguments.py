"""What the binding makes of its arguments before the library sees them.  The tensors are fake ones: they report the GPU, a
type and a shape and own no memory, so a call whose arguments pass ends with a RuntimeError at the stream of a GPU that is not
there, or at their data pointers, and nothing is ever launched."""
from collections import OrderedDict, UserDict
from fractions import Fraction

import numpy as np
import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode

import paper_2604_10597_amd as corey

MODE = FakeTensorMode()


def gpu(*shape, dtype=torch.float32):
    with MODE:
        return torch.empty(shape, dtype=dtype, device="cuda")


def results(nh=1, K=16):
    return dict(counts=gpu(nh, K, dtype=torch.int32), H=gpu(nh, dtype=torch.float64), r=gpu(nh, dtype=torch.float64), range=gpu(nh, 2),
                chunks=gpu(nh, dtype=torch.int32))


X = lambda: gpu(2, 3, 64, dtype=torch.bfloat16)
WS = lambda: gpu(1 << 20, dtype=torch.uint8)          # more than any buffer asked for below

STATISTICS = {
    "hist": lambda **kw: corey.corey_entropy_hist(X(), workspace=WS(), **{"out": results(), "K": 16, **kw}),
    "static": lambda **kw: corey.corey_entropy_hist_static(X(), **{"out": results(), "K": 16, **kw}),
    "route": lambda **kw: corey.corey_route_device(X(), workspace=WS(), **{"out": results(), "K": 16, **kw}),
    "deferred": lambda **kw: corey.corey_route_device_deferred(X(), workspace=WS(), **{"out": results(), "K": 16, **kw}),
    "onesweep": lambda **kw: corey.corey_entropy_hist_onesweep(X(), table_ws=WS(), **{"out": results(), "K": 16, **kw}),
    "from_table": lambda **kw: corey.corey_entropy_hist_from_table(WS(), torch.bfloat16, **{"out": results(), "K": 16, "L": 64, **kw}),
}


@pytest.mark.parametrize("call", STATISTICS)
@pytest.mark.parametrize("value", [16.0, 2.5, "16", Fraction(16), None], ids=repr)
def test_whole_numbers_are_not_truncated_or_parsed(call, value):
    """A float, a string or anything else that does not offer itself as a whole number is refused where one is meant."""
    for name in {"onesweep": ("K",), "from_table": ("K", "L")}.get(call, ("K", "stride", "block")):
        with pytest.raises(TypeError):
            STATISTICS[call](**{name: value})


@pytest.mark.parametrize("call", STATISTICS)
@pytest.mark.parametrize("value", [16, np.int32(16), torch.tensor(16)], ids=repr)
def test_whole_numbers_of_any_kind_are_taken(call, value):
    with pytest.raises(RuntimeError):
        STATISTICS[call](K=value)


def test_arguments_that_are_converted():
    """chunk and the rule's L go through int(), ema_lambda through float()."""
    scan = lambda chunk: corey.selective_scan_fwd(X(), X(), gpu(3, 16), *(gpu(2, 16, 64, dtype=torch.bfloat16) for _ in range(2)),
                                                  chunk=chunk, y=X(), last_state=gpu(2, 3, 16), workspace=WS())
    for chunk in (256, 256.0, "256", np.int64(256)):
        with pytest.raises(RuntimeError):
            scan(chunk)
    with pytest.raises(ValueError):
        scan("x")
    rule = lambda L: corey.corey_select_chunk_device(gpu(1, dtype=torch.float64), L, out=gpu(1, dtype=torch.int32))
    for L in (64, 64.0, "64"):
        with pytest.raises(RuntimeError):
            rule(L)
    for lam in (0.5, 0, "0.5"):
        with pytest.raises(RuntimeError):
            STATISTICS["route"](ema_lambda=lam, ema_state=gpu(1, dtype=torch.float64))


@pytest.mark.parametrize("call", STATISTICS)
@pytest.mark.parametrize("kind", [dict, OrderedDict, UserDict])
def test_results_go_into_any_mapping(call, kind):
    with pytest.raises(RuntimeError):
        STATISTICS[call](out=kind(results()))
    part = results()
    del part["counts"]
    with pytest.raises(KeyError):
        STATISTICS[call](out=kind(part))


BAD_RESULTS = {
    "counts": [gpu(1, 15, dtype=torch.int32), gpu(1, 16), gpu(1, 16, dtype=torch.int64), gpu(2, 16, dtype=torch.int32)[:, ::2]],
    "H": [gpu(1), gpu(0, dtype=torch.float64)],
    "r": [gpu(1), gpu(0, dtype=torch.float64)],
    "range": [gpu(1), gpu(2, dtype=torch.float64)],
    "chunks": [gpu(1, dtype=torch.int64), gpu(0, dtype=torch.int32)],
}


@pytest.mark.parametrize("call", STATISTICS)
def test_results_must_have_room_on_the_gpu(call):
    """A result tensor of another type, with too few values, with gaps or in host memory never reaches a kernel."""
    kw = dict(policy=corey.policy_default()) if call in ("onesweep", "from_table") else {}
    for name, bad in BAD_RESULTS.items():
        if name == "chunks" and call in ("hist", "static"):
            continue
        for t in bad + [torch.zeros(64, dtype=results()[name].dtype)]:
            with pytest.raises((TypeError, ValueError)):
                STATISTICS[call](out=dict(results(), **{name: t}), **kw)


def test_results_of_any_shape_with_room_are_taken():
    for name, t in dict(counts=gpu(16, dtype=torch.uint32), H=gpu(8, dtype=torch.float64), range=gpu(2), chunks=gpu(1, 1, dtype=torch.int32)).items():
        with pytest.raises(RuntimeError):
            STATISTICS["route"](out=dict(results(), **{name: t}))


def test_other_buffers_must_have_room_on_the_gpu():
    bf16 = dict(dtype=torch.bfloat16)
    small = gpu(1000, dtype=torch.uint8)
    host = torch.zeros(1 << 20, dtype=torch.uint8)
    for call in ("hist", "static", "route", "deferred"):
        for parts in (small, host):
            with pytest.raises((TypeError, ValueError)):
                STATISTICS[call](range_parts=parts)
    for call in (corey.corey_entropy_hist, corey.corey_route_device, corey.corey_route_device_deferred):
        with pytest.raises(ValueError):
            call(X(), 16, workspace=host, out=results())
    for call in (corey.corey_route_device, corey.corey_route_device_deferred):
        with pytest.raises(ValueError):
            call(X(), 16, out=dict(results(), workspace=host))
    conv = lambda **kw: corey.causal_conv1d_silu_fwd(X(), gpu(3, 4), **{"u": X(), "range_parts": WS(), **kw})
    for kw in (dict(u=gpu(2, 3, 64)), dict(u=gpu(2, 3, 63, **bf16)), dict(state_in=gpu(2, 3, 3)), dict(state_in=gpu(2, 3, 2, **bf16)),
               dict(bias=gpu(2)), dict(bias=gpu(3, **bf16))):
        with pytest.raises(TypeError):
            conv(**kw)
    with pytest.raises(RuntimeError):
        conv(u=gpu(6, 64, **bf16), state_in=gpu(6, 3, **bf16), bias=gpu(3, 1))
    step = lambda y: corey.selective_state_update(gpu(2, 3, 16), gpu(2, 3, **bf16), gpu(2, 3, **bf16), gpu(3, 16), gpu(2, 16, **bf16),
                                                  gpu(2, 16, **bf16), y=y)
    for y in (gpu(2, 3), gpu(2, 2, **bf16)):
        with pytest.raises(TypeError):
            step(y)
    with pytest.raises(RuntimeError):
        step(gpu(6, **bf16))
    for out in (gpu(1, dtype=torch.int32), gpu(2, dtype=torch.int64)):
        with pytest.raises(TypeError):
            corey.corey_select_chunk_device(gpu(2, dtype=torch.float64), 64, out=out)
