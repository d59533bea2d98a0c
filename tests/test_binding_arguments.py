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
WS = lambda: gpu(1 << 20, dtype=torch.uint8)

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
