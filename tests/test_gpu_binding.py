"""The binding's handling of tensors that only the caller's result dict holds."""
import pytest
import torch

import paper_2604_10597_amd as corey

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["workspace", "counts"])
def test_a_tensor_taken_out_of_the_dict_during_the_call_keeps_its_memory(name):
    """Code that runs inside the call (here an argument's __float__, otherwise another thread) drops the only reference to a
    buffer: the buffer must not become another tensor's memory before the call's work is enqueued on it."""
    print(f"[case] {name} taken out of the result dict", flush=True)
    x = torch.randn(2, 64, 512, device="cuda", dtype=torch.bfloat16)
    out = corey.corey_route_device(x, 256)
    want = {k: out[k].clone() for k in ("counts", "H", "chunks")}
    taken = []

    class Lambda:
        def __float__(self):
            n = out[name].numel() * out[name].element_size()
            del out[name]
            taken.extend(torch.full((n,), 7, dtype=torch.uint8, device="cuda") for _ in range(4))
            return 0.0

    out["H"].fill_(0)
    corey.corey_route_device(x, 256, out=out, ema_lambda=Lambda())
    torch.cuda.synchronize()
    assert len(taken) == 4 and all(bool((t == 7).all()) for t in taken)
    for k in want:
        if k in out:
            assert torch.equal(out[k], want[k]), k
