"""The work a user of this framework has it do, as cases to be timed.

A case is a dict of plain values.  `kind` says which of the public paths it takes:

  layer      a prompt through one layer as the README shows it: causal convolution and SiLU, the statistic of its output on
             the range the convolution left, the chunk rule, the scan with the routed chunk.  Outputs and workspaces are
             left to the calls.
  step       the statistic and the rule on a u that is already there, then the scan with the chunk read from GPU memory:
             the timed step of bench.py, on buffers the program keeps.
  scan       the scan alone at a chunk the caller fixes (the static policies), on buffers the program keeps.
  statistic  histogram, H and r of a tensor, without a scan.
  decode     one generated token of one layer: the convolution's single step and the state update.

Sizes are those of workloads.CONFIGS (layers of 1024 to 5120 channels, 256 to 16384 steps), of bench.py's decode block
(1, 64 and 512 sequences) and of the tests (other N, odd lengths), with the value distributions of workloads.py.
"""
import math

import torch

import paper_2604_10597_amd as corey

DTYPES = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}
SIZE = {"bf16": 2, "fp16": 2, "fp32": 4}
WIDTH = 4          # taps of the convolution: every Mamba layer has four
# most values of [B, D, L] a drawn case may have (x N / 16 states): below the largest listed case's 84 million, so that the
# slower forms (short tiles, odd rows, fp32) do not cost more than that one
MOST = {"bf16": 32e6, "fp16": 32e6, "fp32": 12e6}


def listed():
    return [
        # the smallest layer of the test configurations, everything in binary32: launches and host work are its time
        dict(name="step_tiny_fp32", kind="step", dtype="fp32", B=1, D=64, N=16, L=256, K=16, u="normal", A="init", lens="", h0=False),
        # a 130m-sized layer, one prompt, the recommended cheap routing: guarded rule on the sampled statistic, reduced
        # inside the scan's first kernel
        dict(name="layer_130m", kind="layer", dtype="bf16", B=1, D=1536, N=16, L=2048, K=256, A="trained", route="deferred", mode=4, stride=8),
        # a 370m-sized layer on a prompt of no special length (the paper's prompts have 976, 182, 122 tokens): rows of odd length
        dict(name="layer_370m_prompt_977", kind="layer", dtype="bf16", B=1, D=2048, N=16, L=977, K=256, A="trained", route="deferred", mode=0, stride=1),
        # a batch of four through a 370m-sized layer, exact statistic, one chunk for the batch
        dict(name="step_370m_batch", kind="step", dtype="bf16", B=4, D=2048, N=16, L=4096, K=256, u="mixture", A="trained", lens="", h0=False),
        # a right-padded batch of unequal lengths, every sequence routed on its own
        dict(name="step_1p4b_padded", kind="step", dtype="bf16", B=2, D=4096, N=16, L=8192, K=256, u="normal", A="trained", lens="8192,2048", h0=False),
        # long-context prefill of a 2.8b-sized layer: bench.py's timed step
        dict(name="step_2p8b_long", kind="step", dtype="bf16", B=1, D=5120, N=16, L=16384, K=256, u="outliers", A="trained", lens="", h0=False),
        # the paper's kernel benchmark: batch 1, 1024 channels, 4096 steps, fp16, static chunk 512, freshly initialised A
        dict(name="scan_paper_fp16", kind="scan", dtype="fp16", B=1, D=1024, N=16, L=4096, A="init", chunk=512, h0=False),
        # the next 1000 tokens of two prompts in binary32, from the state the first part left
        dict(name="scan_fp32_continued", kind="scan", dtype="fp32", B=2, D=1536, N=16, L=1000, A="trained", chunk=256, h0=True),
        # the exact statistic of a batch from one pass over it
        dict(name="statistic_one_sweep", kind="statistic", dtype="bf16", B=4, D=2048, L=4096, K=256, u="mixture", lens="", form="one_sweep"),
        # generation: a single sequence, a serving batch, a large one
        dict(name="decode_1", kind="decode", dtype="bf16", B=1, D=5120, N=16, A="trained"),
        dict(name="decode_64", kind="decode", dtype="bf16", B=64, D=5120, N=16, A="trained"),
        dict(name="decode_512", kind="decode", dtype="bf16", B=512, D=5120, N=16, A="trained"),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, even over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _channels(rng):
    """Layers have multiples of 64 channels; now and then any number (a shard of one)."""
    return _spread(rng, 64, 5120) if rng.random() < 0.2 else 64 * _spread(rng, 1, 80)


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "step", "step", "step", "scan", "scan", "statistic", "decode", "decode"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "fp16", "fp32"])
    A = rng.choice(["trained", "trained", "init"])
    N = rng.choice([16, 16, 16, 16, 8, 32, 64])
    if kind == "decode":
        while True:
            B, D = _spread(rng, 1, 512), _channels(rng)
            if B * D * N <= 512 * 5120 * 16:
                return dict(kind=kind, dtype=dtype, B=B, D=D, N=N, A=A)
    chunk = rng.choice([64, 128, 256, 512, 1024, 2048])
    while True:
        B, D = _spread(rng, 1, 8), _channels(rng)
        L = _spread(rng, 16, 16384)
        if rng.random() < 0.3:
            L = (L + 63) // 64 * 64            # padded or packed to a round length
        work = B * D * L * N / 16
        if kind == "scan" and chunk < 256:
            work *= 4                          # short tiles are the slow end of the sweep
        if work <= MOST[dtype]:
            break
    lens = ""
    if kind in ("step", "statistic") and B > 1 and rng.random() < 0.5:
        lens = ",".join(str(L if b == 0 else _spread(rng, min(16, L), L)) for b in range(B))
    u = rng.choice(["normal", "mixture", "outliers"])
    K = rng.choice([64, 256, 256, 256, 1024])
    if kind == "layer":
        route = rng.choice(["deferred", "device"])
        mode, stride = rng.choice([(0, 1), (4, 8)])
        return dict(kind=kind, dtype=dtype, B=B, D=D, N=N, L=L, K=K, A=A, route=route, mode=mode, stride=stride)
    if kind == "step":
        return dict(kind=kind, dtype=dtype, B=B, D=D, N=N, L=L, K=K, u=u, A=A, lens=lens, h0=rng.random() < 0.3)
    if kind == "scan":
        return dict(kind=kind, dtype=dtype, B=B, D=D, N=N, L=L, A=A, chunk=chunk, h0=rng.random() < 0.3)
    form = "one_sweep" if dtype != "fp32" and not lens and rng.random() < 0.4 else "two_sweeps"
    return dict(kind=kind, dtype=dtype, B=B, D=D, L=L, K=K, u=u, lens=lens, form=form)


class _Draws:
    """Tensors of one seed, made on the GPU."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))
        self.dtype = dtype

    def f32(self, *shape):
        return torch.randn(shape, generator=self.g, device="cuda")

    def uniform(self, lo, hi, *shape):
        return torch.rand(shape, generator=self.g, device="cuda") * (hi - lo) + lo

    def normal(self, *shape, scale=1.0):
        return (self.f32(*shape) * scale).to(self.dtype)

    def u(self, kind, B, D, L):
        """The scan's input: N(0,1); or 70 % of that and 30 % Laplace(0,3); or N(0,1) with 1 % of the channels x20."""
        v = self.f32(B, D, L)
        if kind == "mixture":
            e = self.uniform(-0.5, 0.5, B, D, L)
            lap = -3.0 * e.sign() * torch.log1p(-2.0 * e.abs().clamp(max=0.4999999))
            v = torch.where(self.uniform(0.0, 1.0, B, D, L) < 0.3, lap, v)
        elif kind == "outliers":
            ch = torch.randperm(D, generator=self.g, device="cuda")[: max(1, D // 100)]
            v[:, ch] *= 20.0
        return v.to(self.dtype)

    def parameters(self, A, D, N):
        """A, D and the step bias of a layer: A = -(1 .. N) as initialised, or each entry moved as training moves it."""
        a = -torch.arange(1, N + 1, device="cuda", dtype=torch.float32).expand(D, N)
        if A == "trained":
            a = a * torch.exp(0.2 * self.f32(D, N))
        return dict(A=a.contiguous(), Dv=self.f32(D), delta_bias=self.uniform(math.log(1e-3), math.log(1e-1), D))


def prepare(case, seed):
    c = dict(case)
    d = _Draws(seed, DTYPES[c["dtype"]])
    kind, B, D = c["kind"], c["B"], c["D"]
    s = dict(kind=kind, c=c)
    if kind != "statistic":
        N = c["N"]
        s.update(d.parameters(c["A"], D, N))
    if kind in ("layer", "decode"):
        k = WIDTH ** -0.5
        s["conv_weight"], s["conv_bias"] = d.uniform(-k, k, D, WIDTH), d.uniform(-k, k, D)
    if kind == "decode":
        s["state"], s["conv_state"] = d.f32(B, D, N), d.normal(B, D, WIDTH - 1)
        s["x"] = d.normal(B, D, 1)
        s["delta"], s["z"] = d.normal(B, D, scale=0.5), d.normal(B, D)
        s["Bt"], s["Ct"] = d.normal(B, N), d.normal(B, N)
        return s
    L = c["L"]
    if kind == "layer":
        s["x"] = d.normal(B, D, L)
        s["policy"] = corey.policy_default()
        s["policy"].mode = c["mode"]
    else:
        s["u"] = d.u(c.get("u", "normal"), B, D, L)
    lens = [int(v) for v in c.get("lens", "").split(",") if v]
    s["seqlens"] = torch.tensor(lens, dtype=torch.int32, device="cuda") if lens else None
    if kind == "statistic":
        return s
    s["delta"], s["z"] = d.normal(B, D, L, scale=0.5), d.normal(B, D, L)
    s["Bm"], s["Cm"] = d.normal(B, N, L), d.normal(B, N, L)
    s["h0"] = d.f32(B, D, N) if c.get("h0") else None
    if kind in ("step", "scan"):                      # the buffers such a program keeps from call to call
        s["y"] = torch.empty_like(s["u"])
        s["last_state"] = torch.empty((B, D, N), dtype=torch.float32, device="cuda")
        s["workspace"] = torch.empty(corey.selective_scan_fwd_workspace(B, N, L), dtype=torch.uint8, device="cuda")
    if kind == "step":
        nh = B if lens else 1
        s["policy"] = corey.policy_default()
        s["out"] = dict(counts=torch.empty((nh, c["K"]), dtype=torch.int32, device="cuda"),
                        H=torch.empty(nh, dtype=torch.float64, device="cuda"), r=torch.empty(nh, dtype=torch.float64, device="cuda"),
                        range=torch.empty((nh, 2), dtype=torch.float32, device="cuda"),
                        chunks=torch.empty(nh, dtype=torch.int32, device="cuda"))
        s["out"]["workspace"] = torch.empty(corey.corey_entropy_hist_workspace(B, c["K"]), dtype=torch.uint8, device="cuda")
    return s


RESULTS = ("counts", "H", "r", "range", "chunks")


def run(s):
    c = s["c"]
    if s["kind"] == "layer":
        u, conv_state, parts = corey.causal_conv1d_silu_fwd(s["x"], s["conv_weight"], s["conv_bias"], want_state=True)
        sampling = dict(stride=c["stride"], block=512) if c["stride"] > 1 else {}
        call = corey.corey_route_device_deferred if c["route"] == "deferred" else corey.corey_route_device
        route = call(u, c["K"], s["policy"], range_parts=parts, **sampling)
        how = dict(route=route["route"]) if c["route"] == "deferred" else dict(chunks_dev=route["chunks"])
        y, state = corey.selective_scan_fwd(u, s["delta"], s["A"], s["Bm"], s["Cm"], Dv=s["Dv"], z=s["z"],
                                            delta_bias=s["delta_bias"], chunk=512, **how)
        return dict({k: route[k] for k in RESULTS}, u=u, conv_state=conv_state, y=y, state=state)
    if s["kind"] == "step":
        out = corey.corey_route_device(s["u"], c["K"], s["policy"], seqlens=s["seqlens"], out=s["out"])
        y, state = corey.selective_scan_fwd(s["u"], s["delta"], s["A"], s["Bm"], s["Cm"], Dv=s["Dv"], z=s["z"],
                                            delta_bias=s["delta_bias"], h0=s["h0"], seqlens=s["seqlens"], chunk=512,
                                            chunks_dev=out["chunks"], y=s["y"], last_state=s["last_state"], workspace=s["workspace"])
        return dict({k: out[k] for k in RESULTS}, y=y, state=state)
    if s["kind"] == "scan":
        y, state = corey.selective_scan_fwd(s["u"], s["delta"], s["A"], s["Bm"], s["Cm"], Dv=s["Dv"], z=s["z"],
                                            delta_bias=s["delta_bias"], h0=s["h0"], chunk=c["chunk"], y=s["y"],
                                            last_state=s["last_state"], workspace=s["workspace"])
        return dict(y=y, state=state)
    if s["kind"] == "statistic":
        if c["form"] == "one_sweep":
            out = corey.corey_entropy_hist_onesweep(s["u"], c["K"])
        else:
            out = corey.corey_entropy_hist(s["u"], c["K"], seqlens=s["seqlens"])
        return {k: out[k] for k in RESULTS[:4]}
    # one token: the states move on in place, as in a generation loop
    u1, s["conv_state"], _ = corey.causal_conv1d_silu_fwd(s["x"], s["conv_weight"], s["conv_bias"], state_in=s["conv_state"],
                                                          want_state=True)
    y = corey.selective_state_update(s["state"], u1[:, :, 0].contiguous(), s["delta"], s["A"], s["Bt"], s["Ct"], Dv=s["Dv"],
                                     z=s["z"], delta_bias=s["delta_bias"])
    return dict(u=u1, y=y, state=s["state"], conv_state=s["conv_state"])


def work(case):
    """Bytes: every input read once, every output written once (u of a layer is one).  Operations: 7 per state and step (two
    products, two fused multiply-adds, one exponential), 2 per tap, about 3 per value of a histogram."""
    c, s = case, SIZE[case["dtype"]]
    B, D, kind = c["B"], c["D"], c["kind"]
    if kind == "decode":
        rows, N = B * D, c["N"]
        return dict(bytes=8 * rows * N + s * (2 * rows * (WIDTH - 1) + 5 * rows + 2 * B * N) + 4 * D * (N + WIDTH + 3),
                    flops=rows * (7 * N + 2 * WIDTH))
    L = c["L"]
    lens = [int(v) for v in c.get("lens", "").split(",") if v] or [L] * B
    values = D * sum(lens)
    if kind == "statistic":
        return dict(bytes=s * values + 4 * c["K"] * len(lens), flops=3 * values)
    N = c["N"]
    n = 3 * s * values + s * B * D * L + 2 * s * N * sum(lens) + 4 * D * (N + 2) + 4 * B * D * N * (2 if c.get("h0") else 1)
    f = 7 * N * values
    if kind == "layer":
        n += s * values + 4 * D * (WIDTH + 1) + 4 * c["K"]
        f += (2 * WIDTH + 3) * values
    elif kind == "step":
        n += 4 * c["K"] * len(lens)
        f += 3 * values
    return dict(bytes=n, flops=f)


def tolerance(case):
    """Counts, chunks and the statistic of the same bits are the same.  y carries one rounding to the storage type (half an
    ulp: 2^-8, 2^-11 relative) and the differences of binary32 sums in another order."""
    if case["kind"] == "statistic":
        return {"rel": 1e-12}
    return {"rel": {"bf16": 4e-3, "fp16": 5e-4, "fp32": 1e-5}[case["dtype"]]}
