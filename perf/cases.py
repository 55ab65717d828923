"""The work that programs have this library do, as cases to be timed and checked.

A case is a dict of plain values.  `kind` says which call a program makes:

  fwd    attention forward                       (fa_fwd / fa_fwd_gqa)
  bwd    its gradients, forward results in hand  (fa_bwd / fa_bwd_gqa)
  step   one training step of the layer: both in turn
  fp8    quantise Q, K and V, then the FP8 forward (fa_fp8_quant_hadamard, fa_fwd_fp8 / _gqa)

with q [B, H, N, d], k and v [B, H_kv, N, d], d in {64, 128, 256} and scale d^-1/2.
"""
import math

import torch

from paper_2407_08608_amd import binding

_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
_ELEM = {"f32": 4, "bf16": 2, "f16": 2}


def _case(name, kind, dtype, B, H, H_kv, N, d, causal):
    c = {"kind": kind, "dtype": dtype, "B": B, "H": H, "H_kv": H_kv, "N": N, "d": d, "causal": causal}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a short prompt or a patch sequence in one request: launch and latency decide
        _case("fwd_small", "fwd", "bf16", 1, 16, 16, 100, 64, False),
        # 16k tokens of training batch (hidden size 2048) in short sequences, as in the benchmark's sweep
        _case("fwd_short", "fwd", "bf16", 32, 16, 16, 512, 128, True),
        # the same tokens as one long sequence: the sweep's largest forward
        _case("fwd_long", "fwd", "bf16", 1, 16, 16, 16384, 128, False),
        # prefill of a few prompts of odd length with shared key/value heads
        _case("fwd_gqa_ragged", "fwd", "f16", 2, 32, 8, 3001, 128, True),
        # the widest head dimension at a middle sequence length
        _case("fwd_d256", "fwd", "bf16", 8, 8, 8, 2048, 256, True),
        # full precision: reference runs and validation of reduced-precision results
        _case("fwd_f32", "fwd", "f32", 2, 8, 8, 1000, 64, False),
        # low-precision serving, long sequences: pre-pass on the 16-bit tensors and the FP8 forward
        _case("fp8_long", "fp8", "bf16", 2, 16, 16, 8192, 128, False),
        # the same on a narrow head, odd length, under a mask
        _case("fp8_d64", "fp8", "bf16", 4, 32, 32, 2500, 64, True),
        # a small training step: forward and gradients, a few launches each
        _case("step_small", "step", "f16", 2, 8, 8, 333, 64, False),
        # training, the usual middle of the sweep: gradients under the causal mask
        _case("bwd_causal", "bwd", "bf16", 4, 16, 16, 4096, 128, True),
        # gradients at the widest head dimension
        _case("bwd_d256", "bwd", "bf16", 2, 8, 8, 8192, 256, False),
        # fine-tuning with shared key/value heads, one sequence per GPU
        _case("bwd_gqa", "bwd", "bf16", 1, 32, 4, 2048, 128, True),
    ]


# most FLOPs of a drawn case, by kind: each well below the largest listed case's time
_MOST = {"fwd": 1.0e12, "bwd": 1.0e12, "step": 1.0e12, "fp8": 1.0e12, "f32": 2.0e10}


def draw(rng):
    kind = rng.choice(["fwd", "fwd", "fwd", "fp8", "fp8", "bwd", "bwd", "step"])
    dtype = rng.choice(["bf16", "bf16", "f16"])
    d = rng.choice([64, 128, 128, 256])
    if kind == "fwd" and rng.random() < 0.15:
        dtype, d = "f32", 64
    most = _MOST["f32" if dtype == "f32" else kind]
    while True:
        N = int(round(math.exp(rng.uniform(math.log(16), math.log(16384)))))
        if rng.random() < 0.4:  # half-way regular lengths are as common as odd ones
            N = max(16, N // 64 * 64)
        B = int(round(math.exp(rng.uniform(0, math.log(32)))))
        H = rng.choice([1, 2, 4, 8, 12, 16, 32])
        H_kv = rng.choice([h for h in (1, 2, 4, 8, 16) if H % h == 0]) if rng.random() < 0.35 else H
        c = _case(None, kind, dtype, B, H, H_kv, N, d, rng.random() < 0.5)
        if work(c)["flops"] <= most and B * H * N * d <= 1 << 27:
            return c


def _visible(c):
    """Number of (query, key) pairs of one head that enter the softmax."""
    return c["N"] * (c["N"] + 1) / 2 if c["causal"] else float(c["N"]) ** 2


def work(case):
    c = case
    e, n_q, n_kv = _ELEM[c["dtype"]], c["B"] * c["H"] * c["N"], c["B"] * c["H_kv"] * c["N"]
    q, kv, row = n_q * c["d"] * e, n_kv * c["d"] * e, n_q * 4
    product = 2.0 * c["B"] * c["H"] * _visible(c) * c["d"]
    if c["kind"] == "fwd":  # Q, K, V in; O, L out
        return {"bytes": 2 * q + 2 * kv + row, "flops": 2 * product}
    if c["kind"] == "bwd":  # Q, O, dO, K, V, L in; dQ, dK, dV out
        return {"bytes": 4 * q + 4 * kv + row, "flops": 5 * product}
    if c["kind"] == "step":  # Q, K, V, dO in; O, L, dQ, dK, dV out
        return {"bytes": 4 * q + 4 * kv + row, "flops": 7 * product}
    # fp8: 16-bit Q, K, V in; codes, scales, bf16 O and L out
    blocks = -(-c["N"] // 128) * 4 * (c["B"] * c["H"] + 2 * c["B"] * c["H_kv"])
    return {"bytes": (q + 2 * kv) + (q + 2 * kv) // 2 + blocks + 2 * n_q * c["d"] + row, "flops": 2 * product}


def tolerance(case):
    if case["dtype"] == "f32":
        return {"rel": 4e-6}
    if case["kind"] == "fp8":
        # P is rounded to e4m3 (half an ulp: 2^-4) relative to a reference that another tiling would set elsewhere
        return {"rel": 3e-2}
    # about four times the rounding of P, dS and the outputs to the 16-bit type (2^-9 and 2^-12 relative)
    return {"rel": 1e-2 if case["dtype"] == "bf16" else 1.5e-3}


def _inputs(case, seed):
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + 17)

    def normal(heads, heavy):
        x = torch.randn((c["B"], heads, c["N"], c["d"]), generator=g, device="cuda", dtype=torch.float32)
        if heavy:  # activations with outliers, the case that the quantiser's transform is for
            hit = torch.rand(x.shape, generator=g, device="cuda") < 0.001
            x += hit * (10.0 * torch.randn(x.shape, generator=g, device="cuda", dtype=torch.float32))
        return x.to(_DTYPES[c["dtype"]])

    heavy = c["kind"] == "fp8"
    t = {"q": normal(c["H"], heavy), "k": normal(c["H_kv"], heavy), "v": normal(c["H_kv"], heavy)}
    if c["kind"] in ("bwd", "step"):
        t["dout"] = normal(c["H"], False)
    if c["kind"] == "fp8":
        bits = torch.randint(0, 2, (c["d"],), generator=g, device="cuda", dtype=torch.int32)
        t["signs"] = (2 * bits - 1).to(torch.int8)
    return t


def _forward(c, t):
    fn = binding.fa_fwd if c["H_kv"] == c["H"] else binding.fa_fwd_gqa
    return fn(t["q"], t["k"], t["v"], c["d"] ** -0.5, c["causal"])


def prepare(case, seed):
    state = _inputs(case, seed)
    state["case"] = dict(case)
    if case["kind"] == "bwd":
        state["o"], state["lse"] = _forward(case, state)
    return state


def run(state):
    c, t = state["case"], state
    scale, causal, shared = c["d"] ** -0.5, c["causal"], c["H_kv"] != c["H"]
    if c["kind"] == "fwd":
        return _forward(c, t)
    if c["kind"] == "fp8":
        q8, qs = binding.fa_fp8_quant_hadamard(t["q"], t["signs"])
        k8, ks = binding.fa_fp8_quant_hadamard(t["k"], t["signs"])
        v8, vs = binding.fa_fp8_quant_hadamard(t["v"])
        fn = binding.fa_fwd_fp8_gqa if shared else binding.fa_fwd_fp8
        o, lse = fn(q8, k8, v8, qs, ks, vs, scale, causal)
        return q8, k8, v8, qs, ks, vs, o, lse
    bwd = binding.fa_bwd_gqa if shared else binding.fa_bwd
    if c["kind"] == "bwd":
        return bwd(t["q"], t["k"], t["v"], t["o"], t["lse"], t["dout"], scale, causal)
    o, lse = _forward(c, t)
    return (o, lse) + tuple(bwd(t["q"], t["k"], t["v"], o, lse, t["dout"], scale, causal))


# ------------------------------------------------------------------------------------------
# 64-bit reference


def _probabilities(q, k, lo, hi, scale, causal):
    """softmax rows lo..hi of one head, and their logsumexp."""
    s = torch.mm(q[lo:hi], k.t().contiguous()) * scale
    if causal:
        key = torch.arange(k.shape[0], device=s.device)
        s.masked_fill_(key[None, :] > torch.arange(lo, hi, device=s.device)[:, None], -math.inf)
    lse = torch.logsumexp(s, dim=1)
    return torch.exp(s - lse[:, None]), lse


def _quantise(x, signs):
    """Codes and scales as the pre-pass defines them: fp32 butterflies of stride 1, 2, ..., d / 2, one scale per
    128 rows of a head, codes rounded to nearest even."""
    B, H, N, d = x.shape
    y = x.float()
    if signs is not None:
        y = y * signs.float()
        stride = 1
        while stride < d:
            y = y.view(B, H, N, d // (2 * stride), 2, stride)
            a, b = y[..., 0, :], y[..., 1, :]
            y = torch.stack((a + b, a - b), dim=-2).reshape(B, H, N, d)
            stride *= 2
        y = y * torch.tensor(d, dtype=torch.float64).rsqrt().float().to(y.device)
    nb = -(-N // 128)
    pad = torch.zeros((B, H, nb * 128, d), device=y.device)
    pad[:, :, :N] = y
    pad = pad.view(B, H, nb, 128 * d)
    amax = pad.abs().amax(dim=-1)
    one = torch.ones_like(amax)
    scales = torch.where(amax > 0, amax / 448.0, one)
    factor = torch.where(amax > 0, 448.0 / amax, one)
    codes = (pad * factor[..., None]).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
    codes = codes.view(B, H, nb * 128, d)[:, :, :N].contiguous()
    return codes, scales


def _dequantise(codes, scales):
    rows = scales.double().repeat_interleave(128, dim=-1)[:, :, :codes.shape[2]]
    return codes.view(torch.float8_e4m3fn).double() * rows[..., None]


def exact(case, seed):
    c = case
    t = _inputs(c, seed)
    scale, causal, N, group = c["d"] ** -0.5, c["causal"], c["N"], c["H"] // c["H_kv"]
    codes = ()
    if c["kind"] == "fp8":
        pairs = [_quantise(t["q"], t["signs"]), _quantise(t["k"], t["signs"]), _quantise(t["v"], None)]
        q, k, v = (_dequantise(*p) for p in pairs)
        codes = tuple(p[0] for p in pairs) + tuple(p[1] for p in pairs)
    else:
        q, k, v = (t[n].double() for n in ("q", "k", "v"))
    o = torch.empty_like(q)
    lse = torch.empty(q.shape[:3], device=q.device, dtype=torch.float64)
    grads = c["kind"] in ("bwd", "step")
    if grads:
        do = t["dout"].double()
        dq, dk, dv = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
    for b in range(c["B"]):
        for h in range(c["H"]):
            kh, vh = k[b, h // group], v[b, h // group]
            for lo in range(0, N, 4096):
                hi = min(N, lo + 4096)
                p, lse[b, h, lo:hi] = _probabilities(q[b, h], kh, lo, hi, scale, causal)
                o[b, h, lo:hi] = torch.mm(p, vh)
                if grads:
                    g = do[b, h, lo:hi]
                    ds = torch.mm(g, vh.t().contiguous()) - (g * o[b, h, lo:hi]).sum(dim=1, keepdim=True)
                    ds *= p
                    dv[b, h // group] += torch.mm(p.t().contiguous(), g)
                    dq[b, h, lo:hi] = torch.mm(ds, kh) * scale
                    dk[b, h // group] += torch.mm(ds.t().contiguous(), q[b, h, lo:hi]) * scale
    if c["kind"] == "bwd":
        return dq, dk, dv
    if c["kind"] == "step":
        return o, lse, dq, dk, dv
    return codes + (o, lse)
