"""Workloads of the attention library, as its users call it.

Each case is one call (or one pre-pass) through the public entry points of
``paper_2609_09721_amd.binding``, over the range the library is used in: the
smallest self-attention, batched short prompts, single prompts of 2K to 32K
tokens, generation steps against a long key/value cache, cross attention to a
short text, long non-causal self-attention, the MXFP8 Q K^T path, every
probability stage, both head dimensions, the quantisers alone and the offline
(tau, h) calibration.

``exact`` evaluates the same method in 64 bits with plain torch: Algorithm 2's
running row maximum over 64-key tiles, Algorithm 1's (or exp-then-quantize's)
codes and E8M0 scales per 32 keys, and the products with the MXFP4 value
operand (and MXFP8 Q and K on the low-bit path).
"""
import ctypes
import math

import numpy as np
import torch

from paper_2609_09721_amd import binding

LN2 = math.log(2.0)
PARAMS = {"efq": binding.PARAMS_MEAN, "lut": (math.log(1 / 24), 14 / math.log(24))}
C16 = (0, 1, 1, 1, 1, 1, 2, 2, 3, 3, 4, 5, 5, 6, 7, 7)
E2M1 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)


def _case(name, op, batch, seq_q, seq_k, heads_q, heads_kv, head_dim, causal, kind, dist="qwen", **more):
    return dict(name=name, op=op, batch=batch, seq_q=seq_q, seq_k=seq_k, heads_q=heads_q,
                heads_kv=heads_kv, head_dim=head_dim, causal=causal, kind=kind, dist=dist, **more)


def listed():
    return [
        # the smallest workload of the repository, through the one-argument
        # entry point without a workspace: launch and allocation latency
        _case("tiny_256", "efq", 1, 256, 256, 1, 1, 64, False, "efq", "normal"),
        # a batch of eight short evaluation prompts (Qwen3-8B heads)
        _case("prompts_8x333", "attn", 8, 333, 333, 32, 8, 128, True, "efq"),
        # one prompt of ordinary length
        _case("prompt_2k", "attn", 1, 2048, 2048, 32, 8, 128, True, "efq"),
        # one ordinary prompt on the low-bit Q K^T path
        _case("prompt_4k_lowbit", "lowbit", 1, 4096, 4096, 32, 8, 128, True, "efq"),
        # a generation step of eight sequences: one query each, whole call
        _case("step_8x6001", "attn", 8, 1, 6001, 32, 8, 128, False, "efq"),
        # a few queries of one sequence against a long quantised value cache
        _case("few_16x32768", "vhat", 1, 16, 32768, 32, 8, 128, False, "efq"),
        # cross attention of video tokens to a 512-token text (WAN2.2 heads)
        _case("cross_32760x512", "attn", 1, 32760, 512, 24, 24, 128, False, "efq", "wan"),
        # D = 64 heads, ragged, non-causal, the 16-level LUT stage
        _case("d64_4x1500_lut", "attn", 4, 1500, 1500, 12, 12, 64, False, "lut", "normal"),
        # the exp-then-quantize baseline at the paper's shortest length
        _case("prompt_16k_expq", "attn", 1, 16384, 16384, 32, 8, 128, True, "expq"),
        # the headline workload: Qwen3-8B heads, 32K tokens
        _case("prompt_32k", "attn", 1, 32768, 32768, 32, 8, 128, True, "efq"),
        # the offline (tau, h) calibration on a 1K calibration prompt
        _case("calibrate_1k_4x4", "calibrate", 1, 1024, 1024, 32, 8, 128, True, "efq", ntau=4, nh=4),
        # the quantisers alone, filling a long quantised cache
        _case("quantise_65537", "quant", 1, 65537, 65537, 32, 8, 128, False, "efq"),
    ]


def _log(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, n + rng.choice((0, 0, 1))))


def draw(rng):
    fam = rng.choice(("short", "prompt", "prompt", "step", "step", "cross", "self", "calibrate", "quant"))
    heads = rng.choice(((32, 8, 128), (32, 8, 128), (24, 24, 128), (16, 4, 64), (12, 12, 64)))
    kind = rng.choice(("efq", "efq", "efq", "lut", "expq", "expq6"))
    op = rng.choice(("attn", "attn", "lowbit", "vhat"))
    if fam == "short":
        s = _log(rng, 48, 2048)
        return _case("", op, rng.choice((1, 2, 4, 8)), s, s, *heads, rng.random() < 0.6, kind)
    if fam == "prompt":
        s = _log(rng, 1024, 30000)
        return _case("", op, 1, s, s, *heads, True, kind)
    if fam == "step":
        batch = rng.choice((1, 2, 4, 8, 16))
        return _case("", op, batch, _log(rng, 1, 64), _log(rng, 700, 131072 // batch), *heads, False, kind)
    if fam == "cross":
        return _case("", op, 1, _log(rng, 2000, 40000), _log(rng, 77, 1024), 24, 24, 128, False, kind, "wan")
    if fam == "self":
        s = _log(rng, 1500, 22000)
        return _case("", op, 1, s, s, 24, 24, 128, False, kind, "wan")
    if fam == "calibrate":
        s = _log(rng, 200, 2048)
        return _case("", "calibrate", 1, s, s, *heads, True, "efq", ntau=rng.randint(2, 5), nh=rng.randint(2, 5))
    s = _log(rng, 1000, 131072)
    return _case("", "quant", 1, s, s, *heads, False, "efq")


# ------------------------------------------------------------------ inputs
def _qkv(c, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, D, Hq, Hkv = c["batch"], c["head_dim"], c["heads_q"], c["heads_kv"]
    dev = dict(generator=g, device="cuda", dtype=torch.float32)
    q = torch.randn((B, c["seq_q"], Hq, D), **dev)
    k = torch.randn((B, c["seq_k"], Hkv, D), **dev)
    v = torch.randn((B, c["seq_k"], Hkv, D), **dev)
    if c["dist"] == "qwen":      # a magnitude of its own per head, as trained heads have
        for t, h in ((q, Hq), (k, Hkv), (v, Hkv)):
            t *= torch.rand((1, 1, h, 1), **dev) * 1.5 + 0.5
    elif c["dist"] == "wan":     # RMS-normalised Q and K, 1 % outlier K channels
        for t in (q, k):
            t /= torch.sqrt(t.square().mean(-1, keepdim=True) + 1e-6)
        n = Hkv * D
        k.view(B, c["seq_k"], n)[:, :, torch.randperm(n, generator=g, device="cuda")[: n // 100]] *= 8.0
    return tuple(t.to(torch.bfloat16) for t in (q, k, v))


def _candidates(c):
    return (np.linspace(-3.4, -2.2, c["ntau"]).astype(np.float32),
            np.linspace(1.9, 2.8, c["nh"]).astype(np.float32))


def prepare(case, seed):
    c = case
    q, k, v = _qkv(c, seed)
    s = {"c": c, "q": q, "k": k, "v": v}
    sh = binding.shape_of(q, k)
    if c["op"] in ("attn", "vhat", "lowbit"):
        s["out"] = torch.empty(q.shape, dtype=torch.float32, device="cuda")
    if c["op"] == "attn":
        n = binding.lib().efq_attn_workspace_bytes(ctypes.byref(sh))
        s["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
    elif c["op"] == "lowbit":
        s["ws"] = torch.empty(binding.lowbit_workspace_bytes(sh), dtype=torch.uint8, device="cuda")
    elif c["op"] == "vhat":
        s["vhat"] = binding.quant_v(v)
        del s["v"]
    elif c["op"] == "calibrate":
        s["taus"], s["hs"] = _candidates(c)
        s["ref"] = _softmax_attention(q, k, v, c["causal"])
    return s


def run(state):
    s, c = state, state["c"]
    op, causal, kind = c["op"], c["causal"], c["kind"]
    if op == "efq":
        return binding.efq_attn_fwd(s["q"], s["k"], s["v"], causal=causal)
    if op == "attn":
        return binding.attn_fwd(s["q"], s["k"], s["v"], causal=causal, kind=kind, out=s["out"], workspace=s["ws"])
    if op == "vhat":
        return binding.attn_fwd_vhat(s["q"], s["k"], s["vhat"], causal=causal, kind=kind, out=s["out"])
    if op == "lowbit":
        return binding.attn_fwd_lowbit(s["q"], s["k"], s["v"], causal=causal, kind=kind, out=s["out"], workspace=s["ws"])
    if op == "calibrate":
        (tau, h), rho = binding.calibrate(s["q"], s["k"], s["v"], s["ref"], s["taus"], s["hs"], causal=causal)
        return {"tau": float(tau), "h": float(h), "rho": rho}
    qhat, khat = binding.quant_qk(s["q"], s["k"])
    return {"qhat": qhat, "khat": khat, "vhat": binding.quant_v(s["v"])}


def work(case):
    c = case
    B, D, Sq, Sk, Hq, Hkv = (c[n] for n in ("batch", "head_dim", "seq_q", "seq_k", "heads_q", "heads_kv"))
    pairs = B * Hq * (Sk * (Sk + 1) // 2 if c["causal"] else Sq * Sk)
    qn, kn = B * Sq * Hq * D, B * Sk * Hkv * D
    vhat = kn * 17 / 32
    if c["op"] == "quant":
        return {"bytes": 2 * qn + 4 * kn + (qn + kn) * 33 / 32 + vhat, "flops": 0}
    if c["op"] == "calibrate":
        return {"bytes": 2 * qn + 4 * kn + 4 * qn, "flops": 4 * D * pairs * c["ntau"] * c["nh"]}
    return {"bytes": 2 * qn + 2 * kn + (vhat if c["op"] == "vhat" else 2 * kn) + 4 * qn, "flops": 4 * D * pairs}


def tolerance(case):
    """About four times what fp32 sums differ by from 64 bits over the declared
    ranges.  A score that lies within a rounding of a code's threshold takes
    the next code in one of the two, which moves its row: 6e-4 in the 2-norm
    with bf16 Q K^T, 6e-3 with MXFP8, whose products the matrix core sums with
    fewer bits; where a row sees few keys, by up to its own size."""
    if case["op"] == "quant":
        return "exact"
    if case["op"] == "calibrate":
        return {"rel": 1e-5, "max": 2e-5}
    return {"rel": 2e-2 if case["op"] == "lowbit" else 2.5e-3, "max": 0.99}


# ------------------------------------------------------------- 64-bit values
def _softmax_attention(q, k, v, causal):
    """Plain softmax attention in fp32 (the reference output of a calibration)."""
    B, Sq, Hq, D = q.shape
    G = Hq // k.shape[2]
    out = torch.empty(q.shape, dtype=torch.float32, device=q.device)
    for b in range(B):
        for h in range(Hq):
            kt = k[b, :, h // G].float().t().contiguous()
            s = (q[b, :, h].float() @ kt) * D ** -0.5
            if causal:
                s.masked_fill_(torch.ones_like(s, dtype=torch.bool).triu(1), -math.inf)
            out[b, :, h] = torch.softmax(s, -1) @ v[b, :, h // G].float()
    return out


def _e2m1(x):
    """Nearest E2M1 code of x >= 0, ties to the even code, saturating at 6."""
    c = torch.zeros_like(x)
    for i, t in enumerate((0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0)):
        c += (x >= t if i % 2 else x > t).to(c.dtype)
    return c.long()


def _floor_log2(x):
    return torch.frexp(x)[1].to(torch.float64) - 1


def _mx(x, axis, emax, rounded):
    """x (64 bits) through the OCP microscaling rule in blocks of 32 along `axis`."""
    x = x.movedim(axis, -1)
    n = x.shape[-1]
    x = torch.nn.functional.pad(x, (0, -n % 32)).unflatten(-1, (-1, 32))
    amax = x.abs().amax(-1, keepdim=True)
    k = torch.where(amax > 0, _floor_log2(amax) - emax, torch.full_like(amax, -127.0)).clamp_min(-127)
    y = torch.sign(x) * rounded(x.abs() * torch.exp2(-k)) * torch.exp2(k)
    return y.flatten(-2)[..., :n].movedim(-1, axis)


def _e2m1_value(x):
    return torch.tensor(E2M1, dtype=torch.float64, device=x.device)[_e2m1(x)]


def _e4m3_value(x):
    x = x.clamp_max(448.0)
    step = torch.exp2(_floor_log2(x.clamp_min(2.0 ** -6)) - 3)
    return torch.round(x / step) * step


def _probabilities(x, kind, params):
    """Values of the quantised probability operand; x: shifted scores [..., n, 32]."""
    val = torch.tensor(E2M1, dtype=torch.float64, device=x.device)
    mb = x.amax(-1, keepdim=True)
    if kind in ("expq", "expq6"):
        p, amax = torch.exp(x), torch.exp(mb)
        e = _floor_log2(amax.clamp_min(1e-300))
        k = e - 2
        if kind == "expq6":
            k = k + (amax > 1.5 * torch.exp2(e)).to(k.dtype)
        k = k.clamp_min(-126)
        return val[_e2m1(p * torch.exp2(-k))] * torch.exp2(k)
    tau, h = (float(np.float32(t)) for t in params)
    k = torch.floor((mb + math.log(2 / 9)) / LN2).clamp_min(-127)
    u = (x - k * LN2 - math.log(6) - tau) * h
    if kind == "lut":
        c = torch.tensor(C16, device=x.device)[(torch.floor(u) + 1).clamp(0, 15).long()]
    else:
        c = (torch.floor(u) + 1).clamp(0, 7).long()
    return val[c] * torch.exp2(k)


def _attention(q, k, v, causal, kind, params, lowbit):
    B, Sq, Hq, D = q.shape
    Sk, Hkv = k.shape[1], k.shape[2]
    G, scale = Hq // Hkv, float(np.float32(D ** -0.5))
    out = torch.empty((B, Sq, Hq, D), dtype=torch.float64, device=q.device)
    pad = -Sk % 64
    for b in range(B):
        for g in range(Hkv):
            kk = k[b, :, g].double()
            if lowbit:
                kk = _mx(kk, -1, 8, _e4m3_value)
            vv = torch.nn.functional.pad(_mx(v[b, :, g].double(), 0, 2, _e2m1_value), (0, 0, 0, pad))
            kt = torch.nn.functional.pad(kk, (0, 0, 0, pad)).t().contiguous()
            for h in range(g * G, g * G + G):
                qq = q[b, :, h].double()
                if lowbit:
                    qq = _mx(qq, -1, 8, _e4m3_value)
                step = max(1, (1 << 27) // (Sk + pad))
                for i in range(0, Sq, step):
                    r = torch.arange(i, min(Sq, i + step), device=q.device)
                    n = min(Sk + pad, -64 * (-min(Sk, int(r[-1]) + 1) // 64)) if causal else Sk + pad
                    s = (qq[i: i + step] @ kt[:, :n]) * scale
                    t = torch.arange(n, device=q.device)
                    hidden = (t >= Sk)[None] if not causal else (t[None] > r[:, None]) | (t >= Sk)[None]
                    s.masked_fill_(hidden, -math.inf)
                    m = s.view(len(r), -1, 64).amax(-1).cummax(-1).values          # running maximum per tile
                    x = (s.view(len(r), -1, 64) - m[..., None]).view(len(r), -1, 32)
                    p = _probabilities(x, kind, params)
                    w = torch.exp(m - m[:, -1:]).repeat_interleave(2, -1)[..., None]  # the later rescalings
                    p = (p * w).view(len(r), n)
                    out[b, i: i + step, h] = (p @ vv[:n]) / p.sum(-1, keepdim=True)
    return out


def exact(case, seed):
    c = case
    if c["op"] == "quant":
        return None
    pairs = c["batch"] * c["heads_q"] * c["seq_q"] * c["seq_k"] * c.get("ntau", 1) * c.get("nh", 1)
    if pairs > 4e10:
        return None
    q, k, v = _qkv(c, seed)
    if c["op"] != "calibrate":
        return _attention(q, k, v, c["causal"], c["kind"], PARAMS.get(c["kind"]), c["op"] == "lowbit")
    taus, hs = _candidates(c)
    ref = _softmax_attention(q, k, v, c["causal"]).double()
    rho = np.zeros((len(taus), len(hs)))
    for i, tau in enumerate(taus):
        for j, h in enumerate(hs):
            o = _attention(q, k, v, c["causal"], "efq", (tau, h), False)
            rho[i, j] = float((o - ref).norm() / ref.norm())
    i, j = np.unravel_index(int(rho.argmin()), rho.shape)
    return {"tau": float(taus[i]), "h": float(hs[j]), "rho": rho}
