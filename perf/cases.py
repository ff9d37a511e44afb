"""The work a program asks of this library, as timed cases: attention forwards (prefill) and decode steps over a
key/value cache, in both operand types, from calls that are bound by their launch to the largest workloads.

``listed()`` names the cases, ``draw()`` gives more of the same ranges, ``prepare()`` makes what a program holds before
the call, ``run()`` is one call through the public entry points, ``exact()`` the same result in float64 with plain torch.
"""
import math

import numpy as np
import torch

import paper_2609_33586_amd as attn

LOG2E = 1.4426950408889634
TILE = 128  # keys between two moves of the running maximum
MODES = {"exact": attn.ATTN_EXP_EXACT, "h15": attn.ATTN_EXP_H15, "sq4": attn.ATTN_EXP_SQ4, "sq8": attn.ATTN_EXP_SQ8,
         "pot": attn.ATTN_EXP_ROWMAX_POT}
ORDER = {"h15": 1, "sq4": 2, "sq8": 3}  # S(Q_{2^-k}): k


def _fwd(name, dtype, b, hq, hkv, s, d, causal, mode, sharp, tau=0.0, tau_per_wave=False):
    return {"name": name, "kind": "fwd", "dtype": dtype, "B": b, "Hq": hq, "Hkv": hkv, "S": s, "d": d, "causal": causal,
            "mode": mode, "sharp": sharp, "tau": tau, "tau_per_wave": tau_per_wave}


def _dec(name, dtype, b, hq, hkv, sq, sk, cap, d, mode, sharp, noalloc=False):
    return {"name": name, "kind": "decode", "dtype": dtype, "B": b, "Hq": hq, "Hkv": hkv, "Sq": sq, "Sk": sk, "cap": cap,
            "d": d, "causal": True, "mode": mode, "sharp": sharp, "noalloc": noalloc}


def listed():
    return [
        # the smallest forward: a short sequence of a small model, bound by the call and the launch
        _fwd("fwd_bf16_b1h2_s256_d64", "bf16", 1, 2, 2, 256, 64, False, "h15", False),
        # the prefill of one short prompt of an odd length
        _fwd("fwd_fp8_b1h32kv8_s777", "fp8", 1, 32, 8, 777, 128, True, "h15", True),
        # one sequence of 16 heads, the shape of the paper's timing matrix, with the hardware exponential
        _fwd("fwd_bf16_b1h16_s4096", "bf16", 1, 16, 16, 4096, 128, True, "exact", False),
        # a batch of medium prompts with grouped heads
        _fwd("fwd_bf16_b4h32kv8_s2048", "bf16", 4, 32, 8, 2048, 128, True, "h15", True),
        # ragged rows at head dimension 64, a batch that is no power of two
        _fwd("fwd_fp8_b3h24kv8_s3001_d64", "fp8", 3, 24, 8, 3001, 64, True, "h15", False),
        # the headline: FP8 causal at 8K with grouped heads
        _fwd("fwd_fp8_b2h32kv8_s8192", "fp8", 2, 32, 8, 8192, 128, True, "h15", True),
        # an encoder's pass: every key visible, the hardware exponential
        _fwd("fwd_fp8_b2h16_s8192_full", "fp8", 2, 16, 16, 8192, 128, False, "exact", False),
        # the largest: a 16K prompt with 64 query heads
        _fwd("fwd_bf16_b1h64kv8_s16384", "bf16", 1, 64, 8, 16384, 128, True, "h15", True),
        # the smallest decode: one sequence, a short cache of an odd length, no allocation (as under graph capture)
        _dec("dec_bf16_b1h32kv8_sk1000", "bf16", 1, 32, 8, 1, 1000, 1024, 128, "h15", True, noalloc=True),
        # one sequence with a long cache: few heads, many key parts
        _dec("dec_bf16_b1h32kv8_sk32768", "bf16", 1, 32, 8, 1, 32768, 32768, 128, "exact", False),
        # a serving batch with an 8K cache
        _dec("dec_fp8_b16h32kv8_sk8192", "fp8", 16, 32, 8, 1, 8192, 8192, 128, "h15", True),
        # four new tokens at once (speculative decoding) against caches that are not full
        _dec("dec_fp8_b4h32kv8_sq4_sk15000", "fp8", 4, 32, 8, 4, 15000, 16384, 128, "h15", True),
    ]


#: the largest listed case: no drawn one asks for more
_MOST_FLOPS = 4.0 * 64 * 16384 ** 2 * 128 / 2
_MOST_BYTES = 1 << 30


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        dtype = rng.choice(["bf16", "fp8"])
        d = rng.choice([64, 128, 128])
        hkv, g = rng.choice([1, 2, 3, 4, 8, 8, 16]), rng.choice([1, 2, 4, 4, 8])
        mode = rng.choice(["h15"] * 5 + ["exact"] * 4 + ["sq4", "sq8"])
        sharp = rng.random() < 0.5
        if rng.random() < 0.6:
            s = _log_int(rng, 64, 16384)
            if rng.random() < 0.5:
                s = max(128, s // 128 * 128)
            tau, per_wave = 0.0, False
            if dtype == "bf16" and rng.random() < 0.15:
                if rng.random() < 0.5:
                    mode = "pot"
                else:
                    tau, per_wave = 8.0, rng.random() < 0.5
            c = _fwd("", dtype, _log_int(rng, 1, 16), hkv * g, hkv, s, d, rng.random() < 0.7, mode, sharp, tau, per_wave)
            fits = work(c)["flops"] * (2 if dtype == "bf16" else 1) <= 2 * _MOST_FLOPS and work(c)["bytes"] <= _MOST_BYTES
        else:
            sk = _log_int(rng, 128, 65536)
            cap = sk if rng.random() < 0.5 else sk + rng.randrange(1, 2048)
            sq = min(rng.choice([1, 1, 1, 2, 4, 7, 16]), sk)
            c = _dec("", dtype, _log_int(rng, 1, 64), hkv * g, hkv, sq, sk, cap, d, mode, sharp, rng.random() < 0.3)
            fits = work(c)["bytes"] <= _MOST_BYTES
            if c["noalloc"] and attn.attn_decode_workspace_bytes(c["B"], c["Hq"], sq, sk, d, _cut(c)) > 1 << 24:
                c["noalloc"] = False  # more partial results than the built-in workspace holds
        if fits:
            del c["name"]
            return c


def _cut(c):
    """The documented cut of the keys: about 512 workgroups, at least eight tiles of keys in a part."""
    groups = c["B"] * c["Hkv"] * ((c["Hq"] // c["Hkv"] * c["Sq"] + 31) // 32)
    tiles = (c["Sk"] + TILE - 1) // TILE
    parts = min((512 + groups - 1) // groups, tiles // 8)
    return 0 if parts <= 1 else (tiles + parts - 1) // parts * TILE


def _scale(c):
    return float(np.float32(1.0 / math.sqrt(c["d"])))


def _operands(c, seed):
    """q, k, v on the GPU in the operand type, and the descales.  Standard normals; "sharp": 2% of the keys of each
    head are four times as large.  FP8: one scale per tensor, amax / 448."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    sq, sk = (c["S"], c["S"]) if c["kind"] == "fwd" else (c["Sq"], c["cap"])
    x = [torch.randn(c["B"], h, s, c["d"], generator=gen, device="cuda")
         for h, s in ((c["Hq"], sq), (c["Hkv"], sk), (c["Hkv"], sk))]
    if c["sharp"]:
        n = int(round(0.02 * sk))
        at = torch.rand(c["B"], c["Hkv"], sk, generator=gen, device="cuda").argsort(dim=-1)[..., :n]
        x[1].scatter_(2, at.unsqueeze(-1).expand(-1, -1, -1, c["d"]),
                      4 * x[1].gather(2, at.unsqueeze(-1).expand(-1, -1, -1, c["d"])))
    if c["dtype"] == "bf16":
        return [t.to(torch.bfloat16) for t in x], None
    s = [torch.linalg.vector_norm(t, ord=math.inf) / 448.0 for t in x]
    return [(t / u).to(torch.float8_e4m3fn) for t, u in zip(x, s)], tuple(float(u) for u in s)


def prepare(case, seed):
    c = case
    (q, k, v), descale = _operands(c, seed)
    st = {"case": c, "q": q, "k": k, "v": v, "descale": descale, "scale": _scale(c), "mode": MODES[c["mode"]]}
    if c["kind"] == "decode":
        # a decode loop keeps its cut, its outputs and its workspace from step to step
        st["cut"] = attn.attn_decode_split_keys(c["B"], c["Hq"], c["Hkv"], c["Sq"], c["Sk"], c["d"],
                                                attn.ATTN_BF16 if c["dtype"] == "bf16" else attn.ATTN_FP8_E4M3)
        st["out"] = torch.empty(c["B"], c["Hq"], c["Sq"], c["d"], dtype=torch.bfloat16, device="cuda")
        st["lse"] = torch.empty(c["B"], c["Hq"], c["Sq"], dtype=torch.float32, device="cuda")
        st["ws"] = None
        n = attn.attn_decode_workspace_bytes(c["B"], c["Hq"], c["Sq"], c["Sk"], c["d"], st["cut"])
        if n and not c["noalloc"]:
            st["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
    return st


def run(state):
    st, c = state, state["case"]
    if c["kind"] == "fwd":
        o, lse = attn.attn_fwd_ex(st["q"], st["k"], st["v"], causal=c["causal"], scale=st["scale"], exp_mode=st["mode"],
                                  descale=st["descale"], tau=c["tau"], tau_per_wave=c["tau_per_wave"])
    elif c["noalloc"]:
        o, lse = attn.attn_decode_noalloc(st["q"], st["k"], st["v"], causal=True, scale=st["scale"], exp_mode=st["mode"],
                                          split_keys=st["cut"], Sk=c["Sk"], descale=st["descale"], out=st["out"],
                                          lse=st["lse"])
    else:
        o, lse = attn.attn_decode(st["q"], st["k"], st["v"], causal=True, scale=st["scale"], exp_mode=st["mode"],
                                  split_keys=st["cut"], Sk=c["Sk"], descale=st["descale"], out=st["out"], lse=st["lse"],
                                  workspace=st["ws"])
    return {"o": o, "lse": lse}


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 1
    if c["kind"] == "fwd":
        scores = c["B"] * c["Hq"] * float(c["S"]) ** 2 * (0.5 if c["causal"] else 1.0)
        rows, kv = c["B"] * c["Hq"] * c["S"], c["B"] * c["Hkv"] * c["S"]
    else:
        scores = c["B"] * c["Hq"] * float(c["Sq"]) * c["Sk"]
        rows, kv = c["B"] * c["Hq"] * c["Sq"], c["B"] * c["Hkv"] * c["Sk"]
    return {"bytes": rows * (c["d"] * (e + 2) + 4) + 2.0 * kv * c["d"] * e, "flops": 4.0 * scores * c["d"]}


def tolerance(case):
    # A weight on a lattice moves by a third or a half when a logit crosses a rounding boundary.  BF16 logits agree
    # to about 1e-6 between orders of summation; the FP8 matrix core's accumulate to about 2^-13 of sum |q k|.
    # BF16: O is rounded to 8 bits.
    return {"rel": 0.01 if case["dtype"] == "bf16" else 0.03}


def exact(case, seed):
    c = case
    (q, k, v), descale = _operands(c, seed)
    qd, kd, vd = descale or (1.0, 1.0, 1.0)
    c1 = _scale(c) * qd * kd * LOG2E
    dec = c["kind"] == "decode"
    sq, sk = (c["Sq"], c["Sk"]) if dec else (c["S"], c["S"])
    g = c["Hq"] // c["Hkv"]
    cut = (_cut(c) or sk) if dec else sk
    out = torch.empty(c["B"], c["Hq"], sq, c["d"], dtype=torch.float64, device="cuda")
    lse = torch.empty(c["B"], c["Hq"], sq, dtype=torch.float64, device="cuda")
    step = max(32, (1 << 25) // sk // 32 * 32)
    for b in range(c["B"]):
        for h in range(c["Hkv"]):
            kh, vh = k[b, h, :sk].double(), v[b, h, :sk].double()
            for r0 in range(0, sq, step):
                rows = torch.arange(r0, min(r0 + step, sq), device="cuda")
                qh = q[b, h * g:(h + 1) * g, r0:r0 + step].double()
                see = (rows + (sk - sq)) if c["causal"] else torch.full_like(rows, sk - 1)
                for i in range(g):  # one head at a time: the scores are the large array here
                    o, e = _rows(c, qh[i], kh, vh, see, c1, cut)
                    out[b, h * g + i, r0:r0 + step] = o * vd
                    lse[b, h * g + i, r0:r0 + step] = e
    return {"o": out, "lse": lse}


def _rows(c, q, k, v, see, c1, cut):
    """O (without the V descale) and LSE of some query rows of one head; see: each row's last visible key."""
    sk = k.shape[0]
    ms, ls, os = [], [], []
    for j0 in range(0, sk, cut):
        j1 = min(j0 + cut, sk)
        m, l, o = _part(c, q, k[j0:j1], v[j0:j1], see - j0, c1)
        ms.append(m), ls.append(l), os.append(o)
    m = torch.stack(ms).amax(0)
    f = [torch.exp2(c1 * (x - m)) for x in ms]  # 0 for a part that sees no key
    l = sum(x * y for x, y in zip(f, ls))
    o = sum(x.unsqueeze(-1) * y for x, y in zip(f, os)) / l.unsqueeze(-1)
    return o, (m * c1 + torch.log2(l)) * math.log(2.0)


def _part(c, q, k, v, see, c1):
    n, nk = q.shape[0], k.shape[0]
    nt = (nk + TILE - 1) // TILE
    s = q @ k.T
    s.masked_fill_(torch.arange(nk, device=s.device) > see.unsqueeze(-1), -math.inf)
    if nk < nt * TILE:
        s = torch.nn.functional.pad(s, (0, nt * TILE - nk), value=-math.inf)
    s = s.view(n, nt, TILE)
    mt = s.amax(-1)
    if c["mode"] in ("exact", "pot"):
        a = mt.amax(-1, keepdim=True).expand(n, nt)
    elif c.get("tau", 0.0) > 0.0:
        a = _anchors(mt, c1, c["tau"], c["tau_per_wave"])
    else:
        a = mt.cummax(-1).values
    x = (s - a.masked_fill(a == -math.inf, 0.0).unsqueeze(-1)).mul_(c1)  # base-two exponents, -inf where masked
    if c["mode"] == "exact":
        w = torch.exp2(x)
    elif c["mode"] == "pot":
        w = torch.exp2(-torch.floor(0.5 - x).clamp_(max=20.0)).masked_fill_(x == -math.inf, 0.0)
    else:
        f = float(1 << ORDER[c["mode"]])
        n2 = torch.round(x * f).clamp_(min=-126.0 * f) / f  # halves to even
        e = torch.floor(n2)
        w = ((n2 - e + 1.0) * torch.exp2(e)).masked_fill_(x == -math.inf, 0.0)
    m = a[:, -1]
    w *= torch.exp2(c1 * (a - m.unsqueeze(-1))).nan_to_num_(0.0).unsqueeze(-1)
    w = w.view(n, nt * TILE)[:, :nk]
    return m, w.sum(-1), w @ v


def _anchors(mt, c1, tau, per_wave):
    """The anchor of each tile under a conditional rescale: it moves when the maximum grows by more than tau octaves."""
    n, nt = mt.shape
    m, got = mt[:, 0].clone(), [mt[:, 0]]
    for t in range(1, nt):
        move = (mt[:, t] - m) * c1 > tau
        if per_wave:
            w = torch.nn.functional.pad(move, (0, -n % 32)).view(-1, 32).any(-1)
            move = w.repeat_interleave(32)[:n]
        m = torch.where(move, torch.maximum(m, mt[:, t]), m)
        got.append(m)
    return torch.stack(got, -1)
