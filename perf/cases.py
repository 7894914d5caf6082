"""The work that programs have this library do, as cases to time.

A case is one call that a serving program makes for each layer and step: a
decode of the whole cache, a fused append + decode step, a step of several
positions (speculative verification, a chunk of a prompt), or the writing of a
prompt's rows into the cache.  Everything is float32, the library's only data
type; lengths are ragged unless the workload says otherwise.

Keys of a case: ``op`` (decode, noalloc, step, multi, multi_step, append_rows),
``B`` sequences, ``h_q`` / ``h_kv`` query / KV heads, ``d_k`` / ``d_v`` head
sizes, ``n_max`` cache capacity, ``len_lo`` / ``len_hi`` bounds of the lengths
on entry, ``T`` positions that the call submits.
"""
import math
import random
import struct

import torch

from paper_2607_19456_amd import binding


def _case(name, op, B, h_q, h_kv, d_k, d_v, n_max, len_lo, len_hi, T=1):
    c = dict(op=op, B=B, h_q=h_q, h_kv=h_kv, d_k=d_k, d_v=d_v, n_max=n_max,
             len_lo=len_lo, len_hi=len_hi, T=T)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call: one head, one short cache; launch and latency.
        _case("mha1_d64_n128", "decode", 1, 1, 1, 64, 64, 128, 128, 128),
        # One user's decode step: a single sequence of ordinary length.
        _case("gqa32x8_b1_step", "step", 1, 32, 8, 128, 128, 4096, 2900, 2900),
        # A serving batch of ordinary, ragged lengths.
        _case("gqa32x8_b16_ragged_step", "step", 16, 32, 8, 128, 128, 4096, 200, 4000),
        # The MHA workload: 8 sequences of 4096 rows, one step.
        _case("mha32_b8_n4096_step", "step", 8, 32, 32, 128, 128, 4112, 4096, 4096),
        # The GQA workload: group 4, 16 sequences of 8192 rows.
        _case("gqa32x8_b16_n8192", "decode", 16, 32, 8, 128, 128, 8192, 8192, 8192),
        # The MQA workload: 32 query heads on one KV head.
        _case("mqa32_b32_n16384", "decode", 32, 32, 1, 128, 128, 16384, 16384, 16384),
        # The benchmark's workload: long ragged contexts, the largest caches.
        _case("gqa64x8_b4_long_step", "step", 4, 64, 8, 128, 128, 131072, 65536, 131008),
        # The same caches, four draft tokens verified in one step.
        _case("gqa64x8_b4_long_spec4", "multi_step", 4, 64, 8, 128, 128, 131072, 65536,
              131008, 4),
        # Wide heads, odd lengths.
        _case("gqa32x4_d256_b4_odd", "decode", 4, 32, 4, 256, 256, 16381, 9001, 16379),
        # A chunk of 512 prompt positions behind what is cached already.
        _case("gqa32x8_b2_chunk512", "multi_step", 2, 32, 8, 128, 128, 8192, 1000, 7600, 512),
        # A prompt's first chunk: an empty cache, fully causal, an odd size.
        _case("mha16_d64_prompt1500", "multi_step", 1, 16, 16, 64, 64, 2048, 0, 0, 1500),
        # A prompt's rows computed elsewhere, written into the caches.
        _case("append_b8_h8_rows700", "append_rows", 8, 32, 8, 128, 128, 8192, 0, 7000, 700),
    ]


# What a drawn case may cost: below the largest listed ones.
_MAX_KV_BYTES = 2 << 30
_MAX_FLOPS = 40e9
_MAX_ROWS_BYTES = 384 << 20


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        op = rng.choice(["decode", "decode", "decode", "noalloc", "step", "step", "step", "step",
                         "multi_step", "multi_step", "multi_step", "multi", "append_rows"])
        h_kv = rng.choice([1, 2, 4, 8, 8, 16, 32])
        h_q = h_kv * rng.choice([1, 2, 4, 4, 5, 8, 8, 16, 32])
        if h_q > 128:
            continue
        d_k = rng.choice([64, 128, 128, 128, 256])
        d_v = d_k if rng.random() < 0.8 else rng.choice([64, 128, 256])
        B = _log(rng, 1, 256)
        n_max = _log(rng, 64, 131072)
        T = 1
        if op in ("multi_step", "multi", "append_rows"):
            # drafts of a few tokens, or chunks of a prompt
            T = rng.randint(2, 8) if rng.random() < 0.5 else _log(rng, 16, 2048)
        if T >= n_max:
            continue
        hi = n_max - T
        lo = hi if rng.random() < 0.25 else rng.randint(0, hi)
        if op == "multi":
            lo, hi = max(lo, T), max(hi, T)
        c = _case("", op, B, h_q, h_kv, d_k, d_v, n_max, lo, hi, T)
        kv = 4 * B * h_kv * n_max * (d_k + d_v)
        rows = 4 * B * T * (h_kv + h_q) * (d_k + d_v)
        if kv > _MAX_KV_BYTES or rows > _MAX_ROWS_BYTES or work(c)["flops"] > _MAX_FLOPS:
            continue
        if op != "append_rows":
            ws = binding.workspace_bytes(B, h_q * T, h_kv, n_max, d_k, d_v)
            if ws == 0 or ws > (8 << 30):
                continue
            if op == "noalloc" and ws > binding.NOALLOC_MAX_WORKSPACE_BYTES:
                continue
        return c


def _lens(c):
    """The lengths on entry: part of the case, the same for every seed."""
    r = random.Random(c["B"] * 1000003 + c["len_lo"] * 101 + c["len_hi"])
    return [r.randint(c["len_lo"], c["len_hi"]) for _ in range(c["B"])]


def _scale(c):
    return struct.unpack("f", struct.pack("f", 1.0 / math.sqrt(c["d_k"])))[0]


def _fuses(c):
    return c["op"] in ("step", "multi_step")


def _inputs(c, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)

    B, T = c["B"], c["T"]
    rows = (T,) if c["op"] in ("multi", "multi_step", "append_rows") else ()
    s = {"K": normal(B, c["h_kv"], c["n_max"], c["d_k"]),
         "V": normal(B, c["h_kv"], c["n_max"], c["d_v"])}
    if c["op"] != "append_rows":
        s["q"] = normal(B, c["h_q"], *rows, c["d_k"])
    if _fuses(c) or c["op"] == "append_rows":
        s["k_new"] = normal(B, c["h_kv"], *rows, c["d_k"])
        s["v_new"] = normal(B, c["h_kv"], *rows, c["d_v"])
    # The scheduler's lengths, and the tensor that the library reads (and advances).
    s["start"] = torch.tensor(_lens(c), dtype=torch.int32, device="cuda")
    s["lens"] = s["start"].clone()
    return s


def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    s["op"], s["scale"] = c["op"], _scale(c)
    if c["op"] == "append_rows":
        return s
    shape = (c["B"], c["h_q"]) + ((c["T"],) if s["q"].dim() == 4 else ()) + (c["d_v"],)
    s["out"] = torch.empty(shape, dtype=torch.float32, device="cuda")
    if s["q"].dim() == 4:
        s["ws"] = binding.alloc_multi_workspace(s["q"], s["K"], s["V"])
    elif c["op"] != "noalloc":
        s["ws"] = binding.alloc_workspace(s["q"], s["K"], s["V"])
    return s


def run(state):
    """One call.  A call that appends is first given the scheduler's lengths,
    as a serving loop does before each step."""
    s, op = state, state["op"]
    if op == "decode":
        return binding.decode_attn(s["q"], s["K"], s["V"], s["lens"], s["scale"], s["out"],
                                   s["ws"])
    if op == "noalloc":
        return binding.decode_attn_noalloc(s["q"], s["K"], s["V"], s["lens"], s["scale"],
                                           s["out"])
    if op == "multi":
        return binding.decode_multi(s["q"], s["K"], s["V"], s["lens"], s["scale"], s["out"],
                                    s["ws"])
    s["lens"].copy_(s["start"])
    if op == "append_rows":
        binding.kv_append_rows(s["K"], s["V"], s["k_new"], s["v_new"], s["lens"])
        return s["K"], s["V"], s["lens"]
    step = binding.decode_step if op == "step" else binding.decode_multi_step
    out = step(s["q"], s["K"], s["V"], s["k_new"], s["v_new"], s["lens"], s["scale"], s["out"],
               s["ws"])
    return out, s["K"], s["V"], s["lens"]


def _visible(c, n):
    """(query row, key) pairs of one head of a sequence with n rows on entry."""
    T = c["T"]
    first = n + 1 if _fuses(c) else n - T + 1       # keys that row 0 sees
    return T * first + T * (T - 1) // 2


def work(case):
    c = case
    B, T, row = c["B"], c["T"], 4 * (c["d_k"] + c["d_v"])
    lens = _lens(c)
    new = 2 * B * c["h_kv"] * T * row               # rows read and written
    if c["op"] == "append_rows":
        return {"bytes": new, "flops": 0}
    pairs = sum(_visible(c, n) for n in lens)
    return {"bytes": c["h_kv"] * sum(lens) * row + B * c["h_q"] * T * row
                     + (new if _fuses(c) else 0),
            "flops": 2 * (c["d_k"] + c["d_v"]) * c["h_q"] * pairs}


def tolerance(case):
    if case["op"] == "append_rows":
        return "exact"
    # 32-bit products, sums and exponentials: measured 1.8e-7 to 1.0e-6 (rel)
    # against 64 bits; the same sums in another order (the dynamic schedule
    # varies it from call to call) differ by 7e-7 (rel) and 3.7e-6 (max).
    return {"rel": 5e-6, "max": 3e-5}


def exact(case, seed):
    c = case
    s = _inputs(c, seed)
    B, T, G = c["B"], c["T"], c["h_q"] // c["h_kv"]
    lens = _lens(c)
    K, V = s["K"].double(), s["V"].double()
    after = list(lens)
    if "k_new" in s:
        kn = s["k_new"].reshape(B, c["h_kv"], T, -1).double()
        vn = s["v_new"].reshape(B, c["h_kv"], T, -1).double()
        for b, n in enumerate(lens):
            K[b, :, n:n + T] = kn[b]
            V[b, :, n:n + T] = vn[b]
            after[b] = n + T
    end = torch.tensor(after, dtype=torch.int32, device="cuda")
    if c["op"] == "append_rows":
        return K, V, end
    q = s["q"].reshape(B, c["h_kv"], G * T, c["d_k"]).double() * _scale(c)
    out = torch.zeros(B, c["h_kv"], G * T, c["d_v"], dtype=torch.float64, device="cuda")
    for b, n in enumerate(after):
        if n == 0:
            continue
        last = torch.arange(n - T, n, device="cuda").repeat(G)[:, None]
        hidden = torch.arange(n, device="cuda")[None, :] > last
        for g in range(c["h_kv"]):
            score = q[b, g] @ K[b, g, :n].t()
            score.masked_fill_(hidden, -math.inf)
            out[b, g] = torch.softmax(score, 1) @ V[b, g, :n]
    out = out.reshape(B, c["h_q"], *((T,) if s["q"].dim() == 4 else ()), c["d_v"])
    return (out, K, V, end) if _fuses(c) else out
