"""The work that a user of this library has it do, as cases to be timed and compared.

Every case goes through the public functions of the Python package: windowed prefill
(whole prompts, chunks and short turns against long caches, pre-rotated and unrotated
caches), decode (uniform, ragged, paged, unrotated), the cache appends, and one serving
step (append, then decode).  Head shapes, RoPE bases and window settings are those of the
benchmark workloads and of the tests; token counts run from a short prompt to a context of
2^20 keys, odd ones among them.
"""
from __future__ import annotations

import math

import torch

import paper_2608_02947_amd as atf

# head shapes (query heads, KV heads, head dim, RoPE base, llama3 frequency scaling)
SHAPES = {
    "qwen05b": (14, 2, 64, 1e6, False),
    "llama3b": (24, 8, 128, 5e5, True),
    "qwen7b1m": (28, 4, 128, 1e7, False),
    "mha64": (16, 16, 64, 1e4, False),    # no sharing of KV heads
    "gqa8": (32, 4, 128, 1e6, False),     # a group of 8
}

# the largest drawn case: no dearer than the 4096-row chunk at 2^20 keys below
MAX_FLOPS = 3.0e13
MAX_CACHE_BYTES = 2.2e9


def listed():
    return [
        # one token against a short prompt's cache: latency and launches
        dict(name="decode_1k", op="decode", shape="qwen05b", batch=1, n_q=1, n_k=1000,
             window="exact"),
        # one serving step of a batch at the same length: the new token's key is rotated and
        # appended with its value, then every row decodes over its cache
        dict(name="step_b8_8k", op="step", shape="llama3b", batch=8, n_q=1, n_k=8200,
             window="exact"),
        # decode at the longest context served
        dict(name="decode_1m", op="decode", shape="qwen7b1m", batch=1, n_q=1, n_k=1048576,
             window="exact"),
        # a serving batch of requests of different lengths over paged caches, with the
        # window rounded to whole matrix steps
        dict(name="decode_paged_b24", op="decode_paged", shape="llama3b", batch=24, n_q=1,
             n_k=30011, window="rounded", page_tokens=64),
        # a position-free cache shared by requests: keys rotated as they are read
        dict(name="decode_unrotated_100k", op="decode_unrotated", shape="qwen7b1m", batch=2,
             n_q=1, n_k=100003, window="exact"),
        # a short prompt of a small model
        dict(name="prefill_1k_d64", op="prefill", shape="qwen05b", batch=1, n_q=1024, n_k=1024,
             window="exact"),
        # a long prompt of a small model, not a multiple of any tile
        dict(name="prefill_8k_d64", op="prefill", shape="qwen05b", batch=1, n_q=8191, n_k=8191,
             window="exact"),
        # a whole long prompt, with the variable-k profile of the window family
        dict(name="prefill_32k", op="prefill", shape="llama3b", batch=1, n_q=32768, n_k=32768,
             window="variable"),
        # a chunk of a chunked prefill at the end of a 2^20-token context
        dict(name="prefill_chunk_1m", op="prefill", shape="qwen7b1m", batch=1, n_q=4096,
             n_k=1048576, window="exact"),
        # an appended turn of a long session: a few hundred new rows against the session's cache
        dict(name="prefill_turn_64k", op="prefill", shape="qwen7b1m", batch=1, n_q=300,
             n_k=65836, window="exact"),
        # a chunk over an unrotated cache, RoPE applied as it is read
        dict(name="prefill_unrotated_16k", op="prefill_unrotated", shape="llama3b", batch=1,
             n_q=2048, n_k=16384, window="exact"),
        # a prefill chunk's keys and values entering the caches, keys rotated on the way
        dict(name="append_16k", op="append_rotated", shape="llama3b", batch=1, n_q=16384,
             n_k=40000, window="exact"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["decode", "decode", "step", "decode_paged", "decode_ragged",
                     "decode_unrotated", "prefill", "prefill", "prefill", "turn", "turn",
                     "prefill_unrotated", "append", "append_rotated"])
    shape = rng.choice(["qwen05b", "llama3b", "llama3b", "qwen7b1m", "qwen7b1m", "mha64", "gqa8"])
    window = rng.choice(["exact", "exact", "exact", "rounded", "variable", "off"])
    c = dict(op=op, shape=shape, batch=1, n_q=1, n_k=1, window=window)
    if op in ("decode", "decode_unrotated", "step"):
        c["batch"] = rng.choice([1, 1, 2, 3, 8, 16])
        c["n_k"] = _log_int(rng, 500, 300000)
    elif op in ("decode_paged", "decode_ragged"):
        c["batch"] = rng.randint(3, 40)
        c["n_k"] = _log_int(rng, 2000, 60000)
        if op == "decode_paged":
            c["page_tokens"] = rng.choice([32, 64, 128, 256])
    elif op in ("append", "append_rotated"):
        c["batch"] = rng.choice([1, 1, 2, 4])
        c["n_q"] = _log_int(rng, 16, 32768)
        c["n_k"] = c["n_q"] + _log_int(rng, 16, 32768)
    elif op == "turn":
        c["op"] = rng.choice(["prefill", "prefill", "prefill_unrotated"])
        c["batch"] = rng.choice([1, 1, 1, 4])
        c["n_q"] = _log_int(rng, 16, 1024)
        c["n_k"] = c["n_q"] + _log_int(rng, 2000, 200000)
    else:
        c["n_q"] = _log_int(rng, 200, 32768)
        c["n_k"] = c["n_q"] + rng.choice([0, 0, _log_int(rng, 100, 100000)])
    while _cache_bytes(c) > MAX_CACHE_BYTES:
        c["n_k"] = max(c["n_q"], c["n_k"] * 2 // 3)
        if c["n_k"] == c["n_q"]:
            c["batch"] = max(1, c["batch"] // 2)
    while work(c)["flops"] > MAX_FLOPS:
        c["n_q"], c["n_k"] = c["n_q"] * 3 // 4, c["n_k"] - c["n_q"] + c["n_q"] * 3 // 4
    return c


def _cache_bytes(c):
    _, h_kv, d, _, _ = SHAPES[c["shape"]]
    return 4.0 * c["batch"] * h_kv * d * c["n_k"]


# ---- rotation frequencies and window thresholds, from their definitions

def _theta(case):
    """theta_r = base^(-2r/d), or the llama3 rule (factor 32, 1, 4, 8192) over it; fp64."""
    _, _, d, base, llama3 = SHAPES[case["shape"]]
    r = torch.arange(d // 2, dtype=torch.float64)
    th = torch.pow(torch.tensor(base, dtype=torch.float64), -2.0 * r / d)
    if not llama3:
        return th
    lam = 2.0 * math.pi / th
    s = (8192.0 / lam - 1.0) / 3.0
    mid = (1.0 - s) * th / 32.0 + s * th
    return torch.where(lam < 2048.0, th, torch.where(lam > 8192.0, th / 32.0, mid))


def _window(case):
    _, _, d, base, llama3 = SHAPES[case["shape"]]
    th = _theta(case).tolist() if llama3 else None
    kind = case["window"]
    if kind == "off":
        return atf.Window(d, base, math.inf, inv_freq=th)
    if kind == "variable":
        half = d // 2
        return atf.Window(d, base, 2.0, inv_freq=th,
                          k_profile=[16.0 - 14.0 * r / (half - 1) for r in range(half)])
    return atf.Window(d, base, 2.0, inv_freq=th, slice_pairs=8 if kind == "rounded" else 0)


def _thresholds(case):
    """Pair r is kept at distance z iff z <= W[r]; python ints."""
    th = _theta(case).tolist()
    half = len(th)
    kind = case["window"]
    if kind == "off":
        return [2 ** 31 - 1] * half
    k = [16.0 - 14.0 * r / (half - 1) for r in range(half)] if kind == "variable" else [2.0] * half
    W = [int(min(2 ** 31 - 1, math.floor(k[r] * 2.0 * math.pi / th[r]))) for r in range(half)]
    if kind == "rounded":
        W = [W[r // 8 * 8 + 7] for r in range(half)]
    return W


def _q_pos0(case):
    """Position of the first query row (prefill), or of the query (decode)."""
    return case["n_k"] - case["n_q"]


def _lengths(case):
    """Keys of each row of a ragged batch: the longest, the shortest and a spread between."""
    n, B = case["n_k"], case["batch"]
    return [max(1, int(n * math.exp(-3.0 * ((7 * b) % B) / B))) for b in range(B)]


# ---- the states

def _randn(gen, shape, dtype=torch.bfloat16, scale=None):
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    if scale is not None:
        x *= scale
    return x.to(dtype)


def _key_scale(d, cache):
    """Spread of the keys over the pairs, 0.5 at the highest frequency to 2 at the lowest:
    [d] for token-major keys, [d/16, 1, 16] for the pair-chunk-major cache."""
    half = d // 2
    sig = 0.5 + 1.5 * torch.arange(half, dtype=torch.float32, device="cuda") / (half - 1)
    if not cache:
        return torch.cat([sig, sig])
    s = sig.view(half // 8, 1, 8)
    return torch.cat([s, s], dim=2)


def prepare(case, seed):
    h_q, h_kv, d, _, _ = SHAPES[case["shape"]]
    B, n_q, n_k, op = case["batch"], case["n_q"], case["n_k"], case["op"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    s = {"case": case, "window": _window(case)}
    bf, f32 = torch.bfloat16, torch.float32
    paged = op == "decode_paged"
    if paged:
        pt = case["page_tokens"]
        lens = _lengths(case)
        need = [-(-n // pt) for n in lens]
        pages, width = sum(need), max(need)
        order = torch.randperm(pages, generator=gen, device="cuda").to(torch.int32).cpu()
        table = torch.zeros((B, width), dtype=torch.int32)
        at = 0
        for b, n in enumerate(need):
            table[b, :n] = order[at:at + n]
            at += n
        s["table"] = table.cuda()
        s["k"] = _randn(gen, atf.kpages_shape(pages, pt, h_kv, d), scale=_key_scale(d, True))
        s["v"] = _randn(gen, atf.vpages_shape(pages, pt, h_kv, d))
    else:
        s["k"] = _randn(gen, atf.kcache_shape(B, n_k, h_kv, d), scale=_key_scale(d, True))
        s["v"] = _randn(gen, atf.vcache_shape(B, n_k, h_kv, d))
    if op in ("decode_paged", "decode_ragged"):
        lens = torch.tensor(_lengths(case), dtype=torch.int32)
        s["n_k_rows"] = lens.cuda()
        s["q_pos_rows"] = (lens - 1).cuda()
    if op in ("append", "append_rotated", "step"):
        s["k_new"] = _randn(gen, (B, n_q, h_kv, d), scale=_key_scale(d, False))
        s["v_new"] = _randn(gen, (B, n_q, h_kv, d))
    if op.startswith("prefill"):
        s["q"] = _randn(gen, (B, n_q, h_q, d))
        s["lse"] = torch.empty((B, h_q, n_q), dtype=f32, device="cuda")
    elif not op.startswith("append"):
        s["q"] = _randn(gen, (B, h_q, d))
        s["lse"] = torch.empty((B, h_q), dtype=f32, device="cuda")
        s["workspace"] = torch.empty(atf.atf_decode_workspace_bytes(B, h_q, h_kv, n_k, d),
                                     dtype=torch.uint8, device="cuda")
    if "q" in s:
        s["o"] = torch.empty(s["q"].shape, dtype=bf, device="cuda")
    return s


def run(s):
    case = s["case"]
    op, pos = case["op"], _q_pos0(case)
    if op in ("append", "append_rotated", "step"):
        if op == "append":
            atf.atf_cache_append(s["k_new"], s["v_new"], s["k"], s["v"], pos)
        else:
            atf.atf_cache_append_rotated(s["k_new"], s["v_new"], s["k"], s["v"], pos, s["window"])
        if op != "step":
            return {"k": s["k"], "v": s["v"]}
        atf.atf_decode(s["q"], s["k"], s["v"], s["o"], s["lse"], pos, s["window"], s["workspace"])
        return {"o": s["o"], "lse": s["lse"], "k": s["k"], "v": s["v"]}
    if op == "decode":
        atf.atf_decode(s["q"], s["k"], s["v"], s["o"], s["lse"], pos, s["window"], s["workspace"])
    elif op == "decode_unrotated":
        atf.atf_decode_unrotated(s["q"], s["k"], s["v"], s["o"], s["lse"], pos, s["window"],
                                 s["workspace"])
    elif op == "decode_ragged":
        atf.atf_decode_ragged(s["q"], s["k"], s["v"], s["o"], s["lse"], s["n_k_rows"],
                              s["q_pos_rows"], case["n_k"], s["window"], s["workspace"])
    elif op == "decode_paged":
        atf.atf_decode_paged(s["q"], s["k"], s["v"], s["o"], s["lse"], s["table"], s["n_k_rows"],
                             s["q_pos_rows"], case["n_k"], s["window"], s["workspace"])
    elif op == "prefill":
        atf.atf_prefill(s["q"], s["k"], s["v"], s["o"], s["lse"], pos, s["window"])
    elif op == "prefill_unrotated":
        atf.atf_prefill_unrotated(s["q"], s["k"], s["v"], s["o"], s["lse"], pos, s["window"])
    else:
        raise ValueError(op)
    return {"o": s["o"], "lse": s["lse"]}


# ---- the work of one pass

def _attention_work(n_q, pos0, n_k, W, h_q, h_kv, d):
    """(bytes, flops) of one batch entry: 4 flops per kept (cell, pair), 2 d per causal cell;
    q, o and lse, V, and of K the (key, pair)s that some row keeps."""
    pos = torch.arange(pos0, pos0 + n_q, dtype=torch.int64)
    last = torch.clamp(pos, max=n_k - 1)
    cells = int((last + 1).sum())
    terms, key_pairs = 0, 0
    reach = min(pos0 + n_q, n_k)  # keys some row attends
    for w in W:
        first = torch.clamp(pos - w, min=0)
        terms += int(torch.clamp(last - first + 1, min=0).sum())
        key_pairs += max(0, reach - max(0, pos0 - w))
    nbytes = h_kv * (4.0 * key_pairs + 2.0 * d * reach) + n_q * h_q * (4.0 * d + 4.0)
    return nbytes, h_q * (4.0 * terms + 2.0 * d * cells)


def work(case):
    h_q, h_kv, d, _, _ = SHAPES[case["shape"]]
    B, n_q, op = case["batch"], case["n_q"], case["op"]
    W = _thresholds(case)
    moved = 8.0 * B * n_q * h_kv * d  # keys and values, read and written
    turned = 3.0 * B * n_q * h_kv * d
    if op.startswith("append"):
        return {"bytes": moved, "flops": turned if op == "append_rotated" else 0.0}
    lens = _lengths(case) if op in ("decode_paged", "decode_ragged") else [case["n_k"]] * B
    nbytes = flops = 0.0
    done = {}
    for n in lens:
        if n not in done:
            done[n] = _attention_work(n_q, n - n_q, n, W, h_q, h_kv, d)
        nbytes += done[n][0]
        flops += done[n][1]
    if op == "step":
        nbytes, flops = nbytes + moved, flops + turned
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["op"] == "append":
        return "exact"
    if case["op"] == "append_rotated":
        # rotated keys rounded to bf16: 1.7e-3 against 64 bits where every key is new, of
        # which two implementations share all but the rounding of near ties
        return {"rel": 4e-3}
    # outputs of bf16 products rounded to bf16: 2e-3 against 64 bits, 4e-3 where the
    # rotated queries and keys are rounded too
    return {"rel": 1.2e-2}


# ---- the same in 64 bits

def _tokens_of_k(k):
    """[..., d/16, T, 16] pair-chunk-major -> [..., T, d], fp64."""
    *lead, nc, T, _ = k.shape
    n = len(lead)
    x = k.to(torch.float64).view(*lead, nc, T, 2, 8)
    return x.permute(*range(n), n + 1, n + 2, n, n + 3).reshape(*lead, T, nc * 16)


def _tokens_of_v(v):
    """[..., nb, d, 16] -> [..., 16 nb, d]; slot 8h + 4a + b of a row holds token 8a + 4h + b."""
    *lead, nb, d, _ = v.shape
    n = len(lead)
    x = v.to(torch.float64).view(*lead, nb, d, 2, 2, 4)
    return x.permute(*range(n), n, n + 3, n + 2, n + 4, n + 1).reshape(*lead, nb * 16, d)


def _rotate(x, pos, theta):
    """x [..., T, d] (fp64), token t turned to pos[t]; rotate-half pairs (r, r + d/2)."""
    half = x.shape[-1] // 2
    ang = pos.to(torch.float64)[:, None] * theta.to(x.device)[None, :]
    c, s = torch.cos(ang), torch.sin(ang)
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], dim=-1)


def _attend(q, k, v, pos0, W):
    """q [G, n_q, d] at positions pos0 .., k and v [T, d] at 0 ..; (o [G, n_q, d], lse [G, n_q])."""
    G, n_q, d = q.shape
    half, T = d // 2, k.shape[0]
    scale = 1.0 / math.sqrt(d)
    o = torch.empty_like(q)
    lse = torch.empty((G, n_q), dtype=torch.float64, device=q.device)
    rows, keys = (1024, 4096) if n_q > 64 else (n_q, 65536)
    for i0 in range(0, n_q, rows):
        qt = q[:, i0:i0 + rows].reshape(-1, d)
        n = min(rows, n_q - i0)
        p_lo, p_hi = pos0 + i0, pos0 + i0 + n - 1
        pos = torch.arange(p_lo, p_hi + 1, device=q.device).repeat(G)
        m = torch.full((G * n, 1), -math.inf, dtype=torch.float64, device=q.device)
        l = torch.zeros_like(m)
        acc = torch.zeros((G * n, d), dtype=torch.float64, device=q.device)
        for j0 in range(0, min(T, p_hi + 1), keys):
            j1 = min(T, p_hi + 1, j0 + keys)
            kt = k[j0:j1]
            z_lo, z_hi = max(0, p_lo - (j1 - 1)), p_hi - j0
            full = [r for r in range(half) if W[r] >= z_hi]
            part = [r for r in range(half) if z_lo <= W[r] < z_hi]
            z = pos[:, None] - torch.arange(j0, j1, device=q.device)[None, :] \
                if part or j1 - 1 > p_lo else None
            if full:
                at = torch.tensor(full + [r + half for r in full], device=q.device)
                sc = qt[:, at] @ kt[:, at].t().contiguous()
            else:
                sc = torch.zeros((G * n, j1 - j0), dtype=torch.float64, device=q.device)
            for r in part:
                t = qt[:, r:r + 1] * kt[:, r][None, :]
                t += qt[:, r + half:r + half + 1] * kt[:, r + half][None, :]
                sc += t.masked_fill_(z > W[r], 0.0)
            sc *= scale
            if j1 - 1 > p_lo:
                sc.masked_fill_(z < 0, -math.inf)
            m_new = torch.maximum(m, sc.amax(dim=1, keepdim=True))
            a = torch.exp(m - m_new)
            sc.sub_(m_new).exp_()
            l = l * a + sc.sum(dim=1, keepdim=True)
            acc = acc * a + sc @ v[j0:j1]
            m = m_new
        o[:, i0:i0 + n] = (acc / l).view(G, n, d)
        lse[:, i0:i0 + n] = (m + torch.log(l)).view(G, n)
    return o, lse


def exact(case, seed):
    h_q, h_kv, d, _, _ = SHAPES[case["shape"]]
    B, n_q, op, G = case["batch"], case["n_q"], case["op"], h_q // h_kv
    if work(case)["flops"] > 1.5 * MAX_FLOPS:
        return None
    s = prepare(case, seed)
    theta, W, pos0 = _theta(case), _thresholds(case), _q_pos0(case)
    out = {}
    if op in ("append", "append_rotated", "step"):
        new = s["k_new"].to(torch.float64).transpose(1, 2)  # [B, h_kv, n_q, d]
        at = torch.arange(pos0, pos0 + n_q, device="cuda")
        if op != "append":
            new = _rotate(new, at, theta)
        k = _tokens_of_k(s["k"])
        k[:, :, pos0:pos0 + n_q] = new
        v = _tokens_of_v(s["v"])
        v[:, :, pos0:pos0 + n_q] = s["v_new"].to(torch.float64).transpose(1, 2)
        nc, C = d // 16, case["n_k"]
        out["k"] = k.view(B, h_kv, C, 2, nc, 8).permute(0, 1, 4, 2, 3, 5).reshape(s["k"].shape)
        out["v"] = v.view(B, h_kv, -1, 2, 2, 4, d).permute(0, 1, 2, 6, 4, 3, 5).reshape(s["v"].shape)
        if op != "step":
            return out
    prefill = op.startswith("prefill")
    q = s["q"].to(torch.float64)
    q = q.permute(0, 2, 1, 3) if prefill else q[:, :, None, :]  # [B, h_q, n_q, d]
    o = torch.empty((B, h_q, n_q, d), dtype=torch.float64, device="cuda")
    lse = torch.empty((B, h_q, n_q), dtype=torch.float64, device="cuda")
    turn = op.endswith("unrotated")
    lens = _lengths(case) if op in ("decode_paged", "decode_ragged") else [case["n_k"]] * B
    for b in range(B):
        n = lens[b]
        if op == "decode_paged":
            own = s["table"][b, :-(-n // case["page_tokens"])].long()
        for g in range(h_kv):
            if op == "step":
                kg, vg = k[b, g, :n], v[b, g, :n]
            elif op == "decode_paged":
                kg = _tokens_of_k(s["k"][own, g]).reshape(-1, d)[:n]
                vg = _tokens_of_v(s["v"][own, g]).reshape(-1, d)[:n]
            else:
                kg, vg = _tokens_of_k(s["k"][b, g])[:n], _tokens_of_v(s["v"][b, g])[:n]
            qg = q[b, g * G:(g + 1) * G]
            if turn:
                kg = _rotate(kg, torch.arange(n, device="cuda"), theta)
                qg = _rotate(qg, torch.arange(n - n_q, n, device="cuda"), theta)
            o[b, g * G:(g + 1) * G], lse[b, g * G:(g + 1) * G] = _attend(qg, kg, vg, n - n_q, W)
    out["o"] = o.permute(0, 2, 1, 3).contiguous() if prefill else o[:, :, 0]
    out["lse"] = lse if prefill else lse[:, :, 0]
    return out
