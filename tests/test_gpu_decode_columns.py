"""Decode at the edges of its two split kernels: up to 16 query heads per KV head are the
columns of 16x16 matrix tiles, 17 to 32 of 32x32 ones.  Key counts lie at the edges of the
8-, 16- and 32-token groups, windows end inside either chunk of a chunk pair (a table that is
not monotone prunes the upper chunk and keeps the lower one), the caches past n_k hold NaN;
pre-rotated and unrotated caches, against the oracle."""
import math

import numpy as np
import pytest
import torch

from conftest import gpu_available
import oracle
import routes
import workloads as W
from parity import compare, note, pack_kcache, pack_vcache, to_f64, windows_for

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

DEV = "cuda"

CASES = [
    # group, h_kv, n_k, q_pos, d, k, table ("base" or "mixed")
    (1, 2, 7, 6, 64, 2.0, "base"),
    (16, 1, 9, 8, 128, 2.0, "base"),
    (16, 2, 17, 16, 64, math.inf, "base"),
    (15, 1, 127, 126, 128, 2.0, "base"),
    (3, 3, 129, 128, 64, 2.0, "mixed"),
    (7, 1, 641, 640, 128, 2.0, "mixed"),
    (5, 1, 1000, 700, 128, 0.5, "base"),      # keys past the query
    (18, 1, 641, 640, 128, 2.0, "mixed"),
    (32, 1, 129, 200, 64, 2.0, "base"),       # query past the cache's end
]


@pytest.mark.parametrize("unrotated", [False, True], ids=["rotated", "unrotated"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(x) for x in c))
def test_decode_columns(case, unrotated):
    import paper_2608_02947_amd as atf
    G, h_kv, n_k, q_pos, d, kwin, table = case
    B, h_q, cap, base = 2, G * h_kv, n_k + 21, 1e4
    g = torch.Generator(device="cpu").manual_seed(G * 1009 + n_k)
    q = torch.randn((B, 1, h_q, d), generator=g).to(torch.bfloat16)
    k = torch.randn((B, n_k, h_kv, d), generator=g).to(torch.bfloat16)
    v = torch.randn((B, n_k, h_kv, d), generator=g).to(torch.bfloat16)
    th = W.rope_theta(d, base)
    if table == "mixed":
        # thresholds rise and fall from chunk to chunk: 3 to 600 tokens at k = 2
        th = torch.tensor(np.random.default_rng(7).uniform(0.02, 4.0, d // 2)) * \
            torch.tensor([1.0, 6.0]).repeat_interleave(8).repeat(d // 32).double()
    theta = th.numpy() if table == "mixed" else None
    win, widths = windows_for(d, base, kwin, theta, n_ctx=max(n_k, q_pos + 1))
    qr = W.rotate_half(q, torch.tensor([q_pos]), th)
    kr = W.rotate_half(k, torch.arange(n_k), th)
    o_ref, lse_ref, _ = oracle.attend(qr, kr, v, q_pos, widths)

    def cache(x, pack):
        full = torch.full((B, cap, h_kv, d), float("nan"), dtype=torch.bfloat16)
        full[:, :n_k] = x
        return pack(full.to(DEV))

    kp, vp = cache(k if unrotated else kr, pack_kcache), cache(v, pack_vcache)
    qd = (q if unrotated else qr)[:, 0].contiguous().to(DEV)
    ws = torch.full((atf.atf_decode_workspace_bytes(B, h_q, h_kv, n_k, d),), 255, dtype=torch.uint8, device=DEV)
    o = torch.full_like(qd, float("nan"))
    lse = torch.full((B, h_q), float("nan"), dtype=torch.float32, device=DEV)
    note(f"decode columns {case} unrotated={unrotated}")
    fn = atf.atf_decode_unrotated if unrotated else atf.atf_decode
    fn(qd, kp, vp, o, lse, q_pos, win, ws, n_k=n_k)
    torch.cuda.synchronize()
    compare(to_f64(o), to_f64(lse), o_ref[:, 0], lse_ref[:, :, 0], f"columns {case}")


# rows that are split over workgroups of 4 waves, with the merge after them
SPLIT_CASES = [
    (1, 2, 4097, 4096, 64, 2.0, "mixed"),
    (16, 1, 2578, 2577, 128, 2.0, "mixed"),
    (16, 2, 4129, 4128, 64, math.inf, "base"),
    (15, 1, 2561, 2560, 128, 2.0, "base"),
    (7, 1, 2568, 2567, 128, 2.0, "mixed"),
    (3, 3, 4100, 4096, 64, 2.0, "mixed"),
    (5, 1, 2594, 2568, 128, 0.5, "base"),      # keys past the query: the last block is cut
    (12, 1, 2593, 3000, 128, 2.0, "mixed"),    # query past the cache's end
]


@pytest.mark.parametrize("unrotated", [False, True], ids=["rotated", "unrotated"])
@pytest.mark.parametrize("case", SPLIT_CASES, ids=lambda c: "x".join(str(x) for x in c))
def test_decode_columns_split(case, unrotated):
    G, h_kv, n_k, q_pos, d, _, _ = case
    assert routes.decode_cols16(2, G, h_kv, n_k, q_pos, d, cap=n_k + 21)
    assert not routes.decode_direct(2, G, h_kv, n_k, q_pos, d, unrotated, cap=n_k + 21)
    assert routes.decode_splits(2, G, h_kv, n_k, q_pos, d, unrotated)[0] > 1
    test_decode_columns(case, unrotated)


@pytest.mark.parametrize("unrotated", [False, True], ids=["rotated", "unrotated"])
def test_decode_columns_infinite_value(unrotated):
    """An infinite value makes its dimension's output infinite and leaves the others as they
    are: no part of a probability may be 0 where the probability is not."""
    import paper_2608_02947_amd as atf
    n_k, h_q, h_kv, d = 2000, 7, 1, 128
    g = torch.Generator(device="cpu").manual_seed(5)
    q = torch.randn((1, h_q, d), generator=g).to(torch.bfloat16)
    k = 0.1 * torch.randn((1, n_k, h_kv, d), generator=g).to(torch.bfloat16)
    v = torch.randn((1, n_k, h_kv, d), generator=g).to(torch.bfloat16)
    k[0, 0] = k[0, 37] = 0.0  # logits of 0: among them the first of a split
    win, _ = windows_for(d, 1e4, 2.0, None, n_ctx=n_k)
    ws = torch.zeros((atf.atf_decode_workspace_bytes(1, h_q, h_kv, n_k, d),), dtype=torch.uint8, device=DEV)
    outs = []
    for infinite in (False, True):
        if infinite:
            v[0, 0, 0, 3], v[0, 37, 0, 77], v[0, 1999, 0, 5] = math.inf, -math.inf, math.inf
        o, lse = torch.zeros((1, h_q, d), dtype=torch.bfloat16, device=DEV), torch.zeros((1, h_q), device=DEV)
        fn = atf.atf_decode_unrotated if unrotated else atf.atf_decode
        fn(q.to(DEV), pack_kcache(k.to(DEV)), pack_vcache(v.to(DEV)), o, lse, n_k - 1, win, ws, n_k=n_k)
        torch.cuda.synchronize()
        outs.append(o[0].float().cpu())
    want = outs[0].clone()
    want[:, 3], want[:, 77], want[:, 5] = math.inf, -math.inf, math.inf
    assert torch.equal(outs[1], want)
