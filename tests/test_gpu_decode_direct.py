"""Decode at the edges of the rule that leaves a uniform batch unsplit: a row's keys in one
workgroup of 8 waves, which writes the output itself, against the split kernels and merge on
the other side.  Key counts lie at the limits for few and for many rows, at fewer keys than
waves' groups, and windows end inside the rows; the caches past n_k and the workspace hold
NaN; pre-rotated and unrotated caches, against the oracle."""
import math

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
    # batch, group, h_kv, n_k, q_pos, d, k
    (1, 7, 2, 1, 0, 64, 2.0),
    (3, 3, 8, 225, 224, 128, 2.0),
    (1, 7, 4, 256, 255, 128, 2.0),      # limits with fewer than 128 workgroups, and past them
    (1, 7, 4, 257, 256, 128, 2.0),
    (1, 7, 4, 1280, 1279, 128, 0.5),
    (1, 7, 4, 1281, 1280, 128, 0.5),
    (1, 7, 2, 769, 768, 64, math.inf),
    (1, 7, 2, 2560, 2559, 64, 0.5),
    (1, 7, 2, 2561, 2560, 64, 0.5),
    (1, 7, 2, 9000, 2559, 64, 0.5),     # the limit counts keys up to the query
    (64, 2, 2, 769, 768, 128, 2.0),     # 128 workgroups
    (127, 1, 2, 1025, 1030, 64, 2.0),   # 254, the query past the cache's end
    (64, 16, 4, 513, 512, 64, 2.0),     # 256 workgroups, whole tiles of heads
    (32, 3, 8, 1600, 1599, 128, 0.5),
]


@pytest.mark.parametrize("unrotated", [False, True], ids=["rotated", "unrotated"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(x) for x in c))
def test_decode_direct(case, unrotated):
    import paper_2608_02947_amd as atf
    B, G, h_kv, n_k, q_pos, d, kwin = case
    h_q, cap, base = G * h_kv, n_k + 21, 1e4
    g = torch.Generator(device="cpu").manual_seed(B * 1009 + n_k)
    q = torch.randn((B, 1, h_q, d), generator=g).to(torch.bfloat16)
    k = torch.randn((B, n_k, h_kv, d), generator=g).to(torch.bfloat16)
    v = torch.randn((B, n_k, h_kv, d), generator=g).to(torch.bfloat16)
    th = W.rope_theta(d, base)
    win, widths = windows_for(d, base, kwin, None, n_ctx=max(n_k, q_pos + 1))
    qr = W.rotate_half(q, torch.tensor([q_pos]), th)
    kr = W.rotate_half(k, torch.arange(n_k), th)
    rows = torch.tensor([0, B // 2, B - 1]).unique()  # of a large batch three rows are compared
    o_ref, lse_ref, _ = oracle.attend(qr[rows], kr[rows], v[rows], q_pos, widths)

    def cache(x, pack):
        full = torch.full((B, cap, h_kv, d), float("nan"), dtype=torch.bfloat16)
        full[:, :n_k] = x
        return pack(full.to(DEV))

    kp, vp = cache(k if unrotated else kr, pack_kcache), cache(v, pack_vcache)
    qd = (q if unrotated else qr)[:, 0].contiguous().to(DEV)
    ws = torch.full((atf.atf_decode_workspace_bytes(B, h_q, h_kv, n_k, d),), 255, dtype=torch.uint8, device=DEV)
    o = torch.full_like(qd, float("nan"))
    lse = torch.full((B, h_q), float("nan"), dtype=torch.float32, device=DEV)
    note(f"decode direct {case} unrotated={unrotated}")
    fn = atf.atf_decode_unrotated if unrotated else atf.atf_decode
    fn(qd, kp, vp, o, lse, q_pos, win, ws, n_k=n_k)
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all() and torch.isfinite(lse).all()
    compare(to_f64(o[rows.to(DEV)]), to_f64(lse[rows.to(DEV)]), o_ref[:, 0], lse_ref[:, :, 0], f"direct {case}")


# just past whole rounds of 256 workgroups, where long rows are split after all
ROUNDS = [
    # batch, group, h_kv, n_k, d, splits pre-rotated, splits unrotated (0: direct)
    (33, 3, 8, 1000, 128, 0, 0),     # too short for either
    (33, 3, 8, 2100, 128, 4, 4),
    (42, 2, 8, 2049, 128, 3, 3),
    (44, 1, 8, 4000, 128, 2, 2),     # 352 pairs
    (50, 1, 8, 4000, 128, 0, 0),     # 400: nearer two rounds
    (66, 1, 8, 3100, 128, 2, 2),     # 528
    (100, 1, 8, 2000, 128, 2, 2),    # 800
    (17, 1, 16, 2100, 64, 4, 4),
    (24, 1, 16, 1200, 64, 0, 2),     # 384, too short pre-rotated
    (65, 1, 16, 300, 64, 0, 1),      # 1,040: no room for two splits
    (130, 2, 8, 129, 64, 0, 1),
    # 39 heads to a KV head: three workgroups of 13, on 16x16 tiles unless the caches pass 341 MB
    (40, 39, 1, 3500, 128, 6, 4),
    (150, 39, 1, 1200, 128, 0, 0),
    (240, 39, 1, 3400, 128, 5, 5),
]


@pytest.mark.parametrize("unrotated", [False, True], ids=["rotated", "unrotated"])
@pytest.mark.parametrize("case", ROUNDS, ids=lambda c: "x".join(str(x) for x in c))
def test_decode_between_whole_rounds(case, unrotated):
    """Three different rows, each in a third of the batch: all copies of a row agree bit for
    bit, and the rows agree with the oracle."""
    import paper_2608_02947_amd as atf
    B, G, h_kv, n_k, d, *splits = case
    h_q, base, q_pos, cap = G * h_kv, 1e4, n_k - 1, n_k + 21
    direct = routes.decode_direct(B, G, h_kv, n_k, q_pos, d, unrotated, cap=cap)
    plan = 0 if direct else routes.decode_splits(B, G, h_kv, n_k, q_pos, d, unrotated)[0]
    assert plan == splits[unrotated]
    assert routes.decode_cols16(B, G, h_kv, n_k, q_pos, d, cap=cap) == (B < 240)
    g = torch.Generator(device="cpu").manual_seed(B * 1009 + n_k)
    q = torch.randn((3, 1, h_q, d), generator=g).to(torch.bfloat16)
    k = torch.randn((3, n_k, h_kv, d), generator=g).to(torch.bfloat16)
    v = torch.randn((3, n_k, h_kv, d), generator=g).to(torch.bfloat16)
    th = W.rope_theta(d, base)
    win, widths = windows_for(d, base, 2.0, None, n_ctx=n_k)
    qr = W.rotate_half(q, torch.tensor([q_pos]), th)
    kr = W.rotate_half(k, torch.arange(n_k), th)
    o_ref, lse_ref, _ = oracle.attend(qr, kr, v, q_pos, widths)
    row = torch.arange(B, device=DEV) % 3

    def cache(x, pack):
        full = torch.full((3, cap, h_kv, d), float("nan"), dtype=torch.bfloat16)
        full[:, :n_k] = x
        return pack(full.to(DEV))[row]

    kp, vp = cache(k if unrotated else kr, pack_kcache), cache(v, pack_vcache)
    qd = (q if unrotated else qr)[:, 0].to(DEV)[row]
    ws = torch.full((atf.atf_decode_workspace_bytes(B, h_q, h_kv, n_k, d),), 255, dtype=torch.uint8, device=DEV)
    o = torch.full_like(qd, float("nan"))
    lse = torch.full((B, h_q), float("nan"), dtype=torch.float32, device=DEV)
    note(f"decode rounds {case} unrotated={unrotated}")
    fn = atf.atf_decode_unrotated if unrotated else atf.atf_decode
    fn(qd, kp, vp, o, lse, q_pos, win, ws, n_k=n_k)
    torch.cuda.synchronize()
    assert torch.equal(o, o[:3][row]) and torch.equal(lse, lse[:3][row])
    compare(to_f64(o[:3]), to_f64(lse[:3]), o_ref[:, 0], lse_ref[:, :, 0], f"rounds {case}")


# a ragged batch's bound on its rows' keys: at the limits for few and for many workgroups
# and past them; rows of no key, one key, fewer and more keys than the query's position
RAGGED = [
    # batch, group, h_kv, bound, d
    (5, 3, 8, 1280, 128),
    (5, 3, 8, 1281, 128),
    (6, 7, 2, 2560, 64),
    (6, 7, 2, 2561, 64),
    (128, 1, 8, 1300, 128),   # 1,024 workgroups
]


@pytest.mark.parametrize("case", RAGGED, ids=lambda c: "x".join(str(x) for x in c))
def test_decode_direct_ragged(case):
    import paper_2608_02947_amd as atf
    B, G, h_kv, n_k, d = case
    h_q, base = G * h_kv, 1e4
    g = torch.Generator(device="cpu").manual_seed(B * 1009 + n_k)
    q = torch.randn((B, h_q, d), generator=g).to(torch.bfloat16)
    k = torch.randn((B, n_k, h_kv, d), generator=g).to(torch.bfloat16)
    v = torch.randn((B, n_k, h_kv, d), generator=g).to(torch.bfloat16)
    lens = [n_k, 0, 1, 259, n_k // 2] + [(37 * b) % n_k for b in range(5, B)]
    pos = [n_k - 1, 5, 0, 400, n_k // 4] + [max(n - 1, 0) for n in lens[5:]]
    win, widths = windows_for(d, base, 2.0, None, n_ctx=n_k)
    kc, vc = k.clone(), v.clone()
    for b, n in enumerate(lens):
        kc[b, n:], vc[b, n:] = float("nan"), float("nan")
    ws = torch.full((atf.atf_decode_workspace_bytes(B, h_q, h_kv, n_k, d),), 255, dtype=torch.uint8, device=DEV)
    o = torch.full((B, h_q, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    lse = torch.full((B, h_q), float("nan"), dtype=torch.float32, device=DEV)
    note(f"decode direct ragged {case}")
    i32 = dict(dtype=torch.int32, device=DEV)
    atf.atf_decode_ragged(q.to(DEV), pack_kcache(kc.to(DEV)), pack_vcache(vc.to(DEV)), o, lse,
                          torch.tensor(lens, **i32), torch.tensor(pos, **i32), n_k, win, ws)
    torch.cuda.synchronize()
    assert (o[1] == 0).all() and (lse[1] == -math.inf).all()
    for b in (0, 2, 3, 4, B - 1):
        o_ref, lse_ref, _ = oracle.attend(q[b:b + 1, None], k[b:b + 1, :lens[b]], v[b:b + 1, :lens[b]],
                                          pos[b], widths)
        compare(to_f64(o[b:b + 1]), to_f64(lse[b:b + 1]), o_ref[:, 0], lse_ref[:, :, 0], f"ragged {case} row {b}")
