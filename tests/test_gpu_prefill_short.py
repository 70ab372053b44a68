"""The two kernels behind atf_prefill and atf_prefill_unrotated on the same rows.

A call with few rows splits the keys of a row block over 4 or 8 waves; a call with many
gives a workgroup 256 rows.  Each case runs once alone (few rows) and once as every entry
of a batch large enough for the other kernel; both are held to the oracle's tolerances, all
batch entries have to agree bit for bit, and the caches past n_k hold NaN.  Sizes lie at the
edges of the 32-key blocks, of the waves' shares (4 x 32 and 8 x 32 keys) and of the 32-row
blocks; from 4,096 keys the few-row call uses 8 waves.
"""
import math

import numpy as np
import pytest
import torch

from conftest import gpu_available
import oracle
import workloads as W
from parity import compare, note, pack_kcache, pack_vcache, to_f64, windows_for

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

DEV = "cuda"

CASES = [
    # n_q, n_k, q0, h_q, h_kv, d, base, k, slice_pairs
    (1, 33, 32, 3, 1, 128, 1e4, 2.0, 0),          # a second wave with one key
    (5, 31, 26, 7, 1, 64, 1e6, 2.0, 0),           # 35 rows: a row block of 3
    (11, 129, 118, 6, 2, 128, 5e5, 2.0, 0),       # 33 rows, one key past 4 x 32
    (32, 128, 96, 1, 1, 64, 1e4, math.inf, 0),    # exactly one row block, 4 x 32 keys
    (37, 257, 220, 8, 2, 128, 1e7, math.inf, 0),  # one key past 8 x 32
    (40, 97, 70, 2, 1, 64, 1e4, 1.0, 8),          # keys end before the last queries, rounded slice
    (16, 4096, 4080, 14, 2, 64, 1e6, 2.0, 0),     # 8 waves, whole blocks
    (9, 4129, 4120, 7, 1, 128, 1e7, 2.0, 0),      # 8 waves, ragged
    (3, 4200, 4190, 16, 2, 64, 1e4, math.inf, 0),  # 8 waves, keys past the last query
    (20, 4100, 4300, 4, 1, 128, 1e4, 2.0, 8),     # 8 waves, keys end before every query
    (40, 2100, 2060, 7, 1, 64, 100.0, 2.0, 0),    # every window ends inside the keys: far tiles keep no pair
    (33, 2100, 2067, 4, 1, 128, 100.0, 2.0, 0),   # the same at d = 128
    (70, 700, 630, 2, 2, 64, 100.0, 2.0, 8),      # and with the rounded slice
]


def _run(fn, q, kp, vp, q0, win, n_k):
    o = torch.full_like(q, float("nan"))
    lse = torch.full((q.shape[0], q.shape[2], q.shape[1]), float("nan"), dtype=torch.float32, device=DEV)
    fn(q, kp, vp, o, lse, q0, win, n_k=n_k)
    torch.cuda.synchronize()
    return o, lse


@pytest.mark.parametrize("unrotated", [False, True], ids=["rotated", "unrotated"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(x) for x in c))
def test_few_rows_and_many_rows(case, unrotated):
    import paper_2608_02947_amd as atf
    n_q, n_k, q0, h_q, h_kv, d, base, kwin, atom = case
    cap = n_k + 19
    g = torch.Generator(device="cpu").manual_seed(n_q * 7919 + n_k)
    q = torch.randn((1, n_q, h_q, d), generator=g).to(torch.bfloat16)
    k = torch.randn((1, n_k, h_kv, d), generator=g).to(torch.bfloat16)
    v = torch.randn((1, n_k, h_kv, d), generator=g).to(torch.bfloat16)
    th = W.rope_theta(d, base)
    qr = W.rotate_half(q, torch.arange(q0, q0 + n_q), th)
    kr = W.rotate_half(k, torch.arange(0, n_k), th)
    win, widths = windows_for(d, base, kwin, None, n_ctx=max(n_k, q0 + n_q), slice_pairs=atom)
    o_ref, lse_ref, _ = oracle.attend(qr, kr, v, q0, widths, atom=atom)

    def caches(x, pack):
        full = torch.full((1, cap, h_kv, d), float("nan"), dtype=torch.bfloat16)
        full[:, :n_k] = x
        return pack(full.to(DEV))

    fn = atf.atf_prefill_unrotated if unrotated else atf.atf_prefill
    qd = (q if unrotated else qr).to(DEV)
    kp, vp = caches(k if unrotated else kr, pack_kcache), caches(v, pack_vcache)
    note(f"few rows {case} unrotated={unrotated}")
    o1, l1 = _run(fn, qd, kp, vp, q0, win, n_k)
    compare(to_f64(o1), to_f64(l1), o_ref, lse_ref, f"few rows {case}")

    # position tiles x kv heads of one entry, and entries enough for 400 workgroups
    tiles = -(-n_q // ((128 if d == 64 else 256) // (h_q // h_kv))) * h_kv
    B = -(-400 // tiles)
    rep = lambda x: x.expand(B, *x.shape[1:]).contiguous()
    note(f"many rows {case} unrotated={unrotated} B={B}")
    o2, l2 = _run(fn, rep(qd), rep(kp), rep(vp), q0, win, n_k)
    assert torch.equal(o2, o2[:1].expand_as(o2)) and torch.equal(l2, l2[:1].expand_as(l2))
    compare(to_f64(o2[:1]), to_f64(l2[:1]), o_ref, lse_ref, f"many rows {case}")
    # two bf16 roundings of the same output at most, plus the probabilities' rounding
    # against another running maximum (2^-9 of |v| averaged over the keys of a row)
    diff = (o1.double() - o2[:1].double()).abs()
    assert float((diff - 2.0 ** -7 * torch.maximum(o1.double().abs(), o2[:1].double().abs())).max()) <= 1e-2
    assert np.abs(to_f64(l1) - to_f64(l2[:1])).max() <= 1e-4


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("what", ["query", "keys"])
def test_nan_reaches_the_lse(what, d):
    """A row whose scores are NaN, in every wave (its query is NaN) or in one wave only (a
    32-key block is), has a NaN output and LSE with few rows as with many; keys end before
    every query at a whole block, so that no mask touches a score."""
    import paper_2608_02947_amd as atf
    n_q, n_k, q0 = 9, 128, 200
    g = torch.Generator(device="cpu").manual_seed(d)
    q = torch.randn((1, n_q, 2, d), generator=g).to(torch.bfloat16)
    k, v = (torch.randn((1, n_k, 1, d), generator=g).to(torch.bfloat16) for _ in range(2))
    if what == "query":
        q[0, 4, 1] = math.nan
        bad = torch.zeros((2, n_q), dtype=torch.bool)
        bad[1, 4] = True
    else:
        k[0, 32:64] = math.nan
        bad = torch.ones((2, n_q), dtype=torch.bool)
    for kwin in (2.0, math.inf):
        win, _ = windows_for(d, 1e6, kwin, None, n_ctx=q0 + n_q)
        for B in (1, 400):
            rep = lambda x: x.expand(B, *x.shape[1:]).contiguous()
            note(f"nan {what} d={d} k={kwin} B={B}")
            o, lse = _run(atf.atf_prefill, rep(q.to(DEV)), rep(pack_kcache(k.to(DEV))),
                          rep(pack_vcache(v.to(DEV))), q0, win, n_k)
            for b in {0, B - 1}:
                assert torch.equal(lse[b].isnan().cpu(), bad), (kwin, B)
                assert torch.equal(o[b].isnan().cpu(), bad.T[:, :, None].expand(n_q, 2, d)), (kwin, B)
