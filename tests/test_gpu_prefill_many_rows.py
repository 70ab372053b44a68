"""prefill_kernel, which every prefill that fills the chip takes, where small calls would take
prefill_short_kernel: tables that are not monotone, scores that raise the running maximum many
times, groups of 128 and 256 heads, queries at positions past 2^30, and chunks of a prefill
against one call.  A case is repeated as the entries of a batch until the library's own rule
gives it that kernel; all entries have to agree bit for bit, and the first with the oracle."""
import math

import numpy as np
import pytest
import torch

from conftest import gpu_available
import oracle
import routes
import workloads as W
from parity import (compare, compare_rounding_bound, note, pack_kcache, pack_vcache, prefill_budget, to_f64,
                    windows_for, workload_window)
from test_gpu_prefill import _large_score_inputs, _small_inputs

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

DEV = "cuda"


def _batch(win, n_q, n_k, q0, group, h_kv, unrotated=False):
    """The smallest power of 2 of entries that take prefill_kernel."""
    for B in (2 ** i for i in range(10)):
        if routes.prefill_waves(win, B, n_q, n_k, q0, group, h_kv, unrotated) == 0:
            return B
    raise AssertionError("no batch takes prefill_kernel")


def _many(q, k, v, q0, win, label, scale=0.0, unrotated=False):
    """O and LSE of entry 0 of a batch of equal entries."""
    import paper_2608_02947_amd as atf
    (_, n_q, h_q, _), (_, n_k, h_kv, _) = q.shape, k.shape
    B = _batch(win, n_q, n_k, q0, h_q // h_kv, h_kv, unrotated)
    note(f"many rows {label} B={B} q={tuple(q.shape)} k={tuple(k.shape)} q0={q0} unrotated={unrotated}")
    rep = lambda x: x.expand(B, *x.shape[1:]).contiguous()
    qd = rep(q.to(DEV))
    o = torch.full_like(qd, float("nan"))
    lse = torch.full((B, h_q, n_q), float("nan"), dtype=torch.float32, device=DEV)
    fn = atf.atf_prefill_unrotated if unrotated else atf.atf_prefill
    fn(qd, rep(pack_kcache(k.to(DEV))), rep(pack_vcache(v.to(DEV))), o, lse, q0, win, scale)
    torch.cuda.synchronize()
    assert torch.equal(o, o[:1].expand_as(o)) and torch.equal(lse, lse[:1].expand_as(lse))
    return to_f64(o[:1]), to_f64(lse[:1])


def _rotated(q, k, q0, theta):
    return (W.rotate_half(q, torch.arange(q0, q0 + q.shape[1]), theta),
            W.rotate_half(k, torch.arange(k.shape[1]), theta))


@pytest.mark.parametrize("unrotated", [False, True], ids=["rotated", "unrotated"])
@pytest.mark.parametrize("d", [64, 128])
def test_nonmonotone_table(d, unrotated):
    rng = np.random.default_rng(5)
    theta = rng.uniform(0.005, 3.0, d // 2)
    theta[[3, 17, 30]] = 0.0  # position-free pairs: never pruned
    g = torch.Generator(device="cpu").manual_seed(9)
    q = torch.randn((1, 260, 4, d), generator=g).to(torch.bfloat16)
    k, v = (torch.randn((1, 260, 2, d), generator=g).to(torch.bfloat16) for _ in range(2))
    qr, kr = _rotated(q, k, 0, torch.as_tensor(theta))
    win, widths = windows_for(d, 1e4, 3.0, theta, n_ctx=260)
    o_ref, lse_ref, _ = oracle.attend(qr, kr, v, 0, widths)
    o, lse = _many(q if unrotated else qr, k if unrotated else kr, v, 0, win, f"nonmonotone d={d}", unrotated=unrotated)
    compare(o, lse, o_ref, lse_ref, f"nonmonotone d={d}")


@pytest.mark.parametrize("pattern", ["rising", "lognormal"])
@pytest.mark.parametrize("d,h_q,h_kv", [(128, 6, 2), (64, 7, 1)])
def test_large_scores_rescale(pattern, d, h_q, h_kv):
    """Within the error budget derived from the kernel's arithmetic (parity.error_budget)."""
    q, k, v = _large_score_inputs(700, 700, 0, h_q, h_kv, d, 1e4, pattern, seed=77 + d)
    for kwin in (2.0, math.inf):
        win, widths = windows_for(d, 1e4, kwin, None, n_ctx=700)
        o_ref, lse_ref, _ = oracle.attend(q, k, v, 0, widths, scale=1.0)
        o, lse = _many(q, k, v, 0, win, f"large scores {pattern} d={d} k={kwin}", scale=1.0)
        compare_rounding_bound(o, lse, o_ref, lse_ref, prefill_budget(q, k, v, 0, widths, 1.0, o_ref),
                               f"large scores {pattern} d={d} k={kwin}")


@pytest.mark.parametrize("unrotated", [False, True], ids=["rotated", "unrotated"])
@pytest.mark.parametrize("d,group,n_q,n_k,q0", [
    (64, 128, 5, 133, 128),        # a position per workgroup
    (128, 256, 3, 100, 97),
    (128, 7, 37, 97, 2 ** 30 + 5),  # every query far past the keys
    (64, 16, 20, 131, 2 ** 30 + 5),
])
def test_wide_groups_and_far_queries(d, group, n_q, n_k, q0, unrotated):
    g = torch.Generator(device="cpu").manual_seed(group + n_q)
    q = torch.randn((1, n_q, group, d), generator=g).to(torch.bfloat16)
    k, v = (torch.randn((1, n_k, 1, d), generator=g).to(torch.bfloat16) for _ in range(2))
    theta = W.rope_theta(d, 1e6)
    if q0 > 2 ** 30:
        theta = theta.clone()
        theta[-5:] = 0.0  # some pairs reach that far
    qr, kr = _rotated(q, k, q0, theta)
    win, widths = windows_for(d, 1e6, 2.0, theta.numpy(), n_ctx=q0 + n_q)
    o_ref, lse_ref, _ = oracle.attend(qr, kr, v, q0, widths)
    o, lse = _many(q if unrotated else qr, k if unrotated else kr, v, q0, win, f"G={group} d={d}", unrotated=unrotated)
    compare(o, lse, o_ref, lse_ref, f"G={group} d={d} q0={q0}")


@pytest.mark.parametrize("unrotated", [False, True], ids=["rotated", "unrotated"])
@pytest.mark.parametrize("name,tiles,chunks", [("qwen05b_prefill_8k", 28, 4), ("llama3b_prefill_32k", 9, 3)])
def test_chunked_equals_single_shot(name, tiles, chunks, unrotated):
    """Chunks of whole position tiles, each a call that takes prefill_kernel as the whole one
    does, give the whole call's results bit for bit."""
    import paper_2608_02947_amd as atf
    wl = W.WORKLOADS[name]
    d, h_kv, group = wl.head_dim, wl.h_kv, wl.group
    chunk = (128 if d == 64 else 256) // group * tiles
    n = chunk * chunks
    win, _ = workload_window(wl)
    B = max(_batch(win, chunk, s + chunk, s, group, h_kv, unrotated) for s in range(0, n, chunk))
    assert routes.prefill_waves(win, B, n, n, 0, group, h_kv, unrotated) == 0
    note(f"chunked vs single {name} B={B} unrotated={unrotated}")
    q, k, v = (W.random_bf16((B, n, h, d), seed=s).to(DEV) for h, s in ((wl.h_q, 1), (h_kv, 2), (h_kv, 3)))
    kp, vp = pack_kcache(k), pack_vcache(v)
    fn = atf.atf_prefill_unrotated if unrotated else atf.atf_prefill

    def run(a, b):
        qc = q[:, a:b].contiguous()
        o, lse = torch.empty_like(qc), torch.empty((B, wl.h_q, b - a), dtype=torch.float32, device=DEV)
        assert routes.prefill_waves(win, B, b - a, b, a, group, h_kv, unrotated, cap=n) == 0
        fn(qc, kp, vp, o, lse, a, win, n_k=b)
        torch.cuda.synchronize()
        return o, lse

    o, lse = run(0, n)
    for s in range(0, n, chunk):
        oc, lc = run(s, s + chunk)
        assert torch.equal(oc, o[:, s:s + chunk]) and torch.equal(lc, lse[:, :, s:s + chunk]), s
