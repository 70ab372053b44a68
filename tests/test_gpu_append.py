"""The append kernel where a call meets the edges of its 16-token blocks: one token at a
time across a block's edge, whole blocks, and pieces that begin or end inside one, into
contiguous and paged caches; every byte of both caches against the packs of the whole
sequence, the other slots keeping a sentinel."""
import pytest
import torch

from conftest import gpu_available
import workloads as W
from parity import note
from test_gpu_decode import _ref_pack, _ref_vpack

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

DEV = "cuda"


@pytest.mark.parametrize("paged", [False, True], ids=["contiguous", "paged"])
@pytest.mark.parametrize("B,h_kv,d", [(1, 1, 64), (3, 5, 128)])
@pytest.mark.parametrize("cuts", [(14, 15, 16, 17), (16, 32, 48), (3, 16, 33, 95, 96, 128)])
def test_append_block_edges(B, h_kv, d, cuts, paged):
    import paper_2608_02947_amd as atf
    n, pt = 128, 32
    note(f"append edges {B} {h_kv} {d} {cuts} paged={paged}")
    k = W.random_bf16((B, n, h_kv, d), seed=31).to(DEV)
    v = W.random_bf16((B, n, h_kv, d), seed=32).to(DEV)
    lo, hi = cuts[0], cuts[-1]
    full = lambda shape: torch.full(shape, -7.0, dtype=torch.bfloat16, device=DEV)
    kw, vw = full(k.shape), full(v.shape)
    kw[:, lo:hi], vw[:, lo:hi] = k[:, lo:hi], v[:, lo:hi]
    kref, vref = _ref_pack(kw), _ref_vpack(vw)
    if paged:
        order = torch.randperm(B * n // pt, generator=torch.Generator().manual_seed(1))
        table = order.view(B, n // pt).to(torch.int32).to(DEV)
        kc = full(atf.kpages_shape(B * n // pt, pt, h_kv, d))
        vc = full(atf.vpages_shape(B * n // pt, pt, h_kv, d))
        append = lambda a, b: atf.atf_cache_append_paged(
            k[:, a:b].contiguous(), v[:, a:b].contiguous(), kc, vc, table, a)
        # page i of a row holds its tokens pt i .. pt i + pt - 1
        at = table.view(-1).long()
        kref = kref.view(B, h_kv, d // 16, n // pt, pt, 16).permute(0, 3, 1, 2, 4, 5).reshape(-1, h_kv, d // 16, pt, 16)
        vref = vref.view(B, h_kv, n // pt, pt // 16, d, 16).permute(0, 2, 1, 3, 4, 5).reshape(-1, h_kv, pt // 16, d, 16)
        got = lambda c: c[at]
    else:
        kc, vc = full(kref.shape), full(vref.shape)
        append = lambda a, b: atf.atf_cache_append(k[:, a:b].contiguous(), v[:, a:b].contiguous(), kc, vc, a)
        got = lambda c: c
    for a, b in zip(cuts[:-1], cuts[1:]):
        append(a, b)
    torch.cuda.synchronize()
    assert torch.equal(got(kc).view(torch.int16), kref.view(torch.int16))
    assert torch.equal(got(vc).view(torch.int16), vref.view(torch.int16))
