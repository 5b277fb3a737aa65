"""The workgroup-per-chunk kernel (the library's choice for units of few tiles):
one to four waves with tiles, one or several chunks per unit, one or several
row tiles sharing a chunk's keys and values, chunks without a readable page.
Against the fp64 oracle."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from gpu_common import assert_close, assert_lse_close, oracle_call, wrap
from oracle import das_oracle as orc
from paper_2609_34538_amd import _lib as das
from paper_2609_34538_amd import datagen as dg

pytestmark = pytest.mark.gpu
DEV = "cuda"
EDGES = [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 130]


def _data(lens, dtype, hkv, group, dh, w):
    wl = dg.scaled(dg.WORKLOADS[3], dtype=dtype, batch=len(lens), hq=hkv * group, hkv=hkv, dh=dh,
                   layers=1, prefix=(0, max(lens)), draft_depths=(2,), draft_widths=(w,),
                   verify_width=w, paged_random=True)
    cd = dg.make_cache(wl, DEV, prefix_lens=lens)
    return wl, cd, dg.block_inputs(cd, w, 2, DEV)


def _check(wl, cd, batch_args, what):
    cache, batch = wrap(cd)
    q, kb, vb = batch_args
    lse = torch.empty((wl.batch, wl.hq, q.shape[1]), dtype=torch.float32, device=DEV)
    out = das.attn_policy(cache, batch, 0, 2, wl.depth_R, q, kb, vb, lse=lse)
    ref, ref_lse = oracle_call(cd, 0, 2, wl.depth_R, q, kb, vb, range(wl.batch))
    assert_close(out, ref, wl.dtype, what)
    assert_lse_close(lse, ref_lse, what + " lse")


# (KV heads, group, head dim, block width) over EDGES
FEW_TILES = [(1, 1, 64, 1), (3, 1, 96, 16), (2, 1, 128, 33), (3, 1, 64, 64), (1, 8, 96, 2),
             (3, 5, 128, 13), (2, 8, 64, 15), (30, 1, 96, 7)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
@pytest.mark.parametrize("hkv,group,dh,w", FEW_TILES)
def test_few_tiles(dtype, hkv, group, dh, w):
    wl, cd, args = _data(EDGES, dtype, hkv, group, dh, w)
    _check(wl, cd, args, f"{dtype} hkv={hkv} G={group} dh={dh} w={w}")


SEVERAL_CHUNKS = [([3000, 5, 0, 1111], 2, 1, 96, 9), ([9001], 1, 4, 128, 4),
                  ([1200, 700], 3, 2, 64, 25), ([2500, 64], 3, 8, 128, 10),
                  ([40000], 1, 1, 64, 1)]


# the last shape: chunks in fp32, the shared ring in bf16
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
@pytest.mark.parametrize("lens,hkv,group,dh,w", SEVERAL_CHUNKS + [([5000, 700], 3, 2, 64, 25)])
def test_several_chunks(dtype, lens, hkv, group, dh, w):
    wl, cd, args = _data(lens, dtype, hkv, group, dh, w)
    _check(wl, cd, args, f"{dtype} lens={lens} hkv={hkv} G={group} dh={dh} w={w}")


@pytest.mark.parametrize("low", [False, True], ids=["random", "low-logits"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
def test_chunks_without_a_readable_page(dtype, low):
    """Pages 1..20 of a sequence are outside the pool: whole chunks see no
    position, and count with weight 0 also where every logit is far below 0."""
    wl, cd, (q, kb, vb) = _data([3000, 90], dtype, 2, 1, 96, 16)
    if low:
        cd.k_pool.zero_()
        cd.k_pool[..., 0] = 1.0
        for t, x in ((q, -1536.0), (kb, 1.0)):
            t.zero_()
            t[..., 0] = x
    table = cd.block_table.copy()
    table[0, 1:21] = cd.k_pool.shape[3] + np.arange(20)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    cache, batch = wrap(cd, table=table, dev_error=err)
    out = das.attn_policy(cache, batch, 0, 2, wl.depth_R, q, kb, vb)
    assert int(err.item()) == das.DEVERR_PAGE
    ref = []
    for b, s in enumerate([3000, 90]):
        kc = dg.gather_prefix_k(cd, b, cd.k_plane[2], 0, s)
        vc = dg.gather_prefix_v(cd, b, cd.v_plane[wl.depth_R], 0, s)
        keep = np.ones(s, dtype=bool)
        if b == 0:
            keep[64:64 * 21] = False
        ref.append(orc.policy_attention(q[b].double().cpu().numpy(), kc[keep], vc[keep],
                                        kb[b].double().cpu().numpy(),
                                        vb[b].double().cpu().numpy())[0])
    assert_close(out, np.stack(ref), dtype, f"unreadable chunks low={low}")


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
def test_positions_past_the_prefix_add_nothing(dtype):
    lens = [1500, 70, 0]
    wl, cd, (q, kb, vb) = _data(lens, dtype, 2, 1, 128, 5)
    cache, batch = wrap(cd)
    clean = das.attn_policy(cache, batch, 0, 2, wl.depth_R, q, kb, vb).clone()
    for b, s in enumerate(lens):
        page, r = int(cd.block_table[b][s // 64]), s % 64
        cd.k_pool[:, :, :, page, r:] = float("nan")
        cd.v_pool[:, :, :, page].masked_fill_(
            (torch.arange(64, device=DEV) >= r).view(8, 1, 8), float("inf"))
    assert torch.equal(clean, das.attn_policy(cache, batch, 0, 2, wl.depth_R, q, kb, vb))


@pytest.mark.parametrize("scale", [2.0 ** -100, 3.0e5, 2.0 ** 100])
def test_records_over_value_magnitudes(scale):
    """bf16 chunk records hold O / l in fp16 under a per-row power of two."""
    wl, cd, (q, kb, vb) = _data([9001], torch.bfloat16, 1, 4, 96, 4)
    cd.v_pool.mul_(scale)
    cache, batch = wrap(cd)
    out = das.attn_policy(cache, batch, 0, 2, wl.depth_R, q, kb, (vb.float() * scale).to(vb.dtype))
    ref_s, _ = oracle_call(cd, 0, 2, wl.depth_R, q, kb, (vb.float() * scale).to(vb.dtype), [0])
    assert_close(out.float() / scale, ref_s / scale, torch.bfloat16, f"values x {scale}")
