"""fp32 attention on the matrix cores (the library's choice for fp32 caches):
16-token tiles, so the edges are 16 tokens, 16 and 32 query rows, and 64 rows
for the waves that share a tile. Against the fp64 oracle at the fp32 tolerance
(1e-5), and against the vector-ALU kernel."""

from __future__ import annotations

import pytest
import torch

from gpu_common import assert_close, assert_lse_close, oracle_call, wrap
from paper_2609_34538_amd import _lib as das
from paper_2609_34538_amd import datagen as dg

pytestmark = pytest.mark.gpu
DEV = "cuda"
EDGES = [0, 1, 15, 16, 17, 63, 64, 65, 130]


def _data(lens, hkv, group, dh, w):
    wl = dg.scaled(dg.WORKLOADS[3], dtype=torch.float32, batch=len(lens), hq=hkv * group, hkv=hkv,
                   dh=dh, layers=1, prefix=(0, max(lens)), draft_depths=(2,), draft_widths=(w,),
                   verify_width=w, paged_random=True)
    cd = dg.make_cache(wl, DEV, prefix_lens=lens)
    return (wl, cd) + wrap(cd) + dg.block_inputs(cd, w, 2, DEV)


# hkv 2: the split grid; 26 and more heads for 9 sequences: the balanced
# schedule for blocks of up to 32 rows (16 at head dim 128)
@pytest.mark.parametrize("hkv,group,dh,w", [
    (2, 1, 64, 17), (2, 1, 96, 64), (2, 8, 128, 3), (2, 5, 96, 13), (2, 8, 128, 17),
    (2, 4, 64, 33), (26, 1, 64, 16), (26, 1, 64, 31), (26, 2, 96, 8), (26, 1, 96, 32),
    (26, 4, 128, 4), (26, 1, 128, 17)])
def test_matches_oracle(hkv, group, dh, w):
    wl, cd, cache, batch, q, kb, vb = _data(EDGES, hkv, group, dh, w)
    lse = torch.empty((wl.batch, wl.hq, w), dtype=torch.float32, device=DEV)
    out = das.attn_policy(cache, batch, 0, 2, wl.depth_R, q, kb, vb, lse=lse)
    ref, ref_lse = oracle_call(cd, 0, 2, wl.depth_R, q, kb, vb, range(wl.batch))
    assert_close(out, ref, torch.float32, f"f32 hkv={hkv} G={group} dh={dh} w={w}")
    assert_lse_close(lse, ref_lse, "f32 lse")


@pytest.mark.parametrize("hkv,lens", [(2, [9000, 700]), (160, [700, 3000])])
def test_many_partials_and_smaller_workspace(hkv, lens):
    """Many splits or pieces per unit; a workspace that holds only the
    vector-ALU plan's partials is still accepted."""
    wl, cd, cache, batch, q, kb, vb = _data(lens, hkv, 1, 64, 20)
    ref, _ = oracle_call(cd, 0, 2, wl.depth_R, q, kb, vb, range(wl.batch))
    for path in ("auto", "valu"):
        ws = das.alloc_workspace(cache, batch, wl.hq, 20, path)
        out = das.attn_policy(cache, batch, 0, 2, wl.depth_R, q, kb, vb, workspace=ws)
        assert_close(out, ref, torch.float32, f"f32 hkv={hkv}, workspace of {path}")


def test_invisible_positions_and_bad_pages():
    """NaN and Inf past the prefix and on pages outside the pool add nothing."""
    wl, cd, cache, batch, q, kb, vb = _data([70, 16, 129], 90, 1, 96, 20)
    clean = das.attn_policy(cache, batch, 0, 2, wl.depth_R, q, kb, vb).clone()
    pos = {0: 70, 1: 16, 2: 129}
    for b, s in pos.items():
        page = int(cd.block_table[b][s // 64])
        r = s % 64
        cd.k_pool[:, :, :, page, r:] = float("nan")
        v = cd.v_pool[:, :, :, page]  # [nV, L, Hkv, 8, dh, 8]
        mask = (torch.arange(64, device=DEV) >= r).view(8, 1, 8)
        v.masked_fill_(mask, float("inf"))
    assert torch.equal(clean, das.attn_policy(cache, batch, 0, 2, wl.depth_R, q, kb, vb))
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    table = cd.block_table.copy()
    table[2][0] = cd.k_pool.shape[3]
    _, bad = wrap(cd, table=table, dev_error=err)
    out = das.attn_policy(cache, bad, 0, 2, wl.depth_R, q, kb, vb)
    assert int(err.item()) & das.DEVERR_PAGE and torch.isfinite(out).all()
    assert torch.equal(out[:2], clean[:2])


# one to four waves, every head dim, one and two row tiles in one wave
PRECISION = [([4000, 2000], 8, 4, 128, 8, 8), ([4000, 2000], 8, 4, 128, 5, 4),
             ([3000, 1500], 4, 2, 128, 16, 8), ([2000, 1000], 4, 4, 128, 16, 8),
             ([2000, 1000], 4, 8, 128, 12, 8), ([3000, 1500], 8, 4, 96, 8, 8),
             ([3000, 1500], 8, 4, 64, 5, 8), ([3000, 1500], 24, 1, 128, 16, 8)]


@pytest.mark.parametrize("lens,hkv,group,dh,w,pps", PRECISION)
def test_split_grid_no_less_precise_than_the_vector_kernel(lens, hkv, group, dh, w, pps):
    """Keys three times the usual size: the logits' rounding dominates. Relative
    2-norm error against 64 bits, matrix cores and vector ALU on the same inputs."""
    wl, cd, cache, batch, q, kb, vb = _data(lens, hkv, group, dh, w)
    cd.k_pool.mul_(3.0)
    kb = kb * 3.0
    ref, _ = oracle_call(cd, 0, 2, wl.depth_R, q, kb, vb, range(2))
    ref = torch.as_tensor(ref, device=DEV)
    err = {}
    for path in ("auto", "valu"):
        out = das.attn_policy(cache, batch, 0, 2, wl.depth_R, q, kb, vb, path=path,
                              pages_per_split=pps)
        err[path] = float((out.double() - ref).norm() / ref.norm())
    assert err["auto"] <= err["valu"], err
