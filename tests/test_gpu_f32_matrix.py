"""fp32 attention on the matrix cores (the library's choice for fp32 caches):
16-token tiles, so the edges are 16 tokens, 16 and 32 query rows, and 64 rows
for the waves that share a tile. Against the fp64 oracle at the fp32 tolerance
(1e-5), and against the vector-ALU kernel. Which kernel each shape runs is
asserted without a GPU in test_plan_choice."""

from __future__ import annotations

import pytest
import torch

from gpu_common import assert_close, assert_lse_close, oracle_call, wrap
from paper_2609_34538_amd import _lib as das
from paper_2609_34538_amd import datagen as dg

pytestmark = pytest.mark.gpu
DEV = "cuda"
EDGES = [0, 1, 15, 16, 17, 63, 64, 65, 130]

# (prefix lengths, KV heads, group, head dim, block width, pages per split)
CHUNK = [(EDGES, *x, 0) for x in (
    (2, 1, 64, 17), (2, 1, 96, 64), (2, 8, 128, 3), (2, 5, 96, 13), (2, 8, 128, 17),
    (2, 4, 64, 33), (26, 1, 64, 16), (26, 1, 64, 31), (26, 2, 96, 8), (26, 1, 96, 32),
    (26, 4, 128, 4), (26, 1, 128, 17))]
# one and two row tiles (one at head dim 128); the workers' ranges begin and end
# inside units, so a piece waits in LDS
BALANCED = [([3400, 33, 700], 80, 1, 64, 16, 0), ([3400, 0, 700], 66, 1, 64, 31, 0),
            ([2300, 64, 705], 55, 1, 96, 7, 0), ([2300, 1, 640], 44, 4, 96, 8, 0),
            ([1700, 129, 0], 33, 1, 128, 16, 0), ([1700, 15, 64], 33, 4, 128, 3, 0)]
# one wave with one and two row tiles, two and four waves
SPLIT = [([1900, 0, 640], 24, 1, 64, 16, 4), ([1900, 1, 640], 24, 2, 96, 5, 3),
         ([1900, 65, 640], 24, 1, 128, 9, 7), ([700, 130], 2, 1, 64, 31, 2),
         ([700, 130], 2, 1, 128, 20, 2), ([1000, 17, 300], 2, 5, 96, 13, 2),
         ([700, 64], 3, 4, 64, 13, 2), ([700, 1], 2, 2, 128, 32, 2),
         ([1000, 0, 300], 2, 8, 128, 17, 3), ([700, 64], 3, 4, 64, 33, 2)]


def _data(lens, hkv, group, dh, w):
    wl = dg.scaled(dg.WORKLOADS[3], dtype=torch.float32, batch=len(lens), hq=hkv * group, hkv=hkv,
                   dh=dh, layers=1, prefix=(0, max(lens)), draft_depths=(2,), draft_widths=(w,),
                   verify_width=w, paged_random=True)
    cd = dg.make_cache(wl, DEV, prefix_lens=lens)
    return (wl, cd) + wrap(cd) + dg.block_inputs(cd, w, 2, DEV)


@pytest.mark.parametrize("lens,hkv,group,dh,w,pps", CHUNK + BALANCED + SPLIT)
def test_matches_oracle(lens, hkv, group, dh, w, pps):
    wl, cd, cache, batch, q, kb, vb = _data(lens, hkv, group, dh, w)
    lse = torch.empty((wl.batch, wl.hq, w), dtype=torch.float32, device=DEV)
    out = das.attn_policy(cache, batch, 0, 2, wl.depth_R, q, kb, vb, lse=lse, pages_per_split=pps)
    ref, ref_lse = oracle_call(cd, 0, 2, wl.depth_R, q, kb, vb, range(wl.batch))
    assert_close(out, ref, torch.float32, f"f32 hkv={hkv} G={group} dh={dh} w={w} pps={pps}")
    assert_lse_close(lse, ref_lse, "f32 lse")


# what runs in the library's own workspace and in the vector-ALU plan's
SMALLER_WORKSPACE = [(2, [9000, 700], 64, 20, "chunk", "chunk"),
                     (160, [700, 3000], 64, 20, "chunk", "chunk"),
                     (160, [700, 4200], 64, 20, "balanced", "valu"),
                     (140, [700, 4200], 128, 24, "split", "valu")]


@pytest.mark.parametrize("hkv,lens,dh,w,kernel,fallback", SMALLER_WORKSPACE)
def test_many_partials_and_smaller_workspace(hkv, lens, dh, w, kernel, fallback):
    """Many splits or pieces per unit; a workspace that holds only the
    vector-ALU plan's partials is still accepted."""
    wl, cd, cache, batch, q, kb, vb = _data(lens, hkv, 1, dh, w)
    ref, _ = oracle_call(cd, 0, 2, wl.depth_R, q, kb, vb, range(wl.batch))
    for path in ("auto", "valu"):
        ws = das.alloc_workspace(cache, batch, wl.hq, w, path)
        out = das.attn_policy(cache, batch, 0, 2, wl.depth_R, q, kb, vb, workspace=ws)
        assert_close(out, ref, torch.float32, f"f32 hkv={hkv}, workspace of {path}")


@pytest.mark.parametrize("lens,hkv,dh,pps", [([70, 16, 129], 90, 96, 0),
                                             ([2300, 16, 129], 55, 96, 0),
                                             ([2300, 16, 129], 6, 128, 2)])
def test_invisible_positions_and_bad_pages(lens, hkv, dh, pps):
    """NaN and Inf past the prefix and on pages outside the pool add nothing:
    chunks, balanced schedule, split grid (values read after the logits)."""
    wl, cd, cache, batch, q, kb, vb = _data(lens, hkv, 1, dh, 20)
    call = lambda bt: das.attn_policy(cache, bt, 0, 2, wl.depth_R, q, kb, vb,  # noqa: E731
                                      pages_per_split=pps)
    clean = call(batch).clone()
    for b, s in enumerate(lens):
        page = int(cd.block_table[b][s // 64])
        r = s % 64
        cd.k_pool[:, :, :, page, r:] = float("nan")
        v = cd.v_pool[:, :, :, page]  # [nV, L, Hkv, 8, dh, 8]
        mask = (torch.arange(64, device=DEV) >= r).view(8, 1, 8)
        v.masked_fill_(mask, float("inf"))
    assert torch.equal(clean, call(batch))
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    table = cd.block_table.copy()
    table[2][0] = cd.k_pool.shape[3]
    _, bad = wrap(cd, table=table, dev_error=err)
    out = call(bad)
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
