"""Which kernel serves a call and how its work is cut (host_plan: the library's
own host side, no GPU)."""

from __future__ import annotations

import random

import pytest

import test_gpu_chunk as chunk
import test_gpu_f32_matrix as f32
import test_gpu_parity as parity
from host_plan import plan


def _shapes(n, seed):
    """Random calls: (dtype, batch, hkv, group, dh, table pages, block width)."""
    rng = random.Random(seed)
    for _ in range(n):
        yield (rng.choice(["bf16", "f32"]), rng.choice([1, 1, 2, 4, 16, 48]),
               rng.choice([1, 2, 4, 8, 16, 32, 55]), rng.choice([1, 1, 2, 4, 8]),
               rng.choice([64, 96, 128]), int(2 ** rng.uniform(0, 9)), rng.randint(1, 64))


@pytest.mark.parametrize("path,kernel", [("valu", "valu"), ("mfma", "split"),
                                         ("balanced", "balanced")])
def test_a_named_path_runs_its_kernel(path, kernel):
    """A call that names a path runs that path's kernel, with the library's
    split size and with its own."""
    ran = 0
    for dtype, b, hkv, g, dh, pages, w in _shapes(400, 1):
        for pps in (0, 3):
            p = plan(dtype, b, hkv, g, dh, pages, w, path=path, pps=pps)
            if p.status == 0:
                assert p.kernel == kernel, (dtype, b, hkv, g, dh, pages, w, pps, p)
                ran += 1
    assert ran > 50


def test_default_splits_of_the_split_grid():
    """Splits the grid runs with: max(2, the power of two below T / (B * Hkv *
    row tiles)) of 2..32 pages, T = 512, or 2048 for blocks of more than 32
    rows; one more where the division leaves a remainder."""
    for (b, hkv, g, pages, w), n in (((16, 8, 1, 200, 8), 7), ((4, 8, 1, 257, 8), 17),
                                     ((4, 8, 4, 257, 32), 17), ((1, 55, 1, 33, 8), 9),
                                     ((1, 8, 1, 20, 8), 11), ((32, 8, 1, 1000, 8), 32)):
        p = plan("bf16", b, hkv, g, 128, pages, w, path="mfma")
        assert p.nsplit == n, (b, hkv, g, pages, w, p)


@pytest.mark.parametrize("dtype,hkv,group,dh,pages,w,nsplit,pps", [
    # two row tiles: even splits where the rounded-down ones pass three workgroups
    # per CU
    ("bf16", 96, 1, 64, 188, 64, 8, 24), ("bf16", 128, 1, 64, 126, 48, 8, 16),
    ("bf16", 55, 1, 96, 63, 64, 16, 4), ("bf16", 40, 1, 64, 126, 48, 19, 7),
    # four waves: past the first round, where the even ones' rounds take no more
    # pages in turn (not with three row tiles, which need a second round as
    # well), and not for a last split of one page
    ("bf16", 8, 4, 128, 469, 32, 59, 8), ("bf16", 40, 8, 96, 126, 9, 19, 7),
    ("bf16", 32, 4, 128, 257, 32, 17, 16), ("bf16", 990, 4, 64, 5, 58, 2, 3),
    ("bf16", 25, 4, 96, 328, 34, 16, 21),
    # fp32: past the first round only
    ("f32", 96, 1, 96, 126, 64, 9, 15), ("f32", 64, 1, 96, 188, 64, 16, 12)])
def test_even_splits(dtype, hkv, group, dh, pages, w, nsplit, pps):
    path = "mfma" if dtype == "bf16" else "auto"
    p = plan(dtype, 1, hkv, group, dh, pages, w, path=path)
    assert p.kernel == "split" and (p.nsplit, p.pages_per_split) == (nsplit, pps), p
    assert p.nsplit * p.pages_per_split >= pages + 1


@pytest.mark.parametrize("hkv,dh,pages,w,kernel,nsplit", [
    # one chunk per unit at any unit count
    (55, 96, 6, 1, "chunk", 1), (55, 96, 8, 8, "chunk", 1), (180, 96, 33, 8, "chunk", 1),
    # several of one tile per wave
    (24, 96, 17, 8, "chunk", 9),
    # several of more: below 16 units
    (15, 96, 129, 8, "chunk", 17), (16, 96, 129, 8, "split", 33),
    # from there where the power of two of splits leaves over 30 % of 512 waves idle
    (40, 96, 33, 8, "chunk", 6), (44, 96, 33, 8, "chunk", 5), (45, 96, 33, 8, "split", 9),
    (55, 96, 33, 8, "split", 9), (80, 96, 33, 8, "chunk", 3), (89, 96, 129, 8, "chunk", 5),
    (90, 96, 129, 8, "split", 5), (128, 96, 33, 8, "split", 5), (64, 64, 129, 17, "split", 9),
    (160, 96, 33, 8, "chunk", 3),
    # tables of one page and two row tiles
    (512, 128, 1, 31, "chunk", 1), (513, 128, 1, 31, "split", 1), (513, 128, 2, 31, "chunk", 1),
    (513, 128, 1, 16, "chunk", 1)])
def test_chunks_against_the_split_grid(hkv, dh, pages, w, kernel, nsplit):
    p = plan("bf16", 1, hkv, 1, dh, pages, w)
    assert (p.kernel, p.nsplit) == (kernel, nsplit), p


def test_calls_under_a_megabyte_take_one_launch():
    """4 heads x 256 tokens in fp32 (0.5 MB): five tiles per wave in one chunk."""
    p = plan("f32", 1, 4, 1, 64, 4, 4)
    assert (p.kernel, p.nsplit, p.merge) == ("chunk", 1, False), p


def test_any_workspace_that_was_enough_stays_enough():
    """A call's own workspace size is accepted; fp32 calls also run in the
    vector-ALU plan's, and in the library's scratch wherever either fits."""
    for dtype, b, hkv, g, dh, pages, w in _shapes(600, 2):
        p = plan(dtype, b, hkv, g, dh, pages, w)
        if p.workspace == 0:
            assert p.status < 0
            continue
        assert p.status == 0, p
        assert plan(dtype, b, hkv, g, dh, pages, w, workspace=p.workspace + 4096).status == 0
        fits = p.workspace <= 64 << 20
        if dtype == "f32":
            valu = plan(dtype, b, hkv, g, dh, pages, w, path="valu")
            assert plan(dtype, b, hkv, g, dh, pages, w, workspace=valu.workspace).status == 0
            fits = fits or valu.workspace <= 64 << 20
        assert (plan(dtype, b, hkv, g, dh, pages, w, noalloc=True).status == 0) == fits


def _pages(lens, w):
    """Columns of the block table that the GPU tests' caches have."""
    return max(max(1, -(-(s + w) // 64)) for s in lens)


@pytest.mark.parametrize("shapes,kernel", [(f32.CHUNK, "chunk"), (f32.BALANCED, "balanced"),
                                           (f32.SPLIT, "split"), (f32.PRECISION, "split")],
                         ids=["chunk", "balanced", "split", "precision"])
def test_gpu_tests_run_the_kernels_they_name(shapes, kernel):
    for lens, hkv, g, dh, w, pps in shapes:
        p = plan("f32", len(lens), hkv, g, dh, _pages(lens, w), w, pps=pps)
        assert p.kernel == kernel, (lens, hkv, g, dh, w, p)


def test_gpu_tests_of_smaller_workspaces_and_chunks():
    for hkv, lens, dh, w, kernel, fallback in f32.SMALLER_WORKSPACE:
        at = ("f32", len(lens), hkv, 1, dh, _pages(lens, w), w)
        valu = plan(*at, path="valu")
        assert plan(*at).kernel == kernel
        assert plan(*at, workspace=valu.workspace).kernel == fallback
        # what the library asks for holds the vector-ALU plan as well or not
        assert valu.status == 0
    for dtype in ("bf16", "f32"):
        for hkv, g, dh, w in chunk.FEW_TILES:
            n, pages = len(chunk.EDGES), _pages(chunk.EDGES, w)
            assert plan(dtype, n, hkv, g, dh, pages, w).kernel == "chunk"
        for lens, hkv, g, dh, w in chunk.SEVERAL_CHUNKS:
            p = plan(dtype, len(lens), hkv, g, dh, _pages(lens, w), w)
            assert p.kernel == "chunk" and p.nsplit > 1, (dtype, lens, hkv, g, dh, w, p)
    for lens, hkv, g, dh, w in parity.EVEN_SPLITS:
        p = plan("bf16", len(lens), hkv, g, dh, _pages(lens, w), w)
        assert p.kernel == "split" and p.nsplit > 1, (lens, hkv, g, dh, w, p)
