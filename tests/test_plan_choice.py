"""Which kernel serves a call and how its work is cut (host_plan: the library's
own host side, no GPU)."""

from __future__ import annotations

import random

import pytest

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
