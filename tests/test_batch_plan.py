"""The batched step's tile shape, kernel and placement over random batches (host code)."""
import random

import pytest

from batch_form import form, place


@pytest.mark.parametrize("seed", range(60))
def test_every_tile_once(seed):
    """Each (instance, 128 rows, replica tile) is launched once, whatever shape and placement."""
    rng = random.Random(seed)
    n = rng.choice([1, 2, 5, 9, 24, 60])
    lo = rng.choice([1, 100, 1000])
    sizes = [rng.randint(lo, rng.choice([lo, 2 * lo, 4000])) if lo < 4000 else lo for _ in range(n)]
    kinds = [rng.choice(["bf16", "fp8", "bit"]) for _ in sizes]
    R = rng.choice([1, 15, 16, 17, 33, 64, 65, 96, 100, 257])
    f = form(sizes, kinds, R)
    reps = 16 * int(f[-1]) if f.startswith("narrow") else 64
    for f32 in (False, True):
        w = 64 if f32 else reps
        tiles = place(sizes, kinds if not f32 else ["f32"] * n, R, w, f32)
        want = sorted((k, i0, r0) for k, N in enumerate(sizes) for i0 in range(0, N, 128)
                      for r0 in range(0, R, w))
        assert sorted(t for t in tiles if t[0] >= 0) == want
        assert all(t == (-1, 0, 0) for t in tiles if t[0] < 0)
        assert len(tiles) % 8 == 0


@pytest.mark.parametrize("sizes,kinds,R,want", [
    ([8192], ["fp8"], 512, "cached"),                    # 512 tiles, 151 MB
    ([8192], ["bf16"], 512, "cached"),
    ([2048], ["bf16"], 2048, "narrow 4"),
    ([260], ["fp8"], 64 * 200 + 37, "cached"),
    ([800], ["fp8"], 64, "narrow 1"),
    ([654] * 38, ["bf16"] * 38, 200, "narrow 4"),        # 912 tiles of few groups
    ([1200] * 30, ["fp8"] * 30, 64, "narrow 4"),
    ([215] * 34, ["fp8"] * 34, 200, "narrow 2"),
    ([2800] * 60, ["bf16"] * 30 + ["fp8"] * 30, 256, "streamed"),
    ([300] * 8, ["bf16"] * 8, 16, "narrow 1")])
def test_kernel_by_size(sizes, kinds, R, want):
    assert form(sizes, kinds, R) == want


def test_placement_by_balance():
    """Many equal small instances stay whole on an XCD (workgroup b on XCD b mod 8); nine large ones,
    two of them on one XCD otherwise, go tile by tile."""
    def xcds(sizes, R):
        tiles = place(sizes, ["fp8"] * len(sizes), R, 64)
        return [{b % 8 for b, t in enumerate(tiles) if t[0] == k} for k in range(len(sizes))]
    assert all(len(x) == 1 for x in xcds([148] * 32, 256))
    assert all(len(x) == 8 for x in xcds([1947] * 9, 256))


@pytest.mark.parametrize("sizes,kinds,R,want", [
    ([1351] * 1115, ["bit"] * 1115, 64, "narrow 4"),     # 1.9 GB of state, 0.2 of couplings
    ([1351] * 500, ["bit"] * 500, 64, "streamed"),       # 0.9 GB
    ([1376] * 227, ["fp8"] * 227, 256, "narrow 4"),      # couplings 0.29 of the state
    ([1376] * 227, ["bf16"] * 227, 256, "streamed"),     # 0.57 of it
    ([600] * 2400, ["bf16", "bit"] * 1200, 64, "streamed"),   # one bit in half of the tiles
    ([1000] * 200 + [2750] * 220, ["bf16"] * 200 + ["bit"] * 220, 64, "narrow 4"),   # in three of four
    ([8192], ["bit"], 64 * 200, "streamed")])            # one instance
def test_kernel_of_large_batches(sizes, kinds, R, want):
    assert form(sizes, kinds, R) == want
