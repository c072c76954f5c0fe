"""bench.py's counting helpers against brute force on small masks (CPU only)."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


def _mask(S, cols, offs, w):
    i = np.arange(S)[:, None]
    j = np.arange(S)[None, :]
    return (j <= i) & (np.isin(j, cols) | np.isin(i - j, offs) | (i - j < w))


@pytest.mark.parametrize("S,seed", [(700, 1), (515, 2), (1024, 3), (130, 4)])
def test_counts_match_brute_force(S, seed):
    rng = np.random.default_rng(seed)
    cols = np.sort(rng.choice(S, 5, replace=False))
    offs = np.sort(rng.choice(S, 4, replace=False))
    w = 3
    M = _mask(S, cols, offs, w)
    assert bench.mask_density(S, cols, offs, w) == pytest.approx(M.sum() / (S * (S + 1) / 2.0), rel=1e-12)
    blk = 128
    nb = (S + blk - 1) // blk
    touched = sum(M[bi * blk:(bi + 1) * blk, bj * blk:(bj + 1) * blk].any()
                  for bi in range(nb) for bj in range(bi + 1))
    assert bench.touched_block_fraction(S, cols, offs, w) == pytest.approx(touched / (nb * (nb + 1) / 2.0), rel=1e-12)


@pytest.mark.parametrize("S,blk,w,seed", [(1024, 128, 128, 1), (1000, 64, 1, 2), (700, 128, 300, 3), (256, 128, 5, 4)])
def test_block_mask_density_matches_brute_force(S, blk, w, seed):
    # block (I, J) is kept when J is selected, or a full block on diagonal I - J
    # (offsets blk*(I-J) - (blk-1) .. blk*(I-J) + (blk-1)) holds a kept offset
    rng = np.random.default_rng(seed)
    nb = (S + blk - 1) // blk
    Ic = np.sort(rng.choice(nb, rng.integers(0, nb // 2 + 1), replace=False))
    Is = np.sort(rng.choice(nb, rng.integers(0, nb // 2 + 1), replace=False))
    keep_off = np.zeros((nb + 2) * blk, dtype=bool)
    for b in Is:
        keep_off[b * blk:(b + 1) * blk] = True
    keep_off[:w] = True
    kept = 0
    for bi in range(nb):
        for bj in range(bi + 1):
            lo, hi = max(blk * (bi - bj) - (blk - 1), 0), blk * (bi - bj) + blk - 1
            kept += bool(bj in Ic or keep_off[lo:hi + 1].any())
    assert bench.block_mask_density(S, Ic, Is, w, blk) == pytest.approx(kept / (nb * (nb + 1) / 2.0), rel=1e-12)


@pytest.mark.parametrize("S,seed,n_col,n_off,swept", [(700, 1, 150, 6, True), (1024, 2, 150, 6, False), (2000, 3, 150, 6, False),
                                                      (700, 4, 650, 600, True), (1985, 5, 1700, 1900, True),
                                                      (2000, 6, 2000, 0, True), (2000, 7, 0, 2000, False),
                                                      (1500, 8, 700, 1400, True), (3000, 9, 1200, 40, True)])
def test_schedule_slots_match_brute_force(S, seed, n_col, n_off, swept):
    rng = np.random.default_rng(seed)
    cols = np.sort(rng.choice(S, n_col, replace=False))
    offs = np.sort(rng.choice(S, n_off, replace=False))
    w = 5
    keep = np.zeros(S, dtype=bool)
    keep[offs] = True
    keep[:w] = True
    slots = two_pass = sweep = sweep_slots = 0
    for a in range((S + 255) // 256):
        last = min(256 * a + 255, S - 1)
        n_col = -(-int((cols <= last).sum()) // 64)
        n_rng = 0
        for d in range(4 * a + 4):                      # key tile 4 a + 3 - d >= 0
            lo, hi = max(64 * d - 255, 0), min(64 * d + 63, S - 1)
            n_rng += bool(lo <= hi and keep[lo:hi + 1].any())
            waves = 0                                   # of the tile's eight, 32 rows each: with a kept offset
            for u in range(8):
                o = np.arange(64 * d - 255 + 32 * u, 64 * d - 160 + 32 * u)
                waves += bool(keep[o[(o >= 0) & (o < S)]].any())
            two_pass += 76 + 7 * waves if waves else 0
            sweep += 140
        two_pass += 132 * n_col
        slots += 8 * (n_col + n_rng)
        sweep_slots += 8 * (last // 64 + 1)
    assert (two_pass > sweep) == swept
    slots = sweep_slots if swept else slots
    assert bench.schedule_slots(S, cols, offs, w) == slots


def test_the_result_line_stays_short():
    """The tables of the default run (16 threshold pairs on three head patterns, sweeps, blocks) in fewer than 6000 characters,
    nothing lost but digits after the sixth."""
    import json
    rng = np.random.default_rng(0)
    names = ("sparse_flash_ms", "computed_tile_fraction", "mask_density_head0", "mean_k_c", "mean_k_s", "recall_mean", "cra_min")
    grid = [{"head_pattern": p, "alpha_c": a, "alpha_s": b, **{n: float(rng.random()) * 10 ** int(rng.integers(-2, 5)) for n in names}}
            for p in ("column", "slash", "composed") for a in (0.0, 0.8, 0.9, 0.95) for b in (0.0, 0.8, 0.9, 0.95)]
    line = {"grid": grid, "nested": {"t": [1.23456789, 2]}, "one": [{"a": 1}], "none": None}
    got = bench.compact(line)
    assert len(json.dumps(line)) > 10000 and len(json.dumps(got)) < 6000
    rows = [dict(zip(got["grid"]["columns"], r)) for r in got["grid"]["rows"]]
    assert rows == [{k: v if isinstance(v, str) else pytest.approx(v, rel=1e-5) for k, v in r.items()} for r in grid]
    assert got["nested"] == {"t": [1.23457, 2]} and got["one"] == [{"a": 1}] and got["none"] is None
