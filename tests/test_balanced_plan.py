"""The balanced attention plan's arithmetic on the CPU: a model of bal_share, bal_item and
attn_pair_slots (csrc/attn.hpp), constants read from the source, over random ragged batches.  Every
key tile goes to exactly one workgroup, a pair's pieces hold consecutive partial slots from the merge's
first one, no two pieces share a slot, and the slots stay within those the workspace has."""
import os
import re

import numpy as np
import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_31315_amd", "csrc")
ATTN = open(os.path.join(SRC, "attn.hpp")).read()
GRID = int(re.search(r"constexpr int kBalGrid = (\d+);", ATTN).group(1))
COST = int(re.search(r"constexpr int kBalPairCost = (\d+);", ATTN).group(1))
W8 = int(re.search(r"constexpr int kBalWeightMax8 = (\d+);", ATTN).group(1))
KW = [int(x) for x in re.search(r"kw\[9\] = \{([\d, ]+), kBalWeightMax8\}", ATTN).group(1).split(",")] + [W8]
MIN_TILES = int(re.search(r"constexpr int kBalMinTiles = (\d+);",
                          open(os.path.join(SRC, "sd_block.hip")).read()).group(1))
KT = 64


def weight(nmt):
    return KW[nmt] if nmt <= 8 else W8 + 4 * (nmt - 8)


def tile_at(u, p0, w):
    return 0 if u <= p0 else -(-(u - p0) // w)


@pytest.mark.parametrize("seed", range(12))
def test_every_tile_once_and_slots_agree(seed):
    rng = np.random.default_rng(seed)
    for _ in range(12):
        S, Hkv, G = int(rng.integers(1, 100)), int(rng.choice([1, 2, 4, 8])), int(rng.choice([1, 4, 8]))
        ctx = rng.integers(0, int(rng.choice([300, 3000, 33000])), S)
        B = np.where(rng.random(S) < 0.1, 0, rng.integers(1, min(64, 256 // G) + 1, S))
        tiles = np.where(B > 0, -(-(ctx + B) // KT), 0)
        w = np.array([weight(int(G * b + 15) // 16) for b in B])
        units = np.where(tiles > 0, tiles * w + COST, 0)
        starts = np.concatenate([[0], np.cumsum(units * Hkv)])
        total = int(starts[-1])
        per = max(-(-total // GRID), MIN_TILES * weight(1))
        assert COST + w.max() < per  # a workgroup between a pair's first and last holds a tile of it
        first = {}  # (s, g): the merge's first slot and split count
        for s in range(S):
            for g in range(Hkv):
                if B[s] > 0:
                    p0 = int(starts[s] + g * units[s]) + COST
                    wf, wl = p0 // per, (p0 + int(tiles[s] - 1) * int(w[s])) // per
                    first[s, g] = (wf + s * Hkv + g, wl - wf + 1)
        seen, slots = {}, set()
        for wg in range(GRID):
            u0 = min(wg * per, total)
            u1 = min(u0 + per, total)
            while u0 < u1:
                s = int(np.searchsorted(starts, u0, side="right")) - 1
                while units[s] == 0:
                    s += 1
                g = int(u0 - starts[s]) // int(units[s])
                p0 = int(starts[s] + g * units[s]) + COST
                j0 = tile_at(u0, p0, int(w[s]))
                if j0 >= tiles[s]:
                    u0 = p0 + int(tiles[s] * w[s])
                    continue
                if p0 + j0 * w[s] >= u1:
                    break
                j1 = min(tile_at(u1, p0, int(w[s])), int(tiles[s]))
                assert j1 > j0
                assert (p0 + j0 * int(w[s])) // per == wg  # the kernel takes its own index for this
                slot = wg + s * Hkv + g
                base, n = first[s, g]
                assert base <= slot < base + n and slot not in slots
                assert 0 <= slot < GRID + S * Hkv
                slots.add(slot)
                for j in range(j0, j1):
                    assert (s, g, j) not in seen
                    seen[s, g, j] = wg
                u0 = p0 + j1 * int(w[s])
        assert len(seen) == int((tiles * Hkv).sum())
        assert len(slots) == sum(n for _, n in first.values())
