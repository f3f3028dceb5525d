"""The tiles of quake_linear_gelu and the rule that picks one, read from the
kernel's source: the same estimate in the same order, for tests that have to
know which tile a shape takes."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = open(os.path.join(ROOT, "paper_2412_00408_amd", "csrc", "gemm.hip")).read()

# (bm, bn, threads, first, slab, next, next_slab, out, load, split, gelu)
_ROWS = SRC[SRC.index("constexpr Tile kTiles[]"):SRC.index("inline int pick_tile")]
TILES = [tuple(float(v.rstrip("f")) for v in row.split(","))
         for row in re.findall(r"\{(\d+, \d+, [^}]*)\}", _ROWS)]
FIRST_ONE = int(re.search(r"kFirstOne = (\d+);", SRC).group(1))
# (bm, bn, waves in m, waves in n, stages of x, stages of w)
LAUNCHES = [tuple(map(int, v)) for v in re.findall(
    r"launch_tile<DT, (\d+), (\d+), (\d+), (\d+), (\d+), (\d+)>\(g, s\)", SRC)]


def slabs(k):
    return -(-k // 64)


def pick(m, n, k, gelu=True, split=None, cus=256):
    """The tile's index; split: rows of x or w (stride k if not given) off 128-byte lines."""
    split = k % 64 != 0 if split is None else split
    s, best, best_us = slabs(k), 0, -1.0
    fits = [-(-m // int(t[0])) * -(-n // int(t[1])) * t[2] < 2 ** 32 for t in TILES]
    one = k <= 64 and fits[FIRST_ONE]
    for i, (bm, bn, _, first, slab, nxt, nxt_slab, out, load, spl, ge) in enumerate(TILES):
        if (i >= FIRST_ONE) != one or not fits[i]:
            continue
        tiles = -(-m // int(bm)) * -(-n // int(bn))
        us = (first + s * slab + (-(-tiles // cus) - 1) * (nxt + s * nxt_slab) +
              tiles / cus * (out + (ge if gelu else 0.0) + s * (load + (spl if split else 0.0))))
        if best_us < 0 or us < best_us:
            best, best_us = i, us
    return best
