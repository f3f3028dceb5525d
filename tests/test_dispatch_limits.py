"""The softmax kernels' row-length limits and the linear+GELU tiles as the
source defines them, checked against the limits the C header documents and the
boundaries and tiles the GPU tests exercise (CPU only; reads the sources, runs
nothing)."""
import os
import re

import gemm_tiles
from test_gpu_linear import TILE_SHAPES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = open(os.path.join(ROOT, "paper_2412_00408_amd", "csrc", "softmax.hip")).read()
HDR = open(os.path.join(ROOT, "include", "quake.h")).read()


def _int(pattern):
    return int(re.search(pattern, SRC).group(1))


def _shape():
    m = re.search(r"struct ResShape \{(.*?)\};", SRC, re.S).group(1)
    f = {k: (int(a), int(b)) for k, a, b in re.findall(r"(NK2|NK1|NL1) = \(DT == F32\) \? (\d+) : (\d+);", m)}
    return f


def test_resident_capacity_matches_the_header():
    block = _int(r"constexpr int kResBlock = (\d+);")
    s = _shape()
    f32 = (s["NK1"][0] + s["NL1"][0]) * block * 4
    b16 = (s["NK1"][1] + s["NL1"][1]) * block * 8
    assert (f32, b16) == (129024, 131072)
    text = " ".join(" ".join(l.strip().lstrip("*") for l in HDR.splitlines()).split())
    assert "up to 129024 (binary32) or 131072 (16-bit) elements" in text


def test_resident_lds_and_register_shapes_fit():
    block = _int(r"constexpr int kResBlock = (\d+);")
    s = _shape()
    for i, v in ((0, 4), (1, 8)):
        lds = s["NL1"][i] * block * v * 4 + (block // 64) * (4 + 8)
        assert lds <= 160 * 1024
        # the register shapes nest: two workgroups per CU, then one, then LDS
        assert s["NK2"][i] < s["NK1"][i]


def test_gpu_tests_cover_each_resident_shape_boundary():
    src = open(os.path.join(ROOT, "tests", "test_gpu_softmax.py")).read()
    cols = re.search(r"RESIDENT_COLS = \{(.*?)\}\n", src, re.S).group(1)
    f32 = [int(c) for c in re.search(r'"f32": \[([^\]]*)\]', cols).group(1).split(",")]
    bf = [int(c) for c in re.search(r'"bf16": \[([^\]]*)\]', cols).group(1).split(",")]
    block = _int(r"constexpr int kResBlock = (\d+);")
    s = _shape()
    for lst, i, v in ((f32, 0, 4), (bf, 1, 8)):
        for n in (s["NK2"][i], s["NK1"][i], s["NK1"][i] + s["NL1"][i]):
            last = n * block * v
            assert last in lst and last + v in lst, (v, last)


def test_split_chunk_is_the_documented_16384():
    assert _int(r"constexpr int64_t kChunkElems = (\d+);") == 16384
    assert "ceil(cols / 16384)" in HDR


def test_gemm_table_and_launches_agree():
    assert len(gemm_tiles.TILES) == len(gemm_tiles.LAUNCHES) == 14
    for i, (row, (bm, bn, wm, wn, sa, sb)) in enumerate(zip(gemm_tiles.TILES, gemm_tiles.LAUNCHES)):
        assert row[:3] == (bm, bn, 64 * wm * wn)
        assert (i >= gemm_tiles.FIRST_ONE) == ((sa, sb) == (1, 1))
        assert 128 * (sa * bm + sb * bn) <= 160 * 1024


def test_gemm_one_slab_takes_one_stage_and_huge_grids_fit():
    for m, n in ((1, 1), (37, 3072), (4096, 768), (16384, 4096), (2 ** 30, 8), (2 ** 31 - 200, 8),
                 (2 ** 31 - 300, 128)):
        for k in (8, 64, 72, 128, 4096):
            i = gemm_tiles.pick(m, n, k)
            bm, bn, threads = gemm_tiles.TILES[i][:3]
            assert -(-m // int(bm)) * -(-n // int(bn)) * threads < 2 ** 32
            assert (i >= gemm_tiles.FIRST_ONE) == (k <= 64 and m < 2 ** 30)


def test_gpu_tests_cover_every_gemm_tile():
    """Each tile with rows of y aligned and not, with at least as many slabs as
    its stages, and (where some shape of the range is given fewer) with fewer."""
    seen = {}
    for m, n, k in TILE_SHAPES:
        for gelu in (True, False):
            i = gemm_tiles.pick(m, n, k, gelu)
            few = gemm_tiles.slabs(k) < max(gemm_tiles.LAUNCHES[i][4:])
            seen.setdefault(i, set()).update({n % 8 == 0, "few" if few else "more"})
    for i, (bm, bn, wm, wn, sa, sb) in enumerate(gemm_tiles.LAUNCHES):
        want = {True, False, "more"}
        if (bm, bn, sa, sb) in ((256, 256, 3, 2), (256, 192, 2, 3), (128, 128, 2, 3), (64, 64, 4, 4),
                                (64, 32, 4, 4)):
            want.add("few")
        assert want <= seen.get(i, set()), (i, (bm, bn, sa, sb), seen.get(i))
