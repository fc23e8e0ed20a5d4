"""Every tile shape that a projection of the 8B, 32B and 70B layers runs on is
run by a test, epilogue by epilogue: each pair is a kernel of its own. Which
shape a call takes is asked of the library's own choice, so a change of its
constants that leaves a pair untested fails here."""
import ctypes

import pytest

import test_gpu_decode_tiles as decode
import test_gpu_prefill_tiles as prefill
from paper_2607_04181_amd import _lib

# TileId (gemm_prefill.h)
TILES = ("256x224 256x192 256x160 256x128 192x256 160x256 128x256 128x160 128x128 128x64 64x160 "
         "64x128 64x64 64x32 32x32").split()
CUS = 256


class SkinnyPlan(ctypes.Structure):
    _fields_ = [("waves", ctypes.c_int), ("S", ctypes.c_int)]


_choose = _lib._lib._ZN4coco7prefill11choose_tileEiiiii  # (M, N, K, S, num_cus)
skinny_plan = _lib._lib._ZN4coco11skinny_planEii  # (N, K)
skinny_plan.restype = SkinnyPlan


def tile(M, N, K, S=1):
    return TILES[_choose(M, N, K, S, CUS)]


def prefill_pairs(d, hq, hkv, ffn, M):
    return {("qkv", tile(M, (hq + 2 * hkv) * 128, d)), ("residual", tile(M, d, hq * 128)),
            ("swiglu", tile(M, 2 * ffn, d)), ("scatter", tile(M, d, ffn))}


def decode_pairs(d, hq, hkv, ffn, M):
    """Tile kernels of a decode call: above 128 rows every projection's; below,
    by the rules of tile_partial, tile_qkv and tile_swiglu (coco_api.hip)."""
    out = set()
    n_qkv = (hq + 2 * hkv) * 128
    if M > 128 or (M > 64 and n_qkv * d >= 64 << 20):
        out.add(("partial", tile(M, n_qkv, d, skinny_plan(n_qkv, d).S)))
    for N, K in ((d, hq * 128), (d, ffn), (2 * ffn, d)):
        p = skinny_plan(N, K)
        if N == 2 * ffn and K == d and p.S == 1:
            if M > 128 or (M > 64 and (p.waves == 8 or N // 256 >= CUS * 3 // 4)):
                out.add(("swiglu_plain", tile(M, N, K)))
            continue
        full = N // (16 * p.waves) * p.S == CUS
        if M > 128 or (full and p.waves in (4, 8)) or (M > 64 and p.waves == 8):
            out.add(("partial", tile(M, N, K, p.S)))
    return out


# d, query heads, kv heads, F; rows of a prefill chunk, of a decode batch.
LAYERS = [(4096, 32, 8, 14336), (5120, 40, 8, 27648), (8192, 64, 8, 28672)]
PREFILL_ROWS, DECODE_ROWS = 3072, 512


def test_prefill_tile_tests_cover_every_pair():
    need = set().union(*(prefill_pairs(*l, M) for l in LAYERS for M in range(1, PREFILL_ROWS + 1)))
    have = set()
    for dims, lens, shares, _ in prefill.CASES + PREFILL_CASES:
        for M in [sum(lens)] + [sum(lens[s] for s in share) for share in shares]:
            have |= prefill_pairs(*dims, M)
    assert not need - have, sorted(need - have)


def test_decode_tile_tests_cover_every_pair():
    need = set().union(*(decode_pairs(*l, M) for l in LAYERS for M in range(1, DECODE_ROWS + 1)))
    have = set()
    for (d, hq, ffn), rows, shares in decode.CASES + DECODE_CASES:
        for M in [rows] + [n for (n,) in shares]:
            have |= decode_pairs(d, hq, 2, ffn, M)
    assert not need - have, sorted(need - have)


def test_decode_cases_reach_split_plans():
    """QKV and down projections in 8 K-slices, one of them on 8 waves, below
    and above 128 rows."""
    assert {(4096, 16, 512), (4096, 8, 8192)} <= {c[0] for c in DECODE_CASES}
    assert skinny_plan((16 + 4) * 128, 4096).S == 8
    p = skinny_plan(4096, 8192)
    assert (p.waves, p.S) == (8, 8)


# dims, lengths, shares, request checked against the oracle. QKV on 128 x 160,
# 64 x 160 and 64 x 128 tiles (390, 198, 134 rows of 64 + 16 heads; the last
# also gate/up on 64 x 128), on 256 x 224 and 128 x 256 (1729 and 1089 rows of 40
# + 16), on 256 x 192 (1611 rows of 32 + 16); O and down on 256 x 160 and 128 x 160
# (1601 and 801 rows). Every row count leaves a partial row tile.
PREFILL_CASES = [
    ((512, 64, 8, 4480), [134, 58, 198], ([0], [2], [1]), 0),
    ((512, 40, 8, 384), [1089, 600, 40], ([0], [2, 1]), 2),
    ((512, 32, 8, 384), [1300, 270, 41], ([0], [1, 2]), 2),
    ((5120, 4, 1, 512), [801, 767, 33], ([0], [2, 1]), 2),
]

# (d, query heads, F), rows, shares. Partial sums on 256 x 160 and 64 x 160 (385
# rows, d = 5120), 128 x 256 and 128 x 160 (QKV in 8 slices), 192 x 256 and 160 x 256
# (gate/up in 2 slices, down in 8 on 8 waves), 256 x 224 and 256 x 192; SwiGLU
# without 1/rms on 256 x 224, 192 x 256, 160 x 256, 256 x 128, 128 x 256.
DECODE_CASES = [
    ((5120, 16, 384), 385, ([257], [128])),
    ((4096, 16, 512), 300, ([171], [129])),
    ((4096, 16, 512), 127, ([65], [62])),
    ((4096, 8, 8192), 321, ([257], [64])),
    ((4096, 8, 8192), 100, ([67], [33])),
    ((512, 8, 14336), 385, ([321], [64])),
    ((512, 8, 14336), 257, ([193], [64])),
    ((512, 8, 27648), 97, ([65], [32])),
    ((1280, 8, 8192), 257, ([130], [127])),
    ((1024, 8, 7168), 385, ([257], [128])),
    ((1024, 8, 6144), 385, ([321], [64])),
]


@pytest.mark.gpu
@pytest.mark.parametrize("dims,lens,shares,req", PREFILL_CASES)
def test_prefill_tile_pairs(dims, lens, shares, req):
    prefill.test_prefill_tile_shapes_agree_bit_exactly_and_match_oracle(dims, lens, shares, req)


@pytest.mark.gpu
@pytest.mark.parametrize("dims,rows,shares", DECODE_CASES)
def test_decode_tile_pairs(dims, rows, shares):
    decode.test_decode_tile_kernels_agree_bit_exactly_and_match_oracle(dims, rows, shares)
