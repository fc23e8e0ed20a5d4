"""Decode projections on the tile kernel: a batch and its shares run different
kernels (above and below 128 and 64 rows) on the same K-slices and must give
the same bits."""
import numpy as np
import pytest
import torch

from harness import (TOL, PoolSnapshot, Replica, normwise_err, oracle_decode_rows,
                     pool_blocks_of_new_tokens, ragged_decode_batch, small_bf16_shape, to64)
from workloads import device as WD

pytestmark = pytest.mark.gpu

# d, query heads, F: a 4096-wide shape whose O and down projections (4096 x
# 4096) plan 4 waves and gate/up (8192 x 4096) 8, each in one round with 4
# K-slices, its QKV unsplit; and a narrow one with unsplit 4-wave plans of a few
# workgroups. Row counts on both sides of 64 and 128, none a multiple of a tile.
# (8 K-slices and a split QKV: test_tile_coverage.py.)
CASES = [((4096, 32, 4096), 131, ([70], [61])), ((4096, 32, 4096), 97, ([65], [31], [1])),
         ((512, 8, 768), 201, ([128], [72], [1])), ((512, 8, 768), 129, ([65], [64]))]


@pytest.mark.parametrize("dims,rows,shares", CASES)
def test_decode_tile_kernels_agree_bit_exactly_and_match_oracle(dims, rows, shares):
    d, hq, ffn = dims
    shape = small_bf16_shape(d=d, hq=hq, hkv=2, ffn=ffn)
    rng = np.random.default_rng(rows)
    b = ragged_decode_batch(61, rng.integers(0, 300, rows), max_ctx=512, hidden_rows=rows + 5,
                            row_idx=rng.permutation(rows + 5)[:rows])
    rep = Replica.for_batch(shape, "s61", 1, b)
    hidden = WD.hidden_tensor(shape, "s61", b.hidden_rows)
    h0 = to64(hidden)
    snap = PoolSnapshot(rep.layers[0], pool_blocks_of_new_tokens(b))
    whole = hidden.clone()
    rep.forward(0, whole, WD.batch_tensors(b))
    torch.cuda.synchronize()
    pools = {k: rep.layers[0][k].clone() for k in ("k_cache", "v_cache")}
    check = [0, rows // 2, rows - 1]
    ref, _, _ = oracle_decode_rows(shape, "s61", 0, b, check, h0)
    got = to64(whole)[b.row_idx[check]]
    assert normwise_err(got, ref) < TOL
    # The branch y - x: its own bound, plus y's rounding to bf16 (2^-9 of |y|),
    # which the small layers' small branches see (x ~ 3, y - x ~ 0.3).
    x = h0[b.row_idx[check]]
    rounding = 2.0 ** -9 * np.max(np.abs(ref)) / np.max(np.abs(ref - x))
    assert normwise_err(got - x, ref - x) < TOL + rounding
    snap.restore()
    split = hidden.clone()
    at = 0
    for (n,) in shares:
        rep.forward(0, split, WD.batch_tensors(b.select(np.arange(at, at + n))))
        at += n
    assert at == rows
    torch.cuda.synchronize()
    assert torch.equal(split.view(torch.int16), whole.view(torch.int16))
    for k, p in pools.items():
        assert torch.equal(rep.layers[0][k].view(torch.int16), p.view(torch.int16))
