"""The prefill GEMMs run on one of fifteen tile shapes, chosen by the call's
rows: whole batches and their request-aligned shares below take different
shapes for the same rows, and must give the same bits."""
import pytest
import torch

from harness import (TOL, PoolSnapshot, Replica, gpu_cache_tokens, normwise_err,
                     oracle_prefill_seqs, pool_blocks_of_new_tokens, ragged_prefill_batch,
                     small_bf16_shape, to64)
from workloads import device as WD

pytestmark = pytest.mark.gpu

# (d, query heads, kv heads, F), lengths, shares, request checked against the oracle.
# d = 2560, F = 4480: gate/up of 2100 rows on 256 x 160 tiles, 1500 on
# 256 x 224, 1025 on 160 x 256, 513 on 256 x 128, 200 on 64 x 160, 87 on
# 128 x 64; O and down from 256 x 128 to 32 x 32; QKV from 128 x 64 to 32 x 32.
# d = 1792, F = 3584: gate/up of 1025 rows on 128 x 256 tiles. 192- and 160-row
# tiles: gate/up of 381 and 302 rows (F = 14336), O and down of 1340 and 1050
# rows (d = 8192), QKV of 1050 rows (64 + 16 heads) and of 1290 (40 + 8).
# d = 640, F = 5760: gate/up of 2048 and 4096 rows on the persistent 256 x 192
# kernel (8 and 16 row tiles, up to two and four column tiles per workgroup),
# the shares of 1500 and 2296 rows on 256 x 160.
# Lengths leave partial row tiles and rows of several requests in one tile.
CASES = [
    ((2560, 5, 1, 4480), [1500, 513, 33, 54], ([0], [1], [3, 2]), 2),
    ((2560, 5, 1, 4480), [825, 130, 70], ([0], [1, 2]), 2),
    ((1792, 14, 1, 3584), [765, 259, 1], ([2, 1], [0]), 2),
    ((512, 4, 1, 14336), [250, 52, 79], ([0, 1], [2]), 1),
    ((8192, 4, 1, 512), [1050, 250, 40], ([0], [1, 2]), 2),
    ((512, 64, 8, 384), [1000, 50], ([0], [1]), 1),
    ((1024, 40, 4, 384), [1250, 40], ([0], [1]), 1),
    ((640, 5, 1, 5760), [1500, 300, 248], ([0], [2, 1]), 1),
    ((640, 5, 1, 5760), [1500, 300, 1000, 1296], ([0], [1], [3, 2]), 1),
]


@pytest.mark.parametrize("dims,lens,shares,req", CASES)
def test_prefill_tile_shapes_agree_bit_exactly_and_match_oracle(dims, lens, shares, req):
    d, hq, hkv, ffn = dims
    shape = small_bf16_shape(d=d, hq=hq, hkv=hkv, ffn=ffn)
    priors = [(37 * s) % 90 for s in range(len(lens))]
    b = ragged_prefill_batch(41, priors=priors, lens=lens, max_ctx=1600,
                             hidden_rows=sum(lens) + 7)
    rep = Replica.for_batch(shape, "s41", 1, b)
    hidden = WD.hidden_tensor(shape, "s41", b.hidden_rows)
    h0 = to64(hidden)
    snap = PoolSnapshot(rep.layers[0], pool_blocks_of_new_tokens(b))
    whole = hidden.clone()
    rep.forward(0, whole, WD.batch_tensors(b))
    torch.cuda.synchronize()
    pools = {k: rep.layers[0][k].clone() for k in ("k_cache", "v_cache")}
    ref, _, cache, sub = oracle_prefill_seqs(shape, "s41", 0, b, [req], h0)
    got = to64(whole)[sub.row_idx]
    assert normwise_err(got, ref) < TOL
    assert normwise_err(got - h0[sub.row_idx], ref - h0[sub.row_idx]) < TOL
    t0, t1 = int(b.prior_lens[req]), int(b.ctx_lens[req])
    K, V = gpu_cache_tokens(rep.layers[0], b, req, t0, t1)
    assert normwise_err(K, cache.K[0][t0:t1]) < TOL and normwise_err(V, cache.V[0][t0:t1]) < TOL
    snap.restore()
    split = hidden.clone()
    for seqs in shares:
        rep.forward(0, split, WD.batch_tensors(b.select_seqs(seqs)))
    torch.cuda.synchronize()
    assert torch.equal(split.view(torch.int16), whole.view(torch.int16))
    for k, p in pools.items():
        assert torch.equal(rep.layers[0][k].view(torch.int16), p.view(torch.int16))
