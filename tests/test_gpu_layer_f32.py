"""The fp32 layer's kernels against the oracle at the sizes where they can go
wrong: widths that are no multiple of a 32-k chunk or a 16-column tile, every
way the heads share an attention workgroup, one row tile and two, rows that
leave a tile partly empty, contexts around block edges and over several blocks
per wave."""
import numpy as np
import pytest
import torch

import paper_2607_04181_amd as coco
import workloads as W
from harness import (Replica, gpu_cache_tokens, normwise_err, oracle_decode_rows,
                     oracle_prefill_seqs, ragged_decode_batch, ragged_prefill_batch, to64)
from workloads import device as WD

pytestmark = pytest.mark.gpu

# fp32 dot products of up to 700 terms: at most 700 * 2^-24 = 4e-5 of the sum
# of the products' magnitudes, and a few such in a row.
TOL32 = 1e-4


def _shape(d, hq, hkv, hd, ffn):
    return W.LayerShape(d, hq, hkv, hd, ffn, 1.0e4, 1e-6, "f32")


# d, Hq, Hkv, hd, F: chunk tails in d (260) and F (684, 700), column tails
# (d = 260: 8 tiles of 32 and 4 columns; F = 700), groups of 1, 2, 3, 4, 8.
SHAPES = [(260, 4, 2, 64, 684), (128, 3, 1, 32, 700), (64, 8, 1, 32, 36), (96, 2, 2, 96, 100),
          (256, 4, 1, 128, 96), (160, 3, 3, 160, 64), (192, 2, 1, 192, 128),
          (224, 1, 1, 224, 132), (512, 4, 1, 256, 64)]


@pytest.mark.parametrize("dims", SHAPES)
def test_f32_decode_matches_oracle(dims):
    shape = _shape(*dims)
    priors = [0, 1, 14, 15, 16, 127, 128, 129, 300, 5, 40, 63, 64, 65, 255, 256, 31]
    b = ragged_decode_batch(51, priors, max_ctx=512, hidden_rows=20,
                            row_idx=np.random.default_rng(51).permutation(20)[:17])
    rep = Replica.for_batch(shape, "f51", 1, b)
    hidden = WD.hidden_tensor(shape, "f51", b.hidden_rows)
    h0 = to64(hidden)
    rep.forward(0, hidden, WD.batch_tensors(b))
    torch.cuda.synchronize()
    ref, rec, cache = oracle_decode_rows(shape, "f51", 0, b, range(b.n_rows), h0, record=True)
    got = to64(hidden)
    assert normwise_err(got[b.row_idx] - h0[b.row_idx], ref - h0[b.row_idx]) < TOL32
    others = sorted(set(range(b.hidden_rows)) - set(b.row_idx.tolist()))
    assert np.array_equal(got[others], h0[others])
    M, f = b.n_rows, torch.float32
    for name, which, cols in (("h", coco.COCO_WS_H, shape.d_model),
                              ("q", coco.COCO_WS_Q, shape.n_q_heads * shape.head_dim),
                              ("o", coco.COCO_WS_O, shape.n_q_heads * shape.head_dim),
                              ("x1", coco.COCO_WS_X1, shape.d_model),
                              ("h2", coco.COCO_WS_H2, shape.d_model),
                              ("a", coco.COCO_WS_U, shape.d_ffn)):
        if name in rec:
            assert normwise_err(to64(rep.workspace(which, M, cols, f)), rec[name]) < TOL32, name
    for s in range(b.n_seqs):
        p = int(b.positions[s])
        K, V = gpu_cache_tokens(rep.layers[0], b, s, p, p + 1)
        assert normwise_err(K[0], cache.K[s][p]) < TOL32
        assert normwise_err(V[0], cache.V[s][p]) < TOL32


@pytest.mark.parametrize("lens", [[1], [15, 1], [16, 33, 2], [70, 1, 31]])
def test_f32_prefill_matches_oracle_and_splits(lens):
    """One and several row tiles, requests sharing a tile; the requests one by
    one (one or two row tiles per workgroup) give the batch's bits."""
    shape = _shape(260, 4, 2, 64, 684)
    priors = [(61 * s + 9) % 140 for s in range(len(lens))]
    b = ragged_prefill_batch(52, priors=priors, lens=lens, max_ctx=256,
                             hidden_rows=sum(lens) + 3)
    rep = Replica.for_batch(shape, "f52", 1, b)
    hidden = WD.hidden_tensor(shape, "f52", b.hidden_rows)
    h0 = to64(hidden)
    whole = hidden.clone()
    rep.forward(0, whole, WD.batch_tensors(b))
    torch.cuda.synchronize()
    ref, _, cache, _ = oracle_prefill_seqs(shape, "f52", 0, b, range(b.n_seqs), h0)
    assert normwise_err(to64(whole)[b.row_idx] - h0[b.row_idx], ref - h0[b.row_idx]) < TOL32
    for s in range(b.n_seqs):
        t0, t1 = int(b.prior_lens[s]), int(b.ctx_lens[s])
        K, V = gpu_cache_tokens(rep.layers[0], b, s, t0, t1)
        assert normwise_err(K, cache.K[s][t0:t1]) < TOL32
        assert normwise_err(V, cache.V[s][t0:t1]) < TOL32
    split = hidden.clone()
    for s in range(b.n_seqs):
        rep.forward(0, split, WD.batch_tensors(b.select_seqs([s])))
    torch.cuda.synchronize()
    assert torch.equal(split, whole)
