"""The bulk cache append is a bit copy whatever the tokens' order and
alignment: whole pools against the documented tile layout written out in torch
(untouched bytes included)."""
import numpy as np
import pytest
import torch

import paper_2607_04181_amd as coco
import workloads as W
from harness import Replica, ragged_decode_batch, small_bf16_shape
from workloads import device as WD

pytestmark = pytest.mark.gpu

# (sequence, first position, count) pieces in call order: runs that start on
# and off four-token edges and across workgroups of 16 tokens, single tokens,
# a sequence coming back, a run cut by a block edge.
SPANS = {
    "one": [(0, 5, 1)],
    "aligned": [(0, 0, 40)],
    "off by one": [(0, 1, 37)],
    "off by three": [(1, 3, 50), (0, 2, 14)],
    "mixed": [(2, 7, 3), (0, 0, 4), (1, 15, 2), (2, 10, 23), (0, 4, 1), (1, 17, 31), (0, 30, 2)],
}


def _perm(kind, n):
    if kind == "in order":
        return np.arange(n)
    if kind == "reversed":
        return np.arange(n)[::-1].copy()
    return np.random.default_rng(n).permutation(n)


@pytest.mark.parametrize("order", ["in order", "reversed", "shuffled"])
@pytest.mark.parametrize("spans", sorted(SPANS))
@pytest.mark.parametrize("dtype,hd", [("bf16", 128), ("f32", 32), ("f32", 96), ("f32", 256)])
def test_append_of_any_token_order_is_a_bit_copy(dtype, hd, spans, order):
    shape = small_bf16_shape() if dtype == "bf16" else \
        W.LayerShape(64, 2, 2, hd, 64, 1.0e4, 1e-6, "f32")
    b = ragged_decode_batch(7, [80, 80, 80], max_ctx=96)
    rep = Replica.for_batch(shape, "ap", 1, b)
    seq = np.concatenate([np.full(n, s) for s, _, n in SPANS[spans]])
    pos = np.concatenate([np.arange(p, p + n) for _, p, n in SPANS[spans]])
    o = _perm(order, len(seq))
    seq, pos = seq[o], pos[o]
    n, hkv = len(seq), shape.n_kv_heads
    g = torch.Generator(device="cuda").manual_seed(n)
    for shift in (0, 1):  # inputs on and off 16-byte boundaries
        k, v = (torch.randn(n * hkv * hd + shift, device="cuda", generator=g)
                .to(shape.torch_dtype)[shift:].view(n, hkv, hd) for _ in range(2))
        want_k, want_v = (rep.layers[0][x].clone() for x in ("k_cache", "v_cache"))
        blk = torch.from_numpy(b.block_table[seq, pos // 16].astype(np.int64)).cuda()
        slot = torch.from_numpy(pos % 16).cuda()
        want_k.view(-1, hkv, hd // 32, 4, 16, 8)[blk, :, :, :, slot] = \
            k.view(n, hkv, hd // 32, 4, 8)
        want_v.view(-1, hkv, hd // 32, 4, 16, 2, 4)[blk, :, :, slot // 4, :, :, slot % 4] = \
            v.view(n, hkv, hd // 32, 2, 16).transpose(-1, -2)
        coco.coco_kv_append(rep.h, 0, k, v, torch.from_numpy(seq.astype(np.int32)).cuda(),
                            torch.from_numpy(pos.astype(np.int32)).cuda(),
                            WD.batch_tensors(b)["block_table"])
        torch.cuda.synchronize()
        assert torch.equal(rep.layers[0]["k_cache"], want_k)
        assert torch.equal(rep.layers[0]["v_cache"], want_v)
