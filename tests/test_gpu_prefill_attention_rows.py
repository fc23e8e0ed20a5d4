"""Prefill attention on 64-row query tiles (few rows, sequences of more than 64
rows on average) and on 128-row ones: a request gives the same bits under both
and matches the oracle."""
import pytest
import torch

from harness import (TOL, PoolSnapshot, Replica, normwise_err, oracle_prefill_seqs,
                     pool_blocks_of_new_tokens, ragged_prefill_batch, small_bf16_shape, to64)
from workloads import device as WD

pytestmark = pytest.mark.gpu

# Whole batches run 128-row tiles (the single-row requests, or rows past a round
# of workgroups); request 0 alone (65 .. 129 rows, at most 256 / hq tiles of 64)
# the 64-row ones. Contexts end inside a stage of 128 keys and at its edge.
@pytest.mark.parametrize("hq,priors,lens", [
    (8, [0, 17], [65, 1]),
    (8, [1000, 0, 3], [129, 1, 1]),
    (32, [384, 5], [128, 500]),
])
def test_prefill_attention_row_tiles_agree_bit_exactly(hq, priors, lens):
    shape = small_bf16_shape(d=512, hq=hq, hkv=2, ffn=768)
    b = ragged_prefill_batch(43, priors=priors, lens=lens, max_ctx=1600,
                             hidden_rows=sum(lens) + 5)
    rep = Replica.for_batch(shape, "s43", 1, b)
    hidden = WD.hidden_tensor(shape, "s43", b.hidden_rows)
    h0 = to64(hidden)
    snap = PoolSnapshot(rep.layers[0], pool_blocks_of_new_tokens(b))
    whole = hidden.clone()
    rep.forward(0, whole, WD.batch_tensors(b))
    torch.cuda.synchronize()
    snap.restore()
    alone = hidden.clone()
    rep.forward(0, alone, WD.batch_tensors(b.select_seqs([0])))
    torch.cuda.synchronize()
    ref, _, _, sub = oracle_prefill_seqs(shape, "s43", 0, b, [0], h0)
    rows = torch.as_tensor(sub.row_idx, device=whole.device).long()
    assert torch.equal(alone[rows].view(torch.int16), whole[rows].view(torch.int16))
    assert normwise_err(to64(alone)[sub.row_idx], ref) < TOL
