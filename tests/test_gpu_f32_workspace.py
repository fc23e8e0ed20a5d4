"""An fp32 handle holds what its layers use: the activations, and none of the
split-K and decode buffers of the bf16 kernels."""
import re

import pytest
import torch

import paper_2607_04181_amd as coco

pytestmark = pytest.mark.gpu

D, HQ, HKV, HD, F = 256, 4, 2, 64, 688
ROWS = 65536
MIB = 1 << 20


def test_f32_handle_memory_and_noalloc_limit():
    shapes = {"w_qkv": ((HQ + 2 * HKV) * HD, D), "w_o": (D, HQ * HD), "w_gate_up": (2 * F, D),
              "w_down": (D, F), "gamma_attn": (D,), "gamma_mlp": (D,),
              "k_cache": (4, HKV, 16 * HD), "v_cache": (4, HKV, 16 * HD)}
    layer = {k: torch.zeros(s, device="cuda") for k, s in shapes.items()}
    # The first handle on a GPU loads the library there (code, static scratch).
    coco.coco_layer_destroy(coco.coco_layer_init(
        coco.make_config(D, HQ, HKV, HD, F, 1, "f32", 4, 4, 4, 1e4, 1e-6), [layer]))
    cfg = coco.make_config(D, HQ, HKV, HD, F, 1, "f32", ROWS, 4, 4, 1e4, 1e-6)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    h = coco.coco_layer_init(cfg, [layer])
    held = free - torch.cuda.mem_get_info()[0]
    # x, h, q, o, h2, x1 and u in fp32; the constants and the allocator's
    # granularity are far below 16 MiB, the unused pieces 353 MiB.
    used = ROWS * (4 * D + 2 * HQ * HD + F) * 4
    assert used <= held <= used + 16 * MIB, (held / MIB, used / MIB)
    # The no-alloc entry point counts a call as before, part (2 F columns), work
    # list, sums of squares and row slots included: at 12,000 rows 166 MB.
    n = 12000
    hidden = torch.zeros(n, D, device="cuda")
    idx = torch.arange(n, dtype=torch.int32, device="cuda")
    starts = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    table = torch.zeros(1, 4, dtype=torch.int32, device="cuda")
    with pytest.raises(coco.CocoError, match="scratch") as e:
        coco.coco_layer_forward_noalloc(h, 0, hidden, idx, idx, starts, table, starts[1:].clone())
    pieces = [4 * n * D] * 6 + [4 * n * F, 4 * n * 2 * F, 4 * 2, 4 * 32 * n, 8 * n]
    need = sum((p + 255) // 256 * 256 for p in pieces)
    assert int(re.search(r"needs (\d+) bytes", str(e.value)).group(1)) == need
    coco.coco_layer_destroy(h)
