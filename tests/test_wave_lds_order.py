"""Where the lanes of one wave pass values through LDS without a barrier, the
order of the stores and the loads is not the compiler's to choose: it sees one
lane's addresses. Read off the assembly of the kernels that do so (CPU only:
hipcc cross-compiles)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_04181_amd import build as B

pytestmark = pytest.mark.skipif(shutil.which(B.HIPCC) is None, reason="no hipcc")

# Two SwiGLU epilogues of the prefill GEMMs: one tile, and the persistent kernel.
SWIGLU = """
#include "gemm_prefill.h"
namespace coco { namespace prefill {
template __global__ void gemm_prefill_kernel<T64x64, kSwiglu>(
    const bf16_t* __restrict__, const bf16_t* __restrict__, int, int, int, PrefillEpiArgs);
template __global__ void gemm_prefill_swiglu_persistent_kernel<T256x192>(
    const bf16_t* __restrict__, const bf16_t* __restrict__, int, int, int, bf16_t* __restrict__,
    const float* __restrict__, float);
} }
"""


def kernels(source, out):
    """Kernel name -> its assembly lines."""
    cmd = [B.HIPCC, *B.FLAGS, f"-I{B.CSRC}", "--cuda-device-only", "-S", str(source), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    text = out.read_text()
    return {m.group(1): m.group(0).splitlines()
            for m in re.finditer(r"^(_ZN\w+):.*?^\.Lfunc_end", text, re.S | re.M)}


def kind(line, store="ds_write", load="ds_read"):
    op = line.split()[0] if line.split() else ""
    if "wave barrier" in line or op == "s_barrier":
        return "order"
    return "store" if op.startswith(store) else "load" if op.startswith(load) else None


def assert_ordered(lines, **ops):
    seen = [k for k in (kind(l, **ops) for l in lines) if k]
    assert "store" in seen and "load" in seen
    for a, b in zip(seen, seen[1:]):
        assert "order" in (a, b) or a == b, f"{b} next to {a}: {seen}"


def test_fp32_gemm_chunks(tmp_path):
    """A chunk's pieces are stored, then read by other lanes, in every step of
    the main loop (the block with the matrix instructions)."""
    ks = kernels(os.path.join(B.CSRC, "layer_f32.hip"), tmp_path / "f32.s")
    gemms = {n: l for n, l in ks.items() if "layer_f32_gemm_kernel" in n}
    assert len(gemms) == 8
    for lines in gemms.values():
        cuts = [i for i, l in enumerate(lines) if l.startswith(".LBB")] + [len(lines)]
        loops = [lines[a:b] for a, b in zip(cuts, cuts[1:])
                 if any("v_mfma" in l for l in lines[a:b])]
        assert len(loops) == 1
        assert_ordered(loops[0])
        assert kind([l for l in loops[0] if kind(l)][-1]) == "order"  # before the next step's stores


def test_swiglu_output_staging(tmp_path):
    """The epilogue's bf16 outputs (2-byte stores, 16-byte loads)."""
    src = tmp_path / "swiglu.hip"
    src.write_text(SWIGLU)
    ks = kernels(src, tmp_path / "swiglu.s")
    assert len(ks) == 2
    for lines in ks.values():
        last = max(i for i, l in enumerate(lines) if "v_mfma" in l)
        assert_ordered(lines[last:], store="ds_write_b16", load="ds_read_b128")


def test_decode_work_list(tmp_path):
    """The work list's counts: cleared, counted, turned into ranks, counted up
    again; an ordering point between each two."""
    ks = kernels(os.path.join(B.CSRC, "rows.hip"), tmp_path / "rows.s")
    epilogues = {n: l for n, l in ks.items() if "qkv_epilogue_kernel" in n}
    assert epilogues
    for lines in epilogues.values():
        assert sum("wave barrier" in l for l in lines) == 3
