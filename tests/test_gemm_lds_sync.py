"""Static check of the LDS synchronisation of the kernels that load straight from
global memory into LDS (no GPU).

The bf16 GEMM's direct loop frees an LDS stage at a bare s_barrier: after it, other
wavefronts' global->LDS loads overwrite the stage the previous slice was read
from.  Every LDS read a wavefront has issued must therefore have returned
before it reaches that barrier.  The compiler may place the MFMAs that consume
a slice's operands (and with them its own wait for the reads) after the next
barrier, so the kernel waits for its LDS reads explicitly.  The first test compiles
a few instances of the kernel for gfx950 (dense, forward gather, data-gradient
gather with the transposing reads, weight-gradient gather, rows from a halo; four
and eight wavefronts; one, two and three stages) and walks each one's
instructions: at every s_barrier no LDS read issued since the last lgkmcnt(0) wait
may be pending.  The fp32 product whose loading wavefronts refill the stages that
others read is held to the same.  In the kernels whose wavefronts refill their own
stages without a barrier (the MLP's backward, the LSTM's steps) a load into LDS
takes the place of the barrier.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

INSTANCES = """
#include "gemm_bf16_kernel.h"
namespace ckpt {
namespace gb {
template __global__ void k_gemm_bf16<64, 64, 2, 2, true, true, __bf16, GEMM_EPI_BF16STATS, GA_FWDT, G_DENSE, true, 0>(Args);
template __global__ void k_gemm_bf16<64, 64, 4, 2, true, true, __bf16, GEMM_EPI_BF16STATS, GA_FWDT, G_DENSE, true, 0>(Args);
template __global__ void k_gemm_bf16<256, 64, 4, 2, true, false, __bf16, GEMM_EPI_BNBWD, GA_DGRADT, GB_WDGRAD, true, 0>(Args);
template __global__ void k_gemm_bf16<128, 128, 2, 2, false, false, __bf16, GEMM_EPI_STORE, G_DENSE, G_DENSE, true, 3>(Args);
template __global__ void k_gemm_bf16<128, 64, 4, 2, false, false, __bf16, GEMM_EPI_STORE, G_DENSE, GB_WGRAD, true, 0>(Args);
template __global__ void k_gemm_bf16<128, 128, 2, 2, true, true, __bf16, GEMM_EPI_ADDMASK, G_DENSE, G_DENSE, true, 0>(Args);
template __global__ void k_gemm_bf16<128, 128, 2, 2, true, true, __bf16, GEMM_EPI_BF16STATS, G_DENSE, G_DENSE, true, 1>(Args);
template __global__ void k_gemm_bf16<128, 128, 2, 2, true, true, __bf16, GEMM_EPI_BF16STATS, GA_FWDT, G_DENSE, true, 8 + 2>(Args);
template __global__ void k_gemm_bf16<64, 64, 4, 2, true, true, __bf16, GEMM_EPI_BF16STATS, GA_FWDT, G_DENSE, true, 8 + 3>(Args);
template __global__ void k_gemm_bf16<256, 64, 4, 2, true, false, __bf16, GEMM_EPI_BNBWD, GA_DGRADT, GB_WDGRAD, true, 8 + 3>(Args);
template __global__ void k_gemm_bf16<128, 128, 4, 2, true, false, __bf16, GEMM_EPI_BNBWD, GA_DGRADT, GB_WDGRAD, true, 8 + 3>(Args);
}  // namespace gb
}  // namespace ckpt
"""


def pending_reads(asm: str, at):
    """{kernel: instructions for which `at(text)` holds reached with LDS reads
    outstanding}, walking each kernel's instructions in order (an lgkmcnt(0) wait
    clears the reads)."""
    bad, kernel, pending = {}, None, 0
    for line in asm.split("\n"):
        m = re.match(r"^(_Z\S+):", line)
        if m:
            kernel, pending = m.group(1), 0
            continue
        if line.startswith(".Lfunc_end"):
            kernel = None
            continue
        tok = line.strip().split()
        if kernel is None or not tok:
            continue
        op = tok[0]
        if op.startswith(("ds_read", "ds_load")):
            pending += 1
        elif op == "s_waitcnt":
            w = re.search(r"lgkmcnt\((\d+)\)", " ".join(tok[1:]))
            if w and int(w.group(1)) == 0:
                pending = 0
        elif at(line.strip()):
            if pending:
                bad[kernel] = bad.get(kernel, 0) + 1
            pending = 0
    return bad


def is_barrier(text):
    return text.split()[0] == "s_barrier"


def is_lds_load(text):
    """a load from global memory straight into LDS"""
    return re.match(r"(global|buffer)_load_lds", text) is not None or (
        text.startswith("buffer_load") and text.split(";")[0].rstrip().endswith(" lds"))


def pending_reads_at_barriers(asm: str):
    return pending_reads(asm, is_barrier)


def compiled(tmp_path, name, source=None):
    """gfx950 assembly of csrc's `name`, or of `source`"""
    src = os.path.join(ROOT, "paper_1604_06174_amd", "csrc", name)
    if source is not None:
        src = tmp_path / name
        src.write_text(source)
    out = tmp_path / (name + ".s")
    cmd = [HIPCC if os.path.exists(HIPCC) else "hipcc", "-O3", "-std=c++17",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_1604_06174_amd", "csrc"),
           "-x", "hip", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "--cuda-device-only", "-S", str(src), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    return out.read_text()


def body_of(asm, pattern):
    """the functions of asm whose names match, with the number of them"""
    parts = re.findall(r"^(_Z\S*(?:%s)\S*:.*?^\.Lfunc_end\d+:)" % pattern, asm, re.M | re.S)
    return "\n".join(parts), len(parts)


no_hipcc = pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None, reason="hipcc not present")


def test_scan_flags_a_pending_read():
    """The scan itself: a read between the last wait and a barrier is found."""
    asm = "\n".join(["_Zk:", "  ds_read_b128 v[0:3], v4", "  s_waitcnt lgkmcnt(0)", "  s_barrier",
                     "  ds_read_b128 v[0:3], v4", "  s_waitcnt vmcnt(4)", "  s_barrier", ".Lfunc_end0:"])
    assert pending_reads_at_barriers(asm) == {"_Zk": 1}
    asm = asm.replace("s_barrier", "global_load_lds_dwordx4 v[0:1], off")
    assert pending_reads(asm, is_lds_load) == {"_Zk": 1}


@no_hipcc
def test_direct_loop_barriers_have_no_pending_lds_reads(tmp_path):
    asm = compiled(tmp_path, "instances.hip", INSTANCES)
    kernels = re.findall(r"^(_Z\S*k_gemm_bf16\S*):", asm, re.M)
    assert len(kernels) == 11, kernels
    assert sum(1 for l in asm.split("\n") if l.strip().startswith("s_barrier")) > 0
    assert pending_reads_at_barriers(asm) == {}


@no_hipcc
@pytest.mark.parametrize("source,kernel,at", [("gemm_f32.hip", "k_gemm_f32_ks", is_barrier),
                                              ("mlp_bwd.hip", "k_gemm_f32_mlp_bwd", is_lds_load),
                                              ("lstm_step.hip", "k_lstm_step_[fb]wd", is_lds_load)])
def test_stage_refills_have_no_pending_lds_reads(tmp_path, source, kernel, at):
    asm, n = body_of(compiled(tmp_path, source), kernel)
    assert n > 0
    assert sum(1 for l in asm.split("\n") if is_lds_load(l.strip())) > 0
    assert sum(1 for l in asm.split("\n") if l.strip() and at(l.strip())) > 0
    assert pending_reads(asm, at) == {}
