"""The build refuses kernels that spill vector registers or use scratch memory (CPU: hipcc
cross-compiles for gfx950 here). The attention kernels order their LDS DMA with counted
vector-memory waits, which spill traffic would silently shift; the guard keeps a future
change from introducing it unnoticed."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_01701_amd import build as B

pytestmark = pytest.mark.skipif(not os.path.exists(B.HIPCC) and shutil.which("hipcc") is None,
                                reason="hipcc not available")

# 1024 threads per workgroup leave each wave 128 VGPRs; 160 live accumulators must spill.
SPILLING = r"""
#include <hip/hip_runtime.h>
__global__ __launch_bounds__(1024) void spills(const float* __restrict__ x, float* __restrict__ y, int n) {
  float acc[160];
#pragma unroll
  for (int i = 0; i < 160; ++i) acc[i] = x[threadIdx.x + i * 1024];
  for (int r = 0; r < n; ++r) {
#pragma unroll
    for (int i = 0; i < 160; ++i) acc[i] = acc[i] * acc[(i + 1) % 160] + x[r];
  }
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < 160; ++i) s += acc[i] * (i + 1);
  y[threadIdx.x] = s;
}
"""

CLEAN = r"""
#include <hip/hip_runtime.h>
__global__ void clean(const float* __restrict__ x, float* __restrict__ y) { y[threadIdx.x] = 2.0f * x[threadIdx.x]; }
"""


def _compile(tmp_path, name, src):
    p = tmp_path / f"{name}.hip"
    p.write_text(src)
    cmd = [B.HIPCC, *B.HIP_FLAGS, *B.RESOURCE_REMARKS, "-c", str(p), "-o", str(tmp_path / f"{name}.o")]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    return cmd, r.stdout


def test_spilling_kernel_is_rejected(tmp_path):
    cmd, out = _compile(tmp_path, "spills", SPILLING)
    res = B.kernel_resources(out)
    assert any("spills" in k for k in res), out[-2000:]
    bad = B.resource_violations(res)
    assert bad and "spills" in bad[0] and ("Spill" in bad[0] or "Scratch" in bad[0]), bad
    with pytest.raises(RuntimeError, match="spill registers or use scratch"):
        B._run(cmd, verbose=False, check_resources=True)


def test_clean_kernel_passes(tmp_path):
    cmd, out = _compile(tmp_path, "clean", CLEAN)
    res = B.kernel_resources(out)
    assert any("clean" in k for k in res) and not B.resource_violations(res)
    B._run(cmd, verbose=False, check_resources=True)


def test_attention_kernels_are_spill_free(tmp_path):
    """Every kernel of the attention sources reports no spills and no scratch (the same check the
    build applies)."""
    names = {}
    for src in [s for s in B.HIP_SOURCES if s.startswith(("t2v_fwd", "t2v_bwd"))]:
        cmd = [B.HIPCC, *B.HIP_FLAGS, *B.SCHED.get(src, []), *B.RESOURCE_REMARKS, "-c", os.path.join(B.CSRC, src),
               "-o", str(tmp_path / (src + ".o"))]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
        assert r.returncode == 0, r.stdout[-2000:]
        res = B.kernel_resources(r.stdout)
        assert not B.resource_violations(res), B.resource_violations(res)
        names.update(res)
    for kern in ("attn_fwd_kernel", "attn_bwd_pre_kernel", "attn_bwd_dkdv_kernel", "attn_bwd_dkdv_wide_kernel",
                 "attn_bwd_dq_kernel", "attn_bwd_short_kernel", "short_reduce_kernel"):
        assert any(kern in n for n in names), kern


# ------------------------------------------- accumulators of the inline-assembly MFMAs
#
# The kernels that keep their sums in accumulator registers write the MFMAs in assembly, so the
# compiler inserts no wait states for them: a copy or read of an accumulator that it placed too soon
# after one would return stale sums.

_INST = re.compile(r"^\t([a-z]\w+)\s*(.*)$")
_AGPR = re.compile(r"\ba(?:(\d+)\b|\[(\d+):(\d+)\])")


def _agprs(operand):
    return {r for one, lo, hi in _AGPR.findall(operand)
            for r in (range(int(one), int(one) + 1) if one else range(int(lo), int(hi) + 1))}


def _blocks(asm):
    """Basic blocks of a listing, in order: [(instructions, successors)]; and the kernels' first blocks."""
    blocks, labels = [([], [])], {}
    for line in asm.splitlines():
        label = re.match(r"^(\w[\w.$]*|\.LBB\w+):", line)
        m = _INST.match(line)
        if label:
            blocks.append(([], []))
            labels[label.group(1)] = len(blocks) - 1
        elif m:
            op, args = m.group(1), m.group(2).split(";")[0].strip()
            blocks[-1][0].append((op, args))
            if op.startswith(("s_branch", "s_cbranch", "s_endpgm")):
                blocks.append(([], []))
    for i, (insts, succ) in enumerate(blocks):
        op, args = insts[-1] if insts else ("", "")
        if op.startswith(("s_branch", "s_cbranch")):
            succ.append(labels[args])
        if op not in ("s_branch", "s_endpgm") and i + 1 < len(blocks):
            succ.append(i + 1)
    return blocks, [i for name, i in labels.items() if not name.startswith(".L")]


def accumulator_faults(asm):
    """Instructions of a listing that move or read an accumulator register where the result of an
    assembly MFMA may not have arrived (no settling wait since the last one on some path), other than
    moves of a zero; and the number of MFMAs on accumulators."""
    blocks, work = _blocks(asm)
    state = {i: (True, frozenset()) for i in work}
    faults = {}
    while work:
        i = work.pop()
        settled, zero = state[i][0], set(state[i][1])
        for n, (op, text) in enumerate(blocks[i][0]):
            args = text.split(",")
            if op == "s_nop":
                settled = settled or int(text) == 15
            elif op.startswith("v_mfma") and _agprs(args[0]):
                settled = False
                zero -= _agprs(args[0])
            elif op == "v_accvgpr_write_b32" and args[1].strip() == "0":
                zero |= _agprs(args[0])
            elif op == "v_accvgpr_mov_b32" and _agprs(args[1]) <= zero:
                zero |= _agprs(args[0])
            elif _agprs(text) and not settled:
                faults[i, n] = f"{op} {text}"
        for j in blocks[i][1]:
            old = state.get(j)
            new = (settled, frozenset(zero)) if old is None else (old[0] and settled, old[1] & zero)
            if new != old:
                state[j] = new
                work.append(j)
    n_mfma = sum(op.startswith("v_mfma") and text.startswith("a[") for insts, _ in blocks for op, text in insts)
    return list(faults.values()), n_mfma


@pytest.mark.parametrize("flags", [[], B.CHECKED_FLAGS], ids=["product", "checked"])
@pytest.mark.parametrize("src", ["t2v_bwd_dkdv_wide.hip", "t2v_bwd_short.hip"])
def test_accumulators_are_not_moved_before_they_settle(src, flags, tmp_path):
    out = tmp_path / "kernel.asm"
    r = subprocess.run([B.HIPCC, *B.HIP_FLAGS, *flags, *B.SCHED.get(src, []), "-S", "--cuda-device-only",
                        os.path.join(B.CSRC, src), "-o", str(out)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                       text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-2000:]
    asm = out.read_text()
    faults, n_mfma = accumulator_faults(asm)
    assert n_mfma >= 32 and not faults, faults[:5]
    # the check sees what it is there for: a copy in the loop, a read before the wait
    mfma = re.search(r"^\tv_mfma_\w+ a\[(\d+).*\n", asm, re.M)
    for planted in (f"\tv_accvgpr_mov_b32 a0, a{mfma.group(1)}\n", f"\tv_accvgpr_read_b32 v0, a{mfma.group(1)}\n",
                    f"\tds_write_b32 v0, a{mfma.group(1)}\n"):
        assert accumulator_faults(asm[:mfma.end()] + planted + asm[mfma.end():])[0], planted
