"""Registers that the built kernels reserve, read from their kernel descriptors: the
double stage kernel of launches of at most one wavefront per SIMD, and the solve kernel of
two-layer ones, take more than half of a SIMD's 512, so that no two of their wavefronts
share one."""

import os
import re
import shutil
import subprocess

import paper_2605_16082_amd as P

LLVM = "/opt/rocm/llvm/bin"


def _reserved(tmp_path, kernel):
    """Symbol -> registers reserved, of the kernels whose name holds `kernel`."""
    lib = shutil.copy(os.path.join(os.path.dirname(P.__file__), "libslimdg.so"), tmp_path)
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", lib], check=True, capture_output=True)
    found = {}
    for name in sorted(os.listdir(tmp_path)):
        if "amdgcn" not in name:
            continue
        obj = os.path.join(tmp_path, name)
        syms = subprocess.run([f"{LLVM}/llvm-readelf", "-sW", obj], check=True, capture_output=True, text=True).stdout
        kds = sorted(set(re.findall(rf"\S*{kernel}\S*\.kd$", syms, re.M)))
        if not kds:
            continue
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-D", "-j", ".rodata", "--disassemble-symbols=" + ",".join(kds), obj],
                              check=True, capture_output=True, text=True).stdout
        for sym, regs in re.findall(r"\.amdhsa_kernel (\S+).*?\.amdhsa_next_free_vgpr (\d+)", text, re.S):
            found[sym] = int(regs)
    return found


def test_small_stage_launches_get_a_simd_for_each_wavefront(tmp_path):
    regs = _reserved(tmp_path, "12stage_kernel")
    # <double, fields, ..., no LDS>
    small = {k: v for k, v in regs.items() if "kernelId" in k and k.endswith("Lb0EEEvNS_9StageArgsE")}
    assert len(small) == 32 and len(regs) == 128
    assert min(small.values()) > 256, min(small.items(), key=lambda kv: kv[1])


def test_small_two_layer_solves_get_a_simd_for_each_wavefront(tmp_path):
    regs = _reserved(tmp_path, "19column_solve_kernel")
    small = {k: v for k, v in regs.items() if "Li128ELi1ELi1E" in k}     # threads, wavefronts a SIMD
    assert len(small) == 12                                              # 3 precision forms of 1 to 4 fields
    assert min(small.values()) > 256, min(small.items(), key=lambda kv: kv[1])
