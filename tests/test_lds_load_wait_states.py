"""load_to_lds (csrc/fwa_device.h) issues its buffer load from inline assembly, where the compiler does not insert the
wait states it would give a load of its own: a vector instruction that writes a scalar register (v_readfirstlane,
v_readlane) must be 5 wait states ahead of a memory instruction that reads it, and a write of m0 one state ahead of a
load into LDS.  The sequence has to keep both distances whatever stands in front of it; here a descriptor word is written
by v_readfirstlane directly in front, and the distances are counted in the assembly."""
import re
import subprocess

from paper_2501_06480_amd import build

PROBE = r'''
#include <hip/hip_runtime.h>
#include "fwa_device.h"
__global__ void probe(const char* base, const uint32_t* bytes, uint32_t to, float* out) {
    __shared__ __attribute__((aligned(16))) float area[512];
    const uint32_t off = threadIdx.x * 16u, v = bytes[threadIdx.x];
    area[threadIdx.x] = 0.f;
    uint32_t n;
    asm volatile("v_readfirstlane_b32 %0, %1" : "=s"(n) : "v"(v));
    fwa::load_to_lds(base, n, off, to);
    fwa::lds_loads_done();
    __syncthreads();
    out[threadIdx.x] = area[255 - threadIdx.x];
}
'''


def scalar_registers(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return {f"s{i}" for i in range(int(m[1]), int(m[2]) + 1)}
    return {operand} if re.fullmatch(r"s\d+|m0", operand) else set()


def test_descriptor_and_m0_are_old_enough(tmp_path):
    src = tmp_path / "probe.hip"
    src.write_text(PROBE)
    asm = tmp_path / "probe.s"
    subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, "-I", build.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(asm)],
                   check=True, capture_output=True)
    code = [l.strip().split(";")[0].strip() for l in asm.read_text().splitlines() if re.match(r"^\s+[a-z]", l)]
    loads = [i for i, l in enumerate(code) if l.startswith("buffer_load") and l.endswith("lds")]
    assert loads, "no load into LDS in the probe"
    met = 0
    for at in loads:
        operands = [o.strip() for o in code[at].split(None, 1)[1].split(",")]
        wanted = set().union(*(scalar_registers(o) for o in operands)) | {"m0"}
        states = 0
        for l in reversed(code[:at]):
            op, rest = l.split(None, 1) if " " in l else (l, "")
            dst = scalar_registers(rest.split(",")[0].strip())
            if dst & wanted:
                need = 5 if op.startswith("v_") else (1 if "m0" in dst else 0)
                assert states >= need, f"{l} is {states} wait states in front of {code[at]}, {need} are needed"
                met += op.startswith("v_")
                wanted -= dst
            if not wanted or op == "s_barrier":
                break
            states += int(rest, 0) + 1 if op == "s_nop" else 1
    assert met, "the probe has no vector write of a descriptor word to measure from"

