"""What the compiled kernels must hold, read from their device assembly.

Wait states of the loads to LDS that are issued from inline assembly: the
compiler does not look into such a statement, so the waits that the hardware
leaves to software have to be part of it, one state between a scalar write of
m0 and a load to LDS, and five between a vector instruction's write of a scalar
register and a load that takes its address from it.

Registers: the attention's walk and merge kernels keep what they work on in
registers (the fused append's walks excepted, see persist_waves_per_eu)."""
from __future__ import annotations

import functools
import os
import re
import subprocess
import tempfile

import pytest

from paper_2608_24004_amd import build

CSRC = os.path.join(build.PKG, "csrc")
PROBE = """
#include "common.h"
namespace averify {
// the base comes out of a vector register right before the copy
__global__ void probe(const uint8_t* p, const int* at, int* out) {
    __shared__ __attribute__((aligned(16))) uint8_t s[16384];
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)&s[0];
    const uint8_t* q = p + __builtin_amdgcn_readfirstlane(at[threadIdx.x]);
    dma16_run<1>(base, q, threadIdx.x * 16);
    dma16_run<2>(base + 2048, q + 4096, threadIdx.x * 16);
    dma16_run<4>(base + 8192, q + 8192, threadIdx.x * 16);
    wait_vmcnt<0>();
    lds_barrier();
    out[threadIdx.x] = s[threadIdx.x];
}
}
"""


def _scalars(token):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", token)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"s(\d+)", token)
    return {int(m[1])} if m else set()


def _faults(asm):
    """Loads to LDS, and those that a wait is missing for (in program order; a
    label is passed over, as where the block before falls through)."""
    lines = []
    for raw in asm.splitlines():
        line = raw.split(";")[0].strip()
        if line and not line.startswith(".") and not line.endswith(":"):
            lines.append(line)
    loads, bad = 0, []
    for i, line in enumerate(lines):
        if not re.match(r"global_load_lds_dword", line):
            continue
        loads += 1
        ops = [o.split()[0] for o in line.split(None, 1)[1].split(",")]
        base = _scalars(ops[1])
        waited = 0
        for prev in reversed(lines[:i]):
            if waited >= 5:
                break
            op, _, rest = prev.partition(" ")
            dsts = [t.strip() for t in rest.split(",")[:2]]
            if waited < 1 and dsts[0] == "m0":
                bad.append((prev, line))
            # a vector instruction's scalar result: first operand, or the carry
            if op.startswith("v_") and (base & _scalars(dsts[0]) or
                                        ("_co_" in op and base & _scalars(dsts[-1]))):
                bad.append((prev, line))
            nop = re.fullmatch(r"s_nop (\d+)", prev)
            waited += int(nop[1]) + 1 if nop else 1
    return loads, bad


@functools.lru_cache(maxsize=None)
def _assembly(name):
    with tempfile.TemporaryDirectory() as tmp:
        src = os.path.join(CSRC, name)
        if name == "probe.hip":
            src = os.path.join(tmp, name)
            with open(src, "w") as f:
                f.write(PROBE)
        out = os.path.join(tmp, "device.s")
        flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-shared", "-Wall")]
        subprocess.run([build.hipcc()] + flags + ["--cuda-device-only", "-S", "-I", os.path.join(build.ROOT, "include"),
                                                  "-I", CSRC, "-o", out, src], check=True, stderr=subprocess.DEVNULL)
        with open(out) as f:
            return f.read()


@pytest.mark.parametrize("name", ["verify_attention.hip", "verify_lmhead.hip", "probe.hip"])
def test_loads_to_lds_wait_for_their_scalars(name):
    loads, bad = _faults(_assembly(name))
    assert loads >= 7
    assert not bad, "%d of %d loads, first: %s" % (len(bad), loads, bad[0])


def test_attention_kernels_do_not_spill():
    scratch = {}
    for block in re.split(r"\n  - \.agpr_count", _assembly("verify_attention.hip"))[1:]:
        name = re.search(r"\.name:\s+(\S+)", block)[1]
        scratch[name] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", block)[1])
    plain = {n: b for n, b in scratch.items() if re.search(r"attn_(persist|combine|f32)", n) and "Lb1E" not in n}
    assert len(plain) >= 20
    assert not {n: b for n, b in plain.items() if b}
