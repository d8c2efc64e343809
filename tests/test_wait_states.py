"""Wait states around the instructions that csrc/mfma_common.h writes as inline assembly.  The compiler keeps the distances
that the hardware asks for between instructions that it knows; an inline instruction carries its own.  Small kernels
are compiled for gfx950 and the distances counted in the assembly (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2605_30010_amd.build import CSRC, FLAGS, HIPCC

KERNELS = """
#include "mfma_common.h"
namespace et {
template <bool THROUGH>
__global__ void overwrite_behind_store(uint16_t *p, const u32x4 *src) {
  u32x4 v = src[threadIdx.x], w = src[threadIdx.x + 64];
  asm volatile("s_waitcnt vmcnt(0)" : "+v"(v), "+v"(w)::"memory");
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint16_t *q = p + (threadIdx.x + 64 * i) * 8;
    if (THROUGH) store16(q, v, true);
    else *reinterpret_cast<u32x4 *>(q) = v;
    __builtin_amdgcn_sched_barrier(0);
    v ^= w;
    asm volatile("" : "+v"(v));
    __builtin_amdgcn_sched_barrier(0);
  }
}
template __global__ void overwrite_behind_store<true>(uint16_t *, const u32x4 *);
template __global__ void overwrite_behind_store<false>(uint16_t *, const u32x4 *);

// The origin comes out of a vector register right in front of the load.
__global__ void load_from_a_fresh_base(const uint16_t *const *rows, uint16_t *out) {
  __shared__ __align__(16) uint16_t lds[512];
  const uint64_t a = (uint64_t)rows[threadIdx.x];
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)), lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  __builtin_amdgcn_sched_barrier(0);
  lds_dma16_untracked((const uint16_t *)(((uint64_t)hi << 32) | lo), threadIdx.x * 16, lds);
  wait_all();
  *reinterpret_cast<u32x4 *>(out + threadIdx.x * 8) = *reinterpret_cast<const u32x4 *>(lds + threadIdx.x * 8);
}
}
"""


def wait_states(instruction):
    m = re.match(r"s_nop (\d+)", instruction)
    return int(m.group(1)) + 1 if m else 1


def registers(operand):
    m = re.match(r"([vs])\[(\d+):(\d+)\]|([vs])(\d+)$", operand.strip().rstrip(","))
    if not m:
        return set()
    if m.group(4):
        return {m.group(4) + m.group(5)}
    return {m.group(1) + str(i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}


def assemble(src, asm):
    """Labels and instructions by kernel."""
    subprocess.run([HIPCC] + FLAGS + ["--offload-device-only", "-S", src, "-o", asm], check=True, capture_output=True)
    out, name = {}, None
    for line in open(asm):
        m = re.match(r"(_Z\w+):", line)
        if m:
            name = m.group(1)
            out[name] = []
        code = line.split(";")[0].strip()
        if name and code and (line[0] in " \t" and code[0] != "." or code.startswith(".LBB")):
            out[name].append(code)
        if line.startswith(".Lfunc_end"):
            name = None
    return out


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    d = tmp_path_factory.mktemp("wait_states")
    src = str(d / "k.hip")
    with open(src, "w") as f:
        f.write(KERNELS)
    return assemble(src, str(d / "k.s"))


def of(kernels, *parts):
    (body,) = [v for k, v in kernels.items() if all(p in k for p in parts)]
    return body


def distances_to_overwrite(body):
    """Wait states between each 16-byte store and the next vector instruction that writes one of its data registers."""
    out = []
    for i, code in enumerate(body):
        if not code.startswith("global_store_dwordx4"):
            continue
        data, states = registers(code.split()[2]), 0
        assert len(data) == 4, code
        for later in body[i + 1:]:
            if later.startswith("v_") and registers(later.split()[1]) & data:
                out.append(states)
                break
            states += wait_states(later)
    return out


def test_data_of_a_write_through_store_outlive_it(kernels):
    """A store of more than 8 bytes reads its data after it has issued: two wait states on gfx950, which the compiler's own
    stores show, whatever instruction follows (none of the ones behind it in the kernels counts here)."""
    known = distances_to_overwrite(of(kernels, "overwrite_behind_store", "Lb0E"))
    written = distances_to_overwrite(of(kernels, "overwrite_behind_store", "Lb1E"))
    assert len(known) >= 3 and len(written) >= 3
    assert min(known) == 2
    assert min(written) >= 2, written


def test_scalar_base_of_an_untracked_load_is_there_when_it_reads_it(kernels):
    """A vector-memory instruction may read a scalar register five wait states after a vector instruction has written it, and
    M0 one after a scalar move: the load that the compiler does not know brings these along."""
    body = of(kernels, "load_from_a_fresh_base")
    (at,) = [i for i, code in enumerate(body) if code.startswith("global_load_lds_dwordx4")]
    base = registers(body[at].split()[2])
    assert len(base) == 2, body[at]
    states, m0 = 0, None
    for before in reversed(body[:at]):
        if before.startswith("s_mov_b32 m0"):
            m0 = states
        if before.startswith("v_readfirstlane") and registers(before.split()[1]) & base:
            break
        assert not registers(before.split()[1] if " " in before else "") & base, before      # (copied by a scalar instruction since)
        states += wait_states(before)
    else:
        pytest.fail("no vector instruction writes the base: %s" % body[:at + 1])
    assert states >= 5 and m0 is not None and m0 >= 1, body[max(0, at - 8):at + 1]


def test_attention_waits_for_its_lds_reads_in_front_of_each_barrier(tmp_path):
    """The key tiles are refilled behind a barrier by direct loads that the compiler does not know: the reads of the tile
    before have to have returned in front of it, by a wait that stands right there."""
    dense = assemble(os.path.join(CSRC, "dense_kernels.hip"), str(tmp_path / "dense.s"))
    barriers = 0
    for name, body in dense.items():
        if "attention" not in name:
            continue
        for i, code in enumerate(body):
            if code != "s_barrier":
                continue
            barriers += 1
            for before in reversed(body[:i]):
                if before.startswith("s_waitcnt") and "lgkmcnt(0)" in before:
                    break
                assert not re.match(r"ds_|\.LBB|s_c?branch", before), (name, body[max(0, i - 8):i + 1])
    assert barriers >= 40
