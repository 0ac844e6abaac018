"""The written-out loads into LDS (csrc/sc_lds_load.h) carry their own wait
states: the compiler's hazard pass does not look into an asm block.  A probe
whose buffer resource, LDS address and size come straight from vector
registers is compiled, not run, and its assembly read."""

import re
import subprocess

import pytest

from paper_2606_16135_amd import build

PROBE = r"""
#include "sc_lds_load.h"
__shared__ __attribute__((aligned(1024))) unsigned char tiles[2 * 4096];
extern "C" __global__ __launch_bounds__(64) void probe(const uint32_t *p, float *out) {
  const uint32_t *const q = p + 8 * threadIdx.x;
  int voff[LOADS];
  for (int i = 0; i < LOADS; ++i) voff[i] = q[4 + i];
  for (int r = 0; r < 2; ++r) {
    const uint64_t base = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)q[1 + r]) << 32 |
                          (uint32_t)__builtin_amdgcn_readfirstlane((int)q[r]);
    sc::load_to_lds(4096 * r, voff, base, (uint32_t)__builtin_amdgcn_readfirstlane((int)q[3]));
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  out[threadIdx.x] = reinterpret_cast<float *>(tiles)[threadIdx.x];
}
"""


def _instructions(text):
    out = []
    for line in text.splitlines():
        line = line.split(";")[0].strip()
        m = re.match(r"([a-z]\w*)\s+(.*)", line)
        if m and not line.endswith(":"):
            out.append((m[1], re.findall(r"[\w.]+(?:\[[^\]]*\])?", m[2])))
    return out


def _registers(operand, kind="s"):
    if operand == kind:
        return {kind}
    m = re.fullmatch(kind + r"(?:\[(\d+):(\d+)\]|(\d+))", operand)
    return set() if m is None else {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def _wait_states(op, operands):
    return int(operands[0], 0) + 1 if op == "s_nop" else 1


def close_writes(instructions):
    """(load, writer) pairs: a scalar register of the load written by a
    vector instruction fewer than five wait states before it, or M0 written
    by a scalar one with none between."""
    found = []
    for i, (op, operands) in enumerate(instructions):
        if not op.startswith("buffer_load") or "lds" not in operands:
            continue
        used = set().union(*(_registers(x) for x in operands))
        assert used
        states = 0
        for j in range(i - 1, -1, -1):
            o, x = instructions[j]
            if states >= 5:
                break
            if o.startswith("v_") and x and _registers(x[0]) & used:
                found.append((operands, (o, x)))
            if o.startswith("s_") and x and x[0] == "m0" and states < 1:
                found.append((operands, (o, x)))
            states += _wait_states(o, x)
    return found


def test_scanner_finds_a_close_write():
    load = ("buffer_load_dwordx4", ["v1", "s[4:7]", "0", "offen", "lds"])
    bad = [("v_readlane_b32", ["s6", "v9", "3"]), ("s_mov_b32", ["m0", "s8"]), ("s_nop", ["0"]), load]
    assert len(close_writes(bad)) == 1
    assert not close_writes(bad[:1] + [("s_nop", ["4"])] + bad[1:])
    assert len(close_writes([("s_mov_b32", ["m0", "s8"]), load])) == 1


@pytest.mark.parametrize("loads", [1, 4])
def test_loads_into_lds_keep_their_wait_states(loads, tmp_path):
    src, asm = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    cmd = [build._hipcc()] + build.COMMON_FLAGS + [
        "-I" + build.CSRC, f"-DLOADS={loads}", "-x", "hip", "--cuda-device-only", "-S", str(src), "-o", str(asm)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    ins = _instructions(asm.read_text())
    assert sum(op.startswith("buffer_load") and "lds" in x for op, x in ins) == 2 * loads
    assert any(op == "v_readfirstlane_b32" for op, _ in ins)
    assert close_writes(ins) == []
