"""Inline assembly that reads the result of a matrix instruction: the compiler adds wait states between an MFMA and
its own instructions, but does not look into inline assembly, so there the source has to keep the distance.
Checked without a GPU, in the assembly that the compiler writes for the kernels."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2505_19609_amd import build

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")

PROBE = """
#include "mfma.h"
__global__ void probe(const bf16x8 *a, const bf16x8 *b, float *o)
{
    f32x16 s;
    for (int v = 0; v < 16; ++v) s[v] = 0.0f;
    s = mfma32(a[threadIdx.x], b[threadIdx.x], s);
    o[threadIdx.x] = s[0] * s[1];
}
"""
REGS = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+))")


def _assembly(src, out):
    subprocess.run(["hipcc", *build.FLAGS, "-w", "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True,
                   capture_output=True)
    return out.read_text()


def _registers(text):
    found = set()
    for kind, lo, hi, one in REGS.findall(text):
        found |= {(kind, i) for i in (range(int(lo), int(hi) + 1) if lo else (int(one),))}
    return found


def _kernels(text):
    """{name: [label or (opcode, operands, line at which its inline assembly begins or 0, line)]}"""
    found, code, inline = {}, None, 0
    for number, line in enumerate(text.splitlines(), 1):
        if "#ASMSTART" in line or "#ASMEND" in line:
            inline = number if "#ASMSTART" in line else 0
            continue
        label = re.match(r"([\w.$]+):", line)
        if label:
            if label.group(1).startswith("_Z"):
                code = found.setdefault(label.group(1), [])
            elif label.group(1).startswith(".Lfunc_end"):
                code = None
            elif code is not None:
                code.append(label.group(1))
            continue
        words = line.split(";")[0].split(None, 1)
        if code is not None and words and not words[0].startswith("."):
            code.append((words[0], words[1].strip() if len(words) > 1 else "", inline, number))
    return {n: c for n, c in found.items() if any(i[0].startswith("v_mfma") for i in c if not isinstance(i, str))}


def _states(op, operands):
    return int(operands, 0) + 1 if op == "s_nop" else 1


def _too_early(code, needed):
    """Vector and memory instructions that touch a register fewer than `needed` wait states after the MFMA that writes
    it, on any path; every instruction counts as one state, whatever it really takes."""
    at = {c: i for i, c in enumerate(code) if isinstance(c, str)}
    entry, work, bad = {0: {}}, [0], []
    while work:
        i = work.pop()
        left = dict(entry[i])  # register -> wait states still to pass
        leads_to = []
        for j in range(i, len(code)):
            if isinstance(code[j], str):
                if j > i:
                    leads_to.append(j)
                    break
                continue
            op, operands, inline, number = code[j]
            matrix = op.startswith("v_mfma")
            if not matrix and op.startswith(("v_", "ds_", "buffer_", "global_", "flat_")):
                bad += [(number, op, inline, r) for r in _registers(operands) if r in left]
            left = {r: n - _states(op, operands) for r, n in left.items() if n > _states(op, operands)}
            if matrix:
                left.update(dict.fromkeys(_registers(operands.split(",")[0]), needed))
            if op.startswith(("s_branch", "s_cbranch")):
                leads_to.append(at[operands])
            if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                break
        for t in leads_to:
            seen = entry.get(t)
            merged = {r: max(left.get(r, 0), (seen or {}).get(r, 0)) for r in left.keys() | (seen or {}).keys()}
            if seen != merged:
                entry[t] = merged
                work.append(t)
    return bad


@pytest.fixture(scope="module")
def needed(tmp_path_factory):
    """Wait states that the compiler itself puts between the MFMA and a vector instruction that reads its result."""
    d = tmp_path_factory.mktemp("probe")
    (d / "probe.hip").write_text(PROBE)
    (code,) = _kernels(_assembly(d / "probe.hip", d / "probe.s")).values()
    code = [c for c in code if not isinstance(c, str)]
    first = next(i for i, c in enumerate(code) if c[0].startswith("v_mfma"))
    result = _registers(code[first][1].split(",")[0])
    reader = next(i for i in range(first + 1, len(code)) if _registers(code[i][1]) & result)
    n = sum(_states(c[0], c[1]) for c in code[first + 1:reader])
    assert n > 1 and not _too_early(code, n) and _too_early(code, n + 1)
    return n


@pytest.fixture(scope="module", params=["fwd.hip", "bwd.hip"])
def kernels(request, tmp_path_factory):
    out = tmp_path_factory.mktemp("kernels") / (request.param + ".s")
    return _kernels(_assembly(os.path.join(build.CSRC, request.param), out))


def test_waits_written_by_hand_are_as_long_as_the_compiler_s(kernels, needed):
    for name, code in kernels.items():
        blocks = {}
        for c in code:
            if not isinstance(c, str) and c[2]:
                blocks.setdefault(c[2], []).append(c)
        for begin, block in blocks.items():  # (a wait between two instructions of one block is for something else)
            if all(c[0] == "s_nop" for c in block):
                assert sum(_states(c[0], c[1]) for c in block) >= needed, (name, begin)


def test_no_instruction_reads_a_matrix_result_early(kernels, needed):
    for name, code in kernels.items():
        assert not _too_early(code, needed), name
