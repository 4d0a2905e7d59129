"""What the compiler makes of indexed registers beside matrix instructions (fused_slab_bf16.hip): an indexed move must keep 8 wait states
from a 16 x 16 x 32 matrix instruction whose result it touches, and the compiler counts the s_set_gpr_idx_on between them as one.
The kernel puts an addition there; this reads the assembly of this source, built as the library builds it and with the
option under which an addition of plain zero vanishes."""
import re
import subprocess

import pytest

from paper_2306_08367_amd import build

WAIT_STATES = 8


def _registers(operand):
    m = re.match(r"v\[(\d+):(\d+)\]|v(\d+)\b", operand)
    if not m:
        return set()
    return {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def _functions(assembly):
    """Per function: [(mnemonic, operands)], a label as (None, name)."""
    functions, body = [], None
    for line in assembly.splitlines():
        line = line.split(";")[0].strip()
        if re.match(r"_Z\w+:$", line):
            body = []
            functions.append(body)
        elif body is not None and re.match(r"\.LBB\w+:$", line):
            body.append((None, line[:-1]))
        elif body is not None and line and line[0] not in ".#":
            op, _, rest = line.partition(" ")
            body.append((op.strip(), [r.strip() for r in rest.split(",")]))
    return functions


def _waits(body):
    """Wait states on every way from a matrix instruction to the first indexed move that touches its result."""
    at = {operands: i for i, (op, operands) in enumerate(body) if op is None}
    indexed, inside = set(), False
    for i, (op, _) in enumerate(body):
        inside = (inside or op == "s_set_gpr_idx_on") and op != "s_set_gpr_idx_off"
        if inside:
            indexed.add(i)
    for start, (op, operands) in enumerate(body):
        if not (op or "").startswith("v_mfma"):
            continue
        result, ways, seen = _registers(operands[0]), [(start + 1, 0)], {}
        while ways:
            i, waited = ways.pop()
            if i >= len(body) or waited >= 2 * WAIT_STATES or seen.get(i, 99) <= waited:
                continue
            seen[i] = waited
            op, operands = body[i]
            if op is None:
                ways.append((i + 1, waited))
                continue
            if op.startswith(("v_", "ds_", "global_", "flat_", "scratch_")) and any(_registers(r) & result for r in operands):
                if i in indexed:
                    yield waited
                continue                     # (an ordinary instruction: the compiler keeps its distance)
            if op.startswith(("s_branch", "s_cbranch")):
                ways.append((at[operands[0]], waited + 1))
            if op not in ("s_branch", "s_endpgm"):
                ways.append((i + 1, waited + (int(operands[0], 0) + 1 if op == "s_nop" else 0 if op.startswith("s_set_gpr_idx") else 1)))


@pytest.mark.parametrize("options", [[], ["-ffast-math"]], ids=["as-built", "fast-math"])
def test_indexed_moves_keep_their_distance(options, tmp_path):
    out = tmp_path / "slab.s"
    r = subprocess.run([build.hipcc(), *build.FLAGS, *options, "--offload-device-only", "-S", f"{build.CSRC}/fused_slab_bf16.hip", "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    functions = _functions(out.read_text())
    assert any(op == "s_set_gpr_idx_on" for body in functions for op, _ in body) and len(functions) > 48, "the kernels were not found"
    assert all(waited >= WAIT_STATES for body in functions for waited in _waits(body))
