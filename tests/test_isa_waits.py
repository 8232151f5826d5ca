"""Instruction sequences of the built kernels that the hardware needs software to keep apart, read from the disassembly of
the library.  The compiler inserts wait states between its own instructions; inside an inline assembly statement, and
between one and what surrounds it, it does not look."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2509_25401_amd import build as hip_build
from paper_2509_25401_amd import library_path

OBJDUMP = os.path.join(os.path.dirname(hip_build.hipcc_path()), "..", "llvm", "bin", "llvm-objdump")
M0 = 124
WAIT_M0_LDS = 1          # scalar write of M0 -> vector-memory load into LDS
WAIT_SGPR_VMEM = 5       # vector write of a scalar register -> vector-memory instruction that reads it
FAR = 5


def functions(text):
    """{name: [(address, mnemonic, operands, branch target or None)]} of a disassembly listing."""
    out, name, start = {}, None, 0
    for line in text.splitlines():
        head = re.match(r"^([0-9a-f]+) <(.*)>:$", line)
        if head:
            start, name = int(head[1], 16), head[2]
            out[name] = []
            continue
        m = re.match(r"^\t(\S+)(?: (.*?))?\s*// ([0-9A-F]+):(.*)$", line)
        if m and name:
            target = re.search(r"<[^>+]*(?:\+0x([0-9a-f]+))?>\s*$", m[4])
            out[name].append((int(m[3], 16), m[1], (m[2] or "").strip(), start + int(target[1] or "0", 16) if target else None))
    return out


def scalars(operands):
    found = set()
    for m in re.finditer(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", operands):
        found |= {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))
    if "vcc" in operands:
        found |= {106, 107}
    if re.search(r"\bm0\b", operands):
        found.add(M0)
    return found


def written_by_vector(op, operands):
    """Scalar registers that a vector instruction writes."""
    if op.startswith("v_cmp") and op.endswith("_e32"):
        return {106, 107}
    args = [a.strip() for a in operands.split(",")]
    if op.startswith(("v_readfirstlane", "v_readlane", "v_cmp")):
        return scalars(args[0])
    if re.match(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_div_scale|v_mad_[ui]64", op):
        return scalars(args[1])
    return set()


def violations(code):
    """Vector-memory instructions that some path reaches too early, as (address, mnemonic, operands, register).  The state
    in front of an instruction is how many wait states ago each scalar register was written, least over all paths."""
    index = {ins[0]: i for i, ins in enumerate(code)}
    before, todo, bad = {0: {}}, [0], set()
    while todo:
        i = todo.pop()
        address, op, operands, target = code[i]
        state = before[i]
        if op.startswith(("buffer_", "global_", "flat_", "scratch_")):
            for r in scalars(operands):
                if state.get(("vector", r), FAR) < WAIT_SGPR_VMEM:
                    bad.add((address, op, operands, r))
            if ("_lds_" in op or operands.endswith(" lds")) and state.get("m0", FAR) < WAIT_M0_LDS:
                bad.add((address, op, operands, M0))
        waits = int(operands, 0) + 1 if op == "s_nop" else 1
        after = {k: v + waits for k, v in state.items() if v + waits < FAR}
        if op.startswith("v_"):
            after.update({("vector", r): 0 for r in written_by_vector(op, operands)})
        elif op.startswith("s_") and not op.startswith(("s_cmp", "s_bitcmp", "s_nop", "s_waitcnt", "s_cbranch", "s_branch")):
            for r in scalars(operands.split(",")[0]):
                after.pop(("vector", r), None)
                if r == M0:
                    after["m0"] = 0
        following = [] if op in ("s_branch", "s_endpgm", "s_setpc_b64") else [i + 1]
        if op.startswith(("s_branch", "s_cbranch")):
            following.append(index[target])
        for n in following:
            if n >= len(code):
                continue
            old = before.get(n)
            new = after if old is None else {k: min(old.get(k, FAR), after.get(k, FAR)) for k in old.keys() | after.keys()}
            if new != old:
                before[n] = new
                todo.append(n)
    return bad


def unawaited(code):
    """Atomics with a result that are not waited for before anything else than the exec mask is touched: all of them are
    issued in assembly statements, whose outputs the compiler takes for written at the end of the statement."""
    bad = []
    for i, (address, op, operands, _) in enumerate(code):
        if op.startswith("global_atomic") and operands.endswith(" sc0"):
            rest = [ins for ins in code[i + 1:i + 4] if not (ins[1] == "s_mov_b64" and ins[2].startswith("exec"))]
            if not rest or rest[0][1] != "s_waitcnt" or "vmcnt(0)" not in rest[0][2]:
                bad.append((address, op, operands))
    return bad


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    where = tmp_path_factory.mktemp("isa")
    shutil.copy(library_path(), where / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=where, check=True, stdout=subprocess.DEVNULL)
    found = {}
    for part in sorted(where.glob("*gfx950*")):
        if part.stat().st_size:
            listing = subprocess.run([OBJDUMP, "-d", part.name], cwd=where, check=True, stdout=subprocess.PIPE, text=True).stdout
            for name, code in functions(listing).items():
                found[f"{part.name}:{name}"] = code
    assert any("attn_kernel" in name for name in found) and any("gemm_q" in name for name in found)
    return found


def listing(*lines):
    return functions("0000000000000000 <k>:\n" + "".join(f"\t{line} // {4 * n:012X}: 00000000{where}\n" for n, (line, where) in enumerate(lines)))["k"]


@pytest.mark.parametrize("lines,expect", [
    ([("s_mov_b32 m0, s4", ""), ("global_load_lds_dwordx4 v1, s[2:3]", "")], 1),
    ([("s_mov_b32 m0, s4", ""), ("s_nop 0", ""), ("global_load_lds_dwordx4 v1, s[2:3]", "")], 0),
    ([("s_add_u32 m0, s4, 64", ""), ("buffer_load_dwordx4 v1, s[4:7], s2 offen lds", "")], 1),
    ([("s_add_u32 m0, s4, 64", ""), ("s_add_u32 s2, s3, s8", ""), ("buffer_load_dwordx4 v1, s[4:7], s2 offen lds", "")], 0),
    ([("s_mov_b32 m0, s4", ""), ("global_load_dwordx4 v[4:7], v1, s[2:3]", "")], 0),
    ([("v_readfirstlane_b32 s3, v0", ""), ("s_nop 3", ""), ("global_load_dword v1, v2, s[2:3]", "")], 1),
    ([("v_readfirstlane_b32 s3, v0", ""), ("s_nop 4", ""), ("global_load_dword v1, v2, s[2:3]", "")], 0),
    ([("v_readlane_b32 s3, v0, 1", ""), ("s_mov_b32 s3, 0", ""), ("global_load_dword v1, v2, s[2:3]", "")], 0),
    # around a loop: the write stands behind the load
    ([("s_nop 4", ""), ("global_load_lds_dwordx4 v1, s[2:3]", ""), ("s_mov_b32 m0, s4", ""), ("s_cbranch_scc1 65533", " <k+0x4>"), ("s_endpgm", "")], 0),
    ([("s_nop 4", ""), ("global_load_lds_dwordx4 v1, s[2:3]", ""), ("v_readlane_b32 s2, v0, 1", ""), ("s_cbranch_scc1 65533", " <k+0x4>"), ("s_endpgm", "")], 1),
])
def test_what_counts_as_too_early(lines, expect):
    assert len(violations(listing(*lines))) == expect


def test_wait_states_in_front_of_memory_instructions(kernels):
    to_lds = sum("_lds_" in op or args.endswith(" lds") for code in kernels.values() for _, op, args, _ in code)
    assert to_lds > 0
    bad = {name: sorted(violations(code)) for name, code in kernels.items()}
    count = sum(len(v) for v in bad.values())
    first = next((f"{name}: {v[0][1]} {v[0][2]}" for name, v in bad.items() if v), "")
    assert count == 0, f"{count} of them come too early, for instance {first}"


def test_tickets_are_waited_for_where_they_are_drawn(kernels):
    attention = {name: code for name, code in kernels.items() if "attn_kernel" in name}
    assert sum(op.startswith("global_atomic") for code in attention.values() for _, op, _, _ in code) > 0
    bad = {name: unawaited(code) for name, code in attention.items()}
    assert not any(bad.values()), f"{sum(map(len, bad.values()))} of them, for instance {next(v[0] for v in bad.values() if v)}"
