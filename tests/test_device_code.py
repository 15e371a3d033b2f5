"""The built library's gfx950 code as the compiler left it (no GPU needed): what source and results cannot show."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2412_16112_amd.build import LIB

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """Paths of the gfx950 code objects inside the library."""
    where = tmp_path_factory.mktemp("code")
    lib = shutil.copy(LIB, where / "lib.so")
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", str(lib)], check=True, stdout=subprocess.DEVNULL, cwd=where)
    found = sorted(str(f) for f in where.iterdir() if f.name.endswith("gfx950"))
    assert len(found) >= 8
    return found


def instructions(code_object):
    """(kernel, [instruction, ...]) of every kernel, in program order."""
    text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", code_object], check=True, capture_output=True, text=True).stdout
    kernel, body = None, []
    for line in text.splitlines():
        start = re.match(r"[0-9a-f]+ <(\w+)>:$", line)
        if start:
            if kernel:
                yield kernel, body
            kernel, body = start.group(1), []
        elif line.startswith("\t"):
            body.append(line.split("//")[0].strip())
    if kernel:
        yield kernel, body


def scalars(operand):
    """Numbers of the scalar registers that an operand names."""
    m = re.fullmatch(r"s\[(\d+):(\d+)\]|s(\d+)", operand)
    if not m:
        return set()
    return {int(m.group(3))} if m.group(3) else set(range(int(m.group(1)), int(m.group(2)) + 1))


def hazards(body):
    """LDS-direct loads of one kernel that follow too closely on a write of M0 (one wait state between them) or on a vector
    instruction's write of their scalar base (five); the number of such loads beside them.  An instruction is one wait state,
    s_nop N is N + 1.  The states are counted backwards in program order: a jump into the middle would have to land inside them."""
    bad, loads = [], 0
    for at, load in enumerate(body):
        if not load.startswith("global_load_lds"):
            continue
        loads += 1
        base = scalars(load.split()[2])
        states, i = 0, at - 1
        while i >= 0 and states < 5:
            op, _, rest = body[i].partition(" ")
            operands = [x.strip() for x in rest.split(",")]
            written = operands[0]
            if op.startswith("s_") and written == "m0" and states < 1:
                bad.append((body[i], load))
            # (a carry or a comparison writes its first or second operand; v_readlane and v_readfirstlane their first)
            if op.startswith("v_") and any(scalars(x) & base for x in (operands[:2] if re.search("_co_|mad_[ui]64|div_scale", op) else operands[:1])):
                bad.append((body[i], load))
            states += int(operands[0]) + 1 if op == "s_nop" else 1
            i -= 1
    return bad, loads


def test_the_scan_sees_a_hazard():
    assert hazards(["v_readlane_b32 s5, v1, 2", "s_mov_b32 m0, s9", "s_nop 0", "global_load_lds_dwordx4 v7, s[4:5]"])[0]
    assert hazards(["s_mov_b32 m0, s9", "global_load_lds_dword v[6:7], off"])[0]
    assert hazards(["v_readlane_b32 s5, v1, 2", "s_mov_b32 m0, s9", "s_nop 3", "global_load_lds_dwordx4 v7, s[4:5] offset:64"]) == ([], 1)


def test_wait_states_of_lds_direct_loads(code_objects):
    """The loads are inline asm, which the compiler's hazard recogniser does not look into: a base register read while a
    v_readlane is still writing it would be a wild address, and M0 says where in LDS the data goes."""
    loads = 0
    for path in code_objects:
        for kernel, body in instructions(path):
            bad, n = hazards(body)
            loads += n
            assert not bad, "%s: %d of %d loads, the first %s" % (kernel, len(bad), n, bad[0])
    assert loads > 1000


def test_backward_kernels_spill_no_vector_register(code_objects):
    """A reload from scratch memory waits for every load issued before it, the staged tiles in front included."""
    spills = {}
    for path in code_objects:
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", path], check=True, capture_output=True, text=True).stdout
        for kernel in notes.split("- .agpr_count")[1:]:
            name = re.search(r"\.name: +(_Z\w+)\n", kernel).group(1)
            if "clear_bwd" in name:
                spills[name] = int(re.search(r"\.vgpr_spill_count: +(\d+)", kernel).group(1))
    assert len(spills) >= 22
    assert not {k: n for k, n in spills.items() if n}
