"""The machine code that the library's own kernels were compiled to, looked over without a GPU: what their source leaves
to the compiler because it writes matrix instructions as assembly, of which the compiler knows no timing."""
import re
import shutil
import struct
import subprocess

import pytest

from paper_2412_14363_amd import build

OBJDUMP = shutil.which("llvm-objdump", path="/opt/rocm/llvm/bin") or shutil.which("llvm-objdump")


@pytest.fixture(scope="module")
def code_object(tmp_path_factory):
    """the library's own gfx950 code, as a file"""
    if not OBJDUMP:
        pytest.skip("no llvm-objdump")
    data = build.ensure_built().read_bytes()
    bundle = data[data.index(b"__CLANG_OFFLOAD_BUNDLE__"):]
    count, at = struct.unpack_from("<Q", bundle, 24)[0], 32
    code = None
    for _ in range(count):   # offset, size, length of the target's name, the name
        offset, size, length = struct.unpack_from("<QQQ", bundle, at)
        if b"gfx950" in bundle[at + 24:at + 24 + length]:
            code = bundle[offset:offset + size]
        at += 24 + length
    path = tmp_path_factory.mktemp("code") / "gfx950.co"
    path.write_bytes(code)
    return path


@pytest.fixture(scope="module")
def kernels(code_object):
    """name -> instructions of every kernel with matrix instructions in assembly"""
    path = code_object
    symbols = subprocess.run([OBJDUMP, "-t", str(path)], capture_output=True, text=True, check=True).stdout
    names = sorted(set(re.findall(r"\s(_Z\w*(?:gemm_mixed_\w*kernel|project_split_wide_kernel)\w*)$", symbols, re.M)))
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--disassemble-symbols=" + ",".join(names), str(path)],
                          capture_output=True, text=True, check=True).stdout
    found, cur = {}, None
    for line in text.splitlines():
        if m := re.match(r"[0-9a-f]+ <(\S+)>:", line):
            cur = found.setdefault(m[1], [])
        elif cur is not None and line.strip():
            cur.append(re.sub(r"\s*//.*", "", line).strip())
    assert len(found) == len(names) >= 10
    return found


def registers(operand):
    m = re.match(r"([av])(?:(\d+)$|\[(\d+):(\d+)\])", operand.strip().split(" ")[0])
    if not m:
        return set()
    lo, hi = (m[2], m[2]) if m[2] else (m[3], m[4])
    return {(m[1], i) for i in range(int(lo), int(hi) + 1)}


def test_tiles_are_read_behind_the_wait(kernels):
    """The kernels end their products with a wait of 32 states; nothing between the last product and the wait touches a
    register that a product writes."""
    for name, ins in kernels.items():
        ops = [(i.split(" ", 1)[0], i.split(" ", 1)[1].split(",") if " " in i else []) for i in ins]
        tiles = set().union(*(registers(o[0]) for m, o in ops if m.startswith("v_mfma")))
        waits = [i for i in range(len(ins) - 1) if ins[i] == ins[i + 1] == "s_nop 15"]
        assert waits, name
        for w in waits:
            last = max(i for i in range(w) if ops[i][0].startswith("v_mfma"))
            early = [ins[i] for i in range(last + 1, w) if any(registers(x) & tiles for x in ops[i][1])]
            assert not early, (name, len(early), early[:3])


def test_operands_are_ready_two_states_before_a_product(kernels):
    """What the vector ALU writes is read by a matrix instruction two wait states later at the earliest."""
    for name, ins in kernels.items():
        state, written = 0, []
        for i in ins:
            m, _, rest = i.partition(" ")
            ops = rest.split(",")
            if m == "s_nop":
                state += int(ops[0], 0) + 1
                continue
            state += 1
            if m.startswith("v_mfma"):
                used = set().union(*(registers(x) for x in ops[1:4]))
                late = [w for s, r, w in written if state - s <= 2 and r & used]
                assert not late, (name, late, i)
            elif m.startswith("v_"):
                written = written[-3:] + [(state, registers(ops[0]), i)]


def test_stream_kernels_of_one_token_group_leave_room_for_a_second_workgroup(code_object):
    """Launches of more than 256 workgroups count on two to a compute unit: 8 wavefronts each, so 4 on a SIMD, 128 registers
    of 512, and no spills.  (With eight runs to a group LDS holds one workgroup anyway.)"""
    notes = subprocess.run([re.sub("objdump$", "readelf", OBJDUMP), "--notes", str(code_object)], capture_output=True, text=True,
                           check=True).stdout
    found = {}
    for entry in notes.split("- .agpr_count:")[1:]:
        name = re.search(r"\.name:\s+(\S+)", entry)[1]
        if m := re.search(r"gemm_stream_kernelILb0ELi1ELi([124])ELb([01])E", name):
            found[m.groups()] = tuple(int(re.search(r"\.%s:\s+(\d+)" % key, entry)[1])
                                      for key in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size"))
    assert len(found) == 6, found
    assert all(count <= 128 and not spilled and not scratch for count, spilled, scratch in found.values()), found
