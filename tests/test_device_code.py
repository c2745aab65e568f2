"""What the compiler made of the kernels, read from the built library: properties that its resource report or a reader of
the source does not show, and that have cost time without changing a result."""
import ctypes as C
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2412_20185_amd as dd
from paper_2412_20185_amd import build

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _tool(name):
    path = shutil.which(name) or os.path.join(LLVM, name)
    if not os.path.exists(path):
        pytest.skip(f"{name} is not installed")
    return path


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code object of every source file, as files."""
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        data = f.read()
    out = tmp_path_factory.mktemp("code")
    paths = []
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            offset, size, idlen = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in target and size:
                paths.append(out / f"{len(paths)}.co")
                paths[-1].write_bytes(data[at + offset:at + offset + size])
        at = data.find(MAGIC, at + 24)
    assert len(paths) >= len(build.SOURCES) - 1, "code objects not found in the library"
    return paths


def _disassembly(path):
    """(kernel name, its instructions) of a code object."""
    text = subprocess.run([_tool("llvm-objdump"), "-d", "--no-show-raw-insn", path], capture_output=True, text=True,
                          check=True).stdout
    name, lines = None, []
    for line in text.splitlines():
        m = re.match(r"[0-9a-f]+ <(.*)>:", line)
        if m:
            if name:
                yield name, lines
            name, lines = m.group(1), []
        else:
            lines.append(line.split("//")[0].strip())
    if name:
        yield name, lines


def test_no_flat_memory_access(code_objects):
    """A pointer whose address space the compiler does not know is accessed by flat instructions, which count as LDS
    accesses too and are waited for together with all of them.  Every pointer here is to global memory or LDS."""
    flat = {}
    for path in code_objects:
        for name, lines in _disassembly(path):
            n = sum(line.startswith(("flat_load", "flat_store", "flat_atomic")) for line in lines)
            if n:
                flat[name] = n
    assert not flat


def test_registers_of_every_kernel(code_objects):
    """No scratch memory, and of the scalar registers at most 24 set aside in vector lanes: pointers and counts that are
    kept for a workgroup's last step.  The sixteen lane masks of a row loop would be 32 more.  The kernels that are meant to
    run with eight wavefronts a SIMD (64 vector registers) stay within the 80 scalar registers that allow it."""
    seen = 0
    for path in code_objects:
        notes = subprocess.run([_tool("llvm-readelf"), "--notes", path], capture_output=True, text=True, check=True).stdout
        for entry in notes.split("  - .agpr_count")[1:]:
            value = lambda key: int(re.search(rf"\.{key}: +(\d+)", entry).group(1))  # noqa: E731
            name = re.search(r"\.name: +(\S+)", entry).group(1)
            seen += 1
            assert value("private_segment_fixed_size") == 0 and value("vgpr_spill_count") == 0, name
            assert value("sgpr_spill_count") <= 24, (name, value("sgpr_spill_count"))
            if "gemv_kernel" in name and value("vgpr_count") <= 64:
                assert value("sgpr_count") <= 80, (name, value("sgpr_count"))
    assert seen > 100


def test_row_requests_of_a_batch_do_not_wait_for_one_another(code_objects):
    """The residual kernels request a batch of rows (4 KiB a wavefront) before they use the first one.  A wait among the
    requests that is not over until one of them has returned would make the batch several trips over the host link.  (2-bit
    rows with the selection supplied take two rows a request and read the row numbers by vector loads, waited for in two
    groups; all of them first was measured slower.)"""
    batch = {16: ("global_load_dwordx4", 4), 8: ("global_load_dwordx2", 8), 4: ("global_load_dword", 16), 2: ("global_load_dword", 16)}
    seen = set()
    for path in code_objects:
        for name, lines in _disassembly(path):
            m = re.search(r"(?:fetch_kernelI|compensated_gemv_kernelILi\d+E)Li(\d+)ELi(\d+)E", name)
            if not m or m.groups() == ("2", "0"):
                continue
            op, rows = batch[int(m.group(1))]
            run, free, found = 0, True, False  # requests in a row, none of them waited for so far
            for line in lines:
                word = line.split(" ")[0]
                if word == op and not line.endswith(" nt"):  # the weight stream is non-temporal
                    run += 1
                    found |= free and run >= rows
                elif word.startswith(("global_load", "global_store", "global_atomic")):
                    run, free = 0, True
                elif (w := re.search(r"^s_waitcnt.*vmcnt\((\d+)\)", line)) and run and run < rows and int(w.group(1)) < run:
                    free = False
            assert found, name
            seen.add((name.split("kernel")[0][-12:],) + m.groups())
    assert len(seen) >= 4 * 5 - 1


def _wait_state_faults(lines):
    """What the compiler does not see inside the asm dots: a register that a DPP operand names must not have been written by
    either of the two vector instructions in front of it, and for three wait states no other kind of instruction may name the
    result of a dot, nor may a dot read it as a factor.  Nothing is left open where the path goes on elsewhere."""
    recent = []   # registers written by the last vector instructions, one entry per wait state
    pending = {}  # results of dots: wait states left
    for line in lines:
        op, _, rest = line.partition(" ")
        regs = re.findall(r"\bv(?:\[(\d+):(\d+)\]|(\d+))", rest)
        regs = [set(range(int(a), int(b) + 1)) if a else {int(c)} for a, b, c in regs]
        states = int(rest, 0) + 1 if op == "s_nop" else 1
        dot = op == "v_dot2c_f32_f16_dpp"
        if dot and any(written & regs[1] for written in recent[-2:]):
            yield line
        named = regs[1] | regs[2] if dot else set().union(*regs)
        if named & pending.keys():
            yield line
        if pending and op.startswith(("s_branch", "s_cbranch", "s_setpc", "s_endpgm")):
            yield line
        pending = {r: n - states for r, n in pending.items() if n > states}
        written = set()
        if op.startswith("v_") and regs:
            written = regs[0] | regs[1] if "swap" in op else regs[0]
        if dot:
            pending.update({r: 3 for r in regs[0]})
        recent = (recent + [written] + [set()] * (states - 1))[-2:]


def test_dots_with_a_shared_activation_are_given_their_wait_states(code_objects):
    seen = {}
    for path in code_objects:
        for name, lines in _disassembly(path):
            if "row_newbcast" not in "".join(lines):
                continue
            family = re.search(r"[a-z_]*gemv_kernel", name).group(0)
            seen[family] = seen.get(family, 0) + 1
            assert not list(_wait_state_faults(lines)), name
    # formats x (columns x workgroup sizes, then those with several tiles on their way); x row formats x selections
    assert seen == {"gemv_kernel": 3 * (3 * 3 + 3 + 2), "compensated_gemv_kernel": 3 * 4 * (2 * 4 + 1)}


@pytest.mark.parametrize("lines,faults", [
    (["v_mov_b32_e32 v5, v9", "v_dot2c_f32_f16_dpp v1, v5, v2 row_newbcast:0 row_mask:0xf bank_mask:0xf", "s_nop 2"], 1),
    (["v_permlane16_swap_b32_e32 v9, v5", "s_nop 0", "v_dot2c_f32_f16_dpp v1, v5, v2 row_newbcast:0", "s_nop 2"], 1),
    (["v_mov_b32_e32 v5, v9", "s_nop 1", "v_dot2c_f32_f16_dpp v1, v5, v2 row_newbcast:0", "s_nop 2", "v_add_f32_e32 v3, v1, v1"], 0),
    (["v_dot2c_f32_f16_dpp v1, v5, v2 row_newbcast:0", "v_dot2c_f32_f16_dpp v1, v6, v2 row_newbcast:0", "s_nop 2"], 0),
    (["v_dot2c_f32_f16_dpp v1, v5, v2 row_newbcast:0", "s_nop 1", "ds_write_b32 v7, v1"], 1),
    (["v_dot2c_f32_f16_dpp v1, v5, v2 row_newbcast:0", "global_store_dword v[8:9], v1, off"], 1),
    (["v_dot2c_f32_f16_dpp v1, v5, v2 row_newbcast:0", "s_nop 0", "v_dot2c_f32_f16_dpp v3, v5, v1 row_newbcast:1", "s_nop 2"], 1),
    (["v_dot2c_f32_f16_dpp v1, v5, v2 row_newbcast:0", "s_cbranch_scc1 12"], 1),
])
def test_wait_states_that_are_missing_are_seen(lines, faults):
    assert len(list(_wait_state_faults(lines))) == faults


def test_workgroups_of_the_one_grid_kernel_per_compute_unit(code_objects):
    """Three workgroups or more fit a compute unit by their LDS, whatever the kernel's own part of it is; exactly three where a
    small base GEMV runs beside a selection over more than 4096 channels and rows behind the link (with 2-bit rows and the
    smallest of them two), and never fewer than the registers allow with a wide one."""
    lds_of = dd.lib()["_ZN6decdec12one_grid_ldsEiiiilb"]
    lds_of.argtypes = [C.c_int] * 4 + [C.c_long, C.c_bool]
    lds_of.restype = C.c_uint
    cu, wavefronts = 160 * 1024, 8
    seen = 0
    for path in code_objects:
        notes = subprocess.run([_tool("llvm-readelf"), "--notes", path], capture_output=True, text=True, check=True).stdout
        for entry in notes.split("  - .agpr_count")[1:]:
            m = re.search(r"compensated_gemv_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi\d+E", re.search(r"\.name: +(\S+)", entry).group(1))
            if not m:
                continue
            seen += 1
            kind, bits, nch = map(int, m.groups())
            own = int(re.search(r"\.group_segment_fixed_size: +(\d+)", entry).group(1))
            vgprs = int(re.search(r"\.vgpr_count: +(\d+)", entry).group(1))
            by_registers = 4 * min(8, 512 // (-(-vgprs // 8) * 8)) // wavefronts
            fit = lambda *a: cu // (own + lds_of(kind, bits, nch, *a))  # noqa: E731
            for k in (1, 64):
                small, wide, near = fit(k, 900, True), fit(k, 1 << 14, True), fit(k, 900, False)
                assert min(small, by_registers) == (3 if nch >= 2 or bits == 2 else 4), m.groups()
                assert min(wide, near) >= by_registers, m.groups()
            if bits == 2 and nch in (2, 4):  # two beside the smallest
                assert fit(1, 600, True) == 2
            if nch:
                assert fit(4096, 900, True) >= 2
    assert seen == 3 * 4 * (2 * 4 + 1)
