"""Properties of the compiled kernels that no run shows reliably, read from the gfx950 code objects of the built libfc.so
(the AMD assembly of this repository's own sources)."""
import os
import re
import struct
import subprocess

import pytest

from paper_2412_04964_amd import build

LLVM = os.path.join(os.path.dirname(os.path.dirname(build.HIPCC)), "llvm", "bin")
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """the gfx950 ELF images of the offload bundles in a library"""
    blob = open(path, "rb").read()
    at = blob.find(BUNDLE)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + 24)
        entry = at + 32
        for _ in range(n):
            offset, size, name_len = struct.unpack_from("<QQQ", blob, entry)
            name = blob[entry + 24:entry + 24 + name_len]
            entry += 24 + name_len
            if build.ARCH.encode() in name and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(BUNDLE, at + 24)


def test_no_kernel_uses_scratch_memory(tmp_path):
    # a register that spills goes through memory in every wavefront; one of the rotated dequantizers was 1 to 5 % slower for it
    tool = os.path.join(LLVM, "llvm-readelf")
    if not os.path.exists(tool):
        pytest.skip("no llvm-readelf beside the compiler")
    seen, elf = 0, tmp_path / "code.elf"
    for image in code_objects(build.LIB):
        elf.write_bytes(image)
        notes = subprocess.run([tool, "--notes", str(elf)], check=True, capture_output=True, text=True).stdout
        names = re.findall(r"\.name:\s+(_Z\S+)", notes)
        scratch = re.findall(r"\.private_segment_fixed_size:\s+(\d+)", notes)
        assert len(names) == len(scratch)
        spilled = [n for n, size in zip(names, scratch) if int(size)]
        assert not spilled, spilled[0]
        seen += len(names)
    assert seen > 0


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: [instruction, ...]} of every kernel of the library"""
    tool = os.path.join(LLVM, "llvm-objdump")
    if not os.path.exists(tool):
        pytest.skip("no llvm-objdump beside the compiler")
    found = {}
    folder = tmp_path_factory.mktemp("code")
    for i, image in enumerate(code_objects(build.LIB)):
        elf = folder / ("%d.elf" % i)
        elf.write_bytes(image)
        text = subprocess.run([tool, "-d", "--no-show-raw-insn", "--no-leading-addr", str(elf)], check=True,
                              capture_output=True, text=True).stdout
        body = None
        for line in text.splitlines():
            head = re.match(r"(?:[0-9a-f]+ )?<(\S+)>:", line)
            if head:
                body = found.setdefault(head.group(1), [])
            elif body is not None and line.strip():
                body.append(line.split("//")[0].strip())
    assert found, "no code object in %s" % build.LIB
    return found


BUFFER = re.compile(r"buffer_(load|store)\S* (?:(?P<data>\S+), )?\S+, s\[\d+:\d+\], (?P<offset>\S+)")


def scalar_offset(instruction):
    """the match of a buffer access whose scalar offset is a register"""
    m = BUFFER.match(instruction)
    return m if m and not re.fullmatch(r"-?\d+|0x[0-9a-f]+|off", m.group("offset")) else None


def test_partial_rotation_tiles_have_no_scalar_offset(kernels):
    # The last tile of blocks of 1024 and 2048 may be a partial one, so its accesses lean on the range check, which a
    # scalar offset is not part of (what it does where that offset alone passes the end is not documented).
    seen = 0
    for name, body in kernels.items():
        if not re.search(r"(quantize|allreduce)_rotI.*ELi1[01]EE", name):
            continue
        seen += 1
        bad = [i for i in body if scalar_offset(i)]
        assert not bad, "%s: %s" % (name, bad[0])
    assert seen == 2 * (5 + 5 + 3)                 # two blocks; quantizer and dequantizer with five codes, all-reduce with three


def test_partial_tiles_of_sources_side_by_side_have_no_scalar_offset(kernels):
    # the same for the form of the all-reduce in which the sources of a block go side by side
    spread = {name: body for name, body in kernels.items() if re.search(r"allreduce_rot_spreadI.*ELi1[01]EE", name)}
    assert len(spread) == 2 * 3
    for name, body in spread.items():
        bad = [i for i in body if scalar_offset(i)]
        assert not bad, "%s: %s" % (name, bad[0])


def registers(operand):
    """v7 -> {7}, v[4:7] -> {4, 5, 6, 7}; anything else -> empty"""
    m = re.fullmatch(r"v(?:(\d+)|\[(\d+):(\d+)\])", operand)
    return set() if not m else {int(m.group(1))} if m.group(1) else set(range(int(m.group(2)), int(m.group(3)) + 1))


def test_wide_stores_with_a_scalar_offset_keep_their_data(kernels):
    # A 96- or 128-bit store reads its data registers after it has issued; where its scalar offset is a register the compiler
    # does not wait.  The wait state must follow before any of the data registers is written again.
    seen = 0
    for name, body in kernels.items():
        for at, instruction in enumerate(body):
            m = scalar_offset(instruction) if re.match(r"buffer_store_dwordx[34]\b", instruction) else None
            if not m:
                continue
            seen += 1
            data = registers(m.group("data"))
            assert data, instruction
            for later in body[at + 1:]:
                if later.startswith("s_nop"):
                    break
                assert not later.startswith(("s_endpgm", "s_branch", "s_cbranch", "s_setpc")), "%s: no wait after %s" % (name, instruction)
                operands = later.split(None, 1)[1].split(",") if " " in later else [""]
                written = [] if later.startswith(("buffer_store", "global_store", "ds_write", "s_")) else operands[:1]
                assert not any(registers(w.strip()) & data for w in written), "%s: %s overwrites %s" % (name, later, instruction)
    assert seen > 0


def assembled(tmp_path, source):
    """(kernel, [(instruction, number of the asm statement it was written in or None), ...]) of a source file"""
    out = tmp_path / (source + ".s")
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(out)],
                   check=True, capture_output=True)
    name, body, statement, inside = None, [], 0, False
    for line in out.read_text().splitlines():
        head = re.match(r"(_Z\w+):", line)
        if head:
            if name:
                yield name, body
            name, body = head.group(1), []
        elif "#ASMSTART" in line:
            statement, inside = statement + 1, True
        elif "#ASMEND" in line:
            inside = False
        elif name:
            text = line.split(";")[0].strip()
            if text and not text.startswith(".") and not text.endswith(":"):
                body.append((text, statement if inside else None))
    if name:
        yield name, body


@pytest.mark.parametrize("source", ["fc_rot.hip", "fc_rot_rows.hip", "fc_rot_sim.hip"])
def test_lane_exchanges_wait_for_what_assembly_wrote(tmp_path, source):
    # v_permlane*_swap and DPP operands need two wait states behind the vector instruction that wrote them.  The compiler sees to
    # that for its own instructions but not for those of asm statements: there the source has to, by an asm statement of s_nop
    # alone or by what follows the write in its own statement.  What else happens to lie between is the compiler's choice of the day.
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    seen = 0
    for name, body in assembled(tmp_path, source):
        written, waits = {}, {}                           # of every register: the asm statement that wrote it last; wait states since
        for at, (text, statement) in enumerate(body):
            op, _, rest = text.partition(" ")
            operands = [o.strip().split(" ")[0].strip("-|") for o in rest.split(",")]
            swap = op.startswith("v_permlane")
            if swap or "_dpp" in op:
                seen += 1
                if statement is None:
                    for r in set().union(*(registers(o) for o in (operands[:2] if swap else operands[1:2]))):
                        assert r not in written or waits[r] >= 2, "%s: %s, %d wait states behind an asm statement" % (name, text, waits[r])
            if op == "s_nop" and statement is not None:
                near = [s for _, s in body[max(at - 1, 0):at + 2]]
                alone = near.count(statement) == 1        # the only instruction of its statement
                for r in written:
                    if alone or written[r] == statement:
                        waits[r] += int(rest, 0) + 1
            elif statement is not None:
                for r in written:
                    waits[r] += written[r] == statement
            targets = operands[:2] if swap else operands[:1] if op.startswith(("v_", "buffer_load", "global_load", "ds_")) else []
            for r in set().union(*(registers(o) for o in targets)):
                written.pop(r, None)
                if statement is not None and op.startswith("v_"):
                    written[r], waits[r] = statement, 0
    assert seen > 0


def test_rotated_tiles_are_loaded_before_anything_waits(kernels):
    # A wavefront of the rotation kernels loads one tile and lives for it: a load behind the wait for another one costs a launch-bound call
    # the latency of memory once more.  (The all-reduce loads its first source so, and later ones further down.)
    seen = 0
    for name, body in kernels.items():
        if not re.search(r"(quantize|dequantize|allreduce)_rotI", name):
            continue
        seen += 1
        loads = [at for at, i in enumerate(body) if i.startswith("buffer_load")]
        wait = next(at for at, i in enumerate(body) if i.startswith("s_waitcnt") and "vmcnt" in i)
        first = 4 if "allreduce" in name else len(loads)
        assert sum(at < wait for at in loads) >= first >= 4, "%s: %d of %d loads before the first wait" % (name, sum(at < wait for at in loads), first)
    assert seen >= 4 * (5 + 5 + 3)                 # four blocks; quantizer and dequantizer with five codes, all-reduce with three
