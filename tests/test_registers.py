"""What the compiler made of the kernels: the metadata of the code object inside the built library."""
import re
import struct
import subprocess

import pytest

from paper_2508_21230_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def code_object(path):
    """The gfx950 ELF out of a library's offload bundle."""
    raw = open(path, "rb").read()
    at = raw.index(b"__CLANG_OFFLOAD_BUNDLE__")
    (entries,) = struct.unpack_from("<Q", raw, at + 24)
    here = at + 32
    for _ in range(entries):
        offset, size, length = struct.unpack_from("<QQQ", raw, here)
        if b"gfx950" in raw[here + 24:here + 24 + length]:
            return raw[at + offset:at + offset + size]
        here += 24 + length
    raise AssertionError("no gfx950 code object")


@pytest.fixture(scope="module")
def elf(tmp_path_factory):
    import paper_2508_21230_amd as pkg
    pkg.load_library()  # (builds it if it was never built)
    elf = tmp_path_factory.mktemp("code") / "ejoin.elf"
    elf.write_bytes(code_object(build.LIB))
    return elf


@pytest.fixture(scope="module")
def kernels(elf):
    """Name -> (vector registers in scratch memory, bytes of scratch memory a lane)."""
    notes = subprocess.run([READELF, "--notes", str(elf)], check=True, capture_output=True, text=True).stdout
    of = {}
    for kernel in notes.split("- .agpr_count:")[1:]:
        number = {key: int(value) for key, value in re.findall(r"\.(vgpr_spill_count|private_segment_fixed_size):\s+(\d+)", kernel)}
        of[re.search(r"\.name:\s+(\S+)", kernel)[1]] = (number["vgpr_spill_count"], number["private_segment_fixed_size"])
    return of


def test_no_kernel_spills_vector_registers(kernels):
    """A row operand of k_join_strip that lives in scratch memory is read back at every stage, behind the copies just issued: its wait
    drains the copy pipeline."""
    assert len(kernels) > 30 and sum("k_join_strip" in name for name in kernels) >= 18
    assert {name: spilled for name, spilled in kernels.items() if spilled != (0, 0)} == {}


def test_slots_of_the_one_launch_join_are_stored_before_the_ticket(elf):
    """The last workgroup to take a ticket clears the slots: a slot's store that is still under way then would fill it again, for the
    next call to read.  A barrier does not wait for stores, so the wavefront that fills a slot has to, on every way from there."""
    code = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(elf)], check=True, capture_output=True, text=True).stdout
    seen = 0
    for kernel in re.split(r"^[0-9a-f]{16} ", code, flags=re.M):
        if not re.match(r"<\S*k_join_once", kernel):
            continue
        lines = [line.split("//")[0].strip() for line in kernel.splitlines()]
        wait_loop = next(k for k, line in enumerate(lines) if line.startswith("s_sleep"))
        slot = max(k for k in range(wait_loop) if re.match(r"global_store_dword .*\bsc1\b", lines[k]))
        after = next(line for line in lines[slot + 1:] if re.match(r"s_waitcnt|s_c?branch|s_barrier|s_endpgm", line))
        assert re.match(r"s_waitcnt vmcnt\(0\)", after), after
        seen += 1
    assert seen == 4
