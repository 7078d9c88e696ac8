"""The compiled 16-bit GEMMs: the device code in the built library."""
import os
import re
import struct
import subprocess

import pytest

from paper_2504_03871_amd import build

OBJDUMP = os.path.join(os.path.dirname(os.path.realpath(build.hipcc())), "..", "llvm", "bin", "llvm-objdump")


def device_code(lib):
    """The gfx950 code objects in the library, one per source file."""
    data = open(lib, "rb").read()
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at, pos = m.start(), m.start() + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, pos)
            if data[pos + 24:pos + 24 + n].endswith(b"gfx950") and size:
                yield data[at + off:at + off + size]
            pos += 24 + n


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """16-bit GEMM kernel -> its instructions."""
    if not os.path.exists(build.LIB):
        pytest.skip("library not built")
    found, name, path = {}, "", tmp_path_factory.mktemp("code") / "code"
    for code in device_code(build.LIB):
        path.write_bytes(code)
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True).stdout
        for line in listing.splitlines():
            if m := re.match(r"[0-9a-f]+ <(\S+)>:", line):
                name = m[1]
            elif "gemm_bf16" in name:
                found.setdefault(name, []).append(line.strip())
    assert len(found) > 20
    return found


def test_no_gemm_kernel_spills_registers(kernels):
    """A value that comes back from scratch memory waits for every load in flight; in a main loop that is the next stages'."""
    spilled = [name for name, ops in kernels.items() if any(op.startswith("scratch_") for op in ops)]
    assert not spilled, spilled


def test_every_row_tile_kernel_has_an_instance_that_streams_weights(kernels):
    """A layer whose weights are to be requested as streaming data (the last template argument) gets them so from all of its
    row-tile GEMMs, at both tile heights and in shared launches too."""
    row_tiles = [name for name in kernels if name.startswith(("_ZN3moe16gemm_bf16_kernel", "_ZN3moe21gemm_bf16_pair_kernel")) and "kernelIDF16_Li2E" not in name and "kernelIDF16bLi2E" not in name]
    for name in row_tiles:
        assert name.replace("ELb0EEEv", "ELb1EEEv") in kernels, name
        streams = any(op.startswith("buffer_load_dwordx4") and re.search(r"\bnt lds\b", op) for op in kernels[name])
        assert streams == ("ELb1EEEv" in name), name
