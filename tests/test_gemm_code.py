"""The compiled 16-bit GEMMs (the device code in the built library) keep their values in registers."""
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


def test_no_gemm_kernel_spills_registers(tmp_path):
    """A value that comes back from scratch memory waits for every load in flight; in a main loop that is the next stages'."""
    if not os.path.exists(build.LIB):
        pytest.skip("library not built")
    kernels, spilled, name = set(), set(), ""
    for code in device_code(build.LIB):
        (tmp_path / "code").write_bytes(code)
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(tmp_path / "code")], capture_output=True, text=True, check=True).stdout
        for line in listing.splitlines():
            if m := re.match(r"[0-9a-f]+ <(\S+)>:", line):
                name = m[1]
                if "gemm_bf16" in name:
                    kernels.add(name)
            elif line.lstrip().startswith("scratch_") and name in kernels:
                spilled.add(name)
    assert len(kernels) > 20 and not spilled, sorted(spilled)
