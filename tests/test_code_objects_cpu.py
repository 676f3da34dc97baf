"""What the kernels' machine code takes for granted, read from the metadata of
the code objects in the built library."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2609_16915_amd import rosetta as R

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
LLVM = "/opt/rocm/llvm/bin"


def _kernels(tmp):
    """(name, static LDS bytes) of every kernel in the library."""
    dump = os.path.join(tmp, "fatbin")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={dump}", R.LIB_PATH,
                    os.path.join(tmp, "copy.so")], check=True)
    with open(dump, "rb") as f:
        data = f.read()
    out, at = [], data.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + 24)
        e = at + 32
        for _ in range(count):
            off, size, idlen = struct.unpack_from("<QQQ", data, e)
            ident = data[e + 24:e + 24 + idlen].decode()
            e += 24 + idlen
            if "amdgcn" in ident and size:
                elf = os.path.join(tmp, "co.elf")
                with open(elf, "wb") as f:
                    f.write(data[at + off:at + off + size])
                notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", elf], check=True,
                                       capture_output=True, text=True).stdout
                # a kernel's keys come in alphabetical order
                out += [(n, int(lds)) for lds, n in re.findall(
                    r"\.group_segment_fixed_size: (\d+).*?\n\s+\.name:\s+(\S+)", notes, re.S)]
        at = data.find(MAGIC, at + 1)
    return out


@pytest.mark.skipif(not shutil.which(f"{LLVM}/llvm-readelf"), reason="needs ROCm's binary tools")
def test_kernels_that_address_lds_by_number_have_no_static_lds(tmp_path):
    """fft_get and fft_put (csrc/fft.hpp) count from the start of the dynamic
    LDS, which is LDS address 0 only while a kernel has no static LDS."""
    kernels = _kernels(str(tmp_path))
    assert any(lds for _, lds in kernels)  # (some other kernel has: the sizes are read)
    for kind in ("k_expand_key", "k_blind_rotate_fft", "k_trace_fft"):
        found = [(n, lds) for n, lds in kernels if kind in n]
        assert found, kind
        assert not [f for f in found if f[1]], found
