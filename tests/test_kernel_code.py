"""The built gfx950 kernels themselves: what the compiler made of them, read from the library's own code objects (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2412_12639_amd import build

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code objects inside the library, one per translation unit."""
    if not os.path.exists(build.LIB) or not shutil.which(f"{LLVM}/llvm-readelf"):
        pytest.skip("library not built, or no LLVM tools")
    data, out, at = open(build.LIB, "rb").read(), [], 0
    where = tmp_path_factory.mktemp("code")
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        u64 = lambda o: int.from_bytes(data[o:o + 8], "little")
        p = at + 32
        for _ in range(min(u64(at + 24), 16)):
            offset, size, n = u64(p), u64(p + 8), u64(p + 16)
            name = data[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" in name and size:
                out.append(where / f"{len(out)}.co")
                out[-1].write_bytes(data[at + offset:at + offset + size])
        at += 24
    assert len(out) == len(build.UNITS)
    return out


def test_kernels_that_are_meant_to_fit_the_registers_use_no_scratch(code_objects):
    scratch = {}
    for co in code_objects:
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(co)], capture_output=True, text=True, check=True).stdout
        for name, size in re.findall(r"\.name:\s+(_Z\S+).*?\.private_segment_fixed_size:\s+(\d+)", notes, re.S):
            scratch[name] = int(size)
    meant = {n: b for n, b in scratch.items() if re.match(r"_Z(11k_gemm_ring|6k_attnI|13k_gemm_paired|13k_gemm_direct|10k_gemm_fix|12k_lstm_chain)", n)}
    assert len(meant) > 60
    assert not {n: b for n, b in meant.items() if b}
