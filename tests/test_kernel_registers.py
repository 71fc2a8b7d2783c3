"""What the compiler reports about the built kernels (their metadata in the library's gfx950 code objects): kernels on the
decode path keep their registers.  CPU only."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2506_17255_amd import build as skl_build

LLVM = "/opt/rocm/llvm/bin"


def scratch_per_kernel(lib, tmp_path):
    """{kernel name: bytes of scratch per lane} of every gfx950 code object bundled into the library."""
    fat = tmp_path / "fatbin"
    subprocess.check_call([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", lib, str(tmp_path / "rest.so")])
    data = fat.read_bytes()
    found = {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        n, = struct.unpack_from("<Q", data, m.start() + 24)
        at = m.start() + 32
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" not in triple or not size:
                continue
            obj = tmp_path / "object.elf"
            obj.write_bytes(data[m.start() + offset:m.start() + offset + size])
            notes = subprocess.check_output([f"{LLVM}/llvm-readelf", "--notes", str(obj)], text=True)
            for entry in re.split(r"\n  - (?=\.)", notes):
                name, scratch = re.search(r"\.name:\s+(_Z\S+)", entry), re.search(r"\.private_segment_fixed_size:\s+(\d+)", entry)
                if name and scratch:
                    found[name.group(1)] = int(scratch.group(1))
    return found


def test_decode_kernels_keep_their_registers(tmp_path):
    """No scratch in the decode kernels of up to seven sketch rows in either query mode, nor in the kernels of one-pass prompts; the
    batched kernel of eight rows and the prompt kernel of eight rows, 64 tokens and signed values have none left to give."""
    if not os.path.exists(skl_build.LIB) or not shutil.which(f"{LLVM}/llvm-readelf"):
        pytest.skip("needs the built library and the compiler's tools")
    scratch = {k: v for k, v in scratch_per_kernel(skl_build.LIB, tmp_path).items() if re.search(r"k_row_gemv|k_prompt_gemm", k)}
    assert len([k for k in scratch if "k_row_gemvN" in k]) >= 2 * 2 * 2 * 8 and any("k_prompt_gemm" in k for k in scratch)
    spilled = {k: v for k, v in scratch.items() if v}
    allowed = {k for k in spilled if re.search(r"k_row_gemvNILi8E", k) and spilled[k] <= 28 or re.search(r"skl_qm113k_prompt_gemmILi8ELi4E", k)}
    assert not set(spilled) - allowed, spilled
