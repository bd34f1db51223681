"""Registers of the built kernels, read from the notes of the library's own code objects (no GPU needed): a kernel whose
working set does not fit its registers keeps part of it in memory, which costs far more than a shallower ring."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2307_15517_amd import mx

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def scratch_bytes(tmp_path_factory):
    """Demangled kernel name -> bytes of scratch memory per work item."""
    if not os.path.exists(READELF) or shutil.which("c++filt") is None:
        pytest.skip("no llvm-readelf")
    if not os.path.exists(mx.LIB_PATH):
        from paper_2307_15517_amd import build
        build.build(verbose=False)
    data = open(mx.LIB_PATH, "rb").read()
    path = str(tmp_path_factory.mktemp("co") / "object.co")
    found = {}
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            target = data[entry + 24:entry + 24 + length].decode()
            entry += 24 + length
            if "gfx950" in target and size:
                with open(path, "wb") as f:
                    f.write(data[at + offset:at + offset + size])
                notes = subprocess.run([READELF, "--notes", path], stdout=subprocess.PIPE, text=True, check=True).stdout
                for kernel in notes.split(".agpr_count:")[1:]:
                    found[re.search(r"\.name:\s+(\S+)", kernel).group(1)] = \
                        int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", kernel).group(1))
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)
    names = subprocess.run(["c++filt"], input="\n".join(found), stdout=subprocess.PIPE, text=True, check=True).stdout.split("\n")
    return dict(zip((n.replace("mx::(anonymous namespace)::", "") for n in names), found.values()))


@pytest.mark.parametrize("width", [5, 6, 7, 8])
def test_ring_of_wide_records_stays_in_registers(scratch_bytes, width):
    """One-row decode in blocks of 64, sixteen waves: 20 to 32 dwords of weights per lane and chunk."""
    kernels = [n for n in scratch_bytes if re.search(r"\bgemv_dot_kernel<%d, 64, 1, 16, \d>" % width, n)]
    assert len(kernels) == 1 and scratch_bytes[kernels[0]] == 0


def test_product_and_attention_kernels_stay_in_registers(scratch_bytes):
    kernels = [n for n in scratch_bytes
               if re.search(r"\b(gemm_tile|gemm_fragment|gemm_bf16|gemm_bf16_split|gemm_scaled|gemm_scaled_split|"
                            r"attention_bf16|attention_split|linear_splitk)_kernel<", n)]
    assert len(kernels) > 300
    assert not [(n, scratch_bytes[n]) for n in kernels if scratch_bytes[n]]
