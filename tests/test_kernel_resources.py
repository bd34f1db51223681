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
def kernel_notes(tmp_path_factory):
    """Demangled kernel name -> (bytes of scratch memory, vector registers) per work item."""
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
                        tuple(int(re.search(r"\.%s:\s+(\d+)" % key, kernel).group(1))
                              for key in ("private_segment_fixed_size", "vgpr_count"))
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)
    names = subprocess.run(["c++filt"], input="\n".join(found), stdout=subprocess.PIPE, text=True, check=True).stdout.split("\n")
    return dict(zip((n.replace("mx::(anonymous namespace)::", "") for n in names), found.values()))


@pytest.fixture(scope="module")
def scratch_bytes(kernel_notes):
    return {name: scratch for name, (scratch, _) in kernel_notes.items()}


def waves_per_simd(vgprs):
    """512 registers per lane of a SIMD, handed out eight at a time, to no more than eight waves."""
    return min(8, 512 // ((vgprs + 7) // 8 * 8))


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


def test_waves_of_the_fragment_product_are_those_its_forms_are_chosen_by(kernel_notes):
    """The rules for the 32 x 32 form count on 16 waves per compute unit with blocks of 16, or of 32 with few bits, and on 12 of
    the others (8 with blocks of 64 and 7 or 8 bits on both sides); the sums with a bias keep to them."""
    seen = 0
    for name, (_, vgprs) in kernel_notes.items():
        m = re.search(r"\bgemm_tile_kernel<(\d), (\d), (\d+)>", name)
        if not m:
            continue
        wa, wb, block = (int(v) for v in m.groups())
        least = 4 if block == 16 or (block == 32 and wa + wb <= 8) else 2 if block == 64 and min(wa, wb) >= 7 else 3
        assert waves_per_simd(vgprs) >= least, (name, vgprs)
        seen += 1
    assert seen == 3 * 7 * 7


def test_waves_of_the_decode_kernel_are_those_its_split_is_chosen_by(kernel_notes):
    """The rule counts on 16 waves per compute unit, on 12 with blocks of 32 and 8 bits or of 64 and 2 bits, on 8 with the other
    blocks of 64."""
    seen = 0
    for name, (_, vgprs) in kernel_notes.items():
        m = re.search(r"\blinear_splitk_kernel<(\d), (\d+), \d, \d>", name)
        if not m:
            continue
        width, block = (int(v) for v in m.groups())
        least = (3 if width == 2 else 2) if block == 64 else 3 if (block, width) == (32, 8) else 4
        assert waves_per_simd(vgprs) >= least, (name, vgprs)
        seen += 1
    assert seen == 3 * 7 * 4


def test_attention_with_kept_scores_stays_in_registers(scratch_bytes):
    """Up to eight tiles of scores per wave, 128 registers of the 256."""
    kernels = [n for n in scratch_bytes if re.search(r"\battention_(kept|short)_kernel<", n)]
    assert len(kernels) == 16 + 30 and not [n for n in kernels if scratch_bytes[n]]
