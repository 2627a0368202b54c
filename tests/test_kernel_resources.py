"""Wavefronts and workgroups that a CU holds, from the registers and LDS the compiler gave each kernel
of the built library (its code objects' own metadata), against the numbers that the launch plans and
the kernels' layouts count on.  CPU only."""
import os
import re
import struct
import subprocess

import pytest

from paper_1810_08137_amd import ugks

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
CXXFILT = "c++filt"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
LDS = 160 * 1024     # of a CU
VGPRS = 512          # of a SIMD's lane, handed out in eights


def _code_objects(blob):
    """The gfx950 ELF images of the offload bundles in the library: magic, entry count, then offset,
    size and target of each entry."""
    at = blob.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, p)
            target = blob[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in target:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 24)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> (VGPRs of a lane, bytes of LDS, threads of a workgroup)"""
    if not os.path.exists(READELF):
        pytest.skip("ROCm toolchain missing")
    with open(ugks.LIB_PATH, "rb") as fh:
        blob = fh.read()
    out = {}
    for k, image in enumerate(_code_objects(blob)):
        path = str(tmp_path_factory.mktemp("co") / f"{k}.elf")
        with open(path, "wb") as fh:
            fh.write(image)
        text = subprocess.run([READELF, "--notes", path], capture_output=True, text=True,
                              check=True).stdout
        for part in re.split(r"\n\s+- \.a", text)[1:]:
            def field(name):
                m = re.search(r"\." + name + r":\s+(\S+)", part)
                return m.group(1) if m else None
            if field("vgpr_count") is None:
                continue
            name = subprocess.run([CXXFILT, field("name")], capture_output=True,
                                  text=True).stdout.strip()
            name = re.sub(r"\(.*", "", name.replace("(anonymous namespace)::", ""))
            name = name.replace("void ", "").replace("ugks::", "")
            out[name] = (int(field("vgpr_count")), int(field("group_segment_fixed_size")),
                         int(field("max_flat_workgroup_size")))
    return out


def _waves(vgprs):
    """Wavefronts of a SIMD that its registers hold."""
    return min(8, VGPRS // (-(-vgprs // 8) * 8))


@pytest.mark.parametrize("kernel,waves", [
    ("sums_kernel<double, true>", 3),
    ("sums_kernel<float, true>", 3),
    ("sums_kernel<double, false>", 4),
    ("sums_kernel<float, false>", 3),
])
def test_moment_kernel_wavefronts(kernels, kernel, waves):
    assert _waves(kernels[kernel][0]) >= waves, kernels[kernel]


@pytest.mark.parametrize("kernel,workgroups", [
    ("update_kernel<double, 1>", 2),
    ("update_kernel_nodes<double, 1>", 2),
    ("update_kernel_shakhov<double, 1>", 2),
    ("update_kernel<double, 2>", 1),
    ("update_kernel_nodes<double, 2>", 1),
    ("update_kernel_shakhov<double, 2>", 1),
    ("update_kernel<float, 1>", 4),
    ("update_kernel_nodes<float, 1>", 4),
    ("update_kernel_shakhov<float, 1>", 2),
])
def test_update_kernel_workgroups(kernels, kernel, workgroups):
    """By registers and by LDS: the plan's workgroups that run at once on a CU."""
    vgprs, lds, threads = kernels[kernel]
    assert _waves(vgprs) * 4 * 64 // threads >= workgroups, (vgprs, threads)
    assert LDS // lds >= workgroups, lds
