"""The grouped products' kernels keep everything in registers: none of them spills vector registers or uses scratch memory (what a wavefront spills
goes through memory: 24 registers of 256 workgroups are 12.6 MB a launch).  Read from the built library's own code objects."""
import os
import re
import subprocess

import pytest

from paper_2103_13262_amd.build import HIPCC, LIB

LLVM = os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "llvm", "bin")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def kernels(tmp_path):
    """Name and resource figures of every kernel in the library."""
    tool = lambda name, *args: subprocess.run([os.path.join(LLVM, name), *args], check=True, capture_output=True, text=True).stdout
    section = tmp_path / "fatbin"
    tool("llvm-objcopy", "--dump-section", f".hip_fatbin={section}", LIB, str(tmp_path / "copy.so"))
    for i, part in enumerate(section.read_bytes().split(MAGIC)[1:]):
        bundle, code = tmp_path / f"{i}.bundle", tmp_path / f"{i}.co"
        bundle.write_bytes(MAGIC + part)
        tool("clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={bundle}", f"--output={code}")
        for text in tool("llvm-readelf", "--notes", str(code)).split(".agpr_count:")[1:]:
            field = lambda name: re.search(rf"\.{name}:\s+(\S+)", text)[1]
            yield field("name"), int(field("vgpr_spill_count")), int(field("private_segment_fixed_size"))


def test_grouped_products(tmp_path):
    if not os.path.exists(os.path.join(LLVM, "llvm-readelf")):
        pytest.skip("no LLVM tools beside the compiler")
    products = [k for k in kernels(tmp_path) if "ggemm" in k[0]]
    kinds = [sum(f"ggemm_{kind}" in k[0] for k in products) for kind in ("sk_kernel", "cls_kernel", "pair_kernel", "tile_kernel", "f32")]
    assert all(kinds), kinds
    assert [k for k in products if k[1] or k[2]] == []
