"""Registers and scratch of the page kernels, by the metadata of the library that was built: forms whose residency their launch rules and their
comments count on, and which a change elsewhere in a kernel can push over a line of the register file without any other sign."""
import os
import re
import struct
import subprocess

import pytest

from paper_2604_03143_amd import _build, tdk


def code_objects(path):
    """The gfx950 code objects of a library."""
    data, at = open(path, "rb").read(), 0
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        pos = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, name = struct.unpack_from("<QQQ", data, pos)
            if b"gfx950" in data[pos + 24:pos + 24 + name]:
                yield data[at + off:at + off + size]
            pos += 24 + name
        at += 24


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> (registers per lane, bytes of scratch per lane)"""
    if not os.path.exists(tdk.LIB_PATH):
        _build.build(force=True)
    found, llvm = {}, os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
    for code in code_objects(tdk.LIB_PATH):
        path = tmp_path_factory.mktemp("code") / "gfx950.elf"
        path.write_bytes(code)
        notes = subprocess.run([os.path.join(llvm, "llvm-readelf"), "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for entry in notes.split("- .agpr_count:")[1:]:
            name, scratch, regs = (re.search(rf"\.{f}:\s+(\S+)", entry).group(1) for f in ("name", "private_segment_fixed_size", "vgpr_count"))
            found[name] = int(regs), int(scratch)
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True, check=True).stdout.split("\n")
    return {re.sub(r"^void |tdk::|\(.*", "", n): v for n, v in zip(names, found.values())}


def forms(kernels, **of):
    """Kernels of a name with these template arguments (by place; the rest as they come)."""
    for name, args in of.items():
        for k, v in kernels.items():
            m = re.match(rf"tdk_{name}_kernel<(.*)>$", k)
            if m and all(m.group(1).split(", ")[i] == a for i, a in args.items()):
                yield k, v


def waves_per_simd(registers):
    """Of the 512 registers of a SIMD's lane, given out in eights."""
    return 512 // (8 * -(-registers // 8))


def test_long_pages_in_the_masters_order_have_two_wavefronts_per_simd(kernels):
    """32-token pages, one row per access (eight rows per wavefront): all page kernels but the compare kernels that take V, which keep
    both sides of a row."""
    unpacked = {0: "8", 1: "false"}
    some = list(forms(kernels, rerotate={**unpacked, 4: "false"}, keydiff={**unpacked, 3: "false"}, decode={**unpacked, 5: "false"},
                      flag={**unpacked, 3: "1", 4: "false"}))
    assert len(some) == 2 * 2 * 2 + 2 * 2 + 2 * 2 * 3 * 2 + 2 * 2
    assert not {k: v for k, v in some if waves_per_simd(v[0]) < 2}


def test_paired_compare_of_two_accesses_has_three_wavefronts_per_simd(kernels):
    """Several rows per access, two accesses per page and wavefront (four heads with 16-token pages, two with 32), master's order."""
    some = list(forms(kernels, flag={0: "2", 1: "true", 3: "3", 4: "false"}))
    assert len(some) == 4
    assert not {k: v for k, v in some if waves_per_simd(v[0]) < 3}


def test_page_kernels_have_no_scratch(kernels):
    """A reload from scratch waits for every load issued before it, and these kernels count on loads in flight."""
    some = list(forms(kernels, rerotate={}, decode={}, flag={}, keydiff={}))
    assert len(some) > 300
    assert not {k: v for k, v in some if v[1]}


def test_no_form_is_built_that_nothing_launches(kernels):
    """Eight wavefronts per workgroup: the restore takes them for both planes, and nothing with eight loops."""
    eight = {0: "2", 1: "false"}
    assert list(forms(kernels, decode={**eight, 4: "3", 6: "false"})) and list(forms(kernels, rerotate={**eight, 5: "false"}))
    assert not list(forms(kernels, decode={**eight, 4: "1"})) + list(forms(kernels, decode={**eight, 4: "2"}))
    assert not list(forms(kernels, decode={**eight, 6: "true"})) + list(forms(kernels, rerotate={**eight, 5: "true"}))
