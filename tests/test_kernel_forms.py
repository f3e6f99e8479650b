"""What the built library holds, by its symbol table: the forms that flags select and the names that the timing helpers give."""
import os
import re
import subprocess

import pytest

from paper_2604_03143_amd import _build, tdk


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(tdk.LIB_PATH):
        _build.build(force=True)
    out = subprocess.run(["nm", "-C", tdk.LIB_PATH], capture_output=True, text=True, check=True).stdout
    return set(re.findall(r"tdk::(tdk_\w+_kernel(?:<[^>]*>)?)", out))


@pytest.mark.parametrize("form", ["tdk_rerotate_kernel<4, true, false, {}, false, true>", "tdk_decode_kernel<4, true, false, {}, 3, false, true>",
                                  "tdk_flag_kernel<4, true, false, 3, false, {}>", "tdk_keydiff_kernel<4, true, false, false, {}>"])
def test_few_heads_have_both_cache_policies(kernels, form):
    """TDK_TUNE_NT_* choose the policy for models with 1, 2 or 4 KV heads too (several rows per access)."""
    assert form.format("true") in kernels and form.format("false") in kernels


def test_timed_kernels_have_the_names_they_are_given(kernels):
    names = {k.split("<")[0] for k in kernels}
    for kind in range(tdk.KERNEL_KINDS):
        assert tdk.tdk_kernel_name(kind) in names, kind


def test_only_the_direct_loads_use_m0(tmp_path):
    """The loads from memory straight into LDS set M0 in inline assembly, which cannot tell the compiler so (it reserves the
    register): nothing else in the attention kernels may use it, before or behind such a statement."""
    out, src = str(tmp_path / "attend.s"), os.path.join(_build.CSRC, "tdk_attend.hip")
    cmd = [a for a in _build.hipcc_command(out, extra=["--cuda-device-only", "-S"]) if a not in _build.SOURCES and a not in ("-shared", "-fPIC")]
    subprocess.run([*cmd, src], check=True, capture_output=True, timeout=300)
    inside, own, others = False, 0, []
    for line in open(out):
        if "#ASMSTART" in line or "#ASMEND" in line:
            inside = "#ASMSTART" in line
        elif re.search(r"\bm0\b", line.split(";")[0]):
            own += inside
            if not inside:
                others.append(line.strip())
    assert own > 0 and not others, (own, others[:5])
