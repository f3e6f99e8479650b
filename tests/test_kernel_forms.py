"""What the built library holds, by its symbol table: the forms that flags select and the names that the timing helpers give."""
import os
import re
import subprocess

import pytest

from paper_2604_03143_amd import tdk


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(tdk.LIB_PATH):
        from paper_2604_03143_amd import _build
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
