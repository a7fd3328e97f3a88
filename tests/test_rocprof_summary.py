"""The summaries under profiles/ cover every kernel of the library."""
import os
import re

import pytest

from paper_2508_00960_amd.build import CSRC
from paper_2508_00960_amd.rocprof_summary import family_of


def kernels():
    names = set()
    for f in os.listdir(CSRC):
        with open(os.path.join(CSRC, f)) as src:
            names |= set(re.findall(r"__global__[^;{]*?\b(\w+_kernel)\(", src.read()))
    return sorted(names)


def test_every_kernel_has_a_family():
    assert len(kernels()) > 10
    for name in kernels():
        suffixes = ("<0, 0, 8>", "<0, 1, 8>", "<1, 1, 8>") if name == "gemm_mfma_kernel" else ("<8>",)
        for args in suffixes:
            assert family_of(f"void phantom::{name}{args}(phantom::Arguments)")[0], name


def test_an_unknown_kernel_of_the_library_is_an_error():
    assert family_of("void at::native::vectorized_elementwise_kernel<4>(int)")[0] is None
    with pytest.raises(SystemExit, match="another_kernel"):
        family_of("void phantom::another_kernel<8>(phantom::Arguments)")
