"""Kernels launched in place must not promise the compiler that their input
and output differ: the column pass of the four-step windows runs with
src == dst, and the fused step of one window with in == out."""
import os
import re

import pytest

import paper_1101_0086_amd as P

CSRC = os.path.join(os.path.dirname(P.__file__), "csrc")


@pytest.mark.parametrize("source,kernel,pair", [("window_kernels.hip", "win_cols_kernel", ("src", "dst")),
                                                ("mpa_kernels.hip", "mpa_block_kernel", ("in", "out"))])
def test_in_place_kernels_do_not_restrict(source, kernel, pair):
    with open(os.path.join(CSRC, source)) as f:
        text = f.read()
    params = re.search(kernel + r"\(([^{]*?)\)\s*\{", text).group(1)
    for name in pair:
        decl = next(p for p in params.split(",") if re.search(rf"\b{name}$", p.strip()))
        assert "*" in decl and "__restrict__" not in decl, decl
