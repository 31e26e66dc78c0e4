"""Tiles and slices by the host's reciprocals: csrc/tile_order.h itself, which the kernels include, built with the host compiler and
compared with plain division up to the 2^31 - 1 workgroups of a launch."""
import os
import shutil

import pytest

from tests.test_sanitizers import ROOT, SAN, _build_and_run


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_tiles_and_slices_as_by_division(tmp_path):
    exe = str(tmp_path / "tile_order")
    out = _build_and_run(["g++", "-std=c++17", "-Wall", "-Wextra"] + SAN + [os.path.join(ROOT, "tests", "sanitize", "tile_order_main.cpp"), "-o", exe],
                         exe, [], tmp_path)
    assert "tile order clean" in out
