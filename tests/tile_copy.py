"""The kernels' own address arithmetic of the tile copies (csrc/sage_tile_copy.h), compiled for the CPU."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_21136_amd", "csrc")

SOURCE = """
#include "sage_tile_copy.h"
extern "C" {
int k_source(int D, int slot) { return D == 128 ? sage::k_source<128>(slot) : sage::k_source<64>(slot); }
int v_source(int slot) { return sage::v_source(slot); }
int k_off(int D, int row, int c) { return D == 128 ? sage::k_off<128>(row, c) : sage::k_off<64>(row, c); }
int v_off(int row, int c) { return sage::v_off(row, c); }
int copy_left(int bytes, int first) { return sage::copy_left(bytes, first); }
int half_first(int D, int j, int part) { return D == 128 ? sage::half_first<128>(j, part) : sage::half_first<64>(j, part); }
}
"""


class Addresses:
    def __init__(self, lib):
        self._lib = lib
        self.copy_left, self.half_first = lib.copy_left, lib.half_first

    def source(self, is_v, D, slots):
        return np.array([self._lib.v_source(int(s)) if is_v else self._lib.k_source(D, int(s)) for s in slots])

    def place(self, is_v, D, rows, chunks):
        return np.array([self._lib.v_off(int(r), int(c)) if is_v else self._lib.k_off(D, int(r), int(c)) for r, c in zip(rows, chunks)],
                        dtype=np.int64)


@pytest.fixture(scope="session")
def addresses(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile_copy")
    src, lib = str(d / "tile_copy.cpp"), str(d / "tile_copy.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib], check=True)
    return Addresses(ctypes.CDLL(lib))
