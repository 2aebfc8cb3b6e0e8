"""X is read up to column 8 ceil(N / 8) - 1 of every row and no further (include/hinm.h): the last row may end there while the
leading dimension is wider, as in the last columns of a wider matrix."""
import ctypes
import glob
import os
import re
import subprocess

import numpy as np
import pytest

import hinm_synth as synth
from oracle import hinm_oracle as orc
from paper_2407_20496_amd import build

HOST = r"""
#include "column_pieces.h"
extern "C" int half_end(int n0, int half, int N) { return n0 + hinm::half_offset(n0, half, N) + 8; }
extern "C" int piece_end(int first, int N) { return hinm::piece_inside(first, N) ? first + 8 : 0; }
"""


@pytest.fixture(scope="module")
def pieces(tmp_path_factory):
    d = tmp_path_factory.mktemp("pieces")
    (d / "pieces.cpp").write_text(HOST)
    out = str(d / "pieces.so")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-fPIC", "-shared", "-I", build.CSRC,
                    str(d / "pieces.cpp"), "-o", out], check=True)
    return ctypes.CDLL(out)


def test_highest_column_a_block_forms(pieces):
    """The kernels with 16-column blocks form every piece with these two functions of (block, N): nothing past the
    promised extent, and every one of the N columns is covered."""
    for N in range(2, 131):
        extent = (N + 7) // 8 * 8
        for n0 in range(0, N, 16):
            ends = [pieces.half_end(n0, half, N) for half in (0, 1)]
            assert max(ends) <= extent and max(ends) >= min(n0 + 16, N)
        for n0 in range(0, N, 64):          # up to four blocks per workgroup, whole ones beyond N among them
            ends = [pieces.piece_end(n0 + 16 * cb + 8 * half, N) for cb in range(4) for half in (0, 1)]
            assert max(ends) <= extent and max(ends) >= min(n0 + 64, N)


def test_leading_dimensions_stay_64_bit():
    for path in glob.glob(os.path.join(build.CSRC, "*.hip")) + glob.glob(os.path.join(build.CSRC, "*.h")):
        with open(path) as f:
            assert not re.search(r"\(int(32_t)?\)\s*\(?(a\.|c\.)?ld[xy]\b", f.read()), path


@pytest.mark.gpu
@pytest.mark.parametrize("N", [5, 20])
@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("Kv", [64, 72])
def test_last_columns_of_a_wider_matrix(N, prepared, Kv):
    """X ends where the promise ends; its neighbours hold NaN."""
    from tests import gpu_util as gu
    M, K, V, ld, at = 64, 96, 64 if prepared else 16, 128, 128 - (N + 7) // 8 * 8
    case = synth.small_case(M, K, V, Kv, N, "f16", 61)
    vals, nm, vec = orc.pack(case.weights(), "f16", V, Kv)
    Xb = case.activations(N)
    want = orc.product(orc.unpack_fast(vals, nm, vec, M, K, V), Xb, "f16", case.pi_in(), case.pi_out()).astype(np.float64)
    wide = np.full((K, ld), 0x7E00, dtype=np.uint16)
    wide[:, at:at + N] = Xb
    X = gu.dev_bits(wide)[:, at:]
    p = gu.upload_packed(M, K, V, Kv, "f16", vals, nm, vec)
    if prepared:
        pr = gu.gpu_prepare(p, case.pi_in(), case.pi_out())
        for variant in (0, 11):             # by shape, and the 16-row kernel for any column count
            got = gu.gpu_spmm_prepared(pr, Xb, 2, variant, ldx=ld, X_dev=X)
            gu.check_close(got.astype(np.float64), want, what="variant %d" % variant)
    else:
        got = gu.gpu_spmm(p, Xb, case.pi_in(), case.pi_out(), 2, ldx=ld, X_dev=X)
        gu.check_close(got.astype(np.float64), want, what="16-row tiles")
