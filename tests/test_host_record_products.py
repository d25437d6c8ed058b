"""The accumulate pass's reader of a record (csrc/bwd_record.hpp: unpack_products) names the same entries and gives the same
rounded products as the plain reader, for every form of record.  Compiled for the host, no GPU."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2201_05989_amd.build import CSRC, INCLUDE, hipcc

HERE = os.path.dirname(os.path.abspath(__file__))
P = ctypes.c_void_p


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("products") / "libproducts.so")
    subprocess.run([hipcc(), "--cuda-host-only", "-O2", "-ffp-contract=off", "-fPIC", "-shared", f"-I{INCLUDE}", f"-I{CSRC}",
                    os.path.join(HERE, "record_products_check.hip"), "-o", out], check=True, capture_output=True)
    so = ctypes.CDLL(out)
    so.products_check.restype = ctypes.c_uint32
    so.products_check.argtypes = [ctypes.c_uint32, ctypes.c_int, ctypes.c_int, ctypes.c_uint32, P, P, P, P, P, ctypes.c_int,
                                  ctypes.c_uint32, ctypes.c_uint32, ctypes.c_int]
    return so


@pytest.mark.parametrize("F", [1, 2, 4, 8])
@pytest.mark.parametrize("half", [0, 1])
@pytest.mark.parametrize("smooth", [0, 1])
@pytest.mark.parametrize("dense", [0, 1])
@pytest.mark.parametrize("E", [-148, -24, 0, 15, 128])  # largest |dL/dy| just below 2^E, down to the smallest float there is
def test_products_and_entries_are_those_of_the_plain_reader(lib, F, half, smooth, dense, E):
    if half and not -24 <= E <= 15:
        pytest.skip("no such half-precision value")
    rng = np.random.default_rng(F + 100 * half + 1000 * smooth + 10000 * dense + E % 97)
    n = 4000
    cmask = 2047 if F == 8 else 4095
    xmask = int(rng.choice([cmask, 255, 0]))
    la = rng.integers(0, cmask if dense else xmask + 1, n).astype(np.uint32)
    la[:3] = [0, cmask - 1 if dense else xmask, 2047 & (cmask - 1 if dense else xmask)]
    c0 = rng.integers(0, 64, n).astype(np.uint32)
    wf0 = (rng.integers(0, 1 << 23, n) * 2.0 ** -23).astype(np.float32)
    wf0[:2] = [0.0, 1 - 2.0 ** -23]
    tiny = c0 == 0  # the first voxel's fraction can be any float
    wf0[tiny] *= (2.0 ** -rng.integers(0, 70, tiny.sum())).astype(np.float32)
    wrow = (rng.random(n) ** rng.integers(1, 40, n)).astype(np.float32)
    wrow[:4] = [0.0, 1.0, 2.0 ** -62, 2.0 ** -63]
    with np.errstate(over="ignore"):
        g = (rng.uniform(-1, 1, (n, F)) * 2.0 ** E * (1 - 2.0 ** -10)).astype(np.float32)
    g[5:9] = np.sign(g[5:9]) * np.float32(2.0 ** (E - 1))
    for H in (11, 24, 35):
        S = min(62 - H, 51) - E
        assert lib.products_check(F, half, smooth, n, *(a.ctypes.data for a in (la, c0, wf0, wrow, np.ascontiguousarray(g))),
                                  dense, cmask, xmask, S) == 0
