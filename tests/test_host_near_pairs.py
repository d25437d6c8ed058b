"""Records of pairs whose upper corner does not follow from the lower one (table sizes that are no power of two, one dimension),
made and read back on the host (tests/near_check.hip): every corner's entry receives its weight and no other entry anything."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2201_05989_amd import binding, synth
from paper_2201_05989_amd.build import CSRC, INCLUDE, LIB_PATH, hipcc

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def near_check(tmp_path_factory):
    binding.load_library()
    out = str(tmp_path_factory.mktemp("near") / "libnear_check.so")
    lib_dir = os.path.dirname(LIB_PATH)
    subprocess.run([hipcc(), "--cuda-host-only", "-O2", "-ffp-contract=off", "-fPIC", "-shared", f"-I{INCLUDE}", f"-I{CSRC}",
                    os.path.join(HERE, "near_check.hip"), "-o", out, f"-L{lib_dir}", "-lhashgrid", f"-Wl,-rpath,{lib_dir}"],
                   check=True, capture_output=True)
    lib = ctypes.CDLL(out)
    lib.near_check.argtypes = [ctypes.POINTER(binding.hashgrid_config), ctypes.c_uint32, ctypes.c_void_p, ctypes.c_void_p]

    def run(d, L, F, T, N_min, N_max, interp, x):
        cfg = binding.hashgrid_config(d, L, F, T, N_min, N_max, binding.HG_F32, binding.HG_F32, interp, binding.HG_F32)
        x = np.ascontiguousarray(x, dtype=np.float32)
        out3 = (ctypes.c_uint64 * 3)()
        assert lib.near_check(ctypes.byref(cfg), len(x), x.ctypes.data, out3) == 0
        return list(out3)

    return run


def points(rng, d, N_max):
    x = synth.points_uniform(rng, 3000, d)
    x[:50] = 0.0
    x[50:100] = 1 - 2.0 ** -24
    x[100:400] = (rng.integers(0, N_max, (300, d)) / N_max).astype(np.float32)  # vertices: the fraction is 0 or next to it
    x[400:700, 0] = np.float32(rng.random(300) / (4 * N_max))  # first voxel: a fraction finer than the record's unit
    k = 1 << rng.integers(1, 13, 300)  # coordinates that end in many one bits: far steps
    x[700:1000, 0] = ((rng.integers(0, 8, 300) * k + k - 0.5 - rng.random(300) / 3) / N_max).astype(np.float32)
    return np.clip(x, 0, np.float32(1 - 2.0 ** -24))


@pytest.mark.parametrize("interp", [0, 1])
@pytest.mark.parametrize("d,L,F,T,N_min,N_max", [
    (3, 16, 2, 1000003, 16, 2048), (3, 8, 8, 524287, 16, 512), (2, 12, 1, 3 << 18, 4, 32768), (2, 4, 2, 4097, 7, 5000),
    (2, 3, 4, 3, 2, 300), (3, 5, 2, 6, 2, 40), (1, 10, 2, 1 << 16, 16, 1 << 20), (1, 6, 8, 5000, 3, 1 << 18)])
def test_every_corner_gets_its_weight(near_check, d, L, F, T, N_min, N_max, interp):
    bad, pairs, split = near_check(d, L, F, T, N_min, N_max, interp, points(np.random.default_rng(T + d), d, N_max))
    assert bad == 0 and pairs == 3000 * L << (d - 1) and split > 0


def test_nearly_every_pair_of_a_hashed_level_is_one_record(near_check):
    x = synth.points_uniform(np.random.default_rng(1), 4000, 3)
    bad, pairs, split = near_check(3, 8, 2, 1000003, 256, 2048, 0, x)
    # far steps 2^-8 of the pairs, two chunks and the first voxel less than that
    assert bad == 0 and split < 0.01 * pairs


@pytest.mark.parametrize("d,T", [(3, 100003), (2, 1000003), (1, 1 << 16)])
@pytest.mark.parametrize("interp", [0, 1])
def test_points_on_vertices_take_one_record_a_pair(near_check, d, T, interp):
    """Fractions of zero (linear) or a half (smoothstep) on a level of 256 vertices a side.  Two records: chunks' ends, wraps, and the
    last 8 trailing one bits or so."""
    x = (np.random.default_rng(d).integers(0, 256, (4000, d)) / 256).astype(np.float32)
    bad, pairs, split = near_check(d, 1, 2, T, 256, 256, interp, x)
    assert bad == 0 and split < 0.02 * pairs
