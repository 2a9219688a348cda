"""The keys of the assignment search (Eq7), on the CPU: the batch's step takes
no more low bits of a sum than the frame's batches need, a decided pixel's two
smallest sums are at least the required binary32 steps apart, and no pair is
left undecided that lies further apart than the step bits can hide.  The rules
are the kernels' own header, compiled with g++."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_16874_amd", "csrc")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("keys")
    src, so = d / "keys.cpp", d / "keys.so"
    src.write_text('#include "search_keys.hpp"\nextern "C" {\nint step_bits(int n) { return cpe::step_bits(n); }\n'
                   'unsigned key_gap(unsigned g, int b) { return cpe::key_gap(g, b); }\n'
                   'long long fast_search_pixels(int e, int f, int p)\n'
                   '{ return cpe::fast_search_pixels(e, f, p); }\n}\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    lib = ctypes.CDLL(str(so))
    lib.fast_search_pixels.restype = ctypes.c_longlong
    return lib


def _constant(name):
    with open(os.path.join(CSRC, "k_mfma.hpp")) as fh:
        return int(re.search(rf"constexpr int {name} = (\d+);", fh.read()).group(1))


def test_step_bits_are_the_fewest_that_hold_the_steps(rules):
    for nbat in range(8, 2049, 8):
        bits = rules.step_bits(nbat)
        assert 8 << bits >= nbat and (bits == 0 or 8 << (bits - 1) < nbat)
    assert rules.step_bits(128) == _constant("kStepBits")


@pytest.mark.parametrize("nbat", [8, 16, 24, 32, 64, 72, 128, 512, 2048])
def test_gap_of_decided_pixels(rules, nbat):
    gap, bits = _constant("kFastGap"), rules.step_bits(nbat)
    need = rules.key_gap(gap, bits)
    rng = np.random.default_rng(nbat)
    reach = 3 * (1 << bits) + 2 * gap
    s = rng.integers(0x3c000000, 0x44000000, 200000)
    t = s + rng.integers(0, reach + 1, s.size)
    step = lambda v: (v >> bits << bits) | rng.integers(0, nbat // 8, v.size)
    ks, kt = step(s), step(t)
    decided = (np.maximum(ks, kt) >> bits) - (np.minimum(ks, kt) >> bits) >= need
    assert (t - s)[decided].min() >= gap                      # the error bound's requirement
    assert (t - s)[~decided].max() < gap + 3 * (1 << bits)    # what the bits can hide
    assert ((ks < kt)[decided]).all()                         # the winner's key is the smaller sum
    if nbat <= 64:                                            # grids of 32 x 32 rarely have more
        assert decided[t - s >= 16].all()


def test_both_assignment_kernels_take_the_frames_bits():
    for name in ("k_mfma.hpp", "k_assign_big.hpp"):
        with open(os.path.join(CSRC, name)) as fh:
            src = fh.read()
        assert "const int bits = step_bits(nbat);" in src
        calls = re.findall(r"!search_tile<[^;]*?;", src, flags=re.S) + re.findall(r"!search_tile<.*", src)
        assert calls and all("nvalid, bits, force_exact" in c for c in calls)


# element bytes, harmonics, pixels: frames measured at least 1 % slower with the fast search than with the exact one
SLOWER = [(4, 5, 512 * 513), (4, 6, 640 * 640), (4, 7, 512 * 600), (4, 8, 512 * 512), (4, 8, 640 * 640),
          (4, 8, 900 * 900), (4, 9, 1024 * 2048), (4, 12, 1500 * 1500), (4, 16, 1500 * 1500), (2, 6, 512 * 513),
          (2, 8, 512 * 512), (2, 8, 512 * 513), (2, 9, 512 * 512), (2, 10, 640 * 640), (2, 12, 720 * 1024),
          (2, 14, 720 * 1024), (2, 16, 512 * 600), (2, 16, 704 * 704), (2, 16, 720 * 1024)]
# and at least 2 % faster
FASTER = [(4, 2, 704 * 704), (4, 4, 512 * 513), (4, 5, 1100 * 1100), (4, 8, 1500 * 1500), (2, 2, 640 * 640),
          (2, 4, 512 * 512), (2, 7, 512 * 600), (2, 8, 512 * 600), (2, 9, 512 * 600), (2, 10, 1100 * 1100),
          (2, 12, 1100 * 1100), (2, 16, 1024 * 2048)]
# the same for frames without a foreground plane
SLOWER_WITHOUT_PLANE = [(4, 5, 256 * 256), (4, 8, 256 * 256), (4, 9, 1024 * 2048), (2, 6, 256 * 256), (2, 9, 256 * 256),
                        (2, 16, 256 * 256)]
FASTER_WITHOUT_PLANE = [(4, 4, 512 * 513), (4, 5, 640 * 640), (4, 6, 479 * 641), (4, 7, 479 * 641), (2, 5, 512 * 513),
                        (2, 8, 512 * 513), (2, 9, 479 * 641), (2, 10, 512 * 513), (2, 12, 640 * 640),
                        (2, 16, 640 * 640)]


def test_fast_search_follows_the_measurements(rules):
    for elem, F, pixels in SLOWER:
        assert pixels < rules.fast_search_pixels(elem, F, 1), (elem, F, pixels)
    for elem, F, pixels in FASTER:
        assert pixels >= rules.fast_search_pixels(elem, F, 1), (elem, F, pixels)
    for elem, F, pixels in SLOWER_WITHOUT_PLANE:
        assert pixels < rules.fast_search_pixels(elem, F, 0), (elem, F, pixels)
    for elem, F, pixels in FASTER_WITHOUT_PLANE:
        assert pixels >= rules.fast_search_pixels(elem, F, 0), (elem, F, pixels)
