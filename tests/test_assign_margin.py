"""The margin below which the k-means assignment hands a point to its exact pass, against the error that it has to cover:
the header's functions, compiled for the host, over scores that are as wrong as the model of the matrix cores allows."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_13059_amd", "csrc", "mp_margin.h")
ULP = 2.0 ** -23


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("margin")
    src, so = d / "m.cpp", d / "m.so"
    src.write_text(f'''#include "{HEADER}"
extern "C" float tiled(float m, float) {{ return mp::near_margin(m); }}
extern "C" float resident(float m, float best) {{ return mp::near_margin_of_best(m, best); }}
extern "C" float kept(int near, float best, float margin) {{ return mp::kept_score(near != 0, best, margin); }}
extern "C" int tiled_bits() {{ return mp::kTiledSlotBits; }}
extern "C" int resident_bits() {{ return mp::kResidentSlotBits; }}
''')
    subprocess.check_call(["g++", "-std=c++17", "-shared", "-fPIC", "-o", str(so), str(src)])
    h = ctypes.CDLL(str(so))
    for f in (h.tiled, h.resident):
        f.restype, f.argtypes = ctypes.c_float, [ctypes.c_float, ctypes.c_float]
    h.kept.restype, h.kept.argtypes = ctypes.c_float, [ctypes.c_int, ctypes.c_float, ctypes.c_float]
    return h


def _accumulation_error(M, steps):
    # every partial sum is at most 1.5 M, a step loses at most one unit in its last place; half of |c|^2 (at most M): twelve
    return (steps * 1.5 + 12 * 0.5) * ULP * M


def _slotted(v, bits, slot):
    w = np.asarray(v, np.float32).view(np.uint32)
    return ((w & ~np.uint32((1 << bits) - 1)) | slot.astype(np.uint32)).view(np.float32)


@pytest.mark.parametrize("kernel,steps", [("tiled", 131), ("resident", 128)])
def test_every_winner_that_an_error_can_change_is_near(lib, kernel, steps):
    margin, bits = getattr(lib, kernel), getattr(lib, kernel + "_bits")()
    rng = np.random.default_rng(1)
    n = 20000
    changed = 0
    for M in (1.0, 3.7, 1e-6, 250.0, 1e20):
        E = _accumulation_error(M, steps)
        true_best = M * np.concatenate([rng.uniform(-1.5, 0.5, n), np.full(n, -1.5), np.full(n, 0.5), rng.uniform(-1e-3, 1e-3, n)])
        gap = (2.5 * E + 3 * 2.0 ** bits * ULP * M) * rng.uniform(0, 1, true_best.size) ** 6        # (many close to zero)
        # the nearest centroid's score is as low as the model allows, another one's as high
        low = _slotted(true_best - E, bits, np.where(true_best > 0, 0, (1 << bits) - 1))
        high = _slotted(true_best - gap + E, bits, np.where(true_best - gap + E > 0, (1 << bits) - 1, 0))
        wrong = high > low                                   # the other one wins the comparison
        changed += int(wrong.sum())
        for b, s in zip(high[wrong][::7], low[wrong][::7]):
            # (M as the kernel has it is an fp32 sum: up to a hundred roundings too small)
            assert not b - s > margin(M * (1 - 100 * ULP), float(b)), (M, b, s)
    assert changed > 1000


@pytest.mark.parametrize("kernel,steps", [("tiled", 131), ("resident", 128)])
def test_bound(lib, kernel, steps):
    margin, bits = getattr(lib, kernel), getattr(lib, kernel + "_bits")()
    for M in (1.0, 1e-3, 77.0):
        for best in np.linspace(-1.5 * M, 0.5 * M, 401):
            need = 2 * _accumulation_error(M, steps) + 2 * 2.0 ** bits * ULP * abs(best)
            assert margin(M * (1 - 100 * ULP), best) * (1 - 2.0 ** (bits - 23)) > need, (M, best)


def test_candidates_of_the_exact_pass(lib):
    # scores without index bits: whatever can be the nearest is within the margin of the best
    for M in (1.0, 9.0):
        assert lib.tiled(M * (1 - 100 * ULP), 0.0) > 2 * _accumulation_error(M, 131)


@pytest.mark.parametrize("kernel,steps", [("tiled", 131), ("resident", 128)])
def test_below_the_normal_range(lib, kernel, steps):
    # products and sums may be flushed to zero there, and the index bits are most of what is left of a score
    margin, bits = getattr(lib, kernel), getattr(lib, kernel + "_bits")()
    for M in (0.0, 1e-44, 1e-38, 1e-30):
        lost = 2 * (steps + 12) * 2 * 2.0 ** -126
        assert margin(M, 0.0) > lost + 2 * _accumulation_error(M, steps) + 2.0 ** bits * 2.0 ** -149


# A step left the score of a point's centroid B and that has not changed since.  It was a near tie that centroid A led, which has moved away
# and with it, perhaps, the largest |c|^2.  Now another centroid is nearer than B, by anything: with scores as wrong as the model allows in
# both steps, the kept score is not ahead of that one's by the margin of the present step.
@pytest.mark.parametrize("slotted", [True, False])
@pytest.mark.parametrize("shrinks", [1.0, 1.5, 9.0, 100.0])
def test_score_kept_of_a_near_tie(lib, slotted, shrinks):
    rng = np.random.default_rng(2)
    n = 4000
    bits = lib.resident_bits() if slotted else 0
    own = misled = 0
    for M in (1.0, 3.7, 1e-6, 1e20):
        M1, E, E1 = M * shrinks, _accumulation_error(M, 128), _accumulation_error(M * shrinks, 128)
        # B is the nearest, A (on top) no nearer; both within what the one with the larger error can hide
        true_b = M * np.concatenate([rng.uniform(-1.5, 0.5, n), np.full(n, -1.5), np.full(n, 0.5), rng.uniform(-1e-3, 1e-3, n)])
        true_a = true_b - 2 * E1 * rng.uniform(0, 1, true_b.size) ** 3
        up = lambda v: _slotted(v, bits, np.where(v > 0, (1 << bits) - 1, 0)) if bits else np.float32(v)      # noqa: E731
        down = lambda v: _slotted(v, bits, np.where(v > 0, 0, (1 << bits) - 1)) if bits else np.float32(v)    # noqa: E731
        best = up(true_a + E1)
        second = down(np.minimum(true_b - E1, true_a + E1))
        now = down(true_b + 2 * E * rng.uniform(0, 1, true_b.size) ** 6 - E)           # the nearer one's score, as low as can be
        for b, s2, c in zip(best[::5], second[::5], now[::5]):
            # (the margins of the two kernels that leave scores, and of the one that compares them)
            left = lib.resident(M1 * (1 - 100 * ULP), float(b)) if slotted else lib.tiled(M1 * (1 - 100 * ULP), 0.0) + abs(float(b)) / 65536
            assert not float(b) - float(s2) > left             # (a near tie indeed)
            s = lib.kept(1, float(b), left)
            assert not s - float(c) > lib.resident(M * (1 - 100 * ULP), s), (M, shrinks, b, c)
            misled += float(b) - float(c) > lib.resident(M * (1 - 100 * ULP), float(b))
            own += 1
        # a score that is B's own, from any step: its error goes with B, which is still there
        for v, c in zip(up(true_b + E)[::5], now[::5]):
            s = lib.kept(0, float(v), 0.0)
            assert s == float(v) and not s - float(c) > lib.resident(M * (1 - 100 * ULP), s)
    assert own > 10000 and (misled > 1000 or shrinks < 1.2)      # (the best score itself would have been ahead)
