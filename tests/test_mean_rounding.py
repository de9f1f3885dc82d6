"""The bf16 rounding of a k-means mean without a division, against the division, around every kind of number half way between two
bf16 values and at the ends of the exponent range: the header's functions, compiled for the host."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from oracle import mp_oracle as O

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_13059_amd", "csrc", "mp_round.h")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("rounding")
    src, so = d / "r.cpp", d / "r.so"
    src.write_text(f'''#include "{HEADER}"
extern "C" void rounded(const double* a, const double* den, long n, unsigned short* out, unsigned short* divided, unsigned short* plain)
{{
    for (long i = 0; i < n; ++i) {{
        out[i] = mp::quotient_to_bf16(a[i], den[i], 1.0 / den[i]);
        divided[i] = mp::f64_to_bf16_rne(a[i] / den[i]);
        plain[i] = mp::f64_to_bf16_rne(a[i] * (1.0 / den[i]));
    }}
}}
''')
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-o", str(so), str(src)])
    h = ctypes.CDLL(str(so))

    def rounded(a, den):
        a, den = np.ascontiguousarray(a, np.float64), np.ascontiguousarray(den, np.float64)
        out = [np.zeros(a.size, np.uint16) for _ in range(3)]
        h.rounded(*(ctypes.c_void_p(x.ctypes.data) for x in (a, den)), ctypes.c_long(a.size), *(ctypes.c_void_p(x.ctypes.data) for x in out))
        return out
    return rounded


def _steps(x, k):
    """x moved by k units of its last place, away from zero for k > 0."""
    return (x.view(np.int64) + k).view(np.float64)


def test_around_half_way(lib):
    rng = np.random.default_rng(1)
    dens = np.concatenate([np.arange(1, 400), rng.integers(400, 131073, 600), [8191, 8192, 131071, 131072]]).astype(np.float64)
    above = below = 0
    for k in range(-24, 25):
        # (mantissas of seven bits and a half, and the one that carries into the next exponent)
        mantissa = np.concatenate([rng.integers(0, 128, 30), [0, 127]])
        half = (1 + (mantissa + 0.5) / 128) * 2.0 ** rng.integers(-60, 60, mantissa.size) * rng.choice([-1, 1], mantissa.size)
        a = _steps((half[:, None] * dens[None, :]).ravel(), k)
        den = np.broadcast_to(dens, (half.size, dens.size)).ravel()
        got, want, plain = lib(a, den)
        np.testing.assert_array_equal(got, want)
        wrong = plain != want                # what the division is there for, on both sides of the number half way
        side = np.abs(a / den) >= np.abs(np.repeat(half, dens.size))
        above += int((wrong & side).sum())
        below += int((wrong & ~side).sum())
        # (and the division's own rounding is the oracle's)
        np.testing.assert_array_equal((want.astype(np.uint32) << 16).view(np.float32).astype(np.float64), O.round_bf16(a / den))
    assert above > 0 and below > 0, (above, below)


def test_product_is_near_the_quotient():
    # what the window of sixteen units stands on
    rng = np.random.default_rng(2)
    for den in np.concatenate([np.arange(1, 300), rng.integers(300, 131073, 300)]).astype(np.float64):
        a = rng.uniform(0.5, 4, 2000)
        assert np.abs((a * (1 / den)).view(np.int64) - (a / den).view(np.int64)).max() <= 3


@pytest.mark.parametrize("exponent", [-140, -128, -127, -126, -125, -124, -123, -122, 120, 121, 122, 123, 126, 127, 128])
def test_ends_of_the_range(lib, exponent):
    rng = np.random.default_rng(3)
    q = np.concatenate([rng.uniform(1, 2, 300), 1 + (np.arange(128) + 0.5) / 128, [1.0, 2 - 2.0 ** -9, 2 - 2.0 ** -52]]) * 2.0 ** exponent
    for k in range(-20, 21):
        for den in (1.0, 3.0, 7.0, 4095.0, 131071.0):
            a = _steps(q * den, k)
            for sign in (1, -1):
                got, want, _ = lib(sign * a, np.full(a.size, den))
                np.testing.assert_array_equal(got, want)


def test_zero_infinity_and_nan(lib):
    got, want, _ = lib(np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 5e-324]), np.array([3.0, 3.0, 3.0, 3.0, 3.0, 3.0]))
    np.testing.assert_array_equal(got, want)
    assert list(got[:4]) == [0, 0x8000, 0x7f80, 0xff80]
