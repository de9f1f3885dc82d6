"""How the value pass's launch is planned: the header's functions, compiled for the host."""
import ctypes
import os
import subprocess

import pytest

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_13059_amd", "csrc", "mp_plan.h")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "p.cpp", d / "p.so"
    src.write_text(f'''#include "{HEADER}"
extern "C" int chunks(int units) {{ return mp::stream_chunks_per_unit(units); }}
extern "C" int chunk_rows(long long n, int chunks) {{ return mp::stream_chunk_rows(n, chunks); }}
extern "C" void plan(int units, long long first, long long tail, int* out) {{
    const mp::StreamPlan p = mp::plan_streams(units, first, tail);
    out[0] = p.first_rows;
    out[1] = p.tail_rows;
}}
extern "C" int most_selected(int levels, int kb, int cb, int n) {{ return mp::most_selected(levels, kb, cb, n); }}
''')
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-o", str(so), str(src)])
    h = ctypes.CDLL(str(so))
    h.chunk_rows.argtypes = [ctypes.c_longlong, ctypes.c_int]
    h.plan.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_longlong, ctypes.POINTER(ctypes.c_int)]
    return h


def test_keys_selected_are_bounded_by_both_budgets(lib):
    assert lib.most_selected(2, 32768, 4096, 32768) == 4096
    assert lib.most_selected(2, 1024, 4096, 32768) == 1024
    assert lib.most_selected(2, 1024, 0, 32768) == 0
    assert lib.most_selected(1, 1024, 0, 32768) == 1024          # one level: no coarse budget
    assert lib.most_selected(1, 99999, 0, 500) == lib.most_selected(2, 99999, 99999, 500) == 500


def _plan(lib, units, first, tail):
    out = (ctypes.c_int * 2)()
    lib.plan(units, first, tail, out)
    return out[0], out[1]


def test_no_unit_count_leaves_compute_units_idle(lib):
    for units in range(1, 4000):
        wgs = units * lib.chunks(units)
        assert lib.chunks(units) >= 1
        if wgs <= 256:
            assert 3 * wgs >= 2 * 256, units                       # one round: two thirds of the chip at least
        elif wgs <= 512 and units <= 256:
            assert 4 * wgs >= 3 * 512, units                       # two rounds, resident at once
        else:
            # several rounds, up to six: at least three quarters of them
            rounds = -(-wgs // 256)
            assert units > 256 and 4 * wgs >= 3 * 256 * rounds, units
            assert rounds <= 6 or lib.chunks(units) == 1


def test_chunks_cover_the_rows_in_tiles(lib):
    for units in (1, 8, 24, 64, 96, 128, 129, 136, 170, 171, 200, 256, 300, 2000):
        for first in (0, 1, 63, 64, 65, 2048, 4096, 8192, 131072):
            for tail in (0, 1, 130, 255, 8000):
                rows = _plan(lib, units, first, tail)
                counts = [-(-n // r) for n, r in zip((first, tail), rows)]
                assert all(r > 0 and r % 64 == 0 for r in rows)
                assert sum(counts) <= lib.chunks(units) + 1        # (what a context has room for: twice the count and two)
                for n, r, c in zip((first, tail), rows, counts):
                    # even: at most a tile's rounding longer than a share, so that a short chunk occupies all four waves
                    assert c == 0 or r <= -(-n // c) + 63 or r == 64


def test_a_short_tail_takes_no_chunk_from_the_keys(lib):
    for units in (86, 96, 112, 128):
        first, tail = _plan(lib, units, 2048, 130)
        assert -(-2048 // first) == 2 and tail == 192, units
