"""How launches are planned: the header's functions, compiled for the host."""
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
extern "C" int most_chunks(int units) {{ return mp::most_stream_chunks(units); }}
extern "C" void plan(int units, long long first, long long tail, int most, int* out) {{
    const mp::StreamPlan p = mp::plan_streams(units, first, tail, most);
    out[0] = p.first_rows;
    out[1] = p.tail_rows;
}}
extern "C" int short_dense(int group, int units, long long n) {{ return mp::short_dense_on_vector_alu(group, units, n); }}
extern "C" int coarse_level(long long pairs, int pts, int k) {{ return mp::coarse_level_fits(pairs, pts, k); }}
extern "C" int waves(long long pairs) {{ return mp::waves_for_blocks(pairs); }}
extern "C" int most_selected(int levels, int kb, int cb, int n) {{ return mp::most_selected(levels, kb, cb, n); }}
''')
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-o", str(so), str(src)])
    h = ctypes.CDLL(str(so))
    h.coarse_level.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    h.short_dense.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_longlong]
    h.plan.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int, ctypes.POINTER(ctypes.c_int)]
    return h


def test_keys_selected_are_bounded_by_both_budgets(lib):
    assert lib.most_selected(2, 32768, 4096, 32768) == 4096
    assert lib.most_selected(2, 1024, 4096, 32768) == 1024
    assert lib.most_selected(2, 1024, 0, 32768) == 0
    assert lib.most_selected(1, 1024, 0, 32768) == 1024          # one level: no coarse budget
    assert lib.most_selected(1, 99999, 0, 500) == lib.most_selected(2, 99999, 99999, 500) == 500


def _plan(lib, units, first, tail, most=1 << 20):
    out = (ctypes.c_int * 2)()
    lib.plan(units, first, tail, most, out)
    return out[0], out[1]


def _counts(lib, units, first, tail, most=1 << 20):
    return [-(-n // r) for n, r in zip((first, tail), _plan(lib, units, first, tail, most))]


def test_no_unit_count_leaves_compute_units_idle(lib):
    for units in range(1, 4000):
        chunks = _counts(lib, units, 1 << 20, 0)[0]
        wgs = units * chunks
        if wgs <= 256:
            assert 3 * wgs >= 2 * 256, units                       # one round: two thirds of the chip at least
        elif units <= 256:
            assert wgs <= 512 and 4 * wgs >= 3 * 512, units        # two rounds, resident at once
        else:
            # several rounds, up to six: at least three quarters of them
            rounds = -(-wgs // 256)
            assert 4 * wgs >= 3 * 256 * rounds, units
            assert rounds <= 6 or chunks == 1


def test_chunks_cover_the_rows_in_tiles(lib):
    for units in (1, 8, 24, 64, 86, 96, 128, 129, 136, 170, 171, 200, 256, 257, 300, 2000):
        for first in (0, 1, 63, 64, 65, 512, 2048, 4096, 8192, 131072):
            for tail in (0, 1, 130, 255, 1500, 8000):
                for most in (1, 7, 1 << 20):
                    rows = _plan(lib, units, first, tail, most)
                    counts = _counts(lib, units, first, tail, most)
                    assert all(r > 0 and r % 64 == 0 for r in rows)
                    assert sum(counts) <= lib.most_chunks(units) + 1        # (what a context has room for)
                    assert max(counts) <= most
                    for n, r, c in zip((first, tail), rows, counts):
                        # even: at most a tile's rounding longer than a share, so that a short chunk occupies all four waves
                        assert c == 0 or r <= -(-n // c) + 63 or r == 64


def test_a_short_tail_takes_no_chunk_from_the_keys(lib):
    for units in (86, 96, 112, 128):
        first, tail = _plan(lib, units, 2048, 130)
        assert -(-2048 // first) == 2 and tail == 192, units


def test_a_long_tail_does_not_spill_into_a_second_round(lib):
    for units in range(1, 129):        # (beyond, each stream's one chunk is a round of its own)
        for first, tail in ((512, 1500), (1024, 1024), (4096, 3000), (100, 8000)):
            a, b = _counts(lib, units, first, tail)
            rows = _plan(lib, units, first, tail)
            long_ones = units * sum(c for c, r in zip((a, b), rows) if 2 * r > max(rows) + 126)
            # the long chunks fit one round, or fill more than half of the second
            assert long_ones <= 256 or long_ones > 340, (units, first, tail, a, b)


def test_dense_calls_on_the_vector_alu(lib):
    assert lib.short_dense(1, 1, 8192) and lib.short_dense(1, 128, 500) and lib.short_dense(1, 64, 2048)
    assert not lib.short_dense(1, 64, 2049) and not lib.short_dense(1, 128, 1 << 40)
    assert not any(lib.short_dense(g, u, n) for g in (2, 3) for u, n in ((1, 100), (8, 64), (64, 2000), (300, 400)))


def test_waves_of_an_assignments_workgroups(lib):
    narrow = [p for p in range(1, 400) if lib.waves(ctypes.c_longlong(p)) == 8]
    assert narrow == [*range(86, 103), *range(129, 171), *range(257, 400)] and lib.waves(ctypes.c_longlong(1)) == 16
    for p in range(1, 257):         # whole workgroups, of sixteen on 256 places or of eight on 512: at least three quarters of the others' waves
        assert p in narrow or 4 * 16 * (256 // p) >= 3 * 8 * (512 // p), p


def test_coarse_level_in_one_launch_only_where_it_is_the_faster_way(lib):
    # (pairs, points, clusters): measured on both sides of every line
    for case in ((1, 512, 32), (64, 256, 48), (64, 160, 64), (1, 64, 64), (64, 256, 64), (256, 256, 96), (1024, 512, 48), (1, 1, 1)):
        assert lib.coarse_level(*case), case
    for case in ((1, 256, 64), (1, 512, 64), (1, 256, 256), (64, 160, 96), (64, 512, 64), (1024, 512, 64), (256, 512, 128), (1, 513, 16),
                 (64, 256, 96), (1, 0, 0)):
        assert not lib.coarse_level(*case), case
    # the kernel's arrays are made for this many
    assert max(k for k in range(1, 513) for pts in (k, 256, 512) if pts >= k and lib.coarse_level(1 << 20, pts, k)) == 101
