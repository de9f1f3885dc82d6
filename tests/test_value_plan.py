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
extern "C" int most_selected(int levels, int kb, int cb, int n) {{ return mp::most_selected(levels, kb, cb, n); }}
''')
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-o", str(so), str(src)])
    return ctypes.CDLL(str(so))


def test_keys_selected_are_bounded_by_both_budgets(lib):
    assert lib.most_selected(2, 32768, 4096, 32768) == 4096
    assert lib.most_selected(2, 1024, 4096, 32768) == 1024
    assert lib.most_selected(2, 1024, 0, 32768) == 0
    assert lib.most_selected(1, 1024, 0, 32768) == 1024          # one level: no coarse budget
    assert lib.most_selected(1, 99999, 0, 500) == lib.most_selected(2, 99999, 99999, 500) == 500
