"""GPU parity of the value pass whose centroid terms have a wave of their own, at the edges of its tiles, shares and strips (none, one,
sixteen, 64 terms a workgroup and more, workgroups without keys or without terms), with and without a tail, and of the rule that
chooses it; against the oracle, and against the launch they ride along in (a tail off 16 bytes goes another way altogether)."""
import ctypes
import os
import subprocess

import pytest
import torch

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_13059_amd", "csrc", "mp_plan.h")


def test_rule(tmp_path):
    src, so = tmp_path / "t.cpp", tmp_path / "t.so"
    src.write_text(f'''#include "{HEADER}"
extern "C" long long terms(int l, int n, int f, int c, int kb, int cb) {{ return mp::likely_terms(l, n, f, c, kb, cb); }}
extern "C" int own(long long w, long long t, long long k, int r) {{ return mp::terms_have_a_wave(w, t, k, r); }}
''')
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-o", str(so), str(src)])
    h = ctypes.CDLL(str(so))
    h.terms.restype = ctypes.c_longlong
    h.own.argtypes = [ctypes.c_longlong, ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int]
    assert h.terms(1, 4096, 64, 0, 256, 0) == 60 and h.terms(1, 4096, 64, 0, 99999, 0) == 0
    assert h.terms(2, 131072, 4096, 256, 8192, 16384) == 256 + 224 and h.terms(2, 1000, 100, 10, 500, 0) == 10
    assert h.own(256, 480, 2, 4096) and not h.own(257, 1, 2, 4096) and h.own(1, 32, 1, 64) and not h.own(1, 33, 1, 64)


def _case(U, G, nf, nc, n, seed):
    from paper_2506_13059_amd import binding as mp, inputs
    centers = inputs.make_modes(U, max(2, nf // 2), "cuda", seed)
    K, V = inputs.draw_tokens(centers, n, seed + 1)
    Kt, Vt = inputs.draw_tokens(centers, 150, seed + 5)
    q = inputs.draw_queries(centers, G, 1, seed + 2, softness=0.2).view(1, U * G, 128)
    g = torch.Generator(device="cuda").manual_seed(seed + 3)
    fot = torch.randint(0, nf, (U, n), generator=g, device="cuda").to(torch.int32)
    cof = torch.sort(torch.randint(0, nc, (U, nf), generator=g, device="cuda"), dim=1).values.to(torch.int32).contiguous() if nc else None
    ctx = mp.MpContext(1, U * G, U, max_tokens=n, levels=2 if nc else 1, max_fine=nf, max_coarse=nc, max_tail=150)
    ctx.mp_set_clustering(K.view(1, U, n, 128), V.view(1, U, n, 128), fot, nf, cof, nc)
    return ctx, K.view(1, U, n, 128), V.view(1, U, n, 128), Kt.view(1, U, 150, 128), Vt.view(1, U, 150, 128), q


@pytest.mark.gpu
@pytest.mark.parametrize("G", [1, 4, 5, 6, 8])
@pytest.mark.parametrize("U,nf,nc,n,kb,cb", [(1, 40, 0, 900, 400, 0), (1, 300, 0, 9000, 4000, 0), (2, 17, 0, 700, 650, 0), (2, 16, 0, 700, 699, 0),
                                             (3, 70, 9, 2100, 500, 1500), (1, 3000, 0, 30000, 12000, 0), (64, 66, 5, 1600, 700, 1100), (2, 60, 8, 1500, 3, 900)])
def test_terms_beside_the_keys(U, nf, nc, n, kb, cb, G):
    from tests.gpu_util import compare_decode
    ctx, K, V, Kt, Vt, q = _case(U, G, nf, nc, n, 20 + nf + G)
    for tail in (0, 1, 150):
        print(f"U={U} G={G} nf={nf} kb={kb} tail={tail}", flush=True)
        t = dict(k_tail=Kt[:, :, :tail].contiguous(), v_tail=Vt[:, :, :tail].contiguous()) if tail else {}
        compare_decode(ctx, q, K, V, kb, cb, label=f"G={G} nf={nf} tail={tail}", **t)
    ctx.close()
