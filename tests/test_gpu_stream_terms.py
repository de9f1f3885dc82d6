"""GPU parity of the value pass whose centroid terms have a wave of their own, with and without a tail: short shares of a few terms a
workgroup, workgroups without keys or without terms; and at the edges of the terms' tiles and strips of row numbers, none to 250
terms a workgroup, beside the same steps in the launch they ride along in.  Against the oracle; and the rule that chooses the launch."""
import ctypes
import os
import subprocess

import pytest
import torch

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_13059_amd", "csrc", "mp_plan.h")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("terms")
    src, so = d / "t.cpp", d / "t.so"
    src.write_text(f'''#include "{HEADER}"
extern "C" long long terms(int l, int n, int f, int c, int kb, int cb) {{ return mp::likely_terms(l, n, f, c, kb, cb); }}
extern "C" int own(long long w, long long t, long long k, int r) {{ return mp::terms_have_a_wave(w, t, k, r); }}
// one level, as a decode step's launch is planned: do the terms have a wave, and workgroups of selected keys per unit
extern "C" int step(int U, int n, int nf, int kb, int tail, int* chunks) {{
    const int most = mp::most_selected(1, kb, 0, n);
    const mp::StreamPlan p = mp::plan_streams(U, most, tail);
    *chunks = (most + p.first_rows - 1) / p.first_rows;
    const int of_tail = (tail + p.tail_rows - 1) / p.tail_rows;
    return mp::terms_have_a_wave((long long)U * (*chunks + of_tail), mp::likely_terms(1, n, nf, 0, kb, 0), *chunks, p.first_rows);
}}
''')
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-o", str(so), str(src)])
    h = ctypes.CDLL(str(so))
    h.terms.restype = ctypes.c_longlong
    h.own.argtypes = [ctypes.c_longlong, ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int]
    return h


def test_rule(plan):
    h = plan
    assert h.terms(1, 4096, 64, 0, 256, 0) == 60 and h.terms(1, 4096, 64, 0, 99999, 0) == 0
    assert h.terms(2, 131072, 4096, 256, 8192, 16384) == 256 + 224 and h.terms(2, 1000, 100, 10, 500, 0) == 10
    assert h.own(256, 480, 2, 4096) and not h.own(257, 1, 2, 4096) and h.own(1, 32, 1, 64) and not h.own(1, 33, 1, 64)
    # no more terms a workgroup than a wave has keys, or than one strip of row numbers
    for rows, most in ((128, 64), (256, 64), (512, 128), (1024, 256)):
        assert h.own(256, 2 * most, 2, rows) and not h.own(256, 2 * most + 1, 2, rows), rows


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


# Clusters of four keys, so that budgets of whole clusters leave a known number of terms: `terms` a workgroup of the selected keys.
MANY = [(128, 1024, 2, t) for t in (0, 1, 16, 17, 64, 65, 128)] + [(128, 2048, 2, 250), (100, 2000, 2, 129), (200, 800, 1, 193)]


def _sizes(kb, chunks, terms):
    nf = kb // 4 + chunks * terms
    return nf, 4 * nf


@pytest.mark.parametrize("U,kb,chunks,terms", MANY)
def test_shapes_of_many_terms(plan, U, kb, chunks, terms):
    nf, n = _sizes(kb, chunks, terms)
    c = ctypes.c_int()
    assert plan.terms(1, n, nf, 0, kb, 0) == chunks * terms
    assert plan.step(U, n, nf, kb, 0, ctypes.byref(c)) and c.value == chunks           # a wave of their own
    assert not plan.step(U, n, nf, kb, 1, ctypes.byref(c)) and c.value == chunks       # the tail's workgroups are too many


@pytest.mark.gpu
@pytest.mark.parametrize("G", [1, 4, 5, 6, 8])
@pytest.mark.parametrize("U,kb,chunks,terms", MANY)
def test_many_terms_a_workgroup(U, kb, chunks, terms, G):
    from paper_2506_13059_amd import binding as mp
    from tests.gpu_util import compare_decode
    nf, n = _sizes(kb, chunks, terms)
    g = torch.Generator(device="cuda").manual_seed(nf + G)
    fot = (torch.rand(U, n, generator=g, device="cuda").argsort(1) % nf).to(torch.int32)
    near = torch.gather(torch.randn(U, nf, 128, generator=g, device="cuda"), 1, fot.long()[..., None].expand(U, n, 128))
    K, V = ((near + 0.3 * torch.randn(U, n, 128, generator=g, device="cuda")).to(torch.bfloat16).view(1, U, n, 128) for _ in range(2))
    q = torch.randn(1, U * G, 128, generator=g, device="cuda").to(torch.bfloat16)      # (logits of about 1: the terms count)
    ctx = mp.MpContext(1, U * G, U, max_tokens=n, levels=1, max_fine=nf, max_tail=1)
    ctx.mp_set_clustering(K, V, fot, nf, None, 0)
    for tail in (0, 1):
        print(f"U={U} G={G} nf={nf} kb={kb} tail={tail}", flush=True)
        t = dict(k_tail=K[:, :, :1].contiguous(), v_tail=V[:, :, :1].contiguous()) if tail else {}
        compare_decode(ctx, q, K, V, kb, 0, units=(0, U // 2 + 1, U - 1), label=f"G={G} terms={terms} tail={tail}", **t)
    sel = ctx.mp_get_selection()["fine_selected"]
    assert (sel.bool().sum(1) == kb // 4).all()
    ctx.close()
