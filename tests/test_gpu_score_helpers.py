"""Scoring with helper workgroups (logits of all fine clusters worked out beside the coarse level): the rule on the CPU; the
ranks and selections bit for bit those of a launch without helpers, at the edges of a helper's share; what a unit's workgroup takes from
them bit for bit what it works out for itself in the same launch, each way shown to have been gone; and steps one after the other, eager
and from a graph."""
import ctypes
import os
import subprocess

import pytest
import torch

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_13059_amd", "csrc", "mp_plan.h")


def test_rule(tmp_path):
    src, so = tmp_path / "h.cpp", tmp_path / "h.so"
    src.write_text(f'#include "{HEADER}"\nextern "C" int helpers(int u, int c, int l, int f) {{ return mp::score_helpers(u, c, l, f); }}\n')
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-o", str(so), str(src)])
    h = ctypes.CDLL(str(so)).helpers
    for cus in (0, 64, 256, 304):
        for u in (1, 2, 3, 7, 8, 24, 32, 63, 64, 85, 86, 127, 128, 129, 256, 1000, 65535):
            assert h(u, cus, 1, 1024) == 0
            fits = False
            for f in (1, 16, 127, 128, 129, 256, 257, 512, 640, 1024, 1563, 2048, 4096, 8192):
                n = h(u, cus, 2, f)
                fits = fits or n > 0
                assert n >= 0 and u * (1 + n) <= max(cus, u)              # one workgroup a compute unit
                if n:
                    assert -(-f // n) <= 256 and u * f <= 40000 and (n - 1) * -(-f // n) < f + 128
            # (the buffers are made by this: a context that can never have helpers has none, any other has them)
            assert fits <= (h(u, cus, 2, 1) > 0)
    assert h(8, 256, 2, 1024) == 8 and h(24, 256, 2, 1563) == 9 and h(64, 256, 2, 320) == 3 and h(32, 256, 2, 2048) == 0


def test_launched_where_they_are_taken_or_warm_the_caches(tmp_path):
    src, so = tmp_path / "p.cpp", tmp_path / "p.so"
    src.write_text(f'#include "{HEADER}"\nextern "C" int pay(int u, int n, int f, int cb) {{ return mp::helpers_pay(u, n, f, cb); }}\n')
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-o", str(so), str(src)])
    pay = ctypes.CDLL(str(so)).pay
    assert pay(9, 41807, 4096, 9000) and not pay(9, 41807, 4096, 12000) and not pay(9, 41807, 4096, 1 << 30)
    assert pay(9, 41807, 2048, 41807) and pay(8, 32768, 4096, 32768) and not pay(24, 40000, 1600, 40000) and pay(24, 40000, 1600, 24000)
    assert pay(4, 16384, 8192, 16384) and not pay(5, 16384, 8192, 16384) and pay(5, 16384, 8192, 2176) and not pay(5, 16384, 8192, 2178)
    assert pay(1, 0, 1, 0)


def _clustered(U, G, nf, nc, seed, softness=0.2, empty=False):
    from paper_2506_13059_amd import inputs
    n = 3 * nf + 40
    centers = inputs.make_modes(U, max(2, nf // 2), "cuda", seed)
    K, V = inputs.draw_tokens(centers, n, seed + 1)
    q = inputs.draw_queries(centers, G, 3, seed + 2, softness=softness)
    g = torch.Generator(device="cuda").manual_seed(seed + 3)
    fot = torch.randint(0, nf, (U, n), generator=g, device="cuda")
    if empty:
        fot = fot // 2 * 2
    cof = torch.sort(torch.randint(0, nc, (U, nf), generator=g, device="cuda"), dim=1).values.to(torch.int32).contiguous()
    return K.view(U, n, 128), V.view(U, n, 128), q.view(3, U, G, 128), fot.to(torch.int32), cof, n


# one and two rounds of a helper, a last share that is short, candidates past the register path (1200 of them), logits that need a
# shift, empty clusters
@pytest.mark.gpu
@pytest.mark.parametrize("nf,nc,G,softness,empty", [(1, 1, 4, 0.2, False), (17, 3, 1, 0.2, False), (128, 9, 4, 0.2, True), (129, 40, 5, 0.2, False),
                                                    (300, 20, 8, 0.2, False), (1025, 64, 4, 0.2, True), (1300, 30, 3, 6.0, False),
                                                    (2000, 90, 8, 0.2, False)])
def test_same_bits_as_without_helpers(nf, nc, G, softness, empty):
    from paper_2506_13059_amd import binding as mp
    U, many = 2, 258                     # (more units than compute units: no helpers)
    K, V, q, fot, cof, n = _clustered(U, G, nf, nc, 50 + nf, softness, empty)
    got = []
    for B in (1, many // U):
        ctx = mp.MpContext(B, U * G, U, max_tokens=n, levels=2, max_fine=nf, max_coarse=nc)
        rep = [x.repeat(B, *[1] * (x.dim() - 1)).contiguous() for x in (K, V, fot, cof)]
        ctx.mp_set_clustering(rep[0].view(B, U, n, 128), rep[1].view(B, U, n, 128), rep[2], nf, rep[3], nc)
        r = []
        for i, (kb, cb) in enumerate([(n // 8, n // 3), (n // 16, n // 8), (n // 3, n - 5), (n, n)]):
            qs = q[i % 3].repeat(B, 1, 1).reshape(B, U * G, 128).contiguous()
            print(f"nf={nf} nc={nc} G={G} B={B} kb={kb} cb={cb}", flush=True)
            out = ctx.mp_decode_attention(qs, kb, cb)
            s = ctx.mp_get_selection()
            c = ctx.mp_get_counters()
            torch.cuda.synchronize()
            r.append(dict(out=out.view(B * U, G, 128)[:U].float(), counters=c[:U], **{k: v[:U] for k, v in s.items()}))
        got.append(r)
        ctx.close()
    for a, b in zip(*got):
        for k in ("fine_selected", "coarse_promising", "counters"):
            assert torch.equal(a[k], b[k]), k
        for k in ("r_fine", "r_coarse"):
            assert torch.equal(torch.nan_to_num(a[k], nan=7.0), torch.nan_to_num(b[k], nan=7.0)), k
        # (the value pass is cut differently: sums of fp32 in another order behind a bf16 output)
        assert (a["out"] - b["out"]).abs().max() <= 2.0 ** -7 * a["out"].abs().max()


# Both ways of a unit's workgroup, each made certain: it never takes its helpers' logits, or it takes those that the helpers of an earlier call
# with the same query left (with another query they give another result, so taken they are).  Both head groups, one and two chunks of candidates,
# logits that need a shift, empty clusters.
@pytest.mark.gpu
@pytest.mark.parametrize("nf,nc,G,softness,empty", [(1, 1, 4, 0.2, False), (17, 3, 1, 0.2, False), (128, 9, 4, 0.2, True), (129, 40, 5, 0.2, False),
                                                    (300, 20, 8, 0.2, False), (1024, 64, 4, 0.2, True), (1000, 30, 8, 6.0, False), (700, 30, 3, 6.0, True)])
def test_handed_over_and_worked_out(nf, nc, G, softness, empty):
    from paper_2506_13059_amd import binding as mp
    U = 8
    K, V, q, fot, cof, n = _clustered(U, G, nf, nc, 90 + nf, softness, empty)
    ctx = mp.MpContext(1, U * G, U, max_tokens=n, levels=2, max_fine=nf, max_coarse=nc)
    ctx.mp_set_clustering(K.view(1, U, n, 128), V.view(1, U, n, 128), fot, nf, cof, nc)
    qs = [x.reshape(1, U * G, 128).contiguous() for x in q]
    count = ctypes.c_int32()
    how_many = lambda how: mp.lib().mp_test_helpers(ctx.h, how, ctypes.byref(count))      # noqa: E731

    def step(how, x, kb, cb):
        print(f"nf={nf} nc={nc} G={G} how={how} kb={kb} cb={cb}", flush=True)
        assert how_many(how) == 0 and count.value == min(31, -(-nf // 128))
        lse = torch.empty(1, U * G, device="cuda")
        out = ctx.mp_decode_attention(x, kb, cb, lse=lse)
        r = [out, lse, ctx.mp_get_counters(), *ctx.mp_get_selection().values()]
        torch.cuda.synchronize()
        return [t.view(torch.int64) if t.dtype == torch.float64 else t for t in r]

    for i, (kb, cb) in enumerate([(n // 8, n // 3), (n // 3, n - 5), (n, n), (n // 8, 0)]):
        x = qs[i % 3]
        planned = step(0, x, kb, cb)
        handed = step(2, x, kb, cb)
        worked_out = step(1, x, kb, cb)
        for a, b, c in zip(planned, handed, worked_out):
            assert torch.equal(a, c) and torch.equal(b, c)
        if kb < n and cb > 0 and nf > 1:
            step(0, qs[(i + 1) % 3], kb, cb)
            assert not torch.equal(step(2, x, kb, cb)[1], worked_out[1])
    assert how_many(3) != 0 and how_many(0) == 0
    ctx.close()


@pytest.mark.gpu
def test_steps_in_a_row_and_from_a_graph():
    from paper_2506_13059_amd import binding as mp
    U, G, nf, nc = 8, 4, 700, 40
    K, V, q, fot, cof, n = _clustered(U, G, nf, nc, 5)
    ctx = mp.MpContext(1, U * G, U, max_tokens=n + 256, levels=2, max_fine=nf + 40, max_coarse=nc + 4)
    ctx.mp_set_clustering(K.view(1, U, n, 128), V.view(1, U, n, 128), fot, nf, cof, nc)
    qs = [x.reshape(1, U * G, 128).contiguous() for x in q]
    out = torch.empty_like(qs[0])

    def eager():
        r = []
        for x in qs:
            ctx.mp_decode_attention(x, n // 8, n // 3, out=out)
            r.append(out.clone())
        return r
    want = eager()
    static = qs[0].clone()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ctx.mp_decode_attention(static, n // 8, n // 3, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.mp_decode_attention(static, n // 8, n // 3, out=out)
    for i in range(12):
        static.copy_(qs[i % 3])
        graph.replay()
        assert torch.equal(out, want[i % 3]), i
        if i % 4 == 3:
            assert all(torch.equal(a, b) for a, b in zip(eager(), want)), i
    ctx.close()
