"""GPU parity of decode steps whose launch plan is not the ordinary one: a coarse budget below the key budget, unit counts
that do not divide the chip's compute units, and tails beside few selected keys."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _ctx(U, G, n, nf, nc, seed, tail=0):
    from paper_2506_13059_amd import binding as mp, inputs
    centers = inputs.make_modes(U, 30, "cuda", seed)
    K, V = inputs.draw_tokens(centers, n + tail, seed + 1)
    K, V = K.view(1, U, n + tail, 128), V.view(1, U, n + tail, 128)
    q = inputs.draw_queries(centers, G, 1, seed + 2, softness=0.2).view(1, U * G, 128)
    g = torch.Generator(device="cuda").manual_seed(seed + 3)
    fot = torch.randint(0, nf, (U, n), generator=g, device="cuda").to(torch.int32)
    cof = torch.sort(torch.randint(0, nc, (U, nf), generator=g, device="cuda"), dim=1).values.to(torch.int32).contiguous() if nc else None
    ctx = mp.MpContext(1, U * G, U, max_tokens=n, levels=2 if nc else 1, max_fine=nf, max_coarse=nc, max_tail=max(tail, 1))
    Kc, Vc = K[:, :, :n].contiguous(), V[:, :, :n].contiguous()
    ctx.mp_set_clustering(Kc, Vc, fot, nf, cof, nc)
    kt, vt = (K[:, :, n:].contiguous(), V[:, :, n:].contiguous()) if tail else (None, None)
    return ctx, Kc, Vc, q, kt, vt


@pytest.mark.parametrize("G", [1, 4, 8])
@pytest.mark.parametrize("kb,cb", [(3000, 300), (2999, 2500), (1500, 0), (100000, 1)])
def test_coarse_budget_below_the_key_budget(G, kb, cb):
    from tests.gpu_util import compare_decode
    for tail in (0, 70):
        ctx, K, V, q, kt, vt = _ctx(2, G, 3000, 200, 20, 40 + G, tail)
        print(f"G={G} kb={kb} cb={cb} tail={tail}", flush=True)
        compare_decode(ctx, q, K, V, kb, cb, kt, vt, label=f"G={G} kb={kb} cb={cb} tail={tail}")
        ctx.close()


@pytest.mark.parametrize("U,G", [(96, 4), (129, 3), (136, 5), (160, 8), (200, 4), (264, 3)])
def test_unit_counts_that_do_not_divide_the_chip(U, G):
    from paper_2506_13059_amd import binding as mp
    from tests.gpu_util import compare_decode
    from tests.test_gpu_stream import _check
    for tail in (0, 130):
        ctx, K, V, q, kt, vt = _ctx(U, G, 1400, 60, 8, 70 + U, tail)
        print(f"U={U} G={G} tail={tail}", flush=True)
        for kb in (500, 0):
            compare_decode(ctx, q, K, V, kb, 700, kt, vt, units=[0, 1, U // 2, U - 2, U - 1], label=f"U={U} G={G} tail={tail} kb={kb}")
        ctx.close()
    lse = torch.empty(q.shape[:2], dtype=torch.float32, device="cuda")
    out = mp.mp_dense_attention(q, K, V, lse=lse)
    torch.cuda.synchronize()
    _check(out, lse, q, K, V, f"dense U={U} G={G}")
