"""GPU test of the batched copies behind the getters and the local buffer: the same bytes whatever the addresses are multiples
of (sixteen bytes, four or one at a time), rows and tails of any length, and nothing beside them written."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu


def _context(U, n, f, tail):
    from paper_2506_13059_amd import binding as mp
    g = torch.Generator(device="cuda").manual_seed(n)
    K, V = (torch.randn(U, 1, n, 128, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    ids = (torch.arange(n, device="cuda") * 5 % f).int().expand(U, -1).contiguous()
    ctx = mp.MpContext(U, 2, 1, max_tokens=n + 50, levels=1, max_fine=f + 3, max_tail=tail)
    ctx.mp_set_clustering(K, V, ids, f)
    return ctx, K, V


@pytest.mark.parametrize("offset", [0, 4, 2, 1])
@pytest.mark.parametrize("U,n", [(1, 7), (3, 1001), (2, 5000)])
def test_getters(U, n, offset):
    from paper_2506_13059_amd import binding as mp
    print(f"U={U} n={n} offset={offset}", flush=True)
    f = min(n, 13)
    ctx, _, _ = _context(U, n, f, 1)
    want = ctx.mp_get_layout()
    bytes_of = [x.numel() * x.element_size() for x in want]
    got = [torch.full((b + 48,), 0xa5, dtype=torch.uint8, device="cuda") for b in bytes_of]
    st = mp.lib().mp_get_layout(ctx.h, *(C.c_void_p(x.data_ptr() + 16 + offset) for x in got), C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    torch.cuda.synchronize()
    for w, x, b in zip(want, got, bytes_of):
        assert torch.equal(x[16 + offset:16 + offset + b], w.view(-1).view(torch.uint8))
        assert bool((x[:16 + offset] == 0xa5).all()) and bool((x[16 + offset + b:] == 0xa5).all())
    ctx.close()


@pytest.mark.parametrize("offset", [4, 2, 1])
def test_local_buffer(offset):
    # (the library's boundary takes addresses, so the rows may start anywhere)
    from paper_2506_13059_amd import binding as mp
    print(f"offset={offset}", flush=True)
    U, n, tail = 3, 300, 60
    ctx, K, V = _context(U, n, 10, tail)
    g = torch.Generator(device="cuda").manual_seed(1)
    rows = [torch.randn(U, 1, m, 128, generator=g, device="cuda").to(torch.bfloat16) for m in (5, 5, 21, 21)]
    q, kn, vn = (torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16) for s in ((U, 2, 128), (U, 1, 1, 128), (U, 1, 1, 128)))
    out = []
    for by in (0, offset):
        held = [torch.zeros(x.numel() * 2 + 16, dtype=torch.uint8, device="cuda") for x in rows]
        for h, x in zip(held, rows):
            h[by:by + x.numel() * 2] = x.view(-1).view(torch.uint8)
        ks, vs, kr, vr = (C.c_void_p(h.data_ptr() + by) for h in held)
        st = mp.lib().mp_local_buffer_init(ctx.h, 20, ks, vs, 5, kr, None, vr, 21, C.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0
        out.append(ctx.mp_decode_step(q, kn, vn, 100))
    torch.cuda.synchronize()
    assert torch.equal(*out)
    ref = torch.cat([rows[0], rows[2], kn], 2), torch.cat([rows[1], rows[3], vn], 2)
    assert torch.equal(out[0], ctx.mp_decode_attention(q, 100, 0, *ref))
    ctx.close()
