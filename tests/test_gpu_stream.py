"""GPU parity of the matrix-core value pass at the edges of its tiles (16 rows), strips (64 row numbers), waves and
chunks, for every split of the probabilities (three parts of G heads in 16 columns, or a second set of products), and
of the vector-ALU kernel that rows without 16-byte alignment keep using."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _inputs(B, Hkv, G, n, seed, scale=1.0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    q = (scale * torch.randn(B, Hkv * G, 128, generator=g, device="cuda")).to(torch.bfloat16)
    K = torch.randn(B, Hkv, n, 128, generator=g, device="cuda").to(torch.bfloat16)
    V = torch.randn(B, Hkv, n, 128, generator=g, device="cuda").to(torch.bfloat16)
    return q, K, V


def _reference(q, K, V):
    B, Hq, d = q.shape
    Hkv = K.shape[1]
    qd = q.double().view(B, Hkv, Hq // Hkv, d)
    l = qd @ K.double().transpose(2, 3).contiguous() / math.sqrt(d)
    return (torch.softmax(l, 3) @ V.double()).view(B, Hq, d), torch.logsumexp(l, 3).view(B, Hq)


def _check(out, lse, q, K, V, label):
    ref, ref_lse = _reference(q, K, V)
    # one rounding to bf16: half a step of eight significant bits, at most 2^-8 of the value; the fp32 arithmetic
    # before it (sums of up to 128 products and of the rows, relative error around 1e-6) moves the value far less
    err = (out.double() - ref).abs()
    bound = 2.0 ** -8 * ref.abs() + 2e-5 * ref.abs().max()
    assert bool((err <= bound).all()), (label, float((err - bound).max()))
    np.testing.assert_allclose(lse.cpu().numpy(), ref_lse.cpu().numpy(), rtol=2e-6, atol=2e-5, err_msg=label)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 129, 255, 1025, 4100, 20011])
def test_dense_tile_edges(n):
    from paper_2506_13059_amd import binding as mp
    for G in (1, 2, 3, 4, 5, 6, 7, 8):
        q, K, V = _inputs(2, 2, G, n, 10 * n + G, scale=3.0 if G % 2 else 1.0)
        print(f"n={n} G={G}", flush=True)
        lse = torch.empty(q.shape[:2], dtype=torch.float32, device="cuda")
        out = mp.mp_dense_attention(q, K, V, lse=lse)
        torch.cuda.synchronize()
        _check(out, lse, q, K, V, f"n={n} G={G}")


def test_more_units_than_compute_units():
    from paper_2506_13059_amd import binding as mp
    q, K, V = _inputs(150, 2, 2, 700, 5)
    lse = torch.empty(q.shape[:2], dtype=torch.float32, device="cuda")
    out = mp.mp_dense_attention(q, K, V, lse=lse)
    torch.cuda.synchronize()
    _check(out, lse, q, K, V, "300 units")


def _shifted(x, elements):
    """The same rows, starting `elements` 16-bit values behind an aligned address."""
    buf = torch.empty(x.numel() + elements, dtype=x.dtype, device=x.device)
    y = buf[elements:].view(x.shape)
    y.copy_(x)
    assert y.data_ptr() % 16 == 2 * elements
    return y


@pytest.mark.parametrize("G", [1, 4, 5, 6, 8])
@pytest.mark.parametrize("n", [100, 2500])
def test_rows_that_do_not_start_on_16_bytes(G, n):
    from paper_2506_13059_amd import binding as mp
    q, K, V = _inputs(1, 2, G, n, 77 + G)
    for dk, dv in ((4, 0), (0, 4), (2, 6)):
        print(f"G={G} n={n} shifts {dk} {dv}", flush=True)
        lse = torch.empty(q.shape[:2], dtype=torch.float32, device="cuda")
        out = mp.mp_dense_attention(q, _shifted(K, dk) if dk else K, _shifted(V, dv) if dv else V, lse=lse)
        torch.cuda.synchronize()
        _check(out, lse, q, K, V, f"G={G} n={n} {dk} {dv}")


def test_decode_with_a_tail_that_does_not_start_on_16_bytes():
    from paper_2506_13059_amd import binding as mp, inputs
    centers = inputs.make_modes(2, 40, "cuda", 9)
    K, V = inputs.draw_tokens(centers, 1500, 10)
    K, V = K.view(1, 2, 1500, 128), V.view(1, 2, 1500, 128)
    q = inputs.draw_queries(centers, 4, 1, 11, softness=0.2).view(1, 8, 128)
    fot = torch.arange(1500, device="cuda", dtype=torch.int32).remainder(60).expand(2, -1).contiguous()
    ctx = mp.MpContext(1, 8, 2, max_tokens=1500, levels=1, max_fine=60, max_tail=70)
    ctx.mp_set_clustering(K, V, fot, 60)
    kt, vt = K[:, :, :70].contiguous(), V[:, :, 100:170].contiguous()
    a = ctx.mp_decode_attention(q, 400, 0, kt, vt)
    b = ctx.mp_decode_attention(q, 400, 0, _shifted(kt, 4), _shifted(vt, 2))
    torch.cuda.synchronize()
    # two kernels, the same fp32 sums in another order: at most one step of the bf16 output (2^-7 of the value) apart
    assert bool(((a.double() - b.double()).abs() <= 2.0 ** -7 * a.double().abs() + 1e-5).all())
    ctx.close()


def test_results_do_not_depend_on_the_size_of_the_workspace():
    """The stated workspace has room for fewer chunks than the kernel would take for short contexts."""
    from paper_2506_13059_amd import binding as mp
    q, K, V = _inputs(1, 2, 4, 3000, 3)
    need = mp.mp_dense_workspace_bytes(1, 8, 2, 3000)
    outs = []
    for size in (need, 2 * need + 100, 16 * need):
        lse = torch.empty(1, 8, dtype=torch.float32, device="cuda")
        ws = torch.full((size,), 255, dtype=torch.uint8, device="cuda")
        outs.append(mp.mp_dense_attention(q, K, V, lse=lse, workspace=ws))
        torch.cuda.synchronize()
        _check(outs[-1], lse, q, K, V, f"workspace {size}")
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    with pytest.raises(mp.MpError) as e:
        mp.mp_dense_attention(q, K, V, workspace=torch.empty(need - 1, dtype=torch.uint8, device="cuda"))
    assert e.value.status == mp.MP_EINVAL


@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("n", [1, 37, 500, 2511])
def test_infinite_values(G, n):
    """A value row with an infinity: every probability is above zero, so the output's dimension is that infinity, NaN where
    both signs meet or a value is NaN, and the other dimensions are what they are without it."""
    from paper_2506_13059_amd import binding as mp
    q, K, V = _inputs(2, 2, G, n, 900 + 10 * G + n)
    ref, _ = _reference(q, K, V)
    X = V.clone()
    last, some = n - 1, n // 3
    X[:, :, last, 5] = math.inf
    X[:, :, some, 77] = -math.inf
    X[:, :, some, 127] = math.nan
    both = n > 1
    if both:
        X[:, :, last, 64], X[:, :, some, 64] = math.inf, -math.inf
    for shift in (0, 4):          # (rows off 16 bytes: the vector-ALU kernel)
        print(f"G={G} n={n} shift={shift}", flush=True)
        out = mp.mp_dense_attention(q, K, _shifted(X, shift) if shift else X).double()
        torch.cuda.synchronize()
        assert bool((out[..., 5] == math.inf).all()) and bool((out[..., 77] == -math.inf).all())
        assert bool(out[..., 127].isnan().all()) and (not both or bool(out[..., 64].isnan().all()))
        rest = [d for d in range(128) if d not in (5, 77, 127) and not (both and d == 64)]
        err = (out - ref)[..., rest].abs()
        assert bool((err <= 2.0 ** -8 * ref[..., rest].abs() + 2e-5 * ref.abs().max()).all())


def test_infinite_values_of_a_decode_step():
    from paper_2506_13059_amd import binding as mp, inputs
    centers = inputs.make_modes(2, 40, "cuda", 9)
    K, V = inputs.draw_tokens(centers, 1500, 10)
    K, V = K.view(1, 2, 1500, 128).contiguous(), V.view(1, 2, 1500, 128).clone()
    V[:, :, 60 * 7 + 11, 3] = math.inf              # (token 431: a member of cluster 11)
    q = inputs.draw_queries(centers, 4, 1, 11, softness=0.05).view(1, 8, 128)
    fot = torch.arange(1500, device="cuda", dtype=torch.int32).remainder(60).expand(2, -1).contiguous()
    kt, vt = K[:, :, :70].contiguous(), V[:, :, 100:170].clone()
    vt[:, :, 69, 9] = -math.inf
    ctx = mp.MpContext(1, 8, 2, max_tokens=1500, levels=1, max_fine=60, max_tail=70)
    ctx.mp_set_clustering(K, V, fot, 60)
    for budget in (1500, 300, 0):                   # as a row, as a row or a centroid term, as a centroid term
        out = ctx.mp_decode_attention(q, budget, 0, kt, vt)
        torch.cuda.synchronize()
        assert bool((out[..., 3] == math.inf).all()) and bool((out[..., 9] == -math.inf).all()), budget
        rest = [d for d in range(128) if d not in (3, 9)]
        assert bool(out[..., rest].isfinite().all()), budget
    ctx.close()
