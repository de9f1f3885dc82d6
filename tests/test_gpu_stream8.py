"""GPU parity of the matrix-core value pass over 8-bit rows at the edges of its tiles (32 rows), strips (64 row numbers) and
waves, for every split of the probabilities and both column layouts of the logit shares, and of the vector-ALU kernel that
one head to a unit and a tail without 16-byte alignment keep using."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def _context(G, n, tail, seed, clusters=7, values=lambda v: v):
    from paper_2506_13059_amd import binding as mp
    g = torch.Generator(device="cuda").manual_seed(seed)
    q, K, V, kt, vt = (torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
                       for s in ((1, 2 * G, 128), (1, 2, n, 128), (1, 2, n, 128), (1, 2, tail, 128), (1, 2, tail, 128)))
    V, vt = values(V), values(vt)
    k = min(clusters, n)
    fot = (torch.arange(n, device="cuda", dtype=torch.int32) * 5 % k).expand(2, -1).contiguous()
    ctx = mp.MpContext(1, 2 * G, 2, max_tokens=n, levels=1, max_fine=k, max_tail=max(tail, 1), kv_format=mp.MP_KV_E4M3)
    ctx.mp_set_clustering(K, V, fot, k)
    return ctx, q, K, V, kt, vt


def _reference(ctx, q, K, V, kt, vt):
    from tests.test_gpu_fp8 import _dequantised
    Kd, Vd = _dequantised(ctx, K, V)
    out = []
    for u in range(2):
        k, v = torch.cat([Kd[u], kt[0, u].double().cpu()]), torch.cat([Vd[u], vt[0, u].double().cpu()])
        l = q.view(2, -1, 128)[u].double().cpu() @ k.T / math.sqrt(128)
        out.append(torch.softmax(l, 1) @ v)
    return torch.stack(out).view(q.shape)


def _check(got, ref, label):
    # one rounding to bf16 (2^-8 of the value at most), fp32 sums before it
    err = (got.double().cpu() - ref).abs()
    bound = 2.0 ** -8 * ref.abs() + 2e-5 * ref.abs().max() + 2.0 ** -134        # (the last: subnormal bf16)
    assert bool((err <= bound).all()), (label, float((err - bound).max()))


@pytest.mark.parametrize("n", [1, 31, 32, 33, 64, 65, 127, 128, 161, 255, 257, 700, 1025, 9000])
def test_tile_edges(n):
    for G, tail in ((2, 0), (4, 17), (5, 0), (6, 33), (8, 0)):
        print(f"n={n} G={G}", flush=True)
        ctx, q, K, V, kt, vt = _context(G, n, tail, 40 + n + G)
        out = ctx.mp_decode_attention(q, n, 0, kt if tail else None, vt if tail else None)
        _check(out, _reference(ctx, q, K, V, kt, vt), f"n={n} G={G}")
        ctx.close()


def _shifted(x, by):
    flat = torch.empty(x.numel() + by, dtype=x.dtype, device="cuda")[by:]
    flat.copy_(x.reshape(-1))
    return flat.view(x.shape)


@pytest.mark.parametrize("G", [1, 2, 3, 7])
def test_both_kernels(G):
    # a tail off 16 bytes sends the whole launch to the vector ALU; part of the clusters stays behind as centroid terms
    print(f"G={G}", flush=True)
    ctx, q, K, V, kt, vt = _context(G, 1500, 70, 60 + G, clusters=60)
    a = ctx.mp_decode_attention(q, 400, 0, kt, vt)
    b = ctx.mp_decode_attention(q, 400, 0, _shifted(kt, 4), _shifted(vt, 2))
    torch.cuda.synchronize()
    # the same fp32 sums in another order: at most one step of the bf16 output (2^-7 of the value) apart
    assert bool(((a.double() - b.double()).abs() <= 2.0 ** -7 * a.double().abs() + 1e-5).all())
    ctx.close()


@pytest.mark.parametrize("size", [1e-30, 1e-33, 1e-37, 1e15, 1e36, "one large row"])
def test_values_of_any_magnitude(size):
    # (fp32 has the bits of every product that shows in the output; the value scales reach down to 2^-132 and up to 2^116)
    def values(v):
        if size == "one large row":
            x = v.float() * 1e-30
            x[:, :, x.shape[2] // 2] = 1e13 * v.float()[:, :, 0]
            return x.to(torch.bfloat16)
        return (v.float() * size).to(torch.bfloat16)
    for G, n in ((2, 700), (5, 161), (8, 700)):
        print(f"size={size} G={G}", flush=True)
        ctx, q, K, V, kt, vt = _context(G, n, 17, 80 + G, values=values)
        out = ctx.mp_decode_attention(q, n, 0, kt, vt)
        _check(out, _reference(ctx, q, K, V, kt, vt), f"size={size} G={G}")
        ctx.close()


@pytest.mark.parametrize("appended", [False, True])
@pytest.mark.parametrize("G", [2, 4, 8])
def test_infinite_value(G, appended):
    # a row with an infinity has an infinite scale, which leaves no dim of its unit's outputs finite, whichever kernel runs
    from paper_2506_13059_amd import binding as mp

    def values(v):
        v[0, 0, 697 if appended else 233, 9] = float("inf")
        return v
    print(f"G={G} appended={appended}", flush=True)
    ctx, q, K, V, kt, vt = _context(G, 700, 17, 90 + G, values=lambda v: values(v) if v.shape[2] == 700 else v)
    if appended:
        ctx.close()
        ctx = mp.MpContext(1, 2 * G, 2, max_tokens=700, levels=1, max_fine=9, max_tail=17, kv_format=mp.MP_KV_E4M3)
        ctx.mp_cluster_kv(*(x[:, :, :660].contiguous() for x in (K, V)), 7, 0, iters=2, seed=1)
        ctx.mp_update_clusters(*(x[:, :, 660:].contiguous() for x in (K, V)), 1, 0, refine_iters=1, split_iters=1, seed=2)
    a = ctx.mp_decode_attention(q, 700, 0, kt, vt).view(2, G, 128)
    b = ctx.mp_decode_attention(q, 700, 0, _shifted(kt, 4), _shifted(vt, 2)).view(2, G, 128)
    torch.cuda.synchronize()
    assert not bool(torch.isfinite(a[0]).any()) and bool(torch.isfinite(a[1]).all())
    assert torch.equal(torch.nan_to_num(a[0], nan=7.0), torch.nan_to_num(b[0], nan=7.0))
    assert bool(((a[1].double() - b[1].double()).abs() <= 2.0 ** -7 * a[1].double().abs() + 1e-5).all())
    ctx.close()
