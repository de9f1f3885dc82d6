"""GPU parity of the scoring launch at the edges of its register path: a level takes ceil(n / 128) rounds of 16
entries per wave, 512 entries per chunk, up to 1024 entries; beyond that the general path takes over.  Logits beyond
the range that is exponentiated without a shift, scores below the range of a double, and boundary buckets with many
equal scores leave the common path.  Each case against the oracle, to the bar of the other decode tests."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _ctx(G, nf, nc, softness, seed):
    from paper_2506_13059_amd import binding as mp, inputs
    U, n = 2, max(3 * nf, 40)
    centers = inputs.make_modes(U, max(2, nf // 2), "cuda", seed)
    K, V = inputs.draw_tokens(centers, n, seed + 1)
    K, V = K.view(1, U, n, 128), V.view(1, U, n, 128)
    q = inputs.draw_queries(centers, G, 1, seed + 2, softness=softness).view(1, U * G, 128)
    g = torch.Generator(device="cuda").manual_seed(seed + 3)
    fot = torch.randint(0, nf, (U, n), generator=g, device="cuda").to(torch.int32)
    cof = None
    if nc:
        cof = torch.sort(torch.randint(0, nc, (U, nf), generator=g, device="cuda"), dim=1).values.to(torch.int32).contiguous()
    ctx = mp.MpContext(1, U * G, U, max_tokens=n, levels=2 if nc else 1, max_fine=nf, max_coarse=nc)
    ctx.mp_set_clustering(K, V, fot, nf, cof, nc)
    return ctx, K, V, q, n


@pytest.mark.parametrize("nf", [1, 15, 127, 128, 129, 257, 385, 511, 512, 513, 641, 1023, 1024, 1025])
def test_one_level_of_every_shape(nf):
    from tests.gpu_util import compare_decode
    for G in (1, 4, 5):
        ctx, K, V, q, n = _ctx(G, nf, 0, 0.2, 40 + nf)
        print(f"nf={nf} G={G}", flush=True)
        for kb in (n // 16 + 1, n // 2):
            compare_decode(ctx, q, K, V, kb, label=f"nf={nf} G={G} kb={kb}")
        ctx.close()


# coarse x fine levels on either path: both in registers, long coarse level, long candidate list, both long
@pytest.mark.parametrize("nf,nc,G", [(700, 130, 4), (700, 513, 8), (1500, 1100, 3), (1500, 60, 7), (2300, 1200, 2)])
def test_two_levels_on_both_paths(nf, nc, G):
    from tests.gpu_util import compare_decode
    ctx, K, V, q, n = _ctx(G, nf, nc, 0.2, 900 + nf + nc)
    for kb, cb in ((n // 16, n // 4), (n // 3, n - 7)):
        print(f"nf={nf} nc={nc} G={G} kb={kb} cb={cb}", flush=True)
        compare_decode(ctx, q, K, V, kb, cb, label=f"nf={nf} nc={nc} kb={kb}")
    ctx.close()


# logits of several hundred to some thousand: shifts at both levels (or at one of them), scores that leave a double
@pytest.mark.parametrize("softness", [2.0, 6.0, 12.0])
@pytest.mark.parametrize("nf,nc", [(300, 0), (600, 40), (1300, 30)])
def test_far_logits(nf, nc, softness):
    from tests.gpu_util import compare_decode
    ctx, K, V, q, n = _ctx(4, nf, nc, softness, 70 + nf)
    print(f"nf={nf} nc={nc} softness={softness}", flush=True)
    compare_decode(ctx, q, K, V, n // 5, n // 2, label=f"far nf={nf} softness={softness}")
    ctx.close()


@pytest.mark.parametrize("nf", [100, 400, 900])
def test_all_scores_equal(nf):
    """A zero query: every cluster has the same score, the boundary bucket holds the whole level, lower ids go first."""
    from tests.gpu_util import compare_decode
    ctx, K, V, q, n = _ctx(4, nf, 0, 0.2, 300 + nf)
    r = compare_decode(ctx, torch.zeros_like(q), K, V, n // 3, label=f"equal nf={nf}")
    assert r["exempt"] == 0
    ctx.close()


@pytest.mark.parametrize("nf,nc,G", [(400, 0, 1), (900, 0, 3), (1024, 0, 4), (900, 400, 5), (700, 300, 8)])
@pytest.mark.parametrize("softness", [0.0005, 0.004, 0.02])
def test_flat_attention(nf, nc, G, softness):
    """Scores of a whole level within a fraction of an octave and yet all different: the boundary is found by the second
    digit of the selection, or, where even its slices are crowded, by the general search."""
    from tests.gpu_util import compare_decode
    ctx, K, V, q, n = _ctx(G, nf, nc, softness, 600 + nf + G)
    print(f"nf={nf} nc={nc} G={G} softness={softness}", flush=True)
    for kb, cb in ((n // 16, n // 4), (n // 3, n // 2), (n - 5, n - 9)):
        compare_decode(ctx, q, K, V, kb, cb, label=f"flat nf={nf} G={G} kb={kb}")
    ctx.close()
