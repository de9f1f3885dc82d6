"""GPU parity of the assignment steps that look at the changed centroids only (from the fourth iteration of a build, the second of an
update's refinement): bit-identical to the oracle, with centroids that come to rest one after the other, ties that stay ties,
lists longer than their place in LDS, both sizes of workgroup and blocks of several sizes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _keys(kind, n, seed):
    g = torch.Generator().manual_seed(seed)
    if kind == "modes":              # tight modes beside loose ones: some centroids rest early
        c = 3.0 * torch.randn(60, 128, generator=g)
        m = torch.randint(0, 60, (n,), generator=g)
        x = c[m] + torch.where(m < 40, 0.05, 2.0)[:, None] * torch.randn(n, 128, generator=g)
    elif kind == "grid":             # few values: equal distances all over
        x = torch.randint(-1, 2, (n, 128), generator=g) * (torch.arange(128) < 6).float()
    elif kind == "copies":           # many keys of the same few rows, and keys without clusters
        x = torch.randn(n, 128, generator=g)
        x[: n // 2] = x[torch.randint(0, 5, (n // 2,), generator=g)]
    elif kind == "far":              # one key large: every margin is, and all points stay on the lists
        x = torch.randn(n, 128, generator=g)
        x[n // 3] = 20000.0
    else:
        x = torch.randn(n, 128, generator=g)
    return x.to(torch.bfloat16)


@pytest.mark.parametrize("kind,n,k,iters,refine", [
    ("modes", 8192, 256, 9, 0), ("modes", 1024, 17, 8, 0), ("modes", 4000, 289, 7, 0), ("modes", 4000, 288, 7, 0), ("modes", 2500, 512, 6, 0),
    ("modes", 14000, 80, 8, 0), ("modes", 8192, 200, 1, 5), ("modes", 4100, 300, 2, 4), ("grid", 9000, 120, 8, 0), ("grid", 3600, 300, 6, 3),
    ("copies", 8192, 130, 8, 0), ("copies", 8100, 150, 1, 4), ("far", 6000, 180, 6, 0), ("plain", 66000, 17, 6, 0), ("plain", 11000, 1100, 6, 0)])
def test_settled_iterations(kind, n, k, iters, refine):
    from paper_2506_13059_amd import binding as mp, inputs
    from oracle import mp_oracle as O
    from tests.gpu_util import f64, i32
    print(f"{kind} n={n} k={k} iters={iters} refine={refine}", flush=True)
    n_new, seed = (130 if refine else 0), 70 + n + k
    K = _keys(kind, n + n_new, seed)[None]
    V = torch.randn(1, n + n_new, 128, generator=torch.Generator().manual_seed(5)).to(torch.bfloat16)
    W, A = (4096, 2048) if n == 11000 else (0, 0)            # (blocks of two sizes, both sizes of workgroup)
    blocks = mp.mp_plan_blocks(n, W, A, k, 0)
    init_f, _ = inputs.draw_seeds(1, blocks, 1, 17)
    new_f = 5 if refine else 0
    ctx = mp.MpContext(1, 1, 1, max_tokens=n + n_new, levels=1, max_fine=k + new_f, max_coarse=0, block_w=W, block_alpha=A, max_tail=0)
    part = lambda x, a, b: x[:, a:b].contiguous().cuda().view(1, 1, b - a, 128)
    ctx.mp_cluster_kv(part(K, 0, n), part(V, 0, n), k, 0, iters=iters, init_fine=init_f)
    seeds = np.random.default_rng(3).choice(130, 5, replace=False).astype(np.int32)[None]
    if refine:
        ctx.mp_update_clusters(part(K, n, n + n_new), part(V, n, n + n_new), new_f, 0, refine_iters=refine, split_iters=1, seeds=torch.tensor(seeds))
    got = [i32(x) if x.dtype == torch.int32 else f64(x) for x in (ctx.mp_get_assignments()[0], *ctx.mp_get_centroids(0))]
    ctx.close()
    cl = O.cluster_unit(f64(K)[0, :n], f64(V)[0, :n], blocks, init_f[0].numpy(), None, iters, 1)
    if refine:
        cl = O.update_unit(cl, f64(K)[0, n:], f64(V)[0, n:], new_f, 0, seeds[0], refine, 0, 0)
    for g, name in zip(got, ("fine_of_token", "Kc_f", "Vc_f", "N_f")):
        np.testing.assert_array_equal(g[0], cl[name], err_msg=name)


def test_state_only_where_a_block_can_be_large_enough():
    from paper_2506_13059_amd import binding as mp
    n, W = 200000, 1024

    def size(fine):
        ctx = mp.MpContext(1, 1, 1, max_tokens=n, levels=1, max_fine=fine, block_w=W, block_alpha=W)
        b = ctx.device_bytes()
        ctx.close()
        return b

    # blocks of at most 2 W points: 512 clusters make 2^20 pairs, and the state is 8 bytes a token beside what a cluster costs anyway
    a, b, c = (size(f) for f in (510, 511, 512))
    assert abs((c - b) - (b - a) - 8 * n) < 0.01 * 8 * n
