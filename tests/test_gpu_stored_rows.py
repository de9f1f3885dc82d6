"""GPU parity of the stored rows and the tables that come with them (`stored_rows_kernel`): clusters around the batches of a wave (32 and
64 members), empty and long ones, stored by their clusters' waves or by their places (many or few clusters in all), with the rows
of the last block kept for an update, with and without lookup keys, against their definitions: rows in stable cluster order, means of the
members in 64 bits (inputs whose sums are exact) rounded once.  Bit-identical."""
import pytest
import torch

pytestmark = pytest.mark.gpu

SIZES = [0, 1, 2, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 191, 400]


def _rows(U, n, seed):
    # multiples of 2^-6 up to 8: sums of any order are exact
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randint(-512, 513, (U, n, 128), generator=g, device="cuda") / 64.0).to(torch.bfloat16)


def _clusters(U, F, seed):
    """Ids of all units: the sizes of SIZES in turn (so many clusters of each), in random order of the tokens."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    ids = []
    for u in range(U):
        sizes = torch.tensor([SIZES[(f + u) % len(SIZES)] for f in range(F)], device="cuda")
        x = torch.repeat_interleave(torch.arange(F, device="cuda"), sizes)
        ids.append(x[torch.rand(len(x), generator=g, device="cuda").argsort()])
    return torch.stack(ids).to(torch.int32)


def _means(X, ids, F):
    U = X.shape[0]
    s = torch.zeros(U, F, 128, dtype=torch.float64, device="cuda").scatter_add_(1, ids.long()[..., None].expand(-1, -1, 128), X.double())
    n = torch.zeros(U, F, dtype=torch.int64, device="cuda").scatter_add_(1, ids.long(), torch.ones_like(ids, dtype=torch.int64))
    return torch.where(n[..., None] > 0, s / n.clamp(min=1)[..., None], 0.0), n


def _check(ctx, K, V, Kl, ids, F):
    kp, vp, perm, _ = ctx.mp_get_layout()
    order = torch.sort(ids, dim=1, stable=True).indices
    assert torch.equal(perm.long(), order)
    at = order[..., None].expand(-1, -1, 128)
    assert torch.equal(kp, torch.gather(K, 1, at)) and torch.equal(vp, torch.gather(V, 1, at))
    kc, vc, members = ctx.mp_get_centroids(0)[:3]
    for got, X in ((kc, K if Kl is None else Kl), (vc, V)):
        mean, n = _means(X, ids, F)
        assert torch.equal(got.view(mean.shape), mean.to(torch.bfloat16))
        assert torch.equal(members.view(n.shape).long(), n)


# F a multiple of the number of sizes: all units have the same number of tokens; U * F on both sides of the line
@pytest.mark.parametrize("lookup", [False, True])
@pytest.mark.parametrize("U,F,levels", [(1, 16, 1), (3, 32, 2), (24, 32, 2), (25, 32, 1), (50, 16, 2), (400, 16, 2)])
def test_given_clustering(U, F, levels, lookup):
    from paper_2506_13059_amd import binding as mp
    print(f"U={U} F={F} levels={levels} lookup={lookup}", flush=True)
    ids = _clusters(U, F, 5)
    n = ids.shape[1]
    K, V, Kl = _rows(U, n, 1), _rows(U, n, 2), _rows(U, n, 3) if lookup else None
    cof = (torch.arange(F, device="cuda", dtype=torch.int32) // 8)[None].expand(U, -1).contiguous() if levels == 2 else None
    ctx = mp.MpContext(U, 2, 1, max_tokens=n + 128, levels=levels, max_fine=F + 8, max_coarse=F // 8 + 2 if levels == 2 else 0, block_w=1024,
                       block_alpha=512, lookup_keys=lookup)
    b = lambda x: None if x is None else x.view(U, 1, -1, 128)      # noqa: E731
    ctx.mp_set_clustering(b(K), b(V), ids, F, cof, F // 8 if levels == 2 else 0, k_lookup=b(Kl))
    torch.cuda.synchronize()
    _check(ctx, K, V, Kl, ids, F)
    ctx.close()


# a unit has the same index whether its rows were stored by its clusters' waves (among many units) or by their places (alone), and so does
# the update that starts from the rows kept of its last block
@pytest.mark.parametrize("lookup", [False, True])
@pytest.mark.parametrize("given", [False, True])
def test_alone_and_among_others(given, lookup):
    from paper_2506_13059_amd import binding as mp
    U, n, F, C, new = (72, 1459, 16, 2, 64) if given else (72, 2300, 90, 6, 64)
    K, V, Kl = _rows(U, n + new, 11), _rows(U, n + new, 12), _rows(U, n + new, 13) if lookup else None
    ids, cof = _clusters(U, F, 7) if given else None, (torch.arange(F, device="cuda", dtype=torch.int32) // 8)[None].expand(U, -1)
    assert not given or ids.shape[1] == n
    g = torch.Generator().manual_seed(3)
    plan = mp.mp_plan_blocks(n, 1024, 512, F, C)
    pick = lambda of, a, b: torch.cat([torch.randperm(x[of[1]] - x[of[0]], generator=g)[:x[b] - x[a]] for x in plan])      # noqa: E731
    f = torch.stack([pick(("t0", "t1"), "f0", "f1") for _ in range(U)]).to(torch.int32)
    c = torch.stack([pick(("f0", "f1"), "c0", "c1") for _ in range(U)]).to(torch.int32)
    seeds = torch.tensor([[3, 40, 7, 9, 0]], dtype=torch.int32).expand(U, -1)

    def index(units):
        print(f"units={len(units)} given={given} lookup={lookup}", flush=True)
        m = len(units)
        at = lambda x, a, b: None if x is None else x[units, a:b].contiguous().view(m, 1, -1, 128)      # noqa: E731
        ctx = mp.MpContext(m, 2, 1, max_tokens=n + new, levels=2, max_fine=F + 4, max_coarse=C + 1, block_w=1024, block_alpha=512, lookup_keys=lookup)
        if given:
            ctx.mp_set_clustering(at(K, 0, n), at(V, 0, n), ids[units].contiguous(), F, cof[units].contiguous(), C, k_lookup=at(Kl, 0, n))
        else:
            ctx.mp_cluster_kv(at(K, 0, n), at(V, 0, n), F, C, iters=3, init_fine=f[units], init_coarse=c[units], k_lookup=at(Kl, 0, n))
        out = [x.clone() for x in list(ctx.mp_get_layout()) + list(ctx.mp_get_centroids(0)) + list(ctx.mp_get_centroids(1))]
        ctx.mp_update_clusters(at(K, n, n + new), at(V, n, n + new), 4, 1, refine_iters=2, seeds=seeds[units], k_new_lookup=at(Kl, n, n + new))
        out += list(ctx.mp_get_layout()) + list(ctx.mp_get_centroids(0)) + list(ctx.mp_get_centroids(1))
        torch.cuda.synchronize()
        ctx.close()
        return [x.reshape(m, -1) for x in out]

    many = index(list(range(U)))
    assert U * F > (768 if given else 6144) and F <= 768      # (the lines between the two ways)
    for u in (0, 35, U - 1):
        for a, b in zip(many, index([u])):
            assert torch.equal(a[u], b[0])


# many clusters of few rows (batches of up to four, and just above), some empty, workgroups without a long cluster; an update that refines
# nothing (an empty cluster keeps its key centroid)
@pytest.mark.parametrize("lookup", [False, True])
@pytest.mark.parametrize("refine", [0, 1])
def test_small_clusters(lookup, refine):
    from paper_2506_13059_amd import binding as mp
    U, F, new = 61, 396, 40
    g = torch.Generator(device="cuda").manual_seed(9)
    ids = torch.cat([torch.randint(0, F - 8, (U, 1400), generator=g, device="cuda"), torch.full((U, 100), F - 3, device="cuda")], 1).to(torch.int32)
    n = ids.shape[1]
    assert U * F > 6144 >= 8 * F      # (stored by the clusters' waves; alone by places)
    K, V, Kl = _rows(U, n + new, 21), _rows(U, n + new, 22), _rows(U, n + new, 23) if lookup else None
    cof = (torch.arange(F, device="cuda", dtype=torch.int32) // 8)[None].expand(U, -1)
    C = F // 8 + 1
    seeds = torch.tensor([[3, 30, 7]], dtype=torch.int32).expand(U, -1)

    def index(units):
        print(f"units={len(units)} lookup={lookup} refine={refine}", flush=True)
        m = len(units)
        at = lambda x, a, b: None if x is None else x[units, a:b].contiguous().view(m, 1, -1, 128)      # noqa: E731
        ctx = mp.MpContext(m, 2, 1, max_tokens=n + new, levels=2, max_fine=F + 3, max_coarse=C, lookup_keys=lookup)
        ctx.mp_set_clustering(at(K, 0, n), at(V, 0, n), ids[units].contiguous(), F, cof[units].contiguous(), C, k_lookup=at(Kl, 0, n))
        _check(ctx, K[units, :n], V[units, :n], None if Kl is None else Kl[units, :n], ids[units], F)
        out = [x.clone() for x in list(ctx.mp_get_centroids(0)) + list(ctx.mp_get_centroids(1))]
        ctx.mp_update_clusters(at(K, n, n + new), at(V, n, n + new), 3, 0, refine_iters=refine, seeds=seeds[units], k_new_lookup=at(Kl, n, n + new))
        out += list(ctx.mp_get_layout()) + list(ctx.mp_get_centroids(0)) + list(ctx.mp_get_centroids(1))
        torch.cuda.synchronize()
        ctx.close()
        return [x.reshape(m, -1) for x in out]

    many = index(list(range(U)))
    for u in (0, U - 1):
        for a, b in zip(many, index([u])):
            assert torch.equal(a[u], b[0])


# so many clusters that their sums go past the caches, of both tables and (lookup keys) of the values' alone; a unit's tables, the coarse ones
# added up from the sums among them, are those it has alone
@pytest.mark.parametrize("U,lookup", [(305, False), (600, True)])
def test_sums_past_the_caches(U, lookup):
    from paper_2506_13059_amd import binding as mp
    F, n, C = 512, 700, 64
    assert U * F * (1 if lookup else 2) > 300000
    g = torch.Generator(device="cuda").manual_seed(31)
    ids = torch.randint(0, F, (U, n), generator=g, device="cuda").to(torch.int32)
    K, V, Kl = _rows(U, n, 32), _rows(U, n, 33), _rows(U, n, 34) if lookup else None
    cof = (torch.arange(F, device="cuda", dtype=torch.int32) // 8)[None].expand(U, -1)

    def index(units):
        print(f"units={len(units)} lookup={lookup}", flush=True)
        m = len(units)
        at = lambda x: None if x is None else x[units].contiguous().view(m, 1, -1, 128)      # noqa: E731
        ctx = mp.MpContext(m, 2, 1, max_tokens=n, levels=2, max_fine=F, max_coarse=C, lookup_keys=lookup)
        ctx.mp_set_clustering(at(K), at(V), ids[units].contiguous(), F, cof[units].contiguous(), C, k_lookup=at(Kl))
        _check(ctx, K[units], V[units], None if Kl is None else Kl[units], ids[units], F)
        out = [x.clone().reshape(m, -1) for x in list(ctx.mp_get_centroids(0)) + list(ctx.mp_get_centroids(1))]
        torch.cuda.synchronize()
        ctx.close()
        return out

    many = index(list(range(U)))
    for u in (0, U // 2, U - 1):
        for a, b in zip(many, index([u])):
            assert torch.equal(a[u], b[0])
