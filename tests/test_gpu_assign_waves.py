"""GPU parity of the two workgroup widths of `assign_resident_kernel` (sixteen waves for one block of all units, eight for 258): a unit has
the same index alone and among 257 others, at the edges of centroid tiles and chunks of points.  (Alone it is compared with the oracle
in test_gpu_kmeans.py and test_gpu_assign.py.)  Bit-identical."""
import pytest
import torch

from paper_2506_13059_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,F", [(1024, 1), (1025, 16), (1087, 17), (1100, 33), (1500, 100), (1100, 304)])
def test_alone_and_among_others(n, F):
    from paper_2506_13059_amd import binding as mp
    U = 258
    K, V = inputs.draw_tokens(inputs.make_modes(U, 48, "cuda", 7), n, 8)
    K[:, 1::7] = K[:, 0:1]           # (equal keys: near ties)
    g = torch.Generator().manual_seed(n + F)
    seeds = torch.stack([torch.randperm(n, generator=g)[:F] for _ in range(U)]).to(torch.int32)

    def index(units):
        print(f"n={n} F={F} units={len(units)}", flush=True)
        m = len(units)
        ctx = mp.MpContext(m, 2, 1, max_tokens=n, levels=1, max_fine=F)
        ctx.mp_cluster_kv(K[units].contiguous().view(m, 1, n, 128), V[units].contiguous().view(m, 1, n, 128), F, iters=3, init_fine=seeds[units].contiguous())
        ids = ctx.mp_get_assignments()[0]
        out = [ids] + list(ctx.mp_get_centroids(0))
        torch.cuda.synchronize()
        ctx.close()
        return [x.reshape(m, -1) for x in out]

    many = index(list(range(U)))
    for u in (0, 129, U - 1):
        for a, b in zip(many, index([u])):
            assert torch.equal(a[u], b[0])
