"""GPU parity of the k-means assignment at the edges of the kernel that keeps a block's centroids in LDS: tiles of 16
centroids (ragged last tile), slots of sixteen tiles (more than 256 centroids take a second half), eight or sixteen
waves a workgroup (304 centroids and more), the limit of 512, and chunks of 64 points with a ragged end.  Assignments,
counts and centroids are bit-identical to the oracle's."""
import pytest

from tests.test_gpu_kmeans import _run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,n", [(1, 1024), (15, 1025), (16, 1087), (17, 1100), (255, 2113), (256, 1500), (257, 1535),
                                 (273, 2050), (304, 1801), (305, 1801), (400, 1999), (512, 2300), (513, 1600)])
def test_centroid_counts(k, n):
    print(f"k={k} n={n}", flush=True)
    ctx, _, _ = _run_case(1, 2, 2, n, max(2, k // 3), 1, k, 0, 0, 0, iters=2, seed=300 + k)
    ctx.close()


def test_more_near_ties_than_a_workgroup_lists_in_lds():
    # one distinct key row: every point of every workgroup goes to the exact pass
    ctx, _, _ = _run_case(1, 2, 1, 9000, 4, 1, 40, 0, 0, 0, iters=1, seed=21, distinct_rows=1)
    ctx.close()


def test_many_blocks_of_many_units():
    # (block, unit) pairs beyond one round of workgroups are covered by the full-size test; here a handful with ragged ends
    ctx, _, _ = _run_case(2, 4, 2, 5000, 60, 2, 150, 10, 1200, 600, iters=2, seed=22)
    assert ctx.mp_get_sizes()["n_blocks"] == 4
    ctx.close()


@pytest.mark.parametrize("nf", [1130, 1140, 920])
def test_blocks_on_both_sides_of_a_limit(nf):
    """The largest block of a launch decides its kernel: 508 / 513 / 414 centroids in the first block, 622 / 627 / 506 in the
    last, so that one, both or none is beyond 512; the coarse level's points are the same counts."""
    print(f"nf={nf}", flush=True)
    ctx, _, _ = _run_case(1, 4, 2, 4548, 200, 2, nf, 40, 2048, 1024, iters=2, seed=400 + nf)
    assert ctx.mp_get_sizes()["n_blocks"] == 2
    ctx.close()


def test_kernels_in_turn_on_one_context():
    # blocks of 600 centroids keep their near ties in a list that a second launch works off, blocks of 100 decide them
    # at once: each finds the other's counters as it needs them, and gives what a context of its own gives
    import torch
    from paper_2506_13059_amd import binding as mp, inputs
    U, n = 2, 3000
    K, V = inputs.draw_tokens(inputs.make_modes(U, 40, "cuda", 31), n, 32, noise=0.05)
    K, V = K.view(1, U, n, 128), V.view(1, U, n, 128)

    def result(ctx, k):
        seeds, _ = inputs.draw_seeds(U, mp.mp_plan_blocks(n, 0, 0, k, 0), 1, 33 + k)
        ctx.mp_cluster_kv(K, V, k, 0, iters=2, init_fine=seeds)
        got = [ctx.mp_get_assignments()[0].clone()] + [x.clone() for x in ctx.mp_get_centroids(0)]
        torch.cuda.synchronize()
        return got

    def fresh():
        return mp.MpContext(1, U, U, max_tokens=n, levels=1, max_fine=600, max_coarse=0, block_w=0, block_alpha=0, max_tail=0)

    one = fresh()
    for k in (600, 100, 600, 600, 100, 100, 600):
        other = fresh()
        for a, b in zip(result(one, k), result(other, k)):
            assert torch.equal(a, b)
        other.close()
    one.close()


@pytest.mark.parametrize("k,n,distinct", [(300, 3000, 1), (512, 3000, 3), (512, 1100, 40)])
def test_few_points_to_a_workgroup(k, n, distinct):
    # one unit: every workgroup has a chunk or two, the exact decisions of its points are shared by waves without points
    ctx, _, _ = _run_case(1, 1, 1, n, 4, 1, k, 0, 0, 0, iters=2, seed=24 + distinct, distinct_rows=distinct)
    ctx.close()
