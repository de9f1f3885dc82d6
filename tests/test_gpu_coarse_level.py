"""GPU parity of the coarse level in one launch at its edges: chunks of 64 points, tiles of 16 centroids, its limits (512
points, 63 centroids, or more of them over few points; one more takes the launch-per-step path, which the larger cases
are for), sixteen waves up to 256 (block, unit) pairs and eight beyond, and degenerate inputs.  Every result is
bit-identical to the oracle's."""
import pytest

from tests.test_gpu_kmeans import _run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nf,nc", [(1, 1), (2, 1), (63, 15), (64, 16), (65, 17), (129, 64), (500, 255), (511, 256),
                                   (510, 257), (512, 16), (513, 16), (1025, 16)])
def test_edges(nf, nc):
    print(f"nf={nf} nc={nc}", flush=True)
    ctx, _, _ = _run_case(1, 2, 2, nf + 300, max(2, nf // 3), 2, nf, nc, 0, 0, iters=3, seed=500 + nf + nc)
    ctx.close()


@pytest.mark.parametrize("nf,nc", [(512, 63), (512, 64), (160, 64), (161, 64), (101, 101), (102, 102), (255, 40)])
def test_limits(nf, nc):
    print(f"nf={nf} nc={nc}", flush=True)
    ctx, _, _ = _run_case(1, 2, 2, nf + 300, max(2, nf // 3), 2, nf, nc, 0, 0, iters=3, seed=700 + nf + nc)
    ctx.close()


def test_limits_of_many_pairs():
    # 32 pairs take up to 64 centroids over 256 points
    ctx, _, _ = _run_case(8, 4, 4, 700, 90, 2, 250, 64, 0, 0, iters=2, seed=53)
    ctx.close()


def test_more_pairs_than_compute_units():
    ctx, _, _ = _run_case(9, 4, 4, 1100, 20, 2, 130, 20, 128, 64, iters=2, seed=51)
    assert 36 * ctx.mp_get_sizes()["n_blocks"] > 256
    ctx.close()


@pytest.mark.parametrize("distinct", [1, 9])
def test_every_point_a_near_tie(distinct):
    ctx, _, _ = _run_case(1, 2, 2, 600, 4, 2, 200, 40, 0, 0, iters=3, seed=52, distinct_rows=distinct)
    ctx.close()


@pytest.mark.parametrize("W,fine", [(600, 250), (900, 262), (900, 400)])
def test_many_pairs_with_and_without_points_in_lds(W, fine):
    # 264 pairs of 8-wave workgroups: points in LDS up to 311 less the centroids
    ctx, _, _ = _run_case(66, 4, 4, W, 40, 2, fine, 24, 0, 0, iters=3, seed=fine)
    ctx.close()
