"""GPU parity of the member lists at the edges of the kernel that ranks a block's points: segments of sixteen steps of 64
points (kept in registers) and one more (walked twice), with sixteen waves and with fewer (blocks of more clusters than
leave room for sixteen segments' counters), ids of 0, 3 and 3 n + 1 bits.  The index is bit-identical to the oracle's."""
import pytest

from tests.test_gpu_kmeans import _run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(63, 1), (64, 2), (1025, 8), (1024, 9), (16384, 20), (16385, 20), (6000, 1023), (6000, 1025),
                                 (14000, 1100)])
def test_edges(n, k):
    print(f"n={n} k={k}", flush=True)
    ctx, _, _ = _run_case(1, 2, 1, n, max(2, k // 3), 1, k, 0, 0, 0, iters=1, seed=700 + n + k)
    ctx.close()
