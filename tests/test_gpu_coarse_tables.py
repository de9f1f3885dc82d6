"""GPU parity of the coarse tables (`coarse_from_children_kernel`: 64 children's places and counts at a time, eight sums in
flight) at its edges: children of one coarse cluster around eight and 64, one and two coarse clusters.  Bit-identical to the
oracle's."""
import pytest

from tests.test_gpu_kmeans import _run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc", [1, 2])
@pytest.mark.parametrize("nf", [2, 7, 8, 9, 63, 64, 65, 72, 128, 129, 193])
def test_children(nf, nc):
    print(f"nf={nf} nc={nc}", flush=True)
    ctx, _, _ = _run_case(1, 2, 2, nf + 300, max(2, nf // 3), 2, nf, nc, 0, 0, iters=2, seed=900 + nf + nc)
    ctx.close()
