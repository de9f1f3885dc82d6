"""Merging of partial results at the edges of its variants: as many chunks as a dense call of one unit is cut into, against the
definition in 64 bits; and a chunk that has vanished beside the others, whatever its values, as if it were not there."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunks", [1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65, 128, 129])
def test_chunk_counts(chunks):
    from paper_2506_13059_amd import binding as mp
    G, n = 3, 512 * chunks - 5
    g = torch.Generator(device="cuda").manual_seed(chunks)
    q, K, V = (torch.randn(1, h, *s, generator=g, device="cuda").to(torch.bfloat16) for h, s in ((G, (128,)), (1, (n, 128)), (1, (n, 128))))
    q = q * 3.0
    K[0, 0, 300:] *= torch.linspace(0.2, 1.5, max(n - 300, 0), device="cuda")[:, None].to(torch.bfloat16)     # (the chunks' maxima differ)
    lse = torch.empty(1, G, device="cuda")
    out = mp.mp_dense_attention(q, K, V, lse=lse)
    l = q[0].double() @ K[0, 0].double().T / math.sqrt(128)
    want = torch.softmax(l, 1) @ V[0, 0].double()
    # bf16 outputs: half a unit in the last place of each, and fp32 sums
    assert ((out[0].double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5 * want.abs().max()).all()
    assert (lse[0].double() - torch.logsumexp(l, 1)).abs().max() <= 2e-5 * l.abs().max()


# All chunks but one have logits 200 below it, so their weight is zero in fp32, and values with infinities and NaN: whole batches and
# shares of them give what the chunk alone does (one unit's chunks have 512 rows each).
@pytest.mark.parametrize("kept", ["first", "last"])
@pytest.mark.parametrize("chunks", [2, 3, 8, 9, 16, 17, 32, 33, 64, 65, 129, 256])
def test_vanished_chunks_are_not_looked_at(chunks, kept):
    from paper_2506_13059_amd import binding as mp
    G, n = 3, 512 * chunks
    print(f"chunks={chunks} kept={kept}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(chunks)
    q = torch.ones(1, G, 128, device="cuda", dtype=torch.bfloat16)
    K, V = (torch.randn(1, 1, n, 128, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    K *= 0.1
    a, b = (512, n) if kept == "first" else (0, n - 512)
    K[:, :, a:b] -= 200.0 / math.sqrt(128)
    want = mp.mp_dense_attention(q, K, V)
    for x, dim in ((math.inf, 5), (math.nan, 7), (-math.inf, 126)):
        V[:, :, a + dim:b:512, dim] = x
    lse = torch.empty(1, G, device="cuda")
    out = mp.mp_dense_attention(q, K, V, lse=lse)
    assert torch.isfinite(want).all() and torch.isfinite(lse).all()
    assert torch.equal(out, want)
