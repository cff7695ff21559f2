"""Row normalisers of the target stream where chunks and rows meet: rows
shorter than the shortest chunk (one row per chunk, padded to eight logits, so
that chunks cross row ends on odd vocabularies), rows around it, and longer
ones, with and without vector loads.

Tolerance: the stream adds eight binary32 terms, each within 2^-23 of its
value (one FMA and one exponential), before it goes on in binary64; with the
argument's own rounding (|a - max| <= 64: 64 * 2^-24 = 3.8e-6 of a term that
is then below e^-64) the sum is within 8 * 2^-23 = 1e-6 of exact, and ln of it
by the same absolute amount; 2e-6 is allowed.
"""
import pytest
import torch

import paper_2609_33652_amd as tsb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("R,V,B", [(1, 8, 3), (1, 1001, 16), (3, 1024, 16), (2, 8191, 7), (1, 32761, 5), (1, 32768, 5),
                                   (1, 32776, 3), (2, 70001, 3)])
def test_target_rows_over_chunk_edges(R, V, B, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    D, K, T = 4, 4, 1.25
    g = torch.Generator().manual_seed(V * 10 + B)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    draft = (3.0 * torch.randn(R, D, V, generator=g)).to(dt).cuda()
    target = (3.0 * torch.randn(R, B + 1, V, generator=g)).to(dt)
    rnd = tsb.Round(tsb.make_config(R, D, V, B, K, T, dtype, 7), "cuda", target_lse=True)
    rnd.step(draft, target.cuda(), 1)
    h = rnd.host()
    inv_t = torch.tensor(1.0) / torch.tensor(T)
    want = torch.logsumexp((target.float() * inv_t).double(), 2)
    for r in range(R):
        n = int(h["n_nodes"][r])
        assert n == B + 1
        assert torch.allclose(h["target_lse"][r, :n], want[r, :n], rtol=0.0, atol=2e-6), (r, V, B, dtype)
    assert not (h["req_status"] & (tsb.REQ_NONFINITE | tsb.REQ_WALK_TIMEOUT)).any()
