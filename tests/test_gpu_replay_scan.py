"""The replay scan where its branches can go wrong: rows around one tile and
around the shortest sampled row, with and without vector loads; flat rows
(whose hits overflow the list of hits, and whose keys exceed a tile's slots),
peaked and masked ones; calls with and without the sampled threshold. Rows of
more keys than the merge ranks at once, and of 64 tiles (a lane each), 65 and
two times 64 and a part.

Every parent's children are compared with the binary64 oracle (a decision
whose margin is below 1e-5, the binary32 key's resolution, is left out, as in
the parity tests), and the pruned scan with the one that scores every token,
bit for bit.
"""
import numpy as np
import pytest
import torch

import paper_2609_33652_amd as tsb
from oracle import replay as oreplay

pytestmark = pytest.mark.gpu


def _rows(kind, R, D, V, g):
    x = torch.randn(R, D, V, generator=g)
    if kind == "flat":
        return 0.05 * x
    if kind == "peaked":
        x *= 5.0
        x[:, :, V // 2] += 12.0
        return x
    if kind == "masked":  # most tokens -inf, the finite ones near the end of the row
        m = torch.rand(R, D, V, generator=g) < 0.98
        m[:, :, -64:] = False
        return x.masked_fill(m, float("-inf"))
    return x * (1.0 + 5.0 * torch.rand(R, D, 1, generator=g))


@pytest.mark.parametrize("V,R,B,K,kind,dtype,T", [
    (1000, 1, 16, 4, "mixed", "f32", 1.0),
    (4095, 2, 24, 8, "mixed", "bf16", 0.7),
    (4096, 2, 24, 32, "flat", "bf16", 1.0),
    (4100, 2, 24, 8, "peaked", "bf16", 1.0),
    (16380, 4, 64, 16, "flat", "bf16", 1.0),
    (16384, 4, 64, 32, "flat", "bf16", 1.3),
    (16385, 4, 64, 16, "mixed", "bf16", 1.0),
    (20004, 4, 64, 32, "flat", "f32", 1.0),
    (20001, 4, 64, 10, "mixed", "f32", 0.6),
    (40008, 4, 64, 12, "peaked", "bf16", 0.8),
    (40008, 4, 64, 12, "masked", "bf16", 1.0),
    (40008, 1, 64, 12, "flat", "bf16", 1.0),
    (131072, 1, 64, 32, "flat", "bf16", 1.0),
    (262144, 1, 255, 24, "flat", "bf16", 1.0),
    (262208, 1, 64, 8, "mixed", "bf16", 1.0),
    (270336, 1, 255, 16, "flat", "bf16", 1.0),
    (528388, 1, 64, 8, "flat", "bf16", 1.0),
])
def test_scan_edges(V, R, B, K, kind, dtype, T):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    D, seed, step = 3, 77, 9
    g = torch.Generator().manual_seed(V + K)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    draft = _rows(kind, R, D, V, g).to(dt)
    dev = draft.cuda()
    got = []
    for flags in (0, tsb.FLAG_NO_PRUNE):
        rnd = tsb.Round(tsb.make_config(R, D, V, B, K, T, dtype, seed, flags), "cuda")
        rnd.plan(dev)
        rnd.replay(dev, step)
        got.append(rnd.host())
    h = got[0]
    assert torch.equal(h["node_tok"], got[1]["node_tok"])
    tiles = -(-V // 4096)
    if 25 <= tiles <= 64:
        # unpruned, a tile of a flat row fills its parent's slots: more keys than the merge ranks at once (768)
        assert int(h["n_children"].max()) * tiles > 768
    a = (draft.float() * (torch.tensor(1.0) / torch.tensor(T))).double().numpy()
    checked = 0
    for r in range(R):
        for u in range(int(h["n_nodes"][r])):
            m = int(h["n_children"][r, u])
            if m == 0:
                continue
            toks, margin = oreplay.replay_node(a[r, int(h["depth"][r, u])], m, seed, step, r, u)
            if margin < 1e-5:
                continue
            fc = int(h["first_child"][r, u])
            assert np.array_equal(h["node_tok"][r, fc:fc + m].numpy(), toks), (r, u, m)
            checked += 1
    assert checked > 0


@pytest.mark.parametrize("K,bad", [(32, False), (6, False), (6, True)])
def test_unpruned_rows_are_scored_whole(K, bad):
    """Without pruning (by the flag, or for a parent whose candidates repeat) every group of four tokens of the
    scanned rows draws its words and has its keys evaluated, whatever was kept before it."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    R, D, V, B = 2, 3, 20000, 40
    dev = _rows("flat", R, D, V, torch.Generator().manual_seed(K)).to(torch.bfloat16).cuda()
    rnd = tsb.Round(tsb.make_config(R, D, V, B, K, 1.0, "bf16", 5, 0 if bad else tsb.FLAG_NO_PRUNE), "cuda")
    rnd.plan(dev)
    if bad:
        rnd.topk_tok[:, :, 1] = rnd.topk_tok[:, :, 0]
    tsb.stats_enable(True)
    try:
        tsb.stats_read()
        rnd.replay(dev, 3)
        s = tsb.stats_read()
    finally:
        tsb.stats_enable(False)
    parents = int((rnd.host()["n_children"] > 0).sum())
    assert s["replay_tokens"] == parents * V
    assert s["replay_groups_live"] == s["replay_groups_keyed"] == parents * V // 4


@pytest.mark.parametrize("R,B", [(64, 1023), (65, 1023), (192, 700)])
def test_parent_list_of_many_nodes(R, B):
    """Batches whose parent list is one chunk of nodes to a workgroup (the most of them), and several: every parent
    is listed once, and requests from both ends and the middle get the oracle's children."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    D, V, K, seed, step = 4, 64, 12, 6, 2
    draft = (2.0 * torch.randn(R, D, V, generator=torch.Generator().manual_seed(R))).cuda()
    rnd = tsb.Round(tsb.make_config(R, D, V, B, K, 1.0, "f32", seed), "cuda")
    rnd.plan(draft)
    tsb.stats_enable(True)
    try:
        tsb.stats_read()
        rnd.replay(draft, step)
        items = tsb.stats_read()["replay_items"]
    finally:
        tsb.stats_enable(False)
    h = rnd.host()
    assert items == int((h["n_children"] > 0).sum())
    a = draft.cpu().double().numpy()
    for r in (0, R // 3, R // 2, R - 1):
        n = int(h["n_nodes"][r])
        assert (h["node_tok"][r, 1:n] >= 0).all()
        for u in range(n):
            m, fc = int(h["n_children"][r, u]), int(h["first_child"][r, u])
            if m == 0:
                continue
            toks, margin = oreplay.replay_node(a[r, int(h["depth"][r, u])], m, seed, step, r, u)
            assert margin < 1e-5 or np.array_equal(h["node_tok"][r, fc:fc + m].numpy(), toks), (r, u, m)
