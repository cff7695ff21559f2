"""The planner where its threshold search, its list of nodes and the replay's
parent list can go wrong: budgets around a wave's and the workgroup's width and
the largest one, rows whose candidates need one, two and more registers to
merge, scores past the widest histogram (no first guess), more tied nodes than
a counting buffer holds, trees short of their budget, and batches whose nodes
take one and several workgroups of the parent list. For expand-then-prune:
layers narrower than the frontier, of the largest size whose places the whole
workgroup counts, and past it, with and without ties.

Topology, scores and margin must equal the oracle's planner on the same
log-probabilities, bit for bit; the replay must give every listed parent's
children a token.
"""
import numpy as np
import pytest
import torch

import paper_2609_33652_amd as tsb
from oracle import planner as oplan
from oracle import planner_ep as oplan_ep

pytestmark = pytest.mark.gpu


def _draft(kind, R, D, V, g):
    x = torch.randn(R, D, V, generator=g)
    if kind == "flat":  # every candidate of a row ties
        return torch.zeros(R, D, V)
    if kind == "steps":  # a few distinct scores: ties within and across depths
        return torch.randint(0, 3, (R, D, V), generator=g).float()
    if kind == "sharp":  # one token a row takes all: the others score below -100
        x[:, :, V // 3] += 150.0
        return x
    if kind == "short":  # two finite candidates a row
        x[:, :, 2:] = float("-inf")
        return x
    return x * (1.0 + 4.0 * torch.rand(R, D, 1, generator=g))


@pytest.mark.parametrize("V,R,D,B,K,kind,dtype", [
    (64, 3, 6, 0, 4, "mixed", "f32"),
    (1000, 3, 8, 63, 4, "mixed", "f32"),
    (1000, 2, 8, 64, 7, "mixed", "bf16"),
    (1000, 2, 33, 257, 32, "mixed", "bf16"),
    (600, 2, 12, 818, 16, "mixed", "f32"),
    (600, 2, 64, 1023, 32, "mixed", "f32"),
    (600, 2, 64, 1023, 32, "flat", "f32"),
    (600, 2, 5, 130, 11, "flat", "bf16"),
    (600, 3, 9, 200, 5, "steps", "bf16"),
    (600, 2, 16, 300, 6, "sharp", "f32"),
    (600, 2, 16, 40, 1, "mixed", "f32"),
    (600, 2, 4, 100, 6, "short", "f32"),
    (40000, 1, 4, 60, 32, "mixed", "bf16"),
    (151936, 1, 4, 60, 16, "mixed", "bf16"),
    (300, 17, 6, 128, 8, "mixed", "bf16"),
    (300, 64, 6, 129, 8, "mixed", "bf16"),
])
def test_plan_and_parent_list(V, R, D, B, K, kind, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator().manual_seed(V + 7 * B + K)
    draft = _draft(kind, R, D, V, g).to(torch.bfloat16 if dtype == "bf16" else torch.float32).cuda()
    rnd = tsb.Round(tsb.make_config(R, D, V, B, K, 1.0, dtype, 3), "cuda")
    rnd.plan(draft)
    rnd.replay(draft, 2)
    h = rnd.host()
    for r in range(R):
        ref = oplan.plan(h["topk_lp"][r].numpy(), B)
        n = ref["n_nodes"]
        assert int(h["n_nodes"][r]) == n
        for k in ("parent", "depth", "rank", "n_children", "first_child", "score"):
            assert np.array_equal(h[k][r, :n].numpy(), ref[k]), (r, k)
        assert float(h["plan_margin"][r]) == ref["plan_margin"]
        assert (h["parent"][r, n:] == -1).all() and (h["n_children"][r, n:] == 0).all()
        # every node but the root is some parent's child and got a token
        assert ((h["node_tok"][r, 1:n] >= 0) & (h["node_tok"][r, 1:n] < V)).all()
    if kind == "mixed" and B:
        # siblings hold distinct tokens
        for r in range(R):
            for u in range(int(h["n_nodes"][r])):
                m, f = int(h["n_children"][r, u]), int(h["first_child"][r, u])
                if m:
                    assert len(set(h["node_tok"][r, f:f + m].tolist())) == m


@pytest.mark.parametrize("D,B,K,W,kind", [
    (6, 40, 4, 4, "mixed"),
    (5, 100, 8, 8, "steps"),
    (6, 300, 16, 16, "mixed"),
    (6, 300, 16, 16, "flat"),
    (5, 300, 20, 13, "mixed"),
    (5, 300, 20, 13, "steps"),
    (9, 100, 6, 10, "short"),
])
def test_expand_prune_layers(D, B, K, W, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    R, V = 2, 600
    g = torch.Generator().manual_seed(B + K)
    draft = _draft(kind, R, D, V, g).cuda()
    rnd = tsb.Round(tsb.make_config(R, D, V, B, K, 1.0, "f32", 3), "cuda")
    rnd.plan_ep(draft, W)
    h = rnd.host()
    for r in range(R):
        ref = oplan_ep.plan_expand_prune(h["topk_lp"][r].numpy(), B, W)
        n = ref["n_nodes"]
        assert int(h["n_nodes"][r]) == n
        for k in ("parent", "depth", "rank", "n_children", "first_child", "score"):
            assert np.array_equal(h[k][r, :n].numpy(), ref[k]), (r, k)
        assert float(h["plan_margin"][r]) == ref["plan_margin"]
