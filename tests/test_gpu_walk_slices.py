"""The walks where a request's vocabulary slices change shape: one workgroup
(no exchange) and the first vocabulary of several, slices of one, two, three
and five groups a thread, a last slice that is short, odd vocabularies (no
vector loads), slices that leave a compute unit to one workgroup, the longest
held ones, and vocabularies whose slices are recomputed in every pass. Small
and equal draft and target rows make some walks accept and others reject every
child, so both bonus draws and the residual passes run.

A whole round and the staged calls must agree bit for bit, and both with the
oracle's round: path, bonus and status, unless one of its decisions has a
margin below 1e-5 (the repository's near-tie rule).
"""
import numpy as np
import pytest
import torch

import paper_2609_33652_amd as tsb
from oracle import step as ostep

pytestmark = pytest.mark.gpu

SMALL = [(5, 2), (1024, 2), (4096, 2), (4097, 2), (8188, 3), (9601, 2), (32000, 2), (65537, 2), (131070, 1)]
WIDE = [(524288, 1), (614403, 1), (1212416, 1), (1212420, 1), (1212416 + 4096, 1)]


def _round(V, R, dtype, verifier, flags, mix):
    D, B, K, T, seed, step = 3, 7, 3, 1.0, 11, 4
    g = torch.Generator().manual_seed(V + 31 * mix)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    base = 2.0 * torch.randn(R, D + 1, V, generator=g)
    draft = base[:, :D].to(dt)
    cfg = tsb.make_config(R, D, V, B, K, T, dtype, seed, flags)
    whole, staged = tsb.Round(cfg, "cuda", trace=True), tsb.Round(cfg, "cuda", trace=True)
    dev = draft.cuda()
    whole.plan(dev)
    depth = whole.tree["depth"].long().clamp(min=0).cpu()
    # mix 0: the target is near the draft (most tests accept); 1: far from it
    noise = 0.3 if mix == 0 else 3.0
    target = torch.stack([base[r, depth[r]] for r in range(R)]) + noise * torch.randn(R, B + 1, V, generator=g)
    target = target.to(dt)
    tdev = target.cuda()
    if verifier == "rrs":
        whole.step(dev, tdev, step)
    else:
        whole.step_traversal(dev, tdev, step)
    staged.plan(dev)
    staged.replay(dev, step)
    (staged.verify if verifier == "rrs" else staged.verify_traversal)(dev, tdev, step)
    a, b = whole.host(), staged.host()
    for k in ("node_tok", "n_acc", "acc_node", "acc_tok", "bonus", "req_status", "trace"):
        assert torch.equal(a[k], b[k]), k
    d_np, t_np = draft.float().numpy(), target.float().numpy()
    for r in range(R):
        ref = ostep.step_request(d_np[r], t_np[r], T, K, B, seed, step, r, verifier=verifier)
        assert int(a["req_status"][r]) == ref["status"]
        if ostep.near_ties(ref["margins"]):
            continue
        n = int(a["n_acc"][r])
        assert n == ref["n_acc"], (r, n)
        assert list(a["acc_node"][r, :n].numpy()) == [int(x) for x in ref["acc_node"]]
        assert list(a["acc_tok"][r, :n].numpy()) == [int(x) for x in ref["acc_tok"]]
        assert int(a["bonus"][r]) == ref["bonus"], r


@pytest.mark.parametrize("verifier", ["rrs", "traversal"])
@pytest.mark.parametrize("mix", [0, 1])
@pytest.mark.parametrize("V,R", SMALL)
def test_slices(V, R, mix, verifier):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dtype = "f32" if V in (5, 1024, 8188, 65537) else "bf16"
    flags = tsb.FLAG_READ_ROWS if verifier == "rrs" and V % 2 == 0 else 0
    _round(V, R, dtype, verifier, flags, mix)


@pytest.mark.parametrize("verifier", ["rrs", "traversal"])
@pytest.mark.parametrize("V,R", WIDE)
def test_wide_slices(V, R, verifier):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    _round(V, R, "bf16", verifier, tsb.FLAG_READ_ROWS if verifier == "rrs" else 0, 1)
