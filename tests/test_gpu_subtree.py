"""Refinement below the roots (bf16 caches) at the sizes where its two kernels
meet and end: slots of 1 to 20 tokens among long ones, so nodes just above and
just below the longest subtree that one wave takes (16 tokens), subtrees of 2
and 3 tokens, one and more probe tiles, fewer candidate cuts than positions.
Trees, gains, selection and pack match the oracle, every tree is numbered
breadth-first, and the pruned build gives the complete build's result."""
import pytest
import torch

from oracle import gracekv_oracle as O
from synth.workloads import make_case, make_kappa, small_shape

import gpu_harness as H

pytestmark = pytest.mark.gpu


def _partition(N):
    lens = [n for i in range(1, 21) for n in (i, 40 if i % 2 else 33)]
    starts, a, k = [], 0, 0
    while a < N:
        starts.append(a)
        a += lens[k % len(lens)]
        k += 1
    return starts


@pytest.mark.parametrize("d,hpg,W,k_curv,x", [(128, 4, 64, 16, 8.0), (128, 1, 1, 16, 3.0), (64, 2, 17, 16, 6.0),
                                              (128, 2, 48, 5, 8.0), (64, 8, 16, 0, 4.0), (128, 3, 33, 14, 24.0)])
def test_nodes_around_the_subtree_limit(d, hpg, W, k_curv, x):
    sh = small_shape(f"subtree-{d}-{W}-{k_curv}", L=1, G=2, H=2 * hpg, d=d, N_ctx=1131, W=W, dtype="bf16", x=x,
                     n_segments=9, rope_base=5.0e5, channel_scale="outlier")
    case = make_case(sh, 5, with_hidden=False)
    kappa = make_kappa(sh, 5)
    slots = _partition(O.budget(sh.L, sh.G, sh.N_ctx, sh.x).N_c)
    cd = H.to_dev(case)
    g = H.gpu_run(cd, slots=slots, kappa=kappa, k_curv=k_curv)
    H.parity(case, g, sh.name, slots=slots, kappa=kappa, p=O.Params(k_curv=k_curv))
    assert not H.validate_gpu_trees(g)
    pr = H.gpu_run(cd, slots=slots, kappa=kappa, k_curv=k_curv, prune=True)
    assert H.gpu_selected(g) == H.gpu_selected(pr)
    assert g["b_used"] == pr["b_used"] and torch.equal(g["offsets"], pr["offsets"])
    n = int(g["offsets"][-1])
    for k in ("pos_out", "logm_out", "K_out", "V_out"):
        assert torch.equal(g[k][:n], pr[k][:n]), k


# contexts that leave a few tokens to compress: lists of one entry, whose arrays are all rounding
@pytest.mark.parametrize("N_ctx,L,G", [(33, 1, 1), (34, 1, 1), (36, 2, 1), (40, 1, 1), (41, 1, 1), (36, 3, 1), (35, 2, 2),
                                       (49, 1, 1), (50, 1, 2)])
def test_contexts_of_a_few_tokens(N_ctx, L, G):
    sh = small_shape(f"few-{N_ctx}-{L}-{G}", L=L, G=G, H=2 * G, d=64, N_ctx=N_ctx, W=4, dtype="bf16", x=1.0,
                     n_segments=1, rope_base=5.0e5)
    case = make_case(sh, 7, with_hidden=False)
    kappa = make_kappa(sh, 7)
    N_c = O.budget(L, G, N_ctx, 1.0).N_c
    slots = [0] if N_c < 12 else [0, 5]
    cd = H.to_dev(case)
    for prune in (False, True):
        g = H.gpu_run(cd, slots=slots, kappa=kappa, prune=prune)
        if not prune:
            H.parity(case, g, sh.name, slots=slots, kappa=kappa)
        assert not H.validate_gpu_trees(g)
        assert int(g["offsets"][-1]) == L * G * N_ctx
        # all of the budget is spent on singletons: the cache itself
        assert torch.equal(g["K_out"].view(L, G, N_ctx, 64), case["K"][:, :, :N_ctx])
        assert torch.equal(g["V_out"].view(L, G, N_ctx, 64), case["V"][:, :, :N_ctx])
