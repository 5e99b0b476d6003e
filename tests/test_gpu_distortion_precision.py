"""Precision of the child keys in the refinement (bf16 caches).  With equal keys
everywhere and rotations switched off, a child's key is its tokens' key exactly (a
sum of at most 128 equal bf16 numbers is exact), so its logits are theirs bit for
bit, whatever their size, and with the value term off (lam_M = 0) the distortion
D = (Z / Z(C)) ((Z - z) / Z)^2 shows nothing but the rounding of Z, of m_eff and of
the mean: a mean off by one part in 2^24 would move z by that times the logit."""
import math

import pytest
import torch

from paper_2608_07001_amd import gracekv as gk

pytestmark = pytest.mark.gpu


def _lengths(total):
    lens, a = [], 0
    while a < total:
        for n in (128, 97, 85, 63, 61, 47, 33, 31, 27, 23, 19, 17, 16, 15, 13, 11, 7, 6, 5, 3):
            n = min(n, total - a)
            if n > 0:
                lens.append(n)
                a += n
    return lens


@pytest.mark.parametrize("d,W,top", [(128, 64, 300.0), (64, 33, 200.0)])
def test_logits_of_equal_keys(d, W, top):
    dev = "cuda"
    gen = torch.Generator(device=dev).manual_seed(d)
    L, G, H, N = 1, 2, 4, 1600
    cfg = gk.config_for(L=L, G=G, H=H, d=d, W=W, N_ctx=N, x=2.0, dtype=gk.BF16, n_seg=1, D_hidden=64, lam_Z=1.0, lam_M=0.0)
    buf = gk.allocate(cfg)
    p, T = buf.plan, N + W
    key = torch.randn(d, generator=gen, device=dev).bfloat16()
    K = key.expand(L, G, T, d).contiguous()
    V = torch.randn(L, G, T, d, generator=gen, device=dev).bfloat16()
    size = torch.linspace(top / 10, top, H * W, device=dev).view(L, H, W, 1)
    Q = (key.float() * size * math.sqrt(d) / key.float().pow(2).sum()).bfloat16()
    cos, sin = torch.ones(T, d // 2, device=dev), torch.zeros(T, d // 2, device=dev)
    lens = _lengths(p.N_c)
    starts = torch.tensor([0] + lens, device=dev).cumsum(0).int()
    slots = torch.full((p.J_cap + 1,), p.N_c, dtype=torch.int32, device=dev)
    slots[:len(lens)] = starts[:-1]
    n_slots = torch.tensor([len(lens)], dtype=torch.int32, device=dev)
    kappa = torch.rand(T, generator=gen, device=dev)
    buf.trees.zero_()
    gk.build_trees(cfg, K, V, Q, cos, sin, slots, n_slots, kappa, buf.trees)
    gk.check(cfg, buf.trees)
    arr = gk.tree_arrays(p, buf.trees)
    long, short = [], []
    for lg in range(L * G):
        for j, n0 in enumerate(lens):
            base = lg * 2 * p.N_c + 2 * int(starts[j])
            for i in range(1, int(arr["unit_nn"][lg * p.J_cap + j])):
                n, D = int(arr["node_n"][base + i]), float(arr["node_D"][base + i])
                if n > 1:
                    (long if n > 16 else short).append(math.sqrt(D * p.N_c / n))
    print(f"d {d}: (Z - z) / Z rms up to {max(long):.2e} above 16 tokens ({len(long)} nodes), "
          f"{max(short):.2e} below ({len(short)})", flush=True)
    # Z: at most 16 additions inside a tile and 8 of tiles; m_eff: a norm, a mean, a
    # quotient and its square, under ten roundings: 34 x 2^-24 at worst
    assert max(long) < 34 / 2 ** 24
    # a reciprocal to the nearest float moves some channels of the mean by one unit in
    # the last place: 2^-24 of the logit on top
    assert max(short) < (34 + top * 1.45) / 2 ** 24
