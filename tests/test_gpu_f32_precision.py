"""Rounding error of the fp32 kernels: the query absorption and, below, the smallest probabilities of the decode kernel.  A sum of n products whose partial sums are added as a tree carries a
rounding error of sqrt(1.5 + log2(n)) or so roundings of the result, one chain of n additions sqrt(n / 2); a rounding of
an fp32 value is 2.5e-8 of it (root mean square over the mantissas).  The bars are 1.25 times what runs of at most four
products, a tree over 128 of them and a chain over the 128s give: sqrt(1.5 + log2(128) + n / 256) roundings."""
import math

import pytest
import torch

from paper_2603_02188_amd import binding as mlra

pytestmark = pytest.mark.gpu


# depths: one step of each form (32, 64, 128), several steps, a remainder, rows that are not made of runs of four; blocks
# of one and two channel tiles, whose rows the waves share
@pytest.mark.parametrize("batch,h,d_h,nb,d_cb", [(16, 16, 32, 2, 64), (16, 16, 64, 4, 64), (8, 32, 128, 4, 128),
                                                 (17, 12, 200, 2, 100), (5, 8, 1024, 2, 24), (9, 8, 127, 2, 61),
                                                 (40, 8, 128, 2, 16), (33, 8, 200, 2, 17), (18, 8, 258, 2, 31)])
def test_absorb_adds_as_a_tree(batch, h, d_h, nb, d_cb):
    print(f"[case] absorb precision B={batch} h={h} d_h={d_h} NB={nb} d_cb={d_cb}", flush=True)
    gen = torch.Generator().manual_seed(d_h)
    q = torch.randn((batch, h, d_h), generator=gen)
    w = torch.randn((nb, d_cb, h * d_h), generator=gen)
    got = mlra.mlra_absorb_q(q.cuda(), w.cuda()).cpu().double()
    ref = (w.double().view(nb, 1, d_cb, h, d_h) * q.double().view(1, batch, 1, h, d_h)).sum(-1).permute(1, 0, 3, 2)
    err = float((got - ref).norm() / ref.norm())
    bar = 1.25 * 2.5e-8 * math.sqrt(1.5 + math.log2(min(d_h, 128)) + d_h / 256)
    print(f"       error {err:.3e}, bar {bar:.3e}", flush=True)
    assert err <= bar


# A weight of 2^-130 of the largest one is a denormal number, and a value of 2^120 makes it count: scores in the log2 domain
# of 0 and -130 (exact: products of small integers), latents of 0 and 2^120, so that a sequence's merged value is 2^-10 times
# the number of such tokens over the number of the others.  The light tokens come first (the history loses its weight), last,
# in a chunk of their own or in one tile with the heavy ones.
@pytest.mark.parametrize("n_light,n_heavy,light_first", [(1, 1, False), (3, 1, True), (64, 64, True), (64, 64, False),
                                                         (200, 130, True), (100, 300, False)])
def test_decode_keeps_denormal_weights(n_light, n_heavy, light_first):
    print(f"[case] denormal weights light={n_light} heavy={n_heavy} first={light_first}", flush=True)
    n, h, d_cb, d_r, d_h, page = n_light + n_heavy, 18, 32, 4, 32, 64
    pages = -(-n // page)
    light = torch.zeros(pages * page, dtype=torch.bool)
    light[:n_light] = True
    if not light_first:
        light[:n] = light[:n].flip(0)
    latent = torch.where(light[:, None], 2.0 ** 120, 0.0).expand(-1, d_cb).reshape(pages, 1, page, d_cb).contiguous()
    rope = torch.zeros(pages * page, d_r)
    rope[light, 0] = -130.0
    q_abs, q_rope = torch.zeros(1, 1, h, d_cb), torch.ones(1, h, d_r)
    w_uv = torch.eye(d_cb, d_h).repeat(1, h).view(1, d_cb, h * d_h)
    cache = mlra.Cache(latent.cuda(), rope.view(pages, page, d_r).cuda(), torch.arange(pages, dtype=torch.int32).view(1, -1).cuda(),
                       torch.tensor([n], dtype=torch.int32).cuda())
    out = mlra.mlra_decode_attn(cache, q_abs.cuda(), q_rope.cuda(), w_uv.cuda(), mlra.SCALE_FOLDED, out_dtype=torch.float32)
    ref = 2.0 ** -10 * n_light / n_heavy
    # (powers of two and their sums are exact; the division by the sum of the weights rounds)
    assert float((out.cpu().double() / ref - 1.0).abs().max()) <= 1e-6
