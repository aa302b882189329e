"""Rounding error of the fp32 query absorption.  A sum of n products whose partial sums are added as a tree carries a
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
