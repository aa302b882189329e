"""The kernels on the fp32 matrix instructions (absorb, decode, merge + up-projection of every shape outside the bf16
fast paths) at the edges of their tiles, against the fp64 oracle.  Bars as for the other parity tests:
max|gpu - ref| / max|ref| <= 1e-5 (fp32 storage) and 1e-2 (bf16 storage)."""
import math

import numpy as np
import pytest
import torch

from oracle import mlra_oracle as orc
from paper_2603_02188_amd import binding as mlra
from paper_2603_02188_amd import inputs as gen

from gpu_util import device_cache, device_queries_weights, host, max_rel_err, oracle_views, to_device

pytestmark = pytest.mark.gpu

TOL = {"bf16": 1e-2, "f32": 1e-5}


def _shifted(t):
    """The same values one element past an aligned address."""
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    buf[1:] = t.reshape(-1)
    return buf[1:].view(t.shape)


def _lse_reference(v, q_abs, q_rope, groups, scale):
    """Log-sum-exp [B][NB][h / groups] in 64 bits from the absorbed queries as they are stored (so that their rounding, which
    grows with the score, stays out of it)."""
    batch, nb, hb, d_cb = q_abs.shape
    lse = np.full((batch, nb, hb), -np.inf)
    for s in range(batch):
        n = int(v["seq_lens"][s])
        c, kr = orc.gather_sequence(v["latent_pool"], v["rope_pool"], v["page_table"][s], n)
        for b in range(nb if n else 0):
            first = b // (nb // groups) * hb
            x = scale * (c[:, b * d_cb:(b + 1) * d_cb] @ q_abs[s, b].T + kr @ q_rope[s, first:first + hb].T)
            lse[s, b] = x.max(axis=0) + np.log(np.exp(x - x.max(axis=0)).sum(axis=0))
    return lse


def _run(wl, lens, shift=False, folded=False, out_dtype=torch.float32, gated=False):
    print(f"[case] {wl.name} B={wl.batch} NB={wl.n_blocks} d_cb={wl.d_cb} d_r={wl.d_r} h={wl.h} d_h={wl.d_h} "
          f"{wl.dtype} page={wl.page_size} groups={wl.groups} shift={shift} folded={folded} lens={list(lens)}", flush=True)
    inp = gen.make_decode_inputs(wl, poison=True, seq_lens=np.array(lens, dtype=np.int32))
    cache = device_cache(inp)
    tensors = device_queries_weights(inp)
    if shift:
        cache = mlra.Cache(_shifted(cache.latent), _shifted(cache.rope), cache.page_table, cache.seq_lens)
        tensors = [_shifted(t) for t in tensors]
    q_nope, q_rope, w_uk, w_uv = tensors
    two, scale = wl.groups == 2, wl.tau
    if folded:
        q_abs, q_rope = (mlra.mlra2_absorb_q_folded if two else mlra.mlra_absorb_q_folded)(q_nope, w_uk, q_rope, wl.tau)
        scale = mlra.SCALE_FOLDED
    else:
        q_abs = (mlra.mlra2_absorb_q if two else mlra.mlra_absorb_q)(q_nope, w_uk)
    lse = torch.full((wl.batch, wl.n_blocks, wl.h // wl.groups), float("nan"), device="cuda")
    kw = dict(out_dtype=out_dtype, lse=lse)
    if gated:
        gate = gen.to_storage(np.random.default_rng(7).uniform(0.0, 1.0, size=(wl.batch, wl.h, wl.d_h)).astype(np.float32), wl.dtype)
        gate_dev = to_device(gate, "bf16" if wl.dtype == "bf16" else None)
        out = mlra.mlra_decode_attn_gated(cache, q_abs, q_rope, w_uv, gate_dev, scale, 0.5, **kw)
    else:
        out = (mlra.mlra2_decode_attn if two else mlra.mlra_decode_attn)(cache, q_abs, q_rope, w_uv, scale, 0.5, **kw)
    torch.cuda.synchronize()
    v = oracle_views(inp)
    args = (v["latent_pool"], v["rope_pool"], v["page_table"], v["seq_lens"], v["q_nope"], v["q_rope"], v["w_uk"],
            v["w_uv"], wl.tau)
    ref = (orc.mlra2_decode_batch if two else orc.mlra_decode_batch)(*args, 0.5)
    if gated:
        ref = ref * gen.to_f64(gate, wl.dtype)
    err = max_rel_err(host(out), ref)
    print(f"       max rel err {err:.3e}", flush=True)
    assert err <= (1e-2 if out_dtype == torch.bfloat16 else TOL[wl.dtype])
    ref_lse = _lse_reference(v, host(q_abs), host(q_rope), wl.groups, math.log(2.0) if folded else wl.tau)
    got, live = host(lse), np.isfinite(ref_lse)
    assert np.array_equal(np.isneginf(got), ~live) and np.array_equal(np.isfinite(got), live)
    # fp32 scores of size 10 and sums of hundreds: 1e-5 of either.  The bf16 kernels round the scaled queries and the
    # probabilities to bf16: 2^-9 of a score of up to 8 and 2^-9 of the sum
    info = mlra.mlra_decode_plan_info(wl.batch, wl.h, wl.d_h, wl.groups, wl.n_blocks, wl.d_cb, wl.d_r, wl.page_size,
                                      cache.max_seq_len, q_abs.dtype)
    assert (info["kernel"] == "generic") == (wl.d_cb > 256)
    tol = 2e-2 if info["kernel"].startswith("mfma") else 1e-4
    lse_err = float(np.max(np.abs(got[live] - ref_lse[live])))
    print(f"       lse {lse_err:.3e}", flush=True)
    assert lse_err <= tol


def _wl(**kw):
    return gen.WORKLOADS["C1"].scaled(**{**dict(name="f32-kernels", shuffle_pages=True, spare_frac=0.2), **kw})


LENS = [0, 1, 63, 64, 65, 129, 300, 511]


# heads: one tile, its edges, 2 and 4 tiles per workgroup and a remainder; dims: the edges of each register size (32, 96 / 64,
# 192 / 128, 320 / 256 channels), beyond the last one (the plain kernel), odd ones (element loads), one channel
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("h,d_cb,d_r,d_h,nb", [
    (1, 64, 32, 64, 1), (16, 64, 32, 65, 2), (17, 60, 36, 24, 2), (33, 61, 3, 63, 1), (8, 65, 32, 64, 2),
    (64, 128, 64, 128, 1), (65, 96, 32, 128, 1), (20, 127, 65, 66, 1), (130, 68, 24, 40, 2), (33, 129, 64, 64, 1),
    (64, 256, 64, 64, 1), (17, 253, 67, 30, 1), (5, 260, 64, 64, 1), (5, 16, 16, 20, 3),
    (17, 30, 2, 24, 2), (64, 24, 8, 32, 2), (33, 31, 1, 16, 2), (40, 17, 16, 30, 2), (3, 1, 2, 6, 80), (6, 7, 2, 130, 90)])
def test_dims_and_heads(dtype, h, d_cb, d_r, d_h, nb):
    _run(_wl(batch=len(LENS), n_min=0, n_max=511, h=h, d_cb=d_cb, d_r=d_r, d_h=d_h, n_blocks=nb, dtype=dtype), LENS)


# batches around the 16 sequences of an MFMA tile; enough chunks that a piece's chunks are shared by several threads
@pytest.mark.parametrize("batch,n,page", [(1, 9000, 64), (2, 3001, 48), (15, 130, 16), (16, 64, 64), (17, 200, 64), (33, 70, 32)])
def test_batches_and_chunks(batch, n, page):
    rng = np.random.default_rng(batch)
    lens = rng.integers(1, n + 1, size=batch)
    lens[0] = n
    for folded in (False, True):
        _run(_wl(batch=batch, n_min=1, n_max=n, page_size=page, h=12), lens.tolist(), folded=folded)
    _run(_wl(batch=batch, n_min=1, n_max=n, page_size=page, h=12, dtype="bf16"), lens.tolist(), out_dtype=torch.bfloat16)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("h,d_cb,d_r,d_h", [(8, 64, 32, 64), (40, 128, 64, 128), (16, 256, 64, 64)])
def test_bases_that_are_not_aligned_for_wide_loads(dtype, h, d_cb, d_r, d_h):
    _run(_wl(batch=3, n_min=1, n_max=400, h=h, d_cb=d_cb, d_r=d_r, d_h=d_h, n_blocks=2, dtype=dtype), [400, 1, 77],
         shift=True, folded=True)


# merge: heads of up to 128 channels (small slab) and more, blocks that straddle the slabs' ends (96 and 36 channels over
# 512), more blocks than a slab's table has, up to four chunk slots (a thread per pair) and from five on (lane groups: 16
# chunks and more), chunk parts of rows that are not made of runs of four; gate and log-sum-exp of all of them
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("batch,n,h,d_cb,d_r,d_h,nb", [
    (3, 500, 3, 32, 16, 24, 4), (3, 500, 3, 33, 16, 70, 4), (17, 130, 2, 16, 16, 16, 8), (2, 700, 4, 96, 32, 40, 7),
    (2, 300, 2, 36, 4, 20, 30), (1, 9000, 2, 61, 3, 64, 2), (3, 5000, 2, 9, 7, 16, 1), (2, 2500, 2, 4, 2, 8, 70),
    (1, 2300, 5, 30, 2, 128, 20)])
def test_merge_slabs_and_slots(dtype, batch, n, h, d_cb, d_r, d_h, nb):
    lens = np.random.default_rng(d_cb).integers(0, n + 1, size=batch)
    lens[0] = n
    for gated in (False, True):
        _run(_wl(batch=batch, n_min=0, n_max=n, h=h, d_cb=d_cb, d_r=d_r, d_h=d_h, n_blocks=nb, dtype=dtype), lens.tolist(),
             gated=gated)


def test_head_groups():
    _run(_wl(batch=3, n_min=1, n_max=600, h=36, groups=2), [600, 1, 65])
    _run(_wl(batch=3, n_min=1, n_max=600, h=36, groups=2, dtype="bf16"), [600, 0, 65], folded=True)


def test_more_workgroups_than_one_grid_dimension_holds():
    """65535 sequences x 257 blocks are more than 2^32 / 256 workgroups, the most that one dimension of a launch holds."""
    batch, nb, pages = 65535, 257, 64
    print(f"[case] f32 grid B={batch} NB={nb}", flush=True)
    gen_ = torch.Generator(device="cuda").manual_seed(5)
    latent = torch.randn((pages, nb, 1, 1), generator=gen_, device="cuda")
    table = (torch.arange(batch, device="cuda") % pages).to(torch.int32).view(batch, 1)
    cache = mlra.Cache(latent, torch.randn((pages, 1, 1), generator=gen_, device="cuda"), table,
                       torch.ones(batch, dtype=torch.int32, device="cuda"))
    w_uv = torch.randn((nb, 1, 1), generator=gen_, device="cuda")
    q_abs = torch.randn((batch, nb, 1, 1), generator=gen_, device="cuda")
    out = mlra.mlra_decode_attn(cache, q_abs, torch.randn((batch, 1, 1), generator=gen_, device="cuda"), w_uv, 0.5)
    torch.cuda.synchronize()
    # one token: its weight is 1 and the output is the sum of the blocks' channels times their weights
    ref = (latent.double().view(pages, nb) @ w_uv.double().view(nb, 1))[table.long().view(-1)].view(batch, 1, 1)
    assert max_rel_err(host(out), host(ref)) <= 1e-5
