"""Chunk lengths that the decode kernels fit to the sequence lengths themselves (batches of at most 64 sequences), and the
order they give the queries of several tokens per sequence: empty and full sequences, one long one among short ones, all
sizes of the last eight-chunk run, against the fp64 oracle; and against the general path, which the same sequences take when
empty ones bring the batch to 65.  Every case asserts from the call's route that its chunks are fitted, or are not."""
import numpy as np
import pytest
import torch

from oracle import mlra_oracle as orc
from paper_2603_02188_amd import binding as mlra
from paper_2603_02188_amd import inputs as gen

from gpu_util import device_cache, device_queries_weights, host, max_rel_err, oracle_views

pytestmark = pytest.mark.gpu

TOL = {"bf16": 1e-2, "f32": 1e-5}


def _ragged(batch, n_max, seed):
    lens = np.random.default_rng(seed).integers(0, n_max + 1, size=batch).astype(np.int32)
    lens[0] = n_max
    if batch > 2:
        lens[1], lens[-1] = 0, 1
    return lens


def _decode(wl, inp):
    q_nope, q_rope, w_uk, w_uv = device_queries_weights(inp)
    lse = torch.full((wl.batch, wl.n_blocks, wl.h), float("nan"), device="cuda")
    out = mlra.mlra_decode_attn(device_cache(inp), mlra.mlra_absorb_q(q_nope, w_uk), q_rope, w_uv, wl.tau, 0.5,
                                out_dtype=torch.float32, lse=lse)
    torch.cuda.synchronize()
    return host(out), host(lse)


def _fitted(wl, table, q_len=1):
    batch, width = table.shape
    return mlra.mlra_decode_route_info(batch, wl.h, wl.d_h, 1, wl.n_blocks, wl.d_cb, wl.d_r, wl.page_size, width * wl.page_size,
                                       torch.bfloat16 if wl.dtype == "bf16" else torch.float32, q_len)["fitted_from"] > 0


def _check(wl, lens, fitted=True, capacity=None):
    """capacity: the lengths that the page table is made for, where these are not the sequences'."""
    inp = gen.make_decode_inputs(wl, poison=True, seq_lens=lens if capacity is None else capacity)
    inp.seq_lens[:] = lens
    assert _fitted(wl, inp.page_table) == fitted
    out, lse = _decode(wl, inp)
    v = oracle_views(inp)
    ref, ref_lse = orc.mlra_decode_batch(v["latent_pool"], v["rope_pool"], v["page_table"], v["seq_lens"], v["q_nope"],
                                         v["q_rope"], v["w_uk"], v["w_uv"], wl.tau, 0.5, return_lse=True)
    live = np.isfinite(ref_lse)
    assert np.array_equal(np.isfinite(lse), live)
    assert max_rel_err(out, ref) <= TOL[wl.dtype]
    assert not live.any() or np.max(np.abs(lse[live] - ref_lse[live])) <= (2e-2 if wl.dtype == "bf16" else 1e-4)


# fitted: an odd head count, bf16 caches with either epilogue (128 and 64 channels per head), 64 sequences, wide blocks in
# several channel tiles.  Not fitted: chunks too short to pay for it, or no more of them than one round of workgroups.
@pytest.mark.parametrize("batch,n_max,h,d_cb,d_h,dtype,fitted", [
    (8, 2048, 128, 128, 64, "f32", True), (64, 900, 100, 64, 64, "f32", True), (33, 1300, 40, 200, 64, "f32", True),
    (3, 1100, 200, 200, 64, "f32", True), (50, 1200, 17, 64, 128, "bf16", True), (33, 1000, 65, 96, 64, "bf16", True),
    (2, 300, 17, 128, 64, "f32", False), (9, 700, 64, 64, 64, "f32", False), (33, 260, 16, 128, 64, "f32", False),
    (64, 200, 8, 32, 64, "f32", False), (5, 1200, 12, 64, 64, "bf16", False), (3, 600, 32, 200, 64, "f32", False)])
def test_fp32_kernel(batch, n_max, h, d_cb, d_h, dtype, fitted):
    wl = gen.WORKLOADS["C3"].scaled(name="fit-f32", batch=batch, n_min=0, n_max=n_max, h=h, d_h=d_h, d_cb=d_cb, d_r=32,
                                    n_blocks=2, dtype=dtype, index=4000 + batch)
    print(f"[case] fit f32 B={batch} n_max={n_max} h={h} d_cb={d_cb} {dtype}", flush=True)
    _check(wl, _ragged(batch, n_max, batch), fitted)


def test_fp32_kernel_without_tokens():
    wl = gen.WORKLOADS["C3"].scaled(name="fit-empty", batch=6, n_min=0, n_max=2048, h=128, d_h=64, d_cb=64, d_r=32, n_blocks=4,
                                    dtype="f32", index=4100)
    _check(wl, np.zeros(6, dtype=np.int32), capacity=np.full(6, 2048, dtype=np.int32))


@pytest.mark.parametrize("batch,n_max", [(6, 2048), (64, 900)])
def test_same_as_the_general_path(batch, n_max):
    wl = gen.WORKLOADS["C3"].scaled(name="fit-general", batch=65, n_min=0, n_max=n_max, h=128, d_h=64, d_cb=128, d_r=32,
                                    n_blocks=2, dtype="f32", index=4200)
    lens = np.zeros(65, dtype=np.int32)
    lens[:batch] = _ragged(batch, n_max, batch)
    inp = gen.make_decode_inputs(wl, poison=True, seq_lens=lens)
    assert _fitted(wl, inp.page_table[:batch]) and not _fitted(wl, inp.page_table)
    out, lse = _decode(wl, inp)
    q_nope, q_rope, w_uk, w_uv = device_queries_weights(inp)
    cache = device_cache(inp)
    few = mlra.Cache(cache.latent, cache.rope, cache.page_table[:batch].contiguous(), cache.seq_lens[:batch].contiguous())
    lse_few = torch.full((batch, wl.n_blocks, wl.h), float("nan"), device="cuda")
    out_few = mlra.mlra_decode_attn(few, mlra.mlra_absorb_q(q_nope[:batch].contiguous(), w_uk), q_rope[:batch].contiguous(), w_uv,
                                    wl.tau, 0.5, out_dtype=torch.float32, lse=lse_few)
    torch.cuda.synchronize()
    # the same products, chunks cut elsewhere: both within 1e-5 of the exact result
    assert max_rel_err(host(out_few), out[:batch]) <= 2e-5
    live = np.isfinite(lse[:batch])
    assert np.array_equal(np.isfinite(host(lse_few)), live)
    assert np.max(np.abs(host(lse_few)[live] - lse[:batch][live])) <= 2e-4


# the MLRA kernel on long contexts: two blocks per workgroup (16 heads) and one, chunks at their shortest, sequences of one
# chunk and none
@pytest.mark.parametrize("batch,h,n_max", [(16, 128, 24600), (33, 16, 25000)])
def test_mlra_kernel_long(batch, h, n_max):
    wl = gen.WORKLOADS["C3"].scaled(name="fit-long", batch=batch, n_min=0, n_max=n_max, h=h, index=4400 + batch)
    lens = np.resize(np.array([n_max, 0, 1, 63, 64, 65, 3100, 12300], dtype=np.int32), batch)
    lens[8:] = np.minimum(lens[8:], 100)
    info = mlra.mlra_decode_plan_info(batch, h, 128, 1, 4, 128, 64, 64, -(-n_max // 64) * 64, torch.bfloat16)
    print(f"[case] fit MLRA B={batch} h={h} {info}", flush=True)
    assert info["target_chunks"] > 0 and not info["single_if_uniform"]
    _check(wl, lens)


# the MLA kernel: more slots than CUs, one and two head groups
@pytest.mark.parametrize("batch,h,n_max", [(30, 128, 640), (63, 70, 700), (11, 16, 6000)])
def test_mla_kernel(batch, h, n_max):
    wl = gen.WORKLOADS["C5"].scaled(name="fit-mla", batch=batch, n_min=0, n_max=n_max, h=h, index=4500 + batch)
    info = mlra.mlra_decode_plan_info(batch, h, 128, 1, 1, 512, 64, 64, -(-n_max // 64) * 64, torch.bfloat16)
    print(f"[case] fit MLA B={batch} h={h} {info}", flush=True)
    assert info["kernel"] == "mfma-mla" and batch * info["chunk_slots"] * ((h + 63) // 64) > 256 and info["target_chunks"] == 0
    assert mlra.mlra_decode_route_info(batch, h, 128, 1, 1, 512, 64, 64, -(-n_max // 64) * 64, torch.bfloat16)["fitted_from"] > 0
    inp = gen.make_decode_inputs(wl, poison=True, seq_lens=_ragged(batch, n_max, batch))
    q_nope, q_rope, w_uk, w_uv = device_queries_weights(gen.as_single_latent(inp))
    lse = torch.full((batch, 1, h), float("nan"), device="cuda")
    out = mlra.mla_decode_attn(device_cache(gen.as_single_latent(inp)), mlra.mlra_absorb_q(q_nope, w_uk), q_rope, w_uv, wl.tau,
                               out_dtype=torch.float32, lse=lse)
    torch.cuda.synchronize()
    v = oracle_views(gen.as_single_latent(inp))
    ref, ref_lse = orc.mlra_decode_batch(v["latent_pool"], v["rope_pool"], v["page_table"], v["seq_lens"], v["q_nope"],
                                         v["q_rope"], v["w_uk"], v["w_uv"], wl.tau, 1.0, return_lse=True)
    assert max_rel_err(host(out), ref) <= TOL["bf16"]
    got, live = host(lse), np.isfinite(ref_lse)
    assert np.array_equal(np.isfinite(got), live) and np.max(np.abs(got[live] - ref_lse[live])) <= 2e-2
