"""The merge + up-projection kernel of the bf16 path at the edges of its forms: one chunk per sequence (rows only
copied), few and many chunk slots (lane groups of sixteen, remainders), fp32 partials, tiles of 32 sequences, two passes
over the items, gate and log-sum-exp.  Against the fp64 oracle, bar 1e-2 (bf16 operands), lse 2e-2 absolute."""
import numpy as np
import pytest
import torch

from oracle import mlra_oracle as orc
from paper_2603_02188_amd import binding as mlra
from paper_2603_02188_amd import inputs as gen

from gpu_util import device_cache, device_queries_weights, host, max_rel_err, oracle_views, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,nb,h,n_max,slots,gated", [
    (1, 1, 128, 5000, 40, True), (2, 1, 16, 2100, 17, False), (3, 2, 128, 1000, 8, True), (16, 4, 128, 300, 3, True),
    (33, 4, 16, 520, 3, True), (64, 4, 16, 90, 1, True), (33, 8, 128, 70, 1, False), (66, 4, 24, 65, 1, True)])
def test_chunks_tiles_and_gate(batch, nb, h, n_max, slots, gated):
    wl = gen.WORKLOADS["C5"].scaled(name="merge", batch=batch, n_min=0, n_max=n_max, n_blocks=nb, h=h, index=3000 + batch)
    lens = np.random.default_rng(batch).integers(0, n_max + 1, size=batch).astype(np.int32)
    lens[0], lens[-1] = (n_max, 0) if batch > 1 else (n_max, n_max)
    info = mlra.mlra_decode_plan_info(batch, h, 128, 1, nb, 128, 64, 64, -(-n_max // 64) * 64, torch.bfloat16)
    print(f"[case] merge B={batch} NB={nb} h={h} n_max={n_max} gated={gated} {info}", flush=True)
    assert info["merge_mfma"] and info["chunk_slots"] == slots
    inp = gen.make_decode_inputs(wl, poison=True, seq_lens=lens)
    cache = device_cache(inp)
    q_nope, q_rope, w_uk, w_uv = device_queries_weights(inp)
    q_abs = mlra.mlra_absorb_q(q_nope, w_uk)
    lse = torch.full((batch, nb, h), float("nan"), device="cuda")
    gate = np.random.default_rng(7).uniform(0.0, 1.0, size=(batch, h, 128)).astype(np.float32)
    gate16 = gen.to_storage(gate, "bf16")
    kw = dict(out_dtype=torch.float32, lse=lse)
    if gated:
        out = mlra.mlra_decode_attn_gated(cache, q_abs, q_rope, w_uv, to_device(gate16, "bf16"), wl.tau, 0.5, **kw)
    else:
        out = mlra.mlra_decode_attn(cache, q_abs, q_rope, w_uv, wl.tau, 0.5, **kw)
    torch.cuda.synchronize()
    v = oracle_views(inp)
    ref, ref_lse = orc.mlra_decode_batch(v["latent_pool"], v["rope_pool"], v["page_table"], v["seq_lens"], v["q_nope"],
                                         v["q_rope"], v["w_uk"], v["w_uv"], wl.tau, 0.5, return_lse=True)
    if gated:
        ref = ref * gen.to_f64(gate16, "bf16")
    err = max_rel_err(host(out), ref)
    print(f"       max rel err {err:.3e}", flush=True)
    assert err <= 1e-2
    got, live = host(lse), np.isfinite(ref_lse)
    assert np.array_equal(np.isfinite(got), live) and np.max(np.abs(got[live] - ref_lse[live])) <= 2e-2


@pytest.mark.parametrize("batch,h,n_max", [(1, 64, 5000), (5, 128, 2000), (33, 16, 300)])
def test_fp32_partials(batch, h, n_max):
    wl = gen.WORKLOADS["C5"].scaled(name="merge-mla", batch=batch, n_min=1, n_max=n_max, h=h, index=3100 + batch)
    inp = gen.make_decode_inputs(wl, poison=True)
    one = gen.as_single_latent(inp)
    info = mlra.mlra_decode_plan_info(batch, h, 128, 1, 1, 512, 64, 64, n_max, torch.bfloat16)
    print(f"[case] merge fp32 partials B={batch} h={h} {info}", flush=True)
    assert info["kernel"] == "mfma-mla" and info["merge_mfma"]
    cache = device_cache(one)
    q_nope, q_rope, w_uk, w_uv = device_queries_weights(one)
    out = mlra.mla_decode_attn(cache, mlra.mlra_absorb_q(q_nope, w_uk), q_rope, w_uv, wl.tau, out_dtype=torch.float32)
    torch.cuda.synchronize()
    v = oracle_views(one)
    ref = orc.mlra_decode_batch(v["latent_pool"], v["rope_pool"], v["page_table"], v["seq_lens"], v["q_nope"],
                                v["q_rope"], v["w_uk"], v["w_uv"], wl.tau, 1.0)
    assert max_rel_err(host(out), ref) <= 1e-2


# the MLA kernel: chunks of one tile and less, both stages, ragged ends, page turns at every tile and at every third,
# head counts below, at and above the 64 of a workgroup
@pytest.mark.parametrize("h,page,lens", [(64, 32, [1, 31, 32, 33, 64, 65, 0, 400]), (128, 96, [95, 96, 97, 130, 1000]),
                                         (70, 64, [63, 129, 2]), (16, 160, [3000, 161])])
def test_mla_tiles_and_pages(h, page, lens):
    wl = gen.WORKLOADS["C5"].scaled(name="mla-tiles", batch=len(lens), n_min=0, n_max=max(lens), h=h, page_size=page,
                                    index=3200 + h)
    one = gen.as_single_latent(gen.make_decode_inputs(wl, poison=True, seq_lens=np.array(lens, dtype=np.int32)))
    print(f"[case] mla tiles h={h} page={page} lens={lens}", flush=True)
    cache = device_cache(one)
    q_nope, q_rope, w_uk, w_uv = device_queries_weights(one)
    lse = torch.full((len(lens), 1, h), float("nan"), device="cuda")
    out = mlra.mla_decode_attn(cache, mlra.mlra_absorb_q(q_nope, w_uk), q_rope, w_uv, wl.tau, out_dtype=torch.float32,
                               lse=lse)
    torch.cuda.synchronize()
    v = oracle_views(one)
    ref, ref_lse = orc.mlra_decode_batch(v["latent_pool"], v["rope_pool"], v["page_table"], v["seq_lens"], v["q_nope"],
                                         v["q_rope"], v["w_uk"], v["w_uv"], wl.tau, 1.0, return_lse=True)
    assert max_rel_err(host(out), ref) <= 1e-2
    got, live = host(lse), np.isfinite(ref_lse)
    assert np.array_equal(np.isfinite(got), live) and np.max(np.abs(got[live] - ref_lse[live])) <= 2e-2


# whole chunks, none and ragged ends, pages that end inside and at the chunks' ends, in each MLA kernel: the pipelined one (0) on
# uniform chunks, the two-stage one (2: a batch of more than 64 in chunks of little more than 1024 tokens, all first ones
# dispatched before the second ones) and the four-stage one (4: planned chunks, one head group, as many sequences as CUs)
@pytest.mark.parametrize("batch,h,page,stages", [(64, 64, 32, 0), (64, 17, 96, 0), (64, 40, 64, 0), (70, 128, 64, 0), (65, 64, 32, 2),
                                                 (66, 17, 96, 2), (256, 16, 64, 4), (256, 64, 96, 4), (256, 17, 32, 4),
                                                 (256, 40, 64, 4)])
def test_mla_long_chunks(batch, h, page, stages):
    edges = [4090, 0, 1, 31, 32, 33, 64, 65, 96, 97, 127, 129, 160, 1023, 1024, 1025, 1056, 1057, 1088, 1089, 2047, 2049, 3071,
             3073, 3104]
    lens = (edges + [50] * batch)[:batch]
    wl = gen.WORKLOADS["C5"].scaled(name="mla-long", batch=batch, n_min=0, n_max=4090, h=h, page_size=page, index=3300 + h + batch)
    info = mlra.mlra_decode_plan_info(batch, h, 128, 1, 1, 512, 64, page, -(-4090 // page) * page, torch.bfloat16)
    print(f"[case] mla long chunks B={batch} h={h} page={page} {info}", flush=True)
    route = mlra.mlra_decode_route_info(batch, h, 128, 1, 1, 512, 64, page, -(-4090 // page) * page, torch.bfloat16)
    assert info["chunk_slots"] == (2 if batch == 70 else 4) and info["chunk_tokens"] >= 1024
    assert route["mla_stages"] == stages and route["planned"] == (stages == 4) and not route["fitted_from"]
    one = gen.as_single_latent(gen.make_decode_inputs(wl, poison=True, seq_lens=np.array(lens, dtype=np.int32)))
    cache = device_cache(one)
    q_nope, q_rope, w_uk, w_uv = device_queries_weights(one)
    lse = torch.full((batch, 1, h), float("nan"), device="cuda")
    out = mlra.mla_decode_attn(cache, mlra.mlra_absorb_q(q_nope, w_uk), q_rope, w_uv, wl.tau, out_dtype=torch.float32, lse=lse)
    torch.cuda.synchronize()
    v = oracle_views(one)
    ref, ref_lse = orc.mlra_decode_batch(v["latent_pool"], v["rope_pool"], v["page_table"], v["seq_lens"], v["q_nope"],
                                         v["q_rope"], v["w_uk"], v["w_uv"], wl.tau, 1.0, return_lse=True)
    assert max_rel_err(host(out), ref) <= 1e-2
    got, live = host(lse), np.isfinite(ref_lse)
    assert np.array_equal(np.isfinite(got), live) and np.max(np.abs(got[live] - ref_lse[live])) <= 2e-2


# the MLA kernel where the reference maxima move at every tile (scores that grow by 2^40 a tile in some heads, fall in others
# and stay in the rest): short chunks, whole ones and ragged ends, both head groups of a workgroup's waves, one tile to many
@pytest.mark.parametrize("h,page,lens", [(70, 32, [200, 33, 1, 0]), (128, 64, [31, 32, 64, 65, 129, 160, 161, 1000]), (16, 96, [700])])
def test_mla_growing_scores(h, page, lens):
    print(f"[case] mla growing scores h={h} page={page} lens={lens}", flush=True)
    gen_t = torch.Generator().manual_seed(h)
    b, width = len(lens), -(-max(lens) // page)
    total = b * width
    randn = lambda *shape: torch.randn(shape, generator=gen_t)
    u = randn(512) / 512 ** 0.5
    u = u / u.norm()
    ramp = torch.arange(width * page, dtype=torch.float32) * 4.0          # along u: 128 per tile
    c = ramp[None, :, None] * u + 0.5 * randn(b, width * page, 512)
    latent = c.view(b, width, 1, page, 512).reshape(total, 1, page, 512).bfloat16()
    rope = randn(total, page, 64).bfloat16()
    sign = torch.tensor([1.0, -1.0, 0.0])[torch.arange(h) % 3]
    q_abs = (sign[None, :, None] * 3.0 * u + 0.02 * randn(b, h, 512))[:, None].bfloat16()
    q_rope, w_uv = randn(b, h, 64).bfloat16(), (randn(1, 512, h * 128) / 512 ** 0.5).bfloat16()
    table = torch.arange(total, dtype=torch.int32).view(b, width)
    tau = 1.0 / 192 ** 0.5
    cache = mlra.Cache(latent.cuda(), rope.cuda(), table.cuda(), torch.tensor(lens, dtype=torch.int32).cuda())
    lse = torch.full((b, 1, h), float("nan"), device="cuda")
    out = mlra.mla_decode_attn(cache, q_abs.cuda(), q_rope.cuda(), w_uv.cuda(), tau, out_dtype=torch.float32, lse=lse)
    torch.cuda.synchronize()
    ref, ref_lse = np.zeros((b, h, 128)), np.full((b, 1, h), -np.inf)
    w = w_uv.double().view(512, h, 128)
    for i, n in enumerate(lens):
        if n == 0:
            continue
        keys = latent[i * width:(i + 1) * width].double().reshape(-1, 512)[:n]
        ropes = rope[i * width:(i + 1) * width].double().reshape(-1, 64)[:n]
        s = (q_abs[i, 0].double() @ keys.T + q_rope[i].double() @ ropes.T) * tau
        z = torch.softmax(s, dim=-1) @ keys
        ref[i] = torch.stack([z[j] @ w[:, j] for j in range(h)]).numpy()
        ref_lse[i, 0] = torch.logsumexp(s, dim=-1).numpy()
    assert max_rel_err(host(out), ref) <= 1e-2
    got, live = host(lse), np.isfinite(ref_lse)
    assert np.array_equal(np.isfinite(got), live) and np.max(np.abs(got[live] - ref_lse[live])) <= 2e-2


# the two-stage MLA kernel: more workgroups than CUs in short chunks, more sequences than chunks are fitted for
@pytest.mark.parametrize("batch,h,n_max", [(70, 128, 640), (90, 40, 500)])
def test_mla_short_chunks_of_many_workgroups(batch, h, n_max):
    wl = gen.WORKLOADS["C5"].scaled(name="mla-short", batch=batch, n_min=0, n_max=n_max, h=h, index=3400 + batch)
    lens = np.random.default_rng(batch).integers(0, n_max + 1, size=batch).astype(np.int32)
    lens[0], lens[1] = n_max, 0
    info = mlra.mlra_decode_plan_info(batch, h, 128, 1, 1, 512, 64, 64, n_max, torch.bfloat16)
    print(f"[case] mla short chunks B={batch} h={h} {info}", flush=True)
    assert batch * info["chunk_slots"] * ((h + 63) // 64) > 256 and info["chunk_tokens"] < 768 and info["target_chunks"] == 0
    one = gen.as_single_latent(gen.make_decode_inputs(wl, poison=True, seq_lens=lens))
    cache = device_cache(one)
    q_nope, q_rope, w_uk, w_uv = device_queries_weights(one)
    out = mlra.mla_decode_attn(cache, mlra.mlra_absorb_q(q_nope, w_uk), q_rope, w_uv, wl.tau, out_dtype=torch.float32)
    torch.cuda.synchronize()
    v = oracle_views(one)
    ref = orc.mlra_decode_batch(v["latent_pool"], v["rope_pool"], v["page_table"], v["seq_lens"], v["q_nope"],
                                v["q_rope"], v["w_uk"], v["w_uv"], wl.tau, 1.0)
    assert max_rel_err(host(out), ref) <= 1e-2


# absorb: blocks of one to several workgroups of 128 channels, a last one of fewer, batches around its 64 sequences
@pytest.mark.parametrize("batch,nb,d_cb", [(1, 1, 160), (63, 2, 288), (65, 1, 512), (5, 3, 32)])
def test_absorb_channel_passes(batch, nb, d_cb):
    print(f"[case] absorb B={batch} NB={nb} d_cb={d_cb}", flush=True)
    gen_t = torch.Generator().manual_seed(d_cb)
    h, d_h, d_r = 3, 128, 64
    q = torch.randn((batch, h, d_h), generator=gen_t).bfloat16()
    q_rope = torch.randn((batch, h, d_r), generator=gen_t).bfloat16()
    w_uk = (torch.randn((nb, d_cb, h * d_h), generator=gen_t) / d_h ** 0.5).bfloat16()
    ref = torch.einsum("bid,ncid->bnic", q.double(), w_uk.double().view(nb, d_cb, h, d_h)).numpy()
    assert max_rel_err(host(mlra.mlra_absorb_q(q.cuda(), w_uk.cuda())), ref) <= 1e-2
    tau = 1.0 / 192 ** 0.5
    q_abs, folded = mlra.mlra_absorb_q_folded(q.cuda(), w_uk.cuda(), q_rope.cuda(), tau)
    assert max_rel_err(host(q_abs), ref * tau / np.log(2.0)) <= 1e-2
    assert max_rel_err(host(folded), q_rope.double().numpy() * tau / np.log(2.0)) <= 1e-2
