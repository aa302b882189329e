"""Caches whose page tables are wide enough for close to 2^31 tokens (a few pages of many tokens, shared by the sequences): what
the kernels compute from a capacity stays in range, and the short sequences in it come out as in a small cache."""
import numpy as np
import pytest
import torch

from paper_2603_02188_amd import binding as mlra

from gpu_util import host, max_rel_err

pytestmark = pytest.mark.gpu


def _table(batch, width, pages):
    table = torch.zeros((batch, width), dtype=torch.int32)
    table[:, :pages] = torch.arange(pages, dtype=torch.int32)
    return table.cuda()


def _attend(q, keys, values, scale):
    return torch.softmax((q @ keys.T) * scale, dim=-1) @ values


# one chunk per sequence, as long as the capacity; sequences of none, one and more than the 2^31 - capacity tokens
def test_fp32_step_in_one_chunk():
    batch, nb, h, d_cb, d_r, d_h, page, width = 64, 4, 4, 32, 16, 32, 16384, 131071
    print("[case] huge capacity fp32", flush=True)
    assert mlra.mlra_decode_plan_info(batch, h, d_h, 1, nb, d_cb, d_r, page, page * width, torch.float32)["chunk_slots"] == 1
    g = torch.Generator().manual_seed(1)
    latent, rope = torch.randn((2, nb, page, d_cb), generator=g), torch.randn((2, page, d_r), generator=g)
    q_abs, q_rope = torch.randn((batch, nb, h, d_cb), generator=g), torch.randn((batch, h, d_r), generator=g)
    w_uv = torch.randn((nb, d_cb, h * d_h), generator=g) / d_cb ** 0.5
    lens = torch.zeros(batch, dtype=torch.int32)
    lens[0], lens[1], lens[63] = 16500, 1, 300
    cache = mlra.Cache(latent.cuda(), rope.cuda(), _table(batch, width, 2), lens.cuda())
    out = mlra.mlra_decode_attn(cache, q_abs.cuda(), q_rope.cuda(), w_uv.cuda(), 0.1, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = torch.zeros((batch, h, d_h), dtype=torch.float64)
    for s in (0, 1, 63):
        n = int(lens[s])
        kr = rope.double().reshape(-1, d_r)[:n]
        for b in range(nb):
            c = latent[:, b].double().reshape(-1, d_cb)[:n]
            z = _attend(torch.cat((q_abs[s, b], q_rope[s]), -1).double(), torch.cat((c, kr), -1), c, 0.1)
            ref[s] += torch.einsum("hc,chd->hd", z, w_uv[b].double().view(d_cb, h, d_h))
    assert max_rel_err(host(out), ref.numpy()) <= 1e-5


def test_fp32_gqa_in_one_chunk():
    batch, h, g_heads, d_h, page, width = 256, 4, 2, 8, 16384, 131071
    print("[case] huge capacity gqa", flush=True)
    g = torch.Generator().manual_seed(2)
    k, v = (torch.randn((2, g_heads, page, d_h), generator=g) for _ in range(2))
    q = torch.randn((batch, h, d_h), generator=g)
    lens = torch.zeros(batch, dtype=torch.int32)
    lens[0], lens[1], lens[255] = 16500, 1, 300
    out = mlra.gqa_decode_attn(k.cuda(), v.cuda(), _table(batch, width, 2), lens.cuda(), q.cuda(), 0.3, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = np.zeros((batch, h, d_h))
    for s in (0, 1, 255):
        n = int(lens[s])
        for i in range(h):
            keys, values = (t[:, i // (h // g_heads)].double().reshape(-1, d_h)[:n] for t in (k, v))
            ref[s, i] = _attend(q[s, i:i + 1].double(), keys, values, 0.3)[0].numpy()
    assert max_rel_err(host(out), ref) <= 1e-5


# chunk lengths fitted by the kernel: several query tokens in one chunk as long as the capacity, and the MLA kernel, whose
# shortest chunk is 390,168 tiles of 64 tokens here
def test_several_query_tokens_in_one_chunk():
    batch, q_len, nb, h, d_cb, d_r, d_h, page, width = 64, 2, 4, 128, 128, 64, 128, 16384, 131071
    print("[case] huge capacity several query tokens", flush=True)
    route = mlra.mlra_decode_route_info(batch, h, d_h, 1, nb, d_cb, d_r, page, page * width, torch.bfloat16, q_len)
    assert route["chunk_slots"] == 1 and route["fitted_from"] == page * width
    g = torch.Generator().manual_seed(3)
    bf = lambda *shape: torch.randn(shape, generator=g).bfloat16()
    latent, rope = bf(2, nb, page, d_cb), bf(2, page, d_r)
    q_abs, q_rope, w_uv = bf(batch, q_len, nb, h, d_cb), bf(batch, q_len, h, d_r), (bf(nb, d_cb, h * d_h) / 16).bfloat16()
    lens = torch.zeros(batch, dtype=torch.int32)
    lens[0], lens[1], lens[63] = 16500, 1, 300
    cache = mlra.Cache(latent.cuda(), rope.cuda(), _table(batch, width, 2), lens.cuda())
    out = mlra.mlra_decode_attn_multi(cache, q_abs.cuda(), q_rope.cuda(), w_uv.cuda(), 0.05, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = torch.zeros((batch, q_len, h, d_h), dtype=torch.float64)
    for s in (0, 1, 63):
        for j in range(q_len):
            n = int(lens[s]) - (q_len - 1 - j)
            if n <= 0:
                continue
            kr = rope.double().reshape(-1, d_r)[:n]
            for b in range(nb):
                c = latent[:, b].double().reshape(-1, d_cb)[:n]
                z = _attend(torch.cat((q_abs[s, j, b], q_rope[s, j]), -1).double(), torch.cat((c, kr), -1), c, 0.05)
                ref[s, j] += (z[:, None, :] @ w_uv[b].double().view(d_cb, h, d_h).transpose(0, 1))[:, 0]
    assert max_rel_err(host(out), ref.numpy()) <= 1e-2


def test_mla_fitted():
    batch, h, d_c, d_r, d_h, page, width = 3, 64, 512, 64, 128, 4096, (1 << 19) - 1
    print("[case] huge capacity mla", flush=True)
    route = mlra.mlra_decode_route_info(batch, h, d_h, 1, 1, d_c, d_r, page, page * width, torch.bfloat16)
    assert route["chunk_slots"] == 86 and route["fitted_from"] == 390168 * 64
    g = torch.Generator().manual_seed(4)
    bf = lambda *shape: torch.randn(shape, generator=g).bfloat16()
    latent, rope = bf(2, 1, page, d_c), bf(2, page, d_r)
    q_abs, q_rope, w_uv = bf(batch, 1, h, d_c), bf(batch, h, d_r), (bf(1, d_c, h * d_h) / 16).bfloat16()
    lens = torch.tensor([5000, 0, 77], dtype=torch.int32)
    cache = mlra.Cache(latent.cuda(), rope.cuda(), _table(batch, width, 2), lens.cuda())
    out = mlra.mla_decode_attn(cache, q_abs.cuda(), q_rope.cuda(), w_uv.cuda(), 0.03, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = torch.zeros((batch, h, d_h), dtype=torch.float64)
    for s in (0, 2):
        n = int(lens[s])
        c, kr = latent.double().reshape(-1, d_c)[:n], rope.double().reshape(-1, d_r)[:n]
        z = _attend(torch.cat((q_abs[s, 0], q_rope[s]), -1).double(), torch.cat((c, kr), -1), c, 0.03)
        ref[s] = (z[:, None, :] @ w_uv[0].double().view(d_c, h, d_h).transpose(0, 1))[:, 0]
    assert max_rel_err(host(out), ref.numpy()) <= 1e-2


# a cache that is one page of more than 4 GiB of latents: the heavy tokens (a RoPE channel makes the others' weights 0) are the last
# ones, whose latents a 32-bit offset would take from the page's start
def test_mla_page_beyond_32_bit_offsets():
    h, d_c, d_r, d_h, page, heavy = 64, 512, 64, 128, (1 << 22) + 128, 100
    n = page - 13
    print("[case] huge page mla", flush=True)
    assert mlra.mlra_decode_route_info(1, h, d_h, 1, 1, d_c, d_r, page, page, torch.bfloat16)["mla_stages"] == 0
    g = torch.Generator().manual_seed(5)
    bf = lambda *shape: torch.randn(shape, generator=g).bfloat16()
    latent = torch.zeros((1, 1, page, d_c), dtype=torch.bfloat16, device="cuda")
    rope = torch.zeros((1, page, d_r), dtype=torch.bfloat16, device="cuda")
    c, kr, q_abs, q_rope = bf(heavy, d_c), bf(heavy, d_r), bf(1, 1, h, d_c), bf(1, h, d_r)
    kr[:, 0], q_rope[:, :, 0] = 0.0, 64.0
    w_uv = (bf(1, d_c, h * d_h) / 16).bfloat16()
    latent[0, 0, n - heavy:n], rope[0, n - heavy:n] = c.cuda(), kr.cuda()
    rope[0, :n - heavy, 0] = -1000.0                  # scores 0.03 x 64000 below: weights of 0
    cache = mlra.Cache(latent, rope, torch.zeros((1, 1), dtype=torch.int32, device="cuda"),
                       torch.tensor([n], dtype=torch.int32, device="cuda"))
    out = mlra.mla_decode_attn(cache, q_abs.cuda(), q_rope.cuda(), w_uv.cuda(), 0.03, out_dtype=torch.float32)
    torch.cuda.synchronize()
    z = _attend(torch.cat((q_abs[0, 0], q_rope[0]), -1).double(), torch.cat((c, kr), -1).double(), c.double(), 0.03)
    ref = (z[:, None, :] @ w_uv[0].double().view(d_c, h, d_h).transpose(0, 1))[:, 0]
    assert max_rel_err(host(out)[0], ref.numpy()) <= 1e-2


# four slots per sequence that no planning kernel cuts (the epilogue is the fp32 one): each chunk is as long as the capacity, and
# the third and fourth start beyond 2^31
@pytest.mark.parametrize("dtype,kernel", [(torch.bfloat16, "mfma-mla"), (torch.float32, "generic")])
def test_slots_beyond_the_capacity(dtype, kernel):
    batch, h, d_c, d_r, d_h, page, width = 256, 8, 512, 64, 64, 4096, (1 << 19) - 1
    print(f"[case] slots beyond the capacity {kernel}", flush=True)
    info = mlra.mlra_decode_plan_info(batch, h, d_h, 1, 1, d_c, d_r, page, page * width, dtype)
    route = mlra.mlra_decode_route_info(batch, h, d_h, 1, 1, d_c, d_r, page, page * width, dtype)
    assert info["kernel"] == kernel and info["chunk_slots"] == 4 and info["chunk_tokens"] == page * width
    assert not route["planned"] and not route["fitted_from"]
    g = torch.Generator().manual_seed(6)
    draw = lambda *shape: torch.randn(shape, generator=g).to(dtype)
    latent, rope = draw(2, 1, page, d_c), draw(2, page, d_r)
    q_abs, q_rope, w_uv = draw(batch, 1, h, d_c), draw(batch, h, d_r), (draw(1, d_c, h * d_h) / 16).to(dtype)
    lens = torch.zeros(batch, dtype=torch.int32)
    lens[0], lens[1], lens[255] = 4200, 1, 300
    table = torch.zeros((batch, width), dtype=torch.int32, device="cuda")
    table[:, 1] = 1
    cache = mlra.Cache(latent.cuda(), rope.cuda(), table, lens.cuda())
    out = mlra.mla_decode_attn(cache, q_abs.cuda(), q_rope.cuda(), w_uv.cuda(), 0.03, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = torch.zeros((batch, h, d_h), dtype=torch.float64)
    for s in (0, 1, 255):
        n = int(lens[s])
        c, kr = latent.double().reshape(-1, d_c)[:n], rope.double().reshape(-1, d_r)[:n]
        z = _attend(torch.cat((q_abs[s, 0], q_rope[s]), -1).double(), torch.cat((c, kr), -1), c, 0.03)
        ref[s] = (z[:, None, :] @ w_uv[0].double().view(d_c, h, d_h).transpose(0, 1))[:, 0]
    assert max_rel_err(host(out), ref.numpy()) <= (1e-2 if dtype == torch.bfloat16 else 1e-5)
