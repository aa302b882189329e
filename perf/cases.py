"""Performance cases of the decode-attention library: what is timed, on which inputs, and how close two correct
implementations are expected to be.

A case is one decode step as a serving loop runs it (append the new token's cache row, absorb the queries, decode),
or one of the other entry points on its own (pre-attention, the GQA comparison), with every buffer that such a loop
keeps (cache, weights, outputs, workspace) made beforehand.  Inputs are synthetic and are drawn on the GPU from the
seed; sequence lengths are spread evenly between n_min and n_max (so that the work of a case does not depend on the
seed) and dealt to the sequences in an order drawn from the seed.
"""
import math

import torch

from paper_2603_02188_amd import binding as mlra

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}
_SIZE = {"bf16": 2, "f32": 4}
_EPS, _ROPE_BASE = 1e-6, 10000.0


def _step(kind, batch, n_min, n_max, **kw):
    """A decode step.  kind: mlra (Eq. (5)), mlra2 (Eq. (6)), gla2 (Eq. (3)), mla (one latent of d_c channels)."""
    case = {"kind": kind, "batch": batch, "n_min": n_min, "n_max": n_max, "n_blocks": 4, "d_cb": 128, "d_r": 64,
            "h": 128, "d_h": 128, "dtype": "bf16", "page": 64, "shuffle": False, "q_len": 1, "folded": True,
            "gated": False, "static": False, "lse": False, "out": "bf16"}
    case.update(kw)
    return case


def _gqa(batch, n_min, n_max, **kw):
    case = {"kind": "gqa", "batch": batch, "n_min": n_min, "n_max": n_max, "h": 128, "g": 8, "d_h": 128,
            "dtype": "bf16", "page": 64, "shuffle": False, "out": "bf16"}
    case.update(kw)
    return case


def _pre(batch, **kw):
    case = {"kind": "pre", "batch": batch, "n_min": 1, "n_max": 1024, "n_blocks": 4, "d_cb": 128, "d_r": 64, "h": 128,
            "d_h": 128, "d": 7168, "d_cq": 1536, "dtype": "bf16", "page": 64, "shuffle": False}
    case.update(kw)
    return case


def listed():
    return [
        # a unit-sized model in fp32 (debugging, numerics checks): launches and host work are all there is
        dict(_step("mlra", 1, 256, 256, d_cb=64, d_r=32, h=8, d_h=64, dtype="f32", folded=False, lse=True,
                   out="f32"), name="tiny-f32"),
        # one user's request on the full-size layer, small pages, the entry point for callers that cannot allocate
        dict(_step("mlra", 1, 1501, 1501, page=16, shuffle=True, static=True), name="single-request"),
        # one device's share of four-way tensor parallelism: one latent block, 16K contexts
        dict(_step("mlra", 16, 16384, 16384, n_blocks=1), name="tp-share-16x16k"),
        # the headline: MLRA-4, 64 sequences of 8K
        dict(_step("mlra", 64, 8192, 8192), name="mlra4-64x8k"),
        # few users, very long contexts of different lengths
        dict(_step("mlra", 4, 65536, 131072), name="long-4x128k"),
        # a serving batch: mixed lengths, shuffled pages, queries scaled inside the decode call, gated output, lse
        dict(_step("mlra", 128, 512, 8192, shuffle=True, folded=False, gated=True, lse=True), name="serving-128-mixed"),
        # MLRA-2 on the headline's sizes
        dict(_step("mlra2", 64, 8192, 8192), name="mlra2-64x8k"),
        # speculative decoding: four query tokens per sequence, ragged
        dict(_step("mlra", 16, 1000, 4093, q_len=4, shuffle=True, out="f32"), name="draft-16x4"),
        # the MLA comparison on the serving batch
        dict(_step("mla", 128, 512, 8192, n_blocks=1, d_cb=512, shuffle=True), name="mla-128-mixed"),
        # the GQA comparison on the serving batch
        dict(_gqa(128, 512, 8192, shuffle=True), name="gqa-128-mixed"),
        # projections, norms, RoPE and cache append of the new token of 64 sequences
        dict(_pre(64), name="pre-attention-64"),
        # the full-size layer in fp32 (reference runs, checks of a 16-bit deployment)
        dict(_step("mlra", 8, 300, 2048, dtype="f32", folded=False, lse=True, out="f32"), name="f32-8x2k"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["mlra", "mlra", "mlra", "mlra2", "gla2", "multi", "mla", "gqa", "pre", "f32", "f32-small",
                       "bf16-small"])
    page, shuffle = rng.choice([16, 32, 64, 64, 128]), rng.random() < 0.5
    if kind == "pre":
        return _pre(_log(rng, 1, 128), d=rng.choice([1024, 4096, 7168]), d_cq=rng.choice([384, 768, 1536]),
                    h=rng.choice([17, 64, 128]), n_max=_log(rng, 64, 4096), shuffle=shuffle)
    batch = _log(rng, 1, 128)
    # no more tokens than the largest listed cases of the same kind have
    most = {"mlra": 131072, "mlra2": 131072, "gla2": 131072, "multi": 16384, "mla": 65536, "gqa": 65536, "f32": 2048,
            "f32-small": 4096, "bf16-small": 8192}[kind]
    total = {"multi": 40000, "f32": 9000, "f32-small": 60000, "bf16-small": 60000,
             "gqa": 270000}.get(kind, 500000)
    if kind == "f32":
        batch = _log(rng, 1, 16)
    n_max = _log(rng, 64, max(65, min(most, total // batch)))
    n_min = n_max if rng.random() < 0.3 else max(1, int(n_max * rng.uniform(0.05, 1.0)))
    opt = {"page": page, "shuffle": shuffle, "folded": rng.random() < 0.6, "lse": rng.random() < 0.4,
           "out": rng.choice(["bf16", "f32"])}
    if kind == "gqa":
        return _gqa(batch, n_min, n_max, g=rng.choice([4, 8, 16]), page=max(32, page), shuffle=shuffle, out=opt["out"])
    if kind == "mlra":
        return _step("mlra", batch, n_min, n_max, n_blocks=rng.choice([1, 4, 4]), h=rng.choice([64, 128, 128]),
                     gated=rng.random() < 0.3, **opt)
    if kind == "mlra2":
        return _step("mlra2", batch, n_min, n_max, **opt)
    if kind == "gla2":
        return _step("gla2", batch, n_min, n_max, n_blocks=2, d_cb=256, **opt)
    if kind == "multi":
        return _step("mlra", max(1, batch // 4), n_min, n_max, q_len=rng.choice([2, 3, 4]), **opt)
    if kind == "mla":
        return _step("mla", batch, n_min, n_max, n_blocks=1, d_cb=512, h=rng.choice([64, 128]),
                     **dict(opt, page=max(32, page)))
    if kind == "f32":
        return _step("mlra", batch, n_min, n_max, h=rng.choice([16, 64, 128]), dtype="f32",
                     **dict(opt, out="f32"))
    small = dict(d_cb=64, d_r=32, d_h=64, h=rng.choice([8, 12, 16]), n_blocks=rng.choice([2, 4]))
    return _step("mlra", batch, n_min, n_max, dtype="f32" if kind == "f32-small" else "bf16", **small,
                 **dict(opt, out="f32" if kind == "f32-small" else opt["out"]))


# ---- inputs -----------------------------------------------------------------------------------------------------
def _lens(case):
    b, lo, hi = case["batch"], case["n_min"], case["n_max"]
    return [hi if b == 1 else lo + round((hi - lo) * i / (b - 1)) for i in range(b)]


def _groups(case):
    return 2 if case["kind"] in ("mlra2", "gla2") else 1


class _State:
    pass


def _randn(gen, shape, dtype, std=1.0):
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32 if dtype == torch.float32 else dtype)
    return x if std == 1.0 else x.mul_(std)


def _paging(case, gen):
    """Sequence lengths in an order drawn from the seed, and a page table over exactly the pages they need."""
    lens = torch.tensor(_lens(case), dtype=torch.int32, device="cuda")
    lens = lens[torch.randperm(len(lens), generator=gen, device="cuda")].contiguous()
    pages = (lens.cpu() + case["page"] - 1) // case["page"]
    total, width = int(pages.sum()), int(pages.max())
    order = torch.randperm(total, generator=gen, device="cuda") if case["shuffle"] else torch.arange(total, device="cuda")
    order = order.to(torch.int32).cpu()
    table = torch.zeros((len(pages), width), dtype=torch.int32)
    at = 0
    for b, k in enumerate(pages.tolist()):
        table[b, :k] = order[at:at + k]
        at += k
    return lens, table.cuda(), total


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    s = _State()
    s.case, dt, b, h = case, _DT[case["dtype"]], case["batch"], case["h"]
    lens, table, total = _paging(case, gen)
    page = case["page"]
    if case["kind"] == "gqa":
        s.k = _randn(gen, (total, case["g"], page, case["d_h"]), dt)
        s.v = _randn(gen, (total, case["g"], page, case["d_h"]), dt)
        s.lens, s.table = lens, table
        s.q = _randn(gen, (b, h, case["d_h"]), dt)
        s.scale = 1.0 / math.sqrt(case["d_h"])
        s.out = torch.empty((b, h, case["d_h"]), dtype=_DT[case["out"]], device="cuda")
        s.workspace = torch.empty(mlra.gqa_decode_workspace_bytes(b, h, case["d_h"], table.shape[1] * page),
                                  dtype=torch.uint8, device="cuda")
        return s
    nb, d_cb, d_r, d_h = case["n_blocks"], case["d_cb"], case["d_r"], case["d_h"]
    s.cache = mlra.Cache(_randn(gen, (total, nb, page, d_cb), dt), _randn(gen, (total, page, d_r), dt), table, lens)
    s.positions = (lens - 1).contiguous()
    if case["kind"] == "pre":
        d, d_cq, std = case["d"], case["d_cq"], 1.0 / math.sqrt(case["d"])
        s.hidden = _randn(gen, (b, d), dt)
        mats = [_randn(gen, shape, dt, std) for shape in ((d, d_cq), (d, nb * d_cb), (d, d_r), (d_cq, h * d_h),
                                                          (d_cq, h * d_r))]
        gain_q = (1.0 + 0.1 * torch.randn(d_cq, generator=gen, device="cuda")).to(dt)
        gain_kv = (1.0 + 0.1 * torch.randn(nb * d_cb, generator=gen, device="cuda")).to(dt)
        s.weights = mlra.PreWeights(*mats, h, math.sqrt(d / d_cq), math.sqrt(4.0 * d / (nb * d_cb)), gain_q, gain_kv,
                                    _EPS, _ROPE_BASE)
        s.q_nope = torch.empty((b, h, d_h), dtype=dt, device="cuda")
        s.q_rope = torch.empty((b, h, d_r), dtype=dt, device="cuda")
        s.workspace = torch.empty(mlra.mlra_pre_attention_workspace_bytes(b, d, d_cq, nb, d_cb, d_r, h, d_h, dt),
                                  dtype=torch.uint8, device="cuda")
        return s
    q_len, hb = case["q_len"], h // _groups(case)
    rows = b * q_len
    s.tau = 1.0 / math.sqrt(d_h + d_r)
    s.c_kv_new = torch.randn((b, nb * d_cb), generator=gen, device="cuda")
    s.k_rope_new = torch.randn((b, d_r), generator=gen, device="cuda")
    s.q_nope, s.q_rope = _randn(gen, (rows, h, d_h), dt), _randn(gen, (rows, h, d_r), dt)
    s.w_uk = _randn(gen, (nb, d_cb, hb * d_h), dt, 1.0 / math.sqrt(d_cb))
    s.w_uv = _randn(gen, (nb, d_cb, hb * d_h), dt, 1.0 / math.sqrt(d_cb))
    s.gate = torch.sigmoid(torch.randn((b, h, d_h), generator=gen, device="cuda")).to(dt) if case["gated"] else None
    s.q_abs = torch.empty((rows, nb, hb, d_cb), dtype=dt, device="cuda")
    s.q_rope_folded = torch.empty_like(s.q_rope) if case["folded"] else None
    lead = (b, q_len) if q_len > 1 else (b,)
    s.out = torch.empty(lead + (h, d_h), dtype=_DT[case["out"]], device="cuda")
    s.lse = torch.empty(lead + (nb, hb), device="cuda") if case["lse"] else None
    width = table.shape[1]
    if q_len > 1:
        need = mlra.mlra_decode_multi_workspace_bytes(b, q_len, h, nb, d_cb, page, width)
    elif _groups(case) == 2:
        need = mlra.mlra2_decode_workspace_bytes(b, h, nb, d_cb, width * page)
    else:
        need = mlra.mlra_decode_workspace_bytes(b, h, nb, d_cb, width * page)
    s.workspace = None if case["static"] else torch.empty(need, dtype=torch.uint8, device="cuda")
    return s


# ---- one pass ---------------------------------------------------------------------------------------------------
def run(s):
    case = s.case
    if case["kind"] == "gqa":
        mlra.gqa_decode_attn(s.k, s.v, s.table, s.lens, s.q, s.scale, out=s.out, workspace=s.workspace)
        return {"out": s.out}
    if case["kind"] == "pre":
        mlra.mlra_pre_attention(s.cache, s.weights, s.hidden, s.positions, q_nope=s.q_nope, q_rope=s.q_rope,
                                workspace=s.workspace)
        return {"q_nope": s.q_nope, "q_rope": s.q_rope, "latent": s.cache.latent, "rope": s.cache.rope}
    mlra.mlra_append_kv(s.cache, s.c_kv_new, s.k_rope_new, s.positions)
    two = _groups(case) == 2
    if case["folded"]:
        absorb = mlra.mlra2_absorb_q_folded if two else mlra.mlra_absorb_q_folded
        absorb(s.q_nope, s.w_uk, s.q_rope, s.tau, q_abs=s.q_abs, q_rope_out=s.q_rope_folded)
        q_rope, scale = s.q_rope_folded, mlra.SCALE_FOLDED
    else:
        absorb = mlra.mlra2_absorb_q if two else mlra.mlra_absorb_q
        absorb(s.q_nope, s.w_uk, q_abs=s.q_abs)
        q_rope, scale = s.q_rope, s.tau
    if case["q_len"] > 1:
        lead = (case["batch"], case["q_len"])
        mlra.mlra_decode_attn_multi(s.cache, s.q_abs.view(lead + s.q_abs.shape[1:]), q_rope.view(lead + q_rope.shape[1:]),
                                    s.w_uv, scale, out=s.out, lse=s.lse, workspace=s.workspace)
    elif case["static"]:
        mlra.mlra_decode_attn_static(s.cache, s.q_abs, q_rope, s.w_uv, scale, 1.0, s.out, lse=s.lse)
    elif case["gated"]:
        mlra.mlra_decode_attn_gated(s.cache, s.q_abs, q_rope, s.w_uv, s.gate, scale, out=s.out, lse=s.lse,
                                    workspace=s.workspace)
    elif case["kind"] == "mla":
        mlra.mla_decode_attn(s.cache, s.q_abs, q_rope, s.w_uv, scale, out=s.out, lse=s.lse, workspace=s.workspace)
    else:
        decode = mlra.mlra2_decode_attn if two else mlra.mlra_decode_attn
        decode(s.cache, s.q_abs, q_rope, s.w_uv, scale, out=s.out, lse=s.lse, workspace=s.workspace)
    outputs = {"out": s.out, "q_abs": s.q_abs, "latent": s.cache.latent, "rope": s.cache.rope}
    if s.lse is not None:
        outputs["lse"] = s.lse
    if case["folded"]:
        outputs["q_rope"] = s.q_rope_folded
    return outputs


# ---- what a pass cannot do without --------------------------------------------------------------------------------
def work(case):
    e, b, h, d_h = _SIZE[case["dtype"]], case["batch"], case["h"], case["d_h"]
    tokens = sum(_lens(case))
    if case["kind"] == "gqa":
        return {"bytes": tokens * 2 * case["g"] * d_h * e + b * h * d_h * (e + _SIZE[case["out"]]),
                "flops": 4 * tokens * h * d_h}
    nb, d_cb, d_r = case["n_blocks"], case["d_cb"], case["d_r"]
    if case["kind"] == "pre":
        down, up = case["d"] * (case["d_cq"] + nb * d_cb + d_r), case["d_cq"] * h * (d_h + d_r)
        return {"bytes": (down + up + b * (case["d"] + nb * d_cb + d_r + h * (d_h + d_r))) * e,
                "flops": 2 * b * (down + up)}
    q_len, hb = case["q_len"], h // _groups(case)
    rows, out = b * q_len, _SIZE[case["out"]]
    w = nb * d_cb * hb * d_h
    byt = tokens * (nb * d_cb + d_r) * e + b * (nb * d_cb + d_r) * (4 + e) + 2 * w * e
    byt += rows * h * (d_h + d_r) * e + rows * h * d_h * out
    byt += rows * nb * hb * d_cb * e                       # the absorbed queries are an output of the step
    byt += rows * h * d_r * e if case["folded"] else 0
    byt += rows * h * d_h * e if case["gated"] else 0
    byt += rows * nb * hb * 4 if case["lse"] else 0
    flops = 2 * q_len * tokens * nb * hb * (2 * d_cb + d_r) + 4 * rows * w
    return {"bytes": byt, "flops": flops}


def tolerance(case):
    # bf16: the operands of each product (absorbed queries, probabilities, merged values) and the outputs are rounded
    # to 8 bits of mantissa, 2-norm errors of 2e-3 to 4e-3; fp32: sums in another order and hardware exponentials,
    # 4e-7 to 6e-7
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 3e-6}


# ---- the same in 64 bits, in plain torch --------------------------------------------------------------------------
def _attend(q, keys, values, scale):
    s = (q @ keys.t()) * scale
    return torch.softmax(s, dim=-1) @ values, torch.logsumexp(s, dim=-1)


def _pages(table, lens, page):
    return [(int(n), table[b, : -(-int(n) // page)].long()) for b, n in enumerate(lens.cpu().tolist())]


def exact(case, seed):
    s = prepare(case, seed)
    b, h, d_h, page = case["batch"], case["h"], case["d_h"], case["page"]
    f64 = dict(dtype=torch.float64, device="cuda")
    if case["kind"] == "gqa":
        g, r = case["g"], case["h"] // case["g"]
        out = torch.zeros((b, h, d_h), **f64)
        for i, (n, pages) in enumerate(_pages(s.table, s.lens, page)):
            for j in range(g):
                k, v = (t[pages, j].reshape(-1, d_h)[:n].double() for t in (s.k, s.v))
                out[i, j * r:(j + 1) * r] = _attend(s.q[i, j * r:(j + 1) * r].double(), k, v, s.scale)[0]
        return {"out": out}
    nb, d_cb, d_r = case["n_blocks"], case["d_cb"], case["d_r"]
    latent, rope = s.cache.latent.double(), s.cache.rope.double()
    pos = s.positions.long()
    at = s.cache.page_table.long()[torch.arange(b, device="cuda"), pos // page], pos % page
    if case["kind"] == "pre":
        w, x = s.weights, s.hidden.double()

        def norm(v, gain, alpha):
            return alpha * gain.double() * v * torch.rsqrt(v.square().mean(-1, keepdim=True) + _EPS)

        def rotate(v):      # [..., d_r] of row i at position pos[i]
            theta = _ROPE_BASE ** (-2.0 * torch.arange(d_r // 2, **f64) / d_r)
            angle = (pos.double()[:, None] * theta).view((b,) + (1,) * (v.dim() - 2) + (d_r // 2,))
            c, sn, lo, hi = torch.cos(angle), torch.sin(angle), v[..., 0::2], v[..., 1::2]
            return torch.stack((lo * c - hi * sn, lo * sn + hi * c), dim=-1).reshape(v.shape)

        c_q = norm(x @ w.w_dq.double(), w.gain_q, w.alpha_q)
        latent[at[0], :, at[1]] = norm(x @ w.w_dkv.double(), w.gain_kv, w.alpha_kv).view(b, nb, d_cb)
        rope[at[0], at[1]] = rotate(x @ w.w_kr.double())
        return {"q_nope": (c_q @ w.w_uq.double()).view(b, h, d_h),
                "q_rope": rotate((c_q @ w.w_qr.double()).view(b, h, d_r)), "latent": latent, "rope": rope}
    dt = _DT[case["dtype"]]
    latent[at[0], :, at[1]] = s.c_kv_new.to(dt).double().view(b, nb, d_cb)
    rope[at[0], at[1]] = s.k_rope_new.to(dt).double()
    groups, q_len = _groups(case), case["q_len"]
    hb, bpg, rows = h // groups, nb // groups, b * q_len
    w_uk, w_uv = (t.double().view(nb, d_cb, hb, d_h) for t in (s.w_uk, s.w_uv))
    q_nope, q_rope = s.q_nope.double(), s.q_rope.double()
    q_abs = torch.empty((rows, nb, hb, d_cb), **f64)
    for blk in range(nb):
        for i in range(hb):
            q_abs[:, blk, i] = q_nope[:, (blk // bpg) * hb + i] @ w_uk[blk, :, i].t()
    z, lse = torch.zeros((rows, nb, hb, d_cb), **f64), torch.full((rows, nb, hb), -math.inf, **f64)
    for i, (n, pages) in enumerate(_pages(s.cache.page_table, s.cache.seq_lens, page)):
        key_rope = rope[pages].reshape(-1, d_r)
        for blk in range(nb):
            c = latent[pages, blk].reshape(-1, d_cb)
            first = (blk // bpg) * hb
            for j in range(q_len):
                m, row = n - (q_len - 1 - j), i * q_len + j
                if m > 0:
                    q = torch.cat((q_abs[row, blk], q_rope[row, first:first + hb]), dim=-1)
                    z[row, blk], lse[row, blk] = _attend(q, torch.cat((c[:m], key_rope[:m]), dim=-1), c[:m], s.tau)
    out = torch.zeros((rows, h, d_h), **f64)
    for blk in range(nb):
        for i in range(hb):
            out[:, (blk // bpg) * hb + i] += z[:, blk, i] @ w_uv[blk, :, i]
    if case["gated"]:
        out *= s.gate.double()
    lead = (b, q_len) if q_len > 1 else (b,)
    fold = s.tau / math.log(2.0) if case["folded"] else 1.0
    outputs = {"out": out.view(lead + (h, d_h)), "q_abs": q_abs * fold, "latent": latent, "rope": rope}
    if case["lse"]:
        outputs["lse"] = lse.view(lead + (nb, hb))
    if case["folded"]:
        outputs["q_rope"] = q_rope * fold
    return outputs
