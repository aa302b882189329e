"""GQA decode: one chunk per sequence (the decode kernel writes the output) and many (the merge kernel adds them), with
empty and short sequences, both output types, rows that are not made of runs of four channels.  Against the fp64 oracle;
bars 1e-2 (bf16) and 1e-5 (fp32)."""
import numpy as np
import pytest
import torch

from oracle import mlra_oracle as orc
from paper_2603_02188_amd import binding as mlra
from paper_2603_02188_amd import inputs as gen

from gpu_util import host, max_rel_err, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,h,g,d_h,lens", [
    ("bf16", 64, 4, 128, [0, 1, 31, 32, 33, 640] * 12),         # 288 workgroups for 256 CUs: one chunk each
    ("bf16", 128, 128, 128, [0, 65, 300]),                      # one query head per KV head
    ("bf16", 40, 8, 128, [9000]), ("bf16", 8, 1, 128, [20000, 0, 129]),   # 32 and 66 chunk slots
    # two to five slots: every lane's own weights up to four, lanes reduced from five on
    ("bf16", 24, 8, 128, [256, 0, 129]), ("bf16", 40, 8, 128, [300, 0, 129]), ("bf16", 40, 8, 128, [512, 1, 0, 385]),
    ("bf16", 40, 8, 128, [640, 513, 0]), ("f32", 6, 2, 30, [250, 0, 65]), ("f32", 5, 1, 64, [400, 0, 129]),
    ("f32", 6, 2, 30, [100] * 40),                              # one slot, merged (the plain kernel writes partials)
    ("f32", 6, 2, 30, [700, 0, 65]), ("f32", 5, 1, 64, [3000])])
def test_output_written_or_merged(dtype, h, g, d_h, lens):
    wl = gen.WORKLOADS["C5"].scaled(name="gqa-merge", batch=len(lens), n_min=0, n_max=max(lens), h=h, g=g, d_h=d_h,
                                    dtype=dtype, index=3300 + h)
    print(f"[case] gqa {dtype} h={h} g={g} d_h={d_h} lens={lens}", flush=True)
    gi = gen.make_gqa_inputs(wl, seq_lens=np.array(lens, dtype=np.int32))
    args = (to_device(gi.k_pool, dtype), to_device(gi.v_pool, dtype), to_device(gi.page_table), to_device(gi.seq_lens),
            to_device(gi.q, dtype), gi.scale)
    f32, b16 = (host(mlra.gqa_decode_attn(*args, out_dtype=t)) for t in (torch.float32, torch.bfloat16))
    ref = orc.gqa_decode_batch(gen.to_f64(gi.k_pool, dtype), gen.to_f64(gi.v_pool, dtype), gi.page_table, gi.seq_lens,
                               gen.to_f64(gi.q, dtype), gi.scale)
    assert max_rel_err(f32, ref) <= (1e-2 if dtype == "bf16" else 1e-5)
    assert np.array_equal(b16, orc.round_bf16(f32.astype(np.float32)))      # the fp32 output rounded once
    for s, n in enumerate(lens):
        assert n > 0 or np.all(f32[s] == 0.0)
