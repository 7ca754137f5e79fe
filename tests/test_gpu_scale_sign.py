"""Softmax scales of either sign and zero.

Causal masks and running maxima belong to the scaled scores: masking a raw
score with -inf gives +inf under a negative scale and NaN under a zero one.
Every attention path is compared with the oracle at 0 (uniform weights over
the visible tokens) and at -1/sqrt(d), with the bars of tests/util.py.
"""
from __future__ import annotations

import math
import zlib

import numpy as np
import pytest
import torch

import oracle.msa_oracle as O
from paper_2606_13392_amd import msa, synth
from tests.test_gpu_backward import _check_all, _setup
from tests.util import check_outputs, to_dev

pytestmark = pytest.mark.gpu

SCALES = [0.0, -1.0 / math.sqrt(128)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    msa.lib()
    yield
    torch.cuda.synchronize()


# name, q_rows, kv_lens, H_q, H_kv, block, topk, fp8, kernels that run
CASES = [
    ("scale_tiles", [255, 40], [255, 300], 64, 8, 64, 4, False, {"tile_attn_kernel"}),
    ("scale_tiles_fp8_bk128", [500, 63], [500, 63], 64, 4, 128, 4, True, {"tile_attn_kernel"}),
    ("scale_split", [3600], [3600], 64, 8, 64, 4, False, {"tile_attn_kernel", "kvo_attn_kernel"}),
    ("scale_key_block_outer_fp8", [90], [700], 8, 2, 64, 5, True, {"kvo_attn_kernel"}),
    ("scale_dense", [300, 33], [300, 200], 16, 2, 64, 0, False, {"dense_prefill_kernel"}),
]


@pytest.mark.parametrize("scale", SCALES)
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_scale_forward(case, scale):
    name, q_rows, kv_lens, H_q, H_kv, bk, topk, fp8, kernels = case
    p = synth.packed_problem(name, q_rows, kv_lens, num_q_heads=H_q, num_kv_heads=H_kv, block_size=bk,
                             topk=max(topk, 1), seed=zlib.crc32(name.encode()) % 10000)
    x = (synth.generate_fp8_numpy if fp8 else synth.generate_numpy)(p)
    dev = torch.device("cuda")
    up = (lambda a: torch.from_numpy(a).to(dev)) if fp8 else to_dev
    q, k, v, seqs = up(x["q"]), up(x["k"]), up(x["v"]), msa.Seqs.from_problem(p, dev)
    ids = synth.random_block_ids(p)
    ids_d = torch.from_numpy(ids).to(dev)

    def call(kind):
        if kind == "dense":
            return msa.dense_attn(q, k, v, seqs, softmax_scale=scale)
        if fp8:
            return getattr(msa, f"sparse_attn_{kind}_fp8")(q, k, v, synth.FP8_SCALES, ids_d, seqs, bk,
                                                           softmax_scale=scale)
        return getattr(msa, f"sparse_attn_{kind}")(q, k, v, ids_d, seqs, bk, softmax_scale=scale)

    rows = sorted(set(np.linspace(0, p.total_q_rows - 1, 40).astype(int).tolist()))
    lay = O.layout_of(p)
    if topk == 0:
        o_ref, l_ref = O.dense_causal_attention(x["q"], x["k"], x["v"], lay, scale=scale, rows=rows)
    else:
        o_ref, l_ref = O.sparse_attention(x["q"], x["k"], x["v"], ids, lay, bk, scale=scale, rows=rows,
                                          fmt="e4m3" if fp8 else "bf16",
                                          input_scales=synth.FP8_SCALES if fp8 else (1.0, 1.0, 1.0))
    msa.profile_reset()
    msa.profile_enable(True)
    try:
        outs = {kind: call(kind) for kind in (("dense",) if topk == 0 else ("prefill",))}
        torch.cuda.synchronize()
    finally:
        msa.profile_enable(False)
    launched = set(msa.profile_read())
    msa.profile_reset()
    assert {n for n in launched if "attn" in n or "dense" in n} == kernels
    if topk:
        outs["decode"] = call("decode")
    for kind, (o, lse) in outs.items():
        check_outputs(o[rows].float().cpu().numpy(), lse[rows].cpu().numpy(), o_ref, l_ref, f"{name} {kind}")


@pytest.mark.parametrize("scale", SCALES)
@pytest.mark.parametrize("bk", [64, 128])
def test_scale_backward(bk, scale):
    """Blocks partly visible to their rows: a row's own and a sequence's last."""
    p, x, ids = _setup(f"scale_bwd_{bk}", [150, 70], [150, 333], 16, 2, 3, None, bk)
    dev = torch.device("cuda")
    seqs = msa.Seqs.from_problem(p, dev)
    d = {n: to_dev(a) for n, a in x.items()}
    ids_d = torch.from_numpy(ids).to(dev)
    o, lse = msa.sparse_attn_decode(d["q"], d["k"], d["v"], ids_d, seqs, bk, softmax_scale=scale)
    got = msa.sparse_attn_backward(d["q"], d["k"], d["v"], o, lse, d["d_o"], ids_d, seqs, bk, softmax_scale=scale)
    ref = O.sparse_attention_backward(x["q"], x["k"], x["v"], x["d_o"], ids, O.layout_of(p), bk, scale=scale)
    _check_all(f"scale_bwd_{bk}", [t.float().cpu().numpy() for t in got], ref)
