"""Decode attention in slots of 64 keys.

A 128-key block is two slots, of which the second may be partly or wholly past
the row or the sequence.  Contexts sit around halves and ends of blocks; ids
come in any order with padding, out-of-range entries and empty rows; splits
run from one CTA per row to more than the combine takes at once.  A workspace
of the whole-block split's size (and none where that needs none) is accepted
and gives the same attention: the splits' running maxima round weights to bf16
at other points, so the outputs differ by at most two roundings of 2^-9 each
way, 5e-3.
"""
from __future__ import annotations

import zlib

import numpy as np
import pytest
import torch

import oracle.msa_oracle as O
from paper_2606_13392_amd import msa, synth
from tests.test_gpu_paged import _paged_copy
from tests.util import check_outputs, to_dev

pytestmark = pytest.mark.gpu

# name, q_rows, kv_lens, H_q, H_kv, block, topk, fp8, paged
CASES = [
    ("half_edges", [1] * 8, [1, 63, 64, 65, 127, 128, 129, 191], 64, 4, 128, 2, False, False),
    ("half_edges_fp8_pages", [1] * 8, [1, 63, 64, 65, 127, 128, 129, 4000], 64, 4, 128, 3, True, True),
    ("one_row_many_splits", [1], [9001], 16, 1, 128, 63, False, False),
    ("one_row_splits_b64", [1], [5001], 64, 4, 64, 63, True, False),
    ("rows_pages", [4, 2, 7], [1500, 66, 7], 48, 16, 128, 8, False, True),
    # fewer blocks than slots: the waves' slots alternate from six a wave on
    ("padded_lists", [4, 1, 4] * 12, [1451, 2049, 4140] * 12, 32, 4, 128, 63, False, False),
    ("padded_lists_fp8_pages", [2] * 40, [700, 1300] * 20, 64, 16, 128, 15, True, True),
    ("padded_lists_few_slots", [4, 1, 4], [1451, 2049, 4140], 32, 4, 128, 63, False, False),
    ("many_rows_one_cta", [8] * 80, [700] * 80, 32, 8, 128, 4, True, False),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_decode_slots(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    name, q_rows, kv_lens, H_q, H_kv, bk, topk, fp8, paged = case
    p = synth.packed_problem(name, q_rows, kv_lens, num_q_heads=H_q, num_kv_heads=H_kv, block_size=bk, topk=topk,
                             seed=zlib.crc32(name.encode()) % 10000, kv_pad_to=max(kv_lens))
    x = synth.generate_fp8_numpy(p, synth.FP8_SCALES) if fp8 else synth.generate_numpy(p)
    rng = np.random.default_rng(p.seed)
    ids = rng.permuted(synth.random_block_ids(p, pad_slots=1), axis=2)
    pos = p.positions()
    for row in range(p.total_q_rows):
        for g, j in np.argwhere(ids[row] < 0)[:1]:
            ids[row, g, j] = pos[row] // bk + 1           # past the local block: contributes nothing
    if p.total_q_rows > 1:
        ids[0, 0] = -1
    dev = torch.device("cuda")
    up = (lambda a: torch.from_numpy(a).to(dev)) if fp8 else to_dev
    q, k, v, seqs = up(x["q"]), up(x["k"]), up(x["v"]), msa.Seqs.from_problem(p, dev)
    if paged:
        pool, seqs = _paged_copy(p, x, dev, seed=5)
        k, v = up(pool["k"]), up(pool["v"])
    ids_d = torch.from_numpy(ids).to(dev)

    def call(ws=None):
        if fp8:
            return msa.sparse_attn_decode_fp8(q, k, v, synth.FP8_SCALES, ids_d, seqs, bk, workspace=ws)
        return msa.sparse_attn_decode(q, k, v, ids_d, seqs, bk, workspace=ws)

    o, lse = call()
    empty = (ids < 0).all(axis=2).repeat(H_q // H_kv, axis=1)
    assert np.array_equal(empty, np.isneginf(lse.cpu().numpy())) and not o.float().cpu().numpy()[empty].any()
    full = np.flatnonzero(~empty.any(axis=1))
    rows = sorted(rng.choice(full, size=min(24, full.size), replace=False).tolist())
    o_ref, l_ref = O.sparse_attention(x["q"], x["k"], x["v"], ids, O.layout_of(p), bk, rows=rows,
                                      fmt="e4m3" if fp8 else "bf16",
                                      input_scales=synth.FP8_SCALES if fp8 else (1.0, 1.0, 1.0))
    check_outputs(o[rows].float().cpu().numpy(), lse[rows].cpu().numpy(), o_ref, l_ref, name)
    # the whole-block split: ceil(k / (4 ceil(k / waves))) partials of every head row
    k1 = ids.shape[2]
    want = min(max(1, -(-2048 // (4 * p.total_q_rows * H_kv))), -(-k1 // 4))
    nsplit = -(-k1 // (4 * -(-k1 // (4 * want))))
    hr = p.total_q_rows * H_q
    need = 0 if nsplit == 1 else -(-nsplit * hr * 128 * 4 // 256) * 256 + nsplit * hr * 4
    ow, lw = call(torch.empty(need, dtype=torch.uint8, device=dev))
    fin = torch.isfinite(lse)
    assert torch.equal(fin, torch.isfinite(lw)) and float((lse - lw)[fin].abs().max()) <= 1e-5
    assert float((o.double() - ow.double()).norm() / ow.double().norm()) <= 5e-3


@pytest.mark.parametrize("topk,splits", [(3, 1), (4, 1), (5, 3)])
def test_few_blocks_take_one_cta(topk, splits):
    """Up to four 128-key blocks are one CTA's eight slots; from five on (two
    CTAs as whole blocks) every four slots are a split."""
    p = synth.packed_problem(f"one_cta_{topk}", [1], [3000], num_q_heads=64, num_kv_heads=4, block_size=128, topk=topk,
                             seed=topk)
    seqs = msa.Seqs.from_problem(p, torch.device("cuda"))
    need = 0 if splits == 1 else splits * 64 * 128 * 4 + splits * 64 * 4
    assert msa.lib().msa_sparse_attn_decode_workspace_size(seqs.ref(), 64, 4, 128, 128, topk) == need
