"""A row's output depends on the blocks it lists and on nothing else.

The query-tile kernel visits a block for every row of a tile when one of them
lists it; a row that does not list it must not see it, whatever the block
holds.  Each case poisons the keys or values of a block that only some rows of
each tile list (NaN, +-inf, and finite values whose scores overflow) and
compares the rows that do not list it, bit for bit, with the call on finite
inputs; the rows that list it are checked to have seen it.
"""
from __future__ import annotations

import zlib

import numpy as np
import pytest
import torch

from paper_2606_13392_amd import msa, synth
from tests.util import to_dev

pytestmark = pytest.mark.gpu

# name, rows, H_q, H_kv, block, topk, fp8
SHAPES = [
    ("poison_b64", 500, 64, 8, 64, 5, False),
    ("poison_b128_g16", 600, 64, 4, 128, 3, False),
    ("poison_b64_fp8", 500, 64, 8, 64, 5, True),
    ("poison_b128_g3_fp8", 700, 48, 16, 128, 3, True),
]
NAN, INF = float("nan"), float("inf")
# which tensor, values of the poisoned row
POISON = [("v", [NAN]), ("v", [INF, -INF]), ("k", [NAN]), ("k", [INF, -INF]), ("k", [3e38])]


@pytest.mark.parametrize("which,values", POISON, ids=["v_nan", "v_inf", "k_nan", "k_inf", "k_overflow"])
@pytest.mark.parametrize("shape", SHAPES, ids=[s[0] for s in SHAPES])
def test_unselected_block(shape, which, values):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    name, T, H_q, H_kv, bk, topk, fp8 = shape
    if fp8 and values != [NAN]:
        pytest.skip("E4M3 has no infinities")
    p = synth.packed_problem(name, [T], [T], num_q_heads=H_q, num_kv_heads=H_kv, block_size=bk, topk=topk,
                             seed=zlib.crc32(name.encode()) % 10000)
    x = (synth.generate_fp8_numpy if fp8 else synth.generate_numpy)(p)
    # every row lists its local block; odd rows list block 1 as well
    pos = np.arange(T)
    ids = np.full((T, H_kv, topk), -1, dtype=np.int32)
    ids[:, :, 1] = (pos // bk)[:, None]
    ids[:, :, 2] = np.where((pos % 2 == 1) & (pos // bk > 1), 1, -1)[:, None]
    dev = torch.device("cuda")
    up = (lambda a: torch.from_numpy(a).to(dev)) if fp8 else to_dev
    q, k, v, seqs = up(x["q"]), up(x["k"]), up(x["v"]), msa.Seqs.from_problem(p, dev)
    ids_d = torch.from_numpy(ids).to(dev)

    def call(k, v):
        msa.profile_reset()
        msa.profile_enable(True)
        try:
            if fp8:
                out = msa.sparse_attn_prefill_fp8(q, k, v, synth.FP8_SCALES, ids_d, seqs, bk)
            else:
                out = msa.sparse_attn_prefill(q, k, v, ids_d, seqs, bk)
            torch.cuda.synchronize()
        finally:
            msa.profile_enable(False)
        assert "tile_attn_kernel" in msa.profile_read()
        msa.profile_reset()
        return out

    o, lse = call(k, v)
    bad = {"k": k.clone(), "v": v.clone()}
    row = bad[which][bk + 7]                            # a key of block 1, every group
    if fp8:
        row.fill_(0x7F)
    else:
        row.copy_(torch.tensor(values, device=dev).repeat(row.numel() // len(values)).view_as(row).to(row.dtype))
    ob, lb = call(bad["k"], bad["v"])
    lists = torch.from_numpy((pos // bk == 1) | ((pos % 2 == 1) & (pos // bk > 1))).to(dev)
    assert torch.equal(ob[~lists].view(torch.int16), o[~lists].view(torch.int16))
    assert torch.equal(lb[~lists], lse[~lists])
    sees = lists & torch.from_numpy(pos >= bk + 7).to(dev)
    changed = ~torch.isfinite(ob[sees].float()).flatten(1).all(1) | ~torch.isfinite(lb[sees]).all(1)
    assert bool(changed.all()) or values == [3e38]
