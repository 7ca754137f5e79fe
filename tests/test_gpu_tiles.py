"""Prefill Main Branch by query tiles (rows of short causal contexts).

Prefill calls whose rows select much of their causal context run the tile
kernel.  Cases sit where it can go wrong: row counts around a tile, contexts
around key sub-blocks and blocks, group sizes that do not divide a wave's 32
rows, ids in any order with padding, out-of-range entries and empty rows,
E4M3, pages, and calls split between tiles and key-block-outer kernels.
Sampled rows are compared with the float64 oracle, all rows with the decode
call (another kernel for the same attention): both round weights and outputs
to bf16, so they differ by at most two roundings of 2^-9 each way, 5e-3.
"""
from __future__ import annotations

import zlib

import numpy as np
import pytest
import torch

import oracle.msa_oracle as O
from paper_2606_13392_amd import msa, synth
from tests.util import check_outputs, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    msa.lib()
    yield
    torch.cuda.synchronize()


# name, q_rows, kv_lens, H_q, H_kv, block, topk, fp8, paged, tiles only
CASES = [
    ("tile_edges", [255, 256, 257, 1, 15, 16, 17], [255, 256, 257, 1, 15, 16, 17], 64, 8, 64, 4, False, False, True),
    ("bk128_g16_pages", [127, 129, 385, 8, 9], [127, 129, 385, 8, 9], 64, 4, 128, 3, False, True, True),
    ("fp8_pages", [300, 64, 65], [300, 64, 65], 64, 8, 64, 5, True, True, True),
    ("fp8_bk128", [500, 63], [500, 63], 64, 4, 128, 4, True, False, True),
    ("g3_context", [200, 131, 70], [650, 131, 710], 48, 16, 64, 12, False, False, True),
    ("g5_fp8", [190, 77], [190, 77], 80, 16, 64, 6, True, False, True),
    ("g1", [260, 600], [260, 900], 32, 32, 64, 16, False, True, True),
    ("k1_local_only", [256, 130], [256, 130], 64, 8, 64, 1, False, False, True),
    ("k64_many_groups", [400], [400], 64, 32, 64, 63, False, False, True),
    ("split_at_reach", [3600], [3600], 64, 8, 64, 3, False, False, False),
    ("split_bk128_pages_fp8", [3600, 700], [3600, 700], 64, 8, 128, 2, True, True, False),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_tiles(case):
    name, q_rows, kv_lens, H_q, H_kv, bk, topk, fp8, paged, only = case
    p = synth.packed_problem(name, q_rows, kv_lens, num_q_heads=H_q, num_kv_heads=H_kv, block_size=bk, topk=topk,
                             seed=zlib.crc32(name.encode()) % 10000)
    x = (synth.generate_fp8_numpy if fp8 else synth.generate_numpy)(p)
    rng = np.random.default_rng(p.seed)
    ids = synth.random_block_ids(p, pad_slots=1)
    # slots in any order; one entry past the local block, where a slot is free; every 50th (row, group) empty
    ids = rng.permuted(ids, axis=2)
    pos = p.positions()
    for row in range(p.total_q_rows):
        free = np.argwhere(ids[row] < 0)
        for g, j in free[:1]:
            ids[row, g, j] = pos[row] // bk + 1
    ids.reshape(-1, topk + 1)[::50] = -1
    dev = torch.device("cuda")
    up = (lambda a: torch.from_numpy(a).to(dev)) if fp8 else to_dev
    q, k, v, seqs = up(x["q"]), up(x["k"]), up(x["v"]), msa.Seqs.from_problem(p, dev)
    if paged:
        nb = [-(-n // bk) for n in kv_lens]
        pages = rng.permutation(sum(nb) + 3)
        table = np.zeros((len(nb), max(nb)), dtype=np.int32)
        pool = torch.zeros(((sum(nb) + 3) * bk, H_kv, 128), dtype=k.dtype, device=dev)
        pk, pv, at = pool, pool.clone(), 0
        for s, n in enumerate(nb):
            for b in range(n):
                table[s, b] = pages[at]
                at += 1
                rows = min(bk, kv_lens[s] - b * bk)
                src, dst = p.kv_starts[s] + b * bk, int(table[s, b]) * bk
                pk[dst:dst + rows] = k[src:src + rows]
                pv[dst:dst + rows] = v[src:src + rows]
        k, v = pk, pv
        seqs = msa.Seqs(q_rows, kv_lens, [0] * len(nb), pool.shape[0], dev, block_table=torch.from_numpy(table).to(dev),
                        page_size=bk)
    ids_d = torch.from_numpy(ids).to(dev)
    scales = synth.FP8_SCALES

    def call(kind):
        fn = getattr(msa, f"sparse_attn_{kind}" + ("_fp8" if fp8 else ""))
        return fn(q, k, v, scales, ids_d, seqs, bk) if fp8 else fn(q, k, v, ids_d, seqs, bk)

    msa.profile_reset()
    msa.profile_enable(True)
    try:
        o, lse = call("prefill")
        torch.cuda.synchronize()
    finally:
        msa.profile_enable(False)
    launched = msa.profile_read()
    msa.profile_reset()
    assert "tile_attn_kernel" in launched and ("kvo_attn_kernel" not in launched) == only
    od, ld = call("decode")
    torch.cuda.synchronize()
    seen = torch.isfinite(ld)
    assert torch.equal(seen, torch.isfinite(lse)) and not bool(seen.all())
    assert bool((o[~seen] == 0).all()) and bool((lse[~seen] == ld[~seen]).all())
    assert float((lse - ld)[seen].abs().max()) <= 1e-4
    diff = (o.double() - od.double()).norm() / od.double().norm()
    assert float(diff) <= 5e-3
    # the oracle on sampled rows that attend something in every group
    full = [r for r in range(p.total_q_rows) if bool(seen[r].all())]
    rows = sorted(set(rng.choice(full, size=24).tolist() + full[:2] + full[-2:]))
    o_ref, l_ref = O.sparse_attention(x["q"], x["k"], x["v"], ids, O.layout_of(p), bk, rows=rows,
                                      fmt="e4m3" if fp8 else "bf16", input_scales=scales if fp8 else (1.0, 1.0, 1.0))
    check_outputs(o[rows].float().cpu().numpy(), lse[rows].cpu().numpy(), o_ref, l_ref, name)


@pytest.mark.parametrize("keys,kernel", [(6555, "tile_attn_kernel"), (6556, "kvo_attn_kernel")])
def test_chunk_of_few_tiles(keys, kernel):
    """300 rows appended to a context within the reach (8192 positions): past a
    length the longest tile alone takes more than the other path."""
    p = synth.packed_problem(f"chunk_{keys}", [300], [keys], num_q_heads=64, num_kv_heads=8, topk=32, seed=keys)
    x = synth.generate_numpy(p)
    q, k, v, seqs = *(to_dev(x[n]) for n in "qkv"), msa.Seqs.from_problem(p, torch.device("cuda"))
    ids = torch.from_numpy(synth.random_block_ids(p)).cuda()
    msa.profile_reset()
    msa.profile_enable(True)
    try:
        o, lse = msa.sparse_attn_prefill(q, k, v, ids, seqs, 64)
        torch.cuda.synchronize()
    finally:
        msa.profile_enable(False)
    assert {n for n in msa.profile_read() if n.endswith("attn_kernel")} == {kernel}
    msa.profile_reset()
    od, ld = msa.sparse_attn_decode(q, k, v, ids, seqs, 64)
    assert float((lse - ld).abs().max()) <= 1e-4
    assert float((o.double() - od.double()).norm() / od.double().norm()) <= 5e-3


@pytest.mark.parametrize("rows,H_q,H_kv,bk,tiles", [
    ([4245, 1500, 1517], 16, 1, 64, False),               # 128 tiles a sequence, 512 needed
    ([4245, 1500, 1517, 1100], 16, 1, 64, True),
    ([6000, 1500, 1517], 8, 8, 128, False),               # heads alone: 10 tiles a group and sequence, 256 needed
    ([6000, 1500, 1517, 1300, 1300], 8, 8, 128, True),
])
def test_split_counts_tiles_below_the_cut(rows, H_q, H_kv, bk, tiles):
    """k 4: a split needs its number of tiles below position 1024 (1280 of
    128-key blocks), whatever rows lie past."""
    p = synth.packed_problem(f"split_{len(rows)}_{H_kv}", rows, rows, num_q_heads=H_q, num_kv_heads=H_kv, block_size=bk,
                             topk=4, seed=7)
    x = synth.generate_numpy(p)
    q, k, v, seqs = *(to_dev(x[n]) for n in "qkv"), msa.Seqs.from_problem(p, torch.device("cuda"))
    ids = torch.from_numpy(synth.random_block_ids(p)).cuda()
    msa.profile_reset()
    msa.profile_enable(True)
    try:
        o, lse = msa.sparse_attn_prefill(q, k, v, ids, seqs, bk)
        torch.cuda.synchronize()
    finally:
        msa.profile_enable(False)
    assert ("tile_attn_kernel" in msa.profile_read()) == tiles
    msa.profile_reset()
    od, ld = msa.sparse_attn_decode(q, k, v, ids, seqs, bk)
    assert float((lse - ld).abs().max()) <= 1e-4
    assert float((o.double() - od.double()).norm() / od.double().norm()) <= 5e-3


@pytest.mark.parametrize("blocks", [1, 1365, 1366, 5461, 5462])
def test_reverse_index_scan_sizes(blocks):
    """Three groups: 3, 4095 and 4098 tiles around one quad of counts a thread,
    16383 and 16386 around the one-CTA scan's limit."""
    rows, keys = 40, 64 * blocks
    rows = min(rows, keys)
    g = torch.Generator(device="cuda").manual_seed(blocks)
    q, k, v = (torch.randn((n, 3, 128), dtype=torch.bfloat16, device="cuda", generator=g) for n in (rows, keys, keys))
    seqs = msa.Seqs([rows], [keys], [0], keys, torch.device("cuda"))
    local = (torch.arange(keys - rows, keys, device="cuda") // 64).view(-1, 1, 1)
    ids = (torch.rand((rows, 3, 8), device="cuda", generator=g) * local).int()       # may repeat, below the local block
    ids = torch.where((ids[..., :, None] == ids[..., None, :]).tril(-1).any(-1), -1, ids)
    ids[..., :1] = local.int()
    ids = torch.where((torch.arange(8, device="cuda") > 0) & (ids == local), -1, ids).int().contiguous()
    msa.profile_reset()
    msa.profile_enable(True)
    try:
        o, lse = msa.sparse_attn_prefill(q, k, v, ids, seqs, 64)
        torch.cuda.synchronize()
    finally:
        msa.profile_enable(False)
    assert ("kvo_scan_one_kernel" in msa.profile_read()) == (3 * blocks <= 16384)
    msa.profile_reset()
    od, ld = msa.sparse_attn_decode(q, k, v, ids, seqs, 64)
    assert float((lse - ld).abs().max()) <= 1e-4
    assert float((o.double() - od.double()).norm() / od.double().norm()) <= 5e-3
