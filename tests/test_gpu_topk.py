"""The Top-k operator on its own (msa_block_topk) against the CPU oracle
through the C ABI (needs an MI355X).  Ids are integer results: bit-exact on
every row the oracle ranks; at the paper's full sizes every row is also
checked for a valid selection (ascending distinct ids, each selected score
>= every unselected one)."""
from __future__ import annotations

import sys
import zlib

import numpy as np
import pytest
import torch

import oracle.msa_oracle as O
from paper_2606_13392_amd import msa, synth
from tests.util import check_block_ids, to_dev

pytestmark = pytest.mark.gpu

INF = float("inf")
POOL = [-INF, -3.0, -1.0, -0.0, 0.0, 0.25, 1.0, 2.0]


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    msa.lib()
    yield
    torch.cuda.synchronize()


# name, rows, cols, k, row stride (None: cols), value pool (None: N(0, 1)), first column
SMALL = [
    ("k16_B1000", 37, 1000, 16, None, None, 0),
    ("k64_B64", 5, 64, 64, None, None, 0),
    ("k64_B63_fewer_cols_than_k", 9, 63, 64, None, None, 0),
    ("k1_B257", 100, 257, 1, None, None, 0),
    ("k32_B2048", 64, 2048, 32, None, None, 0),
    ("k48_B300_ragged_load", 40, 300, 48, None, None, 0),
    ("ties_k8_B300", 50, 300, 8, None, POOL, 0),
    ("ties_k64_B1000", 20, 1000, 64, None, POOL, 0),
    ("ties_k16_B5000", 8, 5000, 16, None, POOL, 0),
    ("stride_512_vector_loads", 33, 500, 16, 512, None, 0),
    ("stride_503_scalar_loads", 33, 500, 16, 503, None, 0),
    ("unaligned_start_scalar_loads", 17, 300, 12, 304, None, 1),
    ("one_row_B4097", 1, 4097, 20, None, None, 0),
    ("B3_k2", 6, 3, 2, None, POOL, 0),
    ("B0", 3, 0, 4, None, None, 0),
]


@pytest.mark.parametrize("case", SMALL, ids=lambda c: c[0])
def test_block_topk_small(case):
    name, n, B, k, ld, pool, off = case
    _say(f"[block_topk] {name}: rows {n} cols {B} k {k} stride {ld} first column {off}")
    dev = torch.device("cuda", torch.cuda.current_device())
    x = synth.topk_scores(n, off + B, seed=zlib.crc32(name.encode()), device=dev, ld=ld, pool=pool)[:, off:]
    got = msa.block_topk(x, k)
    torch.cuda.synchronize()
    want = O.row_topk(x.cpu().numpy(), k)
    assert np.array_equal(got.cpu().numpy(), want)


def test_block_topk_repeated_calls_agree():
    dev = torch.device("cuda", torch.cuda.current_device())
    x = synth.topk_scores(2000, 3000, seed=5, device=dev, pool=POOL)
    a = msa.block_topk(x, 32)
    b = msa.block_topk(x, 32)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


@pytest.mark.parametrize("shape", synth.TOPK_SHAPES, ids=lambda s: f"N{s[0]}_B{s[1]}_k{s[2]}")
def test_block_topk_paper_shapes(shape):
    N, B, k = shape
    _say(f"[block_topk] paper shape N {N} B {B} k {k}")
    dev = torch.device("cuda", torch.cuda.current_device())
    x = synth.topk_scores(N, B, seed=N + B + k, device=dev)
    got = msa.block_topk(x, k)
    torch.cuda.synchronize()
    # the exact rule on ~1024 rows spread over the matrix, first and last included
    rng = np.random.default_rng(N + k)
    rows = np.unique(np.concatenate([[0, 1, N - 2, N - 1], rng.integers(0, N, size=1020)]))
    want = O.row_topk(x[torch.from_numpy(rows).to(dev)].cpu().numpy(), k)
    assert np.array_equal(got[torch.from_numpy(rows).to(dev)].cpu().numpy(), want)
    # every row: ascending distinct ids in range, selected scores dominate
    g = got.long()
    assert bool(((g >= 0) & (g < B)).all())
    assert bool((g[:, 1:] > g[:, :-1]).all())
    low = torch.gather(x, 1, g).amin(dim=1)
    x.scatter_(1, g, -INF)
    assert bool((low >= x.amax(dim=1)).all())
    _say(f"[block_topk] N {N}: {rows.size} rows exact, {N} rows valid")


@pytest.mark.parametrize("ld_pad", [0, 1])
@pytest.mark.parametrize("k", [1, 16, 40, 41, 63, 64])
def test_block_topk_row_widths(k, ld_pad):
    """Widths around each kernel variant's limit (rows in registers up to 128
    columns, rounds of 256, 512, 1024 and 2048) and k around the one from which
    a round is bounded by the lane halves' maxima: N(0, 1) rows and rows of few
    distinct values; ids equal the oracle's."""
    for B in (1, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025, 2049):
        rng = np.random.default_rng([B, k, ld_pad])
        x = rng.standard_normal((24, B)).astype(np.float32)
        x[12:] = rng.choice(np.array(POOL, dtype=np.float32), size=(12, B))
        buf = torch.zeros((24, B + ld_pad), device="cuda")
        buf[:, :B] = torch.from_numpy(x).to("cuda")
        ids = msa.block_topk(buf[:, :B], k).cpu().numpy()
        assert np.array_equal(ids, O.row_topk(x, k)), f"{B} columns, k {k}"


@pytest.mark.parametrize("k", [16, 64])
def test_block_topk_nan_columns_are_kept(k):
    """A NaN score ranks by its sign and bits (above +inf, or below -inf), in
    rows of every width alike; no column is lost to it."""
    for B in (k, k + 2, 128, 129, 300, 700, 1500, 4000):
        rng = np.random.default_rng([B, k])
        x = rng.standard_normal((12, B)).astype(np.float32)
        x[2:4, rng.choice(B, 5, replace=False)] = INF
        for row in range(1, 12):                        # 1, 3, ... NaNs of either sign, up to all columns
            at = rng.choice(B, B if row == 11 else min(B, 2 * row - 1), replace=False)
            x[row, at] = np.where(rng.random(at.size) < 0.5, np.float32("nan"), -np.float32("nan"))
        u = x.view(np.uint32).astype(np.int64)
        order = np.where(u >> 31, 0xFFFFFFFF - u, u + (1 << 31))      # no zeros among the scores
        want = np.sort(np.argsort(-order, axis=1, kind="stable")[:, :k], axis=1)
        assert np.array_equal(msa.block_topk(torch.from_numpy(x).to("cuda"), k).cpu().numpy(), want), f"{B} columns"


# name, rows, keys, H_kv, block, topk, equal keys
INDEX_CASES = [
    # few units: CTAs score 16-block pieces and write no slice maxima
    ("pieces_edge_of_slice", [130, 40], [64 * 64 + 1, 65 * 64], 2, 64, 16, False),
    ("pieces_ties_pruned_scan", [140], [1100 * 64], 1, 64, 8, True),
    ("rows_of_127_to_129_blocks", [200], [129 * 128 + 5], 4, 128, 40, False),
    ("rows_of_511_to_513_blocks", [140], [513 * 64 + 40], 2, 64, 64, False),
    ("rows_of_1023_to_1025_blocks", [140], [1025 * 64 + 40], 2, 64, 33, False),
    ("units_of_many_sequences", [33, 0, 70, 1, 129, 64, 65] * 10, [300, 5, 900, 64, 129, 64, 2000] * 10, 8, 64, 5, False),
    # decode: waves of 4 blocks, one wave per row up to 2048 blocks, 16 beyond
    ("decode_piece_edges", [1, 2, 1, 1, 1], [1, 256 + 64, 5 * 64, 64 * 64 + 1, 512 * 64 + 7], 8, 64, 16, False),
    ("decode_one_wave_ties", [1, 1, 1], [513 * 64 + 9, 1025 * 64 + 9, 130], 4, 64, 64, True),
    ("decode_one_wave_k64", [1, 1], [2049 * 64, 1030 * 64], 8, 64, 64, False),
    ("decode_16_waves", [1, 1], [2050 * 64, 2100 * 64 + 3], 4, 64, 17, False),
    ("decode_16_waves_ties", [1], [2200 * 64 + 3], 2, 64, 48, True),
    ("decode_wide_pieces", [1, 3, 1], [77 * 128 + 1, 128 * 9, 300], 4, 128, 12, False),
    # wave kernel: one CTA per CU up to 512 of them, more beyond; units numbered without gaps up to 128 sequences
    ("wave_one_cta_per_cu", [4, 1, 7, 4, 0, 3], [600 * 64 + 9, 64, 7, 100 * 64, 0, 1000], 32, 64, 16, False),
    ("wave_wide_one_cta_per_cu", [4, 1, 7, 2], [70 * 128 + 9, 128, 7, 1000], 16, 128, 16, False),
    ("units_of_128_sequences", [4, 1, 0, 3] * 32, [300, 64, 5, 200] * 32, 32, 64, 4, False),
    ("units_of_129_sequences", [4, 1, 0, 3] * 32 + [4], [300, 64, 5, 200] * 32 + [900], 32, 64, 4, False),
    ("wave_many_ctas", [4, 1, 7, 4] * 30, [300 * 64 + 9, 64, 7, 1000] * 30, 16, 64, 16, False),
    ("decode_many_units_slices", [1] * 200, [256 * 64 + 5] + [700] * 199, 8, 64, 8, False),
]


@pytest.mark.parametrize("case", INDEX_CASES, ids=[c[0] for c in INDEX_CASES])
def test_index_topk_paths(case):
    name, rows, keys, H_kv, bk, topk, equal = case
    p = synth.packed_problem(name, rows, keys, num_q_heads=H_kv, num_kv_heads=H_kv, block_size=bk, topk=topk,
                             seed=zlib.crc32(name.encode()) % 10000)
    x = synth.generate_numpy(p)
    if equal:
        x["index_k"][:] = x["index_k"][:1]
    lay = O.layout_of(p)
    pick = sorted(set(range(p.total_q_rows)) & set(np.linspace(0, p.total_q_rows - 1, 60).astype(int).tolist()))
    seqs = msa.Seqs.from_problem(p, torch.device("cuda"))
    ids = msa.index_topk(to_dev(x["index_q"]), to_dev(x["index_k"]), seqs, bk, topk).cpu().numpy()[pick]
    want, gaps = O.select_blocks(x["index_q"], x["index_k"], lay, bk, topk, rows=pick)
    if equal:
        assert np.array_equal(ids, want)
    else:
        check_block_ids(ids, want, gaps, x, lay, bk, topk, rows=pick)
