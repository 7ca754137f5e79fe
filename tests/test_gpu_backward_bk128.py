"""Main Branch backward on 128-key blocks: passes of 64 gathered (query, head)
rows, so group sizes that do not divide 64, tiles around one pass and one work
item (256 queries), partly visible blocks and rows that attend nothing,
against the oracle with the gradient bars of tests/util.py."""
from __future__ import annotations

import pytest

import oracle.msa_oracle as O
from paper_2606_13392_amd import msa
from tests.test_gpu_backward import _check_all, _gpu, _run, _setup  # noqa: F401  (_gpu: the module's fixture)

pytestmark = pytest.mark.gpu

# name, q_rows, kv_lens, H_q, H_kv, topk, kv_pad_to, block_size
CASES = [
    ("bwd_wide_g1", [200], [200], 2, 2, 2, None, 128),
    ("bwd_wide_g3", [150], [150], 6, 2, 4, None, 128),
    ("bwd_wide_g5_chunked", [90, 13], [300, 260], 10, 2, 3, None, 128),
    ("bwd_wide_g7", [129], [129], 7, 1, 2, None, 128),
    ("bwd_wide_g9", [70], [500], 9, 1, 4, None, 128),
    ("bwd_wide_g16_one_pass", [4, 5, 3], [4, 5, 3], 16, 1, 1, None, 128),
    ("bwd_wide_item_edges", [256, 257, 255], [256, 257, 255], 8, 1, 3, None, 128),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_backward_bk128(case):
    p, x, ids = _setup(*case)
    ids[::17] = -1
    got = list(_run(p, x, ids))
    _check_all(case[0], got, O.sparse_attention_backward(x["q"], x["k"], x["v"], x["d_o"], ids, O.layout_of(p), p.block_size))


@pytest.mark.parametrize("rows", [1, 2, 63, 1023, 1024, 1025, 2500])
def test_backward_reproducible_list_lengths(rows):
    """Block 0 is listed by every row: handle lists of `rows` entries, ordered
    in registers up to 1024 and through the scratch list beyond.  dK and dV add
    a list in its order, so three runs agree bit for bit."""
    p, x, ids = _setup(f"bwd_list_{rows}", [rows, 70], [rows, 70], 8, 2, 40, None, 64)
    first, *rest = (list(_run(p, x, ids)) for _ in range(3))
    for r in rest:
        assert all((a == b).all() for a, b in zip(first, r))


@pytest.mark.parametrize("bk,kernel", [(64, "bwd_kvo_kernel"), (128, "bwd_kvo_wide_kernel")])
def test_backward_kernel_by_block_size(bk, kernel):
    p, x, ids = _setup("bwd_names", [70], [70], 4, 2, 2, None, bk)
    msa.profile_reset()
    msa.profile_enable(True)
    try:
        list(_run(p, x, ids))
    finally:
        msa.profile_enable(False)
    assert {n for n in msa.profile_read() if n.startswith("bwd_kvo")} == {kernel}
    msa.profile_reset()
