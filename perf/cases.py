"""The workloads the library's speed is judged on.

A case is a dict of plain values: the kind of call sequence, the head shape,
the number of sequences and the ranges their lengths are drawn from.  Inputs
follow the repository's synthetic recipe: N(0, 1) tensors rounded to bf16 (or
E4M3 at scale 2^-4), with index keys of some key blocks shifted towards one
index query per group ("planted" blocks) for single long prompts.

Kinds (every pass goes through the package's public calls):
  decode   index_topk + sparse_attn_decode      a few new rows per sequence
  prefill  index_topk + sparse_attn_prefill     prompts, or chunks appended to a context
  train    the prefill pair + sparse_attn_backward + sparse_kl_backward
  dense    dense_attn                           full causal attention
  topk     block_topk                           Top-k of a score matrix
"""
import math
import random

import torch

from paper_2606_13392_amd import msa

DEVICE = "cuda"
HEAD_DIM = 128
FP8_SCALE = 2.0 ** -4          # per-tensor scale of E4M3 q, k and v

# Head shapes: 64 query heads on 8 groups with 64-key blocks, and the deployed
# shape with 64 query heads on 4 groups, 128-key blocks and 128-wide indexes.
BK64 = {"heads": 64, "kv_heads": 8, "d_idx": 64, "block": 64}
BK128 = {"heads": 64, "kv_heads": 4, "d_idx": 128, "block": 128}


def _attn(kind, shape, topk, seqs, rows, context, *, planted=0, paged=False, fp8=False, lens=0, name=None):
    """rows, context: (low, high) of a sequence's new rows and cached keys."""
    case = dict(shape, kind=kind, topk=topk, seqs=seqs, rows_lo=rows[0], rows_hi=rows[1], context_lo=context[0],
                context_hi=context[1], planted=planted, paged=paged, fp8=fp8, lens=lens)
    if name is not None:
        case["name"] = name
    return case


def listed():
    return [
        # one user's next token on a short odd-length context: launches and latency
        _attn("decode", BK64, 32, 1, (1, 1), (8208, 8208), name="decode_1x8k"),
        # a full serving batch at long context, contiguous padded cache
        _attn("decode", BK64, 32, 64, (1, 1), (131071, 131071), name="decode_64x128k"),
        # speculative decoding: 4 draft rows per sequence, ragged contexts, paged E4M3 cache
        _attn("decode", BK128, 16, 16, (4, 4), (16000, 65000), paged=True, fp8=True, lens=3, name="decode_spec_paged_fp8"),
        # a short prompt of a small model (8 query heads)
        _attn("prefill", {"heads": 8, "kv_heads": 2, "d_idx": 64, "block": 64}, 8, 1, (4096, 4096), (0, 0),
              name="prefill_4k"),
        # an ordinary long prompt
        _attn("prefill", BK64, 32, 1, (32768, 32768), (0, 0), planted=16, name="prefill_32k"),
        # a serving batch of ragged prompts written to a paged E4M3 cache
        _attn("prefill", BK128, 16, 12, (300, 9000), (0, 0), paged=True, fp8=True, lens=6, name="prefill_packed_fp8"),
        # chunked prefill: new rows appended to long cached contexts
        _attn("prefill", BK64, 48, 4, (2048, 2048), (16384, 131072), lens=2, name="prefill_chunked"),
        # the longest prompt: one million tokens
        _attn("prefill", BK64, 64, 1, (1 << 20, 1 << 20), (0, 0), planted=32, name="prefill_1m"),
        # one layer's attention in a training step at 32K
        _attn("train", BK64, 32, 1, (32768, 32768), (0, 0), planted=16, name="train_32k"),
        # a training step on packed documents of odd lengths, deployed shape
        _attn("train", BK128, 16, 8, (500, 6000), (0, 0), lens=10, name="train_packed"),
        # full attention of ragged prompts (the layers and phases without selection)
        _attn("dense", BK64, 0, 4, (1500, 8000), (0, 0), lens=11, name="dense_packed"),
        # the Top-k operator on scores the caller holds (first row of the paper's latency table)
        {"name": "block_topk_1024", "kind": "topk", "rows": 131072, "cols": 1024, "topk": 16},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "prefill", "prefill", "prefill", "train", "train", "dense", "topk"])
    if kind == "topk":
        cols = _log_uniform(rng, 64, 8192)
        rows = _log_uniform(rng, 1024, min(524288, (1 << 30) // cols))
        return {"kind": kind, "rows": rows, "cols": cols, "topk": rng.choice([8, 16, 16, 31, 32, 48, 64])}
    shape = rng.choice([BK64, BK128])
    topk = rng.choice([16, 32, 48, 64]) if shape is BK64 else rng.choice([8, 16, 16, 32])
    lens = rng.randrange(1 << 20)
    paged = kind != "dense" and rng.random() < 0.4
    fp8 = kind in ("decode", "prefill") and rng.random() < 0.35
    planted = 0
    if kind == "decode":
        seqs = _log_uniform(rng, 1, 64)
        hi = _log_uniform(rng, 2048, 131072)
        rows = (1, 1) if rng.random() < 0.7 else (2, 4)
        context = (max(512, hi // rng.choice([1, 2, 8])), hi)
    elif kind == "prefill" and rng.random() < 0.4:          # chunks on cached contexts
        seqs = _log_uniform(rng, 1, 8)
        rows = (256, _log_uniform(rng, 512, 4096))
        hi = _log_uniform(rng, 4096, 131072)
        context = (hi // 4, hi)
    elif kind == "prefill" and rng.random() < 0.5:          # one prompt
        seqs, context = 1, (0, 0)
        rows = (_log_uniform(rng, 2000, 131072),) * 2
        if rows[0] > 16384 and topk <= 32:
            planted = topk // 2
    else:                                                   # packed prompts or documents
        seqs, context = _log_uniform(rng, 1, 16), (0, 0)
        top = {"prefill": 16384, "train": 8192, "dense": 8192}[kind]
        hi = _log_uniform(rng, 512, top)
        rows = (max(64, hi // rng.choice([1, 4, 16])), hi)
    return _attn(kind, shape, topk, seqs, rows, context, planted=planted, paged=paged, fp8=fp8, lens=lens)


# ------------------------------------------------------------------ layout
def _layout(case):
    """(new rows, keys) per sequence: log-uniform in the case's ranges."""
    rng = random.Random(case["lens"])
    out = []
    for _ in range(case["seqs"]):
        q = _log_uniform(rng, case["rows_lo"], case["rows_hi"])
        c = _log_uniform(rng, case["context_lo"], case["context_hi"]) if case["context_hi"] > 0 else 0
        out.append((q, q + c))
    return [q for q, _ in out], [n for _, n in out]


def _blocks(n, block):
    return (n + block - 1) // block


def _randn(shape, g):
    return torch.randn(shape, dtype=torch.bfloat16, device=DEVICE, generator=g)


def _values(shape, g, fp8):
    """bf16 values, or E4M3 codes of them at FP8_SCALE."""
    if not fp8:
        return _randn(shape, g)
    x = torch.empty(shape, dtype=torch.uint8, device=DEVICE)
    for i in range(0, shape[0], 1 << 18):
        n = min(1 << 18, shape[0] - i)
        x[i:i + n] = (_randn((n,) + tuple(shape[1:]), g) / FP8_SCALE).to(torch.float8_e4m3fn).view(torch.uint8)
    return x


def _inputs(case, seed):
    """The tensors of one pass, from the seed alone."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(0x5EED + 1000003 * seed)
    if case["kind"] == "topk":
        return {"scores": torch.randn((case["rows"], case["cols"]), dtype=torch.float32, device=DEVICE, generator=g)}
    q_rows, kv_lens = _layout(case)
    Tq, B, H, R, D = sum(q_rows), case["block"], case["heads"], case["kv_heads"], case["d_idx"]
    x = {"q_rows": q_rows, "kv_lens": kv_lens, "kv_starts": [0] * len(kv_lens), "table": None}
    if case["paged"]:
        # pages of one key block in shuffled order, a few pages unused
        per = max(_blocks(n, B) for n in kv_lens)
        pages = sum(_blocks(n, B) for n in kv_lens) + 7
        order = torch.randperm(pages, generator=torch.Generator().manual_seed(seed)).tolist()
        table = [[0] * per for _ in kv_lens]
        at = 0
        for s, n in enumerate(kv_lens):
            for b in range(_blocks(n, B)):
                table[s][b] = order[at]
                at += 1
        x["table"] = torch.tensor(table, dtype=torch.int32, device=DEVICE)
        Tk = pages * B
    elif case["kind"] == "decode":
        pad = -(-max(kv_lens) // 64) * 64                  # a padded cache
        x["kv_starts"] = [s * pad for s in range(len(kv_lens))]
        Tk = pad * len(kv_lens)
    else:
        x["kv_starts"] = [sum(kv_lens[:s]) for s in range(len(kv_lens))]
        Tk = sum(kv_lens)
    x["Tk"] = Tk
    x["q"] = _values((Tq, H, HEAD_DIM), g, case["fp8"])
    x["k"] = _values((Tk, R, HEAD_DIM), g, case["fp8"])
    x["v"] = _values((Tk, R, HEAD_DIM), g, case["fp8"])
    if case["kind"] != "dense":
        x["index_q"] = _randn((Tq, R, D), g)
        x["index_k"] = _randn((Tk, D), g)
    if case["planted"]:
        # per group, `planted` blocks shifted towards one of its index queries (never the last block)
        rng = random.Random(seed)
        n = kv_lens[0] // B
        chosen = rng.sample(range(n - 1), case["planted"] * R)
        for r in range(R):
            u = x["index_q"][rng.randrange(Tq), r].float()
            u = 2.0 * math.sqrt(D) * u / u.norm()
            for b in chosen[r * case["planted"]:(r + 1) * case["planted"]]:
                at = _key_rows(x, case, 0, b * B, (b + 1) * B)
                x["index_k"][at] = (x["index_k"][at].float() + u).to(torch.bfloat16)
    if case["kind"] == "train":
        x["d_o"] = _randn((Tq, H, HEAD_DIM), g)
    return x


def _key_rows(x, case, s, lo, hi):
    """Key-side rows of sequence s's keys lo .. hi-1."""
    j = torch.arange(lo, hi, device=DEVICE)
    if x["table"] is None:
        return j + x["kv_starts"][s]
    B = case["block"]
    return x["table"][s].long()[j // B] * B + j % B


def prepare(case, seed):
    x = _inputs(case, seed)
    x["case"] = case
    if case["kind"] != "topk":
        x["seqs"] = msa.Seqs(x["q_rows"], x["kv_lens"], x["kv_starts"], x["Tk"], DEVICE, block_table=x["table"],
                             page_size=case["block"] if case["paged"] else 0)
    return x


def run(x):
    case = x["case"]
    kind = case["kind"]
    if kind == "topk":
        return {"ids": msa.block_topk(x["scores"], case["topk"])}
    q, k, v, seqs = x["q"], x["k"], x["v"], x["seqs"]
    if kind == "dense":
        o, lse = msa.dense_attn(q, k, v, seqs)
        return {"o": o, "lse": lse}
    B = case["block"]
    ids = msa.index_topk(x["index_q"], x["index_k"], seqs, B, case["topk"])
    scales = (FP8_SCALE,) * 3
    if kind == "decode":
        if case["fp8"]:
            o, lse = msa.sparse_attn_decode_fp8(q, k, v, scales, ids, seqs, B)
        else:
            o, lse = msa.sparse_attn_decode(q, k, v, ids, seqs, B)
    elif case["fp8"]:
        o, lse = msa.sparse_attn_prefill_fp8(q, k, v, scales, ids, seqs, B)
    else:
        o, lse = msa.sparse_attn_prefill(q, k, v, ids, seqs, B)
    out = {"ids": ids, "o": o, "lse": lse}
    if kind == "train":
        out["d_q"], out["d_k"], out["d_v"] = msa.sparse_attn_backward(q, k, v, o, lse, x["d_o"], ids, seqs, B)
        grad_scale = 1.0 / (q.shape[0] * case["kv_heads"])
        out["d_index_q"], out["d_index_k"], out["kl"] = msa.sparse_kl_backward(x["index_q"], x["index_k"], q, k, lse,
                                                                               ids, seqs, B, grad_scale=grad_scale)
    return out


# ------------------------------------------------------------------ work
def work(case):
    if case["kind"] == "topk":
        return {"bytes": 4 * case["rows"] * (case["cols"] + case["topk"]), "flops": 0}
    q_rows, kv_lens = _layout(case)
    B, H, R, D, k = case["block"], case["heads"], case["kv_heads"], case["d_idx"], case["topk"]
    Tq, Tk = sum(q_rows), sum(kv_lens)
    elem = 1 if case["fp8"] else 2
    scored = attended = selected = 0          # per group: index keys scored, keys attended, keys of selected blocks
    for q, n in zip(q_rows, kv_lens):
        p = torch.arange(n - q, n)
        lb = p // B
        if case["kind"] == "dense":
            attended += int((p + 1).sum())
            continue
        scored += int((lb * B).sum())
        # the local block up to the row itself, and up to k - 1 whole blocks
        attended += int((p - lb * B + 1 + torch.clamp(lb, max=k - 1) * B).sum())
        selected += min(n, int(((torch.clamp(lb, max=k - 1) + 1) * B).sum()))
    q_bytes = Tq * H * HEAD_DIM
    out = q_bytes * 2 + 4 * Tq * H
    if case["kind"] == "dense":
        return {"bytes": q_bytes * elem + 2 * Tk * R * HEAD_DIM * elem + out, "flops": 4 * HEAD_DIM * H * attended}
    # index tensors, ids, q, o, lse and the K / V rows that some row selects (at most every row)
    nbytes = 2 * Tq * R * D + 2 * Tk * D + 4 * Tq * R * k + q_bytes * elem + 2 * selected * R * HEAD_DIM * elem + out
    flops = 2 * D * R * scored + 4 * HEAD_DIM * H * attended
    if case["kind"] == "train":
        # gradients out, dO in; scores, dP, dV, dK, dQ; teacher scores and the student's forward and two gradients
        nbytes += 2 * (2 * q_bytes + 2 * Tk * R * HEAD_DIM + Tq * R * D + Tk * D) + 4 * Tq * R
        flops += (10 + 2) * HEAD_DIM * H * attended + 6 * D * R * attended
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------ tolerance
def tolerance(case):
    if case["kind"] == "topk":
        return "exact"                        # ranks given scores; ties keep the lower column
    # bf16 outputs and weights, gradients of sums of both signs: 2.3e-3 .. 3.0e-3 from 64 bits
    tol = {"rel": 1e-2, "max": 0.9}
    if case["kind"] != "dense":
        tol["differ"] = 1e-3                  # near-ties of fp32 scores summed in another order
    return tol


# ------------------------------------------------------------------ exact
def _wide(t, fp8):
    return t.view(torch.float8_e4m3fn).float().double() * FP8_SCALE if fp8 else t.double()


def _chunks(n, per_row):
    """Row ranges whose 64-bit score matrices take at most 2 GiB."""
    step = max(1, (1 << 28) // max(1, per_row))
    return [(i, min(n, i + step)) for i in range(0, n, step)]


def _select(case, iq, ik, p):
    """Selected blocks of rows at positions p: (mask [rows, blocks], ids [rows, k])."""
    B, k = case["block"], case["topk"]
    n = ik.shape[0]
    nb = _blocks(n, B)
    s = torch.full((iq.shape[0], nb * B), -math.inf, dtype=torch.float64, device=DEVICE)
    s[:, :n] = iq @ ik.T
    s = s.view(-1, nb, B).amax(2)
    lb = p // B
    block = torch.arange(nb, device=DEVICE)
    s = torch.where(block[None, :] < lb[:, None], s, -math.inf)
    m = block[None, :] == lb[:, None]
    if k > 1:
        top, at = s.topk(min(k - 1, nb), dim=1)
        m.scatter_(1, at, m.gather(1, at) | (top > -math.inf))
    ids = torch.where(m, block[None, :], nb).sort(1).values[:, :k]
    ids = torch.where(ids < nb, ids, -1)
    if ids.shape[1] < k:
        ids = torch.nn.functional.pad(ids, (0, k - ids.shape[1]), value=-1)
    return m, ids.to(torch.int32)


def exact(case, seed):
    if case["kind"] == "topk":
        return None                           # whole numbers alone
    q_rows, kv_lens = _layout(case)
    H, R, B, D = case["heads"], case["kv_heads"], case["block"], case["d_idx"]
    G, train = H // R, case["kind"] == "train"
    if sum(q * n for q, n in zip(q_rows, kv_lens)) * H * HEAD_DIM * (14 if train else 4) > 2e14:
        return None
    x = _inputs(case, seed)
    Tq, Tk, fp8 = sum(q_rows), x["Tk"], case["fp8"]
    new = lambda *shape: torch.zeros(shape, dtype=torch.float64, device=DEVICE)     # noqa: E731
    out = {"o": new(Tq, H, HEAD_DIM), "lse": new(Tq, H)}
    if train:
        out.update(d_q=new(Tq, H, HEAD_DIM), d_k=new(Tk, R, HEAD_DIM), d_v=new(Tk, R, HEAD_DIM),
                   d_index_q=new(Tq, R, D), d_index_k=new(Tk, D), kl=new(Tq, R))
    scale, scale_idx = 1.0 / math.sqrt(HEAD_DIM), 1.0 / math.sqrt(D)
    grad_scale = 1.0 / (Tq * R)
    first = 0
    for s, (q, n) in enumerate(zip(q_rows, kv_lens)):
        rows = _key_rows(x, case, s, 0, n)
        for r in range(R):
            k, v = _wide(x["k"][rows, r], fp8), _wide(x["v"][rows, r], fp8)
            ik = x["index_k"][rows].double() if case["kind"] != "dense" else None
            heads = slice(r * G, (r + 1) * G)
            for i, j in _chunks(q, n * G):
                at = slice(first + i, first + j)
                p = torch.arange(n - q + i, n - q + j, device=DEVICE)
                see = torch.arange(n, device=DEVICE)[None, :] <= p[:, None]
                if ik is not None:
                    iq = x["index_q"][at, r].double()
                    m, _ = _select(case, iq, ik, p)
                    see &= m.repeat_interleave(B, 1)[:, :n]
                qq = _wide(x["q"][at, heads], fp8).reshape(-1, HEAD_DIM)
                z = (qq @ k.T * scale).view(j - i, G, n).masked_fill_(~see[:, None, :], -math.inf)
                lse = torch.logsumexp(z, 2)
                w = torch.exp_(z.sub_(lse[:, :, None])).view(-1, n)
                o = w @ v
                out["o"][at, heads] = o.view(j - i, G, HEAD_DIM)
                out["lse"][at, heads] = lse
                if not train:
                    continue
                d_o = x["d_o"][at, heads].double().reshape(-1, HEAD_DIM)
                out["d_v"][rows, r] += w.T @ d_o
                ds = (d_o @ v.T).sub_((d_o * o).sum(1, keepdim=True)).mul_(w)
                out["d_q"][at, heads] = (scale * (ds @ k)).view(j - i, G, HEAD_DIM)
                out["d_k"][rows, r] += scale * (ds.T @ qq)
                del ds
                teacher = w.view(j - i, G, n).mean(1)
                student = torch.log_softmax((iq @ ik.T * scale_idx).masked_fill_(~see, -math.inf), 1)
                gap = torch.where(see & (teacher > 0), teacher * (teacher.log() - student), 0.0)
                out["kl"][at, r] = gap.sum(1)
                delta = student.exp() - teacher
                out["d_index_q"][at, r] = grad_scale * scale_idx * (delta @ ik)
                out["d_index_k"][rows] += grad_scale * scale_idx * (delta.T @ iq)
        first += q
    if case["kind"] != "dense":
        out = dict(ids=None, **out)
    return out
