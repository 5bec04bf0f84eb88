"""GPU parity of the kernels whose waves own whole query heads, over the head
counts they serve: 16- and 32-token tiles (contexts of one token, one short of and one past
a tile, several tiles, several batches of page-table entries), KV heads that
split over the token streams of a workgroup and KV heads that do not, pages
of one tile and more, and scores that climb so that the softmax reference
moves in the middle of a piece. The pool's memory is filled with NaN first:
rows past a context must not reach any output."""
import math

import numpy as np
import pytest
import torch

import oracle
from parity import LSE_MAX_ABS, OUT_MAX_ABS, OUT_REL_L2
from test_gpu_rescale import _inputs
from paper_2606_24506_amd import crosspool as cpl
from workloads.gen import ModelSpec
from workloads.harness import to_device_u16

pytestmark = pytest.mark.gpu


def gqa(heads, kv, d=128):
    return ModelSpec(f"gqa{heads}x{kv}d{d}", "gqa", heads, kv, head_dim=d, scale=1 / math.sqrt(d))


def mla(heads):
    return ModelSpec(f"mla{heads}", "mla", heads, 1, latent_dim=512, rope_dim=64, scale=1 / math.sqrt(192.0))


def run(specs_lens, page_tokens, schedule, splits, kind="staircase", seed=3):
    """Decodes one request per (spec, length) and compares each with the
    oracle, at the bars of every parity test here."""
    need = sum(-(-n // page_tokens) for _, n in specs_lens)
    pool_bytes = (2 << 20) * (need + 16)
    mem = torch.full((pool_bytes // 2,), 0x7FC0, dtype=torch.int16, device="cuda")  # bf16 NaN
    pool = cpl.Pool(page_tokens=page_tokens, pool_bytes=pool_bytes, placement_seed=seed, device=0, device_mem=mem)
    mids, rids, rows, qs = {}, [], [], []
    for r, (m, n) in enumerate(specs_lens):
        if m.name not in mids:
            mids[m.name] = pool.register_spec(m)
        rids.append(pool.open(mids[m.name], n))
        rw, q, _ = _inputs(m, n, 100 * seed + r, kind)
        rows.append(rw)
        qs.append(q)
        pool.append([rids[-1]], [n], to_device_u16(rw, "cuda"))
    q = to_device_u16(np.concatenate([x.reshape(-1) for x in qs]), "cuda")
    out = torch.zeros(sum(m.n_q_heads * m.d_v for m, _ in specs_lens), dtype=torch.int16, device="cuda")
    lse = torch.zeros(sum(m.n_q_heads for m, _ in specs_lens), dtype=torch.float32, device="cuda")
    pool.decode(rids, q, out, lse, num_splits=splits, schedule=schedule)
    torch.cuda.synchronize()
    o_at = l_at = 0
    for (m, n), rw, qb in zip(specs_lens, rows, qs):
        got = out[o_at:o_at + m.n_q_heads * m.d_v].cpu().numpy().view(np.uint16).reshape(m.n_q_heads, m.d_v)
        got = oracle.bf16_bits_to_f64(got)
        o_ref, l_ref = oracle.decode(rw, qb, m)
        got_l = lse[l_at:l_at + m.n_q_heads].cpu().numpy().astype(np.float64)
        o_at += m.n_q_heads * m.d_v
        l_at += m.n_q_heads
        where = (m.name, n, page_tokens, schedule, splits)
        assert np.isfinite(got).all() and np.isfinite(got_l).all(), where
        d = got - o_ref
        assert np.abs(d).max() <= OUT_MAX_ABS, (where, np.abs(d).max())
        assert np.sqrt((d * d).sum() / (o_ref * o_ref).sum()) <= OUT_REL_L2, where
        assert np.abs(got_l - l_ref).max() <= LSE_MAX_ABS, (where, np.abs(got_l - l_ref).max())
    for r in rids:
        pool.close(r)
    pool.destroy()


BAL, QUE = cpl.CP_SCHED_BALANCED, cpl.CP_SCHED_QUEUE
LENS = [1, 31, 33, 64, 95, 700]


# 64 heads per KV head: two streams, one KV head each (2 KV heads) or
# interleaved tiles (1 or 3); 128: one stream of eight waves
@pytest.mark.parametrize("heads,kv", [(64, 1), (128, 2), (192, 3), (128, 1), (256, 2)])
@pytest.mark.parametrize("page_tokens,schedule,splits", [(64, BAL, 0), (32, QUE, 1), (96, QUE, 3)])
def test_many_heads_per_kv_head(heads, kv, page_tokens, schedule, splits):
    print(f"[case] {heads}:{kv} P{page_tokens} sched{schedule} s{splits}", flush=True)
    m = gqa(heads, kv)
    run([(m, n) for n in LENS], page_tokens, schedule, splits)


def test_many_heads_long_pieces():
    """Unsplit pieces of more than 64 and 128 pages, and two variants in one launch."""
    run([(gqa(64, 1), 2100), (gqa(128, 1), 4300), (gqa(128, 2), 2081)], 32, QUE, 1)


# groups of every kind: 1-4 heads, odd ones, a full unit of 16, two units and
# more; KV heads that fill the eight streams, share them, or are odd
@pytest.mark.parametrize("heads,kv,d", [(8, 8, 64), (16, 4, 64), (40, 8, 64), (6, 1, 64), (32, 8, 128), (16, 16, 128),
                                        (21, 3, 128), (28, 4, 128), (30, 6, 128), (12, 1, 128), (40, 2, 128),
                                        (100, 1, 128)])
@pytest.mark.parametrize("page_tokens,schedule,splits", [(64, BAL, 0), (32, QUE, 1), (96, QUE, 3)])
def test_any_group(heads, kv, d, page_tokens, schedule, splits):
    print(f"[case] {heads}:{kv} d{d} P{page_tokens} sched{schedule} s{splits}", flush=True)
    m = gqa(heads, kv, d)
    run([(m, n) for n in [1, 15, 17, 32, 33, 64, 150, 700]], page_tokens, schedule, splits)


def test_any_group_long_pieces():
    """Unsplit pieces of more than 64 and 128 pages, both head widths in one launch."""
    run([(gqa(28, 4), 2100), (gqa(16, 8, 64), 4300), (gqa(8, 1), 2081), (gqa(12, 12, 64), 2115)], 32, QUE, 1)


# MLA: one unit of 16 (padded), head pairs in two streams (to 32) or one (to
# 64), several units of 64; pages of 16 and 48 tokens take units of 16
@pytest.mark.parametrize("heads", [6, 15, 17, 20, 32, 33, 64, 100, 144])
@pytest.mark.parametrize("page_tokens,schedule,splits", [(64, BAL, 0), (32, QUE, 1), (48, QUE, 3)])
def test_any_mla_head_count(heads, page_tokens, schedule, splits):
    print(f"[case] MLA-{heads} P{page_tokens} sched{schedule} s{splits}", flush=True)
    run([(mla(heads), n) for n in [1, 15, 17, 32, 33, 64, 95, 500]], page_tokens, schedule, splits)


def test_any_mla_head_count_long_pieces():
    """Unsplit pieces of more than 64 and 128 pages, variants sharing a launch."""
    run([(mla(20), 2100), (mla(64), 4300), (mla(7), 2081), (mla(32), 2115)], 32, QUE, 1)


def test_mla_128_on_small_pages():
    """128 heads on pages that 32-token tiles do not fit: units of 16 heads."""
    run([(mla(128), n) for n in (1, 17, 300)], 16, BAL, 0)


@pytest.mark.parametrize("g", [4, 5])
def test_split_probabilities_keep_fp32_precision(g):
    """Probabilities are multiplied as the sum of two bf16 numbers. With V
    equal to a constant (a power of two) in every row the output is that
    constant times (sum of the operands) / (sum of the fp32 probabilities):
    each operand pair is within 2^-17 of its probability, so the result
    rounds to the constant exactly, and an infinite V stays infinite."""
    hq = 4 * g
    m, n = gqa(hq, 4), 1000
    rng = np.random.default_rng(1)
    rows = rng.standard_normal((n, m.row_width), dtype=np.float32)
    rows[:, 4 * 128:] = 0.5
    rows[:, 4 * 128 + 7] = np.inf
    bits = (rows.view(np.uint32) >> 16).astype(np.uint16)
    pool = cpl.Pool(page_tokens=64, pool_bytes=64 << 20, device=0)
    rid = pool.open(pool.register_spec(m), n)
    pool.append([rid], [n], to_device_u16(bits, "cuda"))
    q = to_device_u16((rng.standard_normal((hq, 128), dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16), "cuda")
    out = torch.zeros(hq * 128, dtype=torch.int16, device="cuda")
    lse = torch.zeros(hq, dtype=torch.float32, device="cuda")
    pool.decode([rid], q, out, lse)
    torch.cuda.synchronize()
    got = out.view(torch.bfloat16).float().cpu().numpy().reshape(hq, 128)
    expect = np.full((hq, 128), 0.5, dtype=np.float32)
    expect[:g, 7] = np.inf  # the heads of KV head 0
    assert np.array_equal(got, expect)
    pool.close(rid)
    pool.destroy()
