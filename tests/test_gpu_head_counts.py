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


@pytest.mark.parametrize("model", [gqa(32, 8), gqa(20, 4), gqa(16, 4, 64), gqa(30, 1, 64), mla(12), mla(20), mla(32),
                                   mla(64), mla(100)], ids=lambda m: m.name)
def test_probabilities_keep_fp32_precision(model):
    """Probabilities enter P.V whole (as three bf16 operands). Tokens come in
    pairs of V = +1 and -1 whose scores differ by d = 2^-11.5 to 2^-10.5, so
    the output is -tanh(d / 2), the small difference of nearly equal sums:
    rounding p to 8 bits moves it by as much as itself, and two operands, which
    leave up to 2^-16 of p out, by 2^-5 to 2^-6. What fp32 leaves: the output's
    own rounding (up to 2^-8) and an error of each p of at most 2^-21 or so
    (scores of magnitude 4, two units of the last place), 2^-9.5 of d: together
    below 2^-7. One range per request, so no bf16 partials."""
    hd, lens = model.d_k, (2, 10, 48)
    rng = np.random.default_rng(7)
    off = 512 if model.kind == "mla" else 0     # the score comes from two dimensions, for MLA from rotary ones
    hkv = 1 if model.kind == "mla" else model.n_kv_heads
    specs, rows_all, q_all = [], [], []
    for n in lens:
        k = np.zeros((n, hkv, hd), dtype=np.float32)
        base = rng.uniform(-4, 0, size=(n // 2, hkv)).repeat(2, axis=0)
        k[:, :, off + 1] = base / model.scale
        k[1::2, :, off] = 0.25
        v = np.tile(np.where(np.arange(n) % 2, -1.0, 1.0)[:, None, None], (1, hkv, 1)).astype(np.float32)
        if model.kind == "mla":
            k[:, :, :512] = v
            rows = k.reshape(n, -1)
        else:
            rows = np.concatenate([k.reshape(n, -1), np.broadcast_to(v, (n, hkv, hd)).reshape(n, -1)], axis=1)
        q = np.zeros((model.n_q_heads, hd), dtype=np.float32)
        q[:, off + 1] = rng.uniform(0.5, 1, model.n_q_heads)
        q[:, off] = rng.uniform(1, 2, model.n_q_heads) * 2.0 ** -9.5 / model.scale
        rows_all.append((rows.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16))
        q_all.append((q.view(np.uint32) >> 16).astype(np.uint16))
    pool = cpl.Pool(page_tokens=64, pool_bytes=64 << 20, device=0)
    mid = pool.register_spec(model)
    rids = [pool.open(mid, n) for n in lens]
    for r, rw in zip(rids, rows_all):
        pool.append([r], [rw.shape[0]], to_device_u16(rw, "cuda"))
    out = torch.zeros(len(lens) * model.n_q_heads * model.d_v, dtype=torch.int16, device="cuda")
    lse = torch.zeros(len(lens) * model.n_q_heads, dtype=torch.float32, device="cuda")
    pool.decode(rids, to_device_u16(np.concatenate([x.reshape(-1) for x in q_all]), "cuda"), out, lse, num_splits=1,
                schedule=QUE)
    torch.cuda.synchronize()
    got = oracle.bf16_bits_to_f64(out.cpu().numpy().view(np.uint16)).reshape(len(lens), model.n_q_heads, model.d_v)
    worst = 0.0
    for g, rw, qb in zip(got, rows_all, q_all):
        ref, _ = oracle.decode(rw, qb, model)
        assert np.abs(ref).max() < 2.0 ** -11 and np.abs(ref).min() > 2.0 ** -13
        worst = max(worst, float((np.abs(g - ref) / np.abs(ref)).max()))
    print(f"[precision] {model.name} 2^{np.log2(worst):.2f}", flush=True)
    assert worst <= 2.0 ** -7
    for r in rids:
        pool.close(r)
    pool.destroy()


@pytest.mark.parametrize("model", [gqa(16, 4), gqa(20, 4), gqa(16, 4, 64), mla(12), mla(20), mla(64)], ids=lambda m: m.name)
def test_infinite_values_stay_infinite(model):
    """V constant (a power of two) in every row but for one infinite column:
    the output is that constant exactly, and infinity, not NaN."""
    n, d_v = 1000, model.d_v
    rng = np.random.default_rng(1)
    rows = rng.standard_normal((n, model.row_width), dtype=np.float32)
    q = rng.standard_normal((model.n_q_heads, model.d_k), dtype=np.float32)
    v0 = 0 if model.kind == "mla" else model.n_kv_heads * d_v
    rows[:, v0:v0 + (d_v if model.kind == "mla" else model.n_kv_heads * d_v)] = 0.5
    rows[:, v0 + 7] = np.inf
    if model.kind == "mla":
        q[:, :512] = 0.25
        q[:, 7] = 0  # 0 * inf would be the score
        rows[:, 7] = 0.5  # (an infinite latent value is an infinite key as well)
    bits = (rows.view(np.uint32) >> 16).astype(np.uint16)
    pool = cpl.Pool(page_tokens=64, pool_bytes=64 << 20, device=0)
    rid = pool.open(pool.register_spec(model), n)
    pool.append([rid], [n], to_device_u16(bits, "cuda"))
    qb = (q.view(np.uint32) >> 16).astype(np.uint16)
    out = torch.zeros(model.n_q_heads * d_v, dtype=torch.int16, device="cuda")
    lse = torch.zeros(model.n_q_heads, dtype=torch.float32, device="cuda")
    pool.decode([rid], to_device_u16(qb, "cuda"), out, lse)
    torch.cuda.synchronize()
    expect = np.full((model.n_q_heads, d_v), 0.5, dtype=np.float32)
    if model.kind != "mla":
        expect[:model.n_q_heads // model.n_kv_heads, 7] = np.inf  # the heads of KV head 0
    assert np.array_equal(out.view(torch.bfloat16).float().cpu().numpy().reshape(expect.shape), expect)
    pool.close(rid)
    pool.destroy()


@pytest.mark.parametrize("model", [gqa(64, 1), gqa(128, 1), gqa(32, 8), gqa(28, 1), gqa(16, 4, 64), mla(12), mla(20),
                                   mla(64)], ids=lambda m: m.name)
def test_nan_keys_reach_output_and_lse(model):
    """Keys of NaN in one 32-token tile (one stream has nothing else): the
    heads that read them have NaN outputs and a NaN lse."""
    n = 64
    rng = np.random.default_rng(2)
    rows = rng.standard_normal((n, model.row_width), dtype=np.float32)
    rows[32:, 512 if model.kind == "mla" else 0] = np.nan  # a rotary element, or one of KV head 0's keys
    q = rng.standard_normal((model.n_q_heads, model.d_k), dtype=np.float32)
    pool = cpl.Pool(page_tokens=64, pool_bytes=64 << 20, device=0)
    rid = pool.open(pool.register_spec(model), n)
    pool.append([rid], [n], to_device_u16((rows.view(np.uint32) >> 16).astype(np.uint16), "cuda"))
    out = torch.zeros(model.n_q_heads * model.d_v, dtype=torch.int16, device="cuda")
    lse = torch.zeros(model.n_q_heads, dtype=torch.float32, device="cuda")
    pool.decode([rid], to_device_u16((q.view(np.uint32) >> 16).astype(np.uint16), "cuda"), out, lse, num_splits=1,
                schedule=QUE)
    torch.cuda.synchronize()
    hit = torch.arange(model.n_q_heads) < model.n_q_heads // (1 if model.kind == "mla" else model.n_kv_heads)
    got = out.view(torch.bfloat16).float().cpu().view(model.n_q_heads, model.d_v)
    assert torch.isnan(got[hit]).all() and torch.isfinite(got[~hit]).all()
    assert torch.isnan(lse.cpu()[hit]).all() and torch.isfinite(lse.cpu()[~hit]).all()
    pool.close(rid)
    pool.destroy()
