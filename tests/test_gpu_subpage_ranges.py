"""Balanced schedules that cut ranges inside pages (models whose pages hold more
than 128 KiB): every kernel family that serves such models, against the
oracle, and decode steps whose fused append meets such ranges, bit for bit
against append and decode."""
import numpy as np
import pytest
import torch

from paper_2606_24506_amd import crosspool as cpl
from parity import LSE_MAX_ABS, OUT_REL_L2
from test_gpu_head_counts import BAL, gqa, mla, run
from workloads.harness import to_device_u16

pytestmark = pytest.mark.gpu

LENS = [1, 31, 33, 65, 130, 257, 700]
CUT = [(gqa(32, 8), 64), (gqa(16, 16), 64), (gqa(30, 6), 128), (gqa(32, 16, 64), 128), (gqa(64, 8), 64),
       (gqa(32, 1), 512), (gqa(128, 2), 256), (gqa(256, 2), 192), (mla(16), 128), (mla(12), 256), (mla(20), 128),
       (mla(64), 128), (mla(32), 192)]


def cut_lens(P):
    """Contexts of more than a page (a batch with one-page contexts stays on
    whole pages): test_cost_line.py checks that these are cut inside pages."""
    return [P + 1, P + 31, P + P // 2, 2 * P - 1, 2 * P + 33, 3 * P + P // 2 + 3, 5 * P - 2, 700 + P]


def step_lens(P):
    return [2 * P - 1, 2 * P, 2 * P + P // 2 + 3, 5 * P - 2]


BY_TIME = [[(gqa(40, 8), 8000), (mla(64), 4100), (mla(20), 1), (gqa(40, 8), 5003), (mla(20), 2501), (gqa(28, 4), 65)],
           [(gqa(128, 1), 9000), (gqa(128, 2), 31), (gqa(128, 2), 8001), (gqa(64, 8), 7010), (gqa(128, 1), 64)]]


@pytest.mark.parametrize("model,page_tokens", CUT, ids=lambda x: getattr(x, "name", x))
def test_ranges_inside_pages(model, page_tokens):
    print(f"[case] {model.name} P{page_tokens}", flush=True)
    run([(model, n) for n in LENS], page_tokens, BAL, 0)
    run([(model, n) for n in cut_lens(page_tokens)], page_tokens, BAL, 0)


def test_models_of_different_blocks_in_one_launch():
    run([(gqa(32, 8), 700), (mla(20), 300), (gqa(28, 4), 500), (mla(64), 129), (gqa(32, 8), 65)], 64, BAL, 0)


@pytest.mark.parametrize("model,page_tokens", [(gqa(32, 8), 64), (gqa(64, 8), 64), (mla(16), 256), (mla(64), 128)],
                         ids=lambda x: getattr(x, "name", x))
@pytest.mark.parametrize("first", [1, 2])
def test_fused_step_over_ranges_inside_pages(model, page_tokens, first):
    """Contexts around page ends and in the middle of a page, with a one-page
    one (ranges of whole pages) and without; the step and the two calls it
    stands for run on two pools holding the same rows."""
    lens = step_lens(page_tokens)
    lens[:2] = [first * page_tokens - 1, first * page_tokens]
    rng = np.random.default_rng(3)
    rows = [rng.standard_normal((n + 3, model.row_width), dtype=np.float32) for n in lens]
    bits = [(x.view(np.uint32) >> 16).astype(np.uint16) for x in rows]
    q = rng.standard_normal((len(lens), model.n_q_heads, model.d_k), dtype=np.float32)
    q = to_device_u16((q.view(np.uint32) >> 16).astype(np.uint16), "cuda")
    pools = [cpl.Pool(page_tokens=page_tokens, pool_bytes=128 << 20, placement_seed=s, device=0) for s in (2, 9)]
    res = [[], []]
    for k, pool in enumerate(pools):
        mid = pool.register_spec(model)
        ids = [pool.open(mid, n + 3) for n in lens]
        for r, n in zip(range(len(lens)), lens):
            pool.append([ids[r]], [n], to_device_u16(bits[r][:n], "cuda"))
        for t in range(3):
            new = to_device_u16(np.concatenate([b[n + t] for b, n in zip(bits, lens)]), "cuda")
            out = torch.zeros(len(lens) * model.n_q_heads * model.d_v, dtype=torch.int16, device="cuda")
            lse = torch.zeros(len(lens) * model.n_q_heads, dtype=torch.float32, device="cuda")
            if k == 0:
                pool.decode_step(ids, [1] * len(lens), new, q, out, lse)
            else:
                pool.append(ids, [1] * len(lens), new)
                pool.decode(ids, q, out, lse)
            torch.cuda.synchronize()
            res[k].append((out, lse))
        for r in ids:
            pool.close(r)
        pool.destroy()
    for (o0, l0), (o1, l1) in zip(*res):
        assert torch.equal(o0, o1) and torch.equal(l0.view(torch.int32), l1.view(torch.int32))


@pytest.mark.parametrize("specs_lens,page_tokens", [
    # pages of 144 KiB: cut inside pages the call has 256 ranges (52 MB of
    # partials), of whole pages 150 (31 MB)
    ([(mla(200), 150 * 128)], 128),
    # shared by time, and by bytes, every workgroup has a range of each model
    ([(mla(200), 140 * 128), (gqa(40, 8), 700)], 128),
    ([(gqa(32, 8), 700), (mla(64), 900)], 64)], ids=["mla200", "mla200+gqa40", "within"])
def test_noalloc_plans_as_decode_does(specs_lens, page_tokens):
    """The fixed 40 MiB workspace holds the partials of these batches on ranges
    of whole pages, not of finer ones (or, the last one, holds both): the call
    is accepted and its results are decode's, bit for bit."""
    gen = torch.Generator(device="cuda").manual_seed(4)
    bits = lambda k: torch.randn(k, device="cuda", generator=gen).to(torch.bfloat16).view(torch.int16)
    pool = cpl.Pool(page_tokens=page_tokens, pool_bytes=128 << 20, placement_seed=2, device=0)
    rids = []
    for m, n in specs_lens:
        rids.append(pool.open(pool.register_spec(m), n))
        pool.append([rids[-1]], [n], bits(n * m.row_width))
    q = bits(sum(m.n_q_heads * m.d_k for m, _ in specs_lens))
    res = []
    for call in (pool.decode, pool.decode_noalloc):
        out = torch.zeros(sum(m.n_q_heads * m.d_v for m, _ in specs_lens), dtype=torch.int16, device="cuda")
        lse = torch.zeros(sum(m.n_q_heads for m, _ in specs_lens), dtype=torch.float32, device="cuda")
        call(rids, q, out, lse)
        torch.cuda.synchronize()
        res.append((out, lse))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1].view(torch.int32), res[1][1].view(torch.int32))
    for r in rids:
        pool.close(r)
    pool.destroy()


def test_capped_workspace_falls_back_to_whole_pages():
    """Six 300-token requests on 256 KiB pages: 30 ranges of whole pages, about
    120 cut inside them. A pool whose max_workspace_bytes holds the partials
    of 30 takes every decode call, with one plan for all of them, and the
    result of a pool without a cap (each within the oracle's bars, so within
    twice that of one another)."""
    m, n, k = gqa(32, 8), 300, 6
    cap = 30 * m.n_q_heads * (2 * m.d_v + 4)
    gen = torch.Generator(device="cuda").manual_seed(5)
    bits = lambda c: torch.randn(c, device="cuda", generator=gen).to(torch.bfloat16).view(torch.int16)
    rows, q = [bits(n * m.row_width) for _ in range(k)], bits(k * m.n_q_heads * m.d_k)
    res = []
    for limit in (cap, 0):
        pool = cpl.Pool(page_tokens=64, pool_bytes=64 << 20, placement_seed=2, device=0, max_workspace_bytes=limit)
        mid = pool.register_spec(m)
        ids = [pool.open(mid, n + 8) for _ in range(k)]
        for r, x in zip(ids, rows):
            pool.append([r], [n], x)
        calls = [pool.decode, pool.decode_noalloc, lambda *a: pool.decode_step(ids, [0] * k, None, *a[1:]),
                 lambda *a: pool.decode_layers(ids, [0] * k, None, *a[1:])]
        for call in calls:
            out = torch.zeros(k * m.n_q_heads * m.d_v, dtype=torch.int16, device="cuda")
            lse = torch.zeros(k * m.n_q_heads, dtype=torch.float32, device="cuda")
            call(ids, q, out, lse)
            torch.cuda.synchronize()
            res.append((out, lse))
        for r in ids:
            pool.close(r)
        pool.destroy()
    for g in (res[:4], res[4:]):
        for o, l in g[1:]:
            assert torch.equal(o, g[0][0]) and torch.equal(l.view(torch.int32), g[0][1].view(torch.int32))
    (o0, l0), (o1, l1) = [(o.view(torch.bfloat16).double(), l.double()) for o, l in (res[0], res[4])]
    assert torch.linalg.norm(o0 - o1) <= 2 * OUT_REL_L2 * torch.linalg.norm(o1)
    assert (l0 - l1).abs().max() <= 2 * LSE_MAX_ABS


def test_models_sharing_a_launch_by_time():
    """Launches with work for every workgroup, of models whose kernels take
    different times per byte: ranges of every length, boundaries of every
    cost, with and without sub-page blocks."""
    run([(gqa(40, 8), 6000), (mla(64), 2100), (mla(20), 1), (gqa(40, 8), 5003), (mla(20), 1501), (gqa(28, 4), 65)], 64,
        BAL, 0)
    for batch in BY_TIME:
        run(batch, 64, BAL, 0)
