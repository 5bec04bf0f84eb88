"""The balanced schedule's plan of a launch (cost_line.hpp, compiled here with
g++): every block of every request lies in exactly one range, no range is
empty, batches of whole pages are cut where a line of 8 KiB units cuts them,
and finer ranges are taken only where they shorten the longest share."""
import ctypes
import os
import random
import shutil
import subprocess
from dataclasses import dataclass

import pytest

from paper_2606_24506_amd import build

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no C++ compiler")


@dataclass(frozen=True)
class Model:
    kappa: int        # KV bytes per token
    step: int         # tokens the kernel works through at once
    weight: int = 8   # time per KiB, eighths
    out: int = 0      # output elements of a request
    rereads: int = 1


# kinds of models with the steps and weights of their kernels
MLA16 = Model(1152, 64, out=16 * 512)
MLA20 = Model(1152, 64, 11, 20 * 512)
MLA64 = Model(1152, 32, 18, 64 * 512)
MLA200 = Model(1152, 32, 18, 200 * 512, 4)
MQA32 = Model(512, 128, out=32 * 128)
MQA128 = Model(512, 32, 10, 128 * 128)
GQA32X4 = Model(2048, 32, out=32 * 128)
GQA32X8 = Model(4096, 16, out=32 * 128)
GQA64X8 = Model(4096, 32, out=64 * 128)
GQA16X4D64 = Model(1024, 64, out=16 * 64)
SLOTS = 256


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("cost_line") / "shim.so")
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "c", "cost_line_shim.cpp")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I", build.CSRC, src, "-o", out],
                   check=True)
    lib = ctypes.CDLL(out)
    lib.cost_line.restype = ctypes.c_int64
    return lib


def plan(lib, reqs, page_tokens=64, slots=SLOTS, whole=False):
    """reqs: [(Model, tokens)] -> (workers, total, [(blk_tokens, blk_cost, begin, first, ranges)])"""
    n = len(reqs)
    i32 = lambda v: (ctypes.c_int32 * n)(*v)
    out, total = (ctypes.c_int64 * (5 * n))(), ctypes.c_int64()
    w = lib.cost_line(n, (ctypes.c_int64 * n)(*[t for _, t in reqs]), i32([page_tokens] * n), i32([m.step for m, _ in reqs]),
                      i32([m.kappa for m, _ in reqs]), i32([m.rereads for m, _ in reqs]), i32([m.weight for m, _ in reqs]),
                      i32([m.out for m, _ in reqs]), slots, int(whole), out, ctypes.byref(total))
    return w, total.value, [tuple(out[5 * i:5 * i + 5]) for i in range(n)]


def pieces(reqs, ln):
    """[(request, worker, first token, end token)], as the kernels find them."""
    workers, total, per = ln
    got = []
    for r, ((_, tokens), (blk, cost, begin, first, ranges)) in enumerate(zip(reqs, per)):
        nb = -(-tokens // blk)
        for w in range(max(0, first - 1), min(workers, first + ranges + 1)):
            lo, hi = w * total // workers, (w + 1) * total // workers
            jb = max(0, -(-(lo - begin) // cost))
            je = min(nb, -(-(hi - begin) // cost)) if begin < hi else 0
            if jb < je:
                got.append((r, w, jb * blk, min(tokens, je * blk)))
        assert [w for q, w, _, _ in got if q == r] == list(range(first, first + ranges))
    return got


def whole_pages_by_8_kib(reqs, page_tokens, slots=SLOTS):
    """Ranges per request of a line of 8 KiB units, worked out from its definition."""
    cost = [page_tokens * m.kappa // 8192 * m.rereads for m, _ in reqs]
    nb = [-(-t // page_tokens) for _, t in reqs]
    bare = sum(c * k for c, k in zip(cost, nb))
    w0 = max(1, min(slots, bare // max(cost)))
    begin, at, pre = [], 0, 0
    for i, (c, k) in enumerate(zip(cost, nb)):
        if i and pre * w0 % bare:
            at += 40
        begin.append(at)
        at += c * k
        pre += c * k
    workers = max(1, min(slots, at // max(cost)))
    share = [w * at // workers for w in range(workers + 1)]
    got = []
    for r, (c, k, b) in enumerate(zip(cost, nb, begin)):
        for w in range(workers):
            pages = [j for j in range(k) if share[w] <= b + j * c < share[w + 1]] if b + k * c > share[w] else []
            if pages:
                got.append((r, w, pages[0] * page_tokens, min(reqs[r][1], (pages[-1] + 1) * page_tokens)))
    return got


def random_batch(rng, models, n, hi):
    return [(rng.choice(models), int(2 ** rng.uniform(0, hi))) for _ in range(n)]


@pytest.mark.parametrize("models,page_tokens", [
    ([MLA16], 64), ([MLA16, MQA32, GQA32X4], 64), ([MLA16], 32), ([MLA16], 128), ([GQA32X8], 64), ([GQA64X8, MQA32], 64),
    ([GQA32X8, GQA16X4D64], 64), ([MLA20, MLA64, GQA32X8], 64), ([MQA128, GQA32X4], 64), ([MLA200], 128), ([MQA32], 1)])
def test_ranges_cover_every_request_once(shim, models, page_tokens):
    rng = random.Random(1)
    for k in range(60):
        reqs = random_batch(rng, models, rng.randint(1, 64), 14)
        for whole in (False, True):
            ln = plan(shim, reqs, page_tokens, slots=rng.choice([1, 7, 256]), whole=whole)
            assert ln[1] < 1 << 32
            at = [0] * len(reqs)
            for r, _, lo, hi in pieces(reqs, ln):
                assert lo == at[r] and hi > lo
                at[r] = hi
            assert at == [t for _, t in reqs]


@pytest.mark.parametrize("models,page_tokens", [([MLA16], 64), ([MLA16, MQA32, GQA32X4], 64), ([MQA32, GQA32X4], 32)])
def test_pages_of_8_kib_multiples_keep_their_ranges(shim, models, page_tokens):
    """Launches that nothing makes finer: the ranges, and so the bits of the
    results, are those of a line that counts 8 KiB units."""
    rng = random.Random(2)
    for k in range(40):
        reqs = random_batch(rng, models, rng.randint(1, 64), 15)
        assert pieces(reqs, plan(shim, reqs, page_tokens)) == whole_pages_by_8_kib(reqs, page_tokens)


def longest_share(reqs, ln):
    """KiB-times of the workgroup that has most, each piece with its fixed cost."""
    share = {}
    for r, w, lo, hi in pieces(reqs, ln):
        m = reqs[r][0]
        share[w] = share.get(w, 0) + (hi - lo) * m.kappa * m.rereads * m.weight / 8 / 1024 + 320
    return max(share.values())


@pytest.mark.parametrize("models,page_tokens,hi", [
    ([MLA16], 128, 11), ([GQA64X8], 64, 12), ([GQA32X8, GQA16X4D64], 64, 11), ([MLA20, MLA64, GQA32X8], 64, 12),
    ([MQA128, GQA32X4], 64, 14), ([MLA200], 128, 10), ([MLA16, MQA32, GQA32X4], 128, 12),
    ([Model(512, 8, out=64), Model(65536, 8, out=64)], 16, 10)])
def test_finer_ranges_never_lengthen_the_longest_share(shim, models, page_tokens, hi):
    rng = random.Random(3)
    finer = 0
    for k in range(120):
        reqs = random_batch(rng, models, rng.randint(1, 48), hi)
        ln, whole = plan(shim, reqs, page_tokens), plan(shim, reqs, page_tokens, whole=True)
        if ln != whole:
            finer += 1
            assert longest_share(reqs, ln) < longest_share(reqs, whole)
    assert finer > 0


def split_outputs(reqs, ln):
    return sum(m.out for (m, _), p in zip(reqs, ln[2]) if p[4] > 1)


@pytest.mark.parametrize("models,page_tokens,hi", [
    ([MLA16], 128, 10), ([GQA64X8], 64, 9), ([GQA32X8, GQA16X4D64], 64, 10), ([MLA20, MLA64, GQA32X8], 64, 9)])
def test_more_ranges_split_no_more_outputs(shim, models, page_tokens, hi):
    """Short batches: a request summed in one piece on whole pages is not cut
    into bf16 partials for the sake of more ranges."""
    rng = random.Random(4)
    finer = 0
    for k in range(150):
        reqs = random_batch(rng, models, rng.randint(1, 12), hi)
        ln, whole = plan(shim, reqs, page_tokens), plan(shim, reqs, page_tokens, whole=True)
        if ln[0] > whole[0]:
            finer += 1
            assert split_outputs(reqs, ln) <= split_outputs(reqs, whole)
    assert finer > 0
    one_page = [(models[0], page_tokens - 1)] * 6
    assert split_outputs(one_page, plan(shim, one_page, page_tokens)) == 0


def test_half_pages_are_not_cut_for_nothing(shim):
    """MLA-16 on 128-token pages (two blocks each), half a page to a page for
    every workgroup: cut, the longest share stays a page, or grows to three
    blocks, and there are more partials."""
    for lens in ([18000 // 16] * 16, [28000 // 16] * 16, [1100] * 16, [140 * k for k in range(1, 18)]):
        reqs = [(MLA16, t) for t in lens]
        assert plan(shim, reqs, 128) == plan(shim, reqs, 128, whole=True)


def kernel_of(spec):
    """A model spec as the plan sees it, with the step and weight of its kernel."""
    if spec.kind == "mla":
        step, weight, blocks = (64, 8, 1) if spec.n_q_heads <= 16 else (64, 11, 1) if spec.n_q_heads <= 32 else (32, 18, 64)
        rereads = -(-spec.n_q_heads // blocks) if blocks > 1 else 1
        return Model(1152, step, weight, spec.n_q_heads * 512, rereads)
    hkv, g, d = spec.n_kv_heads, spec.n_q_heads // spec.n_kv_heads, spec.head_dim
    rereads, weight = 1, 8
    if d == 128 and g in (8, 16, 32):
        step = 32 if hkv % 4 == 0 else 128
    elif d == 128 and g in (64, 128):
        step, weight = (32, 10) if g == 128 else (32 if hkv % 2 == 0 else 64, 8)
    else:
        step, rereads = (16 if d == 128 else 32) * 8 // min(8, hkv & -hkv), -(-g // 16)
    return Model(4 * hkv * d, step, weight, spec.n_q_heads * d, rereads)


def test_gpu_batches_have_finer_ranges(shim):
    """The batches by which the GPU tests mean to reach ranges inside pages, and
    launches shared by time, do so."""
    from test_gpu_subpage_ranges import BY_TIME, CUT, cut_lens, step_lens

    for spec, P in CUT:
        reqs = [(kernel_of(spec), n) for n in cut_lens(P)]
        ln = plan(shim, reqs, P)
        assert ln != plan(shim, reqs, P, whole=True) and ln[2][0][0] < P, (spec.name, P)
    for spec, P in [c for c in CUT if c[0].name in ("gqa32x8d128", "gqa64x8d128", "mla64")]:
        reqs = [(kernel_of(spec), n + 2) for n in step_lens(P)]  # the second of three steps
        assert plan(shim, reqs, P)[2][0][0] < P, (spec.name, P)
    for batch in BY_TIME:
        reqs = [(kernel_of(spec), n) for spec, n in batch]
        ln = plan(shim, reqs, 64)
        assert ln[0] == SLOTS and ln != plan(shim, reqs, 64, whole=True)
