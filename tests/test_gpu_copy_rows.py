"""Appends and gathers, bit for bit, over what decides how a workgroup copies
its rows: page sizes that a workgroup's rows divide, straddle or hold several
of, row widths from 128 bytes to more than one pass of the workgroup, KV-head
counts that are no power of two, several KV planes, appends that start in the
middle of a page, and appends whose new page-table entries fit the launch
(up to 352) or need a copy of their own."""
import numpy as np
import pytest
import torch

from paper_2606_24506_amd import crosspool as cpl
from workloads.harness import to_device_u16

pytestmark = pytest.mark.gpu

GEOMS = {
    "mla": dict(kind=cpl.CP_KIND_MLA, n_q_heads=16, n_kv_heads=1, latent_dim=512, rope_dim=64, softmax_scale=0.1),
    "mha1d64": dict(kind=cpl.CP_KIND_GQA, n_q_heads=1, n_kv_heads=1, head_dim=64),
    "gqa3d128": dict(kind=cpl.CP_KIND_GQA, n_q_heads=6, n_kv_heads=3, head_dim=128),
    "gqa5d256": dict(kind=cpl.CP_KIND_GQA, n_q_heads=5, n_kv_heads=5, head_dim=256),
    "mha52d128": dict(kind=cpl.CP_KIND_GQA, n_q_heads=52, n_kv_heads=52, head_dim=128),
}


@pytest.mark.parametrize("page_tokens", [1, 2, 6, 16, 48, 64, 150])
@pytest.mark.parametrize("layers", [1, 2])
def test_appends_and_gathers_bit_exact(page_tokens, layers):
    """Chunks of 1 to 700 tokens per call, two requests of each model; the
    larger calls open more than 352 pages at two tokens per page."""
    print(f"[case] copy P{page_tokens} layers {layers}", flush=True)
    skip = {1: "mla", 150: "mha52d128"}  # pages of no multiple of 256 bytes, or larger than a chunk
    names = [n for n in GEOMS if n != skip.get(page_tokens)]
    pool = cpl.Pool(page_tokens=page_tokens, pool_bytes=600 << 20, placement_seed=5, device=0)
    mids = {n: pool.register(**GEOMS[n], n_layers=layers) for n in names}
    reqs = [n for n in names for _ in range(2)]
    total = 1000
    rids = [pool.open(mids[n], total) for n in reqs]
    width = [pool.info(mids[n])["row_elems"] for n in reqs]
    rng = np.random.default_rng(page_tokens)
    rows = [rng.integers(0, 1 << 16, size=(layers, total, w), dtype=np.uint16) for w in width]
    pos = [0] * len(reqs)
    for most in (1, 3, 40, 700, 256):
        ids, counts, flat = [], [], []
        for r, rid in enumerate(rids):
            k = min(int(rng.integers(0, most + 1)), total - pos[r])
            ids.append(rid)
            counts.append(k)
            flat.append(rows[r][:, pos[r]:pos[r] + k].reshape(-1))
            pos[r] += k
        pool.append(ids, counts, to_device_u16(np.concatenate(flat), "cuda"))
    for r, rid in enumerate(rids):
        n = pos[r]
        assert pool.ctx_len(rid) == n
        for a, b in ((0, n), (n // 3, n), (n // 2, n // 2 + 1)):
            if b <= a:
                continue
            dst = torch.zeros(layers * (b - a) * width[r], dtype=torch.int16, device="cuda")
            pool.gather(rid, a, b - a, dst)
            got = dst.cpu().numpy().view(np.uint16).reshape(layers, b - a, width[r])
            assert np.array_equal(got, rows[r][:, a:b]), (reqs[r], a, b)
    for rid in rids:
        pool.close(rid)
    pool.destroy()
