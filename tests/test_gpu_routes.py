"""Requests that a staged pool keeps on the DMA engines although they are short or fragmented: because its owner
asked for it, or because they are long.  The route of stores and loads is read off their launch count, that of the
no-allocation restore off the copies in a captured graph.

(The layout is that of the direct route's other tests: 1 KiB per token, 256 KiB per chunk.)"""
import numpy as np
import pytest
import torch

import harness
from paper_2609_15021_amd import kvx
from tests.gpu_support import DEV, TINY, bt_tensor, copies_in_graph, device_cache, first_mismatch, to_device, to_host
from tests.test_gpu_direct import EDGE, NB, _expected, _launches

pytestmark = pytest.mark.gpu


def _make(how, nc):
    """A staged pool that keeps every request on the DMA engines, or one that does not, made or switched so."""
    if how == "mode":
        return kvx.kv_pool_create(TINY.kv, nc, "staged_dma", profile=True)
    if how == "mode, one chunk a batch":
        return kvx.kv_pool_create(TINY.kv, nc, "staged_dma", chunks_per_batch=1, profile=True)
    pool = kvx.kv_pool_create(TINY.kv, nc, "zero_copy", staging_slots=2, profile=True,
                              chunks_per_batch=4 if "batch" in how else 0)
    kvx.kv_pool_set_mode(pool, "staged_dma" if "switched mode" in how else "staged")
    return pool


# Twenty chunks in scattered slots: twenty copies, and a launch per batch where requests stay on the DMA engines.
@pytest.mark.parametrize("how,launches,copies,direct_bytes", [
    ("mode", 2, 20, 32 << 20), ("mode, one chunk a batch", 20, 20, 0), ("switched mode", 2, 20, 32 << 20),
    ("switched, batch at creation", 2, 20, 0), ("switched", 1, 0, 32 << 20)])
def test_requests_kept_on_the_dma_engines(how, launches, copies, direct_bytes):
    """The mode that keeps every request on the DMA engines, given at creation or later, and chunks_per_batch, given
    to a pool that is created zero-copy and switched."""
    n, ids = 20 * 256 - 11, np.arange(38, -1, -2)
    A, btA, btB, want_pool, want_B = _expected(n, ids, 39, harness.sub_seed("direct", "kept"))
    pool = _make(how, 39)
    info = kvx.kv_pool_get_info(pool)
    assert info["direct_bytes"] == direct_bytes
    want_mode = kvx.KV_MODE_STAGED_DMA if "mode" in how else kvx.KV_MODE_STAGED
    assert info["mode"] == info["load_mode"] == want_mode
    view = kvx.pool_view(pool)
    view[:] = 0
    dA, dB = to_device(A), device_cache(TINY, NB, fill=0)
    tA, tB = bt_tensor(btA), bt_tensor(btB)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    kvx.kv_store(kvx.Cache(dA, TINY.kv, NB), tA, n, pool, ids, s)
    s.synchronize()
    assert np.array_equal(view, want_pool), first_mismatch(view, want_pool)
    kvx.kv_load(kvx.Cache(dB, TINY.kv, NB), tB, n, pool, ids, s)
    assert _launches(pool) == [launches, launches]
    assert np.array_equal(to_host(dB, A), want_B)
    dB.zero_()
    torch.cuda.synchronize()
    cB = kvx.Cache(dB, TINY.kv, NB)
    kvx.kv_load_noalloc(cB, tB, n, pool, ids, s)
    s.synchronize()
    assert np.array_equal(to_host(dB, A), want_B)
    assert copies_in_graph(lambda: kvx.kv_load_noalloc(cB, tB, n, pool, ids, s), s) == copies
    kvx.kv_pool_destroy(pool)


@pytest.mark.parametrize("n,direct", [(8 * EDGE, True), (8 * EDGE + 1, False)])
def test_long_fragmented_requests_stay_on_the_dma_engines(n, direct):
    """Scattered 256 KiB chunks, 256 MiB and one token more: what is stored comes back, by launches of 256 chunks
    over the link or of 16 in staging."""
    nc, nblk = TINY.nc(n), TINY.nblk(n)
    ids = np.arange(2 * nc - 2, -1, -2)
    pool = kvx.kv_pool_create(TINY.kv, 2 * nc, "staged", profile=True)
    src = torch.randint(-(1 << 15), 1 << 15, (2, nblk, 2, 2, 16, 64), dtype=torch.int16, device=DEV)
    dst = torch.zeros_like(src)
    tA = bt_tensor(harness.block_table(11, nblk, nblk))
    tB = bt_tensor(harness.block_table(12, nblk, nblk))
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    kvx.kv_store(kvx.Cache(src, TINY.kv, nblk), tA, n, pool, ids, s)
    kvx.kv_load(kvx.Cache(dst, TINY.kv, nblk), tB, n, pool, ids, s)
    want = -(-nc // (256 if direct else 16))
    assert _launches(pool) == [want, want]
    got, stored = dst[:, tB.long()], src[:, tA.long()]
    used = n - (nblk - 1) * 16  # tokens in the last block
    stored[:, -1, :, :, used:] = 0
    assert torch.equal(got, stored)
    c = kvx.Cache(dst, TINY.kv, nblk)
    copies = copies_in_graph(lambda: kvx.kv_load_noalloc(c, tB, n, pool, ids, s), s)
    assert copies == (0 if direct else nc)
    kvx.kv_pool_destroy(pool)
