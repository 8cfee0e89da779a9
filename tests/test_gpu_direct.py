"""GPU parity of staged requests at the edges of the rule that moves short and fragmented ones directly
(at most 32 MiB, or 256 MiB in copies averaging under 2 MiB), bit-exact against the CPU oracle, with the route each
took read off its launch count; direct and staged requests ordered against each other on one stream; and
the no-allocation restore by either route, also captured into a graph.

The layout has 1 KiB per token and 256 KiB per chunk: 32,768 tokens are 32 MiB, and a 16-chunk batch of
consecutive slots is one 4 MiB copy."""
import numpy as np
import pytest
import torch

import harness
from paper_2609_15021_amd import kvx
from tests.gpu_support import (DEV, TINY, bt_tensor, device_cache, first_mismatch, host_cache, oracle_pool,
                               oracle_unpack_into, to_device, to_host)

pytestmark = pytest.mark.gpu

EDGE = 32768  # tokens in 32 MiB
NB = EDGE // 16 + 160


def _expected(n, ids, slots, seed):
    A = host_cache(TINY, NB, seed, "raw")
    nblk = TINY.nblk(n)
    btA, btB = harness.block_table(seed + 1, NB, nblk), harness.block_table(seed + 2, NB, nblk)
    pool = oracle_pool(TINY, A, btA, n, ids, slots, 0)
    return A, btA, btB, pool, oracle_unpack_into(TINY, np.zeros_like(A), btB, n, pool, ids)


def _launches(pool):
    torch.cuda.synchronize()
    return [kvx.kv_pool_kernel_stats(pool, w, reset=True)[0] for w in ("pack", "unpack")]


# Slot runs of `run` consecutive chunks (8 are a 2 MiB copy); a pool with chunks_per_batch keeps DMA copies.
@pytest.mark.parametrize("n,run,batch,direct", [
    (EDGE, 128, 0, True), (EDGE + 1, 136, 0, False), (EDGE + 2048, 8, 0, False), (EDGE + 2048, 7, 0, True),
    (EDGE + 1, 1, 0, True), (1, 1, 0, True), (EDGE, 128, 16, False), (300, 1, 16, False)])
def test_direct_rule_edges(n, run, batch, direct):
    nc = TINY.nc(n)
    # Ascending runs in reverse order of slots, so that no two of them join.
    starts = range(0, nc, run)
    ids = np.concatenate([nc - min(a + run, nc) + np.arange(min(run, nc - a)) for a in starts])
    A, btA, btB, want_pool, want_B = _expected(n, ids, nc, harness.sub_seed("direct", n, run))
    pool = kvx.kv_pool_create(TINY.kv, nc, "staged", chunks_per_batch=batch, profile=True)
    view = kvx.pool_view(pool)
    view[:] = 0
    dA, dB = to_device(A), device_cache(TINY, NB, fill=0)
    tA, tB = bt_tensor(btA), bt_tensor(btB)
    torch.cuda.synchronize()
    kvx.kv_store(kvx.Cache(dA, TINY.kv, NB), tA, n, pool, ids)
    torch.cuda.synchronize()
    assert np.array_equal(view, want_pool), first_mismatch(view, want_pool)
    kvx.kv_load(kvx.Cache(dB, TINY.kv, NB), tB, n, pool, ids)
    batches = 1 if direct else -(-nc // 16)
    assert _launches(pool) == [batches, batches]
    assert np.array_equal(to_host(dB, A), want_B)
    dB.zero_()
    torch.cuda.synchronize()
    kvx.kv_load_noalloc(kvx.Cache(dB, TINY.kv, NB), tB, n, pool, ids)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(dB, A), want_B)
    assert kvx.kv_pool_async_error(pool) == 0
    kvx.kv_pool_destroy(pool)


@pytest.mark.parametrize("kind", [kvx.KV_HOST_COHERENT, kvx.KV_HOST_NONCOHERENT])
def test_direct_and_staged_requests_are_ordered_on_one_stream(kind):
    """No host wait in between: direct stores of quarters, a staged load of all of them, a staged store of
    another cache over the same slots, then a direct load of a quarter.  Kernels and copy engines take turns on the
    same bytes, in coherent memory and in memory that the GPU may cache."""
    n, nc = EDGE + 4096, TINY.nc(EDGE + 4096)
    ids = np.arange(nc)
    seed = harness.sub_seed("direct", "mixed")
    nb = TINY.nblk(n) + 32
    A, A2 = host_cache(TINY, nb, seed, "raw"), host_cache(TINY, nb, seed + 9, "raw")
    bt = harness.block_table(seed + 1, nb, TINY.nblk(n))
    pool = kvx.kv_pool_create(TINY.kv, nc, "staged", host_kind=kind)
    dA, dA2 = to_device(A), to_device(A2)
    t = bt_tensor(bt)
    q = nc // 4 * 256
    s = torch.cuda.Stream()
    for rep in range(5):
        B, B2 = device_cache(TINY, nb, fill=0), device_cache(TINY, nb, fill=0)
        kvx.pool_view(pool)[:] = 0
        torch.cuda.synchronize()
        dA, dA2 = dA2, dA  # no byte keeps its value from one repeat to the next
        for k in range(4):
            kvx.kv_store(kvx.Cache(dA, TINY.kv, nb), t[k * q // 16:], q, pool, ids[k * q // 256:], s)
        kvx.kv_load(kvx.Cache(B, TINY.kv, nb), t, n, pool, ids, s)
        kvx.kv_store(kvx.Cache(dA2, TINY.kv, nb), t, n, pool, ids, s)
        kvx.kv_load(kvx.Cache(B2, TINY.kv, nb), t, q, pool, ids, s)
        s.synchronize()
        used, first = torch.from_numpy(bt.astype(np.int64)).to(DEV), TINY.nblk(q)
        assert torch.equal(B[:, used], dA[:, used]), f"rep {rep}: the staged load missed a direct store"
        assert torch.equal(B2[:, used[:first]], dA2[:, used[:first]]), f"rep {rep}: the direct load missed a staged store"
    kvx.kv_pool_destroy(pool)


@pytest.mark.parametrize("batch", [0, 2])
def test_noalloc_short_request_replays_under_graph_capture(batch):
    """Captured by either route (direct, and through the scratch with chunks_per_batch set)."""
    n, nc = 4096 + 77, TINY.nc(4096 + 77)
    ids = harness.chunk_ids(nc, nc + 2, 5)
    A, btA, btB, want_pool, want_B = _expected(n, ids, nc + 2, harness.sub_seed("direct", "graph"))
    pool = kvx.kv_pool_create(TINY.kv, nc + 2, "staged", chunks_per_batch=batch)
    kvx.pool_view(pool)[:] = want_pool
    dB = device_cache(TINY, NB, fill=0)
    cache, tB = kvx.Cache(dB, TINY.kv, NB), bt_tensor(btB)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    kvx.kv_load_noalloc(cache, tB, n, pool, ids, s)  # the first call on a device looks up its scratch
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        kvx.kv_load_noalloc(cache, tB, n, pool, ids, s)
    for rep in range(3):
        dB.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(to_host(dB, A), want_B), f"replay {rep}"
    del g
    kvx.kv_pool_destroy(pool)


@pytest.mark.parametrize("page,direct", [(1 << 20, True), ((1 << 20) + 16, False)])
def test_snapshot_rule_edges(page, direct):
    """Four consecutive snapshots of 8 pages: 32 MiB, and just more (one copy)."""
    G, n = 8, 4
    pool = kvx.kv_pool_create(TINY.kv, 256, "staged", profile=True, num_state_slots=n, state_slot_bytes=G * page)
    src = torch.randint(0, 256, (G, n, page), dtype=torch.uint8, device=DEV)
    dst = torch.zeros_like(src)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    kvx.kv_store_state(kvx.State(src, page, n), [0, 1, 2, 3], pool, [0, 1, 2, 3], s)
    kvx.kv_load_state(kvx.State(dst, page, n), [3, 2, 1, 0], pool, [3, 2, 1, 0], s)
    s.synchronize()
    assert torch.equal(src, dst)
    want = src.transpose(0, 1).reshape(-1).cpu().numpy()
    assert np.array_equal(kvx.state_view(pool), want)
    # A staging slot of 16 x 256 KiB takes nine batches, each one timed launch group.
    assert [kvx.kv_pool_kernel_stats(pool, w)[0] for w in ("state_pack", "state_unpack")] == [1 if direct else 9] * 2
    kvx.kv_pool_destroy(pool)
