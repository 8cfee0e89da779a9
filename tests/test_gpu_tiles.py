"""GPU parity of the gather kernels at the edges of their tiles (256 vectors of 16 bytes), bit-exact
against the CPU oracle: slabs of a wave's 64 vectors, one below and above, of a tile, one above it, and
smaller than any of these; planes that end inside a wave, at a tile's end and just after it; both block
orders; block ids outside the cache among valid ones.  Host pool (zero-copy) and device pool."""
import numpy as np
import pytest
import torch

import harness
import oracle
from paper_2609_15021_amd import build, kvx
from tests.gpu_support import DEV, Layout, bt_tensor, first_mismatch

pytestmark = pytest.mark.gpu

POOL_SENT, CACHE_SENT = 0xA5, 0x5A
ORDERS = {kvx.KV_BLOCK_HND: oracle.BLOCK_HND, kvx.KV_BLOCK_NHD: oracle.BLOCK_NHD}

# (L, H, D, E, BS, C): vectors of a slab are BS*H*D*E/16.
LAYOUTS = {
    "slab 1": (2, 1, 16, 1, 1, 64),
    "slab 63": (1, 3, 112, 1, 3, 12),
    "slab 64": (2, 2, 64, 2, 4, 32),
    "slab 65": (1, 5, 104, 2, 1, 7),
    "slab 192": (2, 3, 64, 2, 8, 64),
    "slab 256": (1, 4, 64, 1, 16, 64),
    "slab 257": (1, 1, 2056, 2, 1, 3),
    "slab 320": (1, 5, 64, 2, 8, 16),
    "slab 2048": (1, 8, 128, 2, 16, 32),
}


def _device_words(pool):
    info = kvx.kv_pool_get_info(pool)

    class View:
        __cuda_array_interface__ = dict(shape=(info["pool_bytes"],), typestr="|u1",
                                        data=(info["device_base"], False), version=2)
    return torch.as_tensor(View(), device=DEV)


@pytest.mark.parametrize("where", ["zero_copy", "device"])
@pytest.mark.parametrize("order", [kvx.KV_BLOCK_HND, kvx.KV_BLOCK_NHD])
@pytest.mark.parametrize("name", LAYOUTS)
def test_tile_edges(name, order, where):
    lay = Layout(*LAYOUTS[name])
    token_vecs = lay.H * lay.D * lay.E // 16
    # Whole chunks, a last chunk of one token, and last chunks whose plane ends next to a wave's or a tile's end.
    tails = {1, lay.C - 1} | {min(lay.C - 1, max(1, e // token_vecs + d)) for e in (64, 256, 512) for d in (-1, 0, 1)}
    for n in [lay.C, 3 * lay.C] + sorted(2 * lay.C + t for t in tails if t > 0):
        print(f"[tiles] {name} order={order} {where} n={n}", flush=True)
        _check(lay, order, where, n, bad=False)
    _check(lay, order, where, 2 * lay.C + lay.BS, bad=True)


def _check(lay, order, where, n, bad):
    seed = harness.sub_seed("tiles", lay.L, lay.H, lay.D, lay.E, lay.BS, n)
    rng = np.random.default_rng(seed)
    nc, nblk = lay.nc(n), lay.nblk(n)
    NB, slots = nblk + 3, nc + 1
    A = [rng.integers(0, 256, NB * lay.block_bytes, dtype=np.uint8) for _ in range(lay.L)]
    table = harness.block_table(seed + 1, NB, nblk)
    ids = harness.chunk_ids(nc, slots, seed + 2)
    want = np.full(slots * lay.slot_bytes, POOL_SENT, dtype=np.uint8)
    assert oracle.pack(lay.orc, A, lay.block_bytes, NB, table, n, want, ids, 4, block_order=ORDERS[order]) == oracle.OK
    to = harness.block_table(seed + 3, NB, nblk)
    back = [np.full(NB * lay.block_bytes, CACHE_SENT, dtype=np.uint8) for _ in range(lay.L)]
    assert oracle.unpack(lay.orc, back, lay.block_bytes, NB, to, n, want, ids, 4, block_order=ORDERS[order]) == oracle.OK
    table, to = table.copy(), to.copy()
    stored = want
    if bad:
        # Every third block is named by an id outside the cache: its rows are stored as zeros, its destination
        # is left alone.
        hit = np.arange(0, nblk, 3)
        table[hit] = np.where(hit % 2, -1, NB)
        stored = want.copy()
        for i in range(nc):
            r = min(lay.C, n - i * lay.C)
            planes = stored[ids[i] * lay.slot_bytes:][:r * lay.token_bytes].reshape(2 * lay.L, r, -1)
            for j in range(-(-r // lay.BS)):
                if (i * (lay.C // lay.BS) + j) in set(hit):
                    planes[:, j * lay.BS:(j + 1) * lay.BS] = 0
        for l in range(lay.L):
            back[l].reshape(NB, -1)[to[hit]] = CACHE_SENT
        to[hit] = np.where(hit % 2, NB + 7, -5)

    if where == "device":
        pool = kvx.kv_pool_create(lay.kv, slots, "zero_copy", host_kind=kvx.KV_POOL_DEVICE)
        view = _device_words(pool)
    else:
        pool = kvx.kv_pool_create(lay.kv, slots, "zero_copy")
        view = torch.from_numpy(kvx.pool_view(pool))
    view.fill_(POOL_SENT)
    dA = [torch.from_numpy(a).to(DEV) for a in A]
    dB = [torch.full((NB * lay.block_bytes,), CACHE_SENT, dtype=torch.uint8, device=DEV) for _ in range(lay.L)]
    tA, tB = bt_tensor(table), bt_tensor(to)
    torch.cuda.synchronize()
    kvx.kv_store(kvx.Cache(dA, lay.kv, NB, 0, order), tA, n, pool, ids)
    torch.cuda.synchronize()
    got = view.cpu().numpy().copy()
    assert np.array_equal(got, stored), f"n={n} pool: " + first_mismatch(got, stored)
    assert kvx.kv_pool_async_error(pool, clear=True) == (kvx.KV_ASYNC_BAD_BLOCK if bad else 0)
    view.copy_(torch.from_numpy(want))
    torch.cuda.synchronize()
    kvx.kv_load(kvx.Cache(dB, lay.kv, NB, 0, order), tB, n, pool, ids)
    torch.cuda.synchronize()
    for l in range(lay.L):
        got = dB[l].cpu().numpy()
        assert np.array_equal(got, back[l]), f"n={n} cache layer {l}: " + first_mismatch(got, back[l])
    assert kvx.kv_pool_async_error(pool) == (kvx.KV_ASYNC_BAD_BLOCK if bad else 0)
    del view
    kvx.kv_pool_destroy(pool)


@pytest.mark.parametrize("where", ["zero_copy", "device"])
@pytest.mark.parametrize("order", [kvx.KV_BLOCK_HND, kvx.KV_BLOCK_NHD])
@pytest.mark.parametrize("name", LAYOUTS)
def test_planes_beyond_the_limits_of_a_launch(name, order, where, monkeypatch):
    """A build of the library in which planes of any size find their blocks as those of 32 GiB and more do, and
    planes of more than 3 tiles are launched as those of 64 GiB and more are."""
    monkeypatch.setattr(kvx, "_lib", kvx._open(build.LIB_LIMITS))
    lay = Layout(*LAYOUTS[name])
    plane = lay.H * lay.D * lay.E * lay.C
    for n in (1, lay.C, 2 * lay.C + 1, 3 * lay.C - 1):
        print(f"[limits] {name} order={order} {where} n={n} tiles={-(-plane // 4096)}", flush=True)
        _check(lay, order, where, n, bad=False)
    _check(lay, order, where, 2 * lay.C + lay.BS, bad=True)


@pytest.mark.parametrize("where", ["zero_copy", "device", "staged"])
@pytest.mark.parametrize("page", [16, 1008, 1024, 1040, 4080, 4096, 4112, 8176, 12304, 65424, 65520])
def test_snapshot_piece_edges(page, where):
    """Pages of one vector, next to a wave's 1 KiB and a piece's 4 KiB, and of several pieces; padded
    pages, more snapshots than one launch carries.  (Staged: a staging slot of 2 KiB, under a piece.)"""
    G, n, stride = 3, 130, page + 48
    lay = Layout(1, 1, 16, 1, 8, 64)
    rng = np.random.default_rng(harness.sub_seed("pieces", page))
    A = rng.integers(0, 256, (G, n + 2, stride), dtype=np.uint8)
    pages, slots = rng.permutation(n + 2)[:n], rng.permutation(n + 1)[:n]
    want = np.full((n + 1) * G * page, POOL_SENT, dtype=np.uint8)
    layers = [np.ascontiguousarray(A[g]).reshape(-1) for g in range(G)]
    assert oracle.state_pack(layers, page, stride, pages, want, slots) == oracle.OK
    back = [np.full((n + 2) * stride, CACHE_SENT, dtype=np.uint8) for _ in range(G)]
    to = rng.permutation(n + 2)[:n]
    assert oracle.state_unpack(back, page, stride, to, want, slots) == oracle.OK
    area = dict(num_state_slots=n + 1, state_slot_bytes=G * page)
    if where == "device":
        pool = kvx.kv_pool_create(lay.kv, 1, "zero_copy", host_kind=kvx.KV_POOL_DEVICE, **area)
        info = kvx.kv_pool_get_info(pool)

        class View:
            __cuda_array_interface__ = dict(shape=(want.size,), typestr="|u1", version=2,
                                            data=(info["device_base"] + -(-info["pool_bytes"] // 4096) * 4096, False))
        view = torch.as_tensor(View(), device=DEV)
    else:
        batch = 1 if where == "staged" else 0
        pool = kvx.kv_pool_create(lay.kv, 1, where, chunks_per_batch=batch, **area)
        view = torch.from_numpy(kvx.state_view(pool))
    view.fill_(POOL_SENT)
    dA = torch.from_numpy(A).to(DEV)
    dB = torch.full_like(dA, CACHE_SENT)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    kvx.kv_store_state(kvx.State(dA, page, n + 2, stride), pages, pool, slots, s)
    s.synchronize()
    assert np.array_equal(view.cpu().numpy(), want), first_mismatch(view.cpu().numpy(), want)
    kvx.kv_load_state(kvx.State(dB, page, n + 2, stride), to, pool, slots, s)
    s.synchronize()
    got = dB.cpu().numpy().reshape(G, -1)
    for g in range(G):
        assert np.array_equal(got[g], back[g]), f"layer {g}: " + first_mismatch(got[g], back[g])
    del view
    kvx.kv_pool_destroy(pool)


@pytest.mark.parametrize("nc", [255, 256, 257])
def test_device_pool_launches_of_many_small_chunks(nc):
    """A device pool takes up to 256 small chunks in one launch."""
    lay = Layout(1, 1, 16, 1, 2, 4)
    pool = kvx.kv_pool_create(lay.kv, 1, "zero_copy", host_kind=kvx.KV_POOL_DEVICE)
    assert kvx.kv_pool_get_info(pool)["chunks_per_batch"] == 256
    kvx.kv_pool_destroy(pool)
    _check(lay, kvx.KV_BLOCK_HND, "device", nc * lay.C - 1, bad=True)
