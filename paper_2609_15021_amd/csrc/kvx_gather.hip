// Pack (store) and unpack (load) kernels for gfx950.
//
// On the cache side the K (or V) slab of one paged block is the contiguous [H][BS][D] region of that
// block (HND, the paper's replica layout, Table 1) or [BS][H][D] (NHD, token-major); on the chunk side a
// plane (layer, K/V) of a chunk is one contiguous run [r][H][D] of token-major rows, the slabs of the
// chunk's blocks one after the other.  A slab differs between the sides only by a permutation of
// D*E-byte rows: cache row (h, s) <-> chunk row (s, h); for NHD blocks not at all.
//
// A plane is cut into tiles of 256 16-byte vectors (4 KiB) in chunk order, wherever its blocks end, and
// a workgroup moves one tile, one vector per lane: the chunk side (host memory over PCIe in zero-copy
// mode) is read or written in contiguous 1 KiB-per-wave runs, the cache side in whole rows.  HBM bounds
// the device-side launches.  With one short tile per workgroup the tiles in flight are neighbours and
// every lane is busy at any slab size.  Measured on MI355X, paired on the same allocations with the
// earlier split (one slab of a block per workgroup, moved 4 KiB at a time, 5 resident per CU), pack /
// unpack TB/s read + written, before -> after:
//   32 KiB slabs (27B-class layout, 2 GiB)         5.75 -> 6.13 / 5.5-5.9 -> 6.0
//   32 KiB NHD slabs (FP8, 32-token pages, 2 GiB)  5.82 -> 6.26 / 5.32 -> 5.98
//   8 KiB slabs (two KV heads)                     4.98 -> 6.13 / 5.05 -> 5.68
//   4 KiB slabs (one KV head)                      3.43 -> 5.92 / 3.45 -> 5.47
//   2 KiB slabs (one KV head, FP8)                 1.92 -> 5.34 / 1.89 -> 5.03
//   3,840-byte slabs of 160-byte rows              3.12 -> 5.07 / 2.98 -> 4.62
// Other tiles, paired the same way (geometric mean over twelve layouts against the earlier split, pack /
// unpack; 4 KiB: 1.46 / 1.42): 1 KiB 1.44 / 1.37, 2 KiB 1.44 / 1.39, 8 KiB 1.45 / 1.40 with 512 lanes,
// 1.39 / 1.37 with two vectors per lane.  Handing each XCD 2, 4, 8 or 16 consecutive tiles changed pack by
// less than 1% and cost unpack 2-3%.
// Values are moved as integers only: no float register ever holds them (NaN payloads, -0
// and subnormals survive).
//
// Streaming data is read and written nontemporally.  Host-side (zero-copy) launches run a few
// dozen workgroups that stride over the tiles (KVX_HOST_WGS_*): the link bounds them, and the rest of
// the chip stays free.
#include <algorithm>
#include <cstring>

#include "kvx_internal.h"

namespace kvx {

namespace {

// One 16-byte vector as a native 128-bit register tuple (kept in VGPRs; never a float).
typedef uint32_t vec16 __attribute__((ext_vector_type(4)));

// Dynamic LDS (unused) reserved per workgroup of a device-side unpack, to cap the workgroups resident per
// CU: 26 KiB of the CU's 160 KiB allows 6 (24 waves).  Paired over twelve layouts, 6 unpacked
// 1.4% more than 8 (the hardware's limit: 32 waves) and 0.4% more than 7, and 3-4% more on the 32 KiB slabs;
// the fp32 layout of 64 KiB slabs loses 4% to it (6.61 -> 6.37 TB/s).  Pack lost 7% with 6 and takes no cap.
#ifndef KVX_LDS_RESERVE_UNPACK
#define KVX_LDS_RESERVE_UNPACK 26624
#endif
#ifndef KVX_LDS_RESERVE_PACK
#define KVX_LDS_RESERVE_PACK 0
#endif
// Workgroups of a host-side (zero-copy) pack / unpack launch; each strides over the launch's tiles
// with the next tile's reads in flight.  Measured on MI355X at the 27B-class layout: 64 for pack gives
// 57.0 GB/s (48: 56.9, 32: 52.9).  Alone, unpack moves 56.8 GB/s with 16, 57.1 with 20, 57.4 with 24 and 32.
// With a store of the same pool running at the same time, the total follows from what the reads in flight leave
// the store (store + load, GB/s, for 16 / 17 / 18 / 20 / 24 / 32 workgroups):
//   store by DMA copies   98.5 / 85.6 / 75.2 / 66.8 / 60.0 / 59.4   (the same at 4 KiB slabs)
//   store by kernels      69.4 / 71.5 / 72.9 / 75.5 / 78.7 / 86.6   (within 5% at 8 and 4 KiB slabs and token-major)
// so loads take 16 in a pool whose stores run on the DMA engines and 32 where they are kernels.  Where each lane
// has its own block (see start_tile) the wait for its table entry also waits for a tile's data, and 18 are best
// beside DMA stores (16 / 17 / 18 / 19 / 20 / 32 in total, 160-byte rows: 90.2 / 82.4 / 93.2 / 81.6 / 73.5 / 59.3;
// 64-byte rows: 90.1 / 91.2 / 96.5 / 82.0 / 73.3 / 60.1; alone 57.0 with 18, 57.4 with 32).
#ifndef KVX_HOST_WGS_PACK
#define KVX_HOST_WGS_PACK 64
#endif
#ifndef KVX_HOST_WGS_UNPACK
#define KVX_HOST_WGS_UNPACK 32
#endif
#ifndef KVX_HOST_WGS_UNPACK_BESIDE_DMA
#define KVX_HOST_WGS_UNPACK_BESIDE_DMA 16
#endif
#ifndef KVX_HOST_WGS_UNPACK_LANES_BESIDE_DMA
#define KVX_HOST_WGS_UNPACK_LANES_BESIDE_DMA 18
#endif
#ifndef KVX_TILE_VECS
#define KVX_TILE_VECS 256
#endif
constexpr int kTileVecs = KVX_TILE_VECS;  // 16-byte vectors of a tile: one per lane of a workgroup
// Vectors of a plane up to which its blocks are found with divide(), whose range ends there (32 GiB).  A test
// build sets 0, so that small planes go the way of the longest.
#ifndef KVX_DIVIDE_VECS
#define KVX_DIVIDE_VECS INT32_MAX
#endif
// Tiles of a plane that one launch dimension takes as workgroups: a dimension holds fewer than 2^32 work-items.
// Longer planes (64 GiB) run the strided kernel on a grid that fills the chip.
#ifndef KVX_GRID_TILES
#define KVX_GRID_TILES ((int64_t{1} << 32) / kTileVecs - 1)
#endif
constexpr int64_t kStridedDeviceWgs = 2048;  // 8 per CU

// Sides with a scalar base are read and written through buffer resources: one lane offset instead of a
// lane address, and the hardware's range check in place of branches (beyond the range a read gives zeros
// and a write does nothing).
constexpr int kNt = 2, kSc1 = 16;            // CDNA3/4 cache-policy bits
constexpr int kRawBufferFlags = 0x00020000;  // descriptor word 3 of a raw (untyped) buffer

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(uint8_t *base, int bytes) {
    // bytes < 2^31: validation caps a block at 2 GiB, so a K or V slab at 1 GiB.
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, kRawBufferFlags);
}

__device__ __forceinline__ vec16 load16(__amdgpu_buffer_rsrc_t from, int offset) {
    return __builtin_amdgcn_raw_buffer_load_b128(from, offset, 0, kNt);
}

// NT_SC1: nontemporal at agent scope instead of plain nontemporal.  Paired on six destination allocations
// of the 27B-class layout, unpack's cache-side stores moved 0.1-2.3% more with it on every one of them
// ("sc1" without "nt" varied by allocation, stores without either lost 2-7%); pack's stores into mapped
// pinned host memory 57.1 GB/s against 55.7-55.9 (56.8 without either bit); its stores into device memory
// and either kernel's loads gained nothing from other policies than plain nontemporal.
template <bool NT_SC1>
__device__ __forceinline__ void store16(__amdgpu_buffer_rsrc_t to, int offset, vec16 v) {
    __builtin_amdgcn_raw_buffer_store_b128(v, to, offset, 0, NT_SC1 ? kNt | kSc1 : kNt);
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Block ids are read-only for the launch: the constant address space makes a uniform read a scalar load.
typedef const __attribute__((address_space(4))) int32_t *TablePtr;

// A tile on its way: kTileVecs chunk-side vectors of one plane (fewer at the plane's end), one per lane.
struct Tile {
    uint8_t *chunk;  // the tile's first byte on the chunk side
    uint8_t *cache;  // the layer's K (or V) slab of block 0
    vec16 data;
    int left;        // vectors in the tile
    int pos;         // this lane's vector inside its block's slab
    int32_t block;   // the block id from the table (not yet checked)
};

// 16-byte-vector offset in the cache-side slab of the slab's chunk-order vector p: chunk row (s, h) =
// (p / VR / H, p / VR % H) is cache row (h, s); token-major slabs are in chunk order already.
__device__ __forceinline__ int cache_vec(const GatherArgs &a, int p) {
    if (a.nhd)
        return p;
    const int row = divide(p, a.by_row), s = divide(row, a.by_head);
    return ((row - s * a.H) * a.BS + s) * a.vec_per_row + (p - row * a.vec_per_row);
}

// Whether the tile's block id is outside the cache (then flagged in the pool's error word).
__device__ __forceinline__ bool bad_block(const GatherArgs &a, const Tile &t) {
    const bool bad = t.block < 0 || t.block >= a.num_blocks;
    if (bad)
        __hip_atomic_store(a.err, KV_ASYNC_BAD_BLOCK, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return bad;
}

// The block's slab as a buffer; of no bytes if the id is outside the cache: no cache byte is then touched,
// and pack's zeros keep stale staging or pool bytes (another request's state) out of the chunk.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t slab_buffer(const GatherArgs &a, const Tile &t) {
    const bool bad = bad_block(a, t);
    return buffer(t.cache + (bad ? 0 : t.block * a.block_stride), bad ? 0 : a.slab_vecs * 16);
}

// Start tile x of plane `plane` (2*layer + kv) of launch chunk c, x < ceil(plane vectors / kTileVecs): find
// its block and issue its reads.  WAVE: a slab is a whole number of waves' vectors, so that a wave's 64
// vectors lie in one block and its table entry and cache base are scalars; otherwise each lane has its own.
template <int DIR, bool WAVE>
__device__ __forceinline__ void start_tile(const GatherArgs &a, int c, int plane, int x, Tile &t) {
    const int32_t slot = a.slot[c];
    uint8_t *const layer = a.layer[plane >> 1];
    // Everything a tile reads from the arguments is needed in scalar registers here, so that the scalar loads
    // go out together: left to itself the compiler spread them over five dependent waits.
    asm volatile("" ::"s"(slot), "s"(layer), "s"(a.chunk_base), "s"(a.block_table), "s"(a.slot_stride),
                 "s"(a.block_stride), "s"(a.num_blocks), "s"(a.plane0), "s"(a.nchunks), "s"(a.C), "s"(a.last_r),
                 "s"(a.blocks_per_chunk), "s"(a.token_vecs), "s"(a.slab_vecs), "s"(a.H), "s"(a.BS),
                 "s"(a.vec_per_row), "s"(a.by_slab.mul), "s"(a.by_slab.shift), "s"(a.by_row.mul), "s"(a.by_row.shift),
                 "s"(a.by_head.mul), "s"(a.by_head.shift), "s"(a.nhd), "s"(a.long_plane));
    const bool last = c == a.nchunks - 1;
    const int r = last ? a.last_r : a.C;  // tokens in the chunk
    const int64_t base = static_cast<int64_t>(x) * kTileVecs;
    const int64_t plane_vecs = static_cast<int64_t>(r) * a.token_vecs;
    const int tiles = last ? a.last_tiles : a.tiles;
    t.left = x == tiles - 1 ? static_cast<int>(plane_vecs - base) : kTileVecs;
    // The tile's first block and the first vector inside its slab.
    const int j0 = a.long_plane ? uniform(divide_long(base, a.slab_vecs)) : divide(static_cast<int>(base), a.by_slab);
    const int first = static_cast<int>(base - static_cast<int64_t>(j0) * a.slab_vecs);
    t.chunk = a.chunk_base + slot * a.slot_stride + ((a.plane0 + plane) * plane_vecs + base) * 16;
    t.cache = layer + (plane & 1) * (static_cast<int64_t>(a.slab_vecs) * 16);
    const TablePtr table = (TablePtr)(a.block_table + static_cast<int64_t>(c) * a.blocks_per_chunk + j0);

    const int v = static_cast<int>(threadIdx.x);
    // Unpack's reads do not wait for the block table.
    if (DIR == kUnpack)
        t.data = load16(buffer(t.chunk, t.left * 16), v * 16);
    if constexpr (WAVE) {
        // A wave beyond the tile's end takes the last block (its vectors are dropped).
        const int wave = first + min(uniform(v & ~63), (t.left - 1) & ~63);
        const int j = divide(wave, a.by_slab);
        t.block = table[j];
        t.pos = wave - j * a.slab_vecs + (v & 63);
        if (DIR == kPack)
            t.data = load16(slab_buffer(a, t), cache_vec(a, t.pos) * 16);
    } else {
        const int inside = first + min(v, t.left - 1);
        const int j = divide(inside, a.by_slab);
        t.block = table[j];
        t.pos = inside - j * a.slab_vecs;
        if (DIR == kPack) {
            const bool bad = bad_block(a, t);
            const uint8_t *slab = t.cache + (bad ? 0 : t.block * a.block_stride);  // bad: read block 0, pass on zeros
            t.data = __builtin_nontemporal_load(reinterpret_cast<const vec16 *>(slab) + cache_vec(a, t.pos));
            if (bad)
                t.data = vec16{0u, 0u, 0u, 0u};
        }
    }
}

// Write a started tile to its place.
template <int DIR, bool WAVE, bool HOST_SIDE>
__device__ __forceinline__ void finish_tile(const GatherArgs &a, const Tile &t) {
    const int v = static_cast<int>(threadIdx.x);
    if constexpr (DIR == kPack) {
        store16<HOST_SIDE>(buffer(t.chunk, t.left * 16), v * 16, t.data);
    } else if constexpr (WAVE) {
        store16<true>(slab_buffer(a, t), v < t.left ? cache_vec(a, t.pos) * 16 : -1, t.data);
    } else if (!bad_block(a, t) && v < t.left) {
        vec16 *slab = reinterpret_cast<vec16 *>(t.cache + t.block * a.block_stride);
        __builtin_nontemporal_store(t.data, slab + cache_vec(a, t.pos));
    }
}

// HOST_SIDE marks launches whose chunk side is mapped pinned host memory (zero-copy mode).
template <int DIR, bool WAVE, bool HOST_SIDE>
__global__ __launch_bounds__(kTileVecs) void gather_kernel(const GatherArgs a) {
    if constexpr (!HOST_SIDE) {
        // One workgroup per tile; the launch's last chunk may have fewer tiles.
        if (static_cast<int>(blockIdx.z) == a.nchunks - 1 && static_cast<int>(blockIdx.x) >= a.last_tiles)
            return;
        Tile t;
        start_tile<DIR, WAVE>(a, blockIdx.z, blockIdx.y, blockIdx.x, t);
        finish_tile<DIR, WAVE, HOST_SIDE>(a, t);
    } else {
        // A capped grid strides over the tiles: the link, not the number of waves in flight, bounds
        // these launches, and the CUs they leave free run other streams' kernels.  The next tile's reads
        // are in flight while a tile is written.  Tiles are numbered over the chunks in order; only the
        // launch's last chunk can have fewer per plane.
        const int planes = 2 * a.nlayers;
        const int full = (a.nchunks - 1) * planes * a.tiles;
        const int total = full + planes * a.last_tiles;
        auto start = [&](int id, Tile &t) {
            int c = a.nchunks - 1, rest = id - full, per = a.last_tiles;
            if (id < full) {
                c = id / (planes * a.tiles);
                rest = id - c * planes * a.tiles;
                per = a.tiles;
            }
            const int plane = rest / per;
            start_tile<DIR, WAVE>(a, c, plane, rest - plane * per, t);
        };
        // Two tiles in turn, by name: copying one to the other would wait for its reads.
        Tile even, odd;
        int id = blockIdx.x;  // the grid has at most `total` workgroups
        start(id, even);
        while (true) {
            id += gridDim.x;
            if (id >= total) {
                finish_tile<DIR, WAVE, HOST_SIDE>(a, even);
                return;
            }
            start(id, odd);
            finish_tile<DIR, WAVE, HOST_SIDE>(a, even);
            id += gridDim.x;
            if (id >= total) {
                finish_tile<DIR, WAVE, HOST_SIDE>(a, odd);
                return;
            }
            start(id, even);
            finish_tile<DIR, WAVE, HOST_SIDE>(a, odd);
        }
    }
}

}  // namespace

template <bool HOST_SIDE>
static const void *kernel_of(Direction dir, bool wave) {
    if (wave)
        return dir == kPack ? reinterpret_cast<const void *>(&gather_kernel<kPack, true, HOST_SIDE>)
                            : reinterpret_cast<const void *>(&gather_kernel<kUnpack, true, HOST_SIDE>);
    return dir == kPack ? reinterpret_cast<const void *>(&gather_kernel<kPack, false, HOST_SIDE>)
                        : reinterpret_cast<const void *>(&gather_kernel<kUnpack, false, HOST_SIDE>);
}

// Launch over the chunks and layers that `a` names; what depends on the layout alone is set.
static hipError_t launch(GatherArgs &a, Direction dir, Packed packed, hipStream_t stream) {
    const bool host_side = packed != kInDevice;
    auto tiles_of = [&](int64_t r) { return (r * a.token_vecs + kTileVecs - 1) / kTileVecs; };
    a.last_tiles = static_cast<int32_t>(tiles_of(a.last_r));
    a.tiles = a.nchunks > 1 ? static_cast<int32_t>(tiles_of(a.C)) : a.last_tiles;
    a.long_plane = static_cast<int64_t>(a.tiles) * kTileVecs > KVX_DIVIDE_VECS;
    dim3 grid(static_cast<uint32_t>(a.tiles), static_cast<uint32_t>(2 * a.nlayers), static_cast<uint32_t>(a.nchunks));
    const bool wave = a.slab_vecs % 64 == 0, strided = host_side || a.tiles > KVX_GRID_TILES;
    if (strided) {
        const int64_t total = 2 * static_cast<int64_t>(a.nlayers) *
                              ((a.nchunks - 1) * static_cast<int64_t>(a.tiles) + a.last_tiles);
        const int64_t wgs = !host_side          ? kStridedDeviceWgs
                            : dir == kPack      ? KVX_HOST_WGS_PACK
                            : packed == kInHost ? KVX_HOST_WGS_UNPACK
                            : wave              ? KVX_HOST_WGS_UNPACK_BESIDE_DMA
                                                : KVX_HOST_WGS_UNPACK_LANES_BESIDE_DMA;
        grid = dim3(static_cast<uint32_t>(std::min(total, wgs)));
    }
    const void *fn = strided ? kernel_of<true>(dir, wave) : kernel_of<false>(dir, wave);
    const unsigned lds = host_side ? 0u : dir == kPack ? KVX_LDS_RESERVE_PACK : KVX_LDS_RESERVE_UNPACK;
    void *kargs[] = {&a};
    // hipLaunchKernel reports launch failures directly (no sticky last-error state).
    return hipLaunchKernel(fn, grid, dim3(kTileVecs), kargs, lds, stream);
}

hipError_t launch_gathers(const kv_cache *cache, const int32_t *block_table, int64_t n_tokens, Direction dir,
                          int64_t chunk0, int nchunks, const int32_t *slots, uint8_t *chunk_base, int64_t slot_stride,
                          Packed packed, int32_t *err, hipStream_t stream) {
    const Geometry g = geometry(cache->layout, cache->block_stride_bytes);
    GatherArgs a;
    std::memset(&a, 0, sizeof(a));
    a.chunk_base = chunk_base;
    a.err = err;
    a.slot_stride = slot_stride;
    a.block_stride = g.block_stride;
    a.num_blocks = cache->num_blocks;
    a.C = static_cast<int32_t>(g.C);
    a.blocks_per_chunk = static_cast<int32_t>(g.blocks_per_chunk);
    a.H = static_cast<int32_t>(g.H);
    a.BS = static_cast<int32_t>(g.BS);
    a.vec_per_row = static_cast<int32_t>(g.vec_per_row);
    a.token_vecs = a.H * a.vec_per_row;
    a.slab_vecs = a.BS * a.token_vecs;
    a.by_slab = divisor(a.slab_vecs);
    a.by_row = divisor(a.vec_per_row);
    a.by_head = divisor(a.H);
    a.nhd = cache->block_order == KV_BLOCK_NHD ? 1 : 0;
    for (int layer0 = 0; layer0 < g.L; layer0 += kMaxLaunchLayers) {
        a.plane0 = 2 * layer0;
        a.nlayers = static_cast<int>(std::min<int64_t>(kMaxLaunchLayers, g.L - layer0));
        for (int l = 0; l < a.nlayers; ++l)
            a.layer[l] = static_cast<uint8_t *>(cache->layer_ptrs[layer0 + l]);
        for (int c0 = 0; c0 < nchunks; c0 += kMaxLaunchChunks) {
            a.nchunks = std::min(kMaxLaunchChunks, nchunks - c0);
            a.last_r = static_cast<int32_t>(std::min<int64_t>(g.C, n_tokens - (chunk0 + c0 + a.nchunks - 1) * g.C));
            a.block_table = block_table + (chunk0 + c0) * g.blocks_per_chunk;
            std::copy(slots + c0, slots + c0 + a.nchunks, a.slot);
            const hipError_t e = launch(a, dir, packed, stream);
            if (e != hipSuccess)
                return e;
        }
    }
    return hipSuccess;
}

}  // namespace kvx
