// Internal declarations shared by the kvx host code and kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <exception>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "kvx.h"

namespace kvx {

#ifndef KVX_THREADS
#define KVX_THREADS 256
#endif
constexpr int kThreads = KVX_THREADS;  // work-items per workgroup (wave64s x 64)
constexpr int kMaxLaunchLayers = 64;   // layer pointers carried in one launch's kernel arguments
constexpr int kMaxLaunchChunks = 256;  // slot ids carried in one launch's kernel arguments
constexpr int kMaxStateLayers = 64;    // recurrent layers of a state snapshot (one launch carries all)
constexpr int kMaxLaunchSnapshots = 128;  // snapshots carried in one state launch's arguments
constexpr int64_t kStatePiece = 4 * 1024;  // bytes of a page one workgroup moves (kvx_state.hip)
constexpr int64_t kHostLine = 256;  // pieces of host memory start at multiples of this (see StatePlan)
constexpr int64_t kMaxLaunchPieces = int64_t(1) << 22;  // workgroups of one state launch

// Derived sizes of a layout (all bytes, 64-bit).
struct Geometry {
    int64_t L, H, D, E, BS, C;
    int64_t row_bytes;     // D*E: one (head, token) row
    int64_t vec_per_row;   // row_bytes / 16
    int64_t block_bytes;   // 2*H*BS*D*E
    int64_t block_stride;  // bytes between blocks in a layer buffer
    int64_t token_bytes;   // TB = 2*L*H*D*E
    int64_t slot_bytes;    // C*TB
    int64_t blocks_per_chunk;  // C / BS
};

Geometry geometry(const kv_layout &lay, int64_t block_stride_bytes);

// Division of 0 <= n < 2^31 by a launch constant d >= 1 as a multiplication: shift = ceil(log2 d), mul =
// floor(2^(31 + shift) / d) + 1 (Granlund and Montgomery, "Division by Invariant Integers using
// Multiplication", PLDI 1994, Theorem 4.2 with N = 31).
struct Divisor {
    uint32_t mul, shift;
};

inline Divisor divisor(int64_t d) {
    Divisor r{};
    while ((int64_t{1} << r.shift) < d)
        ++r.shift;
    r.mul = static_cast<uint32_t>((uint64_t{1} << (31 + r.shift)) / static_cast<uint64_t>(d) + 1);
    return r;
}

__host__ __device__ __forceinline__ int divide(int n, const Divisor &d) {
    const uint64_t high = static_cast<uint64_t>(static_cast<uint32_t>(n) << 1) * d.mul >> 32;
    return static_cast<int>(static_cast<uint32_t>(high) >> d.shift);
}

// floor(n / d) beyond divide()'s range, for 0 <= n < 2^53, d >= 1 and a quotient below 2^31.  n / d is at least 1 / d
// below the next whole number q, and the nearest double would be q only if half the spacing there, at most
// q * 2^-53, reached 1 / d: not while q * d <= 2^53.
__host__ __device__ __forceinline__ int divide_long(int64_t n, int d) {
    return static_cast<int>(static_cast<double>(n) / d);
}

// Kernel arguments of one gather (pack) or scatter (unpack) launch.  A launch covers nchunks
// consecutive chunks of the prefix and nlayers consecutive layers, from those that the block
// table's address and plane0 name on.  Passed by value so that every pointer and id is captured
// at enqueue time.
struct GatherArgs {
    // What every workgroup reads, in one run (scalar loads of up to 64 bytes).
    uint8_t *chunk_base;               // device-visible address of slot 0 (pool or staging)
    const int32_t *block_table;        // device int32[], from the launch's first block on
    int64_t slot_stride;               // bytes between slot ids at chunk_base
    int64_t block_stride;
    int32_t num_blocks;
    int32_t plane0;                    // 2*layer0: the launch's first plane in a chunk
    int32_t nchunks;
    int32_t C;
    int32_t last_r;                    // tokens in the launch's last chunk
    int32_t blocks_per_chunk;
    int32_t token_vecs, slab_vecs;     // 16-byte vectors of one token of a plane, and of one block's K or V slab
    int32_t H, BS, vec_per_row;
    Divisor by_slab, by_row, by_head;  // division by slab_vecs, vec_per_row and H
    int32_t nhd;                       // cache blocks are [2][BS][H][D] (token-major)
    int32_t long_plane;                // a plane's vectors do not fit 31 bits
    int32_t tiles, last_tiles;         // tiles of a plane: of the launch's first chunk, of its last
    int32_t nlayers;
    int32_t *err;                      // device-visible async error word
    uint8_t *layer[kMaxLaunchLayers];  // cache layer base pointers (device) of layers layer0..
    int32_t slot[kMaxLaunchChunks];    // slot id of each chunk of the launch
};

enum Direction { kPack = 0, kUnpack = 1 };

// Where the packed side of a gather launch lies: device memory (staging, a device pool) or the mapped pinned pool,
// in a pool whose stores are kernels too or whose stores run on the DMA engines.
enum Packed { kInDevice = 0, kInHost = 1, kInHostBesideDma = 2 };

// Kernel arguments of one state-snapshot launch.  Pages are cut into ppp pieces of `piece` <=
// kStatePiece bytes (the last piece of a page may be shorter).  The launch covers npieces <=
// kMaxLaunchPieces pieces of its own lists of snapshots, from piece piece0 of page page0 on; page
// p is layer p % G of snapshot p / G.  In a host-side launch with `lines` set, a page is cut at multiples of
// kHostLine of its packed bytes' addresses: its first piece is shorter by the address's low bits.
struct StateArgs {
    uint8_t *base;                     // device-visible packed side (state pool or staging)
    int64_t page_stride, page_bytes;
    int32_t page0, piece0, npieces, piece;
    int32_t G, ppp;
    int32_t last_piece;                // bytes of a page's last piece (set by launch_state, as the next)
    int32_t lines;
    Divisor by_ppp, by_layers;         // division by ppp and G
    uint8_t *layer[kMaxStateLayers];   // device base of each recurrent layer's page buffer
    int64_t page[kMaxLaunchSnapshots];  // device page id of each snapshot
    int64_t off[kMaxLaunchSnapshots];   // byte offset at `base` of each snapshot's packed bytes
};

// Enqueue one launch on `stream`; host_side: the packed side is mapped pinned host memory.  Returns the
// launch error (hipSuccess on success).
hipError_t launch_state(const StateArgs &args, Direction dir, bool host_side, hipStream_t stream);

// Enqueue the pack/unpack launches for chunks [chunk0, chunk0 + nchunks) of a prefix of `cache`
// (split over launches of at most kMaxLaunchLayers layers and kMaxLaunchChunks chunks): slots[c] is the slot of chunk
// chunk0 + c at chunk_base, slot_stride bytes apart.  Returns the first launch error.  No host allocation, no
// event.
hipError_t launch_gathers(const kv_cache *cache, const int32_t *block_table, int64_t n_tokens, Direction dir,
                          int64_t chunk0, int nchunks, const int32_t *slots, uint8_t *chunk_base, int64_t slot_stride,
                          Packed packed, int32_t *err, hipStream_t stream);

// Thread-local error reporting.
kv_status fail(kv_status code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
kv_status hip_fail(hipError_t err, const char *what, const char *file, int line);
void set_last_error(const std::string &msg);

// Runs an entry point's body so that no C++ exception crosses the C ABI: a failed host
// allocation becomes KV_ENOMEM, any other exception KV_EINVAL with its message.
template <class F>
kv_status guarded(F &&body) noexcept {
    try {
        return body();
    } catch (const std::bad_alloc &) {
        return fail(KV_ENOMEM, "host memory allocation failed");
    } catch (const std::exception &e) {
        return fail(KV_EINVAL, "internal error: %s", e.what());
    } catch (...) {
        return fail(KV_EINVAL, "internal error");
    }
}

#define KVX_HIP(expr)                                                         \
    do {                                                                      \
        hipError_t kvx_e_ = (expr);                                           \
        if (kvx_e_ != hipSuccess)                                             \
            return ::kvx::hip_fail(kvx_e_, #expr, __FILE__, __LINE__);        \
    } while (0)

// Host-only request validation shared by kv_check, kv_store and kv_load.
kv_status check_layout(const kv_layout &lay);
kv_status check_request(const kv_cache *cache, const kv_layout *pool_layout, int64_t pool_slots,
                        int64_t n_tokens, const int64_t *chunk_ids, int for_store);
kv_status check_state_request(const kv_state *state, int64_t pool_state_slot_bytes, int64_t pool_state_slots,
                              int64_t n, const int64_t *pages, const int64_t *slot_ids, int for_store);

// Geometry of a pool index (for the tier's consistency check).
int32_t index_chunk_tokens(const kv_index *index);
int64_t index_num_slots(const kv_index *index);
int64_t index_num_state_slots(const kv_index *index);

}  // namespace kvx

// The pool: one pinned host region plus the staging ring and its streams/events.
struct kv_pool {
    kv_layout layout{};
    kvx::Geometry geo{};
    int64_t num_slots = 0, pool_bytes = 0;
    // Recurrent-state snapshot area: num_state_slots slots of state_slot_bytes each, starting
    // state_offset bytes into the pinned region (after the chunk slots).
    int64_t num_state_slots = 0, state_slot_bytes = 0, state_offset = 0;
    int device = 0;
    uint32_t mode_of[2] = {0, 0};     // transfer mode per direction: [kPack] stores, [kUnpack] loads
    uint32_t host_kind = 0;
    uint8_t *host_base = nullptr;   // host address of slot 0 (nullptr for a device pool)
    uint8_t *dev_base = nullptr;    // device address of slot 0
    bool on_device = false;         // KV_POOL_DEVICE: the region is device memory (HBM)
    int32_t *err_host = nullptr;    // async error word (pinned, mapped)
    int32_t *err_dev = nullptr;
    double alloc_seconds = 0.0;
    bool pinned = false;

    // Staged mode: one lane per direction, each with its own staging ring, DMA side streams and
    // events, so a store and a load in flight at once never wait for each other's slots or streams.
    struct Lane {
        uint8_t *staging = nullptr;        // K slots of cpb*slot_bytes each
        std::vector<hipStream_t> sides;    // DMA side streams of this direction
        std::vector<hipEvent_t> ev_free;   // staging slot k may be overwritten once this completes
        std::vector<bool> free_recorded;
        std::vector<hipEvent_t> ev_ready;  // staging slot k holds the current batch
        std::vector<hipEvent_t> ev_join;   // per side stream: exit join of a store
        hipEvent_t ev_entry = nullptr;     // entry gate of a load
        int ring = 0;
    };
    int K = 0, cpb = 0, S = 0;       // ring depth, chunks per slot, side streams: per direction
    uint8_t *staging = nullptr;      // both lanes' staging (one allocation)
    bool staging_contiguous = false;  // always false: staging is plain device memory
    Lane lane[2];                    // [kPack] stores, [kUnpack] loads
    int zc_chunks = 0;                 // chunks per zero-copy launch
    bool dma_only = false;             // chunks_per_batch was given: as KV_MODE_STAGED_DMA in either direction
    // Last use of the pool on each caller stream (recorded after every store/load), so that
    // kv_pool_destroy never frees memory that queued kernels or copies still touch.
    std::vector<std::pair<hipStream_t, hipEvent_t>> last_use;

    // Profiling of pack/unpack and state launches.
    bool profile = false;
    struct Timed {
        hipEvent_t start, stop;
        double bytes;
    };
    // Index: 0 pack, 1 unpack, 2 state pack, 3 state unpack.
    std::vector<Timed> pending[4];
    std::vector<hipEvent_t> spare_events;
    int64_t launches[4] = {0, 0, 0, 0};
    double total_ms[4] = {0.0, 0.0, 0.0, 0.0};
    double total_bytes[4] = {0.0, 0.0, 0.0, 0.0};

    std::mutex mu;
    std::mutex tier_mu;  // serialises tier requests (one request's faults are its own)
    // Tier serving: every request runs under tier_mu on this one stream, its block table staged
    // through these buffers.  Made by the first request (or by kv_tier_run before it accepts a
    // connection) and kept until kv_pool_destroy, so later connections create no runtime objects
    // (a new stream and its first copy measured tens of ms on the request's path).
    hipStream_t tier_stream = nullptr;
    int32_t *tier_table = nullptr;         // device copy of the request's block table
    int32_t *tier_table_pinned = nullptr;  // pinned host staging of it
    size_t tier_table_cap = 0;             // bytes of each
};

namespace kvx {
inline bool is_staged(uint32_t mode) { return mode == KV_MODE_STAGED || mode == KV_MODE_STAGED_DMA; }

// Where the kernels of a request that moves directly find the packed side.
inline Packed packed_in_pool(const kv_pool *pool) {
    return pool->on_device ? kInDevice : pool->mode_of[kPack] == KV_MODE_ZERO_COPY ? kInHost : kInHostBesideDma;
}

// Whether a staged request of `bytes` in `copies` DMA copies moves directly instead: by the zero-copy
// kernels on the caller's stream.  Two kinds of request are better off so.
//  * Short ones: the staged pipeline's kernel, event, cross-queue wait and copy cost 60 to 75 us beyond the
//    link's time, a zero-copy kernel about 20 (loads in one DMA copy, us, staged and direct: 1 MiB 81 and 34,
//    4 MiB 135 and 88, 16 MiB 359 and 309, 32 MiB 657 and 605).  At 32 MiB the gain is down to 8%.
//  * Fragmented ones: a copy costs the DMA engine about 10 us however short (256 KiB: 18 GB/s, 1 MiB: 37,
//    4 MiB: 50 of 57), a fifth of the time at 2 MiB a copy.  256 MiB loaded in copies of 256 KiB, 1 MiB and
//    1.5 MiB: 17.4, 7.6 and 6.7 ms staged, 4.7 direct.
// The kernels hold CUs meanwhile: a stream of large GEMMs ran at 53-58% of its rate beside these loads and
// at 43-53% beside these stores, at 92-99% beside staged ones, and a request that finds the GPU full waits for
// a kernel to end by either route (16 and 32 MiB beside those GEMMs: 870 and 990 us direct, 800 and 810
// staged).  So both kinds are bounded, to about 0.6 and 5 ms of the link's time, and longer requests stay on the
// DMA engines.
constexpr int64_t kDirectBytes = int64_t{32} << 20;
constexpr int64_t kDirectFragmentedBytes = int64_t{256} << 20;
constexpr int64_t kDirectCopyBytes = int64_t{2} << 20;
inline bool moves_directly(const kv_pool *pool, Direction dir, int64_t bytes, int64_t copies) {
    if (pool->dma_only || pool->mode_of[dir] == KV_MODE_STAGED_DMA)
        return false;
    return bytes <= kDirectBytes || (bytes <= kDirectFragmentedBytes && bytes / copies < kDirectCopyBytes);
}

// Make the pool's tier stream and block-table buffers (at least `table_bytes` each) if they are
// missing or too small.  Caller holds pool->tier_mu and has made the pool's device current.
kv_status tier_resources(kv_pool *pool, size_t table_bytes);
}  // namespace kvx
