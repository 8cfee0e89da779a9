// State-snapshot kernels for gfx950: move the recurrent layers' boundary snapshots
// (convolution state, recurrent state and padding as opaque pages, Sec. 2.2) between
// their device page buffers and the packed state slots, [G][page_bytes] per snapshot.
//
// Each page is contiguous on both sides, so the move is a batched copy: pages are cut into pieces of
// 4 KiB (kStatePiece; the last one of a page may be shorter) and a workgroup moves one piece, one 16-byte
// vector per lane.  Device-side launches run one workgroup per piece: HBM bounds them, and short pieces
// keep neighbouring bytes in flight and every CU busy at any page size.  Measured on
// MI355X against the earlier 16 KiB pieces through LDS, paired (store / load, TB/s read + written):
// 8 x 48 pages of 3.06 MiB 5.88 -> 6.33 / 5.71 -> 6.29; one such snapshot 5.52 -> 5.79 / 5.29 -> 5.95;
// 16 x 64 pages of 64 KiB 4.78 -> 5.32 / 4.60 -> 5.71; 64 x 64 pages of 8 KiB 3.45 -> 3.84 / 3.41 -> 4.07.
// A residency cap, which gains the gather unpack, costs the load 1-2% here and the store 3-5%.
// Host-side (zero-copy) launches run a few workgroups that stride over the pieces: the host link bounds
// them.  There is no arithmetic to put on the matrix cores, and bytes never pass through a float register.
#include <algorithm>

#include "kvx_internal.h"

namespace kvx {

namespace {

typedef uint32_t svec16 __attribute__((ext_vector_type(4)));

static_assert(kStatePiece == kThreads * 16, "a piece is one vector per lane");

// Workgroups of a host-side (zero-copy) launch, striding over its pieces with the next piece's reads in
// flight, as the gather kernels' launches do.  Stores, us with 16 / 32 / 64 / 128: 4 x 8 pages of 12,896 bytes 13.3 /
// 13.4 / 14.1 / 14.1, 4 x 8 of 16 KiB 14.6 / 14.7 / 15.5 / 15.6 (the earlier kernel 13.6 and 15.0), 48 pages of
// 3.06 MiB 2,829 / 2,701 / 2,699 / 2,700.  Loads: 48 pages of 3.06 MiB move at 57.0 GB/s with 16, 57.2 with 20, 57.4
// with 24 or 32; 16 x 36 pages of 8 KiB in 95, 94, 92 and 92 us.
#ifndef KVX_STATE_HOST_WGS_PACK
#define KVX_STATE_HOST_WGS_PACK 32
#endif
#ifndef KVX_STATE_HOST_WGS_UNPACK
#define KVX_STATE_HOST_WGS_UNPACK 24
#endif

// Cache-policy bits of buffer loads and stores, and descriptor word 3 of a raw (untyped) buffer.
constexpr int kNt = 2, kSc1 = 16, kRawBuffer = 0x00020000;

// A piece on its way, one vector per lane.
struct Piece {
    uint8_t *dst;
    int bytes;
    int skip;  // bytes of lanes before the piece's first
    svec16 data;
};

// Start piece q of the launch (pieces run [snapshot k][layer g][piece of the page]): issue its reads.  The
// buffer's range ends with the piece, so lanes beyond a short piece's end read zeros and write nothing: no
// branch, no lane address, and so nothing that waits for an earlier piece's reads.
template <int DIR, bool LINES>
__device__ __forceinline__ void start_piece(const StateArgs &a, int q, Piece &p) {
    const int t = a.piece0 + q, pages = divide(t, a.by_ppp);
    const int page_id = a.page0 + pages;  // k*G + g
    const int k = divide(page_id, a.by_layers), g = page_id - k * a.G;
    const int j = t - pages * a.ppp;
    int64_t start = static_cast<int64_t>(j) * a.piece;
    uint8_t *page = a.layer[g] + a.page[k] * a.page_stride;
    uint8_t *packed = a.base + a.off[k] + static_cast<int64_t>(g) * a.page_bytes;
    if constexpr (LINES) {
        const int64_t low = start - (static_cast<int>(reinterpret_cast<uintptr_t>(packed)) & (kHostLine - 1));
        start = max(low, int64_t{0});
        p.skip = static_cast<int>(start - low);
        p.bytes = static_cast<int>(max(min(low + a.piece, a.page_bytes) - start, int64_t{0}));
    } else {
        p.skip = 0;
        p.bytes = j == a.ppp - 1 ? a.last_piece : a.piece;
    }
    page += start;
    packed += start;
    p.dst = DIR == kPack ? packed : page;
    const __amdgpu_buffer_rsrc_t src =
        __builtin_amdgcn_make_buffer_rsrc(DIR == kPack ? page : packed, 0, p.bytes, kRawBuffer);
    // (A lane before the piece has a negative offset, which the range check takes for one far beyond it.)
    p.data = __builtin_amdgcn_raw_buffer_load_b128(src, static_cast<int>(threadIdx.x) * 16 - p.skip, 0, kNt);
}

// Write a started piece to its place; "nt sc1" where the gather kernels' stores take it (into the mapped
// pool and into the cache's pages).
template <int DIR, bool HOST_SIDE>
__device__ __forceinline__ void finish_piece(const Piece &p) {
    const __amdgpu_buffer_rsrc_t dst = __builtin_amdgcn_make_buffer_rsrc(p.dst, 0, p.bytes, kRawBuffer);
    __builtin_amdgcn_raw_buffer_store_b128(p.data, dst, static_cast<int>(threadIdx.x) * 16 - p.skip, 0,
                                           DIR == kUnpack || HOST_SIDE ? kNt | kSc1 : kNt);
}

// LINES: a host-side launch whose pages are cut at the lines of their packed bytes.
template <int DIR, bool HOST_SIDE, bool LINES = false>
__global__ __launch_bounds__(kThreads) void state_kernel(const StateArgs a) {
    if constexpr (!HOST_SIDE) {
        Piece p;
        start_piece<DIR, LINES>(a, blockIdx.x, p);
        finish_piece<DIR, HOST_SIDE>(p);
    } else {
        // Two pieces in turn, by name: copying one to the other would wait for its reads.
        const int end = a.npieces, step = static_cast<int>(gridDim.x);
        int q = static_cast<int>(blockIdx.x);  // the grid has at most npieces workgroups
        Piece even, odd;
        start_piece<DIR, LINES>(a, q, even);
        while (true) {
            q += step;
            if (q >= end) {
                finish_piece<DIR, HOST_SIDE>(even);
                return;
            }
            start_piece<DIR, LINES>(a, q, odd);
            finish_piece<DIR, HOST_SIDE>(even);
            q += step;
            if (q >= end) {
                finish_piece<DIR, HOST_SIDE>(odd);
                return;
            }
            start_piece<DIR, LINES>(a, q, even);
            finish_piece<DIR, HOST_SIDE>(odd);
        }
    }
}

}  // namespace

hipError_t launch_state(const StateArgs &args, Direction dir, bool host_side, hipStream_t stream) {
    if (args.npieces <= 0)
        return hipSuccess;
    const void *fn;
    if (host_side && args.lines)
        fn = dir == kPack ? reinterpret_cast<const void *>(&state_kernel<kPack, true, true>)
                          : reinterpret_cast<const void *>(&state_kernel<kUnpack, true, true>);
    else if (host_side)
        fn = dir == kPack ? reinterpret_cast<const void *>(&state_kernel<kPack, true>)
                          : reinterpret_cast<const void *>(&state_kernel<kUnpack, true>);
    else
        fn = dir == kPack ? reinterpret_cast<const void *>(&state_kernel<kPack, false>)
                          : reinterpret_cast<const void *>(&state_kernel<kUnpack, false>);
    StateArgs a = args;
    a.last_piece = static_cast<int32_t>(a.page_bytes - (a.ppp - 1) * static_cast<int64_t>(a.piece));
    a.by_ppp = divisor(a.ppp);
    a.by_layers = divisor(a.G);
    const int wgs = dir == kPack ? KVX_STATE_HOST_WGS_PACK : KVX_STATE_HOST_WGS_UNPACK;
    const int grid = host_side ? std::min(a.npieces, wgs) : a.npieces;
    void *kargs[] = {&a};
    return hipLaunchKernel(fn, dim3(static_cast<uint32_t>(grid)), dim3(kThreads), kargs, 0, stream);
}

}  // namespace kvx
