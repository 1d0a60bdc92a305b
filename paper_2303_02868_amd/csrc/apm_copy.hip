// Gather / scatter between contiguous tensors and page storage: the layout's segments, each inside
// one page, copied bit for bit.  HBM-bound (read n + write n bytes).
//
// One grid over the fixed-size chunks of all segments (GridMap: classes of segment lengths); chunks beyond a
// segment's end exit at once.  Every lane moves 128 bits with contiguous wavefront accesses, whatever the
// alignment of the two addresses (see apm_seg_copy_kernel).
#include <cstring>
#include <type_traits>
#include "apm_internal.h"

namespace apm {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kNT = 2, kSC1 = 16;  // cache policies: non-temporal; written through
typedef __amdgpu_buffer_rsrc_t Rsrc;
__device__ __forceinline__ Rsrc make_rsrc(const void* base, int bytes) {  // accesses beyond it read zero / are dropped
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00027000);
}

// nvec vectors (at most a workgroup's), both addresses 16-byte aligned.
__device__ __forceinline__ void copy_vectors(const char* src, char* dst, int nvec) {
    const Rsrc S = make_rsrc(src, nvec * 16), D = make_rsrc(dst, nvec * 16);
    const int o = (int)threadIdx.x * 16;
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_amdgcn_raw_buffer_load_b128(S, o, 0, kNT), D, o, 0, kNT | kSC1);
}

// The same from a source at any byte address, which the target's unaligned access mode (the compiler relies
// on it for this type) serves with one 128-bit load.
typedef u32x4 __attribute__((aligned(1))) u32x4_any;
__device__ __forceinline__ void copy_vectors_unaligned(const char* src, char* dst, int nvec) {
    if ((int)threadIdx.x >= nvec) return;
    const u32x4 x = *reinterpret_cast<const u32x4_any*>(src + (int)threadIdx.x * 16);
    __builtin_amdgcn_raw_buffer_store_b128(x, make_rsrc(dst, nvec * 16), (int)threadIdx.x * 16, 0, kNT | kSC1);
}

// The same from a source `off` bytes (1 .. 15) beyond the aligned address `base`; the vectors base[0 .. nvec] are
// read, all of them inside the source.  A lane loads one aligned vector and takes the rest of what it
// stores from the next lane (the last one loads it).
template <int WORDS>
__device__ __forceinline__ u32x4 shifted(const u32x4& x, const u32x4& edge, uint32_t bytes) {
    uint32_t w[8] = {x[0], x[1], x[2], x[3], 0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j <= WORDS; ++j)  // lane i takes lane i + 1's word; the last lane keeps that of `edge`
        w[4 + j] = (uint32_t)__builtin_amdgcn_update_dpp((int)edge[j], (int)x[j], 0x130, 0xf, 0xf, false);
    u32x4 out;
#pragma unroll
    for (int j = 0; j < 4; ++j) out[j] = __builtin_amdgcn_alignbyte(w[j + WORDS + 1], w[j + WORDS], bytes);
    return out;
}
__device__ __forceinline__ void copy_vectors_shifted(const char* base, int off, char* dst, int nvec) {
    const Rsrc S = make_rsrc(base, (nvec + 1) * 16), D = make_rsrc(dst, nvec * 16);
    const int o = (int)threadIdx.x * 16;
    const u32x4 x = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(S, o, 0, 0));
    u32x4 edge = u32x4{0u, 0u, 0u, 0u};
    if (((int)threadIdx.x & 63) == 63) edge = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(S, o + 16, 0, 0));
    const uint32_t bytes = (uint32_t)off & 3u;
    u32x4 y;
    switch (off >> 2) {
        case 0: y = shifted<0>(x, edge, bytes); break;
        case 1: y = shifted<1>(x, edge, bytes); break;
        case 2: y = shifted<2>(x, edge, bytes); break;
        default: y = shifted<3>(x, edge, bytes); break;
    }
    __builtin_amdgcn_raw_buffer_store_b128(y, D, o, 0, kNT | kSC1);
}

// ALIGNED: every address is a multiple of 16; vector for vector, stores written through besides non-temporal: 840 M
// bf16 elements 539 us a call without, 521 with.  From kManyBytes on in workgroups of one wavefront: 502
// (of two, with one, two or four vectors a lane: 517 to 570); below, dispatching those takes longer than it gains (us, of one /
// of four: 43 MB 20.3 / 16.6, 95 MB 34.6 / 33.5, 142 MB 45.2 / 47.4, 202 MB 64.1 / 65.7).  In workgroups of one also
// where no segment has more than kShortBytes, aligned or not: the other three would have nothing to do, but keep
// their places until the stores of the first have gone through (us, of one / of four: 100 000 segments of 128 bytes 22.8 / 43.6, 65 536
// of 1 KB 21.4 / 48.9, 30 000 of 1.2 KB 47 / 54, 65 536 of 2 KB 40.1 / 40.1, 8192 of 4 KB 10.7 / 10.0).
// Otherwise (views of one flat buffer, odd numels) the stores are still aligned
// 128-bit vectors, the destination's first and last bytes go byte by byte (by the segment's first
// workgroup), and the vectors in between take whatever source alignment that leaves:
//   into tensors  the stores start on a cache line, vectors are shifted between lanes, written through besides:
//                 840 M bf16 elements, odd widths, 574 -> 544 us, 122 M fp32 162 -> 157;
//   into pages    that is slower (561 -> 601 us, 159 -> 168): 128-bit loads at the address itself, with the default policy, as a
//                 wavefront's first and last line are its neighbours' too, and stores written through (non-temporal loads and plain
//                 non-temporal stores / like this, bf16, the same buffers again and again: 17 M elements 14.6 / 11.8 us, 34 M 24.4 / 21.2, 47 M
//                 32.6 / 27.4, 122 M 78.4 / 64.8, 870 M 551 / 538; several in turn, 122 M 82.6 / 82.2).
//
// A call brings nothing but the tensors' addresses, and these travel in the kernel arguments
// (SegArgsInline): descriptors staged through a pinned ring cost the GPU an upload and two event packets,
// 15 us between one call's copy and the next one's.  All classes are one grid.  Whole calls with all of the
// above: 124 M fp32 elements out of their pages 160 us -> 151, 840 M bf16 539 -> 495; flat views, 122 M
// bf16 into pages 83.8 -> 81.4, 122 M fp32 out of pages 161 -> 154.
struct SegArgs {
    GridClass small[kMaxExtentClasses - 1];
    const uint64_t* ptrs;     // the tensors' addresses
};
struct SegArgsInline {
    GridClass small[kMaxExtentClasses - 1];
    uint64_t ptrs[kArgWords]; // of the tensors from tensor_begin
};
constexpr int kThreads = 256, kManyThreads = 64;
constexpr int64_t kManyBytes = (int64_t)128 << 20;
constexpr int64_t kShortBytes = 2048;
template <int THREADS> constexpr int64_t kChunk = (int64_t)THREADS * 16;

template <int THREADS, bool ALIGNED, class Args>
__global__ __launch_bounds__(THREADS) void apm_seg_copy_kernel(const SegRec* segs, char* region, uint32_t large_at,
                                                                                    uint32_t per, uint32_t mul, uint32_t shift, int32_t elem_log2,
                                                                                    int32_t to_pages, int32_t tensor_begin, Args args) {
    typedef int i32x8 __attribute__((ext_vector_type(8)));
    typedef const i32x8 __attribute__((address_space(4))) * Const;
    static_assert(sizeof(SegRec) == sizeof(i32x8), "a segment is one scalar load");
    int item;
    uint32_t x;
    grid_item(large_at, GridDiv{per, mul, shift}, args.small, blockIdx.x, &item, &x);
    const SegRec r = __builtin_bit_cast(SegRec, *(Const)reinterpret_cast<const i32x8*>(segs + item));
    char* in_tensor = reinterpret_cast<char*>(args.ptrs[r.tensor - tensor_begin]) + (r.tensor_off << elem_log2);
    char* in_page = region + (r.page_elem << elem_log2);
    const char* src = to_pages ? in_tensor : in_page;
    char* dst = to_pages ? in_page : in_tensor;
    const int64_t nbytes = (int64_t)r.n << elem_log2;
    const int64_t start = (int64_t)x * kChunk<THREADS>;
    if (start >= nbytes) return;
    if (ALIGNED || ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15u) == 0) {
        const int64_t len = nbytes - start < kChunk<THREADS> ? nbytes - start : kChunk<THREADS>;
        src += start;
        dst += start;
        const int nvec = (int)(len >> 4);
        copy_vectors(src, dst, nvec);
        const int tail = (int)(len & 15);  // only the last chunk of a segment can have one
        if ((int)threadIdx.x < tail) dst[((int64_t)nvec << 4) + threadIdx.x] = src[((int64_t)nvec << 4) + threadIdx.x];
        return;
    }
    const uint32_t line = to_pages ? 16u : 128u;
    int64_t head = (int64_t)(-(uint32_t)reinterpret_cast<uintptr_t>(dst) & (line - 1));
    int off = 0;  // of the vectors to be shifted
    if (!to_pages) {
        off = (int)((reinterpret_cast<uintptr_t>(src) + (uint64_t)head) & 15u);
        if (off > head) head += 16;  // the first vector read starts `off` bytes before the first byte stored
    }
    if (head > nbytes) head = nbytes;
    int64_t body = (nbytes - head) & ~(int64_t)15;
    if (off > 0 && body > 0 && nbytes - head - body < 16 - off) body -= 16;  // and the last one ends 16 - off beyond
    if (x == 0) {
        const int64_t tail_at = head + body;
        const int tail = (int)(nbytes - tail_at), t = (int)threadIdx.x;
        for (int k = t; k < (int)head; k += THREADS) dst[k] = src[k];
        if (t < tail) dst[tail_at + t] = src[tail_at + t];
    }
    if (start >= body) return;
    const int nvec = (int)((body - start < kChunk<THREADS> ? body - start : kChunk<THREADS>) >> 4);
    src += head + start;
    dst += head + start;
    if (off > 0) copy_vectors_shifted(src - off, off, dst, nvec);
    else if (!to_pages) copy_vectors(src, dst, nvec);
    else copy_vectors_unaligned(src, dst, nvec);
}

// Both directions of an exchange of the staged mode's ring or the scheduled step in one kernel: the fp32 classes of incoming pages
// move from pinned host pages into staging slots while those of outgoing pages move from
// other slots back to their host pages.  A fixed, small number of wavefronts strides over 4 KiB
// items (one 1 KiB span per wavefront instruction, 4 per class and direction in flight); the link
// is the bound, not the GPU.  One kernel driving both directions keeps them balanced: measured on
// 3 x 1 GiB each way, 49.3 GB/s each way with 48 wavefronts, against 40-42 when half of the
// wavefronts serve each direction (or two kernels do), 48.6 for two runtime copies when the
// runtime overlaps them, and 28 when it does not.  Within an item all host reads are issued first
// (they have the longest latency), then the staging reads; the host writes go out before the
// staging writes (interleaving the two directions instruction by instruction: 47.2 GB/s).
// Only the used extent of each page is moved: the update never touches the rest.
constexpr int kDuplexItem = 4096;  // bytes per class, direction and wavefront iteration
constexpr int kDuplexU = kDuplexItem / (64 * 16);

// A wavefront's position in one direction's run of pages.  A wavefront visits the items congruent
// to its number modulo the wavefront count, and of those only the ones that hold used bytes: items
// beyond a page's used extent are not visited one by one, the cursor hops along its stride to the
// next page.  Skipping them (instead of spending an iteration on an item that is empty in one
// direction) keeps the two directions of an exchange in step when their nearly empty pages sit at
// different positions -- a fifth of the items of a 32-page exchange on a GPT-shaped layout.
// With a page table a page is a whole number of items (items_per_page), so an item lies in one
// page; without one the run is treated as a single page.
struct DuplexCursor {
    unsigned item;        // index in the run (>= n_items: nothing left)
    unsigned page;        // page of the run the item lies in
    unsigned in_page;     // index of the item within that page
    unsigned page_items;  // items of that page that hold used bytes
    int tail;             // bytes of the last of them
    int limit;            // bytes of the current item to move (0: nothing left)
};

struct DuplexRun {
    const int32_t* used;  // page table entry of the run's first page, or nullptr
    unsigned n_items, items_per_page, stride;
    int64_t bytes;
};

__device__ __forceinline__ void duplex_page(const DuplexRun& r, DuplexCursor& c) {
    // The page table does not change while the kernel runs; read through the constant address
    // space it is a scalar load that only its own use waits for (as a plain global load it is a
    // vector load followed by a wait for every outstanding memory operation).
    typedef const int32_t __attribute__((address_space(4))) * ConstTable;
    const int64_t used_bytes = (((int64_t)((ConstTable)r.used)[c.page] + 7) & ~(int64_t)7) * 4;  // up to 2^32
    c.page_items = (unsigned)((used_bytes + kDuplexItem - 1) / kDuplexItem);
    c.tail = (int)(used_bytes - (int64_t)(c.page_items ? c.page_items - 1 : 0) * kDuplexItem);
}

// Settles the cursor on the first item at or after its position, on its stride, that holds used
// bytes.  Every turn of the loop either returns or moves on to a later page of the run.
__device__ __forceinline__ void duplex_settle(const DuplexRun& r, DuplexCursor& c) {
#pragma unroll 1
    for (;;) {
        if (c.item >= r.n_items) {
            c.limit = 0;
            return;
        }
        if (c.in_page >= r.items_per_page) {  // crossed into the next page (item < n_items: it exists)
            c.in_page -= r.items_per_page;
            ++c.page;
            duplex_page(r, c);
            continue;
        }
        if (c.in_page < c.page_items) {
            c.limit = c.in_page + 1 == c.page_items ? c.tail : kDuplexItem;
            return;
        }
        const unsigned hops = (r.items_per_page - c.in_page + r.stride - 1) / r.stride;  // >= 1
        c.item += hops * r.stride;
        c.in_page += hops * r.stride;
    }
}

__device__ __forceinline__ void duplex_start(const DuplexRun& r, DuplexCursor& c, unsigned worker) {
    c.item = c.in_page = worker;
    c.page = 0;
    c.limit = 0;
    if (r.used) {
        c.page_items = 0;
        c.tail = 0;
        if (r.n_items > 0) duplex_page(r, c);
    } else {
        c.page_items = r.n_items;
        c.tail = (int)(r.bytes - (int64_t)(r.n_items ? r.n_items - 1 : 0) * kDuplexItem);
    }
    duplex_settle(r, c);
}

typedef const u32x4 __attribute__((address_space(1))) * DuplexIn;
typedef u32x4 __attribute__((address_space(1))) * DuplexOut;

// One item of each direction: all loads, then all stores, in one basic block (FULL) so that the
// stores wait for their own loads only, in issue order.
template <bool FULL, bool WT>
__device__ __forceinline__ void duplex_item(const DuplexCopy& a, int64_t base_in, int64_t base_out, int lane_off,
                                            int lim_in, int lim_out) {
    u32x4 vin[3][kDuplexU], vout[3][kDuplexU];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int u = 0; u < kDuplexU; ++u)
            if (FULL || lane_off + u * 1024 < lim_in) vin[k][u] = __builtin_nontemporal_load((DuplexIn)(a.in_src[k] + base_in + u * 1024));
    __builtin_amdgcn_sched_barrier(0);  // keep the order written here: host reads first
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int u = 0; u < kDuplexU; ++u)
            if (FULL || lane_off + u * 1024 < lim_out) vout[k][u] = __builtin_nontemporal_load((DuplexIn)(a.out_src[k] + base_out + u * 1024));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int u = 0; u < kDuplexU; ++u)
            if (FULL || lane_off + u * 1024 < lim_out) {
                // WT: written through at system scope.  A non-temporal store to host memory may rest
                // in the L2 as a dirty line, and the write-back that ends every kernel of any other
                // stream then pushes it across PCIe: those kernels pay for this kernel's writes.
                DuplexOut q = (DuplexOut)(a.out_dst[k] + base_out + u * 1024);
                // (hand-written because no builtin takes a cache policy for a 128-bit global store.
                // The compiler does not know that this is a store whose data registers are read a
                // little after issue -- for its own stores of more than 64 bits it keeps the next
                // instruction from overwriting them -- so the wait states go in by hand.)
                if (WT) asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(q), "v"(vout[k][u]) : "memory");
                else __builtin_nontemporal_store(vout[k][u], q);
            }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int u = 0; u < kDuplexU; ++u)
            if (FULL || lane_off + u * 1024 < lim_in) __builtin_nontemporal_store(vin[k][u], (DuplexOut)(a.in_dst[k] + base_in + u * 1024));
}

template <bool WT>
__global__ __launch_bounds__(1024) void apm_duplex_copy_kernel(DuplexCopy a, int n_workers) {
    const int lane = (int)threadIdx.x & 63;
    const int waves_per_wg = (int)blockDim.x / 64;
    const int worker = (int)blockIdx.x * waves_per_wg + __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
    if (worker >= n_workers) return;
    const unsigned in_items = (unsigned)((a.in_bytes + kDuplexItem - 1) / kDuplexItem);
    const unsigned out_items = (unsigned)((a.out_bytes + kDuplexItem - 1) / kDuplexItem);
    const int lane_off = lane * 16;
    // Each direction has its own cursor over the items that hold used bytes; the next positions
    // are worked out (scalar arithmetic, a scalar load per page) before the current item's data moves.
    const unsigned ipp = a.used ? a.items_per_page : 0xffffffffu;
    const DuplexRun rin{a.used ? a.used + a.in_first_page : nullptr, in_items, ipp, (unsigned)n_workers, a.in_bytes};
    const DuplexRun rout{a.used ? a.used + a.out_first_page : nullptr, out_items, ipp, (unsigned)n_workers, a.out_bytes};
    DuplexCursor in, out;
    duplex_start(rin, in, (unsigned)worker);
    duplex_start(rout, out, (unsigned)worker);
#pragma unroll 1
    while (in.limit > 0 || out.limit > 0) {
        // byte counts and used extents are multiples of 16: a 16-byte vector is wholly in or out
        const int cur_in = in.limit, cur_out = out.limit;
        const int64_t base_in = (int64_t)in.item * kDuplexItem + lane_off;
        const int64_t base_out = (int64_t)out.item * kDuplexItem + lane_off;
        if (cur_in > 0) {
            in.item += (unsigned)n_workers;
            in.in_page += (unsigned)n_workers;
            duplex_settle(rin, in);
        }
        if (cur_out > 0) {
            out.item += (unsigned)n_workers;
            out.in_page += (unsigned)n_workers;
            duplex_settle(rout, out);
        }
        if (cur_in >= kDuplexItem && cur_out >= kDuplexItem) duplex_item<true, WT>(a, base_in, base_out, lane_off, cur_in, cur_out);
        else duplex_item<false, WT>(a, base_in, base_out, lane_off, cur_in, cur_out);
    }
}

}  // namespace

hipError_t launch_duplex_copy(const DuplexCopy& d, int wavefronts, int per_wg, hipStream_t s) {
    const int64_t longer = d.in_bytes > d.out_bytes ? d.in_bytes : d.out_bytes;
    if (longer <= 0) return hipSuccess;
    const int64_t n_items = (longer + kDuplexItem - 1) / kDuplexItem;
    const int workers = (int)(n_items < wavefronts ? n_items : wavefronts);
    if (per_wg < 1 || per_wg > 16) per_wg = 1;
    DuplexCopy a = d;
    if (a.page_bytes <= 0 || a.page_bytes % kDuplexItem != 0) a.used = nullptr;
    a.items_per_page = a.used ? (uint32_t)(a.page_bytes / kDuplexItem) : 0u;
    if (n_items >= ((int64_t)1 << 31)) return hipErrorInvalidValue;  // 8 TiB per class and kernel
    const dim3 grid((unsigned)((workers + per_wg - 1) / per_wg)), block((unsigned)(per_wg * 64));
    if (a.host_store_policy != 0) hipLaunchKernelGGL(apm_duplex_copy_kernel<true>, grid, block, 0, s, a, workers);
    else hipLaunchKernelGGL(apm_duplex_copy_kernel<false>, grid, block, 0, s, a, workers);
    return hipGetLastError();
}

hipError_t launch_seg_copy(const SegCopy& c, const SegLaunch* launches, int64_t n_launches, hipStream_t s) {
    for (int64_t i = 0; i < n_launches; ++i) {
        const SegLaunch& l = launches[i];
        SegArgsInline in;
        if (!c.on_device) std::memcpy(in.ptrs, c.ptrs + l.tensor_begin, (size_t)l.tensor_count * sizeof(uint64_t));
        int64_t bytes = 0;
        for (int k = 0; k < l.n_cls; ++k) bytes += l.cls[k].sum_used * c.elem_bytes;
        auto go = [&](auto aligned, auto workgroup) -> int {
            constexpr bool kAligned = decltype(aligned)::value;
            constexpr int threads = decltype(workgroup)::value;
            return for_each_grid(l.cls, l.n_cls, threads, c.max_workgroups,
                [&](const ExtentClass& e) { return (e.max_used * c.elem_bytes + kChunk<threads> - 1) / kChunk<threads>; },
                [&](const GridMap& map, int64_t workgroups, int64_t first) -> int {
                    auto start = [&](auto kernel, auto& args, int32_t tensor_begin) {
                        std::memcpy(args.small, map.small, sizeof map.small);
                        hipLaunchKernelGGL(kernel, dim3((unsigned)workgroups), dim3(threads), 0, s, c.segs + first, c.region, map.large_at, map.large.per,
                                           map.large.mul, map.large.shift, c.elem_bytes == 4 ? 2 : 1, c.to_pages, tensor_begin, args);
                    };
                    SegArgs on_device{{}, c.ptrs};
                    if (c.on_device) start(apm_seg_copy_kernel<threads, kAligned, SegArgs>, on_device, 0);
                    else start(apm_seg_copy_kernel<threads, kAligned, SegArgsInline>, in, l.tensor_begin);
                    return (int)hipGetLastError();
                });
        };
        const bool is_short = l.n_cls > 0 && l.cls[0].max_used * c.elem_bytes <= kShortBytes;
        const std::integral_constant<int, kThreads> four;
        const std::integral_constant<int, kManyThreads> one;
        const hipError_t e = (hipError_t)(c.aligned ? (is_short || bytes >= kManyBytes ? go(std::true_type{}, one) : go(std::true_type{}, four))
                                                    : (is_short ? go(std::false_type{}, one) : go(std::false_type{}, four)));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace apm
