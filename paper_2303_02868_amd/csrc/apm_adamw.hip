// Page AdamW kernels for gfx950:
//   apm_grad_reduce_kernel    per (page, slice) sum of squares (fp64) and any-nonzero of g16
//   apm_grad_finalize_kernel  per page: norm, clip scale, skip decision -> the page's record
//   apm_page_recs_kernel      the page records when no reduce pass is needed
//   apm_stage_kernel          the same from a call's page list and tensor addresses
//   apm_adamw_kernel          the fused update (optionally gathering g16 from / scattering p16 to
//                             the caller's tensors), one workgroup per page slice;
//                             apm_adamw_run_kernel the same over consecutive pages of the classes
//   apm_adamw_call_kernel     the same where a call's list and addresses fit its arguments: no pass before it
//   apm_adamw_live_kernel     the same over the pages that the finalize pass did not skip
//   apm_adamw_clip_kernel     norms, clip scales and the update in one grid
//   apm_adamw_stride_kernel   the same slice body run by a fixed, small number of wavefronts that
//                             stride over all slices (fp32 classes in host memory across PCIe);
//                             apm_adamw_staged_kernel through staging slots in device memory
//   apm_grad_take_kernel      g' <- g or g' += g for the buffered gradient of the delayed path
//
// All are HBM-bandwidth bound (no reuse, ~50 VALU operations per element at most), so the design
// is about memory access only: every wavefront instruction touches one fully contiguous span
// (1 KiB for the 128-bit fp32 accesses, 512 B for the 64-bit bf16 accesses), each lane keeps
// several independent loads in flight, and a workgroup never straddles a page.
//
// Work decomposition: one grid over the fixed-size slices of all listed pages (GridMap; for a run of pages
// grid.y walks the pages); slices that start beyond the page's used extent exit at once.  The page table (`used`) is read
// on the device; the host, which knows the extents from the layout, only sizes the grids (pages
// grouped into extent classes) so that few workgroups are launched for nothing.  All classes are one
// grid, the nearly empty pages first: as a launch of their own they cost 8 to 11 us after the large
// ones, and behind the large ones in the same grid their latencies come at the end of the call.  us a call from and
// to tensors, launches of their own / one grid / nearly empty pages last: 124 M parameters 538 / 525 / 526; 4.8 M in 256 K
// pages 31.3 / 26.2 / 25.8, with clipping 40.5 / 32.7 / 36.7; 11 M with clipping 67.9 / 59.5 / 62.7.
#include <cstring>
#include <type_traits>

#include "apm_internal.h"

namespace apm {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kWave = 64;

__device__ __forceinline__ double shfl_xor_f64(double x, int off) {
    int lo = __double2loint(x), hi = __double2hiint(x);
    lo = __shfl_xor(lo, off, kWave);
    hi = __shfl_xor(hi, off, kWave);
    return __hiloint2double(hi, lo);
}

// Sum over the wavefront in a fixed butterfly order; every lane ends with the same value.
__device__ __forceinline__ double wave_sum_f64(double x) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x += shfl_xor_f64(x, off);
    return x;
}

__device__ __forceinline__ uint32_t wave_or_u32(uint32_t x) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x |= (uint32_t)__shfl_xor((int)x, off, kWave);
    return x;
}

__device__ __forceinline__ float bf16lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Round-to-nearest-even of an fp32 value to bf16 bits, on the integer representation.
__device__ __forceinline__ uint32_t f32_to_bf16_rne(float x) {
    const uint32_t u = __float_as_uint(x);
    // both forms are computed and one is selected: a branch here would split the update kernel's
    // body into basic blocks (see full_slice)
    const uint32_t nan = (u >> 16) | 0x0040u;
    const uint32_t rne = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    return (u & 0x7FFFFFFFu) > 0x7F800000u ? nan : rne;
}

// ---- tunables (defaults measured on MI355X; see the sweep notes next to each) ----------------
#ifndef APM_FAST_RCP_SQRT
// 1: hardware 1-ulp reciprocal and square root instead of the correctly rounded sequences.
// Measured slower (6.0 vs 6.25 TB/s): the kernel is not ALU-bound, so the exact forms stay.
#define APM_FAST_RCP_SQRT 0
#endif
#ifndef APM_REDUCE_U
#define APM_REDUCE_U 4          // 128-bit loads in flight per lane in the reduce kernel
#endif
// The update's wavefronts are workgroups of their own, one per page slice of U vectors per lane and
// fp32 class, and request dynamic LDS for no purpose other than capping how many of them a CU
// (160 KiB) holds: with four read and four write streams per wavefront, more resident wavefronts
// lower the achieved HBM bandwidth, and short wavefronts started in address order keep the streams
// closer together than long ones.  Measured on 1.07 G elements, TB/s, U = 1 at 16 / 12 / 10 wavefronts per
// CU: 6.43 / 6.60 / 6.55; U = 2 at 10 / 8 / 6: 6.25 / 6.31 / 6.45; U = 4 at 5 / 4: 6.32 / 6.33; a
// fixed grid of wavefronts that walk the slices with their next loads in flight: 5.3.
// Whole calls, U = 4 at 5, U = 2 at 8, U = 1 at 12, U = 1 at 11: 124 M parameters 563 / 580 / 548 / 544 us, 1.3 B with
// clipping 6308 / 6361 / 6050 / 5990.
#ifndef APM_UPDATE_U
#define APM_UPDATE_U 1
#endif
#ifndef APM_UPDATE_LDS
#define APM_UPDATE_LDS 14848
#endif
// Launches with few elements: here workgroups of short pages that find nothing to do weigh more, and a CU takes
// 17 wavefronts.  From and to tensors (us a call at 11 / 17: 4 M elements in 64 K pages 26.9 / 24.5, 16 M in 1 M
// pages 95.1 / 89.3, 64 M 326 / 343; with clipping, at 12 / 17: 35.8 / 31.5, 112 / 101) up to kFewElems; from and
// to the page classes only where all wavefronts then run at once (1 M 5.9 / 5.5, 2 M 10.3 / 9.5, 8 M 36.7 / 37.1;
// with clipping 14.3 / 13.9, 18.8 / 18.2, 45.2 / 45.5).
constexpr int64_t kFewElems = (int64_t)24 << 20, kFewRunElems = (int64_t)2 << 20;
constexpr int kFewLds = 9216;
// Bare runs up to this size store state non-temporal only.  Their state fits the L2s (12 B an element of 32 MiB), where what a
// call leaves serves the next one on the same pages, and written-through stores end later: one state again and again gains,
// three states in turn lose, and the line is where the first stops gaining (us a call, written through / not, again and again; in turn:
// 1 M elements 6.2 / 5.0; 6.4 / 6.0, 1.6 M 9.1 / 8.2; 8.9 / 9.0, 2.1 M 11.1 / 10.2; 11.0 / 11.5, 2.4 M 11.6 / 11.7; 11.9 / 12.5, 2.9 M 13.7 /
// 14.0; 13.8 / 14.6, 3.7 M 16.6 / 17.6; 17.9 / 18.1).  The other forms are written through at every size: in turn they gain
// up to 4 % or lose up to 2; again and again they take up to 0.7 us more below 1 M elements (0.6 M with clipping 12.5 / 12.2 in pages,
// 14.0 / 14.1 from tensors; 0.9 M 14.0 / 14.1, 14.2 / 13.3), from there on the sign of the difference varies with the layout.
constexpr int64_t kNtRunElems = (int64_t)2 << 20;
constexpr int kWideU = 4;  // see wide_pays
unsigned update_lds(bool tensors, int64_t elems, unsigned lds) { return elems <= (tensors ? kFewElems : kFewRunElems) ? kFewLds : lds; }

// When pages may be skipped on the device (APM_SKIP_UNTOUCHED) the pages to update are known only there.
// Few slices: the plain grid, whose wavefronts leave if their page's record says skipped.  More: the finalize
// pass notes the other pages, and a grid of 1 / kSkipSpread of all slices' wavefronts (but kSkipWaves
// where there are that many slices) walks the slices of the noted pages, so that workgroups without work are
// few when most pages are skipped and no wavefront has more than kSkipSpread slices when none is.  A
// wavefront without work costs 0.2 ns of the call, one with many slices loses the address order that keeps
// the streams together, and in a small call its slices run one after the other on an idle chip.
// us a call, every page / every eighth page / no page with a gradient:
//   plain grid / grid of an eighth to a twelfth of the slices / two to four times that
//   512 slices       12 / 12 / 11      27 / 14 / 12      17 / 13 / 12
//   8 K              18 / 13 / 12      26 / 14 / 12      19 / 12 / 12
//   32 K             48 / 19 / 16      59 / 18 / 12      51 / 18 / 12
//   128 K           157 / 49 / 43     180 / 40 / 18     170 / 42 / 22
//   4 M            4877 / 1448 / 1194 5919 / 907 / 392 5424 / 999 / 537
constexpr int kSkipU = 1, kSkipSpread = 12, kSkipWaves = 8192, kSkipLds = 14848;
constexpr uint32_t kThroughSlack = 12288;  // see apm_adamw_live_kernel

// Gradient elements [e, e+8) of a page, read from its tenant tensors; elements that belong to no
// tenant (alignment gap, padding) read as zero.  e is a multiple of 8, as every tenant offset is,
// so a vector never straddles the start of the second tenant.
__device__ __forceinline__ u32x4 gather_g8(const PageRec& r, int e) {
    const int k = e >= r.off1 ? 1 : 0;
    const int left = r.end[k] - e;
    u32x4 w = u32x4{0u, 0u, 0u, 0u};
    if (left >= 8) {
        w = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(r.g[k] + e));
    } else if (left > 0) {  // last, partial vector of the tensor: never read past its end
        const uint16_t* src = r.g[k] + e;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (j < left) w[j >> 1] |= (uint32_t)src[j] << (16 * (j & 1));
    }
    return w;
}

__device__ __forceinline__ u32x2 gather_g4(const PageRec& r, int e) {
    const int k = e >= r.off1 ? 1 : 0;
    const int left = r.end[k] - e;
    u32x2 w = u32x2{0u, 0u};
    if (left >= 4) {
        w = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(r.g[k] + e));
    } else if (left > 0) {
        const uint16_t* src = r.g[k] + e;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j < left) w[j >> 1] |= (uint32_t)src[j] << (16 * (j & 1));
    }
    return w;
}

// bf16 parameters of page elements [e, e+4) written to the tenant tensor they belong to; elements
// of no tenant are dropped.
__device__ __forceinline__ void scatter_q4(const PageRec& r, int e, u32x2 o) {
    const int k = e >= r.off1 ? 1 : 0;
    const int left = r.end[k] - e;
    if (left >= 4) {
        __builtin_nontemporal_store(o, reinterpret_cast<u32x2*>(r.q[k] + e));
    } else if (left > 0) {
        uint16_t* dst = r.q[k] + e;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j < left) dst[j] = (uint16_t)(o[j >> 1] >> (16 * (j & 1)));
    }
}

typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
static_assert(sizeof(PageRec) == sizeof(i32x16) && sizeof(PageRun) == sizeof(i32x2), "a record is one scalar load");

// Through the constant address space these are scalar loads also in kernels that store before them; what
// they read was written by an earlier kernel (the one-pass kernel does not use the scale it gets this way).
// The empty statement keeps it one load: the compiler otherwise loads field by field where each is used, a round
// trip after the other.
__device__ __forceinline__ PageRec load_rec(const PageRec* at) {
    typedef const i32x16 __attribute__((address_space(4))) * Const;
    i32x16 w = *(Const)reinterpret_cast<const i32x16*>(at);
    asm("" : "+s"(w));
    return __builtin_bit_cast(PageRec, w);
}
__device__ __forceinline__ PageRun load_run(const PageRun* at) {
    typedef const i32x2 __attribute__((address_space(4))) * Const;
    return __builtin_bit_cast(PageRun, *(Const)reinterpret_cast<const i32x2*>(at));
}

static_assert(sizeof(PagePlace) == sizeof(i32x16) && sizeof(CallTables) == sizeof(i32x16), "one scalar load each");
__device__ __forceinline__ i32x16 load_16(const void* at) {
    typedef const i32x16 __attribute__((address_space(4), aligned(4))) * Const;
    return *(Const)reinterpret_cast<const i32x16*>(at);
}
// The record of a list position, which a stage kernel would have made (with GATHER / SCATTER the tensors' addresses): one dependent scalar
// load more than a record in memory, two with a list, from tables that stay in the scalar caches.  All that a step needs is fetched
// at once, the words of both tenants too.
__device__ __forceinline__ uint32_t call_word(const CallWords* c, uint32_t k) {
    typedef const uint32_t __attribute__((address_space(4))) * Const;
    return ((Const)c->word)[k];
}
template <bool GATHER, bool SCATTER>
__device__ __forceinline__ PageRec call_rec(const CallTables& t, const PagePlace& p, const CallWords* c) {
    uint32_t g[2] = {0, 0}, q[2] = {0, 0};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (GATHER) g[k] = call_word(c, (uint32_t)(t.g_at + p.tensor[k]));
        if (SCATTER) q[k] = call_word(c, (uint32_t)(t.q_at + p.tensor[k]));
    }
    if (GATHER || SCATTER) asm("" : "+s"(g[0]), "+s"(g[1]), "+s"(q[0]), "+s"(q[1]));
    PageRec r;
    r.used = p.used;
    r.scale = 1.0f;
    r.pofs = p.pofs;
    r.off1 = GATHER || SCATTER ? p.off1 : INT32_MAX;
    r.pad = 0;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        r.end[k] = GATHER || SCATTER ? p.end[k] : k == 0 ? (p.used + 7) & ~7 : 0;
        r.g[k] = reinterpret_cast<const uint16_t*>(t.g_base + ((uint64_t)g[k] << 4)) + (GATHER ? p.shift[k] : p.pofs);
        r.q[k] = reinterpret_cast<uint16_t*>(t.q_base + ((uint64_t)q[k] << 4)) + (SCATTER ? p.shift[k] : p.pofs);
    }
    return r;
}

// The workgroup's sum (wavefront butterfly, then wave 0..3) and OR, written by thread 0.
__device__ __forceinline__ void block_sum(double acc, uint32_t nz, double* s_acc, uint32_t* s_nz, double* sum, uint32_t* flag) {
    acc = wave_sum_f64(acc);
    nz = wave_or_u32(nz);
    const int wave = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        s_acc[wave] = acc;
        s_nz[wave] = nz;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double t = s_acc[0];
    uint32_t z = s_nz[0];
#pragma unroll
    for (int k = 1; k < kThreads / kWave; ++k) {
        t += s_acc[k];
        z |= s_nz[k];
    }
    *sum = t;
    *flag = z;
}

struct ReduceArgs {
    const uint16_t* g16;
    const int32_t* used;
    const int64_t* grad_pages;
    int64_t grad_first;
    int64_t list_offset;
    int64_t E;
    double* partials;
    uint32_t* nzflags;
    int32_t S;
    int32_t* live;        // nullable: its counts are to be cleared
    GridClass small[kMaxExtentClasses - 1];
};

// Per (page, slice): sum of squares in fp64 and OR of the magnitude bits of the slice's used
// gradient elements.  Slice 0 always writes (a zero for an empty page); other slices only when
// they hold used elements.  The fixed order (lane-sequential, wavefront butterfly, wave 0..3)
// makes the result independent of scheduling.  recs (gather only): from position a.list_offset.
// Without SUMS only whether any element is not zero is wanted: a slice whose first eighth says so is not read any further.
// (Whole calls, us, with sums / without: 1.08 G elements, an eighth of them live 946 / 896; 541 M, all live 3008 / 2860; 27 M, half live 85.3 /
// 78.2; 52 M, a tenth live 56.7 / 54.)
// Call: CallWords if the records are made from those (`recs` is not used then).
struct CallNone {};
template <bool GATHER, bool SUMS, class Call>
__global__ __launch_bounds__(kThreads) void apm_grad_reduce_kernel(const PageRec* recs, uint32_t large_at, uint32_t per, uint32_t mul,
                                                                   uint32_t shift, ReduceArgs a, Call call) {
    int item;
    uint32_t tile;
    grid_item(large_at, GridDiv{per, mul, shift}, a.small, blockIdx.x, &item, &tile);
    const int64_t i = a.list_offset + item;
    PageRec rec{};
    int64_t page = 0;
    int used;
    if constexpr (!std::is_same<Call, CallNone>::value) {
        uint32_t place = (uint32_t)i;
        if (call.t.listed) place = call_word(&call, 2 * place);
        const i32x16 at = load_16(call.t.places + place);
        rec = call_rec<GATHER, false>(call.t, __builtin_bit_cast(PagePlace, at), &call);
        used = rec.used;
        page = __builtin_bit_cast(PagePlace, at).page;
    } else if (GATHER) {
        rec = load_rec(recs + item);
        used = rec.used;
    } else {
        page = a.grad_pages ? a.grad_pages[i] : a.grad_first + i;
        used = a.used[page];
    }
    if (a.live && blockIdx.x == 0 && threadIdx.x < kMaxExtentClasses) a.live[threadIdx.x] = 0;
    const int start = (int)tile * kReduceTile;
    if (start >= used && tile != 0) return;
    const int end = min(start + kReduceTile, used);
    const uint16_t* g = GATHER ? nullptr : a.g16 + page * a.E;
    bool edge = false;  // gather only: this slice is not wholly inside one tenant
    if (GATHER) {
        const int k = start >= rec.off1 ? 1 : 0;
        // Wholly inside tenant k, counted in whole 8-element vectors (the fast path below loads
        // 16 bytes at a time and must not read past the tensor's last element): the slice reads
        // that tensor like a page.  A slice that holds a tensor's ragged end takes the per-vector
        // path, which reads that end element by element.
        if (start + (((end - start) + 7) & ~7) <= rec.end[k]) g = rec.g[k];
        else edge = true;
    }

    // the vector at e; elements at or beyond the extent are zero
    auto load = [&](int e) {
        u32x4 w = u32x4{0u, 0u, 0u, 0u};
        if (e < end) {
            if (GATHER && edge) w = gather_g8(rec, e);
            else w = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(g + e));
        }
        return w;
    };
    auto cut = [&](u32x4& w, int e) {
        if (e + 8 > end && e < end) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t x = w[j];  // selected: written in place, the compiler branches for every one of them
                if (e + 2 * j >= end) x = 0u;
                else if (e + 2 * j + 1 >= end) x &= 0x0000FFFFu;
                w[j] = x;
            }
        }
    };
    if (!SUMS) {
        constexpr int kSpans = kReduceTile / (kThreads * 8);
        const int e0 = start + (int)threadIdx.x * 8;
        auto any = [&](u32x4 w, int e) {
            cut(w, e);
            return (w[0] | w[1] | w[2] | w[3]) & 0x7FFF7FFFu;
        };
        uint32_t nz = any(load(e0), e0);
        if (!__syncthreads_or(nz != 0u) && start + kThreads * 8 < end) {
            u32x4 w[kSpans - 1];
#pragma unroll
            for (int u = 1; u < kSpans; ++u) w[u - 1] = load(e0 + u * (kThreads * 8));
#pragma unroll
            for (int u = 1; u < kSpans; ++u) nz |= any(w[u - 1], e0 + u * (kThreads * 8));
        }
        const int found = __syncthreads_or(nz != 0u);
        if (threadIdx.x == 0) a.nzflags[i * a.S + tile] = (uint32_t)found;
        return;
    }
    double acc0 = 0.0, acc1 = 0.0;
    uint32_t nz = 0;
    constexpr int U = APM_REDUCE_U;
    constexpr int kOuter = kReduceTile / (kThreads * 8 * U);
    static_assert(kOuter * kThreads * 8 * U == kReduceTile, "reduce tile must be a multiple of the unrolled span");
#pragma unroll 1
    for (int o = 0; o < kOuter; ++o) {
        const int e0 = start + o * (kThreads * 8 * U) + (int)threadIdx.x * 8;
        if (e0 - (int)threadIdx.x * 8 >= end) break;   // uniform: the whole span is beyond the extent
        u32x4 w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = load(e0 + u * (kThreads * 8));
#pragma unroll
        for (int u = 0; u < U; ++u) {
            cut(w[u], e0 + u * (kThreads * 8));
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t x = w[u][j];
                nz |= x & 0x7FFF7FFFu;
                const double lo = (double)bf16lo(x), hi = (double)bf16hi(x);
                acc0 = fma(lo, lo, acc0);
                acc1 = fma(hi, hi, acc1);
            }
        }
    }
    __shared__ double s_acc[kThreads / kWave];
    __shared__ uint32_t s_nz[kThreads / kWave];
    block_sum(acc0 + acc1, nz, s_acc, s_nz, a.partials + i * a.S + tile, a.nzflags + i * a.S + tile);
}

struct FinalizeArgs {
    const int32_t* used;
    const int64_t* grad_pages;
    const int64_t* state_pages;
    int64_t grad_first;
    int64_t state_first;
    int64_t n_listed;
    const double* partials;
    const uint32_t* nzflags;
    int32_t S;
    int32_t skip_mode;
    double max_norm;
    PageRec* recs;     // [n_listed]; as PageRun if `run`
    const uint16_t* g16;
    uint16_t* p16;
    int64_t E;
    int32_t* live;     // nullable: see kLiveInts
    int64_t cls_begin[kMaxExtentClasses];
    int32_t n_cls;
    bool by_page;      // partials and flags are indexed by page, not by position
    bool run;
    bool staged;       // the records hold everything but the scale already (caller's tensors)
    uint64_t* sums;    // one-pass launches: [n_listed * S], to be marked as not there yet
    float* grad_norm;  // nullable
    uint8_t* skip_mask;  // nullable
    const int32_t* out_index;  // nullable: list position -> index into grad_norm / skip_mask
    bool gather, scatter;
};

// The record of a page that is read from / written to the page classes.
__device__ __forceinline__ PageRec class_rec(int used, float scale, int64_t gpage, int64_t spage, int64_t E,
                                             const uint16_t* g16, uint16_t* p16) {
    PageRec r;
    r.used = used;
    r.scale = scale;
    r.pofs = spage * E;
    r.g[0] = r.g[1] = g16 + gpage * E;
    r.q[0] = r.q[1] = p16 + gpage * E;
    r.off1 = INT32_MAX;
    r.end[0] = (used + 7) & ~7;
    r.end[1] = 0;
    r.pad = 0;
    return r;
}

// min(1, c / (norm + 1e-6)) with plain IEEE propagation: an infinite norm gives 0, a NaN norm a NaN
// scale (the comparison is false for NaN), as the library optimizers do.  c <= 0: no clipping.
__device__ __forceinline__ float clip_scale(double norm, double c) {
    if (!(c > 0.0)) return 1.0f;
    const double sc = c / (norm + 1e-6);
    return sc > 1.0 ? 1.0f : (float)sc;
}

// What the one-pass kernel's wavefronts read until the value is there: bit patterns that no sum of
// squares and no scale has (a NaN with every bit set; the NaNs of the arithmetic carry at most the
// payload of a bf16).
constexpr uint64_t kNoSum = ~(uint64_t)0;
constexpr uint32_t kNoScale = ~(uint32_t)0;

// One wavefront per listed page (R pages, one after the other): combines the page's slice partials in a
// fixed order and turns them into the page's clip scale / skip decision and the optional outputs.
// The pages that are not skipped are noted by workgroup, WAVES * R pages with one atomic per extent
// class: each atomic takes 10 ns of the one counter's time (131 072 pages of 64 elements, one atomic a page
// 1780 us a call, 64 pages 330; 32 768 of 512 elements 522 and 159).  Small workgroups for few pages, where
// the launch's own latency counts.
// Call: CallWords if no stage kernel has written the records (a.gather, a.scatter: what of them is the caller's tensors).
// SUMS: else `partials` holds none.  (Asked at run time, a page's sums and flags come one after the other: norms of 100 000 pages of 64 elements 250 us a
// call, like this 244.)
template <int WAVES, int R, bool SUMS, class Call>
__global__ __launch_bounds__(WAVES * kWave) void apm_grad_finalize_kernel(FinalizeArgs a, Call call) {
    static_assert(WAVES * R <= kWave, "one wavefront notes a workgroup's pages");
    constexpr bool kCall = std::is_same<Call, CallWords>::value;
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int64_t first = (int64_t)blockIdx.x * (WAVES * R);
    __shared__ int32_t s_cls[WAVES * R];  // extent class of a page to note, or -1
#pragma unroll 1
    for (int r = 0; r < R; ++r) {
        const int slot = r * WAVES + wave;
        const int64_t i = first + slot;
        int c = -1;
        if (i < a.n_listed) {
            PagePlace place{};
            int64_t page, o = i;
            int used;
            if constexpr (kCall) {
                uint32_t k = (uint32_t)i;
                if (call.t.listed) {
                    k = call_word(&call, 2 * (uint32_t)i);
                    o = (int64_t)call_word(&call, 2 * (uint32_t)i + 1);
                }
                place = __builtin_bit_cast(PagePlace, load_16(call.t.places + k));
                page = place.page;
                if (!call.t.listed) o = page;
                used = place.used;
            } else {
                page = a.grad_pages ? a.grad_pages[i] : a.grad_first + i;
                used = a.used[page];
            }
            const int n_slices = max(1, (used + kReduceTile - 1) / kReduceTile);
            double s = 0.0;
            uint32_t nz = 0;
            for (int k = lane; k < n_slices; k += kWave) {
                const int64_t at = (a.by_page ? page : i) * a.S + k;
                if (SUMS) s += a.partials[at];
                nz |= a.nzflags[at];
            }
            s = wave_sum_f64(s);
            nz = wave_or_u32(nz);
            const bool skip = a.skip_mode == APM_SKIP_UNTOUCHED && nz == 0u;
            if (lane == 0) {
                const double norm = sqrt(s);
                const float scale = clip_scale(norm, a.max_norm);
                const float sc = skip ? -1.0f : scale;
                if constexpr (kCall) {
                    PageRec rec;
                    if (a.gather && a.scatter) rec = call_rec<true, true>(call.t, place, &call);
                    else if (a.gather) rec = call_rec<true, false>(call.t, place, &call);
                    else if (a.scatter) rec = call_rec<false, true>(call.t, place, &call);
                    else rec = call_rec<false, false>(call.t, place, &call);
                    rec.scale = sc;
                    a.recs[i] = rec;
                } else if (a.run) reinterpret_cast<PageRun*>(a.recs)[i] = PageRun{used, sc};
                else if (a.staged) a.recs[i].scale = sc;
                else a.recs[i] = class_rec(used, sc, page, a.state_pages ? a.state_pages[i] : a.state_first + i, a.E, a.g16, a.p16);
                if (!kCall && a.out_index) o = (int64_t)a.out_index[i];
                if (a.grad_norm) a.grad_norm[o] = skip ? 0.0f : (float)norm;
                if (a.skip_mask) a.skip_mask[o] = skip ? 1 : 0;
            }
            if (!skip) {
                c = 0;
                while (c + 1 < a.n_cls && i >= a.cls_begin[c + 1]) ++c;
            }
        }
        if (lane == 0) s_cls[slot] = c;
    }
    if (!a.live) return;
    __syncthreads();
    if (wave != 0) return;
    const int mine = lane < WAVES * R ? s_cls[lane] : -1;
    for (int c = 0; c < max(1, a.n_cls); ++c) {
        const uint64_t noted = __ballot(mine == c);
        if (noted == 0) continue;
        int at = lane == 0 ? atomicAdd(a.live + c, __popcll(noted)) : 0;
        at = __shfl(at, 0, kWave) + __popcll(noted & (((uint64_t)1 << lane) - 1));
        if (mine == c) a.live[kMaxExtentClasses + a.cls_begin[c] + at] = (int32_t)(first + lane);
    }
}

// Clears the counts where no reduce pass does it.
__global__ void apm_live_clear_kernel(int32_t* live) {
    if (threadIdx.x < kMaxExtentClasses) live[threadIdx.x] = 0;
}

__device__ __forceinline__ void clear_sums(uint64_t* sums, int64_t n) {
    for (int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x; j < n; j += (int64_t)gridDim.x * kThreads) sums[j] = kNoSum;
}

// No reduce pass: one thread per listed page fills its record with scale 1, or with the mark that the
// one-pass kernel waits on.
__global__ __launch_bounds__(kThreads) void apm_page_recs_kernel(FinalizeArgs a) {
    if (a.sums) clear_sums(a.sums, a.n_listed * a.S);
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= a.n_listed) return;
    const int64_t page = a.grad_pages ? a.grad_pages[i] : a.grad_first + i;
    const int used = a.used[page];
    const float scale = a.sums ? __uint_as_float(kNoScale) : 1.0f;
    if (a.run) reinterpret_cast<PageRun*>(a.recs)[i] = PageRun{used, scale};
    else a.recs[i] = class_rec(used, scale, page, a.state_pages ? a.state_pages[i] : a.state_first + i, a.E, a.g16, a.p16);
}

// Brings a call's page list and tensor addresses to where the kernels below read them, one thread per
// listed page.  The words travel in the kernel arguments (an upload from pinned memory would cost
// an extra kernel and two event packets, 20 us and more of idle GPU per call: 124 M parameters from
// and to tensors 582 us a call staged that way, 560 like this; 5 M in small pages
// with clipping 48 and 41); bound by launch latency and its chain of loads: addresses fetched beside the page's own
// loads, not after them, 4.8 M in small pages with clipping 32.6 -> 31.8 us a call.
struct StageArgs {
    const int32_t* used;
    const int64_t* pages;       // positions' pages, or nullptr: first + i
    int64_t first;
    int64_t n_listed;
    const TenantRec* tenants;
    PageRec* recs;
    const uint16_t* g16;        // the page classes, for what is not the caller's
    uint16_t* p16;
    int64_t E;
    int64_t* list;              // written from the list words
    int32_t* out;
    uint64_t* sums;             // one-pass launches: as in FinalizeArgs
    int64_t n_sums;
    const uint64_t* words;      // list, g, q words, unless they follow inline
    int64_t list_begin;         // the list words are those of positions [list_begin, + list_n)
    int32_t list_n;
    int32_t n_runs;             // StageArgsRuns: runs that the positions come in
    int32_t t_begin, t_n;       // the g / q words are those of tensors [t_begin, + t_n)
    int32_t has_g, has_q;
    uint64_t g_base, q_base;    // StageArgsNarrow
};
struct StageArgsInline {
    StageArgs a;
    uint64_t word[kArgWords];
};
// Half words: pages, then output indices, of the list; addresses as multiples of 16 from their list's base.  A launch less for
// 220 to 440 tensors, two for 150 listed pages of 274: 4 to 5 us each.
struct StageArgsNarrow {
    StageArgs a;
    uint32_t word[2 * kArgWords];
};

// The same with the list as runs (StageRun) in the first words.
struct StageArgsRuns {
    StageArgs a;
    uint32_t word[2 * kArgWords];
};

template <class Args>
__global__ __launch_bounds__(kThreads) void apm_stage_kernel(Args args) {
    const StageArgs* ap;
    if constexpr (sizeof(Args) > sizeof(StageArgs)) ap = &args.a;
    else ap = &args;
    const StageArgs& a = *ap;
    constexpr bool kRuns = std::is_same<Args, StageArgsRuns>::value, kNarrow = kRuns || std::is_same<Args, StageArgsNarrow>::value;
    constexpr int kRunWords = sizeof(StageRun) / sizeof(uint32_t);
    constexpr bool kInline = sizeof(Args) > sizeof(StageArgs);
    auto word = [&](int64_t k) -> uint64_t {
        if constexpr (kInline) return args.word[k];
        else return a.words[k];
    };
    const int64_t list_words = kRuns ? (int64_t)kRunWords * a.n_runs : (kNarrow ? 2 : 1) * (int64_t)a.list_n;
    int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x, page = 0;
    const bool mine = i < (a.list_n > 0 ? a.list_n : a.n_listed), tenants = (a.has_g || a.has_q) && a.t_n > 0;
    // Argument words read lane by lane come from as far as anything else: all addresses are fetched beside the page's
    // own loads, not after them.
    using Word = typename std::conditional<kNarrow, uint32_t, uint64_t>::type;
    __shared__ Word s_address[kInline ? (kNarrow ? 2 : 1) * kArgWords : 1];
    if (kInline && tenants && (int64_t)blockIdx.x * kThreads < a.n_listed)
        for (int k = (int)threadIdx.x; k < (a.has_g + a.has_q) * a.t_n; k += kThreads) s_address[k] = (Word)word(list_words + k);
    if constexpr (kRuns) {
        __shared__ StageRun s_run[2 * kArgWords / kRunWords];
        for (int k = (int)threadIdx.x; k < (int)list_words; k += kThreads) reinterpret_cast<uint32_t*>(s_run)[k] = args.word[k];
        __syncthreads();
        if (mine && a.list_n > 0) {
            i += a.list_begin;
            int low = 0, high = a.n_runs;  // the last run that begins at or before i
            while (high - low > 1) {
                const int mid = (low + high) / 2;
                if ((int64_t)s_run[mid].at <= i) low = mid;
                else high = mid;
            }
            const StageRun r = s_run[low];
            const int64_t k = i - (int64_t)r.at;
            page = (int64_t)(r.page & 0x7FFFFFFFu) + (r.page >> 31 ? -k : k);
            a.list[i] = page;
            a.out[i] = (int32_t)(r.out + (uint32_t)k);
        }
    }
    if (mine && !(kRuns && a.list_n > 0)) {
        if (a.list_n > 0) {
            const uint64_t w = word(i), out = kNarrow ? word(a.list_n + i) : w >> 32;
            i += a.list_begin;
            page = (int64_t)(uint32_t)w;
            a.list[i] = page;
            a.out[i] = (int32_t)out;
        } else {
            page = a.pages ? a.pages[i] : a.first + i;
        }
    }
    int used = 0;
    TenantRec t{};
    if (mine) {
        used = a.used[page];
        if (tenants) t = a.tenants[page];
    }
    if (kInline) __syncthreads();
    if (mine) {
        const PageRec own = class_rec(used, a.n_sums > 0 ? __uint_as_float(kNoScale) : 1.0f, page, page, a.E, a.g16, a.p16);
        PageRec* out = a.recs + i;
        if (!a.has_g && !a.has_q) {
            *out = own;
        } else if (tenants) {
            auto address = [&](int64_t k, uint64_t base) -> uint64_t {
                const uint64_t w = kInline ? s_address[k] : word(list_words + k);
                return kNarrow ? base + (w << 4) : w;
            };
            // Tenant by tenant: with several launches each fills in the tenants whose addresses it carries.
            out->used = used;
            out->scale = own.scale;
            out->pofs = own.pofs;
            out->off1 = t.off1;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int64_t at = t.tensor[k] - a.t_begin;
                if (t.tensor[k] < 0) {
                    out->end[k] = 0;
                } else if (at >= 0 && at < a.t_n) {
                    const int off = k == 0 ? 0 : t.off1;
                    out->end[k] = off + t.n[k];
                    out->g[k] = a.has_g ? reinterpret_cast<const uint16_t*>(address(at, a.g_base)) + t.tensor_off[k] - off : own.g[0];
                    out->q[k] = a.has_q ? reinterpret_cast<uint16_t*>(address((a.has_g ? a.t_n : 0) + at, a.q_base)) + t.tensor_off[k] - off : own.q[0];
                }
            }
        }
    }
    if (a.sums) clear_sums(a.sums, a.n_sums);  // behind the loads, which would wait for these stores
}

struct UpdateArgs {
    float b1, omb1, b2, omb2, inv_sqrt_bc2, eps, step_size, lr_wd;
};

__device__ __forceinline__ void adamw_elem(float& p, float& m, float& v, float g, const UpdateArgs& a,
                                           float scale) {
    const float gs = g * scale;
    m = fmaf(a.b1, m, a.omb1 * gs);
    v = fmaf(a.b2, v, a.omb2 * (gs * gs));
#if APM_FAST_RCP_SQRT
    const float denom = fmaf(__builtin_amdgcn_sqrtf(v), a.inv_sqrt_bc2, a.eps);
    const float upd = m * __builtin_amdgcn_rcpf(denom);
#else
    const float denom = fmaf(sqrtf(v), a.inv_sqrt_bc2, a.eps);
    const float upd = m / denom;
#endif
    // p' = p - (lr wd p + (lr/bc1) m'/denom): the two small terms are summed first, so the only
    // rounding at the magnitude of p is the final subtraction (half an ulp per step).
    const float delta = fmaf(a.step_size, upd, a.lr_wd * p);
    p = p - delta;
}

constexpr int kUpdThreads = kWave;
template <int U> constexpr int kTile = kUpdThreads * 4 * U;  // elements per wavefront

// The vectors of a slice that lies inside one tenant (all slices of a page but the last one or two) go
// through buffer accesses: the five streams' addresses are scalar (a descriptor each, made from the
// page record), the lanes share one 32-bit offset, and the cache policy is an operand: of the loads
// non-temporal, of the state's stores
//   kStoreHbm   non-temporal and written through, for state in device memory.  Non-temporal alone leaves the
//               lines in the L2 until they are evicted, in another order than the slices': 201 M parameters
//               876 us a call without, 868 with; with clipping 907 and 892 (written through alone: 867, but
//               with clipping 946);
//   kStoreNT    non-temporal, for state in host memory, and for state in device memory that is updated beside a
//               kernel that moves pages across the link (124 M parameters from pinned memory, staged: 34.5 ms a
//               step written through besides, 34.0 without; driven by a schedule: 42.2 and 41.9, 355 M 101.9 and 100.1);
//   kStoreHostWT  written through, for the same while other kernels run on the GPU: a non-temporal store
//               to host memory may rest in the L2 as a dirty line; the write-back that ends every kernel of any
//               other stream then has to push it across PCIe, so those kernels pay for this kernel's writes.
// Gradients are read with the default policy where state is stored with kStoreHbm: a slice of a tensor that does not
// start on a cache line shares its first and last line with its neighbours, and with clipping g is read a second time
// (213 M parameters in tensors of odd sizes: 957 us non-temporal, 943 default; with clipping 987 and 967).
// (As an operand because the compiler drops the hint of its non-temporal builtin from stores that it
// merges or moves between this body and the checked one below: 124 M parameters 599 us a call without
// the hint at one vector per lane, 548 with it.)
constexpr int kNT = 2, kSC1 = 16;
constexpr int kStoreHbm = kNT | kSC1, kStoreNT = kNT, kStoreHostWT = kSC1;
typedef __amdgpu_buffer_rsrc_t Rsrc;

// [base, base + bytes): accesses beyond it read zero / are dropped.
__device__ __forceinline__ Rsrc make_rsrc(const void* base, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00027000);
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    return f32_to_bf16_rne(lo) | (f32_to_bf16_rne(hi) << 16);
}

// The update of a lane's vector; returns the bf16 parameters.
__device__ __forceinline__ u32x2 update_vector(const UpdateArgs& a, float scale, u32x2 g, f32x4& p, f32x4& m, f32x4& v) {
    const float gf[4] = {bf16lo(g[0]), bf16hi(g[0]), bf16lo(g[1]), bf16hi(g[1])};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float pj = p[j], mj = m[j], vj = v[j];
        adamw_elem(pj, mj, vj, gf[j], a, scale);
        p[j] = pj;
        m[j] = mj;
        v[j] = vj;
    }
    return u32x2{pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3])};
}

// All loads are issued back to back, one wait, all stores back to back, in one basic block: on this
// target loads and stores share one counter, and at the entry of a basic block the compiler must
// assume the worst about what is outstanding.
// get_scale() is called when the loads are under way.  n: elements of the slice (a multiple of 8), the rest is neither read nor written.
template <int U, int STORE, class GetScale>
__device__ __forceinline__ void full_slice(const UpdateArgs& a, GetScale&& get_scale, int lane, float* p_, float* m_, float* v_,
                                           const uint16_t* g_, uint16_t* q_, int n = kTile<U>) {
    const Rsrc P = make_rsrc(p_, n * 4), M = make_rsrc(m_, n * 4), V = make_rsrc(v_, n * 4);
    const Rsrc G = make_rsrc(g_, n * 2), Q = make_rsrc(q_, n * 2);
    f32x4 p[U], m[U], v[U];
    u32x2 g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int o = lane * 16 + u * (kWave * 16);
        g[u] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(G, lane * 8 + u * (kWave * 8), 0, STORE == kStoreHbm ? 0 : kNT));
        p[u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(P, o, 0, kNT));
        m[u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(M, o, 0, kNT));
        v[u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(V, o, 0, kNT));
    }
    // without the barrier the scheduler sinks half of the loads between the vectors' arithmetic to
    // save registers
    __builtin_amdgcn_sched_barrier(0);
    const float scale = get_scale();
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int o = lane * 16 + u * (kWave * 16);
        const u32x2 q = update_vector(a, scale, g[u], p[u], m[u], v[u]);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, p[u]), P, o, 0, STORE);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, m[u]), M, o, 0, STORE);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v[u]), V, o, 0, STORE);
        __builtin_amdgcn_raw_buffer_store_b64(q, Q, lane * 8 + u * (kWave * 8), 0, kNT);
    }
}

// A slice that a tenant's end or the page's used extent cuts: one vector at a time, each checked against
// the used extent; with GATHER / SCATTER g is gathered / p16 scattered lane by lane through the tenants.
template <int U, bool GATHER, bool SCATTER>
__device__ __forceinline__ void cut_slice(const UpdateArgs& a, const PageRec& rec, int v0, float* p_, float* m_, float* v_) {
    f32x4* P = reinterpret_cast<f32x4*>(p_);
    f32x4* M = reinterpret_cast<f32x4*>(m_);
    f32x4* V = reinterpret_cast<f32x4*>(v_);
    // The class pointers come out of memory, so the compiler knows no address space for them and
    // would use flat accesses.  They are device (or pinned host) memory: say so.
    typedef const u32x2 __attribute__((address_space(1))) * GlobalIn;
    typedef u32x2 __attribute__((address_space(1))) * GlobalOut;
    const GlobalIn G = (GlobalIn) reinterpret_cast<const u32x2*>(rec.g[0]);
    const GlobalOut Q = (GlobalOut) reinterpret_cast<u32x2*>(rec.q[0]);
    const int nvec = ((rec.used + 7) & ~7) >> 2;
#pragma unroll 1
    for (int u = 0; u < U; ++u) {
        const int vi = v0 + u * kWave;
        if (vi >= nvec) break;
        const u32x2 g = GATHER ? gather_g4(rec, vi << 2) : __builtin_nontemporal_load(G + vi);
        f32x4 p = __builtin_nontemporal_load(P + vi), m = __builtin_nontemporal_load(M + vi), v = __builtin_nontemporal_load(V + vi);
        const u32x2 q = update_vector(a, rec.scale, g, p, m, v);
        __builtin_nontemporal_store(p, P + vi);  // whatever the slices' policy: such slices are few
        __builtin_nontemporal_store(m, M + vi);
        __builtin_nontemporal_store(v, V + vi);
        if (SCATTER) scatter_q4(rec, vi << 2, q);
        else __builtin_nontemporal_store(q, Q + vi);
    }
}

// Fused update of one slice (kTile<U> elements from `start`) of one page by one wavefront:
// 12 B + 2 B read and 12 B + 2 B written per element.  Each lane keeps U 128-bit vectors per
// fp32 class in flight; every wavefront-wide access is one contiguous 1 KiB (fp32) or 512 B (bf16)
// span.  p, m, v: the page's first element.
template <int U, bool GATHER, bool SCATTER, int STORE>
__device__ __forceinline__ void update_slice(const UpdateArgs& a, const PageRec& rec, int start, int lane,
                                             float* p, float* m, float* v) {
    const int k = start >= rec.off1 ? 1 : 0;
    if (start + kTile<U> <= rec.end[k])
        full_slice<U, STORE>(a, [&] { return rec.scale; }, lane, p + start, m + start, v + start, rec.g[k] + start, rec.q[k] + start);
    else cut_slice<U, GATHER, SCATTER>(a, rec, (start >> 2) + lane, p, m, v);
}

// The HBM-resident form: one grid over the slices of all listed pages (GridMap: classes of extents).  The arguments
// are single values, what the prologue needs first, because the hardware hands the leading 14 dwords
// of such an argument list to every wavefront in registers: the record's load is then the only round
// trip before the first vector load.
struct SmallClasses {
    GridClass small[kMaxExtentClasses - 1];
};
template <int U, bool GATHER, bool SCATTER, int STORE>
__global__ __launch_bounds__(kUpdThreads) void apm_adamw_kernel(const PageRec* recs, float* p32, float* m32, float* v32, uint32_t large_at,
                                                                uint32_t per, uint32_t mul, uint32_t shift, UpdateArgs a, SmallClasses classes) {
    int item;
    uint32_t x;
    grid_item(large_at, GridDiv{per, mul, shift}, classes.small, blockIdx.x, &item, &x);
    const PageRec rec = load_rec(recs + item);
    const int start = (int)x * kTile<U>;
    if (rec.scale < 0.0f || start >= ((rec.used + 7) & ~7)) return;  // a skipped page, beyond the extent
    update_slice<U, GATHER, SCATTER, STORE>(a, rec, start, (int)threadIdx.x, p32 + rec.pofs, m32 + rec.pofs, v32 + rec.pofs);
}

// The same with records made from the call's words.  first: list position of the map's first item.
template <int U, bool GATHER, bool SCATTER>
__global__ __launch_bounds__(kUpdThreads) void apm_adamw_call_kernel(const PagePlace* places, float* p32, float* m32, float* v32, uint32_t large_at,
                                                                     uint32_t per, uint32_t mul, uint32_t shift, uint32_t first, int listed, UpdateArgs a,
                                                                     SmallClasses classes, CallWords c) {
    int item;
    uint32_t x;
    grid_item(large_at, GridDiv{per, mul, shift}, classes.small, blockIdx.x, &item, &x);
    uint32_t place = first + (uint32_t)item;
    if (listed) place = call_word(&c, 2 * place);
    // Side by side: issued as soon as its address is known, the second would be waited for before the first starts.
    uint32_t none = 0;
    asm("" : "+s"(none) : "s"(place));
    i32x16 at = load_16(places + place), t = load_16(reinterpret_cast<const char*>(&c.t) + none);
    asm("" : "+s"(t), "+s"(at));
    const PageRec rec = call_rec<GATHER, SCATTER>(__builtin_bit_cast(CallTables, t), __builtin_bit_cast(PagePlace, at), &c);
    const int start = (int)x * kTile<U>;
    if (start >= ((rec.used + 7) & ~7)) return;
    update_slice<U, GATHER, SCATTER, kStoreHbm>(a, rec, start, (int)threadIdx.x, p32 + rec.pofs, m32 + rec.pofs, v32 + rec.pofs);
}

// The same for a run of pages in the page classes; all pointers are those of the launch's first page.
// BARE: nothing has written records, `runs` is the page table (int32_t) and the scale is 1: a launch less,
// eight quarter pages 13.2 -> 10.8 us a call.
template <int U, bool BARE, int STORE>
__global__ __launch_bounds__(kUpdThreads) void apm_adamw_run_kernel(const void* runs, float* p32, float* m32, float* v32,
                                                                    const uint16_t* g16, uint16_t* p16, int E, UpdateArgs a) {
    PageRun run{0, 1.0f};
    if (BARE) run.used = static_cast<const int32_t*>(runs)[blockIdx.y];
    else run = load_run(static_cast<const PageRun*>(runs) + blockIdx.y);
    const int64_t at = (int64_t)blockIdx.y * E;
    const PageRec rec = class_rec(run.used, run.scale, 0, 0, 0, g16 + at, p16 + at);
    const int start = (int)blockIdx.x * kTile<U>;
    if ((!BARE && rec.scale < 0.0f) || start >= rec.end[0]) return;
    update_slice<U, false, false, STORE>(a, rec, start, (int)threadIdx.x, p32 + at, m32 + at, v32 + at);
}

// Over the pages that the finalize pass noted, a class's `slices.per` slices each.  live: see kLiveInts;
// recs (as PageRun if RUN) and, if RUN, the other pointers are those of list position 0.
// Entry 0 is the class of the largest pages, which comes last in the grid and is there with the first load; the others follow,
// the smallest pages first; unused ones (the last) start where entry 0 does.
struct LiveClasses {
    struct Class {
        uint32_t first;         // of its workgroups
        int32_t begin, number;  // its first position, its count's place
        GridDiv slices;
        uint32_t di, dx;        // it has di * slices.per + dx workgroups
    } cls[kMaxExtentClasses];
};
__device__ __forceinline__ LiveClasses::Class load_class(const LiveClasses::Class* at) {
    typedef int i32x8 __attribute__((ext_vector_type(8)));
    static_assert(sizeof(LiveClasses::Class) == sizeof(i32x8), "a class is one scalar load");
    typedef const i32x8 __attribute__((address_space(4), aligned(4))) * Const;
    i32x8 w = *(Const)reinterpret_cast<const i32x8*>(at);
    asm("" : "+s"(w));
    return __builtin_bit_cast(LiveClasses::Class, w);
}
template <int U, bool RUN, bool GATHER, bool SCATTER, int STORE>
__global__ __launch_bounds__(kUpdThreads) void apm_adamw_live_kernel(const int32_t* live, const PageRec* recs, float* p32, float* m32, float* v32,
                                                                     const uint16_t* g16, uint16_t* p16, int64_t E, UpdateArgs a, LiveClasses lc) {
    typedef const int32_t __attribute__((address_space(4))) * Const;
    uint32_t w = blockIdx.x;
    LiveClasses::Class c = load_class(lc.cls);
    if (w < c.first) c = load_class(lc.cls + 1 + (w >= lc.cls[2].first) + (w >= lc.cls[3].first));
    const uint32_t n = ((Const)live)[c.number], nx = c.slices.per;
    const Const positions = (Const)live + kMaxExtentClasses + c.begin;
    w -= c.first;
    // a wavefront's items are the class's workgroups apart; page and slice advance by that without another division
    uint32_t i = c.slices.quotient(w), x = w - i * nx;
    auto walk = [&](auto store) {
#pragma unroll 1
        for (; i < n; i += c.di, x += c.dx) {
            if (x >= nx) {
                x -= nx;
                if (++i >= n) return;
            }
            const int64_t pos = positions[i];
            PageRec rec;
            int64_t at;
            if (RUN) {
                at = pos * E;
                const PageRun run = load_run(reinterpret_cast<const PageRun*>(recs) + pos);
                rec = class_rec(run.used, run.scale, 0, 0, 0, g16 + at, p16 + at);
            } else {
                rec = load_rec(recs + pos);
                at = rec.pofs;
            }
            const int start = (int)x * kTile<U>;
            if (start < ((rec.used + 7) & ~7))
                update_slice<U, GATHER, SCATTER, decltype(store)::value>(a, rec, start, (int)threadIdx.x, p32 + at, m32 + at, v32 + at);
        }
    };
    // A wavefront waits for one slice's stores before the next slice's loads, and written through they take longer: with many
    // slices a wavefront, of many wavefronts, that costs more than it gains.  us a call, written through / not, one GPU, elements
    // (slices per wavefront): all live, 7 M (3.5) 46.7 / 47.7, 13 M (6.3) 79.2 / 79.9, 19 M (9.2) 116 / 116,
    // 26 M (12) 151 / 148, 124 M (12) 707 / 691, 1.3 G (12) 7486 / 7353; 541 M, a quarter live (3) 804 / 806, 3 in 8 (4.5) 1164 / 1152, half
    // (6) 1534 / 1514; 1.08 G, an eighth (1.5) 951 / 954.
    const uint64_t wavefronts = c.di * nx + c.dx;
    if (STORE == kStoreNT || (uint64_t)n * nx > 4 * (wavefronts + kThroughSlack)) walk(std::integral_constant<int, kStoreNT>{});
    else walk(std::integral_constant<int, STORE>{});
}

// The form for fp32 classes that live in pinned host memory, read and written across PCIe by the kernel itself: a
// fixed number of wavefronts shares all slices of `count` list positions.  The link needs only some hundred KiB in
// flight, so a few dozen wavefronts saturate it.  The launch chooses how many of them share a workgroup (and with it a
// CU): one per workgroup gives the highest transfer rate; packed 8 or 16 to a workgroup they occupy few CUs, which
// matters beside kernels whose workgroups need a CU's whole register file or LDS (dense matrix products), because a
// wavefront that lives as long as the whole transfer keeps those off its CU.
//
// The slices that hold used elements of pages not skipped are numbered in list order and dealt out in turn.  A wavefront
// finds its own by a scan over the extents of 64 positions at a time, one lane each, fetched while it works on the 64
// before: it never stands on a slice without elements (dealt out by position and slice of the largest page instead, 19 M
// parameters of 230 pages, 154 of them nearly empty, 5.42 ms a step = 42.9 GB/s each way, like this 4.78 = 48.7; 31 M
// 7.69 and 7.49; 124 M 30.5 and 30.3).
//
// STAGED: a wavefront brings its next slice into its staging slot in device memory while it updates the one before
// from the other slot and writes it to the host, so both directions of the link are busy from the second slice to the
// last but one and nothing but the wavefront itself orders the two.  (A batch of pages at a time instead, one copy
// kernel for both directions beside the update's, each direction idle for two batches of the step: 124 M parameters
// 34.1 ms a step, like this 30.7; 11 M 4.22 and 2.80; 5 M 1.83 and 1.34.)
constexpr int kStrideMaxThreads = 1024;
constexpr int kStrideU = 4;
static_assert(kTile<kStrideU> * 4 == kLinkSlotBytes, "a staging slot holds a slice");

struct StrideArgs {
    const PageRec* recs;  // as PageRun if RUN
    float* p32;           // RUN: of the launch's first page, as g16 and p16; otherwise of the class
    float* m32;
    float* v32;
    const uint16_t* g16;
    uint16_t* p16;
    int64_t E;
    int64_t count;
    int n_workers;
    float* slots[3];      // STAGED: two slices a wavefront
};

struct LinkSlice {
    int64_t page;  // list position
    int start, n;  // elements; n == 0: none
    int used;
    float scale;
};
template <bool RUN, int U>
struct LinkWalk {
    const PageRec* recs;
    int64_t count, base;
    int stride, total, t;      // t: of the worker's next slice, among the `total` of positions [base, base + 64)
    int used, upto;            // lane by lane: extent (0: skipped), slices of [base, base + lane]
    float scale;
    PageRun ahead;             // of position base + 64 + lane

    __device__ __forceinline__ PageRun fetch(int64_t at) const {
        PageRun r{0, 1.0f};
        at += (int)threadIdx.x & (kWave - 1);
        if (at < count) r = RUN ? reinterpret_cast<const PageRun*>(recs)[at] : *reinterpret_cast<const PageRun*>(recs + at);
        return r;
    }
    static __device__ __forceinline__ int slices(int used) { return (int)(((uint32_t)used + (kTile<U> - 1)) / kTile<U>); }
    __device__ __forceinline__ void enter(const PageRun& r) {
        used = r.scale < 0.0f ? 0 : (r.used + 7) & ~7;
        scale = r.scale;
        upto = slices(used);
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int x = __shfl_up(upto, off, kWave);
            if (((int)threadIdx.x & (kWave - 1)) >= off) upto += x;
        }
        total = __builtin_amdgcn_readlane(upto, kWave - 1);
        ahead = fetch(base + kWave);
    }
    __device__ __forceinline__ LinkWalk(const PageRec* r, int64_t n, int worker, int workers) : recs(r), count(n), base(0), stride(workers), t(worker) {
        enter(fetch(0));
    }
    __device__ __forceinline__ LinkSlice next() {
#pragma unroll 1
        while (t >= total) {
            if (base + kWave >= count) return LinkSlice{0, 0, 0, 0, 1.0f};
            t -= total;
            base += kWave;
            enter(ahead);
        }
        const int l = __popcll(__ballot(upto <= t));  // < 64, as t < total
        LinkSlice s;
        s.page = base + l;
        s.used = __builtin_amdgcn_readlane(used, l);
        s.scale = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(scale), l));
        s.start = (t - (__builtin_amdgcn_readlane(upto, l) - slices(s.used))) * kTile<U>;
        s.n = min(kTile<U>, s.used - s.start);
        t += stride;
        return s;
    }
};

// Where a slice lies.
struct LinkPlace {
    float *p, *m, *v;
    const uint16_t* g;
    uint16_t* q;
};
template <bool RUN>
__device__ __forceinline__ LinkPlace link_place(const StrideArgs& s, const LinkSlice& x) {
    if (RUN) {
        const int64_t at = x.page * s.E + x.start;
        return LinkPlace{s.p32 + at, s.m32 + at, s.v32 + at, s.g16 + at, s.p16 + at};
    }
    PageRec rec{};
    if (x.n > 0) rec = load_rec(s.recs + x.page);
    const int64_t at = rec.pofs + x.start;
    return LinkPlace{s.p32 + at, s.m32 + at, s.v32 + at, rec.g[0] + x.start, rec.q[0] + x.start};
}

template <bool RUN, bool WT>
__global__ __launch_bounds__(kStrideMaxThreads) void apm_adamw_stride_kernel(StrideArgs s, UpdateArgs a) {
    const int lane = (int)threadIdx.x & (kWave - 1);
    const int worker = (int)blockIdx.x * ((int)blockDim.x / kWave) + __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    if (worker >= s.n_workers) return;
    // Pages of one slice at most are dealt out one by one, vector by vector: of a slice that is mostly beyond its page the accesses that the
    // descriptors drop cost time too (8.4 M parameters in pages of 64 elements 8.9 ms a step with the walk, 5.7 like this; 16.8 M in pages of
    // 512 4.67 and 4.20; but few elements in each larger page, whose slices without any have to be found: 20 000 of 300 in pages of 8192
    // 1.67 ms with the walk, 1.89 by position and slice).
    if (s.E <= kTile<kStrideU>) {
#pragma unroll 1
        for (int64_t i = worker; i < s.count; i += s.n_workers) {
            PageRec rec;
            int64_t at;
            if (RUN) {
                const PageRun run = load_run(reinterpret_cast<const PageRun*>(s.recs) + i);
                at = i * s.E;
                rec = class_rec(run.used, run.scale, 0, 0, 0, s.g16 + at, s.p16 + at);
            } else {
                rec = load_rec(s.recs + i);
                at = rec.pofs;
            }
            if (rec.scale < 0.0f || rec.end[0] == 0) continue;
            update_slice<kStrideU, false, false, WT ? kStoreHostWT : kStoreNT>(a, rec, 0, lane, s.p32 + at, s.m32 + at, s.v32 + at);
        }
        return;
    }
    LinkWalk<RUN, kStrideU> walk(s.recs, s.count, worker, s.n_workers);
#pragma unroll 1
    for (;;) {
        const LinkSlice x = walk.next();
        if (x.n == 0) return;
        const LinkPlace at = link_place<RUN>(s, x);
        full_slice<kStrideU, WT ? kStoreHostWT : kStoreNT>(a, [&] { return x.scale; }, lane, at.p, at.m, at.v, at.g, at.q, x.n);
    }
}

// Loads and stores of both directions are one basic block, host reads first: a wait for the slice that came in before
// then waits for nothing that is issued after it.  Accesses beyond a slice's elements, or of a direction that has no slice,
// are dropped by the descriptors.
// For a run of pages.
// UPDATE: else the slices come and go as they are.
// THREADS: a workgroup's most.  More than 8 wavefronts leave each other 128 registers: there the slice that comes is read when the one
// that goes is on its way (356 M parameters, 128 wavefronts, 16 a workgroup, GB/s each way: 46.3; read first, with registers spilled, 39; slices
// of half the size 42).
template <bool WT, bool UPDATE, int THREADS>
__global__ __launch_bounds__(THREADS) void apm_adamw_staged_kernel(StrideArgs s, UpdateArgs a) {
    constexpr int U = kStrideU, STORE = WT ? kStoreHostWT : kStoreNT;
    constexpr bool kTight = THREADS > kStrideMaxThreads / 2;
    const int lane = (int)threadIdx.x & (kWave - 1);
    const int worker = (int)blockIdx.x * ((int)blockDim.x / kWave) + __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    if (worker >= s.n_workers) return;
    LinkWalk<true, U> walk(s.recs, s.count, worker, s.n_workers);
    LinkSlice out{0, 0, 0, 0, 1.0f};
    LinkPlace out_at{};
    int slot = 2 * worker;
    const int o = lane * 16;
#pragma unroll 1
    for (;;) {
        const LinkSlice in = walk.next();
        if (in.n == 0 && out.n == 0) return;
        const LinkPlace in_at = link_place<true>(s, in);
        const int n_in = in.n * 4, n_out = out.n;
        float* const src[3] = {in_at.p, in_at.m, in_at.v};
        float* const dst[3] = {out_at.p, out_at.m, out_at.v};
        u32x4 come[3][U], go[3][U];
        u32x2 g[U];
        auto load_in = [&] {
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int u = 0; u < U; ++u)
                    come[k][u] = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc(src[k], n_in), o + u * (kWave * 16), 0, kNT);
        };
        if (!kTight) load_in();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                go[k][u] = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc(s.slots[k] + (int64_t)(slot ^ 1) * kTile<U>, n_out * 4), o + u * (kWave * 16), 0, 0);
            if (UPDATE) g[u] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(make_rsrc(out_at.g, n_out * 2), lane * 8 + u * (kWave * 8), 0, kNT));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (UPDATE) {
                f32x4 p = __builtin_bit_cast(f32x4, go[0][u]), m = __builtin_bit_cast(f32x4, go[1][u]), v = __builtin_bit_cast(f32x4, go[2][u]);
                const u32x2 q = update_vector(a, out.scale, g[u], p, m, v);
                go[0][u] = __builtin_bit_cast(u32x4, p);
                go[1][u] = __builtin_bit_cast(u32x4, m);
                go[2][u] = __builtin_bit_cast(u32x4, v);
                __builtin_amdgcn_raw_buffer_store_b64(q, make_rsrc(out_at.q, n_out * 2), lane * 8 + u * (kWave * 8), 0, kNT);
            }
#pragma unroll
            for (int k = 0; k < 3; ++k)
                __builtin_amdgcn_raw_buffer_store_b128(go[k][u], make_rsrc(dst[k], n_out * 4), o + u * (kWave * 16), 0, STORE);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (kTight) load_in();
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int u = 0; u < U; ++u)
                __builtin_amdgcn_raw_buffer_store_b128(come[k][u], make_rsrc(s.slots[k] + (int64_t)slot * kTile<U>, n_in), o + u * (kWave * 16), 0, 0);
        out = in;
        out_at = in_at;
        slot ^= 1;
    }
}

// ---- norms, clip scales and update in one kernel -----------------------------------------------
//
// A page is updated with a scale that depends on its whole gradient, so the gradient is read twice.
// As a reduce pass in front of the update pass that is another 2 B per element from HBM (30 instead
// of 28).  Here both are in one grid, one wavefront per item, in this order:
//
//     sums of pages 0 .. D-1 | for every page j: sums of page j+D, update slices of page j
//
// for every class of extents, the smallest pages first (the largest class's sums run beside the small ones'
// waiting), where the sums of a page are its kReduceTile-element tiles and one wavefront that adds them up and
// publishes the page's scale.  The second reading of a page's gradient follows the first by D pages;
// the first reading uses ordinary loads and all else is non-temporal, so the gradient is still in the
// memory-side cache (256 MiB) then: D pages are kLookAhead elements, 32 MiB of gradient (4, 8, 16, 32, 64, 100 M
// elements ahead, 1.3 B parameters: 6567, 6005, 5862, 5970, 6000, 6100 us a call).  Against a reduce
// pass, a pass over its results and the update: 1.3 B parameters 5963 -> 5780 us, 127 M 596 -> 568,
// 4.8 M in small pages 38.4 -> 34.0; for smaller pages see one_pass_pays.
//
// Wavefronts hand results on through single words in device memory (a tile's sum, a page's scale)
// which the stage / prepare pass has marked as not there yet; value and mark are one word, so
// nothing else needs ordering.  Workgroups start in grid order, so whoever waits waits for wavefronts
// that are already running, and by its turn an update slice almost always finds its scale in place.
// Nothing relies on that order, though: after wait_limit polls (more for a page of many tiles) a wavefront
// computes what it waits for by itself, with the same result, or until a look between two tiles finds it there.
constexpr int64_t kLookAhead = (int64_t)16 << 20;
constexpr int kClipLds = 13312;  // 12 wavefronts per CU: 5832 us; 16, 13, 11, 10: 6000, 5840, 5873, 6164

typedef uint64_t __attribute__((address_space(1))) * GlobalU64;
typedef uint32_t __attribute__((address_space(1))) * GlobalU32;
__device__ __forceinline__ uint64_t poll64(GlobalU64 p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ uint32_t poll32(GlobalU32 p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Sum of squares of one tile by one wavefront, with the additions in the order of apm_grad_reduce_kernel
// (its four wavefronts' accumulators side by side).  Every lane returns it.
template <bool GATHER>
__device__ __forceinline__ double tile_sum(const PageRec& rec, int tile, int lane) {
    constexpr int kWaves = kThreads / kWave, U = APM_REDUCE_U, kSpan = kThreads * 8 * U;
    const int start = tile * kReduceTile, end = min(start + kReduceTile, rec.used);
    const int k = start >= rec.off1 ? 1 : 0;
    const bool inside = !GATHER || start + (((end - start) + 7) & ~7) <= rec.end[k];
    double acc0[kWaves], acc1[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) acc0[w] = acc1[w] = 0.0;
    // elements from `end` on read as zero: the descriptor ends with the last vector that holds one
    const Rsrc G = make_rsrc(rec.g[k] + start, inside && end > start ? (((end - start) + 7) & ~7) * 2 : 0);
#pragma unroll 1
    for (int at = start; at < end; at += kSpan) {
        u32x4 x[U * kWaves];
        if (inside) {
#pragma unroll
            for (int u = 0; u < U * kWaves; ++u)
                x[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(G, (at - start + (u * kWave + lane) * 8) * 2, 0, 0));
        } else {
            // a tenant ends in this tile: whole vectors, all under way at once ...
            typedef const u32x4 __attribute__((address_space(1))) * GlobalIn;
#pragma unroll
            for (int u = 0; u < U * kWaves; ++u) {
                const int e = at + (u * kWave + lane) * 8, kk = e >= rec.off1 ? 1 : 0;
                x[u] = u32x4{0u, 0u, 0u, 0u};
                if (e < end && e + 8 <= rec.end[kk]) x[u] = *(GlobalIn) reinterpret_cast<const u32x4*>(rec.g[kk] + e);
            }
            // ... and the one with a tenant's last few elements, never read past them
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const int last = rec.end[kk] & ~7;
                if (last == rec.end[kk] || last < at || last >= min(at + kSpan, end)) continue;
                const int at_u = (last - at) / (8 * kWave), at_lane = (last - at) / 8 % kWave;
                const u32x4 y = lane == at_lane ? gather_g8(rec, last) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
                for (int u = 0; u < U * kWaves; ++u)
                    if (u == at_u && lane == at_lane) x[u] = y;
            }
        }
        if (at + kSpan > end) {
#pragma unroll
            for (int u = 0; u < U * kWaves; ++u) {
                const int left = end - (at + (u * kWave + lane) * 8);  // boundary vector: drop elements at or beyond the extent
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    x[u][j] = left <= 2 * j ? 0u : left == 2 * j + 1 ? x[u][j] & 0x0000FFFFu : x[u][j];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int w = 0; w < kWaves; ++w)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double lo = (double)bf16lo(x[u * kWaves + w][j]), hi = (double)bf16hi(x[u * kWaves + w][j]);
                    acc0[w] = fma(lo, lo, acc0[w]);
                    acc1[w] = fma(hi, hi, acc1[w]);
                }
    }
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const double s = wave_sum_f64(acc0[w] + acc1[w]);
        t = w == 0 ? s : t + s;
    }
    return t;
}

// What wavefront w of the reduce kernel's workgroup adds up of a tile, all loads under way at once.  In a small call every update slice is
// on the chip before the first page's scale is there, so how long that takes is lost (us a call with a tile / a quarter of it a
// wavefront: 0.6 M elements 10.9 / 9.4, 4.8 M 29.2 / 27.6, 18 M 88.9 / 84.9).
constexpr int kTileParts = kThreads / kWave;
template <bool GATHER>
__device__ __forceinline__ double part_sum(const PageRec& rec, int tile, int w, int lane) {
    constexpr int kVectors = kReduceTile / (kThreads * 8);  // of this lane; the next one is a workgroup's span further
    const int start = tile * kReduceTile, end = min(start + kReduceTile, rec.used);
    const int k = start >= rec.off1 ? 1 : 0;
    const bool inside = !GATHER || start + (((end - start) + 7) & ~7) <= rec.end[k];
    const int first = (w * kWave + lane) * 8;  // element of the tile
    u32x4 x[kVectors];
    if (inside) {
        const Rsrc G = make_rsrc(rec.g[k] + start, end > start ? (((end - start) + 7) & ~7) * 2 : 0);
#pragma unroll
        for (int u = 0; u < kVectors; ++u)
            x[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(G, (first + u * (kThreads * 8)) * 2, 0, 0));
    } else {  // a tenant ends in this tile: its whole vectors (beyond them a descriptor reads zero), and the one with its last few elements
#pragma unroll
        for (int u = 0; u < kVectors; ++u) x[u] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int low = kk == 0 ? start : max(start, rec.off1), high = min(end, rec.end[kk]);
            if (high <= low) continue;
            const Rsrc G = make_rsrc(rec.g[kk] + low, ((high - low) & ~7) * 2);
#pragma unroll
            for (int u = 0; u < kVectors; ++u)
                x[u] |= __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(G, (start - low + first + u * (kThreads * 8)) * 2, 0, 0));
            const int last = rec.end[kk] & ~7, at = (last - start) / 8;
            if (last == rec.end[kk] || last < start || last >= end) continue;
            const u32x4 y = at % kThreads == w * kWave + lane ? gather_g8(rec, last) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int u = 0; u < kVectors; ++u) x[u] |= u == at / kThreads ? y : u32x4{0u, 0u, 0u, 0u};
        }
    }
    double acc0 = 0.0, acc1 = 0.0;
#pragma unroll
    for (int u = 0; u < kVectors; ++u) {
        const int left = end - (start + first + u * (kThreads * 8));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t v = left >= 2 * j + 2 ? x[u][j] : left == 2 * j + 1 ? x[u][j] & 0x0000FFFFu : 0u;
            const double lo = (double)bf16lo(v), hi = (double)bf16hi(v);
            acc0 = fma(lo, lo, acc0);
            acc1 = fma(hi, hi, acc1);
        }
    }
    return wave_sum_f64(acc0 + acc1);
}

// A page's sum by one wavefront on its own, in the order of apm_grad_finalize_kernel.  needless() is asked
// before every tile: if it says yes, the page's scale has come after all.
template <bool GATHER, class Needless>
__device__ __forceinline__ double page_sum(const PageRec& rec, int n_tiles, int lane, Needless&& needless) {
    double s = 0.0;
#pragma unroll 1
    for (int t = 0; t < n_tiles; ++t) {
        if (needless()) return 0.0;
        const double x = tile_sum<GATHER>(rec, t, lane);
        if ((t & (kWave - 1)) == lane) s += x;
    }
    return wave_sum_f64(s);
}

struct ClipArgs {
    PageRec* recs;         // of the launch's first page; as PageRun if RUN
    float* p32;            // RUN: of the launch's first page, as g16 and p16; otherwise of the class
    float* m32;
    float* v32;
    const uint16_t* g16;
    uint16_t* p16;
    int64_t E;
    uint64_t* sums;        // [count * S] of the launch
    float* grad_norm;      // nullable
    uint8_t* skip_mask;    // nullable: nothing is skipped here
    const int32_t* out_index;  // of the launch's first page, or nullptr: out_first + position
    int64_t out_first;
    double max_norm;
    int32_t S;
    // The launch's classes of extents, each with the workgroups from `first` on.  Entry 0 is the class of the largest pages, which
    // comes last in the grid and is there with the first load; the others follow, the smallest pages first; unused ones (the last)
    // start where entry 0 does.
    struct Class {
        uint32_t first;
        uint32_t n_ahead, n_mixed;  // workgroups of the class's first part, and of its first two
        int32_t begin;              // the class's first page, from the launch's first
        int32_t ahead;              // D
        int32_t wait_limit;
        uint32_t after;             // count - D
        GridDiv sum, both, slices;  // per page: the tiles of the largest and 1, that and the slices, the slices
    } cls[kMaxExtentClasses];
};

// One scalar load, as load_rec.
__device__ __forceinline__ ClipArgs::Class load_class(const ClipArgs::Class* at) {
    static_assert(sizeof(ClipArgs::Class) == sizeof(i32x16), "a class is one scalar load");
    typedef const i32x16 __attribute__((address_space(4), aligned(4))) * Const;
    i32x16 w = *(Const)reinterpret_cast<const i32x16*>(at);
    asm("" : "+s"(w));
    return __builtin_bit_cast(ClipArgs::Class, w);
}

// How wavefronts hand results on: through words that an earlier kernel has marked ...
struct CallMarked {};
struct HandedMarked {
    GlobalU64 sum;    // of the page's tiles
    GlobalU32 scale;
    __device__ __forceinline__ void put_sum(int t, double x) const { __hip_atomic_store(sum + t, (uint64_t)__double_as_longlong(x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ bool sum_there(int t, double* x) const {
        const uint64_t v = poll64(sum + t);
        *x = __longlong_as_double((long long)v);
        return v != kNoSum;
    }
    __device__ __forceinline__ void put_scale(float x) const { __hip_atomic_store(scale, __float_as_uint(x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ bool scale_there(uint32_t* v) const { return (*v = (uint32_t)__builtin_amdgcn_readfirstlane((int)poll32(scale))) != kNoScale; }
};
// ... or that carry the call's number beside the value.  Pages share no cache line (with lines shared: 4.9 M elements 31.9 / 30.8 us a
// call with words marked / tagged, 25 M 122 / 128; with lines of their own 29.6 and 121).
struct HandedTagged {
    GlobalU64 sum, scale;
    uint32_t number;
    __device__ __forceinline__ void put(GlobalU64 at, uint32_t x) const { __hip_atomic_store(at, (uint64_t)x << 32 | number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ void put_sum(int part, double x) const {  // of part % kTileParts of tile part / kTileParts
        const uint64_t u = (uint64_t)__double_as_longlong(x);
        put(sum + 2 * part, (uint32_t)(u >> 32));
        put(sum + 2 * part + 1, (uint32_t)u);
    }
    __device__ __forceinline__ bool sum_there(int t, double* x) const {
        uint64_t v[2 * kTileParts];
#pragma unroll
        for (int k = 0; k < 2 * kTileParts; ++k) v[k] = poll64(sum + t * (2 * kTileParts) + k);
        bool there = true;
#pragma unroll
        for (int k = 0; k < 2 * kTileParts; ++k) there = there && (uint32_t)v[k] == number;
#pragma unroll
        for (int w = 0; w < kTileParts; ++w) {
            const double s = __longlong_as_double((long long)((v[2 * w] & 0xFFFFFFFF00000000u) | v[2 * w + 1] >> 32));
            *x = w == 0 ? s : *x + s;
        }
        return there;
    }
    __device__ __forceinline__ void put_scale(float x) const { put(scale, __float_as_uint(x)); }
    __device__ __forceinline__ bool scale_there(uint32_t* v) const {
        const uint64_t x = poll64(scale);
        *v = (uint32_t)__builtin_amdgcn_readfirstlane((int)(x >> 32));
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)x) == number;
    }
};

// Call: CallMarked, or CallTables / CallWords if no other kernel has prepared anything (a run: `recs` is then the page table).
template <bool RUN, bool GATHER, bool SCATTER, class Call>
__global__ __launch_bounds__(kUpdThreads) void apm_adamw_clip_kernel(ClipArgs c, UpdateArgs a, Call call) {
    constexpr int U = APM_UPDATE_U;
    constexpr bool kMarked = std::is_same<Call, CallMarked>::value;
    const int lane = (int)threadIdx.x;
    uint32_t w = blockIdx.x, i, x;
    PageRec* recs = c.recs;  // with the first round trip
    asm("" : "+s"(recs));
    ClipArgs::Class k_;
    CallTables tables{};
    if constexpr (kMarked) {
        k_ = load_class(c.cls);
    } else {
        i32x16 k0 = load_16(c.cls), t = load_16(&call);  // the tables come first
        asm("" : "+s"(k0), "+s"(t));
        k_ = __builtin_bit_cast(ClipArgs::Class, k0);
        tables = __builtin_bit_cast(CallTables, t);
    }
    if (w < k_.first) k_ = load_class(c.cls + 1 + (w >= c.cls[2].first) + (w >= c.cls[3].first));
    // item -> page, index among the page's sums (tiles, then the adder) or among its slices
    bool sums = true;
    w -= k_.first;
    if (w < k_.n_ahead) {
        i = k_.sum.quotient(w);
        x = w - i * k_.sum.per;
    } else if (w < k_.n_mixed) {
        w -= k_.n_ahead;
        i = k_.both.quotient(w);
        x = w - i * k_.both.per;
        sums = x < k_.sum.per;
        if (sums) i += (uint32_t)k_.ahead;
        else x -= k_.sum.per;
    } else {
        w -= k_.n_mixed;
        i = k_.slices.quotient(w);
        x = w - i * k_.slices.per;
        i += k_.after;
        sums = false;
    }
    i += (uint32_t)k_.begin;
    const int32_t wait_limit = k_.wait_limit;
    PageRec rec;
    int64_t at;
    typename std::conditional<kMarked, HandedMarked, HandedTagged>::type hand;
    if constexpr (RUN) {
        PageRun* r = reinterpret_cast<PageRun*>(recs) + i;
        at = (int64_t)i * c.E;
        typedef const int32_t __attribute__((address_space(4))) * Const;
        const int used = kMarked ? load_run(r).used : ((Const)reinterpret_cast<const int32_t*>(recs))[i];
        rec = class_rec(used, 0.0f, 0, 0, 0, c.g16 + at, c.p16 + at);
        if constexpr (kMarked) hand.scale = (GlobalU32) reinterpret_cast<uint32_t*>(&r->scale);
    } else if constexpr (kMarked) {
        rec = load_rec(recs + i);
        at = rec.pofs;
        hand.scale = (GlobalU32) reinterpret_cast<uint32_t*>(&recs[i].scale);
    } else {
        uint32_t place = (uint32_t)tables.first + i;
        if (tables.listed) place = call_word(&call, 2 * place);
        rec = call_rec<GATHER, SCATTER>(tables, __builtin_bit_cast(PagePlace, load_rec(reinterpret_cast<const PageRec*>(tables.places) + place)), &call);
        at = rec.pofs;
    }
    if constexpr (kMarked) {
        hand.sum = (GlobalU64)(c.sums + (int64_t)i * c.S);
    } else {
        hand.sum = (GlobalU64)(tables.sums + (int64_t)i * tag_sums(c.S));
        hand.scale = (GlobalU64)(tables.scales + (int64_t)i * kTagLine);
        hand.number = tables.number;
    }
    const int n_tiles = max(1, (rec.used + kReduceTile - 1) / kReduceTile);
    if (sums && x + 1 < k_.sum.per) {
        const int tile = (int)x / (kMarked ? 1 : kTileParts);
        if (tile >= n_tiles) return;
        double t;
        if constexpr (kMarked) t = tile_sum<GATHER>(rec, tile, lane);
        else t = part_sum<GATHER>(rec, tile, (int)x % kTileParts, lane);
        if (lane == 0) hand.put_sum((int)x, t);
        return;
    }
    if (sums) {
        double s = 0.0;
        bool all = true;
#pragma unroll 1
        for (int t = 0; t < n_tiles && all; t += kWave) {
            double v = 0.0;
            for (int polls = 0;; ++polls) {
                bool there = true;
                if (t + lane < n_tiles) there = hand.sum_there(t + lane, &v);
                all = __all(there);
                if (all || polls >= wait_limit) break;
                __builtin_amdgcn_s_sleep(4);
            }
            if (t + lane < n_tiles) s += v;
        }
        s = all ? wave_sum_f64(s) : page_sum<GATHER>(rec, n_tiles, lane, [] { return false; });
        const double norm = sqrt(s);
        if (lane != 0) return;
        hand.put_scale(clip_scale(norm, c.max_norm));
        int64_t o = c.out_first + i;
        if constexpr (!RUN && !kMarked) o = tables.listed ? (int64_t)call_word(&call, 2 * (uint32_t)o + 1) : (int64_t)tables.places[o].page;
        else if (c.out_index) o = (int64_t)c.out_index[i];
        if (c.grad_norm) c.grad_norm[o] = (float)norm;
        if (c.skip_mask) c.skip_mask[o] = 0;
        return;
    }
    const int start = (int)x * kTile<U>;
    if (start >= ((rec.used + 7) & ~7)) return;
    // called when the slice's loads are under way: the first poll comes back with them
    auto get_scale = [&]() -> float {
        uint32_t seen = 0;
        bool there = false;
        auto look = [&] { return there = hand.scale_there(&seen); };
        for (int polls = 0; !look(); ++polls) {
            if (polls >= wait_limit) {
                const double s = page_sum<GATHER>(rec, n_tiles, lane, [&] { return wait_limit > 0 && look(); });
                return there ? __uint_as_float(seen) : clip_scale(sqrt(s), c.max_norm);
            }
            __builtin_amdgcn_s_sleep(2);
        }
        return __uint_as_float(seen);
    };
    const int k = start >= rec.off1 ? 1 : 0;
    float *p = c.p32 + at, *m = c.m32 + at, *v = c.v32 + at;
    if (start + kTile<U> <= rec.end[k]) {
        full_slice<U, kStoreHbm>(a, get_scale, lane, p + start, m + start, v + start, rec.g[k] + start, rec.q[k] + start);
    } else {
        rec.scale = get_scale();
        cut_slice<U, GATHER, SCATTER>(a, rec, (start >> 2) + lane, p, m, v);
    }
}

struct TakeArgs {
    uint16_t* dst;
    const uint16_t* src;
    const int32_t* used;
    const int64_t* order;  // or nullptr: first + position
    int64_t first;
    int64_t E;
    double* sums;
    uint32_t* nzflags;
    int32_t S;
    int32_t at;            // position of the map's first item
    GridMap map;
};
struct TakeArgsInline {
    TakeArgs a;
    int32_t page[kTakePages];
};

// dst <- src, or g' <- bf16_rne(fp32(g') + fp32(g)) (Alg. 2, buffering thread: "accumulate buffered
// gradients"), over the used extent of each listed page; 4 or 6 B per element, HBM-bound.  Only used
// extents move: of the 533 pages of a 24-layer model 195 hold a bias or a norm.
// SUMS: also the tile's sum of squares and non-zero flag of what was written, with the additions in the
// order of apm_grad_reduce_kernel, so that the update that follows does not read the gradient twice.
// 355 M parameters with clipping, hand-over beside the update: 2041 us an iteration with copies of whole
// pages and the sums worked out by the update, 1877 like this; 124 M, four micro-batches, no clipping: 1116
// and 1030.  A workgroup then takes a tile; without, 8 elements per lane, the fastest form of a copy.  Stores are written
// through as the state's are (355 M, hand-over beside the update: 1766 -> 1760 us), but for sums over what is added, where a
// workgroup goes through its tile in two spans and loads wait behind stores (added with clipping, written through / not:
// 0.6 M elements 11.6 / 9.4 us, 4.8 M 14.2 / 12.8, 135 M 143.1 / 141.7; without clipping 26 M 25.8 / 27.6).
// It runs beside the update, where its wavefronts add to those in flight, which like the update's own lower the bandwidth
// beyond some number: so it requests LDS as well, and shares a CU's with the update's (by itself, 21 of one wavefront, or 6 of four where
// sums are worked out, fit a CU).  Without sums a workgroup is one wavefront: four of them end when the last one does (but see take_by_four).
// us an iteration with four-wavefront workgroups / of one / of one with LDS of 5120 / 7680 / 10240: 124 M, one hand-over and three
// additions 1026 / 1021 / 974 / 966 / 970; 303 M 1535 / 1515 / 1488 / 1495 / 1520; 355 M with sums and LDS of 0 / 14336 / 27136 / 40960: 1798 /
// 1776 / 1772 / 1800.  From how many elements on, without / with LDS: three additions 6.6 M 77.3 / 76.9, 9.8 M 97.8 / 93.1, 22 M 192 / 177 (4.8 M by
// itself 10.2 / 11.0), with sums (0 / 14336 / 27136) 13 M 144 / 138 / 146, in 64 K pages 15 M 143 / 141 / 148, 93 M 813 / 783 / 794; a hand-over alone 6.6 M
// 39.3 / 39.6, 22 M 116.4 / 116.8, 31 M 160.9 / 159.9, with sums 30 M 155 / 159 / 156, 93 M 477 / 489 / 491 and 474 / 471 / 472, 231 M 1211 / 1194 / 1177.
struct TakeCap {
    int64_t few;   // elements up to which no LDS is requested
    unsigned lds;
};
constexpr TakeCap take_cap(bool accumulate, bool sums) {
    const int64_t m = (int64_t)1 << 20;
    return accumulate ? TakeCap{8 * m, sums ? 14336u : 7680u} : sums ? TakeCap{128 * m, 27136u} : TakeCap{24 * m, 7680u};
}
// With sums, pages that hold less than a quarter of a tile on average go without LDS: their workgroups end after a load or two, and more of them have
// to be on a CU.  us an iteration with clipping and one / three additions, without / with it: 9 M elements, 300 a page, 159 / 172 and 286 / 284;
// 24 M, 300 a page, 477 / 477 and 680 / 711; 8.6 M, 2867 on average, 106.7 / 108.1 and 126.6 / 130.0; 20 M, 4096 a page, 140.6 / 139.5 and 186.4 / 182.8.
//
// Without sums, small calls over pages that hold much less than their class's largest (`spanned` elements in all, if they did not) take four
// wavefronts a workgroup, as there are four times fewer that find nothing to do: in pages of up to 8 K elements always, where those come between the
// others, in larger ones, where they come in long rows, if they are most of the grid.  us an iteration with one / three additions, a workgroup of
// one wavefront / of four, spanned / elems 2 but where stated: 6 M elements in pages of 2048 61.2 / 61.1 and 75.3 / 70.8, 4096 60.7 / 56.2 and 75.0 / 73.4
// (1.3: 60.0 / 57.8 and 78.7 / 78.5), 8192 59.3 / 57.4 and 75.1 / 74.3, 16 K 50.4 / 50.7 and 68.6 / 69.2, 32 K 46.3 / 47.5 and 64.9 / 70.3, 64 K 48.6 / 50.3 and
// 66.7 / 74.1; 4.8 M in 1 M pages (2.6) 40.2 / 40.0 and 60.6 / 57.6, an addition alone 9.9 / 8.8; full pages of 64 elements, an addition alone 26.8 / 40.8.
constexpr bool take_by_four(int64_t elems, int64_t spanned, int64_t largest) {
    return elems <= (int64_t)8 << 20 && (largest <= 8192 ? 4 * spanned > 5 * elems : 4 * spanned > 9 * elems);
}

template <bool ACCUM, bool SUMS, int T, class Args>
__global__ __launch_bounds__(T) void apm_grad_take_kernel(Args args) {
    const TakeArgs* ap;
    if constexpr (sizeof(Args) > sizeof(TakeArgs)) ap = &args.a;
    else ap = &args;
    const TakeArgs& a = *ap;
    int pos;
    uint32_t tile;
    grid_item(a.map.large_at, a.map.large, a.map.small, blockIdx.x, &pos, &tile);
    pos += a.at;
    int64_t page;
    if constexpr (sizeof(Args) > sizeof(TakeArgs)) page = args.page[pos];
    else page = a.order ? a.order[pos] : a.first + pos;
    constexpr int U = SUMS ? APM_REDUCE_U : 1, kSpan = T * 8 * U, kItem = SUMS ? kReduceTile : kSpan;
    const int used = a.used[page], used8 = (used + 7) & ~7;
    const int start = (int)tile * kItem;
    if (start >= used8 && !(SUMS && tile == 0)) return;
    const int end = min(start + kItem, used8);
    u32x4* dst = reinterpret_cast<u32x4*>(a.dst + page * a.E);
    const Rsrc D = make_rsrc(a.dst + page * a.E + start, end > start ? (end - start) * 2 : 0);
    const u32x4* src = reinterpret_cast<const u32x4*>(a.src + page * a.E);
    double acc0 = 0.0, acc1 = 0.0;
    uint32_t nz = 0;
#pragma unroll 1
    for (int at = start; at < end; at += kSpan) {
        u32x4 x[U], y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = at + (u * T + (int)threadIdx.x) * 8;
            x[u] = u32x4{0u, 0u, 0u, 0u};
            if (e < end) {
                x[u] = __builtin_nontemporal_load(src + (e >> 3));
                if (ACCUM) y[u] = __builtin_nontemporal_load(dst + (e >> 3));
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = at + (u * T + (int)threadIdx.x) * 8;
            if (e < end) {
                if (ACCUM) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float lo = bf16lo(y[u][j]) + bf16lo(x[u][j]);
                        const float hi = bf16hi(y[u][j]) + bf16hi(x[u][j]);
                        x[u][j] = f32_to_bf16_rne(lo) | (f32_to_bf16_rne(hi) << 16);
                    }
                }
                __builtin_amdgcn_raw_buffer_store_b128(x[u], D, (e - start) * 2, 0, ACCUM && SUMS ? kStoreNT : kStoreHbm);
            }
            if (SUMS) {
                const int left = used - e;  // boundary vector: elements at or beyond the extent do not count
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t v = left >= 2 * j + 2 ? x[u][j] : left == 2 * j + 1 ? x[u][j] & 0x0000FFFFu : 0u;
                    nz |= v & 0x7FFF7FFFu;
                    const double lo = (double)bf16lo(v), hi = (double)bf16hi(v);
                    acc0 = fma(lo, lo, acc0);
                    acc1 = fma(hi, hi, acc1);
                }
            }
        }
    }
    if (!SUMS) return;
    __shared__ double s_acc[kThreads / kWave];
    __shared__ uint32_t s_nz[kThreads / kWave];
    block_sum(acc0 + acc1, nz, s_acc, s_nz, a.sums + page * a.S + tile, a.nzflags + page * a.S + tile);
}

constexpr int kMaxGridY = 65535;

}  // namespace

hipError_t launch_grad_take(const GradTake& t, hipStream_t s) {
    TakeArgsInline in;
    in.a = TakeArgs{t.dst, t.src, t.used, t.order, t.first, t.E, t.sums, t.nzflags, t.S, 0, {}};
    int64_t elems = 0, spanned = 0, pages = 0;
    for (int k = 0; k < t.n_cls; ++k) {
        spanned += t.cls[k].count * t.cls[k].max_used;
        elems += t.cls[k].sum_used > 0 ? t.cls[k].sum_used : t.cls[k].count * t.cls[k].max_used;  // at most
        pages += t.cls[k].count;
    }
    const TakeCap cap = take_cap(t.accumulate, t.sums != nullptr);
    const unsigned lds = elems <= cap.few || (t.sums && elems < kOnePassElems * pages) ? 0 : cap.lds;
    const int threads = t.sums || take_by_four(elems, spanned, t.n_cls > 0 ? t.cls[0].max_used : 0) ? kThreads : kWave, item = t.sums ? kReduceTile : threads * 8;
    // positions of the given classes in one grid
    auto go = [&](const ExtentClass* cls, int n_cls) -> hipError_t {
        while (n_cls > 0 && cls[n_cls - 1].max_used <= 0 && !t.sums) --n_cls;  // nothing to take
        return (hipError_t)for_each_grid(cls, n_cls, threads, t.max_workgroups,
            [&](const ExtentClass& c) { return c.max_used > 0 ? (c.max_used + item - 1) / item : 1; },
            [&](const GridMap& m, int64_t workgroups, int64_t first) -> int {
                in.a.at = (int32_t)first;
                in.a.map = m;
                const dim3 grid((unsigned)workgroups);
#define APM_TAKE(ACCUM, SUMS, T)                                                                                    \
    do {                                                                                                           \
        if (t.host_pages) hipLaunchKernelGGL((apm_grad_take_kernel<ACCUM, SUMS, T, TakeArgsInline>), grid, dim3(T), lds, s, in); \
        else hipLaunchKernelGGL((apm_grad_take_kernel<ACCUM, SUMS, T, TakeArgs>), grid, dim3(T), lds, s, in.a);      \
    } while (0)
                if (t.accumulate && t.sums) APM_TAKE(true, true, kThreads);
                else if (t.sums) APM_TAKE(false, true, kThreads);
                else if (t.accumulate && threads == kThreads) APM_TAKE(true, false, kThreads);
                else if (t.accumulate) APM_TAKE(true, false, kWave);
                else if (threads == kThreads) APM_TAKE(false, false, kThreads);
                else APM_TAKE(false, false, kWave);
#undef APM_TAKE
                return (int)hipGetLastError();
            });
    };
    if (!t.host_pages) return go(t.cls, t.n_cls);
    // kTakePages positions a launch, whatever their classes
    int64_t n = 0;
    for (int k = 0; k < t.n_cls; ++k) n += t.cls[k].count;
    for (int64_t at = 0; at < n; at += kTakePages) {
        ExtentClass part[kMaxExtentClasses];
        int n_part = 0;
        for (int k = 0; k < t.n_cls; ++k) {
            const int64_t b = t.cls[k].begin > at ? t.cls[k].begin : at, end = t.cls[k].begin + t.cls[k].count;
            const int64_t e = end < at + kTakePages ? end : at + kTakePages;
            if (b < e) part[n_part++] = ExtentClass{b - at, e - b, t.cls[k].max_used, 0};
        }
        for (int64_t i = at; i < n && i < at + kTakePages; ++i) in.page[i - at] = (int32_t)t.host_pages[i];
        const hipError_t e = go(part, n_part);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

namespace {
// Calls f(first list position, pages, largest used extent, the class's used elements) for every launch of a pass: per extent
// class, in pieces of at most kMaxGridY pages.
template <class F>
hipError_t for_each_launch(const AdamwLaunch& L, F&& f) {
    const ExtentClass all{0, L.n_listed, L.E, L.n_listed * L.E};
    const ExtentClass* c = L.n_cls > 0 ? L.cls : &all;
    const int n = L.n_cls > 0 ? L.n_cls : 1;
    for (int k = 0; k < n; ++k) {
        for (int64_t off = 0; off < c[k].count; off += kMaxGridY) {
            const int64_t ny = c[k].count - off < kMaxGridY ? c[k].count - off : kMaxGridY;
            f(c[k].begin + off, ny, c[k].max_used > 0 ? c[k].max_used : 1, c[k].sum_used);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}
}  // namespace

// Workgroups for one thread per listed page, or, if sums have to be marked, up to eight of those per thread.
static unsigned record_grid(const AdamwLaunch& L) {
    int64_t threads = L.n_listed;
    if (L.one_pass && threads < L.n_listed * L.S / 8) threads = L.n_listed * L.S / 8;
    return (unsigned)((threads + kThreads - 1) / kThreads);
}

// The classes that the grid over noted pages walks: of the launch's, those that would not be worth a launch of their own
// join the next larger one if that one's wavefronts are more than the least.  How many a class gets depends on what
// it could hold, so the few slots of small pages keep some more of them for the large ones: 135 M parameters, half / all
// of them live, 64 experts and their norms, 332 / 698 us with the norms' pages in the experts' class, 338 / 710 apart.  With the least
// number of wavefronts the empty slices only lengthen each one's walk: 4.8 M in 1 M pages 36.4 us a call apart, 37.9 together.
static int live_classes(const AdamwLaunch& L, ExtentClass out[kMaxExtentClasses]) {
    if (L.n_cls == 0) {
        out[0] = ExtentClass{0, L.n_listed, L.E, L.n_listed * L.E};
        return 1;
    }
    for (int c = 0; c < L.n_cls; ++c) out[c] = L.cls[c];
    int n = L.n_cls;
    for (int c = n - 1; c > 0; --c) {
        if (out[c].count * ((out[c - 1].max_used - out[c].max_used) / 1024) >= kWorthLaunch) continue;
        if (out[c - 1].count * ((out[c - 1].max_used + kTile<kSkipU> - 1) / kTile<kSkipU>) <= (int64_t)kSkipWaves * kSkipSpread) continue;
        out[c - 1].count += out[c].count;
        out[c - 1].sum_used += out[c].sum_used;
        for (int k = c + 1; k < n; ++k) out[k - 1] = out[k];
        --n;
    }
    return n;
}

// Whether the finalize pass notes the pages that are not skipped, for the grid over noted pages (see kSkipSpread).
static bool notes_live(const AdamwLaunch& L) {
    if (L.skip_mode != APM_SKIP_UNTOUCHED || L.stride_wavefronts > 0) return false;
    ExtentClass cls[kMaxExtentClasses];
    int64_t n = 0;
    for (int c = live_classes(L, cls) - 1; c >= 0; --c) n += cls[c].count * ((cls[c].max_used + kTile<kSkipU> - 1) / kTile<kSkipU>);
    return n > kSkipWaves;
}

hipError_t launch_grad_reduce(const AdamwLaunch& L, hipStream_t s) {
    hipError_t e = hipSuccess;
    int32_t* live = notes_live(L) ? L.live : nullptr;
    ReduceArgs a{L.g16, L.used, L.grad_pages, L.grad_first, 0, L.E, L.partials, L.nzflags, L.S, live, {}};
    if (L.sums_ready && live) hipLaunchKernelGGL(apm_live_clear_kernel, dim3(1), dim3(kWave), 0, s, live);
    const bool sums = L.max_norm > 0.0 || L.grad_norm;
    const ExtentClass all{0, L.n_listed, L.E, L.n_listed * L.E};
    if (!L.sums_ready) e = (hipError_t)for_each_grid(L.n_cls > 0 ? L.cls : &all, L.n_cls > 0 ? L.n_cls : 1, kThreads, L.max_workgroups,
        [](const ExtentClass& c) { return c.max_used > 0 ? (c.max_used + kReduceTile - 1) / kReduceTile : 1; },
        [&](const GridMap& m, int64_t workgroups, int64_t first) -> int {
            a.list_offset = first;
            std::memcpy(a.small, m.small, sizeof a.small);
            auto go = [&](const auto& call) {
                typedef typename std::decay<decltype(call)>::type Call;
                auto kernel = L.gather ? (sums ? apm_grad_reduce_kernel<true, true, Call> : apm_grad_reduce_kernel<true, false, Call>)
                                       : (sums ? apm_grad_reduce_kernel<false, true, Call> : apm_grad_reduce_kernel<false, false, Call>);
                hipLaunchKernelGGL(kernel, dim3((unsigned)workgroups), dim3(kThreads), 0, s, L.recs + first, m.large_at, m.large.per, m.large.mul, m.large.shift,
                                   a, call);
            };
            if (L.call) go(*L.call);
            else go(CallNone{});
            return (int)hipGetLastError();
        });
    if (e != hipSuccess) return e;
    FinalizeArgs f{L.used, L.grad_pages, L.state_pages, L.grad_first, L.state_first, L.n_listed,
                   L.partials, L.nzflags, L.S, L.skip_mode, L.max_norm, L.recs, L.g16, L.p16, L.E, live, {}, 0, L.sums_ready, L.is_run(),
                   L.gather || L.scatter, nullptr, L.grad_norm, L.skip_mask, L.out_index, L.gather, L.scatter};
    ExtentClass live_cls[kMaxExtentClasses];
    f.n_cls = live_classes(L, live_cls);
    for (int c = 0; c < f.n_cls; ++c) f.cls_begin[c] = live_cls[c].begin;
    auto go = [&](const auto& call) {
        typedef typename std::decay<decltype(call)>::type Call;
        auto start = [&](auto kernel, int waves, int pages) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)((L.n_listed + pages - 1) / pages)), dim3((unsigned)(waves * kWave)), 0, s, f, call);
        };
        auto sized = [&](auto with_sums) {
            constexpr bool SUMS = decltype(with_sums)::value;
            if (L.n_listed <= 1024) start(apm_grad_finalize_kernel<4, 1, SUMS, Call>, 4, 4);
            else if (L.n_listed <= 4096) start(apm_grad_finalize_kernel<16, 1, SUMS, Call>, 16, 16);
            else start(apm_grad_finalize_kernel<16, 4, SUMS, Call>, 16, 64);
        };
        if (sums) sized(std::true_type{});
        else sized(std::false_type{});
    };
    if (L.call) go(*L.call);
    else go(CallNone{});
    return hipGetLastError();
}

hipError_t launch_prepare(const AdamwLaunch& L, hipStream_t s) {
    FinalizeArgs f{L.used, L.grad_pages, L.state_pages, L.grad_first, L.state_first, L.n_listed,
                   nullptr, nullptr, L.S, L.skip_mode, 0.0, L.recs, L.g16, L.p16, L.E, nullptr, {}, 0, false, L.is_run(),
                   false, L.one_pass ? reinterpret_cast<uint64_t*>(L.partials) : nullptr, nullptr, nullptr, nullptr, false, false};
    hipLaunchKernelGGL(apm_page_recs_kernel, dim3(record_grid(L)),
                       dim3(kThreads), 0, s, f);
    return hipGetLastError();
}

int64_t stage_launches_runs(int64_t n_runs, int64_t lists, int64_t n_tensors) {
    if (run_words(n_runs) + lists * n_tensors <= 2 * kArgWords) return 1;
    const int64_t per = lists ? 2 * kArgWords / lists : 1;
    return (n_runs + kStageRuns - 1) / kStageRuns + (lists ? (n_tensors + per - 1) / per : 0);
}

int64_t stage_launches(int64_t n_list, int64_t lists, int64_t n_tensors, bool narrow) {
    const int64_t room = narrow ? 2 * kArgWords : kArgWords;
    if ((narrow ? 2 : 1) * n_list + lists * n_tensors <= room) return 1;
    const int64_t per = lists ? room / lists : room;
    return (n_list + kArgWords - 1) / kArgWords + (lists ? (n_tensors + per - 1) / per : 0);
}

hipError_t launch_stage(const AdamwLaunch& L, const StageCall& c, hipStream_t s) {
    const bool has_g = c.g_ptrs != nullptr, has_q = c.q_ptrs != nullptr;
    const bool listed = c.list || c.runs;
    const int64_t n_list = listed ? L.n_listed : 0, n_t = has_g || has_q ? c.n_tensors : 0;
    StageArgsInline in;
    StageArgsNarrow half;
    StageArgsRuns runs;
    StageArgs a{L.used, listed ? c.d_list : L.grad_pages, L.grad_first, L.n_listed, c.tenants, L.recs, L.g16, L.p16, L.E,
                  c.d_list, c.d_out, L.one_pass ? reinterpret_cast<uint64_t*>(L.partials) : nullptr,
                  L.one_pass ? L.n_listed * L.S : 0, c.d_words, 0, 0, 0, 0, 0, has_g, has_q, c.g_base, c.q_base};
    auto go = [&](int64_t list_begin, int64_t list_n, int64_t t_begin, int64_t t_n) -> hipError_t {
        a.list_begin = list_begin;
        a.list_n = (int32_t)list_n;
        a.t_begin = (int32_t)t_begin;
        a.t_n = (int32_t)t_n;
        const int64_t threads = list_n > 0 ? list_n : L.n_listed;
        const unsigned pages_grid = (unsigned)((threads + kThreads - 1) / kThreads), sums_grid = a.sums ? record_grid(L) : 0u;
        const dim3 grid(pages_grid > sums_grid ? pages_grid : sums_grid);
        if (c.d_words) {
            hipLaunchKernelGGL(apm_stage_kernel<StageArgs>, grid, dim3(kThreads), 0, s, a);
        } else if (c.narrow) {
            uint32_t* w = half.word;
            for (int64_t k = 0; k < list_n; ++k) *w++ = (uint32_t)c.list[list_begin + k];
            for (int64_t k = 0; k < list_n; ++k) *w++ = (uint32_t)(c.list[list_begin + k] >> 32);
            // an empty tensor's address may be anything: it is nobody's tenant
            for (int64_t k = 0; has_g && k < t_n; ++k) *w++ = (uint32_t)((c.g_ptrs[t_begin + k] - c.g_base) >> 4);
            for (int64_t k = 0; has_q && k < t_n; ++k) *w++ = (uint32_t)((c.q_ptrs[t_begin + k] - c.q_base) >> 4);
            half.a = a;
            hipLaunchKernelGGL(apm_stage_kernel<StageArgsNarrow>, grid, dim3(kThreads), 0, s, half);
        } else {
            in.a = a;
            uint64_t* w = in.word;
            if (list_n > 0) std::memcpy(w, c.list + list_begin, (size_t)list_n * sizeof(uint64_t));
            w += list_n;
            if (t_n > 0 && has_g) std::memcpy(w, c.g_ptrs + t_begin, (size_t)t_n * sizeof(uint64_t));
            if (has_g) w += t_n;
            if (t_n > 0 && has_q) std::memcpy(w, c.q_ptrs + t_begin, (size_t)t_n * sizeof(uint64_t));
            hipLaunchKernelGGL(apm_stage_kernel<StageArgsInline>, grid, dim3(kThreads), 0, s, in);
        }
        a.sums = nullptr;  // marked by the first launch
        return hipGetLastError();
    };
    // runs [r, r + n) and, with the last of them, all addresses
    auto go_runs = [&](int64_t r, int64_t n, int64_t t_n) -> hipError_t {
        const int64_t begin = (int64_t)c.runs[r].at, end = r + n < c.n_runs ? (int64_t)c.runs[r + n].at : n_list;
        uint32_t* w = runs.word;
        std::memcpy(w, c.runs + r, (size_t)n * sizeof(StageRun));
        w += n * (int64_t)(sizeof(StageRun) / sizeof(uint32_t));
        for (int64_t k = 0; has_g && k < t_n; ++k) *w++ = (uint32_t)((c.g_ptrs[k] - c.g_base) >> 4);
        for (int64_t k = 0; has_q && k < t_n; ++k) *w++ = (uint32_t)((c.q_ptrs[k] - c.q_base) >> 4);
        runs.a = a;
        runs.a.list_begin = begin;
        runs.a.list_n = (int32_t)(end - begin);
        runs.a.n_runs = (int32_t)n;
        runs.a.t_n = (int32_t)t_n;
        const unsigned pages_grid = (unsigned)((end - begin + kThreads - 1) / kThreads), sums_grid = a.sums ? record_grid(L) : 0u;
        hipLaunchKernelGGL(apm_stage_kernel<StageArgsRuns>, dim3(pages_grid > sums_grid ? pages_grid : sums_grid), dim3(kThreads), 0, s, runs);
        a.sums = nullptr;
        return hipGetLastError();
    };
    if (c.runs && run_words(c.n_runs) + (has_g + has_q) * n_t <= 2 * kArgWords) return go_runs(0, c.n_runs, n_t);
    if (c.d_words || (!c.runs && stage_launches(n_list, has_g + has_q, n_t, c.narrow) == 1)) return go(0, n_list, 0, n_t);
    // list words first: the launches with the addresses read the list that they wrote
    for (int64_t k = 0; c.runs && k < c.n_runs; k += kStageRuns) {
        hipError_t e = go_runs(k, c.n_runs - k < kStageRuns ? c.n_runs - k : kStageRuns, 0);
        if (e != hipSuccess) return e;
    }
    for (int64_t k = 0; !c.runs && k < n_list; k += kArgWords) {
        hipError_t e = go(k, n_list - k < kArgWords ? n_list - k : kArgWords, 0, 0);
        if (e != hipSuccess) return e;
    }
    const int64_t per = (c.narrow ? 2 : 1) * kArgWords / (has_g && has_q ? 2 : 1);
    for (int64_t k = 0; k < n_t; k += per) {
        hipError_t e = go(0, 0, k, n_t - k < per ? n_t - k : per);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// f(the stores' policy as a constant)
template <class F>
static void with_stores(bool non_temporal_only, F&& f) {
    if (non_temporal_only) f(std::integral_constant<int, kStoreNT>{});
    else f(std::integral_constant<int, kStoreHbm>{});
}

// Workgroups a page of the class takes.
template <int U> int64_t slices_of(const ExtentClass& c) { return c.max_used > 0 ? (c.max_used + kTile<U> - 1) / kTile<U> : 1; }

hipError_t launch_adamw(const AdamwLaunch& L, hipStream_t s) {
    const UpdateArgs a{L.b1, L.omb1, L.b2, L.omb2, L.inv_sqrt_bc2, L.eps, L.step_size, L.lr_wd};
    const bool run = L.is_run();
    const PageRun* runs = reinterpret_cast<const PageRun*>(L.recs);
    // of the page at list position `at` of a run
    auto state = [&](float* c, int64_t at) { return run ? c + (L.state_first + at) * L.E : c; };
    auto g16 = [&](int64_t at) { return L.g16 + (L.grad_first + at) * L.E; };
    auto p16 = [&](int64_t at) { return L.p16 + (L.grad_first + at) * L.E; };
    if (L.stride_wavefronts > 0) {
        if (L.gather || L.scatter) return hipErrorInvalidValue;  // host-resident state goes with the page classes
        const int64_t slices = L.n_listed * ((L.E + kTile<kStrideU> - 1) / kTile<kStrideU>);
        const int workers = (int)(slices < L.stride_wavefronts ? slices : L.stride_wavefronts);
        const int per_wg = L.stride_waves_per_wg >= 1 && L.stride_waves_per_wg <= kStrideMaxThreads / kWave ? L.stride_waves_per_wg : 1;
        const dim3 grid((unsigned)((workers + per_wg - 1) / per_wg)), block((unsigned)(per_wg * kWave));
        const StrideArgs t{L.recs, state(L.p32, 0), state(L.m32, 0), state(L.v32, 0), run ? g16(0) : nullptr, run ? p16(0) : nullptr,
                           L.E, L.n_listed, workers, {L.link_slots[0], L.link_slots[1], L.link_slots[2]}};
        auto go = [&](auto in_a_run, auto written_through) {
            constexpr bool RUN = decltype(in_a_run)::value, WT = decltype(written_through)::value;
            hipLaunchKernelGGL((apm_adamw_stride_kernel<RUN, WT>), grid, block, 0, s, t, a);
        };
        const std::true_type yes;
        const std::false_type no;
        if (L.link_slots[0]) {
            // the streamer's pages are a run, and without the update they are not written through (it has another form of that)
            if (!run || (L.host_write_through && !L.link_update)) return hipErrorInvalidValue;
            constexpr int kMost = kStrideMaxThreads, kHalf = kMost / 2;
            const bool half = (int)block.x <= kHalf;
            auto kernel = L.host_write_through ? (half ? apm_adamw_staged_kernel<true, true, kHalf> : apm_adamw_staged_kernel<true, true, kMost>)
                          : L.link_update      ? (half ? apm_adamw_staged_kernel<false, true, kHalf> : apm_adamw_staged_kernel<false, true, kMost>)
                                               : (half ? apm_adamw_staged_kernel<false, false, kHalf> : apm_adamw_staged_kernel<false, false, kMost>);
            hipLaunchKernelGGL(kernel, grid, block, 0, s, t, a);
        } else if (run && L.host_write_through) go(yes, yes);
        else if (run) go(yes, no);
        else if (L.host_write_through) go(no, yes);
        else go(no, no);
        return hipGetLastError();
    }
    if (L.partials && notes_live(L)) {
        constexpr int U = kSkipU;
        ExtentClass cls[kMaxExtentClasses];
        const int n_cls = live_classes(L, cls);
        const bool wide = run && L.wide;
        const int tile = wide ? kTile<kWideU> : kTile<U>;
        const int64_t cap = L.max_workgroups > 0 ? L.max_workgroups : max_workgroups(kUpdThreads);
        int64_t wgs[kMaxExtentClasses], total = 0;
        for (int c = 0; c < n_cls; ++c) {
            const int64_t slices = cls[c].count * ((cls[c].max_used + tile - 1) / tile);
            wgs[c] = (slices + kSkipSpread - 1) / kSkipSpread;
            if (wgs[c] < kSkipWaves) wgs[c] = slices < kSkipWaves ? slices : kSkipWaves;
            total += wgs[c];
        }
        const bool together = total <= cap;
        for (int c0 = n_cls - 1; c0 >= 0; --c0) {  // all classes at once, or one after the other
            LiveClasses lc{};
            int64_t at = 0;
            int k = 1;
            const int last = together ? 0 : c0;
            for (int c = c0; c >= last; --c) {
                if (wgs[c] <= 0 && c > last) continue;
                if (wgs[c] > cap) wgs[c] = cap;  // each walks further
                LiveClasses::Class& q = lc.cls[c == last ? 0 : k++];
                q.first = (uint32_t)at;
                q.begin = (int32_t)cls[c].begin;
                q.number = c;
                q.slices = grid_div(cls[c].max_used > 0 ? (cls[c].max_used + tile - 1) / tile : 1);
                q.di = (uint32_t)wgs[c] / q.slices.per;
                q.dx = (uint32_t)wgs[c] - q.di * q.slices.per;
                at += wgs[c];
            }
            for (; k < kMaxExtentClasses; ++k) lc.cls[k].first = lc.cls[0].first;
            if (at > 0) {
                const dim3 grid((unsigned)at), block(kUpdThreads);
#define APM_LAUNCH_LIVE(...) hipLaunchKernelGGL((apm_adamw_live_kernel<__VA_ARGS__>), grid, block, kSkipLds, s, L.live, \
                                                     L.recs, state(L.p32, 0), state(L.m32, 0), state(L.v32, 0), run ? g16(0) : nullptr,  \
                                                     run ? p16(0) : nullptr, L.E, a, lc)
                with_stores(L.beside_link, [&](auto store) {
                    constexpr int STORE = decltype(store)::value;
                    if (wide) APM_LAUNCH_LIVE(kWideU, true, false, false, STORE);
                    else if (run) APM_LAUNCH_LIVE(U, true, false, false, STORE);
                    else if (L.gather && L.scatter) APM_LAUNCH_LIVE(U, false, true, true, kStoreHbm);
                    else if (L.gather) APM_LAUNCH_LIVE(U, false, true, false, kStoreHbm);
                    else if (L.scatter) APM_LAUNCH_LIVE(U, false, false, true, kStoreHbm);
                    else APM_LAUNCH_LIVE(U, false, false, false, STORE);
                });
#undef APM_LAUNCH_LIVE
                const hipError_t e = hipGetLastError();
                if (e != hipSuccess) return e;
            }
            if (together) break;
        }
        return hipSuccess;
    }
    constexpr int U = APM_UPDATE_U;
    if (!run) {
        const ExtentClass all{0, L.n_listed, L.E, L.n_listed * L.E};
        const ExtentClass* cls = L.n_cls > 0 ? L.cls : &all;
        const int n_cls = L.n_cls > 0 ? L.n_cls : 1;
        int64_t elems = 0;
        for (int c = 0; c < n_cls; ++c) elems += cls[c].sum_used;
        const unsigned lds = update_lds(L.gather || L.scatter, elems, APM_UPDATE_LDS);
        const bool by_call = L.call && !L.partials;  // after a reduce pass the records are there
        return (hipError_t)for_each_grid(cls, n_cls, kUpdThreads, L.max_workgroups, slices_of<U>, [&](const GridMap& m, int64_t workgroups, int64_t first) -> int {
            SmallClasses classes;
            std::memcpy(classes.small, m.small, sizeof classes.small);
#define APM_LAUNCH_UPDATE(G, Q, STORE) hipLaunchKernelGGL((apm_adamw_kernel<U, G, Q, STORE>), dim3((unsigned)workgroups), dim3(kUpdThreads), lds, s, L.recs + first, \
                                                   L.p32, L.m32, L.v32, m.large_at, m.large.per, m.large.mul, m.large.shift, a, classes)
#define APM_LAUNCH_CALL(G, Q) hipLaunchKernelGGL((apm_adamw_call_kernel<U, G, Q>), dim3((unsigned)workgroups), dim3(kUpdThreads), lds, s, L.call->t.places, \
                                                 L.p32, L.m32, L.v32, m.large_at, m.large.per, m.large.mul, m.large.shift, (uint32_t)first, L.call->t.listed, a, classes, *L.call)
            if (by_call && L.gather && L.scatter) APM_LAUNCH_CALL(true, true);
            else if (by_call && L.gather) APM_LAUNCH_CALL(true, false);
            else if (by_call && L.scatter) APM_LAUNCH_CALL(false, true);
            else if (by_call) APM_LAUNCH_CALL(false, false);
            else if (L.gather && L.scatter) APM_LAUNCH_UPDATE(true, true, kStoreHbm);
            else if (L.gather) APM_LAUNCH_UPDATE(true, false, kStoreHbm);
            else if (L.scatter) APM_LAUNCH_UPDATE(false, true, kStoreHbm);
            else if (L.beside_link) APM_LAUNCH_UPDATE(false, false, kStoreNT);
            else APM_LAUNCH_UPDATE(false, false, kStoreHbm);
#undef APM_LAUNCH_UPDATE
#undef APM_LAUNCH_CALL
            return (int)hipGetLastError();
        });
    }
    return for_each_launch(L, [&](int64_t begin, int64_t ny, int64_t max_used, int64_t sum_used) {
        const bool wide = L.wide;
        const int tile = wide ? kTile<kWideU> : kTile<U>;
        const dim3 grid((unsigned)((max_used + tile - 1) / tile), (unsigned)ny), block(kUpdThreads);
        const unsigned lds = update_lds(false, sum_used, APM_UPDATE_LDS);
#define APM_LAUNCH_RUN(U, BARE, STORE, RUNS) hipLaunchKernelGGL((apm_adamw_run_kernel<U, BARE, STORE>), grid, block, lds, s, RUNS, state(L.p32, begin), \
                                                         state(L.m32, begin), state(L.v32, begin), g16(begin), p16(begin), (int)L.E, a)
        const bool few = L.bare_run && sum_used <= kNtRunElems;
        with_stores(few || L.beside_link, [&](auto store) {
            constexpr int STORE = decltype(store)::value;
            if (wide && L.bare_run) APM_LAUNCH_RUN(kWideU, true, kStoreHbm, L.used + L.grad_first + begin);
            else if (wide) APM_LAUNCH_RUN(kWideU, false, STORE, runs + begin);
            else if (L.bare_run) APM_LAUNCH_RUN(U, true, STORE, L.used + L.grad_first + begin);
            else APM_LAUNCH_RUN(U, false, STORE, runs + begin);
        });
#undef APM_LAUNCH_RUN
    });
}

// In one grid a page takes at least three wavefronts, two of them with next to nothing to do when the page is
// small; with few pages a launch less counts for more, unless the form without a stage kernel has no more launches
// either.  us a call, in one grid / as passes, pages of 512, 1024, 2048, 4096, 8192 elements:
//   64 M elements, consecutive pages   811 / 521  461 / 411  362 / 353  323 / 324  310 / 316
//   8 M, consecutive                    91 / 71    67 / 60    54 / 52    48 / 49    46 / 48
//   256 K, from and to tensors        12.8 / 14.7  12.3 / 14.8  11.7 / 14.7
//   4096 pages of 256, reversed / from and to tensors   47.6 / 43.7, 21.4 / 20.3; 2048 of 512   31.7 / 34.7, 16.5 / 18.9
// What counts is what the pages hold on average: 30 000 tensors of 300 elements alone in pages of 4096, 160 / 113.
bool one_pass_pays(const AdamwLaunch& L, bool staged) {
    int64_t elems = 0;
    for (int c = 0; c < L.n_cls; ++c) elems += L.cls[c].sum_used;
    return L.skip_mode == APM_SKIP_NONE && (elems >= kOnePassElems * L.n_listed || (staged && L.n_listed <= kOnePassPages));
}

hipError_t launch_clip_update(const AdamwLaunch& L, hipStream_t s) {
    const UpdateArgs a{L.b1, L.omb1, L.b2, L.omb2, L.inv_sqrt_bc2, L.eps, L.step_size, L.lr_wd};
    const bool run = L.is_run();
    if (!L.one_pass || !L.partials || L.skip_mode != APM_SKIP_NONE || L.stride_wavefronts > 0) return hipErrorInvalidValue;
    const ExtentClass all{0, L.n_listed, L.E, L.n_listed * L.E};
    const ExtentClass* cls = L.n_cls > 0 ? L.cls : &all;
    const int n_cls = L.n_cls > 0 ? L.n_cls : 1;
    struct Items { int64_t sums, slices, all; };
    const int64_t per_tile = L.call ? kTileParts : 1;
    auto items_of = [&](const ExtentClass& e) {
        const int64_t max_used = e.max_used > 0 ? e.max_used : 1;
        const int64_t sums = (max_used + kReduceTile - 1) / kReduceTile * per_tile + 1, slices = slices_of<APM_UPDATE_U>(e);
        return Items{sums, slices, sums + slices};
    };
    int64_t total = 0, elems = 0;
    for (int k = 0; k < n_cls; ++k) {
        total += cls[k].count * items_of(cls[k]).all;
        elems += cls[k].sum_used;
    }
    const unsigned lds = update_lds(L.gather || L.scatter, elems, kClipLds);
    // pages [begin, begin + count) of each of n classes, the largest first, in one grid
    auto go = [&](const ExtentClass* part, int n) -> hipError_t {
        const int64_t begin = part[0].begin;
        ClipArgs c{};
        c.E = L.E;
        c.S = L.S;
        c.grad_norm = L.grad_norm;
        c.skip_mask = L.skip_mask;
        c.max_norm = L.max_norm;
        int64_t at = 0;
        for (int k = 0; k < n; ++k) {
            const ExtentClass& e = part[n - 1 - k];
            const Items it = items_of(e);
            const int64_t max_used = e.max_used > 0 ? e.max_used : 1, want = (kLookAhead + max_used - 1) / max_used;
            const int64_t ahead = want < e.count ? want : e.count;
            ClipArgs::Class& q = c.cls[k == n - 1 ? 0 : k + 1];
            q.first = (uint32_t)at;
            q.n_ahead = (uint32_t)(ahead * it.sums);
            q.n_mixed = q.n_ahead + (uint32_t)((e.count - ahead) * it.all);
            q.begin = (int32_t)(e.begin - begin);
            q.ahead = (int32_t)ahead;
            // a page's sums are added up 64 at a time, a round trip each
            q.wait_limit = L.wait_limit + (int32_t)((int64_t)L.wait_limit * ((max_used + kReduceTile - 1) / kReduceTile) / 4096);
            q.after = (uint32_t)(e.count - ahead);
            q.sum = grid_div(it.sums);
            q.both = grid_div(it.all);
            q.slices = grid_div(it.slices);
            at += e.count * it.all;
        }
        for (int k = n; k < kMaxExtentClasses; ++k) c.cls[k].first = c.cls[0].first;
        c.recs = run ? reinterpret_cast<PageRec*>(reinterpret_cast<PageRun*>(L.recs) + begin) : L.recs + begin;
        c.sums = reinterpret_cast<uint64_t*>(L.partials) + begin * L.S;
        c.out_index = L.out_index ? L.out_index + begin : nullptr;
        c.out_first = begin;
        const int64_t fp32 = run ? (L.state_first + begin) * L.E : 0, b16 = run ? (L.grad_first + begin) * L.E : 0;
        c.p32 = L.p32 + fp32;
        c.m32 = L.m32 + fp32;
        c.v32 = L.v32 + fp32;
        c.g16 = L.g16 + b16;
        c.p16 = L.p16 + b16;
        const dim3 grid((unsigned)at), block(kUpdThreads);
        auto start = [&](auto call) {
            typedef decltype(call) Call;
            if (L.gather && L.scatter) hipLaunchKernelGGL((apm_adamw_clip_kernel<false, true, true, Call>), grid, block, lds, s, c, a, call);
            else if (L.gather) hipLaunchKernelGGL((apm_adamw_clip_kernel<false, true, false, Call>), grid, block, lds, s, c, a, call);
            else if (L.scatter) hipLaunchKernelGGL((apm_adamw_clip_kernel<false, false, true, Call>), grid, block, lds, s, c, a, call);
            else hipLaunchKernelGGL((apm_adamw_clip_kernel<false, false, false, Call>), grid, block, lds, s, c, a, call);
        };
        if (!L.call) {
            if (run) hipLaunchKernelGGL((apm_adamw_clip_kernel<true, false, false, CallMarked>), grid, block, lds, s, c, a, CallMarked{});
            else start(CallMarked{});
        } else {
            CallWords call = *L.call;
            call.t.sums += begin * tag_sums(L.S);
            call.t.scales += begin * kTagLine;
            call.t.first = (int32_t)begin;
            if (run) c.recs = reinterpret_cast<PageRec*>(const_cast<int32_t*>(L.used + L.grad_first + begin));
            if (run) hipLaunchKernelGGL((apm_adamw_clip_kernel<true, false, false, CallTables>), grid, block, lds, s, c, a, call.t);
            else start(call);
        }
        return hipGetLastError();
    };
    if (total <= (L.max_workgroups > 0 ? L.max_workgroups : max_workgroups(kUpdThreads))) return n_cls > 0 ? go(cls, n_cls) : hipSuccess;
    for (int k = 0; k < n_cls; ++k) {
        const int64_t piece = pages_per_launch(items_of(cls[k]).all, kUpdThreads, L.max_workgroups);
        for (int64_t off = 0; off < cls[k].count; off += piece) {
            ExtentClass part = cls[k];
            part.begin += off;
            part.count = cls[k].count - off < piece ? cls[k].count - off : piece;
            const hipError_t e = go(&part, 1);
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

}  // namespace apm
