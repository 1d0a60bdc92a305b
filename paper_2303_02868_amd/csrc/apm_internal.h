// Internal declarations shared by the library's translation units (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <exception>
#include <functional>
#include <new>
#include <vector>

#include "apm.h"

#if defined(__HIPCC__)
#define APM_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define APM_HOST_DEVICE inline
#endif

namespace apm {

// ---- errors -------------------------------------------------------------------------------
int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));

// Every int-returning entry point runs inside this: no C++ exception crosses the C boundary.
template <class F>
int guarded(F&& f) noexcept {
    try {
        return f();
    } catch (const std::bad_alloc&) {
        return fail(APM_ENOMEM, "out of host memory");
    } catch (const std::exception& e) {
        return fail(APM_EDEVICE, "unexpected failure: %s", e.what());
    } catch (...) {
        return fail(APM_EDEVICE, "unexpected failure");
    }
}

#define APM_HIP(expr)                                                                   \
    do {                                                                                \
        hipError_t apm_e_ = (expr);                                                     \
        if (apm_e_ != hipSuccess)                                                       \
            return ::apm::fail(APM_EDEVICE, "%s failed: %s", #expr, hipGetErrorString(apm_e_)); \
    } while (0)

// ---- packing plan -------------------------------------------------------------------------
constexpr int64_t kAlign = 8;  // elements; keeps 128-bit accesses aligned for both widths

struct PageEntry {
    int64_t used = 0;
    int32_t n_tensors = 0;
    int64_t tensor[2] = {-1, -1};  // index in the tensor list
    int64_t tensor_elems[2] = {0, 0};
};

struct Plan {
    int64_t E = 0;
    int64_t total = 0;
    std::vector<apm_segment> segs;
    std::vector<PageEntry> pages;
};

int make_plan(int64_t E, const int64_t* numels, int64_t n, Plan* out);
int emit_plan(const Plan& plan, apm_segment* segs, int64_t* n_segs, int64_t* n_pages,
              double* fragmentation);

inline int elem_bytes(int state) { return state <= APM_V32 ? 4 : 2; }

// ---- sizes launched together --------------------------------------------------------------
// Items of very different sizes (a page's used extent, a segment) are grouped into at most this many
// classes, largest first, in which an item takes as many workgroups as the class's largest needs:
// a nearly empty page (a small tensor alone in its page) does not cost a full page's worth
// of workgroups that only find out they have nothing to do.
constexpr int kMaxExtentClasses = 4;
struct ExtentClass {
    int64_t begin;     // first position
    int64_t count;     // items
    int64_t max_used;  // largest size among them (elements)
    int64_t sum_used;  // and the sum of their sizes
};
// A class that would save fewer idle workgroups than it is worth joins the next larger one.  Counted in spans of 1024 elements,
// four workgroups of the update or half a copy's:
//
// For a launch, or a page list, of its own.  From and to tensors, us a call with the line at 2048 / 4096 / 16384 / 65536
// spans: 4.8 M elements in 64 K pages with clipping 41 / 33 / 33 / 33, in 256 K pages 30 / 30 / 28 / 28, in 1 M pages
// 32 / 32 / 32 / 53; 124 M 537 / 537 / 538 / 544; 350 M 1520 / 1518 / 1529 / 1555.
constexpr int64_t kWorthLaunch = 16384;
// For its part of the pages' common grid; line at 64 / 2048 / 16384 spans: 124 M 524 / 525 / 529; 7 M in 64 K pages
// 28.5 / 28.5 / 27.4; 16 M in 1 M pages 22.6 / 21.0 / 23.2.
constexpr int64_t kWorthGrid = 2048;
// For its part of the segments' common grid, where a class costs nothing but its entry; line at 64 / 2048 / 16384 spans / one class:
// 124 M fp32 out of pages 151.7 / 151.7 / 156.3 / 239, 73 M into 256 K pages 91.9 / 92.9 / 101 / 121, 122 M bf16 flat views
// 81.5 / 81.5 / 83.2 / 88.7, 12 M out of 256 K pages 9.5 / 9.6 / 10.1 / 11.9.
constexpr int64_t kWorthSegs = 64;
// Sizes come as an array, and are counted once whatever is asked of them: a call's host time is spent here
// when its pages are many and small.
class ExtentGroups {
public:
    // E = the size that the class limits are fractions of; the sizes are read until the last call.
    ExtentGroups(int64_t n, int64_t E, const int32_t* size);
    // Returns the number of classes.  worth: spans that a class has to save (kWorthLaunch, kWorthGrid, kWorthSegs).
    int fold(int64_t worth, ExtentClass cls[kMaxExtentClasses]);
    // With the classes of the last fold:
    // out[pos] = index of the item at position pos (classes one after the other, the given order kept inside each);
    void order(int64_t* out) const;
    // whether that is 0, 1, 2, ...
    bool in_order() const;

private:
    int class_of(int64_t used) const { return (used <= limit_[0]) + (used <= limit_[1]) + (used <= limit_[2]); }
    int64_t n_;
    const int32_t* size_;
    int64_t limit_[kMaxExtentClasses - 1];
    int64_t cnt_[kMaxExtentClasses] = {}, mx_[kMaxExtentClasses] = {}, sum_[kMaxExtentClasses] = {};
    int into_[kMaxExtentClasses] = {};
    int64_t begin_[kMaxExtentClasses] = {};
    int n_cls_ = 0;
};

// In which classes, and in which order, the pages of a whole layout are launched: decided here, once, for every call over all of it.
struct LayoutOrder {
    // In one grid (kWorthGrid): list positions, whose pages `order` names.  plain: position k is page k, and there is no table of it.
    ExtentClass cls[kMaxExtentClasses];
    int n_cls;
    bool plain;
    // As a run (position k is page k, class after class) if `run`, in these classes: those that are worth a launch of their own
    // (kWorthLaunch) or, where they would not leave the pages in order, the ones above if they do.  The two do not nest: a class that
    // joins the next larger one at the higher line can make that one large enough to stay apart, in another order.  So that plain
    // implies run, and who has neither has an `order`.
    ExtentClass run_cls[kMaxExtentClasses];
    int run_n_cls;
    bool run;
};
LayoutOrder layout_order(int64_t n, int64_t E, const int32_t* used, int64_t* order);

// One dimension of a grid holds fewer than 2^32 work-items (the runtime refuses more): the workgroups of
// `threads` work-items that a one-dimensional launch can have.
constexpr int64_t max_workgroups(int threads) { return (((int64_t)1 << 32) - 1) / threads; }
// Pages that one such launch takes if a page is `per_page` workgroups; at least one (the largest page, 2^30
// elements, is under 2^23 of any kernel here).  limit > 0: at most that many workgroups.
int64_t pages_per_launch(int64_t per_page, int threads, int64_t limit = 0);

// All classes in one one-dimensional grid, the classes of small items first: a launch of its own for them
// costs 5 to 9 us, because it starts when the last workgroup of the one before has ended.
//
// w / per for w < 2^26 (more workgroups than a grid of 64 work-items each has) as a multiplication:
// mul = ceil(2^shift / per) with shift = 26 + ceil(log2 per) is off by less than 1 / per at any such w.
struct GridDiv {
    uint32_t per, mul, shift;
    APM_HOST_DEVICE uint32_t quotient(uint32_t w) const { return (uint32_t)(((uint64_t)w * mul) >> shift); }
};
GridDiv grid_div(int64_t per);  // 1 <= per <= 2^23
// Workgroups [0, large_at): the classes of small items, the smallest first, small[k] from workgroup `first` on, unused
// entries (the last ones) with first = large_at; from large_at on the largest class.  begin: first position of the class, counted
// from the largest class's.
struct GridClass {
    uint32_t first;
    int32_t begin;
    GridDiv div;
};
struct GridMap {
    uint32_t large_at;
    GridDiv large;
    GridClass small[kMaxExtentClasses - 1];
};
// Workgroup w's item (a position, counted from the largest class's first) and its number within the item.
// What the largest class needs are single kernel arguments: the leading ones arrive in registers.
APM_HOST_DEVICE void grid_item(uint32_t large_at, GridDiv d, const GridClass* small, uint32_t w, int* item, uint32_t* x) {
    int begin = 0;
    uint32_t first = large_at;
    if (w < large_at) {
        const int c = (w >= small[1].first) + (w >= small[2].first);
        d = small[c].div;
        begin = small[c].begin;
        first = small[c].first;
    }
    w -= first;
    const uint32_t q = d.quotient(w);
    *item = begin + (int)q;
    *x = w - q * d.per;
}
// Calls launch(map, workgroups, first position of the largest class in it) for all classes at once, or, where
// that is more than one grid holds (or more than `limit` > 0), class by class in pieces that it holds; not at all where
// there are no items.  per(class): workgroups an item takes, >= 1.  Returns the first non-zero result.
template <class Per, class Launch>
int for_each_grid(const ExtentClass* cls, int n_cls, int threads, int64_t limit, Per&& per, Launch&& launch) {
    int64_t total = 0;
    const int64_t cap = limit > 0 ? limit : max_workgroups(threads);
    for (int c = 0; c < n_cls; ++c) total += cls[c].count * per(cls[c]);
    if (total == 0) return 0;
    if (total <= cap) {
        GridMap m{};
        int64_t at = 0;
        for (int c = n_cls - 1; c >= 1; --c) {
            m.small[n_cls - 1 - c] = GridClass{(uint32_t)at, (int32_t)(cls[c].begin - cls[0].begin), grid_div(per(cls[c]))};
            at += cls[c].count * per(cls[c]);
        }
        m.large_at = (uint32_t)at;
        m.large = grid_div(per(cls[0]));
        for (int k = n_cls - 1; k < kMaxExtentClasses - 1; ++k) m.small[k] = GridClass{m.large_at, 0, GridDiv{1, 0, 0}};
        return launch(m, total, cls[0].begin);
    }
    for (int c = 0; c < n_cls; ++c) {
        GridMap m{};
        m.large = grid_div(per(cls[c]));
        const int64_t piece = pages_per_launch(m.large.per, threads, limit);
        for (int64_t off = 0; off < cls[c].count; off += piece) {
            const int64_t n = cls[c].count - off < piece ? cls[c].count - off : piece;
            const int rc = launch(m, n * m.large.per, cls[c].begin + off);
            if (rc != 0) return rc;
        }
    }
    return 0;
}

// Words of 8 bytes that a launch carries in its kernel arguments: 3.4 KB, which leaves room for the
// rest under the 4 KB that argument blocks may have.
constexpr int kArgWords = 440;

// ---- pinned staging ring: small host arrays (page lists, copy descriptors) to the device ----
struct StageRing {
    static constexpr int K = 8;
    void* h[K] = {};
    void* d[K] = {};
    size_t cap[K] = {};
    hipEvent_t ev[K] = {};
    bool busy[K] = {};
    int next = 0;
    // Returns a slot whose previous use has completed, with at least `bytes` capacity.
    int acquire(size_t bytes, int* slot);
    // Copies the first `bytes` of the slot's host buffer to its device buffer on `s`.
    int commit(int slot, size_t bytes, hipStream_t s);
    // To be called after the kernels that read the slot's device buffer have been enqueued on `s`:
    // the slot is not handed out again before they have run (commit alone only covers the copy).
    int seal(int slot, hipStream_t s);
    void destroy();
};

// ---- kernels ------------------------------------------------------------------------------
constexpr int kReduceTile = 16384;  // gradient elements per workgroup of the reduce kernel

// The tenants of a page as the layout has them: tenant k is n[k] elements of tensor tensor[k] from
// tensor_off[k] on; the first starts at page element 0, the second at off1 (a multiple of 8).  The table depends on the layout alone and is uploaded
// with it; a fused call only brings the tensors' addresses.
struct TenantRec {
    int64_t tensor_off[2];
    int32_t off1;
    int32_t n[2];
    int32_t tensor[2];  // -1: no such tenant
};

// What the update kernel needs to know of one listed page, in one record that a workgroup fetches with
// a single scalar load: every workgroup is one wavefront with a few KB of work, so what it does
// before its first vector load counts.
//
// Pages first, first + 1, ... read from and written to the page classes (a run) need this much; where
// the page lies follows from the position.
struct PageRun {
    int32_t used;   // used extent of the page (elements)
    float scale;    // clip scale; negative = the page is skipped
};
// Any other page, and pages whose gradient / bf16 parameters are the caller's tensors.  Element e of
// the page has its gradient at g[k] + e and its bf16 parameter at q[k] + e, where k = 1 from the
// second tenant's first element off1 on; tenant k ends before element end[k].  A page class is one
// tenant over the used extent rounded up to 8.
struct __attribute__((aligned(64))) PageRec {
    int32_t used;
    float scale;
    int64_t pofs;   // the page's first element in the fp32 classes
    const uint16_t* g[2];
    uint16_t* q[2];
    int32_t off1;   // INT32_MAX: no second tenant
    int32_t end[2];
    int32_t pad;
};

// A page in use as the layout has it, in launch order (apm_pool::d_places): element e of the page is element e + shift[k] of tensor
// tensor[k], where k = 1 from off1 on, and tenant k ends before page element end[k] (0, and some tensor: no such tenant).
struct __attribute__((aligned(64))) PagePlace {
    int64_t shift[2];
    int64_t pofs;  // the page's first element in the classes
    int32_t used;
    int32_t page;
    int32_t off1;
    int32_t end[2];
    int32_t tensor[2];
    int32_t pad[3];
};
// A call whose words fit the arguments of its one launch needs no stage kernel before it: the wavefronts make the records they need
// from the layout's table and the words.  What one wavefront of the clipped update hands to another (a tile's sum, a page's scale) then
// carries the call's number, so nothing needs marking either.
constexpr int kTagLine = 8;  // words of a cache line: pages share none, they are polled from all over the chip
APM_HOST_DEVICE int tag_sums(int S) { return kTagLine * S; }  // a tile is summed up in four parts
struct CallTables {
    const PagePlace* places;
    uint64_t g_base, q_base;  // the tensors' addresses are multiples of 16 from there; or the page class, if it is not the caller's tensors
    uint64_t* sums;           // [n_listed * tag_sums(S)] per tile: upper and lower half of each part's sum above the call's number
    uint64_t* scales;         // [n_listed * kTagLine] a page's scale above the call's number
    uint32_t number;          // never 0, which is what the words hold at first
    int32_t g_at, q_at;       // words of the tensors' addresses
    int32_t listed;           // words 2 i, 2 i + 1: place in the table and output index of list position i; else the position itself and its page
    int32_t first;            // list position of the launch's first page
    int32_t pad;
};
constexpr int kCallWords = 2 * kArgWords;
// Up to how many elements: where a call is large, a longer way to a wavefront's first load costs as much as the stage kernel did (us a
// call, with a stage / prepare kernel / without; no norms, from and to tensors, and a reversed list: 0.6 M 9.3 / 6.3, 8 M - and 41.7 / 38.5, 10 M 49.7 /
// 47.9 and 52.0 / 50.7, 22 M 97.9 / 95.9 and 101.1 / 99.6, 49 M 212 / 211 and 213 / 211, 67 M 299 / 298 and 292 / 289, 124 M 528 / 531 and - ; with norms:
// 0.6 M 13.3 / 9.4, 2.5 M 26.8 / 20.6, 4.9 M 32.3 / 28.0 and 31.4 / 27.5, 18 M 90.6 / 84.9 and 90.1 / 86.4, 25 M 122 / 120 and 132 / 132, 31 M 150 / 149 and
// 147.5 / 145.2, 39 M 180 / 185 and 180 / 180, 49 M 226 / 232 and 222 / 223).
constexpr int64_t kCallElems = (int64_t)64 << 20, kCallSumElems = (int64_t)32 << 20;
// Elements a page from which norms, scales and update go in one grid, and pages up to which they do whatever they hold (one_pass_pays).
constexpr int64_t kOnePassElems = 4096, kOnePassPages = 2048;
// Pages up to which that grid hands results on under the call's number: it has three wavefronts more a page, and a page two cache lines more that are
// polled.  us a call with a stage / prepare kernel / without, from and to tensors, and consecutive pages: 1000 of 4096 elements 26.2 / 22.7 and 27.2 / 23.5,
// 1984 of 16 K 149.7 / 147.1 and 146.7 / 142.3, 2000 of 4096 46.7 / 44.2 and 46.2 / 46.7, 2560 of 8192 99.3 / 98.1 and 100.0 / 100.7, 3072 of 4096 67.1 / 67.0 and
// 68.2 / 69.7, 3584 of 8192 138.8 / 144.4 and 135.5 / 138.4, 4096 of 4096 85.4 / 86.7 and 87.7 / 90.6, 7168 147.7 / 164.0 and 144.5 / 155.5.
constexpr int64_t kTaggedPages = 2048;
// The passes of a step that skips (or of norms of many small pages), whose finalize pass then writes the records: with a stage kernel / without, 4.5 M
// elements 20.9 / 17.8 us, 52 M 55.1 / 51.7, 153 M 134.4 / 130.5, 382 M 295 / 291 and with clipping 312 / 313, 541 M 469 / 468, 1.08 G 915 / 919.
constexpr int64_t kCallPassElems = (int64_t)512 << 20;
struct CallWords {
    CallTables t;
    uint32_t word[kCallWords];
};

// Wavefronts of the update kernel when it reads and writes fp32 classes in host memory across
// PCIe (the streamer's direct mode, the file tier's window); see apm_stream.hip for the sweep.
constexpr int kDirectWavefronts = 48;
// The staged form of it: what a wavefront has in one slot of a class.
constexpr int kLinkSlotBytes = 4096;

// Where the pages that a launch does not skip are noted: a count per extent class, then their positions,
// those of a class from its first position on.  Part of a pool's array belongs to every page
// (kLiveInts(1)), so that launches over disjoint pages can run side by side.
constexpr int64_t kLiveInts(int64_t n_listed) { return (kMaxExtentClasses + 1) * n_listed; }

struct AdamwLaunch {
    float* p32;
    float* m32;
    float* v32;
    const uint16_t* g16;
    uint16_t* p16;
    const int32_t* used;          // device, indexed by grad page id
    PageRec* recs;                // device scratch, [n_listed], filled by the stage / reduce / prepare
                                  // pass; as PageRun [n_listed] if the pages are a run (see is_run)
    bool gather;                  // read g from the tenant tensors instead of g16
    bool scatter;                 // write p16 to the tenant tensors instead of p16
    const int64_t* state_pages;   // device list or nullptr (then state_first + i)
    const int64_t* grad_pages;    // device list or nullptr (then grad_first + i)
    int64_t state_first;
    int64_t grad_first;
    int64_t n_listed;
    ExtentClass cls[kMaxExtentClasses];  // n_cls == 0: one class, all positions, extent E
    int n_cls;
    const int32_t* out_index;     // device: list position -> index into grad_norm / skip_mask;
                                  // nullptr = the position itself
    int64_t E;
    double* partials;             // [n_listed][S] per-slice sums of squares; nullptr = no reduce pass
    uint32_t* nzflags;            // [n_listed][S] per-slice OR of magnitude bits
    int32_t S;                    // slices per page = ceil(E / kReduceTile)
    float* grad_norm;             // device, nullable
    uint8_t* skip_mask;           // device, nullable
    float b1, omb1, b2, omb2, inv_sqrt_bc2, eps, step_size, lr_wd;
    double max_norm;
    int32_t skip_mode;
    int32_t stride_wavefronts;    // > 0: the update runs as that many wavefronts striding over all
                                  // page slices (fp32 classes in host memory); 0: one per slice
    int32_t stride_waves_per_wg;  // how many of them share a workgroup, 1..16
    float* link_slots[3];         // stride form: per class two staging slots of kLinkSlotBytes per wavefront; nullptr: none
    bool link_update;             // with slots: else the pages come and go as they are
    bool beside_link;             // g16 / p16 in the page classes, while a kernel on another stream moves pages across PCIe
    bool host_write_through;      // stride form: fp32 state stores written through at system scope
    bool wide;                    // a run whose grid holds many workgroups without work: fewer, larger slices
    bool bare_run;                // a run without a reduce or prepare pass: the update reads `used` itself
    int32_t* live;                // scratch of a launch that may skip pages, kLiveInts(n_listed) entries
    bool sums_ready;              // partials / nzflags hold the sums already, indexed by page
    bool one_pass;                // launch_clip_update follows: the stage / prepare pass marks every scale and
                                  // every sum in `partials` as not there yet
    int32_t wait_limit;           // polls after which a wavefront of it computes what it waits for by itself
    int64_t max_workgroups;       // of a one-dimensional launch; 0: what the hardware takes
    const CallWords* call;        // nullptr: recs (and sums) are written by a stage / prepare pass
    bool is_run() const { return !state_pages && !grad_pages && !gather && !scatter; }
};

// Reduce pass (fills the records with clip scale / skip); or, when no reduce pass is needed, the
// prepare pass (fills them with scale 1).  One of the two must precede launch_adamw on the same stream.
hipError_t launch_grad_reduce(const AdamwLaunch& a, hipStream_t s);
hipError_t launch_prepare(const AdamwLaunch& a, hipStream_t s);

// What a call brings to the device besides scalars: its page list (a word per position: page, and the
// index of its outputs in the upper half) and its tensors' addresses.  Written to where the step's
// kernels read it (list / out / L.recs, with scale 1) by apm_stage_kernel.
struct StageCall {
    const uint64_t* list;         // n_listed words, or nullptr: as `runs`, or as L.grad_pages / L.grad_first say
    const uint64_t* g_ptrs;       // n_tensors addresses each, nullptr if not gathered / scattered
    const uint64_t* q_ptrs;
    int64_t n_tensors;
    const TenantRec* tenants;
    int64_t* d_list;              // written if `list` or `runs`
    int32_t* d_out;
    const uint64_t* d_words;      // list, g_ptrs, q_ptrs one after the other in device memory, or nullptr
    // Carried in kernel arguments, the words are halved if every address lies less than 64 GiB beyond its list's
    // base, as they do but for lists that several allocations far apart make up.
    bool narrow;
    uint64_t g_base, q_base;      // multiples of 16, as all addresses are
    // The list as runs in place of `list`, or nullptr; the addresses then as half words.
    const struct StageRun* runs;
    int64_t n_runs;
};
// List positions at, at + 1, ... up to the next run's: pages one after the other, downwards if the upper bit of `page` is set, output indices
// out, out + 1, ...
struct StageRun {
    uint32_t at, page, out;
};
constexpr int64_t run_words(int64_t n_runs) { return n_runs * (int64_t)(sizeof(StageRun) / sizeof(uint32_t)); }
constexpr int64_t kStageRuns = 2 * kArgWords * sizeof(uint32_t) / sizeof(StageRun);  // that a launch carries
int64_t stage_launches_runs(int64_t n_runs, int64_t lists, int64_t n_tensors);  // as stage_launches
// Launches it takes to carry a call's words in kernel arguments (StageCall::d_words == nullptr): n_list list
// words and `lists` (0..2) lists of n_tensors addresses.  narrow: as 32-bit words, two per list word.
int64_t stage_launches(int64_t n_list, int64_t lists, int64_t n_tensors, bool narrow);
hipError_t launch_stage(const AdamwLaunch& L, const StageCall& c, hipStream_t s);
hipError_t launch_adamw(const AdamwLaunch& a, hipStream_t s);
// Norms, clip scales and update in one kernel, after the stage / prepare pass of a launch with
// one_pass set; for skip_mode NONE and fp32 classes in device memory.
hipError_t launch_clip_update(const AdamwLaunch& a, hipStream_t s);
// Whether that is the better form; staged: a stage kernel writes the launch's records.
bool one_pass_pays(const AdamwLaunch& a, bool staged);
constexpr int32_t kWaitLimit = 4096;
// Takes a gradient in page layout over into a buffered half: dst <- src, or (accumulate) dst <- dst + src, over
// the used extents of the listed pages, and if `sums` is set works out the tiles' sums of squares and
// non-zero flags of what it wrote, as the reduce pass would, indexed by page.
constexpr int64_t kTakePages = 2 * kArgWords;
struct GradTake {
    const uint16_t* src;
    uint16_t* dst;
    bool accumulate;
    const int32_t* used;
    int64_t E;
    int32_t S;
    double* sums;       // [pool pages * S] or nullptr
    uint32_t* nzflags;
    // The pages: the device list `order` in the given classes, or host_pages, which are carried in the kernel
    // arguments, kTakePages a launch, or neither: pages first, first + 1, ...
    const int64_t* order;
    const int64_t* host_pages;
    int64_t first;
    const ExtentClass* cls;
    int n_cls;
    int64_t max_workgroups;  // see AdamwLaunch
};
hipError_t launch_grad_take(const GradTake& t, hipStream_t s);

// One segment of the layout as the copy kernel reads it: n elements from `tensor_off` of tensor
// `tensor`, in the class region from element `page_elem`.  The table depends on the layout alone and
// is uploaded with it; a call only brings the tensors' addresses.
struct __attribute__((aligned(32))) SegRec {  // one scalar load
    int64_t tensor_off;
    int64_t page_elem;
    int32_t tensor;
    int32_t n;
    int64_t pad;
};
// Segments of the table in classes of their lengths, all of tensors [tensor_begin, tensor_begin + kArgWords).
struct SegLaunch {
    ExtentClass cls[kMaxExtentClasses];
    int n_cls;
    int32_t tensor_begin, tensor_count;
};
// Pack (to_pages) or unpack over the given launches.  ptrs = the tensors' addresses: in host memory
// (carried in the kernel arguments), or on_device: in device memory.
struct SegCopy {
    const SegRec* segs;
    char* region;
    int32_t elem_bytes;
    bool to_pages;
    const uint64_t* ptrs;
    bool on_device;
    bool aligned;  // every tensor starts on a multiple of 16 bytes
    int64_t max_workgroups;  // see AdamwLaunch
};
hipError_t launch_seg_copy(const SegCopy& c, const SegLaunch* launches, int64_t n_launches, hipStream_t s);

// One kernel that moves an incoming batch (3 fp32 classes, in_bytes each, host -> staging) and an
// outgoing batch (out_bytes each, staging -> host) at once; either byte count may be 0.  All
// addresses are device-side addresses, 16-byte aligned; byte counts are multiples of 16.
struct DuplexCopy {
    const char* in_src[3];
    char* in_dst[3];
    const char* out_src[3];
    char* out_dst[3];
    int64_t in_bytes, out_bytes;
    // Optional: move only the used extent of each page.  used = the device page table (elements per
    // page), *_first_page = the table index of each batch's first page, page_bytes = E * 4.
    const int32_t* used;
    int64_t in_first_page, out_first_page, page_bytes;
    uint32_t items_per_page;  // filled in by launch_duplex_copy
    int host_store_policy;    // stores to the host pages: 0 non-temporal, 3 written through at system scope
};
hipError_t launch_duplex_copy(const DuplexCopy& d, int wavefronts, int per_wg, hipStream_t s);

// Fills the scalar fields of `a` from the hyper-parameters (all derived in double, rounded once).
int prepare_hyper(const apm_hyper* h, int64_t step, AdamwLaunch* a);

}  // namespace apm

struct apm_pool {
    apm_pool_desc desc{};
    void* base[APM_N_STATES] = {};
    void* alloc[APM_N_STATES] = {};  // what the library allocated for the class (base = alloc + skew)
    bool owned[APM_N_STATES] = {};

    bool has_layout = false;
    std::vector<int64_t> layout_numels;
    std::vector<int64_t> layout_ids;
    apm::Plan plan;
    std::vector<int32_t> used;  // used extent of every page of the pool (0 beyond the layout); empty before a layout
    std::vector<int64_t> used_sum;  // used_sum[k]: of pages [0, k) in use

    int fd[APM_N_STATES] = {-1, -1, -1, -1, -1};  // FILE pools: one file per stored class

    int32_t* d_used = nullptr;      // device page table: used extent per page
    char* d_tables = nullptr;       // the layout's tables below, in one allocation
    apm::SegRec* d_segs = nullptr;  // the layout's segments, ordered as seg_launches lists them
    std::vector<apm::SegLaunch> seg_launches;
    int32_t seg_ranges = 0;         // groups of kArgWords tensors they are split into
    apm::TenantRec* d_tenants = nullptr;  // by page in use
    apm::PagePlace* d_places = nullptr;   // pages in use in launch order; nullptr: more than kMaxPlaces
    std::vector<int32_t> place_of;        // by page in use: its index there
    // All pages in use.  The launch order of whole.cls, and the same as 32-bit output indices; nullptr if whole.plain.
    apm::LayoutOrder whole{};
    int64_t* d_order = nullptr;
    int32_t* d_order_out = nullptr;
    int64_t layout_epoch = 0;  // counts the layouts installed
    char* d_scratch = nullptr;      // the five below, allocated on first use
    double* d_partials = nullptr;   // reduce scratch, n_pages * S
    uint32_t* d_nzflags = nullptr;
    apm::PageRec* d_recs = nullptr;   // n_pages entries
    uint64_t* d_tagged = nullptr;     // CallTables: scales, then sums, of up to kTaggedPages each; d_tagged_own if it is not part of the
    uint64_t* d_tagged_own = nullptr; // scratch, which the first call that hands results on then allocates
    uint32_t call_number = 0;         // of the last call that used it
    int32_t* d_live = nullptr;        // kLiveInts(n_pages) entries
    // what a call's list comes to (apm_stage_kernel), n_pages entries each, allocated on first use; like the scratch above they belong to the one step that is running on the pool
    int64_t* d_list = nullptr;
    int32_t* d_list_out = nullptr;
    int32_t S = 0;
    apm::StageRing ring;
    int64_t max_workgroups = 0;  // see AdamwLaunch; set by tests only, as
    int32_t wait_limit = apm::kWaitLimit;

    // one-step-stale update state
    hipStream_t upd_stream = nullptr;
    bool upd_overlaps = false;  // measured: its kernels run beside the producer stream's
    uint16_t* gbuf[2] = {nullptr, nullptr};
    hipEvent_t ev_staged[2] = {};
    hipEvent_t ev_applied[2] = {};
    bool applied_valid[2] = {false, false};
    hipEvent_t ev_flush = nullptr;
    // Sums of squares and non-zero flags of what each half holds, worked out while it was taken over
    // (n_pages * S entries, allocated when first wanted); gsum_ok: complete for the half's contents
    // under the layout of gsum_epoch.
    double* gsum[2] = {nullptr, nullptr};
    uint32_t* gnz[2] = {nullptr, nullptr};
    bool gsum_ok[2] = {false, false};
    int64_t gsum_epoch[2] = {0, 0};
    int cur = 0;
    bool buffered = false;
    int64_t applied = 0;
    // What the buffered gradient was handed over with: it is applied, one call later, with the
    // hyper-parameters and the page list of the call that brought it.
    apm_hyper buf_hyper{};
    std::vector<int64_t> buf_pages;  // copy of the caller's list (unused if buf_pages_null)
    bool buf_pages_null = true;      // the call listed pages [0, buf_n_pages)
    int64_t buf_n_pages = 0;
    // Its half holds the used extents of the layout it was handed over under (buf_by_extent; else whole
    // pages).  buf_extents: those extents, kept by the first layout that replaces that one; empty until then.
    bool buf_by_extent = false;
    std::vector<int32_t> buf_extents;
    float* delayed_norm = nullptr;
    uint8_t* delayed_skip = nullptr;

    // kernel timing (measurement aid)
    bool timing = false;
    struct TimedLaunch { int cls; hipEvent_t begin, end; };
    std::vector<TimedLaunch> timed;

    bool stores(int s) const { return s >= 0 && s < APM_N_STATES && (desc.state_mask >> s) & 1u; }
};

namespace apm {
// Validates a page list and enqueues the kernels of one step: what brings the call's list and addresses to
// the device, the passes over the gradient, and the update, or the last two in one grid.  g16_override != nullptr
// replaces the pool's G16 region as the gradient source; page_sums / page_nzflags: its tiles' sums
// and flags, indexed by page, if they are known.
int enqueue_step(apm_pool* pool, const int64_t* pages, int64_t n_pages, int64_t step,
                 const apm_hyper* hyper, const uint16_t* g16_override, float* grad_norm,
                 uint8_t* skip_mask, hipStream_t stream, const apm_tensor* grad_tensors = nullptr,
                 const apm_tensor* p16_tensors = nullptr, int64_t n_tensors = 0,
                 double* page_sums = nullptr, uint32_t* page_nzflags = nullptr);
int ensure_scratch(apm_pool* pool, bool list = false);
// Whether work enqueued on the stream now is captured, as far as that can be told.
bool is_captured(hipStream_t s);
// The number of the next call, on stream s, and where it hands results on (kTaggedPages); false if there is no memory for that.
bool next_call(apm_pool* pool, hipStream_t s, CallTables* out);
// Pages in use beyond which a call's words do not fit its arguments, or a launch more costs it little.
constexpr int64_t kMaxPlaces = 16384;
// Pages [first, first + n) as one class, each launched with the grid of the layout's largest page.
ExtentClass run_class(const apm_pool* pool, int64_t first, int64_t n);
bool wide_pays(const ExtentClass& c);  // AdamwLaunch::wide for it
// Allocates the ping-pong gradient halves, the events and the update stream of the delayed path.
// caller != nullptr-able: the stream the producer works on; the update stream is chosen so that
// its kernels run beside that stream's (see make_overlapping_stream).
int ensure_delayed(apm_pool* pool, hipStream_t caller, bool probe);

// Whether kernels on two streams of one process run at the same time is not something the API
// states: the runtime maps streams onto a few hardware queues, and work of two streams that share
// a queue runs in order.  These helpers measure it with two short spin kernels (a few hundred
// microseconds each; both streams are synchronised first).
int streams_overlap(hipStream_t a, hipStream_t b, bool* out);
// A new non-blocking stream whose kernels overlap with those of `with` (and of `*also`, if given);
// tries a few candidates and keeps the last one (*overlaps = false) if none does.
int make_overlapping_stream(hipStream_t with, hipStream_t* out, bool* overlaps, const hipStream_t* also = nullptr);
// FILE <-> HOST page copy (synchronous).
int file_page_copy(apm_pool* dst, int64_t dst_page, apm_pool* src, int64_t src_page, int64_t n_pages,
                   int state, hipStream_t stream);

// The one-step-stale hand-over shared by apm_step_delayed and the streamer's delayed step:
// applies the buffered gradient through `apply` (which enqueues one update reading the gradient
// half it is given, with the step number, page list and hyper-parameters it is given -- those of
// the call that handed that gradient over -- on the pool's update stream), then stages new_g16
// into the other half on `caller` together with this call's page list and hyper-parameters
// (nullptr = flush).
using DelayedApply = std::function<int(const uint16_t* g16, int64_t step, hipStream_t upd_stream,
                                       const int64_t* pages, int64_t n_pages, const apm_hyper* hyper)>;
// want_sums: the hand-over also leaves the sums of what it staged in gsum / gnz.
int delayed_call(apm_pool* pool, const int64_t* pages, int64_t n_pages, const void* new_g16,
                 const apm_hyper* hyper, hipStream_t caller, const DelayedApply& apply, bool want_sums = false);

// Brackets one kernel launch with events when the pool's timing is on.
struct ScopedTiming {
    apm_pool* pool;
    hipStream_t stream;
    hipEvent_t end = nullptr;
    ScopedTiming(apm_pool* p, int cls, hipStream_t s) : pool(p), stream(s) {
        if (!p->timing) return;
        hipEvent_t b = nullptr;
        if (hipEventCreate(&b) != hipSuccess || hipEventCreate(&end) != hipSuccess) { end = nullptr; return; }
        (void)hipEventRecord(b, s);
        p->timed.push_back({cls, b, end});
    }
    ~ScopedTiming() { if (end) (void)hipEventRecord(end, stream); }
};
}  // namespace apm

// For tests, not part of the C ABI: caps the workgroups of the pool's one-dimensional launches (0: no cap), so that
// small pools exercise what otherwise takes tens of millions of pages.
extern "C" int apm_test_set_max_workgroups(apm_pool* pool, int64_t max_workgroups);
// The same for AdamwLaunch::wait_limit (0: wavefronts that would wait for another one's result never do).
extern "C" int apm_test_set_wait_limit(apm_pool* pool, int32_t wait_limit);
// The number of the pool's last call that handed results on under one (0: the next one clears them).
extern "C" int apm_test_set_call_number(apm_pool* pool, uint32_t number);
