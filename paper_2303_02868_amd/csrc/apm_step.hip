// Host side of the update: scalar preparation, page-list handling, the synchronous step and the
// one-step-stale (delayed) step.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>

#include "apm_internal.h"

namespace apm {

int prepare_hyper(const apm_hyper* h, int64_t step, AdamwLaunch* a) {
    if (!h) return fail(APM_EINVAL, "NULL hyper");
    if (step < 1) return fail(APM_EINVAL, "step must be >= 1 (got %lld): bias correction divides by 1 - beta^step", (long long)step);
    if (!(h->beta1 >= 0.0 && h->beta1 < 1.0) || !(h->beta2 >= 0.0 && h->beta2 < 1.0)) return fail(APM_EINVAL, "betas must lie in [0, 1)");
    if (!(h->eps >= 0.0) || !std::isfinite(h->lr) || !std::isfinite(h->weight_decay) || std::isnan(h->max_grad_norm)) return fail(APM_EINVAL, "bad hyper-parameter");
    if (h->skip_mode != APM_SKIP_NONE && h->skip_mode != APM_SKIP_UNTOUCHED) return fail(APM_EINVAL, "unknown skip_mode %d", h->skip_mode);
    // Every scalar is formed in double and rounded to fp32 exactly once: 1 - 0.999f evaluated in
    // fp32 would already be off by 1e-5 relative.
    const double bc1 = 1.0 - std::pow(h->beta1, (double)step);
    const double bc2 = 1.0 - std::pow(h->beta2, (double)step);
    a->b1 = (float)h->beta1;
    a->omb1 = (float)(1.0 - h->beta1);
    a->b2 = (float)h->beta2;
    a->omb2 = (float)(1.0 - h->beta2);
    a->inv_sqrt_bc2 = (float)(1.0 / std::sqrt(bc2));
    a->eps = (float)h->eps;
    a->step_size = (float)(h->lr / bc1);
    a->lr_wd = (float)(h->lr * h->weight_decay);
    a->max_norm = h->max_grad_norm > 0.0 ? h->max_grad_norm : 0.0;
    a->skip_mode = h->skip_mode;
    return APM_OK;
}

namespace {
// Checks a bf16 tensor list against the installed layout for the gather / scatter kernels.
int check_fused_list(const apm_pool* pool, const apm_tensor* t, int64_t n, const char* what) {
    if (!pool->has_layout || (int64_t)pool->layout_numels.size() != n) return fail(APM_ESTATE, "%s list does not match the pool's installed layout", what);
    for (int64_t i = 0; i < n; ++i) {
        if (t[i].numel != pool->layout_numels[(size_t)i]) return fail(APM_ESTATE, "%s list does not match the pool's installed layout", what);
        if (t[i].numel == 0) continue;
        if (t[i].dtype != APM_BF16) return fail(APM_EINVAL, "%s tensor %lld is not bf16", what, (long long)i);
        if (!t[i].data || (reinterpret_cast<uintptr_t>(t[i].data) & 15u)) return fail(APM_EINVAL, "%s tensor %lld: data must be a 16-byte aligned device pointer", what, (long long)i);
    }
    return APM_OK;
}

// The used extents of a call's pages; `room` holds them where the pool has no array of them.
const int32_t* page_extents(const apm_pool* pool, const int64_t* pages, int64_t n, std::vector<int32_t>* room) {
    if (pool->used.empty()) room->assign((size_t)n, 0);
    else if (pages) room->resize((size_t)n);
    for (int64_t k = 0; pages && !pool->used.empty() && k < n; ++k) (*room)[(size_t)k] = pool->used[(size_t)pages[k]];
    return room->empty() ? pool->used.data() : room->data();
}

bool consecutive(const int64_t* pages, int64_t n) {
    for (int64_t k = 1; pages && k < n; ++k)
        if (pages[k] != pages[0] + k) return false;
    return true;
}

}  // namespace

// A workgroup that finds nothing to do costs 0.2 ns, hidden behind the others' work if they are not too many in a row.
// Slices of four vectors per lane are a quarter as many, but move a few percent less (us a call, 64 full pages
// and as many nearly empty ones as stated, with norms, one vector in one grid / four as passes; in brackets
// without norms; 1 M elements a page, none 298 / 318 (289 / 292), 150 % 329 / 331 (303 / 300), 400 % 440 / 332
// (395 / 298); 128 K elements a page, 400 % 57 / 57 (43 / 43), 1000 % 91 / 66 (79 / 49)).  Skipping: 1000 nearly empty
// and 4 full pages of 1 M elements 336 / 148, 10 000 and 100 of 16 K 111 / 74.
bool wide_pays(const ExtentClass& c) {
    const int64_t idle = c.count * c.max_used - c.sum_used;
    return c.max_used >= 4096 && (c.max_used >= (int64_t)1 << 19 ? 2 * idle > 3 * c.sum_used : idle > 4 * c.sum_used);
}

// (30 000 tensors of 300 elements in pages of 8192 without a list: 622 us a call with a full page's grid each, 125
// with the largest page's; skipping 577 and 132.)
ExtentClass run_class(const apm_pool* pool, int64_t first, int64_t n) {
    const int64_t in_use = (int64_t)pool->used_sum.size() - 1;
    auto upto = [&](int64_t k) { return in_use < 0 ? (int64_t)0 : pool->used_sum[(size_t)(k < in_use ? k : in_use)]; };
    return ExtentClass{0, n, pool->whole.n_cls > 0 ? pool->whole.cls[0].max_used : 0, upto(first + n) - upto(first)};
}

namespace {
// Launches that may carry a call's page list and tensor addresses in their arguments; beyond that
// they are staged through the pinned ring.  The ring costs the GPU an upload and two event packets,
// 20 us and more between one call's update and the next one's; a stage launch costs 3 us.
constexpr int64_t kMaxStageLaunches = 4;
}  // namespace

// The base from which a list's addresses are multiples of 16 that fit half words, if there is one.
static bool base_of(const apm_tensor* t, int64_t n, uint64_t* base) {
    uint64_t low = UINT64_MAX, high = 0;
    for (int64_t i = 0; i < n; ++i) {
        if (t[i].numel == 0) continue;
        const uint64_t at = reinterpret_cast<uint64_t>(t[i].data);
        if (at < low) low = at;
        if (at > high) high = at;
    }
    *base = low <= high ? low : 0;
    return low > high || (high - low) >> 4 <= UINT32_MAX;
}

// A list in launch order as runs; their number, or -1 if there are more than `most`.  A run's pages are compared with where its first two lead, not
// each with the one before: 100 000 pages last to first 62 us in place of 180 (a word a page: 67).
static int64_t runs_of(const int64_t* pages, const std::vector<int64_t>& order, int64_t most, StageRun* out) {
    auto page_at = [&](int64_t i) { return pages ? pages[i] : i; };
    const int64_t n = (int64_t)order.size(), *o = order.data();
    int64_t n_runs = 0;
    for (int64_t k = 0, end; k < n; k = end) {
        if (n_runs == most) return -1;
        const int64_t at = o[k], page = page_at(at);
        const int64_t step = k + 1 < n && o[k + 1] == at + 1 ? page_at(at + 1) - page : 0;
        end = k + 1;
        if (step == 1 || step == -1)
            for (++end; end < n && o[end] - end == at - k && page_at(at + (end - k)) - page == step * (end - k); ++end) {}
        out[n_runs++] = StageRun{(uint32_t)k, (uint32_t)page | (step == -1 ? 0x80000000u : 0u), (uint32_t)at};
    }
    return n_runs;
}

bool is_captured(hipStream_t s) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &capture) == hipSuccess) return capture != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// The words of a call: the list (in launch order) and the addresses.  False if they do not go into half words or a page is not the
// layout's.
static bool fill_call(const apm_pool* pool, const int64_t* pages, int64_t n_placed, const std::vector<int64_t>& order, const apm_tensor* g,
                      int64_t n_g, const apm_tensor* q, int64_t n_q, CallWords* call) {
    if (!base_of(g, n_g, &call->t.g_base) || !base_of(q, n_q, &call->t.q_base)) return false;
    uint32_t* w = call->word;
    for (int64_t k = 0; k < n_placed; ++k) {
        const int64_t at = order.empty() ? k : order[(size_t)k], page = pages ? pages[at] : at;
        if (page >= (int64_t)pool->place_of.size()) return false;
        *w++ = (uint32_t)pool->place_of[(size_t)page];
        *w++ = (uint32_t)at;
    }
    // an empty tensor's address may be anything: it is nobody's tenant
    call->t.g_at = (int32_t)(w - call->word);
    for (int64_t i = 0; i < n_g; ++i) *w++ = (uint32_t)((reinterpret_cast<uint64_t>(g[i].data) - call->t.g_base) >> 4);
    call->t.q_at = (int32_t)(w - call->word);
    for (int64_t i = 0; i < n_q; ++i) *w++ = (uint32_t)((reinterpret_cast<uint64_t>(q[i].data) - call->t.q_base) >> 4);
    call->t.places = pool->d_places;
    return true;
}

int enqueue_step(apm_pool* pool, const int64_t* pages, int64_t n_pages, int64_t step,
                 const apm_hyper* hyper, const uint16_t* g16_override, float* grad_norm,
                 uint8_t* skip_mask, hipStream_t stream, const apm_tensor* grad_tensors,
                 const apm_tensor* p16_tensors, int64_t n_tensors, double* page_sums, uint32_t* page_nzflags) {
    if (!pool) return fail(APM_EINVAL, "NULL pool");
    if (pool->desc.device != APM_DEV_GPU) return fail(APM_EDEVICE, "the update runs on GPU pools only");
    for (int st = 0; st < APM_N_STATES; ++st) {
        if (st == APM_G16 && (g16_override || grad_tensors)) continue;
        if (st == APM_P16 && p16_tensors) continue;
        if (!pool->stores(st)) return fail(APM_ESTATE, "pool does not store state class %d", st);
    }
    if (grad_tensors) {
        int rc0 = check_fused_list(pool, grad_tensors, n_tensors, "gradient");
        if (rc0 != APM_OK) return rc0;
    }
    if (p16_tensors) {
        int rc0 = check_fused_list(pool, p16_tensors, n_tensors, "bf16 parameter");
        if (rc0 != APM_OK) return rc0;
    }
    if (n_pages < 0 || n_pages > pool->desc.n_pages) return fail(APM_ERANGE, "page count %lld out of range", (long long)n_pages);
    AdamwLaunch L{};
    int rc = prepare_hyper(hyper, step, &L);
    if (rc != APM_OK) return rc;
    if (n_pages == 0) return APM_OK;
    APM_HIP(hipSetDevice(pool->desc.hip_device));

    // List positions are grouped into extent classes (largest extents first, the caller's order
    // kept inside a class).  order[pos] = the caller's index of the page launched at position pos.
    const int64_t E = pool->desc.page_elems;
    const int64_t in_use = pool->has_layout ? (int64_t)pool->plan.pages.size() : 0;
    auto page_at = [&](int64_t k) { return pages ? pages[k] : k; };
    if (pages) {
        // Two workgroups updating one page at once would race: a listed page is listed once.
        std::vector<uint8_t> seen((size_t)pool->desc.n_pages, 0);
        for (int64_t k = 0; k < n_pages; ++k) {
            if (pages[k] < 0 || pages[k] >= pool->desc.n_pages) return fail(APM_ERANGE, "pages[%lld] = %lld out of range [0, %lld)", (long long)k, (long long)pages[k], (long long)pool->desc.n_pages);
            if (seen[(size_t)pages[k]]) return fail(APM_EINVAL, "pages[%lld] = %lld is listed twice", (long long)k, (long long)pages[k]);
            seen[(size_t)pages[k]] = 1;
        }
    }
    if (grad_tensors || p16_tensors) {  // the tensors cover the pages of the layout and no others
        if (!pages && n_pages > in_use) return fail(APM_ERANGE, "page count %lld exceeds the %lld pages in use", (long long)n_pages, (long long)in_use);
        if (pages)
            for (int64_t k = 0; k < n_pages; ++k)
                if (pages[k] >= in_use) return fail(APM_ERANGE, "pages[%lld] = %lld is not in use by the layout", (long long)k, (long long)pages[k]);
    }
    // The whole layout in its own order is the common case: its launch order came with the layout.
    // An ascending run launched in the caller's order needs no indirection; on the page classes that is worth
    // more than the finer classes of a common grid.
    const bool whole = !pages && n_pages == in_use;
    const bool tensors = grad_tensors || p16_tensors;
    std::vector<int64_t> order;
    // (With norms in one launch that makes its own records finer classes are worth more: 4.9 M elements in 256 K pages with clipping, us a call,
    // as a run 34.1, in classes 27.9; 24 M 114.3 and 107.2.)
    const bool norms = (L.max_norm > 0.0 || grad_norm) && L.skip_mode == APM_SKIP_NONE && !page_sums;
    // A captured launch makes no records of its own: a replay would hand results on under the same number, and may come after a layout that
    // replaces the tables.
    const bool captured = is_captured(stream);
    bool run = whole && (tensors || (norms && !captured && pool->d_places && pool->used_sum.back() <= kCallSumElems) ? pool->whole.plain : pool->whole.run);
    if (whole) {
        const bool as_run = run && !tensors;
        L.n_cls = as_run ? pool->whole.run_n_cls : pool->whole.n_cls;
        for (int c = 0; c < L.n_cls; ++c) L.cls[c] = as_run ? pool->whole.run_cls[c] : pool->whole.cls[c];
    } else {
        std::vector<int32_t> room;
        ExtentGroups groups(n_pages, E, page_extents(pool, pages, n_pages, &room));
        if (consecutive(pages, n_pages)) {
            L.n_cls = groups.fold(tensors ? kWorthGrid : kWorthLaunch, L.cls);
            run = groups.in_order();
        }
        if (!run) {
            L.n_cls = groups.fold(kWorthGrid, L.cls);
            order.resize((size_t)n_pages);
            groups.order(order.data());
        }
    }
    const bool need_reduce = grad_norm || skip_mask || L.max_norm > 0.0 || L.skip_mode != APM_SKIP_NONE;
    rc = ensure_scratch(pool, !run && !whole);
    if (rc != APM_OK) return rc;

    // What the kernels need of this call's list and tensors, as words (see StageCall).
    StageCall sc{};
    const int64_t n_list = run || whole ? 0 : n_pages;
    const int64_t n_g = grad_tensors ? n_tensors : 0, n_q = p16_tensors ? n_tensors : 0;
    int ring_slot = -1;
    // Half words take a look at every address: only where they save launches and the call does not go through the ring.
    const int64_t lists = (n_g > 0) + (n_q > 0), n_words = tensors ? n_tensors : 0;
    int64_t launches = stage_launches(n_list, lists, n_words, false);
    const int64_t narrow_launches = stage_launches(n_list, lists, n_words, true);
    if (narrow_launches < launches && narrow_launches <= kMaxStageLaunches) {
        sc.narrow = base_of(grad_tensors, n_g, &sc.g_base) && base_of(p16_tensors, n_q, &sc.q_base);
        if (sc.narrow) launches = narrow_launches;
    }
    // A long list that is mostly runs (a model's pages last to first, the pages of some experts) goes as those.  us a call, word by word / as
    // runs: 57 M elements in 64 K pages last to first 262 / 250, with clipping 269 / 262, 216 M (word by word through the ring) 955 / 945 and
    // 994 / 981; of 1.08 G elements of 64 experts in 64 K pages an eighth, from and to tensors, 656 / 614.
    StageRun runs[kStageRuns * kMaxStageLaunches];  // not on the heap: most lists that come here are no runs
    const int64_t n_runs = n_list > 0 && launches > 1 ? runs_of(pages, order, kStageRuns * std::min<int64_t>(launches - 1, kMaxStageLaunches), runs) : -1;
    if (n_runs > 0) {
        const int64_t as_runs = stage_launches_runs(n_runs, lists, n_words);
        if (as_runs < launches && as_runs <= kMaxStageLaunches && base_of(grad_tensors, n_g, &sc.g_base) && base_of(p16_tensors, n_q, &sc.q_base)) {
            sc.runs = runs;
            sc.n_runs = n_runs;
            sc.narrow = true;
            launches = as_runs;
        }
    }
    const bool by_ring = launches > kMaxStageLaunches;
    // A list alone that goes through the ring is read there by the step's kernels: no stage kernel.
    bool staged = tensors || (n_list > 0 && !by_ring);
    L.n_listed = n_pages;
    // One launch whose arguments hold all the words needs no kernel before it.
    CallWords call;
    const bool places = !run || tensors;  // else the page table will do
    call.t.listed = places && !whole;
    const int64_t n_placed = call.t.listed ? n_pages : 0;
    int64_t elems = 0;
    for (int c = 0; c < L.n_cls; ++c) elems += L.cls[c].sum_used;
    const bool words_fit = !captured && 2 * n_placed + n_g + n_q <= kCallWords && (!places || pool->d_places);
    const bool one_launch = words_fit && (need_reduce ? norms && elems <= kCallSumElems && n_pages <= kTaggedPages : places && elems <= kCallElems);  // a bare run has nothing to save
    L.one_pass = need_reduce && !page_sums && one_pass_pays(L, staged || one_launch);
    // As passes the finalize pass writes the records.
    if (need_reduce && !L.one_pass ? words_fit && staged && elems <= kCallPassElems : one_launch) {
        if (fill_call(pool, pages, n_placed, order, grad_tensors, n_g, p16_tensors, n_q, &call) && (!L.one_pass || next_call(pool, stream, &call.t))) {
            if (!grad_tensors) call.t.g_base = reinterpret_cast<uint64_t>(g16_override ? g16_override : static_cast<const uint16_t*>(pool->base[APM_G16]));
            if (!p16_tensors) call.t.q_base = reinterpret_cast<uint64_t>(pool->base[APM_P16]);
            L.call = &call;
            staged = false;
        }
    }
    const int64_t* d_list = whole ? pool->d_order : pool->d_list;
    const int32_t* d_out = whole ? pool->d_order_out : pool->d_list_out;
    const int64_t list_words = sc.runs ? 0 : n_list;
    const bool ring = by_ring && !L.call;
    size_t bytes = (size_t)(list_words + n_g + n_q) * sizeof(uint64_t);
    std::vector<uint64_t> own;
    uint64_t* words = nullptr;
    if (ring) {  // written where they are read from
        if (!staged) bytes = (size_t)n_list * (sizeof(int64_t) + sizeof(int32_t));
        rc = pool->ring.acquire(bytes, &ring_slot);
        if (rc != APM_OK) return rc;
        words = static_cast<uint64_t*>(pool->ring.h[ring_slot]);
    } else if (staged) {
        own.resize((size_t)(list_words + n_g + n_q));
        words = own.data();
    }
    sc.list = list_words ? words : nullptr;
    sc.g_ptrs = n_g ? words + list_words : nullptr;
    sc.q_ptrs = n_q ? words + list_words + n_g : nullptr;
    sc.n_tensors = tensors ? n_tensors : 0;
    sc.tenants = pool->d_tenants;
    sc.d_list = pool->d_list;
    sc.d_out = pool->d_list_out;
    if (staged) {
        for (int64_t k = 0; k < list_words; ++k) words[k] = (uint64_t)page_at(order[(size_t)k]) | (uint64_t)order[(size_t)k] << 32;
        for (int64_t i = 0; i < n_g; ++i) words[list_words + i] = reinterpret_cast<uint64_t>(grad_tensors[i].data);
        for (int64_t i = 0; i < n_q; ++i) words[list_words + n_g + i] = reinterpret_cast<uint64_t>(p16_tensors[i].data);
    } else if (ring) {
        int64_t* list = reinterpret_cast<int64_t*>(words);
        int32_t* out = reinterpret_cast<int32_t*>(list + n_list);
        for (int64_t k = 0; k < n_list; ++k) {
            list[k] = page_at(order[(size_t)k]);
            out[k] = (int32_t)order[(size_t)k];
        }
    }
    if (ring) {
        rc = pool->ring.commit(ring_slot, bytes, stream);
        if (rc != APM_OK) return rc;
        if (staged) {
            sc.d_words = static_cast<const uint64_t*>(pool->ring.d[ring_slot]);
        } else {
            d_list = static_cast<const int64_t*>(pool->ring.d[ring_slot]);
            d_out = reinterpret_cast<const int32_t*>(d_list + n_list);
        }
    }
    L.p32 = static_cast<float*>(pool->base[APM_P32]);
    L.m32 = static_cast<float*>(pool->base[APM_M32]);
    L.v32 = static_cast<float*>(pool->base[APM_V32]);
    L.g16 = g16_override ? g16_override : static_cast<const uint16_t*>(pool->base[APM_G16]);
    L.p16 = static_cast<uint16_t*>(pool->base[APM_P16]);
    L.used = pool->d_used;
    if (!run) {
        L.state_pages = L.grad_pages = d_list;
        L.out_index = d_out;
    }
    L.state_first = L.grad_first = page_at(0);
    L.gather = grad_tensors != nullptr;
    L.scatter = p16_tensors != nullptr;
    L.E = E;
    L.S = pool->S;
    L.grad_norm = grad_norm;
    L.skip_mask = skip_mask;
    L.recs = pool->d_recs;
    L.live = pool->d_live;
    L.sums_ready = need_reduce && page_sums;
    L.wait_limit = pool->wait_limit;
    L.max_workgroups = pool->max_workgroups;
    if (need_reduce) {
        L.partials = page_sums ? page_sums : pool->d_partials;
        L.nzflags = page_sums ? page_nzflags : pool->d_nzflags;
    }
    if (staged) APM_HIP(launch_stage(L, sc, stream));
    if (need_reduce && !L.one_pass) {
        ScopedTiming t(pool, APM_K_REDUCE, stream);
        APM_HIP(launch_grad_reduce(L, stream));
    } else if (!staged && !L.call) {
        L.bare_run = run && !need_reduce;
        if (!L.bare_run) APM_HIP(launch_prepare(L, stream));
    }
    {
        ScopedTiming t(pool, APM_K_UPDATE, stream);
        APM_HIP(L.one_pass ? launch_clip_update(L, stream) : launch_adamw(L, stream));
    }
    return ring_slot >= 0 ? pool->ring.seal(ring_slot, stream) : APM_OK;
}

namespace {
// Spins for `ticks` of the constant-rate device clock; the iteration cap makes it end regardless.
__global__ void apm_spin_kernel(long long ticks, int max_iters) {
    const long long t0 = wall_clock64();
    for (int i = 0; i < max_iters; ++i) {
        if (wall_clock64() - t0 >= ticks) break;
        __builtin_amdgcn_s_sleep(32);
    }
}
}  // namespace

int streams_overlap(hipStream_t a, hipStream_t b, bool* out) {
    int dev = 0, khz = 0;
    APM_HIP(hipGetDevice(&dev));
    APM_HIP(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
    if (khz <= 0) khz = 100000;
    constexpr double kSpinMs = 0.5;
    const long long ticks = (long long)(kSpinMs * khz);
    const int cap = 20000;  // >= 1 us per iteration: the kernel ends after some tens of ms at most
    auto both = [&](long long t, double* ms) -> int {
        APM_HIP(hipStreamSynchronize(a));
        APM_HIP(hipStreamSynchronize(b));
        const auto t0 = std::chrono::steady_clock::now();
        hipLaunchKernelGGL(apm_spin_kernel, dim3(1), dim3(1), 0, a, t, cap);
        hipLaunchKernelGGL(apm_spin_kernel, dim3(1), dim3(1), 0, b, t, cap);
        APM_HIP(hipGetLastError());
        APM_HIP(hipStreamSynchronize(a));
        APM_HIP(hipStreamSynchronize(b));
        *ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
        return APM_OK;
    };
    double warm, ms1, ms2;
    int rc = both(0, &warm);  // loads the kernel
    if (rc == APM_OK) rc = both(ticks, &ms1);
    if (rc == APM_OK) rc = both(ticks, &ms2);
    if (rc != APM_OK) return rc;
    const double ms = ms1 < ms2 ? ms1 : ms2;
    *out = ms < 1.6 * kSpinMs;  // side by side: ~0.5 ms; one after the other: ~1 ms
    return APM_OK;
}

int make_overlapping_stream(hipStream_t with, hipStream_t* out, bool* overlaps, const hipStream_t* also) {
    constexpr int kTries = 8;
    hipStream_t cand[kTries] = {};
    int n = 0, pick = -1;
    int rc = APM_OK;
    // Rejected candidates stay alive until the choice is made: a destroyed stream's queue slot
    // would be handed straight to the next one created.
    for (; n < kTries && pick < 0; ++n) {
        if (hipStreamCreateWithFlags(&cand[n], hipStreamNonBlocking) != hipSuccess) {
            (void)hipGetLastError();
            rc = fail(APM_EDEVICE, "creating a stream failed");
            break;
        }
        bool ok = false;
        rc = streams_overlap(with, cand[n], &ok);
        if (rc == APM_OK && ok && also) rc = streams_overlap(*also, cand[n], &ok);
        if (rc != APM_OK) { ++n; break; }
        if (ok) pick = n;
    }
    if (rc == APM_OK && pick < 0 && n > 0) pick = n - 1;
    for (int k = 0; k < n; ++k)
        if (k != pick && cand[k]) (void)hipStreamDestroy(cand[k]);
    if (rc != APM_OK) {
        if (pick >= 0 && cand[pick]) (void)hipStreamDestroy(cand[pick]);
        return rc;
    }
    *out = cand[pick];
    bool ok = false;
    rc = streams_overlap(with, cand[pick], &ok);
    if (rc == APM_OK && ok && also) rc = streams_overlap(*also, cand[pick], &ok);
    if (overlaps) *overlaps = rc == APM_OK && ok;
    return APM_OK;
}

int ensure_delayed(apm_pool* pool, hipStream_t caller, bool probe) {
    if (pool->upd_stream) return APM_OK;
    const size_t bytes = (size_t)pool->desc.n_pages * (size_t)pool->desc.page_elems * 2u;
    for (int k = 0; k < 2; ++k) {
        if (pool->gbuf[k]) continue;  // kept from an attempt that failed further down
        hipError_t e = hipMalloc((void**)&pool->gbuf[k], bytes);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            for (int j = 0; j < 2; ++j) {
                if (pool->gbuf[j]) (void)hipFree(pool->gbuf[j]);
                pool->gbuf[j] = nullptr;
            }
            return fail(APM_ENOMEM, "allocating the %zu-byte buffered-gradient halves failed: %s", bytes, hipGetErrorString(e));
        }
    }
    // Zero once: a producer that fills a half in place writes its tensors' elements only, and the
    // alignment gaps inside a page's used extent are read as gradient.
    for (int k = 0; k < 2; ++k) APM_HIP(hipMemset(pool->gbuf[k], 0, bytes));
    for (int k = 0; k < 2; ++k) {
        if (!pool->ev_staged[k]) APM_HIP(hipEventCreateWithFlags(&pool->ev_staged[k], hipEventDisableTiming));
        if (!pool->ev_applied[k]) APM_HIP(hipEventCreateWithFlags(&pool->ev_applied[k], hipEventDisableTiming));
    }
    if (!pool->ev_flush) APM_HIP(hipEventCreateWithFlags(&pool->ev_flush, hipEventDisableTiming));
    // The update stream must run beside the producer's stream, which is the point of the
    // one-step-stale form; which streams do is measured, once, here.
    if (probe) return make_overlapping_stream(caller, &pool->upd_stream, &pool->upd_overlaps);
    APM_HIP(hipStreamCreateWithFlags(&pool->upd_stream, hipStreamNonBlocking));
    return APM_OK;
}

// Sums are worked out by the hand-over if a page fills the greater part of the workgroup that takes a tile (us
// with and without, 16 M elements: pages of 512 elements 133 and 36 a sum, 283 and 400 an update; 2048: 81 and 63,
// 378 and 386; 4096: 66 and 64, 343 and 357), else the update works them out itself.
constexpr int64_t kSumsPage = 4096;

// Room for the sums of half k; without it the update works them out itself.
static bool ensure_sums(apm_pool* pool, int k) {
    if (pool->desc.page_elems < kSumsPage) return false;
    const size_t n = (size_t)pool->desc.n_pages * (size_t)pool->S;
    if (!pool->gsum[k] && hipMalloc((void**)&pool->gsum[k], n * sizeof(double)) != hipSuccess) pool->gsum[k] = nullptr;
    if (!pool->gnz[k] && hipMalloc((void**)&pool->gnz[k], n * sizeof(uint32_t)) != hipSuccess) pool->gnz[k] = nullptr;
    if (pool->gsum[k] && pool->gnz[k]) return true;
    (void)hipGetLastError();
    return false;
}

// Launches that may carry a hand-over's page list in their arguments; beyond that it is staged through the
// pinned ring (reversed lists, 4 / 5 / 8 launches of 880 pages of 512 elements against the ring: 31 and 35,
// 37 and 37, 56 and 44 us).
constexpr int64_t kMaxTakeLaunches = 4;

// Copies or adds the used extents of the listed pages of g16 into half k.
static int take_gradient(apm_pool* pool, int k, const uint16_t* g16, const int64_t* pages, int64_t n_pages, bool accumulate,
                         bool sums, hipStream_t s) {
    if (n_pages == 0) return APM_OK;
    const int64_t in_use = (int64_t)pool->plan.pages.size();
    GradTake t{g16, pool->gbuf[k], accumulate, pool->d_used, pool->desc.page_elems, pool->S, sums ? pool->gsum[k] : nullptr,
               sums ? pool->gnz[k] : nullptr, nullptr, nullptr, 0, pool->whole.cls, pool->whole.n_cls, pool->max_workgroups};
    if (!pages && n_pages == in_use) {
        t.order = pool->whole.plain ? nullptr : pool->d_order;
        APM_HIP(launch_grad_take(t, s));
        return APM_OK;
    }
    auto page_at = [&](int64_t i) { return pages ? pages[i] : i; };
    ExtentClass cls[kMaxExtentClasses];
    t.cls = cls;
    const bool run = consecutive(pages, n_pages);
    // Consecutive pages need no list, and with the extents taken as the layout's largest no look-up, at the price of
    // workgroups without work where pages differ much: a list is the better form then.
    if (run && (n_pages > kTakePages || pool->whole.run_n_cls <= 1)) {
        cls[0] = run_class(pool, page_at(0), n_pages);
        t.n_cls = 1;
        t.first = page_at(0);
        APM_HIP(launch_grad_take(t, s));
        return APM_OK;
    }
    std::vector<int64_t> order((size_t)n_pages);
    std::vector<int32_t> room;
    ExtentGroups groups(n_pages, pool->desc.page_elems, page_extents(pool, pages, n_pages, &room));
    t.n_cls = groups.fold(kWorthGrid, cls);
    groups.order(order.data());
    for (int64_t& i : order) i = page_at(i);
    const int64_t launches = (n_pages + kTakePages - 1) / kTakePages;
    int slot = -1;
    if (launches > kMaxTakeLaunches) {
        const size_t bytes = (size_t)n_pages * sizeof(int64_t);
        int rc = pool->ring.acquire(bytes, &slot);
        if (rc != APM_OK) return rc;
        std::memcpy(pool->ring.h[slot], order.data(), bytes);
        rc = pool->ring.commit(slot, bytes, s);
        if (rc != APM_OK) return rc;
        t.order = static_cast<const int64_t*>(pool->ring.d[slot]);
    } else {
        t.host_pages = order.data();
    }
    APM_HIP(launch_grad_take(t, s));
    return slot >= 0 ? pool->ring.seal(slot, s) : APM_OK;
}

// Whether the buffered gradient holds every element that the layout installed now gives the listed pages.
static int check_buffered(const apm_pool* pool, const int64_t* pages, int64_t n_pages) {
    if (pool->buf_extents.empty()) return APM_OK;
    for (int64_t i = 0; i < n_pages; ++i) {
        const int64_t p = pages ? pages[i] : i;
        if (pool->used[(size_t)p] > ((pool->buf_extents[(size_t)p] + 7) & ~7))
            return fail(APM_ESTATE, "page %lld has %d elements in the layout installed since the gradient was handed over, %d were handed over", (long long)p, pool->used[(size_t)p], pool->buf_extents[(size_t)p]);
    }
    return APM_OK;
}

// Applies the buffered gradient (half `cur`) on the update stream.
static int apply_buffered(apm_pool* pool, const DelayedApply& apply) {
    const int k = pool->cur;
    const int held = check_buffered(pool, pool->buf_pages_null ? nullptr : pool->buf_pages.data(), pool->buf_n_pages);
    if (held != APM_OK) {  // it cannot be applied any more
        pool->buffered = false;
        return held;
    }
    APM_HIP(hipStreamWaitEvent(pool->upd_stream, pool->ev_staged[k], 0));
    int rc = apply(pool->gbuf[k], pool->applied + 1, pool->upd_stream,
                   pool->buf_pages_null ? nullptr : pool->buf_pages.data(), pool->buf_n_pages, &pool->buf_hyper);
    if (rc != APM_OK) return rc;
    pool->applied += 1;
    APM_HIP(hipEventRecord(pool->ev_applied[k], pool->upd_stream));
    pool->applied_valid[k] = true;
    return APM_OK;
}

int delayed_call(apm_pool* pool, const int64_t* pages, int64_t n_pages, const void* new_g16,
                 const apm_hyper* hyper, hipStream_t s, const DelayedApply& apply, bool want_sums) {
    APM_HIP(hipSetDevice(pool->desc.hip_device));
    int rc = ensure_delayed(pool, s, true);
    if (rc != APM_OK) return rc;
    if (pool->buffered) {
        rc = apply_buffered(pool, apply);
        if (rc != APM_OK) return rc;
        pool->buffered = false;
    }
    if (!new_g16) {  // flush: the caller's stream joins the update stream
        APM_HIP(hipEventRecord(pool->ev_flush, pool->upd_stream));
        APM_HIP(hipStreamWaitEvent(s, pool->ev_flush, 0));
        return APM_OK;
    }
    // Stage the new gradient into the other half; that half was last read by the update enqueued
    // two calls ago, which must have finished before it is overwritten.
    const int nxt = pool->cur ^ 1;
    const size_t pb = (size_t)pool->desc.page_elems * 2u;
    // The gradient travels with the list and the hyper-parameters of this call (copied before
    // anything is enqueued: an allocation failure leaves the pool as it was).
    std::vector<int64_t> list_copy;
    if (pages) list_copy.assign(pages, pages + n_pages);
    const char* src = static_cast<const char*>(new_g16);
    char* dst = reinterpret_cast<char*>(pool->gbuf[nxt]);
    // A producer that wrote its gradient straight into the half handed out by
    // apm_delayed_grad_buffer has already staged it (and waited for the half to be free there).
    const bool in_place = src == dst;
    if (!in_place && pool->applied_valid[nxt]) APM_HIP(hipStreamWaitEvent(s, pool->ev_applied[nxt], 0));
    pool->gsum_ok[nxt] = false;
    const bool by_extent = !in_place && pool->has_layout && (reinterpret_cast<uintptr_t>(new_g16) & 15u) == 0;
    if (by_extent) {
        want_sums = want_sums && ensure_sums(pool, nxt);
        rc = take_gradient(pool, nxt, static_cast<const uint16_t*>(new_g16), pages, n_pages, false, want_sums, s);
        if (rc != APM_OK) return rc;
        pool->gsum_ok[nxt] = want_sums;
        pool->gsum_epoch[nxt] = pool->layout_epoch;
    } else if (!in_place) {  // no layout yet, so no extents, or no vectors: whole pages, a copy per run of consecutive ones
        for (int64_t k = 0; k < n_pages;) {
            const int64_t p0 = pages ? pages[k] : k;
            int64_t len = 1;
            while (k + len < n_pages && (pages ? pages[k + len] : k + len) == p0 + len) ++len;
            APM_HIP(hipMemcpyAsync(dst + (size_t)p0 * pb, src + (size_t)p0 * pb, pb * (size_t)len, hipMemcpyDeviceToDevice, s));
            k += len;
        }
    }
    APM_HIP(hipEventRecord(pool->ev_staged[nxt], s));
    pool->buf_hyper = *hyper;
    pool->buf_pages.swap(list_copy);
    pool->buf_pages_null = pages == nullptr;
    pool->buf_n_pages = n_pages;
    pool->buf_by_extent = by_extent;
    pool->buf_extents.clear();
    pool->cur = nxt;
    pool->buffered = true;
    return APM_OK;
}

}  // namespace apm

using namespace apm;

extern "C" int apm_page_adamw_step(apm_pool* pool, const int64_t* pages, int64_t n_pages,
                                   int64_t step, const apm_hyper* hyper, float* grad_norm,
                                   uint8_t* skip_mask, void* stream) {
    return apm::guarded([&]() -> int {
        return enqueue_step(pool, pages, n_pages, step, hyper, nullptr, grad_norm, skip_mask,
                            static_cast<hipStream_t>(stream));
    });
}

extern "C" int apm_page_adamw_step_fused(apm_pool* pool, const int64_t* pages, int64_t n_pages,
                                         int64_t step, const apm_hyper* hyper,
                                         const apm_tensor* grad_tensors,
                                         const apm_tensor* p16_tensors, int64_t n_tensors,
                                         float* grad_norm, uint8_t* skip_mask, void* stream) {
    return apm::guarded([&]() -> int {
        if (!grad_tensors && !p16_tensors) return fail(APM_EINVAL, "neither a gradient nor a parameter tensor list was given");
        if (n_tensors < 0) return fail(APM_EINVAL, "negative tensor count");
        return enqueue_step(pool, pages, n_pages, step, hyper, nullptr, grad_norm, skip_mask,
                            static_cast<hipStream_t>(stream), grad_tensors, p16_tensors, n_tensors);
    });
}

extern "C" int apm_step_delayed(apm_pool* pool, const int64_t* pages, int64_t n_pages,
                                const void* new_g16, const apm_hyper* hyper, void* stream) {
    return apm::guarded([&]() -> int {
        if (!pool) return fail(APM_EINVAL, "NULL pool");
        if (pool->desc.device != APM_DEV_GPU) return fail(APM_EDEVICE, "the update runs on GPU pools only");
        if (n_pages < 0 || n_pages > pool->desc.n_pages) return fail(APM_ERANGE, "page count %lld out of range", (long long)n_pages);
        AdamwLaunch probe{};
        int rc = prepare_hyper(hyper, 1, &probe);  // validate before any state changes
        if (rc != APM_OK) return rc;
        if (pages)
            for (int64_t k = 0; k < n_pages; ++k)
                if (pages[k] < 0 || pages[k] >= pool->desc.n_pages) return fail(APM_ERANGE, "pages[%lld] out of range", (long long)k);
        return delayed_call(pool, pages, n_pages, new_g16, hyper, static_cast<hipStream_t>(stream),
                            [&](const uint16_t* g16, int64_t step, hipStream_t upd, const int64_t* b_pages,
                                int64_t b_n, const apm_hyper* b_hyper) {
                                const int k = g16 == pool->gbuf[1] ? 1 : 0;
                                const bool sums = pool->gsum_ok[k] && pool->gsum_epoch[k] == pool->layout_epoch;
                                return enqueue_step(pool, b_pages, b_n, step, b_hyper, g16, pool->delayed_norm,
                                                    pool->delayed_skip, upd, nullptr, nullptr, 0,
                                                    sums ? pool->gsum[k] : nullptr, sums ? pool->gnz[k] : nullptr);
                            },
                            hyper->max_grad_norm > 0.0 || hyper->skip_mode != APM_SKIP_NONE || pool->delayed_norm || pool->delayed_skip);
    });
}

extern "C" int apm_delayed_accumulate(apm_pool* pool, const int64_t* pages, int64_t n_pages,
                                      const void* g16, void* stream) {
    return apm::guarded([&]() -> int {
        if (!pool || !g16) return fail(APM_EINVAL, "NULL argument");
        if (pool->desc.device != APM_DEV_GPU) return fail(APM_EDEVICE, "GPU pools only");
        if (!pool->buffered) return fail(APM_ESTATE, "no gradient is being collected: call apm_step_delayed with a gradient first");
        if (n_pages < 0 || n_pages > pool->desc.n_pages) return fail(APM_ERANGE, "page count %lld out of range", (long long)n_pages);
        if (n_pages == 0) return APM_OK;
        APM_HIP(hipSetDevice(pool->desc.hip_device));
        hipStream_t s = static_cast<hipStream_t>(stream);
        if (pages)
            for (int64_t k = 0; k < n_pages; ++k)
                if (pages[k] < 0 || pages[k] >= pool->desc.n_pages) return fail(APM_ERANGE, "pages[%lld] out of range", (long long)k);
        int rc = check_buffered(pool, pages, n_pages);
        if (rc != APM_OK) return rc;
        // The collecting half was staged on the producer's stream; the sum is ordered after it there,
        // and the "staged" event moves behind the sum so that the update sees the accumulated values.
        const int k = pool->cur;
        APM_HIP(hipStreamWaitEvent(s, pool->ev_staged[k], 0));
        if (pool->has_layout) {  // without a layout no page has a used extent
            if (pool->gsum_epoch[k] != pool->layout_epoch) pool->gsum_ok[k] = false;
            rc = take_gradient(pool, k, static_cast<const uint16_t*>(g16), pages, n_pages, true, pool->gsum_ok[k], s);
            if (rc != APM_OK) return rc;
        }
        APM_HIP(hipEventRecord(pool->ev_staged[k], s));
        return APM_OK;
    });
}

extern "C" void* apm_delayed_grad_buffer(apm_pool* pool, void* stream) {
    if (!pool || pool->desc.device != APM_DEV_GPU) {
        fail(APM_EINVAL, "NULL or non-GPU pool");
        return nullptr;
    }
    if (hipSetDevice(pool->desc.hip_device) != hipSuccess ||
        ensure_delayed(pool, static_cast<hipStream_t>(stream), true) != APM_OK) return nullptr;
    const int nxt = pool->cur ^ 1;
    if (pool->applied_valid[nxt] &&
        hipStreamWaitEvent(static_cast<hipStream_t>(stream), pool->ev_applied[nxt], 0) != hipSuccess) {
        fail(APM_EDEVICE, "hipStreamWaitEvent failed");
        return nullptr;
    }
    return pool->gbuf[nxt];
}

extern "C" int64_t apm_delayed_applied(const apm_pool* pool) { return pool ? pool->applied : 0; }

extern "C" int apm_delayed_set_outputs(apm_pool* pool, float* grad_norm, uint8_t* skip_mask) {
    return apm::guarded([&]() -> int {
        if (!pool) return fail(APM_EINVAL, "NULL pool");
        pool->delayed_norm = grad_norm;
        pool->delayed_skip = skip_mask;
        return APM_OK;
    });
}

extern "C" int apm_test_set_max_workgroups(apm_pool* pool, int64_t max_workgroups) {
    if (!pool || max_workgroups < 0) return fail(APM_EINVAL, "bad argument");
    pool->max_workgroups = max_workgroups;
    return APM_OK;
}

extern "C" int apm_test_set_wait_limit(apm_pool* pool, int32_t wait_limit) {
    if (!pool || wait_limit < 0) return fail(APM_EINVAL, "bad argument");
    pool->wait_limit = wait_limit;
    return APM_OK;
}

extern "C" int apm_test_set_call_number(apm_pool* pool, uint32_t number) {
    if (!pool) return fail(APM_EINVAL, "bad argument");
    pool->call_number = number;
    return APM_OK;
}
