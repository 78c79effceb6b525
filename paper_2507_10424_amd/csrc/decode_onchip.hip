// On-chip Min-Sum decoder, host side: variant choice, launch geometry, the
// single-graph and multi-graph launches.  The kernels are in onchip_kernel.h
// (one instantiation per source file and register budget).
#include <algorithm>
#include <mutex>
#include <new>

#include "onchip_kernel.h"

namespace ldpc {
namespace {
using namespace onchip;

// The widest masked variant is left out of the multi-code kernel: the
// register demand of a kernel is that of its largest variant, and that one
// alone would push every variant of the launch into spills.  Jobs that need
// it get a launch of their own.  So is the bank-conflict-free layout: its
// tables are built for the graph's own thread count, and the shared launch
// runs the largest thread count of its jobs.
constexpr int kWideVariant = 6;
constexpr bool shared_launch_ok(int v) { return v != kWideVariant && kVariants[v].cf == 0 && v < 16; }
static_assert(kNumVariants == 42, "k_onchip_multi dispatches variants 0-5 and 7-13");

__global__ __launch_bounds__(kMaxThreads) void k_onchip_multi(const JobTable jt, int32_t L, int32_t early) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    for (int32_t c = 0; c < jt.njobs; ++c) {
        switch (jt.job[c].variant) {
        case 0: run_v<0, false>(jt.job[c], L, early, lds); break;
        case 1: run_v<1, false>(jt.job[c], L, early, lds); break;
        case 2: run_v<2, false>(jt.job[c], L, early, lds); break;
        case 3: run_v<3, false>(jt.job[c], L, early, lds); break;
        case 4: run_v<4, false>(jt.job[c], L, early, lds); break;
        case 5: run_v<5, false>(jt.job[c], L, early, lds); break;
        case 7: run_v<7, false>(jt.job[c], L, early, lds); break;
        case 8: run_v<8, false>(jt.job[c], L, early, lds); break;
        case 9: run_v<9, false>(jt.job[c], L, early, lds); break;
        case 10: run_v<10, false>(jt.job[c], L, early, lds); break;
        case 11: run_v<11, false>(jt.job[c], L, early, lds); break;
        case 12: run_v<12, false>(jt.job[c], L, early, lds); break;
        case 13: run_v<13, false>(jt.job[c], L, early, lds); break;
        default: break; // the host places no variant here that fails shared_launch_ok
        }
        __syncthreads();
    }
}

// [register budget][learned][variant]; register budgets: the compiler's, at
// least 4 and at least 3 waves per SIMD
const KernelFn (*const kKernels[3])[kNumVariants] = {kKernelsW0, kKernelsW4, kKernelsW3};
// Index of a register budget (waves per SIMD: 0, 4 or 3) in kKernels.
inline int budget_index(int waves_per_simd) { return waves_per_simd == 4 ? 1 : waves_per_simd == 3 ? 2 : 0; }
inline int tuned_budget(const ldpc_graph &g) { return g.tuned() ? budget_index(g.tuning.waves_per_simd) : 0; }

// Threads: whole wavefronts, enough for RPT rows and CPT bits per thread.
int threads_for(const ldpc_graph &g, const Variant &v) {
    const int a = (g.m + v.rpt - 1) / v.rpt, b = (g.n + v.cpt - 1) / v.cpt;
    const int want = a > b ? a : b;
    const int t = ((want + 63) / 64) * 64;
    return t < 64 ? 64 : t;
}

// Every column's degree is within the profile at any slot index.
bool profile_holds(const ldpc_graph &g, const Variant &v) {
    const int t = threads_for(g, v);
    for (int c = 0; c * t < g.n; ++c)
        if (c >= v.cpt || (int)((v.dvp >> (4 * c)) & 15u) < g.dv_max) return false;
    return true;
}

bool variant_ok(const ldpc_graph &g, int k) {
    if (k < 0 || k >= kNumKernels) return false;
    const Variant &v = kVariants[k];
    const bool rows_ok = v.rx ? (g.dc_min == v.dc && g.dc_max == v.dc) : g.dc_max <= v.dc;
    // (a padded layout variant, cf & 4, takes columns of any degree up to its dv)
    const bool cols_ok = (v.cx && !(v.cf & 4)) ? (g.dv_min == v.dv && g.dv_max == v.dv) : g.dv_max <= v.dv;
    // the layout's tables are for their own geometry, stride and thread count
    const bool regular = k >= kFirstRegular && k < kFirstOwnLayout; // on the tables without a profile
    const bool cf_ok = v.cf == 0 || (g.cf.edge != nullptr && g.cf.rpt == v.rpt && g.cf.cpt == v.cpt &&
                                     g.cf.dvs == v.dv && g.cf.dvp == (regular ? 0u : v.dvp) &&
                                     threads_for(g, v) == g.cf.nt && (!regular || profile_holds(g, v)));
    const size_t state = v.cf != 0 ? cf_state_bytes(g, v.f) : state_bytes(g, v.f);
    return rows_ok && cols_ok && cf_ok && threads_for(g, v) <= kMaxThreads && g.edge_tab != nullptr &&
           state + sizeof(Shared) + 1024 <= (size_t)g.lds_max;
}

size_t state_of(const ldpc_graph &g, int variant) {
    return kVariants[variant].cf != 0 ? cf_state_bytes(g, kVariants[variant].f) : state_bytes(g, kVariants[variant].f);
}
size_t lds_of(const ldpc_graph &g, int variant) { return state_of(g, variant) + sizeof(Shared); }

// Default preference when nothing is tuned: the bank-conflict-free layout,
// then exact degrees, a column mask of 6 before one of 8, two frame slots
// before four.
constexpr int kPickOrder[] = {15, 14, 33, 32, 35, 34, 37, 36, 39, 38, 41, 40, 22, 23, 24, 25, 26, 27, 28, 29, 30,
                              31, 0,  7,  10, 1,  11, 2,  12, 3,  13, 4,  5,  6,  8,  9,  16, 17, 18, 19, 20, 21};
static_assert(sizeof(kPickOrder) / sizeof(kPickOrder[0]) == kNumVariants, "every variant has a place");

// The tuned variant if one is set and valid, else the first that fits.
int pick(const ldpc_graph &g) {
    if (g.tuned() && variant_ok(g, g.tuning.variant)) return g.tuning.variant;
    for (int k : kPickOrder)
        if (variant_ok(g, k)) return k;
    return -1;
}

// Layout variants whose two-slot kernel takes more than 128 registers, so that
// at most three of its waves share a SIMD: their one-slot form is the faster
// one at every batch size (n = 1152, rows of 9, 20,000 frames: 0.406 ms with
// two slots, 0.286 with one; rows of 12: 0.459 and 0.327) where the GPU holds
// more workgroups of it (kernel_of).
constexpr bool one_slot_always(int v) {
    return v == 23 || v == 27 || v == 29 || v == 31 || v == 33 || v == 37 || v == 39 || v == 41;
}

// The kernel for a regular graph's own row and column degree, -1 if there is
// none.  Faster than the padded layout's one-slot kernels, which read six
// messages (four with rows of 16) of any bit, and than the LDS-resident decoder,
// which takes rows of 8 and 10 otherwise (20 iterations, 300 and 16,000 frames,
// before and now: (3,9) n = 2,007 0.047 and 0.522 ms, 0.026 and 0.457; (3,12) n =
// 2,004 0.036 and 0.320, 0.017 and 0.215; (4,16) n = 2,016 0.037 and 0.409, 0.019
// and 0.251; (4,8) n = 2,008 0.062 and 1.389, 0.042 and 0.701; (5,10) n = 1,010
// 0.049 and 1.028, 0.034 and 0.572).
int regular_form(const ldpc_graph &g) {
    for (int k = kFirstRegular; k < kNumKernels; ++k)
        if (variant_ok(g, k)) return k;
    return -1;
}

int64_t room_of(const ldpc_graph &g, int v, bool learned) { // resident workgroups, with the compiler's registers
    const KernelFn fn = v >= kNumVariants ? kKernelsOne[learned ? 1 : 0][v - kNumVariants] : kKernels[0][learned ? 1 : 0][v];
    return resident_workgroups((const void *)fn, threads_for(g, kVariants[v]), lds_of(g, v), g);
}

// The kernel (index into kVariants) that decodes B frames: the picked variant,
// or, without a tuning record, its one-slot form or the regular graph's own,
// whose rounds are about half as long, while no more than four frames (five where
// they stop early, and a slot waits less for its neighbour) fall to each resident
// workgroup of it ((3,6) n = 1024, B = 1,000: 0.069 ms with two slots and 0.045
// with one; 4,000: 0.097 and 0.092; 20,000: 0.233 and 0.253; early exit, n = 576,
// rows of 6, 6,000 of 1,280 at a time, 0.137 and 0.123; to the end, n = 1530, 2,500
// of 512, 0.094 and 0.113), and at every size where the two-slot kernel is short of
// registers.  Rows of 9 and workgroups of more than four wavefronts are the
// exception: a CU holds one workgroup of either kernel, so that the one-slot form
// decodes half the frames at a time.  There it is taken at every size for a
// regular graph's own and plain decoding, and where other launches fill the GPU;
// else while the frames of each workgroup are few: 12 where they stop early (6
// for a profile's learned decoding), 3 where they do not (6 for a regular graph's
// own).  (Two slots and one, (3,9) n = 1800: to the end, 600 frames 0.063 and 0.049
// ms, 20,000 1.12 and 1.08; learned, 2,600 frames 0.207 and 0.203, 7,000 0.462 and
// 0.484; learned to the end, 1,200 frames 0.101 and 0.095, 7,000 0.441 and 0.494.
// Columns of 2, 3 and 6, n = 2304: early exit, 2,100 frames 0.216 and 0.193, 7,000
// 0.471 and 0.513; learned, 1,200 frames 0.131 and 0.128, 7,000 0.480 and 0.575; to
// the end, 600 frames 0.057 and 0.051, 7,000 0.343 and 0.398.)
int kernel_of(const ldpc_graph &g, int64_t B, bool learned, bool early, bool shared = false) {
    const int v = pick(g), r = onchip_regular(g) ? regular_form(g) : -1;
    const int o = r >= 0 ? r : v >= 0 ? one_slot(v) : -1;
    if (g.tuned() || o < 0 || !variant_ok(g, o)) return v;
    if (r >= 0 && (v < 0 || !kVariants[v].rx)) return r; // (no two-slot kernel for rows of its degree)
    const int64_t room = room_of(g, o, learned);
    if (r < 0 && !one_slot_always(v)) return B <= (early ? 5 : 4) * room ? o : v;
    if (shared || (r >= 0 && !learned) || 4 * room >= 5 * room_of(g, v, learned)) return o;
    const bool few = early ? learned && r < 0 : r < 0;
    return B <= (early ? 12 : 6) / (few ? 2 : 1) * room ? o : v;
}
KernelFn kernel_fn(const ldpc_graph &g, int v, bool learned) {
    return v >= kNumVariants ? kKernelsOne[learned ? 1 : 0][v - kNumVariants]
                             : kKernels[tuned_budget(g)][learned ? 1 : 0][v];
}

Job make_job(const ldpc_graph &g, int variant, const float *llr, int32_t B, uint8_t *bits, float *post,
             int32_t *iters, uint8_t *ok, const float *alpha, const float *beta, uint32_t *queue) {
    Job J;
    J.row_ptr = g.row_ptr;
    J.edge_tab = g.edge_tab;
    J.col_ptr = g.col_ptr;
    J.row_class = g.row_class;
    J.m = g.m;
    J.n = g.n;
    J.E = (int32_t)g.E;
    J.sh_off = (uint32_t)state_of(g, variant);
    J.cf_edge = g.cf.edge;
    J.cf_bitpos = g.cf.bitpos;
    J.cf_slot_bit = g.cf.slot_bit;
    J.cf_row_class = g.cf.row_class;
    J.cf_eta_off = cf_eta_offset(g, kVariants[variant].f);
    J.cf_npos = g.cf.npos;
    J.llr = llr;
    J.B = B;
    J.bits = bits;
    J.post = post;
    J.iters = iters;
    J.ok = ok;
    J.alpha = alpha;
    J.beta = beta;
    J.ncls = (int32_t)g.class_degrees.size();
    J.variant = variant;
    J.dealt = J.grid = J.rounds = 0;
    J.queue = queue;
    J.nq = queues_for(B);
    return J;
}

// A launch of `grid` workgroups for one job with a one-slot kernel: the first
// `rounds` frames of each workgroup are dealt (it holds one and knows the
// next), and where those are all, no counter is needed (nor the launch that
// clears it).  Two where all workgroups start at once: drawn, the second ones
// come with an atomic of every workgroup, and most of a batch of little more
// than `grid` finds every counter exhausted one by one (n = 108, rows of 9,
// 4,000 frames: 0.059 ms with one dealt, 0.034 with two).  One where the launch
// shares the GPU with others (the eight quasi-cyclic codes take 1 % longer
// with two).
void deal(Job &J, int grid, int rounds) {
    if (J.variant < kNumVariants) return;
    J.grid = grid;
    J.rounds = rounds;
    J.dealt = (int32_t)std::min<int64_t>(rounds * (int64_t)grid, J.B);
    if (J.dealt == J.B) J.queue = nullptr;
    else J.nq = queues_for(std::max(J.B - J.dealt, 4 * grid)); // (every workgroup draws at about the same time)
}

// Grid of a persistent launch: every CU filled to its occupancy, but no more
// workgroups than there are groups of `per_wg` frames.  `rounds` frames of each
// workgroup may be dealt: where that is every frame, up to the runtime's count of
// workgroups, since those that wait for a CU take it as the first ones end (n =
// 2304, rows of 9, 430 frames: 0.076 ms with 430, 0.093 with the 256 that run at
// once and two frames to each; (3,12) n = 1200, 1,100 frames to the end, 512 at
// once and 768: 0.060 ms with 768, 0.072 with 550).  `among`: other launches share
// the GPU, and the grid is the runtime's count: workgroups waiting for a CU take
// it from launches that end (the eight quasi-cyclic codes at 0.3 of their
// batches, 1.5 dB: 0.599 ms, 0.668 with those that run at once).
int launch_grid(const void *fn, int threads, size_t lds, const ldpc_graph &g, int64_t frames, int cap_per_cu,
                int *grid, int per_wg, int rounds = 0, bool among = false) {
    int64_t promised = 0, want = resident_workgroups(fn, threads, lds, g, &promised);
    if (want < 0) return LDPC_EHIP;
    if (among) want = promised;
    if (rounds > 0 && cap_per_cu == 0 && frames <= rounds * promised) {
        *grid = (int)std::min(frames, promised);
        return LDPC_OK;
    }
    if (cap_per_cu > 0) want = std::min(want, (int64_t)g.num_cu * cap_per_cu);
    const int64_t groups = (frames + per_wg - 1) / per_wg;
    *grid = (int)(want < groups ? want : groups);
    if (*grid < 1) *grid = 1;
    return LDPC_OK;
}

// Side streams of the multi-code decoder, one set per device, created on
// first use (default priority, non-blocking) and kept until the process
// ends; `mu` serialises the calls that fork onto them.
constexpr int kSideStreams = 3;
struct SideStreams {
    hipStream_t s[kSideStreams];
    hipEvent_t fork, join[kSideStreams];
    std::mutex mu;
};
SideStreams *side_streams() {
    constexpr int kMaxDevices = 64;
    static SideStreams *sets[kMaxDevices] = {};
    static bool failed[kMaxDevices] = {};
    static std::mutex make;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(make);
    if (!sets[dev] && !failed[dev]) {
        failed[dev] = true; // until the set is complete
        SideStreams *x = new (std::nothrow) SideStreams();
        if (!x) return nullptr;
        bool ok = hipEventCreateWithFlags(&x->fork, hipEventDisableTiming) == hipSuccess;
        for (int k = 0; k < kSideStreams && ok; ++k)
            ok = hipStreamCreateWithFlags(&x->s[k], hipStreamNonBlocking) == hipSuccess &&
                 hipEventCreateWithFlags(&x->join[k], hipEventDisableTiming) == hipSuccess;
        if (!ok) return nullptr; // (a partial set is left to the process end; every call runs on `stream`)
        sets[dev] = x;
        failed[dev] = false;
    }
    return sets[dev];
}

} // namespace

bool onchip_cf_geometry(const ldpc_graph &g, const std::vector<int32_t> &col_deg, int32_t *rpt, int32_t *cpt,
                        int32_t *dvs, uint32_t *dvp) {
    // Among the layout variants for the graph's row degree whose stride (or
    // degree profile) holds its columns: the least lane work issued per round
    // (threads round up to whole wavefronts; a check edge weighs about four
    // bit-side adds, and a bit slot index reads its profile entry's messages),
    // then the exact stride, then more threads (more wavefronts to hide LDS
    // latency when LDS limits the workgroups per CU).
    std::vector<int32_t> sorted(col_deg);
    std::sort(sorted.begin(), sorted.end());
    int best = -1;
    int64_t best_cost = 0;
    for (int k = 0; k < kNumKernels; ++k) {
        if (k >= kNumVariants && k < kFirstOwnLayout) continue; // (on the tables of the others)
        const Variant &v = kVariants[k];
        if (v.cf == 0 || g.dc_min != g.dc_max || g.dc_max != v.dc || g.dv_max > v.dv) continue;
        if (!(v.cf & 4) && (g.dv_min != v.dv || g.dv_max != v.dv)) continue; // exact columns only
        const int t = threads_for(g, v);
        if (t > kMaxThreads) continue;
        int64_t reads = (int64_t)v.cpt * v.dv;
        if (v.dvp != 0u) { // bits in ascending degree: slot index c holds sorted[c t .. c t + t)
            bool holds = true;
            for (size_t p = 0; p < sorted.size() && holds; ++p)
                holds = (int32_t)((v.dvp >> (4 * (p / t))) & 15u) >= sorted[p];
            if (!holds) continue;
            reads = 0;
            for (int c = 0; c < v.cpt; ++c) reads += (v.dvp >> (4 * c)) & 15u;
        }
        const int64_t cost = (int64_t)t * (4 * v.rpt * v.dc + reads);
        const Variant *b = best >= 0 ? &kVariants[best] : nullptr;
        if (best < 0 || cost < best_cost ||
            (cost == best_cost && (v.dv < b->dv || (v.dv == b->dv && t > threads_for(g, *b))))) {
            best = k;
            best_cost = cost;
        }
    }
    if (best < 0) return false;
    *rpt = kVariants[best].rpt;
    *cpt = kVariants[best].cpt;
    *dvs = kVariants[best].dv;
    *dvp = kVariants[best].dvp;
    return true;
}

bool onchip_regular(const ldpc_graph &g) {
    return g.edge_tab != nullptr && !g.tuned() && regular_form(g) >= 0;
}

bool onchip_fits(const ldpc_graph &g) { return g.edge_tab != nullptr && pick(g) >= 0; }

bool onchip_masks_rows(const ldpc_graph &g) {
    const int v = pick(g);
    return v >= 0 && !kVariants[v].rx;
}

bool onchip_variant_fits(const ldpc_graph &g, int variant) { return variant_ok(g, variant); }

int onchip_num_variants() { return kNumVariants; }

bool onchip_kernel_spill_free(int variant, int waves_per_simd) { return onchip_kernel_spill_bytes(variant, waves_per_simd) == 0; }

int64_t onchip_kernel_spill_bytes(int variant, int waves_per_simd) {
    if (variant < 0 || variant >= kNumVariants) return -1;
    hipFuncAttributes a{};
    if (hipFuncGetAttributes(&a, (const void *)kKernels[budget_index(waves_per_simd)][0][variant]) != hipSuccess)
        return -1;
    return (int64_t)a.localSizeBytes;
}

int onchip_kernel_vgprs(int variant, int waves_per_simd) {
    if (variant < 0 || variant >= kNumVariants) return -1;
    hipFuncAttributes a{};
    if (hipFuncGetAttributes(&a, (const void *)kKernels[budget_index(waves_per_simd)][0][variant]) != hipSuccess)
        return -1;
    return a.numRegs;
}

size_t onchip_workspace_bytes(const ldpc_graph &g, int32_t B) {
    (void)g;
    (void)B;
    return 4ull * kQueueWords; // frame counters
}

int onchip_decode(const ldpc_graph &g, const float *llr, int32_t B, int32_t L, uint32_t flags, const float *alpha,
                  const float *beta, int32_t T, uint8_t *bits, float *post, int32_t *iters, uint8_t *ok, void *ws,
                  size_t ws_bytes, hipStream_t stream) {
    (void)T;
    if (!onchip_fits(g) && !onchip_regular(g)) return LDPC_EUNSUPPORTED;
    if (ws == nullptr || ws_bytes < onchip_workspace_bytes(g, B)) return LDPC_EWORKSPACE;
    const int32_t early = test_period(flags);
    const int v = kernel_of(g, B, alpha != nullptr, early > 0);
    const KernelFn fn = kernel_fn(g, v, alpha != nullptr);
    const int threads = threads_for(g, kVariants[v]), per_wg = v >= kNumVariants ? 1 : 2 * kVariants[v].f;
    const size_t lds = lds_of(g, v);
    int grid = 0;
    constexpr int kDealt = 2; // frames dealt to each workgroup of a one-slot kernel
    int st = launch_grid((const void *)fn, threads, lds, g, B, g.tuned() ? g.tuning.wg_per_cu : 0, &grid, per_wg,
                         v >= kNumVariants ? kDealt : 0);
    if (st) return st;
    JobTable jt{};
    jt.njobs = 1;
    Job &J = jt.job[0] = make_job(g, v, llr, B, bits, post, iters, ok, alpha, beta, (uint32_t *)ws);
    deal(J, grid, kDealt);
    if (J.queue) k_zero_words<<<(kQueueWords + 255) / 256, 256, 0, stream>>>(J.queue, kQueueWords);
    timed_launch(K_ONCHIP, fn, grid, threads, lds, stream, jt, L, early);
    return hipGetLastError() == hipSuccess ? LDPC_OK : LDPC_EHIP;
}

size_t onchip_multi_workspace_bytes(int32_t njobs) {
    return align_up(4ull * kQueueWords * (size_t)(njobs > 0 ? njobs : 1), 256);
}

int onchip_decode_multi(const ldpc_job *jobs, int32_t njobs, int32_t L, uint32_t flags, void *ws, size_t ws_bytes,
                        hipStream_t stream) {
    if (njobs > kMaxJobs) return LDPC_EUNSUPPORTED;
    if (ws == nullptr || ws_bytes < onchip_multi_workspace_bytes(njobs)) return LDPC_EWORKSPACE;
    // largest jobs first, so the last frames of the shared launch come from small jobs
    std::vector<int32_t> order(njobs);
    for (int32_t k = 0; k < njobs; ++k) order[k] = k;
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
        return (int64_t)jobs[a].B * jobs[a].g->E > (int64_t)jobs[b].B * jobs[b].g->E;
    });
    // A job whose batch alone fills every CU at least once (by the runtime's
    // count: three of the eight codes at 0.07 of their batches 0.084 ms, 0.112
    // with the 430 frames of n = 2304 in a launch of their own, of which 256 run
    // at once and 512 by that count) gets a launch of its own kernel (its own LDS
    // size, workgroup size, register budget and tuned workgroups per CU); so does
    // a job that only the widest variant fits.  The other jobs share one
    // persistent launch, whose workgroup size and LDS are the maxima over them.
    constexpr int64_t kOwnLaunchRounds = 1;
    JobTable jt{};
    int threads = 64;
    size_t lds = 0;
    int64_t frames = 0;
    const ldpc_graph *any = nullptr; // one of the shared launch's
    uint32_t *queues = (uint32_t *)ws;
    struct Own {
        Job J;
        KernelFn fn;
        int threads;
        size_t lds;
        const ldpc_graph *g;
        int wg_per_cu; // tuned cap, 0 for none
    };
    std::vector<Own> own;
    Own sharer{};
    int32_t nj = 0;
    for (int32_t k = 0; k < njobs; ++k) {
        const ldpc_job &jb = jobs[order[k]];
        const ldpc_graph &g = *jb.g;
        if (!onchip_fits(g)) return LDPC_EUNSUPPORTED;
        if (jb.B == 0) continue;
        const int v_own = kernel_of(g, jb.B, false, test_period(flags) > 0, njobs > 1);
        int v = v_own;
        if (!shared_launch_ok(v)) // another variant that fits keeps the job eligible for the shared launch
            for (int c : kPickOrder)
                if (shared_launch_ok(c) && variant_ok(g, c)) {
                    v = c;
                    break;
                }
        const KernelFn fn = kernel_fn(g, v_own, false);
        const int t_own = threads_for(g, kVariants[v_own]);
        const size_t l_own = lds_of(g, v_own);
        bool alone = !shared_launch_ok(v);
        if (!alone) {
            int64_t room = 0;
            if (resident_workgroups((const void *)fn, t_own, l_own, g, &room) < 0) return LDPC_EHIP;
            const int64_t in_flight = room * kVariants[v_own].f;
            alone = (int64_t)jb.B >= kOwnLaunchRounds * in_flight;
        }
        own.push_back(Own{make_job(g, v_own, jb.llr_dev, jb.B, jb.bits_dev, jb.post_dev, jb.iters_dev, jb.ok_dev,
                                   nullptr, nullptr, queues + (size_t)k * kQueueWords),
                          fn, t_own, l_own, &g, g.tuned() ? g.tuning.wg_per_cu : 0});
        if (alone) continue;
        sharer = own.back();
        own.pop_back();
        const int t = threads_for(g, kVariants[v]);
        threads = t > threads ? t : threads;
        lds = lds_of(g, v) > lds ? lds_of(g, v) : lds;
        frames += jb.B;
        any = &g;
        jt.job[nj++] = make_job(g, v, jb.llr_dev, jb.B, jb.bits_dev, jb.post_dev, jb.iters_dev, jb.ok_dev, nullptr,
                                nullptr, queues + (size_t)k * kQueueWords);
    }
    // A job that would share with none runs its own kernel too (four frames of it
    // in turn to a workgroup otherwise: two quasi-cyclic codes, 1,638 and 51
    // frames, 0.158 ms with the 51 in the shared kernel, 0.132 in their own).
    if (nj == 1) {
        own.push_back(sharer);
        nj = 0;
        frames = 0;
    }
    jt.njobs = nj;
    const int32_t early = test_period(flags);
    if (frames == 0 && own.empty()) return LDPC_OK;
    k_zero_words<<<(njobs * kQueueWords + 255) / 256, 256, 0, stream>>>(queues, njobs * kQueueWords);
    // Jobs with a launch of their own that use the same kernel, workgroup size,
    // LDS size and workgroup cap (the same graph, or graphs of one shape) go
    // into one launch of it, in order (largest first), so that each job's last
    // frames overlap the next job's first ones.
    struct Launch {
        KernelFn fn;
        int threads;
        size_t lds;
        JobTable jt;
        const ldpc_graph *g;
        int64_t frames;
        int wg_per_cu, per_wg, grid;
    };
    std::vector<Launch> launches;
    std::vector<bool> placed(own.size(), false);
    for (size_t a = 0; a < own.size(); ++a) {
        if (placed[a]) continue;
        JobTable ot{};
        int t = 0;
        size_t l = 0;
        int64_t fr = 0;
        for (size_t b = a; b < own.size(); ++b) {
            if (placed[b] || own[b].fn != own[a].fn || own[b].wg_per_cu != own[a].wg_per_cu ||
                own[b].threads != own[a].threads || own[b].lds != own[a].lds)
                continue;
            placed[b] = true;
            ot.job[ot.njobs++] = own[b].J;
            t = own[b].threads > t ? own[b].threads : t;
            l = own[b].lds > l ? own[b].lds : l;
            fr += own[b].J.B;
        }
        const int per_wg = ot.njobs == 1 && own[a].J.variant >= kNumVariants ? 1 : 2 * kVariants[own[a].J.variant].f;
        launches.push_back(Launch{own[a].fn, t, l, ot, own[a].g, fr, own[a].wg_per_cu, per_wg, 0});
    }
    if (frames > 0) launches.push_back(Launch{k_onchip_multi, threads, lds, jt, any, frames, 0, 4, 0});
    // Several launches run side by side: all but the first go round-robin to
    // the library's side streams of the device, which wait for everything
    // enqueued on `stream` so far and which `stream` waits for at the end.
    // Each launch's last frames (and the shared launch of small jobs) then
    // overlap the others instead of leaving CUs idle.
    const bool among = launches.size() > 1;
    for (Launch &x : launches) {
        const int rounds = among ? 1 : 2; // dealt to each workgroup of a one-slot kernel for one job
        const int st = launch_grid((const void *)x.fn, x.threads, x.lds, *x.g, x.frames, x.wg_per_cu, &x.grid, x.per_wg,
                                   x.per_wg == 1 ? rounds : 0, among);
        if (st) return st;
        if (x.jt.njobs == 1) deal(x.jt.job[0], x.grid, rounds);
    }
    SideStreams *side = among ? side_streams() : nullptr;
    const int sides = (int)std::min<size_t>(kSideStreams, launches.size() - 1); // of the side streams, those in use
    std::unique_lock<std::mutex> hold;
    if (side) {
        hold = std::unique_lock<std::mutex>(side->mu);
        LDPC_HIP_TRY(hipEventRecord(side->fork, stream));
        for (int k = 0; k < sides; ++k) LDPC_HIP_TRY(hipStreamWaitEvent(side->s[k], side->fork, 0));
    }
    for (size_t k = 0; k < launches.size(); ++k) {
        const Launch &x = launches[k];
        const hipStream_t on = (side && k % (kSideStreams + 1) != 0) ? side->s[k % (kSideStreams + 1) - 1] : stream;
        timed_launch(K_ONCHIP, x.fn, x.grid, x.threads, x.lds, on, x.jt, L, early);
    }
    if (side) {
        for (int k = 0; k < sides; ++k) {
            LDPC_HIP_TRY(hipEventRecord(side->join[k], side->s[k]));
            LDPC_HIP_TRY(hipStreamWaitEvent(stream, side->join[k], 0));
        }
    }
    return hipGetLastError() == hipSuccess ? LDPC_OK : LDPC_EHIP;
}

} // namespace ldpc
