// The persistent fire-growth kernel.
//
// Model (Sections 3.1 and 3.4, Algorithm 1 Step 2).  Once a cell ignites at
// minute a, its fire advances q_k(p) metres along axis k in each later minute
// of period p (the FBP rates of the cell in that period through eq. (1)),
// and reaches neighbour k once the distance D_k between the two centres is
// covered.  The neighbour ignites in that minute if its own head rate passes
// the threshold, else at the start of the first later period that passes
// (the message persists).  Every hop takes at least one minute and rates do
// not depend on the order of ignitions, so the arrival minutes are the least
// solution of arrival(j) = min_i accept_j(reach_ij(arrival(i))): any
// evaluation order that only commits arrivals of the current period and
// carries per-axis progress across period ends gives exactly the minute-
// stepping result.
//
// Work decomposition.  One work group per replication (persistent groups
// take replications from a counter).  Per weather period p:
//   - cells waiting for a passing rate (pending) are re-tested;
//   - cells whose axes were still travelling at the end of p-1
//     (continuations, with the metres left on each axis) are advanced
//     through p, those listed last (lit latest, at the fire front) first;
//   - label correcting: each cell that received a smaller arrival in p is
//     advanced from that minute to the end of p.
// The period's weather rows and the coefficient tables are read from LDS.
// Advancing a cell through a period costs one FBP evaluation; axes that
// reach their neighbour inside p offer that minute with atomicMin on the
// neighbour's 32-bit label, the rest become a continuation for p+1.
// Improved cells go to the period's work queue (LDS, spilling to the slot's
// global list): each wave reserves a range with one LDS atomic, writes its
// entries and commits the range in reservation order; waves take committed
// chunks of up to 16 entries as soon as they are free, so no wave waits for
// the others between hops.  The period ends when no wave holds a chunk and
// every reserved entry has been taken.
//
// Lanes a cell.  The kernel is bound by a chain of dependent passes (a hop of
// the fire front is one) and, with many replications, by vector instructions.
// A narrow pass gives a cell to four lanes, 16 cells a pass: each lane takes
// two opposite axes, and the three rate curves and three random blocks of a
// cell run side by side.  It takes about 620 vector instructions and, alone on
// its SIMD, 3 thousand cycles of evaluation, 2 thousand of loads, 1 thousand
// of label atomics and 1.7 thousand of appends.  A wide pass gives a cell to
// one lane, 64 cells a pass, in about 1100 instructions, so it costs half as
// many a cell but takes longer from a cell's arrival to its neighbours'.
// Continuations go wide when there are more of them than the group's waves
// take in one narrow pass, queue entries when more than 32 are waiting and the
// idle waves could not take them all narrow.  FP64 evaluations are called from
// narrow passes only: inlined, or called from wide ones, their constants and
// the registers saved around the call made the loop spill.
// Against one lane a cell throughout with inlined FP64 code (1900 instructions
// a pass at 40 cells on average, 256 registers, 8 waves a compute unit), in ms:
// 8192^2 x 64 replications x 72 periods 7.70 -> 4.50, 1024^2 x 2048 x 48
// 39.1 -> 19.6, one FP32 fire on 2048^2 x 48 3.61 -> 2.23, 20 x 20 cells x 10
// 0.24 -> 0.13.  Drawing the random part (three Philox blocks, the noise)
// between a pass's loads and their first use, and loading in every lane: 6.91 ->
// 6.25 and 13.8 -> 12.9 on other weather of the first two.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device.h"
#include "kernels.h"
#include "types.h"

namespace c2f {

constexpr int32_t kNever = 0x7FFFFFFF;
typedef __attribute__((address_space(1))) CellRec GCellRec;

constexpr int kChunk = 16;   // cells a wave takes at a time, four lanes each
// More queue entries than this may be taken as one pass of one lane each
// (1024^2 x 2048 replications x 48 periods: 13.9 ms at 24, 32 and 47).
constexpr int kWideMin = 32;

// Had the cell not burned when it held label v (an older tag, or pending)?
__device__ __forceinline__ bool unburned(uint32_t v, uint32_t tag) {
    return (v >> kMinuteBits) != tag || (v & kMinuteMask) == kPendingMinute;
}

__device__ __forceinline__ uint32_t load_label(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int wave_rank(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Value of x in lane `lane` (wave-uniform) without a trip through LDS.
__device__ __forceinline__ int lane_value(int x, int lane) { return __builtin_amdgcn_readlane(x, lane); }

// One LDS atomic per wave reserves slots for the appending lanes.
__device__ __forceinline__ int wave_reserve(bool pred, int* counter, uint64_t& m) {
    m = __ballot(pred);
    if (m == 0) return 0;
    const int leader = __ffsll((unsigned long long)m) - 1;
    int base = 0;
    if (__lane_id() == leader) base = atomicAdd(counter, (int)__popcll(m));
    return lane_value(base, leader) + wave_rank(m);
}

template <typename T>
__device__ __forceinline__ void append_g(bool pred, const T& val, T* glob, uint32_t cap, int* counter, int* flag) {
    uint64_t m;
    const int idx = wave_reserve(pred, counter, m);
    if (pred) {
        if ((uint32_t)idx < cap) glob[idx] = val;
        else *flag = 1;
    }
}


// ceil(r / q) for 0 < q < r < 2^16.  The float quotient x = r rcp(q) (rcp
// within one ulp) differs from r / q by less than (r / q) 2^-22, which is
// below 1 / q because r < 2^22.  With r / q = k + f: for f = 0, x lies in
// (k - 1, k + 1) and truncates to k - 1 or k; for f >= 1 / q, x lies in
// (k, k + 1) and truncates to k.  One exact 24-bit product then takes the
// truncation up to ceil(r / q) where it is one short.
__device__ __forceinline__ int32_t ceil_div_small(int32_t r, int32_t q) {
    uint32_t t = (uint32_t)((float)r * __builtin_amdgcn_rcpf((float)q));
    t += __umul24(t, (uint32_t)q) < (uint32_t)r;
    return (int32_t)t;
}

// One axis of a cell advanced through the n minutes left of a period at the
// integer rate q: rem > 0 holds the metres left and is below 2^16 (at most the
// diagonal of a 20 km cell).  Returns the number of minutes the fire needs to
// reach the neighbour (1..n, rem becomes 0), or 0 if it does not in this
// period.
__device__ __forceinline__ int32_t step_axis(int32_t q, int32_t& rem, int32_t n) {
    // 1 where q >= rem: the quotient truncates to 0, which the correction takes
    // to 1 (24 bits of q hold enough: the product is 0), or to 1, and then q is
    // below 2^17
    const int32_t t = ceil_div_small(rem, max(q, 1));
    const bool reach = q > 0 && t <= n;
    // q n < rem < 2^16 when the neighbour is not reached
    rem = reach ? 0 : rem - (int32_t)__umul24((uint32_t)q, (uint32_t)n);
    return reach ? t : 0;
}

__device__ __forceinline__ CellRec load_rec(const GCellRec* p) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(1))) const u32x4 g4;
    const u32x4 a = ((g4*)p)[0], b = ((g4*)p)[1];
    CellRec r;
    r.info = a.x;
    r.grad = a.y;
    r.ux = __uint_as_float(a.z);
    r.uy = __uint_as_float(a.w);
    r.sfc = __hiloint2double((int)b.y, (int)b.x);
    r.sfd = __hiloint2double((int)b.w, (int)b.z);
    return r;
}

// Is an axis with rem metres left still worth following from minute m0?  d is
// the neighbour's label less the tag's part: its minute if it has burned in
// this replication, kPendingMinute if it waits for a passing rate (its
// ignition minute is then already determined), more if it has not burned.  No
// once the neighbour holds a label no later candidate can beat.
__device__ __forceinline__ bool axis_live(int32_t rem, uint32_t d, int32_t m0) {
    return rem > 0 && d > (uint32_t)m0 && d != kPendingMinute;
}

// Up to 95 VGPRs are used, so 5 waves a SIMD would fit; groups of 256 threads are the
// ones whose LDS then takes five a compute unit (queues of 2048 entries), and
// are built for it, wider ones for 4.  At 5 against 4 groups of 256 a unit:
// 64^2 x 5000 replications x 24 periods 2.49 against 2.82 ms, 256^2 x 4800 x 48
// 9.47 against 10.44, 512^2 x 4800 x 48 13.5 against 14.7; at five replications
// a unit and fewer it is no faster (128^2 x 1280 x 24: 1.50 against 1.41).
// (With narrow passes alone, 6 and 8 waves spilled 144 and 208 bytes a lane and
// were 22 and 60 % slower at 1024 threads.)
template <typename R, int BLOCK>
__global__ __launch_bounds__(BLOCK, BLOCK == 256 ? 5 : 4) void propagate_kernel(const Job* __restrict__ jobs, int n_jobs,
                                                          int total_items, Slots slots,
                                                          RunCounters* __restrict__ rc) {
    constexpr int LQ = BLOCK <= 64 ? 1024 : (BLOCK <= 256 ? 2048 : 4096);   // LDS part of the period queue
    __shared__ uint2 s_Q[LQ];
    __shared__ int s_res, s_commit;   // queue entries reserved, committed (in order)
    // queue entries taken (high 32 bits) and waves holding a chunk (low 32),
    // one word so that taking a chunk and becoming a holder is one step
    __shared__ unsigned long long s_hb;
    __shared__ int s_nC[2], s_nP[2];
    __shared__ int s_ctake;           // continuations taken
    __shared__ int s_item, s_flag;
    __shared__ uint32_t s_tag;
    __shared__ int s_scen, s_ign;
    // Decisions that steer every wave through the same barriers.  Each is
    // written by thread 0 only between two barriers and read by all
    // threads after the second, so no wave can read a value meant for a
    // later step: s_refill (the slot's plane needs refilling) and s_stop
    // (leave the period loop after this period).
    __shared__ int s_refill, s_stop;
    // of the replication, and of all the group has run: its replications' sums
    // go to the launch's counters together.  Nine device atomics a replication,
    // all on one line, were most of a launch of many short fires: 5000 fires of
    // 20^2 that hardly spread took 0.77 ms, 0.15 with the sums; 300 took 57 and
    // 34 us.
    __shared__ unsigned long long s_cnt[kNumCounters], s_sum[kNumCounters];
    // what the evaluations read: the curves, the weather rows of the period
    // being propagated (staged at the start of each period) and the
    // landscape's constants, in both precisions
    __shared__ EvalLds<double> s_x64;
    __shared__ EvalLds<float> s_x32;
    __shared__ EvalRep s_e;

    constexpr int NW = BLOCK / 64;
    const int tid = threadIdx.x;
    const int slot = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int quad = (tid & 63) >> 2, role = tid & 3;   // the lane's cell of a chunk, its axes there
    __builtin_amdgcn_s_setprio(1);
    if (tid < kNumCounters) s_sum[tid] = 0;
    if (tid < kNumCurves) {
        s_x64.coef[tid] = curve_entry<double>(tid);
        s_x32.coef[tid] = curve_entry<float>(tid);
    }
    uint32_t* __restrict__ plane = slots.planes + (size_t)slot * (size_t)slots.plane_cells;
    const int64_t stride = slots.list_cap;   // entries allocated per list
    const uint32_t cap = (uint32_t)slots.list_limit;   // entries used per list (<= stride, <= 2^30)
    uint8_t* lb = slots.lists + (size_t)slot * (size_t)stride * (size_t)kSlotListBytesPerEntry;
    uint2* const gQ = (uint2*)lb;        // global part of the period queue: 2 x cap entries
    // continuation and pending lists, one of each pair current
    auto gC = [&](int w) __attribute__((always_inline)) { return (Cont*)(lb + 16 * stride) + (w ? stride : 0); };
    auto gP = [&](int w) __attribute__((always_inline)) { return (uint32_t*)(lb + 64 * stride) + (w ? stride : 0); };

    for (int taken = 0;; ++taken) {
        // With deferred dense outputs (item_slot set) a slot's plane must
        // still hold its item's labels when the launch ends, so a group runs
        // at most one item; the launch then has a group for every item.
        if (slots.item_slot && taken > 0) break;
        if (tid == 0) {
            int it = atomicAdd(&rc->next_item, 1);
            if (__hip_atomic_load(&rc->overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) it = total_items;
            else if (slots.order && it < total_items) it = slots.order[it];
            s_item = it;
        }
        __syncthreads();
        // values every thread reads from LDS after a barrier are the same in
        // every lane: readfirstlane tells the compiler so, which keeps the
        // job record and everything derived from it in scalar registers
        const int item = __builtin_amdgcn_readfirstlane(s_item);
        if (item >= total_items) break;

        // job lookup (jobs are sorted by item_base)
        int lo = 0, hi = n_jobs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (jobs[mid].item_base <= item) lo = mid;
            else hi = mid - 1;
        }
        const Job& job = jobs[lo];
        const int lr = item - job.item_base;
        const uint32_t rep = (uint32_t)(job.rep_offset + lr);
        const int cols = job.cols;
        const int rows = job.rows;
        const int P = job.period_min;
        // a global pointer: loads through a generic one wait on LDS as well
        const GCellRec* const cells = (const GCellRec*)job.cells;
        const bool use_thr = job.threshold > 0.0f;
        const R thr = (R)job.threshold;
        // the lane's axes `role` and `role` + 4: centre distance, and the
        // neighbours' index offsets offk and -offk
        const int32_t Dk = (role & 1) ? job.d_diag : job.d_orth;
        const int32_t offk = role == 0 ? 1 : role == 1 ? 1 - cols : role == 2 ? -cols : -cols - 1;
        const uint32_t last_cell = (uint32_t)((int64_t)rows * cols - 1);

        // ------------------------------------------- replication set-up
        if (tid < kNumFuels) {
            load_land<double>(job.land, s_x64.L, tid);
            load_land<float>(job.land, s_x32.L, tid);
        }
        if (tid == 0) {
            const uint32_t prev = slots.tags[slot];
            s_refill = prev <= 1u;   // tags exhausted: refill this slot's plane
            s_tag = prev <= 1u ? kTagFresh : prev;
            s_res = s_commit = 0;
            s_hb = 0ull;
            s_nC[0] = s_nC[1] = s_nP[0] = s_nP[1] = 0;
            s_ctake = 0;
            s_flag = 0;
            s_stop = 0;
            for (int k = 0; k < kNumCounters; ++k) s_cnt[k] = 0;
            int scen, ign;
            rep_draws(job, rep, scen, ign);
            s_scen = scen;
            s_ign = ign;
            s_e = EvalRep{job.seed, rep, job.rounding, job.sigma, job.hfi_min, 0.f};
        }
        __syncthreads();
        if (s_refill) {
            for (size_t i = tid; i < (size_t)slots.plane_cells; i += BLOCK) plane[i] = kPlaneFill;
            __syncthreads();
        }
        if (tid == 0) {
            const uint32_t tag = s_tag - 1u;
            s_tag = tag;
            slots.tags[slot] = tag;
            const int ign = s_ign;
            if (job.ign_mode != 4 && ign >= 0 && rec_fuel(cells[ign].info) != 0) {
                // the ignition takes the last minute before its period
                const uint32_t v = (tag << kMinuteBits) | (uint32_t)(job.ign_period * P);
                plane[ign] = v;
                s_Q[0] = make_uint2((uint32_t)ign, v);
                s_res = s_commit = 1;
                s_cnt[kCntIgnitions] = 1;
                if (job.count) atomicAdd(&job.count[ign], 1u);
            }
        }
        __syncthreads();
        const uint32_t tag = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_tag);
        const int scen_r = __builtin_amdgcn_readfirstlane(s_scen);
        const uint32_t pendv = (tag << kMinuteBits) | kPendingMinute;
        const size_t so = (size_t)scen_r * job.n_wp * kRowLen;
        const double* const g_rows64 = job.table64 + so;
        const R* const g_rows = (const R*)job.table + so;   // in the precision of the results
        const EvalRep erep{job.seed, rep, job.rounding, job.sigma, job.hfi_min, mix_margin(job.sigma)};
        const float burnout = job.burnout;
        // a global pointer: through a generic one each count would wait on
        // LDS and memory both
        typedef __attribute__((address_space(1))) uint32_t gu32;
        gu32* const count = (gu32*)job.count;
        auto count_one = [&](uint32_t j) __attribute__((always_inline)) {
            (void)__hip_atomic_fetch_add(count + j, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        // the receiving cell's ignition test: its head rate exceeds the threshold
        auto ignites = [&](uint32_t j, int p) __attribute__((always_inline)) {
            if constexpr (sizeof(R) == 8) return head_rate_lds<double>(&s_x64, &s_x64, &s_e, job.cells, j, (uint32_t)p) > thr;
            else return head_rate_lds<float>(&s_x32, &s_x64, &s_e, job.cells, j, (uint32_t)p) > thr;
        };

        uint32_t c_entries = 0, c_conts = 0, c_evals = 0, c_cand = 0, c_impr = 0, c_ign = 0, c_rounds = 0;
        int max_list = 0;
        int cc = 0, pc = 0;   // which buffer of each list pair is current

        // Append one entry per lane where `pred` holds: one reservation per
        // wave, entries written, then the range committed in reservation
        // order (earlier reservations never wait on later ones).  Called in
        // wave-uniform control flow.
        auto q_commit = [&](int wbase, int wtot) __attribute__((always_inline)) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            if (__lane_id() == 0) {
                while (__hip_atomic_load(&s_commit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != wbase)
                    __builtin_amdgcn_s_sleep(1);
                __hip_atomic_store(&s_commit, wbase + wtot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        };
        auto q_put = [&](int idx, uint2 val) __attribute__((always_inline)) {
            if (idx < LQ) s_Q[idx] = val;
            else if ((uint32_t)(idx - LQ) < 2 * cap) gQ[idx - LQ] = val;
            else s_flag = 1;
        };
        auto q_append1 = [&](bool pred, uint2 val) __attribute__((always_inline)) {
            const uint64_t m = __ballot(pred);
            if (m == 0) return;
            int wbase = 0;
            if (__lane_id() == 0) wbase = atomicAdd(&s_res, (int)__popcll(m));
            wbase = lane_value(wbase, 0);
            if (pred) q_put(wbase + wave_rank(m), val);
            q_commit(wbase, (int)__popcll(m));
        };

        // the list's entries are sorted by period and the loop starts at the
        // earliest, so the entries of period p are those with period p, and
        // none is still to come after the last entry's period: both follow
        // from p alone, which every thread knows
        const int last_seed_period = job.n_seeds > 0 ? job.seeds[job.n_seeds - 1].y : -1;
        for (int p = job.ign_period; p < job.n_periods; ++p) {
            // list ignitions of period p take minute p P, inside or outside
            // the burning window, on cells with fuel that have not burned
            // (a pending cell included).  Lit by one thread between periods,
            // when no other thread touches the plane or the queue; an
            // improved label joins the queue like the set-up ignition.
            if (p <= last_seed_period && seeds_at(job, p)) {
                if (tid == 0) {
                    for (int k = 0; k < job.n_seeds; ++k) {
                        if (job.seeds[k].y != p) continue;
                        const uint32_t c = (uint32_t)job.seeds[k].x;
                        if (rec_fuel(cells[c].info) == 0) continue;
                        const uint32_t v = (tag << kMinuteBits) | (uint32_t)(job.seeds[k].y * P);
                        const uint32_t old = atomicMin(&plane[c], v);
                        if (v < old) {
                            if (unburned(old, tag)) {
                                ++c_ign;
                                if (job.count) atomicAdd(&job.count[c], 1u);
                            }
                            q_put(s_res, make_uint2(c, v));
                            s_commit = ++s_res;
                        }
                    }
                }
                __syncthreads();
            }
            // outside the daily burning window nothing spreads or ignites:
            // the continuations and pending cells wait, unchanged
            if (!burning_period(job, p)) continue;
            // every wave has left the previous period (its end barriers)
            for (int i = tid; i < kRowLen; i += BLOCK) {
                s_x64.row[i] = g_rows64[(size_t)p * kRowLen + i];
                s_x32.row[i] = (float)g_rows[(size_t)p * kRowLen + i];
            }
            __syncthreads();
            const int32_t s = p * P + 1;   // first minute of period p
            const int32_t e = (p + 1) * P; // last minute of period p

            // Each wave counts as a holder of the queue until it has done its
            // share of the pending cells and continuations below, so that no
            // wave finds the queue drained while another may still append to
            // it.  The waves then join the queue without a barrier: a wave
            // done early takes entries while others still advance
            // continuations (the labels are a least fixed point, whatever
            // the order).
            if (__lane_id() == 0) atomicAdd(&s_hb, 1ull);
            // Pending cells ignite at the start of p if their rate now passes;
            // the new labels join this period's queue.
            {
                const int nP = min(s_nP[pc], (int)cap);
                for (int base = 0; base < nP; base += BLOCK) {
                    const int i = base + tid;
                    bool act = i < nP;
                    uint32_t j = 0;
                    if (act) {
                        j = gP(pc)[i];
                        act = load_label(&plane[j]) == pendv;
                    }
                    bool ok = false;
                    if (act) {
                        ++c_evals;
                        ok = ignites(j, p);
                    }
                    bool improved = false, first = false;
                    const uint32_t v = (tag << kMinuteBits) | (uint32_t)s;
                    if (ok) {
                        const uint32_t old = atomicMin(&plane[j], v);
                        improved = v < old;
                        first = improved && unburned(old, tag);
                        if (first && count) count_one(j);
                    }
                    c_impr += (uint32_t)__popcll(__ballot(improved));
                    c_ign += (uint32_t)__popcll(__ballot(first));
                    q_append1(improved, make_uint2(j, v));
                    append_g(act && !ok, j, gP(pc ^ 1), cap, &s_nP[pc ^ 1], &s_flag);
                }
            }
            // The waves' loop over the period's work: chunks of up to 16
            // cells, four lanes a cell.  First the continuations of p-1 from
            // the start of p, last listed first: the cells listed last were
            // lit latest in p-1, at the front of the fire, and tend to start
            // the longest chains of p, which then reach the queue in the
            // first rounds.  Then label correcting over the period's queue:
            // cells whose arrival improved inside p, advanced from that
            // minute.  Labels are a least fixed point whatever the order.  A
            // wave waiting for entries drops to the lowest issue priority, so
            // that its polling takes no issue slots from the waves working on
            // the chain.
            const int n_conts = min(s_nC[cc], (int)cap);
            if (n_conts > max_list) max_list = n_conts;
            bool conts = true;
            const int csize = n_conts > kChunk * NW && !use_thr ? 64 : kChunk;
            int cbase = wave * csize;   // the first chunk of continuations by wave, later ones from s_ctake
            uint64_t redo = 0;   // lanes of the last one-lane pass whose cells a quad takes
            int base = 0;
            for (;;) {
                int cnt = 0;
                const bool again = redo != 0;
                if (again) {
                    cnt = min((int)__popcll(redo), kChunk);
                } else if (conts) {
                    if (cbase >= n_conts) {
                        conts = false;
                        if (__lane_id() == 0) atomicAdd(&s_hb, ~0ull);   // no longer a holder
                        continue;
                    }
                    base = cbase;
                    cnt = min(csize, n_conts - base);
                } else {
                    bool done = false;
                    base = 0;
                    __builtin_amdgcn_s_setprio(0);
                    if (__lane_id() == 0) {
                        for (;;) {
                            if (__hip_atomic_load(&s_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) {
                                done = true;
                                break;
                            }
                            const unsigned long long hb =
                                __hip_atomic_load(&s_hb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            const int h = (int)(hb >> 32), holders = (int)(uint32_t)hb;
                            const int cm =
                                __hip_atomic_load(&s_commit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            if (h < cm) {
                                const int avail = cm - h;
                                const bool many = avail > kWideMin && avail > kChunk * (NW - holders) && !use_thr;
                                const int take = min(many ? 64 : kChunk, avail);
                                const unsigned long long nhb = ((unsigned long long)(uint32_t)(h + take) << 32) |
                                                               (unsigned long long)(uint32_t)(holders + 1);
                                if (atomicCAS(&s_hb, hb, nhb) == hb) {
                                    base = h;
                                    cnt = take;
                                    break;
                                }
                                continue;
                            }
                            // finished when no wave holds a chunk (so none can
                            // append) and every reserved entry has been taken
                            const int rs =
                                __hip_atomic_load(&s_res, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            if (holders == 0 && h == cm && cm == rs) {
                                done = true;
                                break;
                            }
                            __builtin_amdgcn_s_sleep(1);
                        }
                    }
                    base = lane_value(base, 0);
                    cnt = lane_value(cnt, 0);
                    done = lane_value((int)done, 0) != 0;
                    __builtin_amdgcn_s_setprio(1);
                    if (done) break;
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                    ++c_rounds;
                }

                if (!again) {
                    if (conts) c_conts += (uint32_t)cnt;
                    else c_entries += (uint32_t)cnt;
                }
                if (cnt > kChunk) {
                    // one lane a cell; cells that need FP64 are set aside in
                    // `redo` for quads
                    const int lane = (int)__lane_id();
                    const int i = base + lane;
                    bool act = lane < cnt && (conts || i < LQ || (uint32_t)(i - LQ) < 2 * cap);
                    uint32_t c = 0, lab = 0;
                    uint32_t rem[4] = {0u, 0u, 0u, 0u};   // metres left, axis k low and k + 4 high
                    if (act) {
                        if (conts) {
                            const uint2* ct = (const uint2*)(gC(cc) + (n_conts - 1 - i));
                            const uint2 a = ct[0], r0 = ct[1], r1 = ct[2];
                            c = a.x;
                            lab = a.y;
                            rem[0] = r0.x, rem[1] = r0.y, rem[2] = r1.x, rem[3] = r1.y;
                        } else {
                            uint2 ent;
                            if (i < LQ) {
                                ent = s_Q[i];
                            } else {
                                const uint64_t v = __hip_atomic_load((const uint64_t*)&gQ[i - LQ], __ATOMIC_RELAXED,
                                                                     __HIP_MEMORY_SCOPE_AGENT);
                                ent = make_uint2((uint32_t)v, (uint32_t)(v >> 32));
                            }
                            c = ent.x;
                            lab = ent.y;
                            rem[0] = rem[2] = (uint32_t)job.d_orth * 0x10001u;
                            rem[1] = rem[3] = (uint32_t)job.d_diag * 0x10001u;
                        }
                    }
                    const int off[4] = {1, 1 - cols, -cols, -cols - 1};
                    // every lane loads (an empty one cell 0): a branch here
                    // would copy the loads' registers behind it and wait
                    const uint32_t own = load_label(&plane[c]);
                    const CellRec rec = load_rec(cells + c);
                    uint32_t v[8];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        v[k] = plane[min(c + (uint32_t)off[k], last_cell)];
                        v[k + 4] = plane[min(c - (uint32_t)off[k], last_cell)];
                    }
                    // the random part while the loads are on their way (the
                    // empty asm keeps it there: it would sink to its use)
                    uint32_t w[8];
                    float mu = lane_draws<sizeof(R) == 8>(erep, c, (uint32_t)p, w);
                    asm volatile("" : "+v"(mu), "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(w[4]), "+v"(w[5]),
                                 "+v"(w[6]), "+v"(w[7]));
                    act = act && own == lab;
                    const int32_t m0 = max((int32_t)(lab & kMinuteMask) + 1, s);
                    const uint32_t nb = act ? rec_nbmask(rec.info) : 0u;
                    uint32_t settled = 0;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const uint32_t dA = v[k] - (tag << kMinuteBits), dB = v[k + 4] - (tag << kMinuteBits);
                        const bool a = ((nb >> k) & 1u) && axis_live((int32_t)(rem[k] & 0xFFFFu), dA, m0);
                        const bool b = ((nb >> (k + 4)) & 1u) && axis_live((int32_t)(rem[k] >> 16), dB, m0);
                        rem[k] = (a ? rem[k] & 0xFFFFu : 0u) | (b ? rem[k] & 0xFFFF0000u : 0u);
                        settled |= (dA <= (uint32_t)(e + 1) ? 1u << k : 0u) | (dB <= (uint32_t)(e + 1) ? 16u << k : 0u);
                    }
                    const bool want = (rem[0] | rem[1] | rem[2] | rem[3]) != 0u && m0 <= e;
                    int32_t t[8];   // minutes to the neighbour, 0 = not reached in p
#pragma unroll
                    for (int k = 0; k < 8; ++k) t[k] = 0;
                    if (__any(want)) {
                        int32_t q[8];
                        bool done;
                        bool out = lane_axis_q<sizeof(R) == 8>(s_x32, erep, rec, mu, w, q, done);
                        redo = __ballot(want && !done);
                        if (want && !done) rem[0] = rem[1] = rem[2] = rem[3] = 0u;
                        if (want && done) {
                            ++c_evals;
                            if (burnout > 0.f) {
                                int32_t qm = 0;
#pragma unroll
                                for (int k = 0; k < 8; ++k) qm = max(qm, (nb >> k) & 1u ? q[k] : 0);
                                out = out || (double)qm < (double)burnout;
                            }
                            const int32_t n = e - m0 + 1;
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                int32_t rA = out ? 0 : (int32_t)(rem[k] & 0xFFFFu), rB = out ? 0 : (int32_t)(rem[k] >> 16);
                                if (rA > 0) t[k] = step_axis(q[k], rA, n);
                                if (rB > 0) t[k + 4] = step_axis(q[k + 4], rB, n);
                                if ((settled >> k) & 1u) rA = 0;
                                if ((settled >> k) & 16u) rB = 0;
                                rem[k] = (uint32_t)rA | ((uint32_t)rB << 16);
                            }
                        }
                    }
                    const bool keep = (rem[0] | rem[1] | rem[2] | rem[3]) != 0u;
                    const uint32_t lab0 = (tag << kMinuteBits) | (uint32_t)(m0 - 1);   // + t: the neighbour's label
                    uint32_t old[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        old[k] = 0u;   // not offered: nothing is below 0
                        const uint32_t j = k < 4 ? c + (uint32_t)off[k & 3] : c - (uint32_t)off[k & 3];
                        if (t[k] != 0) old[k] = atomicMin(&plane[j], lab0 + (uint32_t)t[k]);
                    }
                    uint32_t impr = 0, first = 0;
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const bool i_k = lab0 + (uint32_t)t[k] < old[k];
                        impr |= i_k ? 1u << k : 0u;
                        first |= i_k && unburned(old[k], tag) ? 1u << k : 0u;
                        c_cand += (uint32_t)__popcll(__ballot(t[k] != 0));
                    }
                    uint64_t am[8];
                    int wtot = 0;
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        am[k] = __ballot((impr >> k) & 1u);
                        wtot += (int)__popcll(am[k]);
                    }
                    const uint64_t mk = __ballot(keep);
                    const int ktot = (int)__popcll(mk);
                    if ((wtot | ktot) != 0) {
                        int got = 0;
                        if (lane < 2) got = atomicAdd(lane == 0 ? &s_res : &s_nC[cc ^ 1], lane == 0 ? wtot : ktot);
                        const int wbase = lane_value(got, 0), kbase = lane_value(got, 1);
                        if (wtot > 0) {
                            int idx = wbase;
#pragma unroll
                            for (int k = 0; k < 8; ++k) {
                                const uint32_t j = k < 4 ? c + (uint32_t)off[k & 3] : c - (uint32_t)off[k & 3];
                                if ((impr >> k) & 1u) q_put(idx + wave_rank(am[k]), make_uint2(j, lab0 + (uint32_t)t[k]));
                                idx += (int)__popcll(am[k]);
                            }
                            q_commit(wbase, wtot);
                            c_impr += (uint32_t)wtot;
#pragma unroll
                            for (int k = 0; k < 8; ++k) {
                                const uint32_t j = k < 4 ? c + (uint32_t)off[k & 3] : c - (uint32_t)off[k & 3];
                                const bool f = (first >> k) & 1u;
                                c_ign += (uint32_t)__popcll(__ballot(f));
                                if (count && f) count_one(j);
                            }
                        }
                        const int k = kbase + wave_rank(mk);
                        if (keep) {
                            if ((uint32_t)k < cap) {
                                uint2* ct = (uint2*)(gC(cc ^ 1) + k);
                                ct[0] = make_uint2(c, lab);
                                ct[1] = make_uint2(rem[0], rem[1]);
                                ct[2] = make_uint2(rem[2], rem[3]);
                            } else {
                                s_flag = 1;
                            }
                        }
                    }
                } else {
                    // the quad's entry: cell, label, metres left on the lane's
                    // two axes (a cell lit in p starts with the whole distance)
                    int i = base + quad;
                    if (again) {
                        for (int j = 0; j < cnt; ++j) {
                            if (quad == j) i = base + __ffsll((unsigned long long)redo) - 1;
                            redo &= redo - 1;
                        }
                    }
                    bool act = quad < cnt && (conts || i < LQ || (uint32_t)(i - LQ) < 2 * cap);
                    uint32_t c = 0, lab = 0;
                    int32_t remA = 0, remB = 0;
                    if (act) {
                        if (conts) {
                            const Cont* ct = gC(cc) + (n_conts - 1 - i);
                            const uint32_t rr = ct->rem[role];
                            c = ct->c;
                            lab = ct->label;
                            remA = (int32_t)(rr & 0xFFFFu);
                            remB = (int32_t)(rr >> 16);
                        } else {
                            uint2 ent;
                            if (i < LQ) {
                                ent = s_Q[i];
                            } else {
                                const uint64_t v = __hip_atomic_load((const uint64_t*)&gQ[i - LQ], __ATOMIC_RELAXED,
                                                                     __HIP_MEMORY_SCOPE_AGENT);
                                ent = make_uint2((uint32_t)v, (uint32_t)(v >> 32));
                            }
                            c = ent.x;
                            lab = ent.y;
                            remA = remB = Dk;
                        }
                    }

                    // issue every load of the entry at once: own label, cell
                    // record and the labels of the lane's two neighbours.  A
                    // neighbour outside the grid is read at an index clamped into
                    // the plane (an index below 0 wraps to a large unsigned value
                    // and clamps too) and never used: the record's neighbour mask
                    // (in-grid burnable cells) excludes its axis.  Grids hold
                    // fewer than 2^31 cells.
                    const uint32_t cA = c + (uint32_t)offk, cB = c - (uint32_t)offk;
                    uint32_t own = load_label(&plane[c]);
                    const CellRec rec = load_rec(cells + c);
                    const uint32_t vA = plane[min(cA, last_cell)], vB = plane[min(cB, last_cell)];
                    // the random part while the loads are on their way
                    // (the empty asm keeps it there: it would sink to its use)
                    QuadDraws draws = quad_draws<sizeof(R) == 8>(erep, c, (uint32_t)p, role);
                    asm volatile("" : "+v"(draws.mu), "+v"(draws.w.n1), "+v"(draws.w.n2), "+v"(draws.w.wa), "+v"(draws.w.wb));
                    // other waves lower the label meanwhile, and the quad's lanes
                    // must agree on what follows: the first lane's load counts
                    own = quad_lane<0>(own);
                    act = act && own == lab;

                    int32_t candA = kNever, candB = kNever;
                    bool keep = false;
                    if (act) {
                        // a cell lit before p (a continuation, or an ignition
                        // waiting out the hours outside the burning window)
                        // advances from p's start
                        const int32_t m0 = max((int32_t)(lab & kMinuteMask) + 1, s);
                        const uint32_t nb = rec_nbmask(rec.info) >> role;
                        const uint32_t dA = vA - (tag << kMinuteBits), dB = vB - (tag << kMinuteBits);
                        if (!(nb & 1u) || !axis_live(remA, dA, m0)) remA = 0;
                        if (!(nb & 16u) || !axis_live(remB, dB, m0)) remB = 0;
                        if (quad_or((uint32_t)(remA | remB)) != 0u && m0 <= e) {
                            int32_t qA, qB;
                            bool out = quad_axis_q<sizeof(R) == 8>(s_x32, s_x64, erep, &s_e, rec, draws, role, qA, qB);
                            c_evals += role == 0;
                            // burn-out (A5 (iv)): the head fire intensity is below
                            // the threshold; (A5 (i)): every rate toward a burnable
                            // neighbour is below delta.  The cell spreads no further.
                            if (burnout > 0.f) {
                                const int32_t qm = max(nb & 1u ? qA : 0, nb & 16u ? qB : 0);
                                out = out || quad_or((double)qm >= (double)burnout ? 1u : 0u) == 0u;
                            }
                            if (out) remA = remB = 0;
                            const int32_t n = e - m0 + 1;
                            const int32_t tA = remA > 0 ? step_axis(qA, remA, n) : 0;
                            const int32_t tB = remB > 0 ? step_axis(qB, remB, n) : 0;
                            if (tA) candA = m0 + tA - 1;
                            if (tB) candB = m0 + tB - 1;
                            // nothing after the period can beat a label of at most e + 1
                            if (dA <= (uint32_t)(e + 1)) remA = 0;
                            if (dB <= (uint32_t)(e + 1)) remB = 0;
                        }
                        keep = quad_or((uint32_t)(remA | remB)) != 0u;
                    }

                    // offer the candidates: atomicMin of real labels, or a
                    // pending mark where the neighbour's rate is below the
                    // threshold.  Both atomics are issued before any result is
                    // used so that their latencies overlap.
                    const bool hasA = candA != kNever, hasB = candB != kNever;
                    bool pendA = false, pendB = false;
                    if (use_thr) {
                        if (hasA) pendA = !ignites(cA, p);
                        if (hasB) pendB = !ignites(cB, p);
                        c_evals += (uint32_t)hasA + (uint32_t)hasB;
                    }
                    const uint32_t labA = pendA ? pendv : (tag << kMinuteBits) | (uint32_t)candA;
                    const uint32_t labB = pendB ? pendv : (tag << kMinuteBits) | (uint32_t)candB;
                    uint32_t oldA = 0, oldB = 0;   // not offered: nothing is below 0
                    if (hasA) oldA = atomicMin(&plane[cA], labA);
                    if (hasB) oldB = atomicMin(&plane[cB], labB);
                    c_cand += (uint32_t)__popcll(__ballot(hasA)) + (uint32_t)__popcll(__ballot(hasB));
                    const bool imprA = labA < oldA && !pendA, imprB = labB < oldB && !pendB;
                    // improved neighbours join the queue and axes still travelling
                    // at the end of p continue in p+1, one entry per quad: one
                    // ballot for each gives every lane its place in the wave's
                    // ranges, which lanes 0 and 1 reserve in one LDS instruction
                    const uint64_t mA = __ballot(imprA), mB = __ballot(imprB), mk = __ballot(keep);
                    const int nA = (int)__popcll(mA), wtot = nA + (int)__popcll(mB), ktot = (int)(__popcll(mk) >> 2);
                    if ((wtot | ktot) != 0) {
                        int got = 0;
                        if (__lane_id() < 2)
                            got = atomicAdd(__lane_id() == 0 ? &s_res : &s_nC[cc ^ 1], __lane_id() == 0 ? wtot : ktot);
                        const int wbase = lane_value(got, 0), kbase = lane_value(got, 1);
                        if (wtot > 0) {
                            if (imprA) q_put(wbase + wave_rank(mA), make_uint2(cA, labA));
                            if (imprB) q_put(wbase + nA + wave_rank(mB), make_uint2(cB, labB));
                            q_commit(wbase, wtot);
                            const bool newA = imprA && unburned(oldA, tag), newB = imprB && unburned(oldB, tag);
                            c_impr += (uint32_t)wtot;
                            c_ign += (uint32_t)__popcll(__ballot(newA)) + (uint32_t)__popcll(__ballot(newB));
                            if (count) {
                                if (newA) count_one(cA);
                                if (newB) count_one(cB);
                            }
                        }
                        const int k = kbase + (wave_rank(mk) >> 2);
                        if (keep) {
                            if ((uint32_t)k < cap) {
                                Cont* ct = gC(cc ^ 1) + k;
                                if (role == 0) *(uint2*)&ct->c = make_uint2(c, lab);
                                ct->rem[role] = (uint32_t)remA | ((uint32_t)remB << 16);
                            } else {
                                s_flag = 1;
                            }
                        }
                    }
                    if (use_thr) {
                        append_g(pendA && oldA > pendv, cA, gP(pc ^ 1), cap, &s_nP[pc ^ 1], &s_flag);
                        append_g(pendB && oldB > pendv, cB, gP(pc ^ 1), cap, &s_nP[pc ^ 1], &s_flag);
                    }
                }
                if (redo != 0) continue;   // still a holder
                if (conts) {
                    if (__lane_id() == 0) cbase = atomicAdd(&s_ctake, csize);
                    cbase = csize * NW + lane_value(cbase, 0);
                } else if (__lane_id() == 0) {
                    atomicAdd(&s_hb, ~0ull);   // one holder fewer
                }
            }
            {
                const int n = s_res;
                if (n > max_list) max_list = n;
            }
            // ------------------------------------------------- period end
            // Thread 0 decides whether to stop between the two barriers: a
            // list overflowed, or the fire is out (no continuation and no
            // pending cell for p+1) and no listed ignition is still to
            // come.  Reading s_flag or the list lengths after the second
            // barrier could see values a faster wave already wrote in p+1.
            __syncthreads();
            if (tid == 0) {
                s_stop = s_flag || (s_nC[cc ^ 1] == 0 && s_nP[pc ^ 1] == 0 && last_seed_period <= p);
                s_nC[cc] = 0;
                s_nP[pc] = 0;
                s_res = s_commit = 0;
                s_ctake = 0;
                s_hb = 0ull;
            }
            cc ^= 1;
            pc ^= 1;
            __syncthreads();
            if (s_stop) break;
        }
        if (s_flag && tid == 0) atomicOr(&rc->overflow, 1);

        // per-replication counters and outputs
        atomicAdd(&s_cnt[kCntEvals], (unsigned long long)c_evals);   // per lane, the others per wave
        if (__lane_id() == 0) {
            atomicAdd(&s_cnt[kCntIgnitions], (unsigned long long)c_ign);
            atomicAdd(&s_cnt[kCntEntries], (unsigned long long)c_entries);
            atomicAdd(&s_cnt[kCntConts], (unsigned long long)c_conts);
            atomicAdd(&s_cnt[kCntCandidates], (unsigned long long)c_cand);
            atomicAdd(&s_cnt[kCntImprovements], (unsigned long long)c_impr);
            atomicAdd(&s_cnt[kCntRounds], (unsigned long long)c_rounds);
        }
        atomicMax(&s_cnt[kCntMaxList], (unsigned long long)max_list);
        if (slots.item_slot) {
            if (tid == 0) slots.item_slot[item] = make_int2(slot, (int)tag);
        } else if (job.scar || job.arr_minute || job.arr_period) {
            __syncthreads();
            const size_t n = (size_t)job.rows * cols;
            const size_t o = (size_t)lr * n;
            for (size_t i = tid; i < n; i += BLOCK) {
                const uint32_t v = load_label(&plane[i]);
                const bool on = (v >> kMinuteBits) == tag && (v & kMinuteMask) != kPendingMinute;
                const int32_t t = on ? (int32_t)(v & kMinuteMask) : -1;
                if (job.scar) job.scar[o + i] = (uint8_t)on;
                if (job.arr_minute) job.arr_minute[o + i] = t;
                if (job.arr_period) job.arr_period[o + i] = !on ? -1 : (t == 0 ? 0 : (t - 1) / P);
            }
        }
        __syncthreads();
        if (tid == 0) {
            if (job.burned) job.burned[lr] = (int64_t)s_cnt[kCntIgnitions];
            if (job.ign_out) job.ign_out[lr] = s_ign;
            if (job.scen_out) job.scen_out[lr] = s_scen;
        }
        if (tid < kNumCounters) s_sum[tid] = tid == kCntMaxList ? max(s_sum[tid], s_cnt[tid]) : s_sum[tid] + s_cnt[tid];
        __syncthreads();
    }
    if (tid < kNumCounters && s_sum[tid] != 0) {   // each by the thread that summed it
        if (tid == kCntMaxList) atomicMax(&rc->c[tid], s_sum[tid]);
        else atomicAdd(&rc->c[tid], s_sum[tid]);
    }
}

// Dense per-replication outputs from the final arrival planes, one thread
// per (item, cell): used when every item of the launch kept its own slot.
__global__ __launch_bounds__(256) void dense_outputs_kernel(const Job* __restrict__ jobs, int n_jobs,
                                                            int total_items, int n_slots, Slots slots,
                                                            const RunCounters* __restrict__ rc) {
    const int item = blockIdx.y;
    if (item >= total_items || rc->overflow) return;   // an overflowed launch is repeated
    int lo = 0, hi = n_jobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].item_base <= item) lo = mid;
        else hi = mid - 1;
    }
    const Job& job = jobs[lo];
    if (!(job.scar || job.arr_minute || job.arr_period)) return;
    const int2 st = slots.item_slot[item];
    if (st.x < 0 || st.x >= n_slots) return;   // item not run (cleared to -1 before the launch)
    const uint32_t tag = (uint32_t)st.y;
    const uint32_t* __restrict__ plane = slots.planes + (size_t)st.x * (size_t)slots.plane_cells;
    const size_t n = (size_t)job.rows * (size_t)job.cols;
    const size_t o = (size_t)(item - job.item_base) * n;
    const int P = job.period_min;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const uint32_t v = plane[i];
        const bool on = (v >> kMinuteBits) == tag && (v & kMinuteMask) != kPendingMinute;
        const int32_t t = on ? (int32_t)(v & kMinuteMask) : -1;
        if (job.scar) job.scar[o + i] = (uint8_t)on;
        if (job.arr_minute) job.arr_minute[o + i] = t;
        if (job.arr_period) job.arr_period[o + i] = !on ? -1 : (t == 0 ? 0 : (t - 1) / P);
    }
}

hipError_t launch_dense_outputs(const Job* jobs, int n_jobs, int total, int n_slots, int64_t max_cells,
                                const Slots& slots, const RunCounters* rc, hipStream_t s) {
    if (total <= 0 || total > 65535 || !slots.item_slot) return hipErrorInvalidValue;
    const int64_t want = (max_cells + 255) / 256;
    const int gx = (int)std::max<int64_t>(1, std::min<int64_t>(want, 4096 / std::min(total, 16)));
    hipLaunchKernelGGL(dense_outputs_kernel, dim3(gx, total), dim3(256), 0, s, jobs, n_jobs, total, n_slots, slots,
                       rc);
    return hipGetLastError();
}

template <typename R>
static hipError_t launch_prop_t(int block, int grid, const Job* jobs, int n_jobs, int total, const Slots& sl,
                                RunCounters* rc, hipStream_t s) {
    switch (block) {
        case 64: hipLaunchKernelGGL((propagate_kernel<R, 64>), dim3(grid), dim3(64), 0, s, jobs, n_jobs, total, sl, rc); break;
        case 128: hipLaunchKernelGGL((propagate_kernel<R, 128>), dim3(grid), dim3(128), 0, s, jobs, n_jobs, total, sl, rc); break;
        case 256: hipLaunchKernelGGL((propagate_kernel<R, 256>), dim3(grid), dim3(256), 0, s, jobs, n_jobs, total, sl, rc); break;
        case 512: hipLaunchKernelGGL((propagate_kernel<R, 512>), dim3(grid), dim3(512), 0, s, jobs, n_jobs, total, sl, rc); break;
        case 768: hipLaunchKernelGGL((propagate_kernel<R, 768>), dim3(grid), dim3(768), 0, s, jobs, n_jobs, total, sl, rc); break;
        case 1024: hipLaunchKernelGGL((propagate_kernel<R, 1024>), dim3(grid), dim3(1024), 0, s, jobs, n_jobs, total, sl, rc); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_propagate(int precision, int block, int grid, const Job* jobs, int n_jobs, int total,
                            const Slots& slots, RunCounters* rc, hipStream_t s) {
    return precision == 1 ? launch_prop_t<float>(block, grid, jobs, n_jobs, total, slots, rc, s)
                          : launch_prop_t<double>(block, grid, jobs, n_jobs, total, slots, rc, s);
}

template <typename R>
static int occ_t(int block) {
    int nb = 0;
    hipError_t e = hipErrorInvalidValue;
    switch (block) {
        case 64: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, propagate_kernel<R, 64>, 64, 0); break;
        case 128: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, propagate_kernel<R, 128>, 128, 0); break;
        case 256: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, propagate_kernel<R, 256>, 256, 0); break;
        case 512: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, propagate_kernel<R, 512>, 512, 0); break;
        case 768: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, propagate_kernel<R, 768>, 768, 0); break;
        case 1024: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, propagate_kernel<R, 1024>, 1024, 0); break;
        default: break;
    }
    return (e == hipSuccess) ? nb : 0;
}

int propagate_blocks_per_cu(int precision, int block) {
    return precision == 1 ? occ_t<float>(block) : occ_t<double>(block);
}

}  // namespace c2f
