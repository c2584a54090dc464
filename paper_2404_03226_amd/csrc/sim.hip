// Event-driven list-scheduling simulation with INSPIRIT priorities.
//
// One wave of a work-group owns one DAG at a time and runs its whole event loop
// (a persistent grid takes DAGs, largest first, from an atomic dispenser);
// beside it, up to 128 workers, a second wave keeps the workers' best queue
// entries and a third reads ahead.
// Per event time t, in order (Section 2 DMDA push, Section 4.1 per-worker
// queues, Section 4.4 adaptive pop rule):
//   push     newly ready tasks in ascending id, each to the worker with the
//            least expected termination time (free time + queued estimates +
//            own estimate; ties to the lower worker id) -- a wave-wide argmin
//            over packed (cost, worker) keys;
//   regulate Nready = queued tasks; the Section 4.4 state machine picks the
//            pop rule (scalar code);
//   pop      every idle worker takes the best task of its own queue under the
//            rule -- two wave-wide argmax steps over 64-slot blocks;
//   advance  t = earliest finish among running tasks (wave min);
//   release  for each completing task c and edge c -> s, one 64-bit
//            read-modify-write (the wave owns the DAG) subtracts (1 << 43) + c
//            from word[s] = rem << 43 | sum of unfinished predecessor ids.  rem reaching 0 makes s ready; rem
//            reaching 1 leaves exactly one unfinished predecessor
//            u = remaining sum, whose IE grows by one when tau(u) + tau(s)
//            <= U (IE counts successors with rem == 1).  Newly ready ids of
//            one completing task arrive ascending (rows are sorted); several
//            such runs are merged by rank.
//
// Queue entry of the general loop (two 64-bit words):  k = IA << 42 | IE << 21 | (2^21-1-seq),
//                                  x = task << 42 | dur << 21 | est
// (all fields < 2^21).  Under the ability rule the key is k itself; under the
// efficiency rule IA and IE swap places; FIFO keeps only the seq field.  Keys
// are unique (seq), so a max identifies one entry.  Each block keeps the max
// key of its entries under two rules (ability-or-FIFO, efficiency); IE only
// grows while a task waits, so increments update block maxima with atomicMax
// and a pop rescans only the block it touched.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <string>
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"
#include "keys.hpp"

namespace insp {

constexpr uint64_t M43 = (1ull << 43) - 1;

#ifdef INSP_PHASE_CLOCKS
// Diagnostic build only: per-DAG core-clock totals of each event phase.
__device__ unsigned long long g_phase_clk[8192 * 32];
#define PCLK(i) do { unsigned long long c_ = clock64(); pc[i] += c_ - pc_last; pc_last = c_; } while (0)
#else
#define PCLK(i) do {} while (0)
#endif

// Makes the compiler wait for a global load inside the branch that issued it.
// A value read from LDS on one side of a uniform branch and from global memory
// on the other otherwise arrives at the join with a pending global load, and
// every later use waits for all outstanding global accesses -- stores
// included -- even when the LDS side ran.
template <typename T>
__device__ __forceinline__ void settle(const T &x) {
    asm volatile("" ::"v"(x));
}

// The popped task's schedule, written over its dead dependency word and
// push order (see TaskRec): one 16-byte store.
__device__ __forceinline__ void put_record(TaskRec *r, int64_t start, int32_t dur, int32_t w, int32_t ie, int mode) {
    const uint64_t wd = (uint64_t)start | (uint64_t)dur << 42;
    int4 q;
    q.x = (int32_t)(uint32_t)wd;
    q.y = (int32_t)(uint32_t)(wd >> 32);
    q.z = -2 - w;
    q.w = ie | mode << 22;
    *reinterpret_cast<int4 *>(r) = q;
}

struct SimArgs {
    const DagDesc *desc;
    const int32_t *order;
    int32_t count, max_w, sum_cap, policy, lb, slot_cap;
    int32_t key_cap;           // queue blocks whose keys live in LDS (>= slot_cap, whose payload does too)
    const int32_t *col;
    const int32_t *dur, *est;
    int64_t base;
    TaskRec *tr;
    unsigned long long *dep;   // dependency words: remaining in-degree << 43 | sum of unfinished predecessor ids
    int32_t *fbuf;
    SlotPool slots;
    unsigned long long *sums;
    int32_t *paux;
    int64_t freeb_base;
    const int32_t *dag_u, *dag_taubar;
    const int64_t *rank;  // HEFT upward ranks (global task index)
    const int32_t *tia, *tie;  // transitive IA, IE (global task index)
    int32_t attr_mode;
    int32_t data_bw;           // data model: bytes per tick between memory nodes (0 = off)
    const int32_t *dkib;       // data model: output KiB per task (global task index)
    const int32_t *pprp, *ppred;  // predecessor lists (local row pointers as rp, ids as col)
    long long *barr;           // data model: per queue block, the latest input arrival pushed into it
    int32_t *dxc;              // data model: transfer ticks of each task's output (global task index)
    int32_t *stat;
    int32_t *counter;
    int64_t *makespan;
    insp_trace_rec *trace;     // DAG di's events from record (toff - base) + di on: n + 1 slots per DAG
    int32_t *n_events;
    int32_t s_inc, s_dec, dec_step, c, k_num, k_den, max_events;
    int32_t prio_top;          // DAGs dispensed before this one run at raised wave priority
};

// LDS-resident state of the DAG a work-group is simulating.
constexpr int kPF = 8;    // successors of a running task prefetched into registers at its pop
constexpr int kFC = 256;  // frontier slots in LDS (larger frontiers use global memory)
constexpr int kCC = 128;  // candidate slots in LDS
constexpr int kScan = 16;  // most blocks the tune key's "scan=" may name (it has no effect: see keep_best)
constexpr int64_t kHelperSpin = 1ll << 40;
// Which way a branch of the one-wave loop nearly always goes.
#define USUALLY(x) __builtin_expect(!!(x), 1)
#define RARELY(x) __builtin_expect(!!(x), 0)

constexpr int32_t kReqSpin = 1 << 24;  // polls of a rescan request (it takes a few)

struct Lds {
    int64_t *fin, *expend, *qest;                    // [MW]
    int32_t *run, *len, *nb, *last, *seg, *rsr, *dgr; // [MW]
    int32_t *blist;                                  // [MW * lb] first block ids of each worker
    unsigned long long *sum;                         // [2 * sum_cap] block max keys
    int32_t *fr0, *fr1;                              // [kFC]
    int32_t *cs, *cu;                                // [kCC]
    int32_t *pre;                                    // [8 * kWave] staged frontier rows
    unsigned long long *sk;                          // [64 * key_cap] keys of the low blocks' entries
    unsigned long long *sx;                          // [64 * slot_cap] payload (task, durations) of the lowest
    int32_t *srs;                                    // [64 * slot_cap] ... and their first edges
    int32_t *hs;                                     // [4] DAG index
};

__host__ __device__ inline size_t lds_bytes(int mw, int sc, int lb, int slc, int slk) {
    return (size_t)mw * (3 * 8 + 7 * 4 + (size_t)lb * 4) + (size_t)sc * 16 + kFC * 8 + kCC * 8 +
           8 * 64 * 4 + (size_t)slc * 64 * 12 + (size_t)slk * 64 * 8 + 64 + 32;
}

// The general loop, for machines of more than 128 workers: their state in LDS
// arrays, a lane's workers lane, lane + 64, ... in turn.
__device__ void sim_dag(const SimArgs &A, int32_t di, const Lds &L) {
    constexpr int WPL = INSP_MAX_WORKERS / kWave;
    const int lane = lane_id();
    const DagDesc d = A.desc[di];
    const int32_t n = d.n, ncpu = d.n_cpu, W = d.n_cpu + d.n_gpu;
    int32_t status = A.stat[2 * d.id];
    if (n == 0 || status != 0) {
        if (lane == 0) {
            A.makespan[di] = status ? -1 : 0;
            if (A.n_events) A.n_events[di] = 0;
        }
        return;
    }
    const int64_t ub = d.toff - A.base;
    const int32_t *col = A.col + d.eoff;
    TaskRec *tr = A.tr + d.toff;
    unsigned long long *dep = A.dep + d.toff;
    int32_t *fbuf = A.fbuf + 3 * d.toff;      // [0,n) runs, [n,2n) merged, [2n,3n) candidates
    const int2 *est2 = reinterpret_cast<const int2 *>(A.est) + ub;
    const int2 *dur2 = reinterpret_cast<const int2 *>(A.dur) + ub;
    const SlotPool slots = A.slots.at(64 * d.blk_off);
    unsigned long long *sums = A.sums + 2 * d.blk_off;
    int32_t *wblk = A.paux + d.wl_off;
    int32_t *freeb = A.paux + A.freeb_base + d.blk_off;
    const int32_t maxb = d.maxb;
    const int32_t SC = A.sum_cap;
    const int32_t kLB = A.lb;
    const int32_t SLC = A.slot_cap;  // blocks [0, SLC) keep their slots in LDS
    const int32_t U = A.dag_u[d.id];

    // regulator parameters (defaults: the paper names them, prints no values)
    const int32_t s_inc = A.s_inc > 0 ? A.s_inc : max(1, (W + 3) / 4);
    const int32_t s_dec = A.s_dec > 0 ? A.s_dec : max(1, (W + 1) / 2);
    const int32_t dec_step = A.dec_step > 0 ? A.dec_step : s_dec;
    const int32_t cc = A.c >= 0 ? A.c : s_dec / 2;
    const bool kset = A.k_num > 0 && A.k_den > 0;
    const int32_t k_num = kset ? A.k_num : W;
    const int32_t k_den = kset ? A.k_den : A.dag_taubar[d.id];
    const bool heft = A.policy == INSP_POLICY_HEFT;
    const bool tattr = A.attr_mode == INSP_ATTR_TRANSITIVE;
    const bool trans = !heft && tattr;  // keys built from the transitive attributes
    const bool skey = heft || trans;  // keys fixed while queued
    const int64_t *rk = A.rank + d.toff;
    const int32_t *tia = A.tia + d.toff, *tie = A.tie + d.toff;
    // data model: inputs move between memory nodes (host for the CPU
    // workers, one per GPU worker); see the push and the pop below
    const bool data = A.data_bw > 0;
    const int32_t *dkib = A.dkib + d.toff, *prp = A.pprp + d.toff + d.id, *pred = A.ppred + d.eoff;
    long long *barr = A.barr + d.blk_off;
    int32_t *dxc = A.dxc + d.toff;
    // block arrival bounds matter only where the locality rule can be used
    const bool lrule = data && (A.policy == INSP_POLICY_INSPIRIT || A.policy == INSP_POLICY_LOCALITY);
    const int slot0 = A.policy == INSP_POLICY_FIFO ? 2 : heft ? 3 : 0;
    const int32_t max_events = A.max_events > 0 ? A.max_events : n + 1;

    for (int32_t w = lane; w < W; w += kWave) {
        L.run[w] = -1;
        L.len[w] = 0;
        L.nb[w] = 0;
        L.last[w] = -1;
        L.fin[w] = 0;
        L.expend[w] = 0;
        L.qest[w] = 0;
        L.rsr[w] = 0;
        L.dgr[w] = 0;
    }
    for (int32_t i = lane; i < d.nblk; i += kWave) freeb[i] = d.nblk - 1 - i;
    int32_t nfree = d.nblk;
    if (data)  // each output's transfer ticks, once per run (no division at the pushes)
        for (int32_t i = lane; i < n; i += kWave)
            dxc[i] = (int32_t)(((int64_t)1024 * dkib[i] + A.data_bw - 1) / A.data_bw);

    // initial frontier: tasks without predecessors, ascending
    int32_t r = 0;
    for (int32_t i0 = 0; i0 < n; i0 += kWave) {
        int32_t i = i0 + lane;
        bool ok = i < n && (dep[i] >> 43) == 0;
        uint64_t mk = ballot(ok);
        if (ok) {
            int32_t pos = r + lanes_below(mk);
            fbuf[pos] = i;
            if (pos < kFC) L.fr0[pos] = i;
        }
        r += __popcll(mk);
    }
    bool merged = false, staged = false;
    wg_fence();
    __builtin_amdgcn_wave_barrier();

    int64_t t = 0, prev_t = 0;
    int32_t nready = 0, events = 0, done = 0, seq = 0;
    int32_t peak = 0, prev_n = 0, cnt = 0;
    int mode = INSP_MODE_ABILITY;
#ifdef INSP_PHASE_CLOCKS
    unsigned long long pc[32] = {0}, pc_last = clock64();
#endif

    for (;;) {
        PCLK(9);
        if (++events > max_events) {
            status |= ST_HANG;
            break;
        }
        // ------------------------------------------------------------ push
        int64_t ld[WPL];
#pragma unroll
        for (int k = 0; k < WPL; k++) {
            int32_t w = lane + k * kWave;
            ld[k] = INT64_MAX / 4;
            if (w < W) {
                int64_t B = t;
                if (L.run[w] >= 0 && L.expend[w] > t) B = L.expend[w];
                ld[k] = B + L.qest[w];
            }
        }
        for (int32_t i0 = 0; i0 < r; i0 += kWave) {
            const int32_t idx = i0 + lane;
            const bool ok = idx < r;
            int32_t v_l = 0;
            int2 e_l = make_int2(1, 1), d_l = make_int2(1, 1);
            int32_t ia_l = 0, ie_l = 0, rs_l = 0;
            uint64_t rk_l = 0;
            if (staged) {
                // rows loaded during the previous candidate round trip
                if (ok) {
                    v_l = L.pre[idx];
                    e_l = make_int2(L.pre[64 + idx], L.pre[128 + idx]);
                    d_l = make_int2(L.pre[192 + idx], L.pre[256 + idx]);
                    ia_l = L.pre[320 + idx];
                    rs_l = L.pre[384 + idx];
                    ie_l = L.pre[448 + idx];
                }
            } else {
                if (ok) {
                    if (r <= kFC) v_l = merged ? L.fr1[idx] : L.fr0[idx];
                    else v_l = merged ? fbuf[n + idx] : fbuf[idx];
                }
                if (ok) {
                    e_l = est2[v_l];
                    d_l = dur2[v_l];
                    ia_l = tr[v_l].ia;
                    rs_l = tr[v_l].rs;
                    ie_l = wg_load(&tr[v_l].iev);
                }
            }
            if (heft && ok) rk_l = (uint64_t)rk[v_l];
            if (trans && ok) {
                ia_l = tia[v_l];
                ie_l = tie[v_l];
            }
            if (ballot(ok && (d_l.x < 1 || d_l.x > INSP_MAX_TICK || d_l.y < 1 || d_l.y > INSP_MAX_TICK)))
                status |= ST_DUR;
            const int32_t cntj = min(kWave, r - i0);
            for (int32_t j = 0; j < cntj; j++) {
                const int32_t v = read_lane(v_l, j);
                const int32_t e0 = read_lane(e_l.x, j), e1 = read_lane(e_l.y, j);
                // DMDA's transfer term: ticks to move the inputs whose home
                // node is not the worker's (an item stays where it was made)
                int64_t xk[WPL];
#pragma unroll
                for (int k = 0; k < WPL; k++) xk[k] = 0;
                if (data) {
                    const int32_t pa = prp[v], pz = prp[v + 1];
                    for (int32_t c0 = pa; c0 < pz; c0 += kWave) {
                        int32_t nu = 0;
                        int64_t cu = 0;
                        if (c0 + lane < pz) {
                            const int32_t u = pred[c0 + lane];
                            const int32_t wu = -2 - tr[u].qpos;  // worker of a finished task
                            nu = wu < ncpu ? 0 : 1 + wu - ncpu;
                            cu = dxc[u];
                        }
                        const int32_t cnt = min(kWave, pz - c0);
                        for (int32_t jj = 0; jj < cnt; jj++) {
                            const int32_t nj = read_lane(nu, jj);
                            const int64_t cj = (int64_t)read_lane64((uint64_t)cu, jj);
#pragma unroll
                            for (int k = 0; k < WPL; k++) {
                                const int32_t w = lane + k * kWave;
                                if ((w < ncpu ? 0 : 1 + w - ncpu) != nj) xk[k] += cj;
                            }
                        }
                    }
                }
                uint64_t best = ~0ull;
#pragma unroll
                for (int k = 0; k < WPL; k++) {
                    int32_t w = lane + k * kWave;
                    if (w < W) {
                        uint64_t cst = (uint64_t)(ld[k] + (w < ncpu ? e0 : e1) + xk[k]);
                        uint64_t key = cst << 11 | (uint64_t)w;
                        best = key < best ? key : best;
                    }
                }
                best = wave_min_u64(best);
                const int32_t ws = (int32_t)(best & 2047);
                const bool gpu = ws >= ncpu;
                int64_t xs = 0;
                if (data) {
                    int64_t mine = 0;
#pragma unroll
                    for (int k = 0; k < WPL; k++)
                        if (lane + k * kWave == ws) mine = xk[k];
                    xs = (int64_t)read_lane64((uint64_t)mine, ws & 63);
                    if (xs > INSP_MAX_TICK) status |= ST_XFER;
                }
                const int32_t ek = gpu ? e1 : e0;
                const int32_t dk = read_lane(gpu ? d_l.y : d_l.x, j);
#pragma unroll
                for (int k = 0; k < WPL; k++)
                    if (lane + k * kWave == ws) ld[k] += ek;
                const int32_t len = L.len[ws];
                const int32_t pos = len & 63;
                int32_t blk;
                if (pos == 0) {
                    nfree--;
                    blk = wg_load(&freeb[nfree]);
                    if (lane == 0) {
                        const int32_t nbw = L.nb[ws];
                        if (nbw < kLB) L.blist[ws * kLB + nbw] = blk;
                        else wblk[(int64_t)ws * maxb + nbw] = blk;
                        L.nb[ws] = nbw + 1;
                        L.last[ws] = blk;
                    }
                } else {
                    blk = L.last[ws];
                }
                const int32_t p = blk * 64 + pos;
                const uint64_t kw =
                    heft ? read_lane64(rk_l, j) << 21 | (M21 - (uint64_t)seq)
                         : (uint64_t)read_lane(ia_l, j) << 42 | (uint64_t)read_lane(ie_l, j) << 21 | (M21 - (uint64_t)seq);
                const uint64_t xw = (uint64_t)v << 42 | (uint64_t)(dk & M21) << 21 | (uint64_t)(ek & M21);
                const int32_t rs = read_lane(rs_l, j);
                if (lane == 0) {
                    if (blk < SLC) {
                        L.sk[p] = kw;
                        L.sx[p] = xw;
                        L.srs[p] = rs;
                    } else {
                        slots.k[p] = kw;
                        slots.x[p] = xw;
                        slots.rs[p] = rs;
                    }
                    tr[v].qpos = p;
                    tr[v].seq = seq;
                    // the dependency word is dead once a task is queued: it
                    // holds the time its inputs arrive (transfers start now)
                    if (data) tr[v].word = (unsigned long long)(t + xs);
                    // never lowered by pops: an upper bound for the block
                    if (lrule) barr[blk] = pos == 0 ? t + xs : max(barr[blk], (long long)(t + xs));
                    const uint64_t a0 = key_of(kw, slot0), a1 = key_of(kw, 1);
                    if (blk < SC) {
                        if (pos == 0) {
                            L.sum[2 * blk] = a0;
                            L.sum[2 * blk + 1] = a1;
                        } else {
                            atomicMax(&L.sum[2 * blk], (unsigned long long)a0);
                            atomicMax(&L.sum[2 * blk + 1], (unsigned long long)a1);
                        }
                    } else if (pos == 0) {
                        sums[2 * blk] = a0;
                        sums[2 * blk + 1] = a1;
                    } else {
                        wg_fetch_max(&sums[2 * blk], (unsigned long long)a0);
                        wg_fetch_max(&sums[2 * blk + 1], (unsigned long long)a1);
                    }
                    L.len[ws] = len + 1;
                    L.qest[ws] += ek;
                }
                seq++;
                nready++;
            }
        }
        PCLK(0);
        wg_fence();
        __builtin_amdgcn_wave_barrier();
        PCLK(1);
        // -------------------------------------------------------- regulate
        const int32_t observed = nready;
        if (A.policy == INSP_POLICY_INSPIRIT) {
            if (nready > peak) peak = nready;
            const int32_t dn = nready - prev_n;
            if ((dn < 0 ? -dn : dn) >= s_inc) {
                const int64_t dt = t - prev_t;
                prev_n = nready;
                prev_t = t;
                if (nready >= peak - dec_step) {
                    cnt = 0;
                    if (dn >= s_inc) {
                        const int64_t lhs = (int64_t)dn * k_den, rhs = (int64_t)k_num * dt;
                        if (dt == 0 || lhs > rhs) mode = INSP_MODE_ABILITY;
                        else if (lhs < rhs) mode = INSP_MODE_EFI;
                    }
                } else if ((int64_t)nready > (int64_t)peak - (int64_t)s_dec * cnt) {
                    mode = INSP_MODE_ABILITY;
                } else if ((int64_t)nready <= (int64_t)peak - (int64_t)s_dec * (cnt + 1) + cc) {
                    mode = INSP_MODE_EFI_LOC;
                    if ((int64_t)nready <= (int64_t)peak - (int64_t)s_dec * (cnt + 1)) cnt++;
                }
            }
        }
        const int pmode = A.policy == INSP_POLICY_FIFO ? INSP_MODE_FIFO
                        : A.policy == INSP_POLICY_ABILITY_ONLY ? INSP_MODE_ABILITY
                        : A.policy == INSP_POLICY_EFI_ONLY ? INSP_MODE_EFI
                        : A.policy == INSP_POLICY_LOCALITY ? INSP_MODE_EFI_LOC
                        : heft ? INSP_MODE_RANK : mode;
        // efficiency with locality: tasks whose inputs have arrived first
        const bool loc = data && pmode == INSP_MODE_EFI_LOC;
        const int ord = heft ? 3 : pmode == INSP_MODE_FIFO ? 2 : pmode == INSP_MODE_ABILITY ? 0 : 1;
        const int slot = ord == 1 ? 1 : 0;
        // ------------------------------------------------------------- pop
        int32_t popped = 0;
        for (int32_t w0 = 0; w0 < W; w0 += kWave) {
            const int32_t wl = w0 + lane;
            uint64_t mask = ballot(wl < W && L.run[wl] < 0 && L.len[wl] > 0);
            while (mask) {
                const int32_t w = w0 + (int32_t)__builtin_ctzll(mask);
                mask &= mask - 1;
                int32_t nb = L.nb[w], len = L.len[w];
                const int32_t last = L.last[w];
                int32_t bb = last;
                bool lsel = false;
                if (loc) {
                    // the arrival times are not in the keys.  A block whose
                    // latest input arrival has passed holds only tasks whose
                    // inputs are in place, so its efficiency maximum stands;
                    // the other blocks are scanned entry by entry
                    uint64_t bestk = 0;
                    int32_t bestb = -1;
                    const int32_t lp = (len - 1) & 63;
                    for (int32_t i0 = 0; i0 < nb; i0 += kWave) {
                        const int32_t i = i0 + lane;
                        uint64_t kk = 0;
                        int32_t b = -1;
                        bool mix = false;
                        if (i < nb) {
                            b = i < kLB ? L.blist[w * kLB + i] : wg_load(&wblk[(int64_t)w * maxb + i]);
                            if ((int64_t)wg_load(&barr[b]) <= t) kk = b < SC ? L.sum[2 * b + 1] : wg_load(&sums[2 * b + 1]);
                            else mix = true;
                        }
                        const uint64_t km = wave_max_u64(kk);
                        if (km > bestk) {
                            bestk = km;
                            bestb = read_lane(b, (int)__builtin_ctzll(ballot(kk == km && i < nb)));
                        }
                        uint64_t mm = ballot(mix);
                        while (mm) {
                            const int32_t bm = read_lane(b, (int)__builtin_ctzll(mm));
                            mm &= mm - 1;
                            uint64_t ke = 0;
                            if (lane < (bm == last ? lp + 1 : 64)) {
                                const uint64_t kv = bm < SLC ? L.sk[bm * 64 + lane] : wg_load(&slots.k[bm * 64 + lane]);
                                const uint64_t xv = bm < SLC ? L.sx[bm * 64 + lane] : wg_load(&slots.x[bm * 64 + lane]);
                                if ((int64_t)wg_load(&tr[(int32_t)(xv >> 42)].word) <= t) ke = key_of(kv, 1);
                            }
                            const uint64_t kme = wave_max_u64(ke);
                            if (kme > bestk) {
                                bestk = kme;
                                bestb = bm;
                            }
                        }
                    }
                    if (bestb >= 0) {
                        bb = bestb;
                        lsel = true;
                    }
                }
                if (!lsel && nb > 1) {
                    uint64_t bk = 0;
                    int32_t bid = -1;
                    for (int32_t i0 = 0; i0 < nb; i0 += kWave) {
                        const int32_t i = i0 + lane;
                        if (i < nb) {
                            const int32_t b = i < kLB ? L.blist[w * kLB + i] : wg_load(&wblk[(int64_t)w * maxb + i]);
                            const uint64_t k = b < SC ? L.sum[2 * b + slot] : wg_load(&sums[2 * b + slot]);
                            if (k > bk) {
                                bk = k;
                                bid = b;
                            }
                        }
                    }
                    const uint64_t km = wave_max_u64(bk);
                    const uint64_t wm = ballot(bk == km && bid >= 0);
                    bb = read_lane(bid, (int)__builtin_ctzll(wm));
                }
                const int32_t lastpos = (len - 1) & 63;
                const int32_t cntb = bb == last ? lastpos + 1 : 64;
                const bool ok = lane < cntb;
                const int32_t eb = bb * 64, el = last * 64;
                const bool okl = last != bb && lane <= lastpos;
                uint64_t kw = 0, xw = 0, kl = 0, xl = 0;
                int32_t rw = 0, rl = 0;
                if (ok) {
                    if (bb < SLC) {
                        kw = L.sk[eb + lane];
                        xw = L.sx[eb + lane];
                        rw = L.srs[eb + lane];
                    } else {
                        kw = wg_load(&slots.k[eb + lane]);
                        xw = wg_load(&slots.x[eb + lane]);
                        rw = wg_load(&slots.rs[eb + lane]);
                    }
                }
                if (okl) {
                    if (last < SLC) {
                        kl = L.sk[el + lane];
                        xl = L.sx[el + lane];
                        rl = L.srs[el + lane];
                    } else {
                        kl = wg_load(&slots.k[el + lane]);
                        xl = wg_load(&slots.x[el + lane]);
                        rl = wg_load(&slots.rs[el + lane]);
                    }
                }
                bool here = true;
                if (lsel && ok) here = (int64_t)wg_load(&tr[(int32_t)(xw >> 42)].word) <= t;
                const uint64_t key = ok && here ? key_of(kw, ord) : 0;
                const uint64_t km = wave_max_u64(key);
                const int win = (int)__builtin_ctzll(ballot(key == km && ok));
                const uint64_t vk = read_lane64(kw, win), vx = read_lane64(xw, win);
                const int32_t vr = read_lane(rw, win);
                const int32_t p = eb + win;
                const int32_t q = el + lastpos;
                const int32_t v = (int32_t)(vx >> 42);
                const int32_t dk = (int32_t)((vx >> 21) & M21), ek = (int32_t)(vx & M21);
                uint64_t mk = 0, mx = 0;
                int32_t mr = 0;
                if (p != q) {
                    if (last == bb) {
                        mk = read_lane64(kw, lastpos);
                        mx = read_lane64(xw, lastpos);
                        mr = read_lane(rw, lastpos);
                    } else {
                        mk = read_lane64(kl, lastpos);
                        mx = read_lane64(xl, lastpos);
                        mr = read_lane(rl, lastpos);
                    }
                    if (lane == 0) {
                        if (bb < SLC) {
                            L.sk[p] = mk;
                            L.sx[p] = mx;
                            L.srs[p] = mr;
                        } else {
                            slots.k[p] = mk;
                            slots.x[p] = mx;
                            slots.rs[p] = mr;
                        }
                        tr[(int32_t)(mx >> 42)].qpos = p;
                        // the moved entry keeps block bb's arrival bound valid
                        if (lrule && last != bb) barr[bb] = max(barr[bb], barr[last]);
                    }
                }
                len--;
                const bool freed = (len & 63) == 0;
                int32_t newlast = last;
                if (freed) {
                    if (lane == 0) freeb[nfree] = last;
                    nfree++;
                    nb--;
                    newlast = nb <= 0 ? -1 : nb - 1 < kLB ? L.blist[w * kLB + nb - 1]
                                                         : wg_load(&wblk[(int64_t)w * maxb + nb - 1]);
                }
                if (!(bb == last && freed)) {
                    // block bb after the removal: the winner's slot holds the
                    // moved entry; if bb is the last block its final slot left
                    const uint64_t nk = (p != q && lane == win) ? mk : kw;
                    const bool valid = ok && !(bb == last && lane == lastpos);
                    const uint64_t s0 = wave_max_u64(valid ? key_of(nk, slot0) : 0);
                    const uint64_t s1 = wave_max_u64(valid ? key_of(nk, 1) : 0);
                    if (lane == 0) {
                        if (bb < SC) {
                            L.sum[2 * bb] = s0;
                            L.sum[2 * bb + 1] = s1;
                        } else {
                            sums[2 * bb] = s0;
                            sums[2 * bb + 1] = s1;
                        }
                    }
                }
                if (last != bb && !freed) {
                    // the last block lost its final entry to bb
                    const bool valid = okl && lane != lastpos;
                    const uint64_t s0 = wave_max_u64(valid ? key_of(kl, slot0) : 0);
                    const uint64_t s1 = wave_max_u64(valid ? key_of(kl, 1) : 0);
                    if (lane == 0) {
                        if (last < SC) {
                            L.sum[2 * last] = s0;
                            L.sum[2 * last + 1] = s1;
                        } else {
                            sums[2 * last] = s0;
                            sums[2 * last + 1] = s1;
                        }
                    }
                }
                // fixed keys carry the rank or the transitive attributes, not
                // the out-degree
                const int32_t deg = skey ? tr[v].ia : (int32_t)(vk >> 42);
                const int32_t iep = tattr ? tie[v] : heft ? wg_load(&tr[v].iev) : (int32_t)((vk >> 21) & M21);
                // a task whose inputs are still moving holds the worker until
                // they arrive
                int64_t s0 = t;
                if (data) s0 = max(t, (int64_t)wg_load(&tr[v].word));
                if (lane == 0) {
                    L.len[w] = len;
                    L.nb[w] = nb;
                    L.last[w] = newlast;
                    L.run[w] = v;
                    L.fin[w] = s0 + dk;
                    L.expend[w] = s0 + ek;
                    L.qest[w] -= ek;
                    L.rsr[w] = vr;
                    L.dgr[w] = deg;
                    put_record(&tr[v], s0, dk, w, iep, pmode);  // running, then done
                }
                nready--;
                popped++;
            }
        }
        PCLK(2);
        if (A.trace && lane == 0 && events <= max_events) {
            insp_trace_rec rec;
            rec.t = t;
            rec.nready = observed;
            rec.mode = pmode;
            rec.cnt = cnt;
            rec.peak = peak;
            rec.pushed = r;
            rec.popped = popped;
            A.trace[(d.toff - A.base) + di + events - 1] = rec;
        }
        if (done == n) break;
        // --------------------------------------------------------- advance
        uint64_t tm = ~0ull;
        for (int32_t w = lane; w < W; w += kWave)
            if (L.run[w] >= 0 && (uint64_t)L.fin[w] < tm) tm = (uint64_t)L.fin[w];
        tm = wave_min_u64(tm);
        if (tm == ~0ull) {
            status |= ST_HANG;
            break;
        }
        t = (int64_t)tm;
        PCLK(3);
        // --------------------------------------------------------- release
        r = 0;
        int32_t nc = 0, nseg = 0, ndone = 0;
        for (int32_t w0 = 0; w0 < W; w0 += kWave) {
            const int32_t wl = w0 + lane;
            const bool fin_now = wl < W && L.run[wl] >= 0 && L.fin[wl] == t;
            uint64_t mask = ballot(fin_now);
            const int32_t c_l = fin_now ? L.run[wl] : -1;
            if (fin_now) L.run[wl] = -1;
            while (mask) {
                const int l = (int)__builtin_ctzll(mask);
                mask &= mask - 1;
                const int32_t w = w0 + l;
                const int32_t c = read_lane(c_l, l);
                done++;
                ndone++;
                const int32_t deg = L.dgr[w], rs = L.rsr[w];
                const int32_t r0 = r;
                const unsigned long long dec = 0ull - ((1ull << 43) + (unsigned long long)c);
                for (int32_t e0 = 0; e0 < deg; e0 += kWave) {
                    const int32_t e = e0 + lane;
                    const bool ok = e < deg;
                    const int32_t s = ok ? col[rs + e] : 0;
                    // one wave owns the DAG's words and a row's successors are
                    // distinct (rows are deduplicated), so a plain
                    // read-modify-write replaces the atomic (a wave's accesses
                    // to one address complete in program order)
                    uint64_t old = 0;
                    if (ok) {
                        old = dep[s];
                        dep[s] = old + dec;
                    }
                    const int32_t nr = (int32_t)(old >> 43) - 1;
                    const bool rdy = ok && nr == 0, cd = ok && nr == 1;
                    const uint64_t m1 = ballot(rdy), m2 = ballot(cd);
                    if (rdy) {
                        const int32_t pos = r + lanes_below(m1);
                        fbuf[pos] = s;
                        if (pos < kFC) L.fr0[pos] = s;
                    }
                    if (cd) {
                        const int32_t pos = nc + lanes_below(m2);
                        if (pos < kCC) {
                            L.cs[pos] = s;
                            L.cu[pos] = (int32_t)((old + dec) & M43);
                        } else {
                            fbuf[2 * n + pos] = s;
                        }
                    }
                    r += __popcll(m1);
                    nc += __popcll(m2);
                }
                if (r > r0) {
                    if (lane == 0) L.seg[nseg] = r;
                    nseg++;
                }
            }
        }
        PCLK(4);
        wg_fence();
        __builtin_amdgcn_wave_barrier();
        PCLK(5);
        // successors left with one unfinished predecessor raise its IE.  The
        // predecessor is named by the atomic's result (rem 1, remaining sum);
        // that result is final unless a later completion of the same event
        // made the successor ready, in which case it is not a candidate.
        const bool single = ndone == 1;
        merged = false;
        staged = false;
        if (nc <= kWave && r <= kFC) {
            // one round trip: candidate records and the next push's frontier rows
            const bool hc = lane < nc;
            const int32_t s = hc ? L.cs[lane] : 0;
            int32_t u = hc ? L.cu[lane] : -1;
            if (hc && !single)
                for (int32_t k = 0; k < r; k++)
                    if (L.fr0[k] == s) {
                        u = -1;
                        break;
                    }
            staged = r <= kWave;
            const bool hf = staged && lane < r;
            const int32_t fv = hf ? L.fr0[lane] : 0;
            int32_t tu = 0, ts = 0, iu = 0, qu = -1, au = 0, sq = 0;
            if (u >= 0) {
                tu = tr[u].tau;
                ts = tr[s].tau;
                iu = wg_load(&tr[u].iev);
                qu = wg_load(&tr[u].qpos);
                au = tr[u].ia;
                sq = wg_load(&tr[u].seq);
            }
            int2 fe = make_int2(1, 1), fd = make_int2(1, 1);
            int32_t fa = 0, frs = 0, fie = 0;
            if (hf) {
                fe = est2[fv];
                fd = dur2[fv];
                fa = tr[fv].ia;
                frs = tr[fv].rs;
                fie = wg_load(&tr[fv].iev);
            }
            const bool cond = u >= 0 && (int64_t)tu + ts <= (int64_t)U;
            // several successors may name the same predecessor: the first lane
            // applies all of its increments
            int32_t mult = 0;
            bool lead = cond;
            for (int32_t j = 0; j < nc; j++) {
                const int32_t uj = read_lane(u, j);
                const int32_t cj = read_lane(cond ? 1 : 0, j);
                if (cj && cond && uj == u) {
                    mult++;
                    if (j < lane) lead = false;
                }
            }
            if (lead) {
                const int32_t nie = iu + mult;
                tr[u].iev = nie;
                if (qu >= 0 && !skey) {
                    const uint64_t nk = (uint64_t)au << 42 | (uint64_t)nie << 21 | (M21 - (uint64_t)sq);
                    const int32_t bk = qu >> 6;
                    if (bk < SLC) L.sk[qu] = nk;
                    else slots.k[qu] = nk;
                    if (bk < SC) {
                        atomicMax(&L.sum[2 * bk], (unsigned long long)key_of(nk, slot0));
                        atomicMax(&L.sum[2 * bk + 1], (unsigned long long)key_of(nk, 1));
                    } else {
                        wg_fetch_max(&sums[2 * bk], (unsigned long long)key_of(nk, slot0));
                        wg_fetch_max(&sums[2 * bk + 1], (unsigned long long)key_of(nk, 1));
                    }
                }
            }
            // a raised predecessor that became ready in this very event: its
            // staged row must carry the new IE
            uint64_t lm = ballot(lead && qu == -1);
            while (lm) {
                const int l = (int)__builtin_ctzll(lm);
                lm &= lm - 1;
                const int32_t uu = read_lane(u, l), kk = read_lane(mult, l);
                const uint64_t fm = ballot(hf && fv == uu);
                if (fm && lane == (int)__builtin_ctzll(fm)) fie += kk;
            }
            int32_t pos = lane;
            if (nseg > 1 && hf) {
                // rank of this entry among the ascending runs of the completions
                int32_t rank = 0, lo = 0;
                for (int32_t g = 0; g < nseg; g++) {
                    const int32_t hi = L.seg[g];
                    if (lane >= lo && lane < hi) {
                        rank += lane - lo;
                    } else {
                        int32_t a = lo, b = hi;
                        while (a < b) {
                            const int32_t mid = (a + b) >> 1;
                            if (L.fr0[mid] < fv) a = mid + 1;
                            else b = mid;
                        }
                        rank += a - lo;
                    }
                    lo = hi;
                }
                pos = rank;
            }
            if (!staged && nseg > 1) {
                // frontier too large to stage: merge ids in LDS, rows loaded at push
                for (int32_t i = lane; i < r; i += kWave) {
                    const int32_t x = L.fr0[i];
                    int32_t rank = 0, lo = 0;
                    for (int32_t g = 0; g < nseg; g++) {
                        const int32_t hi = L.seg[g];
                        if (i >= lo && i < hi) {
                            rank += i - lo;
                        } else {
                            int32_t a = lo, b = hi;
                            while (a < b) {
                                const int32_t mid = (a + b) >> 1;
                                if (L.fr0[mid] < x) a = mid + 1;
                                else b = mid;
                            }
                            rank += a - lo;
                        }
                        lo = hi;
                    }
                    L.fr1[rank] = x;
                }
                merged = true;
            }
            if (hf) {
                L.pre[pos] = fv;
                L.pre[64 + pos] = fe.x;
                L.pre[128 + pos] = fe.y;
                L.pre[192 + pos] = fd.x;
                L.pre[256 + pos] = fd.y;
                L.pre[320 + pos] = fa;
                L.pre[384 + pos] = frs;
                L.pre[448 + pos] = fie;
            }
        } else {
            for (int32_t i0 = 0; i0 < nc; i0 += kWave) {
                const int32_t i = i0 + lane;
                if (i < nc) {
                    const int32_t s = i < kCC ? L.cs[i] : wg_load(&fbuf[2 * n + i]);
                    int32_t u = -1;
                    if (single && i < kCC) {
                        u = L.cu[i];
                    } else {
                        const uint64_t wd = wg_load(&dep[s]);
                        if ((wd >> 43) == 1) u = (int32_t)(wd & M43);
                    }
                    if (u >= 0) {
                        const int32_t tu = tr[u].tau, ts = tr[s].tau;
                        const int32_t pu = wg_load(&tr[u].qpos);
                        if ((int64_t)tu + ts <= (int64_t)U) {
                            wg_fetch_add(&tr[u].iev, 1);
                            if (pu >= 0 && !skey) {
                                const int32_t bk = pu >> 6;
                                const uint64_t nk = (bk < SLC ? (uint64_t)atomicAdd(&L.sk[pu], 1ull << 21)
                                                              : (uint64_t)wg_fetch_add(&slots.k[pu], 1ull << 21)) +
                                                    (1ull << 21);
                                if (bk < SC) {
                                    atomicMax(&L.sum[2 * bk], (unsigned long long)key_of(nk, slot0));
                                    atomicMax(&L.sum[2 * bk + 1], (unsigned long long)key_of(nk, 1));
                                } else {
                                    wg_fetch_max(&sums[2 * bk], (unsigned long long)key_of(nk, slot0));
                                    wg_fetch_max(&sums[2 * bk + 1], (unsigned long long)key_of(nk, 1));
                                }
                            }
                        }
                    }
                }
            }
            wg_fence();
            // several completions: merge their ascending runs by rank
            if (nseg > 1) {
                const bool in_lds = r <= kFC;
                for (int32_t i0 = 0; i0 < r; i0 += kWave) {
                    const int32_t i = i0 + lane;
                    if (i < r) {
                        const int32_t x = in_lds ? L.fr0[i] : fbuf[i];
                        int32_t rank = 0, lo = 0;
                        for (int32_t g = 0; g < nseg; g++) {
                            const int32_t hi = L.seg[g];
                            if (i >= lo && i < hi) {
                                rank += i - lo;
                            } else {
                                int32_t a = lo, b = hi;  // count of run g below x
                                while (a < b) {
                                    const int32_t mid = (a + b) >> 1;
                                    const int32_t y = in_lds ? L.fr0[mid] : fbuf[mid];
                                    if (y < x) a = mid + 1;
                                    else b = mid;
                                }
                                rank += a - lo;
                            }
                            lo = hi;
                        }
                        if (in_lds) L.fr1[rank] = x;
                        else fbuf[n + rank] = x;
                    }
                }
                merged = true;
            }
        }
        PCLK(7);
        wg_fence();
        __builtin_amdgcn_wave_barrier();
        PCLK(8);
    }
#ifdef INSP_PHASE_CLOCKS
    if (lane == 0 && d.id < 8192)
        for (int i = 0; i < 32; i++) g_phase_clk[d.id * 32 + i] = pc[i];
#endif
    if (lane == 0) {
        A.makespan[di] = (status & ST_HANG) ? -1 : t;
        if (A.n_events) A.n_events[di] = events;
        if (status) atomicOr(&A.stat[2 * d.id], status);
        A.stat[2 * d.id + 1] = events;
    }
}

// ---------------------------------------------------------------------------
// Machines of at most 64 workers (WPL = 1) or 128 (WPL = 2): lane w holds
// the state of worker w (and of worker w + 64) in registers -- running task,
// its finish and expected-end times, queue length, block count, last block,
// the running task's row and first successors -- so pushes, pops and the
// advance read no memory for it.  Same event order and results as the
// general loop above.
//
// What bounds it is one wave's chain of dependent steps per event: waits on
// LDS and L2 round trips, and the issue of several hundred instructions at
// 4 clocks and more each.  The loop keeps everything else off that chain:
//   - 32-bit keys.  IA and IE take `a` bits each (a = bit length of the DAG's
//     largest out-degree; IE <= IA) and the push order `s` bits (s = bit length
//     of n - 1), under a valid bit.  Each entry keeps both rules' keys,
//       kA = V | IA << (a+s) | IE << s | (2^s-1-seq)   (ability; under the
//                                                        FIFO policy V | (2^s-1-seq))
//       kE = V | IE << (a+s) | IA << s | (2^s-1-seq)   (efficiency),
//     so a pop compares plain words.  Launches with a DAG whose keys need more
//     than 32 bits keep one 64-bit key per entry instead (see Keys).
//   - A worker's best entry is known before it is popped.  Per worker and
//     rule, `best` holds the queue's largest key and its slot (key << 32 | slot).
//     Pushes and IE increments raise it with an LDS atomicMax; a pop empties
//     it and asks the work-group's second wave (keep_best) to find the next
//     one, which it does while this wave simulates the following events.  The
//     second wave rescans only the block the pop changed, merges its maximum
//     into the per-block maxima with atomicMax and takes the largest of
//     those.  Keys only grow while a task is queued, so maxima raised by
//     this wave meanwhile and scanned values that are out of date by then
//     merge to the right result in any order; a pop waits for a rescan still
//     under way.  Every slot without a live entry holds zero keys, so scans
//     read whole blocks unpredicated: valid keys carry the top bit.
//   - A popped entry's slot stays empty for one of the worker's next pushes
//     (empty slots are chained through their first-edge field), so a pop
//     moves no other entry; a queue keeps its blocks, of which each push adds
//     at most one entry's share: n / 64 + W blocks hold any run.
//   - All workers that are idle pop at once, a lane each.
//   - An event with one completion of at most 64 successors (most are) keeps
//     its newly ready tasks in the lanes that released them: their rows are
//     loaded there and the pushes take them in lane (ascending id) order, with
//     no list in between.  Its loads are unpredicated (lanes without a task
//     read element 0) so that the compiler issues them together.
//   - Pointers and parameters that only uncommon paths use are kept in LDS
//     (kCold*), not in scalar registers, whose spills cost the common path.
//   - A wave that runs alone issues an instruction every 4 clocks; a scalar
//     instruction that reads what a vector compare has just written waits 16
//     more, a taken branch costs 21, an untaken one 7 and an LDS round trip 48
//     (measured).  So uniform tests are made on scalar state where it allows
//     (no queue block past the ones in LDS, no bad duration), lane updates are
//     selects instead of masked blocks, and uncommon code is out of line.
// Measured: layered DAG of 1,000 tasks 1.6 us an event, tiled Cholesky of 11,480
// 1.55 and a power-law DAG of 20,000 on 77 workers 2.1, against 3.0, 3.0 and 4.9
// with the scan in the simulating wave (above 64 workers in the general loop),
// pops one by one and frontier lists.

__device__ __forceinline__ uint32_t wave_max_k(uint32_t x) { return wave_max_u32f(x); }
__device__ __forceinline__ unsigned long long wave_max_k(unsigned long long x) { return wave_max_u64f(x); }

// Order this wave's LDS and global accesses as written (the hardware already
// takes them in issue order within a work-group).
__device__ __forceinline__ void keep_order() { __atomic_signal_fence(__ATOMIC_SEQ_CST); }

template <typename T>
__device__ __forceinline__ T lds_load(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T>
__device__ __forceinline__ void lds_store(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Element i of a per-task array (n <= 2^21, elements of at most 32 bytes: the
// byte offset fits 32 bits, so the access is a scalar base plus one register).
template <typename T>
__device__ __forceinline__ T *at(T *base, int32_t i) {
    return reinterpret_cast<T *>(
        reinterpret_cast<typename std::conditional<std::is_const<T>::value, const char, char>::type *>(base) +
        (uint32_t)i * (uint32_t)sizeof(T));
}

// LDS of the one-wave loop: arrays of fixed size first (their offsets are
// instruction immediates), then the ones whose size the launch picks.
template <int WPL>
struct LaneLds {
    static constexpr int kMW = WPL * kWave;
    static constexpr int kBest = 0;                     // uint64 [2 * kMW]: each worker's best entry under either rule
    static constexpr int kRun = kBest + 16 * kMW;       // int2 [kMW]: running task or -1 and its finish (read-ahead)
    static constexpr int kCold = kRun + 8 * kMW;        // uint64 [8]: pointers of the uncommon paths
    static constexpr int kBpos = kCold + 64;            // int32 [2 * kMW], 64-bit keys: slots of the best entries
    static constexpr int kReq = kBpos + 8 * kMW;        // int32 [kMW]: block to rescan + 1, or 0
    static constexpr int kRnb = kReq + 4 * kMW;         // int32 [kMW]: blocks of the queue
    static constexpr int kSeg = kRnb + 4 * kMW;         // int32 [kMW]: ends of the runs of newly ready tasks
    static constexpr int kSucc = kSeg + 4 * kMW;        // int32 [kPF]: a completing task's first successors
    static constexpr int kPre = kSucc + 4 * kPF;        // int32 [8 * 64]: staged frontier rows
    static constexpr int kFr0 = kPre + 4 * 8 * kWave;   // int32 [kFC]
    static constexpr int kFr1 = kFr0 + 4 * kFC;         // int32 [kFC]
    static constexpr int kCs = kFr1 + 4 * kFC;          // int32 [kCC]
    static constexpr int kCu = kCs + 4 * kCC;           // int32 [kCC]
    static constexpr int kHs = kCu + 4 * kCC;           // int32 [4]: DAG index, finished, read-ahead's sink, rescans on
    static constexpr int kFixed = kHs + 16;
    unsigned long long *mx;  // [2 * sum_cap] block maxima
    unsigned long long *sk;  // [64 * key_cap] keys of the low blocks' entries
    unsigned long long *sx;  // [64 * slot_cap] payload (task, durations) of the lowest
    int32_t *srs;            // [64 * slot_cap] ... and their first edges
    int32_t *blist;          // [W * lb] first block ids of each worker
    static constexpr size_t bytes(int mw, int sc, int lb, int slc, int slk) {
        return (size_t)kFixed + (size_t)sc * 16 + (size_t)slk * 512 + (size_t)slc * 768 + (size_t)mw * lb * 4;
    }
    __device__ __forceinline__ static char *raw() {
        extern __shared__ int64_t lds64[];
        return reinterpret_cast<char *>(lds64);
    }
    template <typename T>
    __device__ __forceinline__ static T *arr(int off) { return reinterpret_cast<T *>(raw() + off); }
    __device__ __forceinline__ explicit LaneLds(const SimArgs &A) {
        mx = arr<unsigned long long>(kFixed);
        sk = mx + 2 * A.sum_cap;
        sx = sk + 64 * A.key_cap;
        srs = reinterpret_cast<int32_t *>(sx + 64 * A.slot_cap);
        blist = srs + 64 * A.slot_cap;
    }
};
static_assert(LaneLds<1>::kFixed % 16 == 0 && LaneLds<2>::kFixed % 16 == 0, "aligned for 64-bit arrays");

// Pointers kept in LDS (LaneLds::kCold).
enum ColdPtr { kColdFbuf = 0, kColdWblk, kColdKeys, kColdPayload, kColdEdges, kColdSums };

template <int WPL, typename T>
__device__ __forceinline__ T *cold(int i) {
    const uint64_t v = (uint64_t)uniform64((int64_t)LaneLds<WPL>::template arr<uint64_t>(LaneLds<WPL>::kCold)[i]);
    return (T *)(__attribute__((address_space(1))) T *)v;
}

template <int WPL, int KK>
__device__ __forceinline__ Keys<KK> make_keys(const SimArgs &A, const LaneLds<WPL> &L) {
    Keys<KK> K;
    K.ka = reinterpret_cast<typename Keys<KK>::T *>(L.sk);
    K.ke = Keys<KK>::kBig ? nullptr : K.ka + 64 * A.key_cap;  // the two 32-bit arrays fill the 64-bit key storage
    K.o0 = A.policy == INSP_POLICY_FIFO ? 2 : A.policy == INSP_POLICY_HEFT ? 3 : 0;
    return K;
}

// The work-group's second wave: answers rescan requests until the DAG is done.
template <int WPL, int KK>
__device__ void keep_best(const SimArgs &A, int32_t di) {
    using KT = typename Keys<KK>::T;
    using LL = LaneLds<WPL>;
    constexpr bool kBig = Keys<KK>::kBig;
    const LL L(A);
    const int lane = lane_id();
    const DagDesc d = A.desc[di];
    const SlotPool slots = A.slots.at(64 * d.blk_off);
    unsigned long long *sums = A.sums + 2 * d.blk_off;
    const int32_t *wblk = A.paux + d.wl_off;
    const Keys<KK> K = make_keys<WPL, KK>(A, L);
    const int32_t SC = A.sum_cap, SLK = A.key_cap, kLB = A.lb;
    unsigned long long *mx = L.mx, *best = LL::template arr<unsigned long long>(LL::kBest);
    int32_t *bpos = LL::template arr<int32_t>(LL::kBpos), *req = LL::template arr<int32_t>(LL::kReq);
    const int32_t *rnb = LL::template arr<int32_t>(LL::kRnb), *hs = LL::template arr<int32_t>(LL::kHs);
    // rule-r key of block b's entry in this lane
    auto entry = [&](int32_t b, int r) -> KT {
        if (b < SLK) return K.lds(b * 64 + lane, r);
        const uint64_t raw = wg_load(&slots.k[b * 64 + lane]);
        settle(raw);
        return K.rule(raw, r);
    };
    for (int64_t it = 0; it < kHelperSpin; it++) {
        if (lds_load(&hs[1])) break;
        if (!lds_load(&hs[3])) {
            __builtin_amdgcn_s_sleep(2);
            continue;
        }
        bool any = false;
#pragma unroll
        for (int k = 0; k < WPL; k++) {
            const int32_t wl = lane + k * kWave, rq = lds_load(&req[wl]);
            uint64_t m = ballot(rq != 0);
            any |= m != 0;
            keep_order();
            while (m) {
                const int l = (int)__builtin_ctzll(m);
                const int32_t w = l + k * kWave;
                m &= m - 1;
                const int32_t b = read_lane(rq, l) - 1, nbw = uniform(min(lds_load(&rnb[w]), d.maxb));
                keep_order();
                if (b < 0 || b >= d.nblk) continue;  // never
                // the changed block's maxima under both rules, and their slots
                const KT k0 = entry(b, 0), k1 = entry(b, 1);
                const KT s0 = wave_max_k(k0), s1 = wave_max_k(k1);
                int32_t bp0 = b * 64 + (int32_t)__builtin_ctzll(ballot(k0 == s0));
                int32_t bp1 = b * 64 + (int32_t)__builtin_ctzll(ballot(k1 == s1));
                unsigned long long bm0, bm1;
                if constexpr (kBig) {
                    bm0 = s0;
                    bm1 = s1;
                } else {
                    bm0 = s0 ? (unsigned long long)s0 << 32 | (uint32_t)bp0 : 0ull;
                    bm1 = s1 ? (unsigned long long)s1 << 32 | (uint32_t)bp1 : 0ull;
                }
                const bool glob = b >= SC;
                bool found = true;
                if (lane == 0) {
                    if (!glob) {
                        atomicMax(&mx[2 * b], bm0);
                        atomicMax(&mx[2 * b + 1], bm1);
                    } else {
                        wg_fetch_max(&sums[2 * b], bm0);
                        wg_fetch_max(&sums[2 * b + 1], bm1);
                    }
                }
                if (nbw > 1) {
                    // the largest block maximum under each rule
                    keep_order();
                    bm0 = bm1 = 0;
                    int32_t b0 = -1, b1 = -1;
                    for (int32_t i0 = 0; i0 < nbw; i0 += kWave) {
                        const int32_t i = i0 + lane;
                        int32_t bi = -1;
                        if (i < nbw) {
                            bi = i < kLB ? L.blist[w * kLB + i] : wg_load(&wblk[(int64_t)w * d.maxb + i]);
                            if (bi >= d.nblk) bi = -1;
                        }
                        unsigned long long m0 = 0, m1 = 0;
                        if (bi >= 0) {
                            if (bi < SC) {
                                m0 = lds_load(&mx[2 * bi]);
                                m1 = lds_load(&mx[2 * bi + 1]);
                            } else {
                                m0 = __hip_atomic_load(&sums[2 * bi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                m1 = __hip_atomic_load(&sums[2 * bi + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            }
                        }
                        if (m0 > bm0) {
                            bm0 = m0;
                            b0 = bi;
                        }
                        if (m1 > bm1) {
                            bm1 = m1;
                            b1 = bi;
                        }
                    }
                    const unsigned long long g0 = wave_max_u64f(bm0), g1 = wave_max_u64f(bm1);
                    if constexpr (kBig) {
                        // the entries those maxima stand for
                        const int32_t c0 = read_lane(b0, (int)__builtin_ctzll(ballot(bm0 == g0)));
                        const int32_t c1 = read_lane(b1, (int)__builtin_ctzll(ballot(bm1 == g1)));
#pragma unroll
                        for (int r = 0; r < 2; r++) {
                            const int32_t br = r ? c1 : c0;
                            if (br < 0) continue;
                            const uint64_t hit = ballot(entry(br, r) == (r ? g1 : g0));
                            if (hit) (r ? bp1 : bp0) = br * 64 + (int32_t)__builtin_ctzll(hit);
                            else found = false;
                        }
                    }
                    bm0 = g0;
                    bm1 = g1;
                }
                // a maximum raised while it was looked for (kWide): the request
                // stands and is answered again
                if (!found) continue;
                if (glob) __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the maxima in global memory are merged
                if (lane == 0) {
                    if constexpr (kBig) {
                        best[2 * w] = bm0;
                        best[2 * w + 1] = bm1;
                        bpos[2 * w] = bp0;
                        bpos[2 * w + 1] = bp1;
                    } else {
                        atomicMax(&best[2 * w], bm0);
                        atomicMax(&best[2 * w + 1], bm1);
                    }
                    keep_order();
                    lds_store(&req[w], 0);
                }
            }
        }
        if (!any) __builtin_amdgcn_s_sleep(1);
    }
}

// Worker w's value of a per-worker register (w is wave-uniform).
template <int WPL>
__device__ __forceinline__ int32_t of_worker(const int32_t (&x)[WPL], int32_t w) {
    if constexpr (WPL == 1) return read_lane(x[0], w);
    else return w < kWave ? read_lane(x[0], w) : read_lane(x[1], w - kWave);
}

typedef int32_t row4 __attribute__((ext_vector_type(4), aligned(4)));

// DATA: the data model (A.data_bw > 0), as the general loop runs it: a push
// adds each worker's input transfer ticks to its cost and records the task's
// input arrival time, a pop starts its task when the inputs are in, and the
// efficiency-with-locality rule prefers tasks whose inputs are.
// With kNarrow the keys of every DAG of the launch fit (launch_sim checks).
template <int WPL, int KK, bool DATA>
__device__ void sim_lane(const SimArgs &A, int32_t di) {
    static_assert(WPL == 1 || WPL == 2, "a lane holds one or two workers");
    using LL = LaneLds<WPL>;
    using KT = typename Keys<KK>::T;
    constexpr bool kBig = Keys<KK>::kBig;
    constexpr int WB = WPL == 1 ? 6 : 7;              // bits of a worker id
    constexpr uint32_t kLim = (1u << (32 - WB)) - 1;  // costs this far past now are compared in 64 bits
    constexpr int kPred = 8;                          // predecessors of a task read together
    const LL L(A);
    const int lane = lane_id();
    const DagDesc d = A.desc[di];
    const int32_t n = d.n, ncpu = d.n_cpu, W = d.n_cpu + d.n_gpu;
    int32_t status = A.stat[2 * d.id];
    if (n == 0 || status != 0) {
        if (lane == 0) {
            A.makespan[di] = status ? -1 : 0;
            if (A.n_events) A.n_events[di] = 0;
        }
        return;
    }
    const int64_t ub = d.toff - A.base;
    const int32_t *col = A.col + d.eoff;
    TaskRec *tr = A.tr + d.toff;
    unsigned long long *dep = A.dep + d.toff;
    const int2 *est2 = reinterpret_cast<const int2 *>(A.est) + ub;
    const int2 *dur2 = reinterpret_cast<const int2 *>(A.dur) + ub;
    const int32_t maxb = d.maxb;
    const int32_t SC = A.sum_cap;
    const int32_t kLB = A.lb;
    const int32_t SLC = A.slot_cap;  // blocks [0, SLC) keep their entries' payload in LDS
    const int32_t SLK = A.key_cap;   // blocks [0, SLK) (SLK >= SLC) keep their keys in LDS
    const int32_t NB = min(SLC, SC); // blocks [0, NB) are in LDS with all they have
    unsigned long long *mx = L.mx, *best = LL::template arr<unsigned long long>(LL::kBest);
    int2 *lrun = LL::template arr<int2>(LL::kRun);
    int32_t *req = LL::template arr<int32_t>(LL::kReq), *rnb = LL::template arr<int32_t>(LL::kRnb);
    int32_t *bpos = LL::template arr<int32_t>(LL::kBpos), *seg = LL::template arr<int32_t>(LL::kSeg);
    int32_t *succ = LL::template arr<int32_t>(LL::kSucc), *pre = LL::template arr<int32_t>(LL::kPre);
    int32_t *fr0 = LL::template arr<int32_t>(LL::kFr0), *fr1 = LL::template arr<int32_t>(LL::kFr1);
    int32_t *cs = LL::template arr<int32_t>(LL::kCs), *cu = LL::template arr<int32_t>(LL::kCu);
    // the global queue pool and block maxima, for blocks not held in LDS
    auto pool = [&]() {
        SlotPool s;
        s.k = cold<WPL, unsigned long long>(kColdKeys);
        s.x = cold<WPL, unsigned long long>(kColdPayload);
        s.rs = cold<WPL, int32_t>(kColdEdges);
        return s;
    };
    auto gsums = [&]() { return cold<WPL, unsigned long long>(kColdSums); };

    // initial frontier (tasks without predecessors, ascending) and the
    // largest out-degree, which sizes the key fields
    int32_t r = 0;
    uint32_t mdeg = 0, longest = 0;
    {
        int32_t *fbuf = A.fbuf + 3 * d.toff;  // [0,n) runs, [n,2n) merged, [2n,3n) candidates
        for (int32_t i0 = 0; i0 < n; i0 += kWave) {
            int32_t i = i0 + lane;
            bool ok = false;
            if (i < n) {
                ok = (dep[i] >> 43) == 0;
                mdeg = max(mdeg, (uint32_t)tr[i].ia);
                const int2 du = dur2[i];
                longest = max(longest, max((uint32_t)(du.x - 1), (uint32_t)(du.y - 1)));
            }
            uint64_t mk = ballot(ok);
            if (ok) {
                int32_t pos = r + lanes_below(mk);
                fbuf[pos] = i;
                if (pos < kFC) fr0[pos] = i;
            }
            r += __popcll(mk);
        }
        mdeg = wave_max_u32f(mdeg);
        longest = wave_max_u32f(longest);
        if (lane == 0) {
            uint64_t *c = LL::template arr<uint64_t>(LL::kCold);
            const SlotPool slots = A.slots.at(64 * d.blk_off);
            c[kColdFbuf] = (uint64_t)fbuf;
            c[kColdWblk] = (uint64_t)(A.paux + d.wl_off);
            c[kColdKeys] = (uint64_t)slots.k;
            c[kColdPayload] = (uint64_t)slots.x;
            c[kColdEdges] = (uint64_t)slots.rs;
            c[kColdSums] = (uint64_t)(A.sums + 2 * d.blk_off);
        }
    }
    const bool bad_dur = longest >= (uint32_t)INSP_MAX_TICK;  // some duration is out of range: the pushes look for it
    const uint32_t abits = field_bits(mdeg), sbits = field_bits(n - 1);
    KeyFmt kf;
    kf.sa = sbits;
    kf.sb = abits + sbits;
    kf.smask = (1u << sbits) - 1;
    kf.amask = (1u << abits) - 1;
    kf.fifo = A.policy == INSP_POLICY_FIFO;
    const bool heft = KK == kFixed && A.policy == INSP_POLICY_HEFT;
    const bool tattr = KK == kFixed && A.attr_mode == INSP_ATTR_TRANSITIVE;
    const int64_t *rk = A.rank + d.toff;
    const int32_t *tia = A.tia + d.toff, *tie = A.tie + d.toff;
    const Keys<KK> K = make_keys<WPL, KK>(A, L);
    const int32_t U = A.dag_u[d.id];
    // data model: inputs move between memory nodes (the host for the CPU
    // workers, one per GPU worker)
    const int32_t *prp = A.pprp + d.toff + d.id, *pred = A.ppred + d.eoff;
    int32_t *dxc = A.dxc + d.toff;
    long long *barr = A.barr + d.blk_off;
    // block arrival bounds matter only where the locality rule can be used
    const bool lrule = DATA && (A.policy == INSP_POLICY_INSPIRIT || A.policy == INSP_POLICY_LOCALITY);
    if constexpr (DATA)  // each output's transfer ticks, once per run (no division at the pushes)
        for (int32_t i = lane; i < n; i += kWave)
            dxc[i] = (int32_t)(((int64_t)1024 * A.dkib[d.toff + i] + A.data_bw - 1) / A.data_bw);

    const int32_t s_inc = A.s_inc > 0 ? A.s_inc : max(1, (W + 3) / 4);
    const int32_t s_dec = A.s_dec > 0 ? A.s_dec : max(1, (W + 1) / 2);
    const int32_t dec_step = A.dec_step > 0 ? A.dec_step : s_dec;
    const int32_t cc = A.c >= 0 ? A.c : s_dec / 2;
    const bool kset = A.k_num > 0 && A.k_den > 0;
    const int32_t k_num = kset ? A.k_num : W;
    const int32_t k_den = kset ? A.k_den : A.dag_taubar[d.id];
    const int32_t max_events = A.max_events > 0 ? A.max_events : n + 1;
    const int policy = A.policy;

    // this lane's workers
    bool wok[WPL], wcpu[WPL];
    int32_t run[WPL], len[WPL], nb[WPL], rsr[WPL], dgr[WPL];
    int32_t hole[WPL], tail[WPL];  // slots for the next pushes: an empty one (or -1), and the one past the last entry
    row4 pfa[WPL], pfb[WPL];  // the running task's first successors
    int64_t fin[WPL], expend[WPL], qest[WPL];  // expend is 0 while the worker is idle
    unsigned long long pk0[WPL], pk1[WPL];  // 64-bit keys: the best entry pushed or raised since the last pop, by rule ...
    int32_t pp0[WPL], pp1[WPL];             // ... and its slot
#pragma unroll
    for (int k = 0; k < WPL; k++) {
        const int32_t w = lane + k * kWave;
        wok[k] = w < W;
        wcpu[k] = w < ncpu;
        run[k] = -1;
        len[k] = nb[k] = rsr[k] = dgr[k] = 0;
        hole[k] = tail[k] = -1;
        pfa[k] = pfb[k] = row4{0, 0, 0, 0};
        fin[k] = expend[k] = qest[k] = 0;
        pk0[k] = pk1[k] = 0;
        pp0[k] = pp1[k] = 0;
        best[2 * w] = 0;
        best[2 * w + 1] = 0;
        if constexpr (kBig) bpos[2 * w] = bpos[2 * w + 1] = 0;
        req[w] = 0;
    }

    // blocks are taken in order, lowest first; every slot starts empty (zero keys)
    int32_t nused = 0;
    {
        unsigned long long *sums = A.sums + 2 * d.blk_off, *sk = A.slots.at(64 * d.blk_off).k;
        for (int32_t b = lane; b < d.nblk; b += kWave) {
            if (b < SC) {
                mx[2 * b] = 0;
                mx[2 * b + 1] = 0;
            } else {
                sums[2 * b] = 0;
                sums[2 * b + 1] = 0;
            }
            if constexpr (DATA) barr[b] = 0;
        }
        for (int32_t b = 0; b < d.nblk; b++) {
            if (b < SLK) K.put(b * 64 + lane, 0);
            else sk[b * 64 + lane] = 0;
        }
    }
    wg_fence();
    if (lane == 0) lds_store(LL::template arr<int32_t>(LL::kHs) + 3, 1);

    // where this event's frontier is: in the lanes of `fm` (their rows in the
    // f_ registers), staged by rank in `pre`, or listed in fr0 / fr1 / fbuf
    bool merged = false, staged = false, inlane = false;
    uint64_t fm = 0;
    int32_t f_v = 0, f_ia = 0, f_ie = 0, f_rs = 0, f_pa = 0, f_pz = 0;
    int2 f_e = make_int2(1, 1), f_d = make_int2(1, 1);

    int64_t t = 0, prev_t = 0;
    int32_t nready = 0, events = 0, done = 0, seq = 0;
    int32_t peak = 0, prev_n = 0, cnt = 0;
    int mode = INSP_MODE_ABILITY;
#ifdef INSP_PHASE_CLOCKS
    unsigned long long pc[32] = {0}, pc_last = clock64();
#endif

    // lanes with `on`: the IE of queued task (slot qu; push order and worker
    // qw) is now nie with out-degree ia: its keys and the maxima they enter
    auto raise = [&](bool on, int32_t qu, int32_t qw, int32_t ia, int32_t nie) {
        const int32_t wu = qw >> 21, bk = qu >> 6;
        const uint32_t sq = (uint32_t)qw & (uint32_t)M21;
        uint64_t word;
        unsigned long long m0, m1;
        if constexpr (kBig) {
            word = K.big((uint64_t)ia << 21 | (uint64_t)nie, sq);
            m0 = K.rule(word, 0);
            m1 = K.rule(word, 1);
        } else {
            const uint32_t na = kf.ka((uint32_t)ia, (uint32_t)nie, sq), ne = kf.ke((uint32_t)ia, (uint32_t)nie, sq);
            word = (uint64_t)ne << 32 | na;
            m0 = (unsigned long long)na << 32 | (uint32_t)qu;
            m1 = (unsigned long long)ne << 32 | (uint32_t)qu;
        }
        if (USUALLY(nused <= NB) || (ballot(on) & ballot(bk >= NB)) == 0) {
            if (on) {
                K.put(qu, word);
                keep_order();
                atomicMax(&mx[2 * bk], m0);
                atomicMax(&mx[2 * bk + 1], m1);
            }
        } else {
            unsigned long long *gk = pool().k, *sums = gsums();
            if (on) {
                if (bk < SLK) K.put(qu, word);
                else gk[qu] = word;
                keep_order();
                if (bk < SC) {
                    atomicMax(&mx[2 * bk], m0);
                    atomicMax(&mx[2 * bk + 1], m1);
                } else {
                    wg_fetch_max(&sums[2 * bk], m0);
                    wg_fetch_max(&sums[2 * bk + 1], m1);
                }
            }
        }
        if constexpr (!kBig) {
            if (on) {
                atomicMax(&best[2 * wu], m0);
                atomicMax(&best[2 * wu + 1], m1);
            }
        } else {
            uint64_t left = ballot(on);
            while (left) {
                const int l = (int)__builtin_ctzll(left);
                left &= left - 1;
                const unsigned long long a0 = read_lane64(m0, l), a1 = read_lane64(m1, l);
                const int32_t w = read_lane(wu, l), q = read_lane(qu, l);
#pragma unroll
                for (int k = 0; k < WPL; k++)
                    if (lane + k * kWave == w) {
                        if (a0 > pk0[k]) {
                            pk0[k] = a0;
                            pp0[k] = q;
                        }
                        if (a1 > pk1[k]) {
                            pk1[k] = a1;
                            pp1[k] = q;
                        }
                    }
            }
        }
    };

    for (;;) {
        PCLK(9);
        if (RARELY(++events > max_events)) {
            status |= ST_HANG;
            break;
        }
        // ------------------------------------------------------------ push
        if (r > 0) {
            // this lane's loads past now: the rest of the running task's estimate
            // plus the estimates queued, saturated at kLim (as are lanes without a
            // worker), and the slot of the next push (-1: a new block)
            uint32_t ld[WPL];
            int32_t nslot[WPL], used[WPL];  // used: the empty slot a push took
#pragma unroll
            for (int k = 0; k < WPL; k++) {
                const uint64_t x = (uint64_t)(max(expend[k], t) - t) + (uint64_t)qest[k];
                ld[k] = wok[k] && x < kLim ? (uint32_t)x : kLim;
                nslot[k] = hole[k] >= 0 ? hole[k] : tail[k];
                used[k] = -1;
            }
            for (int32_t i0 = 0;; i0 += kWave) {
                if (RARELY(!inlane)) {
                    const int32_t idx = i0 + lane;
                    const bool in = idx < r;
                    fm = ballot(in);
                    if (staged) {
                        if (in) {
                            f_v = pre[idx];
                            f_e = make_int2(pre[64 + idx], pre[128 + idx]);
                            f_d = make_int2(pre[192 + idx], pre[256 + idx]);
                            f_ia = pre[320 + idx];
                            f_rs = pre[384 + idx];
                            f_ie = pre[448 + idx];
                        }
                    } else {
                        const int32_t *fbuf = cold<WPL, int32_t>(kColdFbuf);
                        if (in) {
                            if (r <= kFC) f_v = merged ? fr1[idx] : fr0[idx];
                            else f_v = merged ? fbuf[n + idx] : fbuf[idx];
                            f_e = est2[f_v];
                            f_d = dur2[f_v];
                            const int4 fx = *reinterpret_cast<const int4 *>(&tr[f_v].iev);  // IE, IA, tau, first edge
                            f_ie = fx.x;
                            f_ia = fx.y;
                            f_rs = fx.w;
                            // fixed keys: the rank (low and high words), or the transitive attributes
                            if (heft) {
                                const int64_t rv = rk[f_v];
                                f_ia = (int32_t)(uint32_t)rv;
                                f_ie = (int32_t)(uint32_t)((uint64_t)rv >> 32);
                            } else if (tattr) {
                                f_ia = tia[f_v];
                                f_ie = tie[f_v];
                            }
                        }
                    }
                    if constexpr (DATA) {
                        if (in) {
                            f_pa = prp[f_v];
                            f_pz = prp[f_v + 1];
                        }
                    }
                }
                const bool ok = __builtin_amdgcn_inverse_ballot_w64(fm);
                if (RARELY(bad_dur))
                    if (fm & ballot(max((uint32_t)(f_d.x - 1), (uint32_t)(f_d.y - 1)) >= (uint32_t)INSP_MAX_TICK))
                        status |= ST_DUR;
                // data model: memory node and transfer ticks of each task's first
                // predecessors' outputs (two round trips for all tasks together)
                int32_t pn[kPred], px[kPred];
                if constexpr (DATA) {
                    const int32_t np = ok ? f_pz - f_pa : 0;
                    int32_t pu[kPred];
#pragma unroll
                    for (int k = 0; k < kPred; k++) pu[k] = pred[ok && k < np ? f_pa + k : 0];
#pragma unroll
                    for (int k = 0; k < kPred; k++) {
                        const int32_t u = k < np ? pu[k] : 0;
                        pn[k] = at(tr, u)->qpos;
                        px[k] = *at(dxc, u);
                    }
#pragma unroll
                    for (int k = 0; k < kPred; k++) {
                        const int32_t wu = -2 - pn[k];  // worker of a finished task
                        pn[k] = wu < ncpu ? 0 : 1 + wu - ncpu;
                    }
                }
                PCLK(16);
                // lane j: slot, push order and worker of its task, and (data
                // model) its input transfer ticks
                int32_t pq = 0, wsj = 0;
                int64_t xsj = 0;
                const int32_t sqj = seq + lanes_below(fm);
                uint64_t todo = fm;
                while (todo) {
                    const int j = (int)__builtin_ctzll(todo);
                    todo &= todo - 1;
                    const int32_t e0 = read_lane(f_e.x, j), e1 = read_lane(f_e.y, j);
                    // DMDA's transfer term: ticks to move the inputs whose home
                    // node is not the worker's (an item stays where it was made)
                    int64_t xk[WPL];
#pragma unroll
                    for (int k = 0; k < WPL; k++) xk[k] = 0;
                    if constexpr (DATA) {
                        const int32_t pa = read_lane(f_pa, j), np = read_lane(f_pz, j) - pa;
#pragma unroll
                        for (int q = 0; q < kPred; q++) {
                            if (q >= np) break;
                            const int32_t nj = read_lane(pn[q], j), cj = read_lane(px[q], j);
#pragma unroll
                            for (int k = 0; k < WPL; k++)
                                if ((wcpu[k] ? 0 : 1 + lane + k * kWave - ncpu) != nj) xk[k] += cj;
                        }
                        for (int32_t c0 = kPred; c0 < np; c0 += kWave) {
                            int32_t nu = 0, cx = 0;
                            if (c0 + lane < np) {
                                const int32_t u = pred[pa + c0 + lane];
                                const int32_t wu = -2 - tr[u].qpos;
                                nu = wu < ncpu ? 0 : 1 + wu - ncpu;
                                cx = dxc[u];
                            }
                            const int32_t cn = min(kWave, np - c0);
                            for (int32_t jj = 0; jj < cn; jj++) {
                                const int32_t nj = read_lane(nu, jj), cj = read_lane(cx, jj);
#pragma unroll
                                for (int k = 0; k < WPL; k++)
                                    if ((wcpu[k] ? 0 : 1 + lane + k * kWave - ncpu) != nj) xk[k] += cj;
                            }
                        }
                    }
                    // least expected termination, ties to the lower worker: a
                    // 32-bit key (cost - t) << WB | worker while the cost is below kLim
                    uint32_t k32 = ~0u;
#pragma unroll
                    for (int k = 0; k < WPL; k++) {
                        uint32_t rc = ld[k] + (uint32_t)(wcpu[k] ? e0 : e1);
                        if constexpr (DATA) rc = (uint32_t)min((uint64_t)rc + (uint64_t)xk[k], (uint64_t)kLim);
                        else rc = min(rc, kLim);
                        k32 = min(k32, rc << WB | (uint32_t)(lane + k * kWave));
                    }
                    const uint32_t m32 = wave_min_u32f(k32);
                    int32_t ws = (int32_t)(m32 & ((1u << WB) - 1));
                    if (RARELY(m32 >> WB == kLim)) {
                        uint64_t k64 = ~0ull;
#pragma unroll
                        for (int k = 0; k < WPL; k++) {
                            const int64_t rc = max(expend[k], t) - t + qest[k] + (wcpu[k] ? e0 : e1) + xk[k];
                            if (wok[k]) k64 = min(k64, (uint64_t)rc << WB | (uint64_t)(lane + k * kWave));
                        }
                        ws = (int32_t)(wave_min_u64f(k64) & ((1u << WB) - 1));
                    }
                    const int32_t ek = ws >= ncpu ? e1 : e0;
                    int64_t xs = 0;
                    if constexpr (DATA) {
                        xs = (int64_t)read_lane64((uint64_t)xk[0], ws & 63);
                        if constexpr (WPL == 2)
                            if (ws >= kWave) xs = (int64_t)read_lane64((uint64_t)xk[WPL - 1], ws & 63);
                        if (xs > INSP_MAX_TICK) status |= ST_XFER;
                    }
                    int32_t slot = of_worker<WPL>(nslot, ws);
                    if (RARELY(slot < 0)) {  // a new block
                        const int32_t blk = nused++;
                        const int32_t nbw = of_worker<WPL>(nb, ws);
                        if (nbw < kLB) {
                            if (lane == 0) L.blist[ws * kLB + nbw] = blk;
                        } else {
                            int32_t *wblk = cold<WPL, int32_t>(kColdWblk);
                            if (lane == 0) wblk[(int64_t)ws * maxb + nbw] = blk;
                        }
                        slot = blk * 64;
#pragma unroll
                        for (int k = 0; k < WPL; k++)
                            if (lane + k * kWave == ws) {
                                nb[k] = nbw + 1;
                                tail[k] = slot;
                                // (the second wave reads the count first, then that many ids)
                                keep_order();
                                lds_store(&rnb[lane + k * kWave], nbw + 1);
                            }
                    }
                    // the slot was the worker's empty one or its tail
                    const int32_t next = (slot + 1) & 63 ? slot + 1 : -1;
#pragma unroll
                    for (int k = 0; k < WPL; k++) {
                        const bool is = lane + k * kWave == ws, h = is && slot == hole[k], tl = is && slot != hole[k];
                        len[k] += is ? 1 : 0;
                        qest[k] += is ? ek : 0;
                        ld[k] = min(ld[k] + (is ? (uint32_t)ek : 0u), kLim);
                        used[k] = h ? slot : used[k];
                        hole[k] = h ? -1 : hole[k];
                        tail[k] = tl ? next : tail[k];
                        nslot[k] = is ? tail[k] : nslot[k];
                    }
                    pq = lane == j ? slot : pq;
                    wsj = lane == j ? ws : wsj;
                    xsj = lane == j ? xs : xsj;
                    if constexpr (kBig) {
                        // the best entry pushed since the worker's last pop
                        const uint64_t hi = (uint32_t)read_lane(f_ie, j), lo = (uint32_t)read_lane(f_ia, j);
                        const uint64_t raw = K.big(heft ? hi << 32 | lo : lo << 21 | hi, seq + __popcll(fm & ((1ull << j) - 1)));
                        const unsigned long long a0 = K.rule(raw, 0), a1 = K.rule(raw, 1);
#pragma unroll
                        for (int k = 0; k < WPL; k++)
                            if (lane + k * kWave == ws) {
                                if (a0 > pk0[k]) {
                                    pk0[k] = a0;
                                    pp0[k] = slot;
                                }
                                if (a1 > pk1[k]) {
                                    pk1[k] = a1;
                                    pp1[k] = slot;
                                }
                            }
                    }
                }
                PCLK(17);
                const int32_t np = __popcll(fm);
                seq += np;
                nready += np;
                // the chunk's queue entries and task records, a lane each, then the
                // maxima of their blocks and workers
                const int32_t bq = pq >> 6;
                const bool g = wsj >= ncpu;
                const int32_t ekl = g ? f_e.y : f_e.x, dkl = g ? f_d.y : f_d.x;
                uint64_t word;
                unsigned long long m0, m1;
                if constexpr (kBig) {
                    // the general loop's key: rank << 21 or IA << 42 | IE << 21, then the push order
                    word = K.big(heft ? (uint64_t)(uint32_t)f_ie << 32 | (uint32_t)f_ia : (uint64_t)f_ia << 21 | (uint64_t)f_ie, sqj);
                    m0 = K.rule(word, 0);
                    m1 = K.rule(word, 1);
                } else {
                    const uint32_t a0 = kf.ka((uint32_t)f_ia, (uint32_t)f_ie, (uint32_t)sqj);
                    const uint32_t a1 = kf.ke((uint32_t)f_ia, (uint32_t)f_ie, (uint32_t)sqj);
                    word = (uint64_t)a1 << 32 | a0;
                    m0 = (unsigned long long)a0 << 32 | (uint32_t)pq;
                    m1 = (unsigned long long)a1 << 32 | (uint32_t)pq;
                }
                const uint64_t xw = (uint64_t)f_v << 42 | (uint64_t)(dkl & M21) << 21 | (uint64_t)(ekl & M21);
                // the next empty slot of each worker whose first one was taken
                // (read before the entries overwrite the chain)
#pragma unroll
                for (int k = 0; k < WPL; k++) {
                    int32_t nh;
                    if (USUALLY(nused <= SLC) || ballot(used[k] >= SLC * 64) == 0) {
                        nh = L.srs[max(used[k], 0)];
                    } else {
                        const int32_t *grs = pool().rs;
                        nh = -1;
                        if (used[k] >= 0) {
                            if ((used[k] >> 6) < SLC) nh = L.srs[used[k]];
                            else nh = wg_load(&grs[used[k]]);
                        }
                        settle(nh);
                    }
                    hole[k] = used[k] >= 0 ? nh : hole[k];
                    used[k] = -1;
                }
                keep_order();
                if (USUALLY(nused <= NB) || (fm & ballot(bq >= NB)) == 0) {
                    if (ok) {
                        K.put(pq, word);
                        L.sx[pq] = xw;
                        L.srs[pq] = f_rs;
                        keep_order();
                        atomicMax(&mx[2 * bq], m0);
                        atomicMax(&mx[2 * bq + 1], m1);
                    }
                } else {
                    const SlotPool slots = pool();
                    unsigned long long *sums = gsums();
                    if (ok) {
                        if (bq < SLK) K.put(pq, word);
                        else slots.k[pq] = word;
                        if (bq < SLC) {
                            L.sx[pq] = xw;
                            L.srs[pq] = f_rs;
                        } else {
                            slots.x[pq] = xw;
                            slots.rs[pq] = f_rs;
                        }
                        keep_order();
                        if (bq < SC) {
                            atomicMax(&mx[2 * bq], m0);
                            atomicMax(&mx[2 * bq + 1], m1);
                        } else {
                            wg_fetch_max(&sums[2 * bq], m0);
                            wg_fetch_max(&sums[2 * bq + 1], m1);
                        }
                    }
                }
                if (ok) {
                    // queue slot, then push order and worker
                    *reinterpret_cast<int2 *>(&at(tr, f_v)->qpos) = make_int2(pq, sqj | wsj << 21);
                    if constexpr (!kBig) {
                        atomicMax(&best[2 * wsj], m0);
                        atomicMax(&best[2 * wsj + 1], m1);
                    }
                    // data model: the record's first word holds the time the
                    // task's inputs arrive (transfers start now) until its pop
                    if constexpr (DATA) at(tr, f_v)->word = (unsigned long long)(t + xsj);
                }
                // never lowered by pops: an upper bound for the block
                if constexpr (DATA)
                    if (lrule && ok)
                        wg_fetch_max(reinterpret_cast<unsigned long long *>(&barr[bq]), (unsigned long long)(t + xsj));
                if (inlane || i0 + kWave >= r) break;
            }
        }
        PCLK(0);
        // -------------------------------------------------------- regulate
        const int32_t observed = nready;
        if (policy == INSP_POLICY_INSPIRIT) {
            peak = max(peak, nready);
            const int32_t dn = nready - prev_n;
            if ((dn < 0 ? -dn : dn) >= s_inc) {
                const int64_t dt = t - prev_t;
                prev_n = nready;
                prev_t = t;
                if (nready >= peak - dec_step) {
                    cnt = 0;
                    if (dn >= s_inc) {
                        const int64_t lhs = (int64_t)dn * k_den, rhs = (int64_t)k_num * dt;
                        if (dt == 0 || lhs > rhs) mode = INSP_MODE_ABILITY;
                        else if (lhs < rhs) mode = INSP_MODE_EFI;
                    }
                } else if ((int64_t)nready > (int64_t)peak - (int64_t)s_dec * cnt) {
                    mode = INSP_MODE_ABILITY;
                } else if ((int64_t)nready <= (int64_t)peak - (int64_t)s_dec * (cnt + 1) + cc) {
                    mode = INSP_MODE_EFI_LOC;
                    if ((int64_t)nready <= (int64_t)peak - (int64_t)s_dec * (cnt + 1)) cnt++;
                }
            }
        }
        const int pmode = policy == INSP_POLICY_INSPIRIT ? mode
                        : policy == INSP_POLICY_FIFO ? INSP_MODE_FIFO
                        : policy == INSP_POLICY_ABILITY_ONLY ? INSP_MODE_ABILITY
                        : policy == INSP_POLICY_EFI_ONLY ? INSP_MODE_EFI
                        : policy == INSP_POLICY_LOCALITY ? INSP_MODE_EFI_LOC : INSP_MODE_RANK;
        const int slot = pmode == INSP_MODE_EFI || pmode == INSP_MODE_EFI_LOC ? 1 : 0;
        // efficiency with locality under the data model: tasks whose inputs
        // have arrived first
        const bool loc = DATA && pmode == INSP_MODE_EFI_LOC;
        // ------------------------------------------------------------- pop
        int32_t popped = 0;
#pragma unroll
        for (int k = 0; k < WPL; k++) {
            // (only workers have queues)
            const uint64_t wm = ballot(run[k] < 0) & ballot(len[k] > 0);
            if (wm == 0) continue;
            const bool want = __builtin_amdgcn_inverse_ballot_w64(wm);
            const int32_t w = lane + k * kWave;
            const int32_t np = __popcll(wm);
            popped += np;
            nready -= np;
            // the best entry of each queue, once its rescan is done (the
            // second wave answers every request)
            unsigned long long bk;
            int32_t bp = 0;
            for (int32_t spin = 0;; spin++) {
                const int32_t rq = lds_load(&req[w]);
                keep_order();
                bk = lds_load(&best[2 * w + slot]);
                if constexpr (kBig) bp = lds_load(&bpos[2 * w + slot]);
                if (USUALLY((wm & ballot(rq != 0)) == 0)) break;
                if (RARELY(spin > kReqSpin)) {
                    // never: a wait that ends all the same.  What is popped then is
                    // some task whose slot the queue has used; the DAG fails
                    status |= ST_HANG;
                    done = n;
                    break;
                }
            }
            keep_order();
            int32_t p;
            if constexpr (kBig) p = (slot ? pk1[k] : pk0[k]) > bk ? (slot ? pp1[k] : pp0[k]) : bp;
            else p = (int32_t)(uint32_t)bk;
            p = want ? p : 0;
            uint32_t key = (uint32_t)(bk >> 32);  // 32-bit keys: the entry's key under the rule
            PCLK(11);
            if constexpr (DATA) {
                if (loc) {
                    // the arrival times are not in the keys: a queue whose best
                    // entry's inputs are still moving is searched, a block whose
                    // latest input arrival has passed by its maximum (all its tasks
                    // have their inputs), other blocks entry by entry
                    bool late = false;
                    const SlotPool slots = pool();
                    const int32_t *wblk = cold<WPL, int32_t>(kColdWblk);
                    unsigned long long *sums = gsums();
                    if (want) {
                        const uint64_t xv = (p >> 6) < SLC ? L.sx[p] : wg_load(&slots.x[p]);
                        late = (int64_t)wg_load(&tr[(int32_t)(xv >> 42)].word) > t;
                    }
                    uint64_t lm = ballot(late);
                    while (lm) {
                        const int l = (int)__builtin_ctzll(lm);
                        lm &= lm - 1;
                        const int32_t wl = l + k * kWave;
                        const int32_t nbw = read_lane(nb[k], l);
                        KT bestk = 0;
                        int32_t bestb = -1;
                        for (int32_t i0 = 0; i0 < nbw; i0 += kWave) {
                            const int32_t i = i0 + lane;
                            int32_t b = -1;
                            if (i < nbw) {
                                if (i < kLB) {
                                    b = L.blist[wl * kLB + i];
                                } else {
                                    b = wg_load(&wblk[(int64_t)wl * maxb + i]);
                                    settle(b);
                                }
                            }
                            KT kk = 0;
                            bool mix = false;
                            if (b >= 0) {
                                if ((int64_t)wg_load(&barr[b]) <= t)
                                    kk = K.of_max(b < SC ? lds_load(&mx[2 * b + 1])
                                                         : __hip_atomic_load(&sums[2 * b + 1], __ATOMIC_RELAXED,
                                                                             __HIP_MEMORY_SCOPE_AGENT));
                                else mix = true;
                            }
                            const KT km = wave_max_k(kk);
                            if (km > bestk) {
                                bestk = km;
                                bestb = read_lane(b, (int)__builtin_ctzll(ballot(kk == km && b >= 0)));
                            }
                            uint64_t mm = ballot(mix);
                            while (mm) {
                                const int32_t bm = read_lane(b, (int)__builtin_ctzll(mm));
                                mm &= mm - 1;
                                const int32_t pe = bm * 64 + lane;
                                const KT kr = bm < SLK ? K.lds(pe, 1) : K.rule(wg_load(&slots.k[pe]), 1);
                                KT ke = 0;
                                if (kr != 0) {
                                    const uint64_t xv = bm < SLC ? L.sx[pe] : wg_load(&slots.x[pe]);
                                    if ((int64_t)wg_load(&tr[(int32_t)(xv >> 42)].word) <= t) ke = kr;
                                }
                                const KT kme = wave_max_k(ke);
                                if (kme > bestk) {
                                    bestk = kme;
                                    bestb = bm;
                                }
                            }
                        }
                        if (bestb >= 0) {  // the entry of that block with this key
                            const int32_t pe = bestb * 64 + lane;
                            const KT kr = bestb < SLK ? K.lds(pe, 1) : K.rule(wg_load(&slots.k[pe]), 1);
                            const int32_t pn2 = bestb * 64 + (int32_t)__builtin_ctzll(ballot(kr == bestk));
                            if (lane == l) {
                                p = pn2;
                                if constexpr (!kBig) key = (uint32_t)bestk;
                            }
                        }
                    }
                }
            }
            // take the entry at p: its slot joins the worker's empty ones, and its
            // block's maxima and the worker's best wait for the rescan
            const int32_t bb = p >> 6;
            uint64_t vx = 0;
            int32_t vr = 0;
            if (USUALLY(nused <= NB) || (wm & ballot(bb >= NB)) == 0) {
                if (want) {
                    vx = L.sx[p];
                    vr = L.srs[p];
                    if constexpr (!kBig)
                        if (kf.fifo) key = K.ke[p];  // the FIFO key holds no attributes
                    K.put(p, 0);
                    L.srs[p] = hole[k];
                    mx[2 * bb] = 0;
                    mx[2 * bb + 1] = 0;
                }
            } else {
                const SlotPool slots = pool();
                unsigned long long *sums = gsums();
                if (want) {
                    if constexpr (!kBig)
                        if (kf.fifo) key = bb < SLK ? K.ke[p] : (uint32_t)(wg_load(&slots.k[p]) >> 32);
                    if (bb < SLC) {
                        vx = L.sx[p];
                        vr = L.srs[p];
                        L.srs[p] = hole[k];
                    } else {
                        vx = wg_load(&slots.x[p]);
                        vr = wg_load(&slots.rs[p]);
                        slots.rs[p] = hole[k];
                    }
                    if (bb < SLK) K.put(p, 0);
                    else slots.k[p] = 0;
                    if (bb < SC) {
                        mx[2 * bb] = 0;
                        mx[2 * bb + 1] = 0;
                    } else {
                        sums[2 * bb] = 0;
                        sums[2 * bb + 1] = 0;
                    }
                }
                settle(vx);
                settle(vr);
            }
            PCLK(12);
            if (want) {
                best[2 * w] = 0;
                best[2 * w + 1] = 0;
                keep_order();
                lds_store(&req[w], bb + 1);
            }
            const int32_t v = (int32_t)(vx >> 42);
            const int32_t dk = (int32_t)((vx >> 21) & M21), ek = (int32_t)(vx & M21);
            // a task whose inputs are still moving holds the worker until they arrive
            int64_t s0 = t;
            if constexpr (DATA)
                if (want) s0 = max(t, (int64_t)wg_load(&at(tr, v)->word));
            int32_t deg = 0, iev = 0;
            if constexpr (kBig) {
                if (want) {
                    const int4 fx = *reinterpret_cast<const int4 *>(&at(tr, v)->iev);  // IE, IA, tau, first edge
                    deg = fx.y;
                    iev = tattr ? tie[v] : fx.x;
                    pk0[k] = pk1[k] = 0;
                }
            } else {
                const int32_t f1 = (int32_t)((key >> kf.sb) & kf.amask), f0 = (int32_t)((key >> kf.sa) & kf.amask);
                const bool efi = slot || kf.fifo;
                deg = efi ? f0 : f1;
                iev = efi ? f1 : f0;
            }
            if (want) {
                // the first successors, for the release (past the row's end
                // they are never used; the successor array is padded)
                pfa[k] = *reinterpret_cast<const row4 *>(col + vr);
                pfb[k] = *reinterpret_cast<const row4 *>(col + vr + 4);
                put_record(at(tr, v), s0, dk, w, iev, pmode);
                len[k]--;
                hole[k] = p;
                run[k] = v;
                fin[k] = s0 + dk;
                expend[k] = s0 + ek;
                qest[k] -= ek;
                rsr[k] = vr;
                dgr[k] = deg;
                // for the wave that reads ahead
                lrun[w] = make_int2(v, (int32_t)fin[k]);
            }
            PCLK(13);
        }
        PCLK(2);
        if (RARELY(A.trace != nullptr) && lane == 0 && events <= max_events) {
            insp_trace_rec rec;
            rec.t = t;
            rec.nready = observed;
            rec.mode = pmode;
            rec.cnt = cnt;
            rec.peak = peak;
            rec.pushed = r;
            rec.popped = popped;
            A.trace[(d.toff - A.base) + di + events - 1] = rec;
        }
        if (RARELY(done == n)) break;
        // --------------------------------------------------------- advance
        // every running task ends within 2^21 ticks of t
        uint32_t dl = ~0u;
#pragma unroll
        for (int k = 0; k < WPL; k++)
            if (run[k] >= 0) dl = min(dl, (uint32_t)(fin[k] - t));
        const uint32_t dtm = wave_min_u32f(dl);
        if (RARELY(dtm == ~0u)) {
            status |= ST_HANG;
            break;
        }
        t += dtm;
        PCLK(3);
        // --------------------------------------------------------- release
        r = 0;
        uint64_t cm[WPL];
        int32_t c_l[WPL];
        int32_t ndone = 0;
#pragma unroll
        for (int k = 0; k < WPL; k++) {
            cm[k] = ballot(run[k] >= 0) & ballot(fin[k] == t);
            const bool fin_now = __builtin_amdgcn_inverse_ballot_w64(cm[k]);
            ndone += __popcll(cm[k]);
            c_l[k] = run[k];
            if (fin_now) {
                run[k] = -1;
                expend[k] = 0;
                lrun[lane + k * kWave].x = -1;
            }
        }
        done += ndone;
        merged = staged = inlane = false;
        // the only completing worker, or the first
        const int32_t w1 = WPL == 2 && cm[0] == 0 ? kWave + (int32_t)__builtin_ctzll(cm[WPL - 1])
                                                  : (int32_t)__builtin_ctzll(cm[0]);
        const int32_t deg1 = of_worker<WPL>(dgr, w1);
        if (USUALLY(ndone == 1) && USUALLY(deg1 <= kWave)) {
            const int32_t c = of_worker<WPL>(c_l, w1);
            // the first successors go from the worker's lane to a lane each
#pragma unroll
            for (int k = 0; k < WPL; k++)
                if (lane + k * kWave == w1) {
                    *reinterpret_cast<int4 *>(succ) = make_int4(pfa[k].x, pfa[k].y, pfa[k].z, pfa[k].w);
                    *reinterpret_cast<int4 *>(succ + 4) = make_int4(pfb[k].x, pfb[k].y, pfb[k].z, pfb[k].w);
                }
            keep_order();
            const bool in = lane < deg1;
            int32_t s = lds_load(&succ[lane & (kPF - 1)]);
            if (RARELY(deg1 > kPF)) {
                const int32_t rs = of_worker<WPL>(rsr, w1);
                if (in && lane >= kPF) s = col[rs + lane];
            }
            s = in ? s : 0;
            PCLK(19);
            // one wave owns the DAG's words and a row's successors are
            // distinct (rows are deduplicated), so a plain read-modify-write
            // replaces the atomic (a wave's accesses to one address complete in
            // program order)
            unsigned long long *dp = at(dep, s);
            const uint64_t now = *dp - ((1ull << 43) + (unsigned long long)c);
            if (in) *dp = now;
            const uint32_t nr = (uint32_t)(now >> 43);
            const uint64_t inm = deg1 < 64 ? (1ull << deg1) - 1 : ~0ull;
            const uint64_t cdm = inm & ballot(nr == 1);
            fm = inm & ballot(nr == 0);
            r = __popcll(fm);
            inlane = r > 0;
            const bool rdy = __builtin_amdgcn_inverse_ballot_w64(fm), cd = __builtin_amdgcn_inverse_ballot_w64(cdm);
            PCLK(20);
            if (USUALLY(fm | cdm)) {
                // rows of the newly ready tasks; records of the others' remaining
                // predecessors u, whose IE may grow
                const int32_t u = cd ? (int32_t)(now & M43) : 0;
                TaskRec *ru = at(tr, u);
                const int4 fx = *reinterpret_cast<const int4 *>(&at(tr, s)->iev);  // IE, IA, tau, first edge
                const int2 uq = *reinterpret_cast<const int2 *>(&ru->qpos);        // queue slot; push order and worker
                const int4 ux = *reinterpret_cast<const int4 *>(&ru->iev);
                f_e = *at(est2, s);
                f_d = *at(dur2, s);
                if constexpr (DATA) {
                    f_pa = *at(prp, s);
                    f_pz = at(prp, s)[1];
                }
                f_v = s;
                f_ie = fx.x;
                f_ia = fx.y;
                f_rs = fx.w;
                if constexpr (KK == kFixed) {
                    if (heft) {
                        const int64_t rv = rk[s];
                        f_ia = (int32_t)(uint32_t)rv;
                        f_ie = (int32_t)(uint32_t)((uint64_t)rv >> 32);
                    } else if (tattr) {
                        f_ia = tia[s];
                        f_ie = tie[s];
                    }
                }
                PCLK(23);
                // (taus are at most 2^20, U at most 2^31 - 1)
                uint64_t left = cdm & ballot(ux.z + fx.z <= U);
                const bool cond = __builtin_amdgcn_inverse_ballot_w64(left);
                if (left) {
                    // several successors may name the same predecessor: the
                    // first lane applies all of its increments
                    int32_t mult = 1;
                    bool lead = cond;
                    if (RARELY(left & (left - 1))) {
                        lead = false;
                        while (left) {
                            const int l = (int)__builtin_ctzll(left);
                            const uint64_t same = left & ballot(u == read_lane(u, l));
                            left &= ~same;
                            if (lane == l) {
                                lead = true;
                                mult = __popcll(same);
                            }
                        }
                    }
                    const int32_t nie = ux.x + mult;
                    if (lead) ru->iev = nie;
                    if constexpr (KK != kFixed) {
                        raise(lead && uq.x >= 0, uq.x, uq.y, ux.y, nie);
                        // a raised IE of a task about to be pushed goes into its key
                        uint64_t lm = ballot(lead && uq.x == -1);
                        if (fm)
                            while (lm) {
                                const int l = (int)__builtin_ctzll(lm);
                                lm &= lm - 1;
                                const int32_t uu = read_lane(u, l), kk = read_lane(mult, l);
                                if (rdy && s == uu) f_ie += kk;
                            }
                    }
                }
            }
            PCLK(24);
            continue;
        }
        // several completions, or a long row: successors through lists
        int32_t *fbuf = cold<WPL, int32_t>(kColdFbuf);
        int32_t nc = 0, nseg = 0;
#pragma unroll
        for (int k = 0; k < WPL; k++) {
            uint64_t mask = cm[k];
            while (mask) {
                const int l = (int)__builtin_ctzll(mask);
                mask &= mask - 1;
                const int32_t c = read_lane(c_l[k], l);
                const int32_t deg = read_lane(dgr[k], l), rs = read_lane(rsr[k], l);
                const int32_t r0 = r;
                const unsigned long long dec = 0ull - ((1ull << 43) + (unsigned long long)c);
                for (int32_t e0 = 0; e0 < deg; e0 += kWave) {
                    const int32_t e = e0 + lane;
                    const bool ok = e < deg;
                    int32_t s = 0;
                    if (ok) s = col[rs + e];
                    uint64_t old = 0;
                    if (ok) {
                        old = dep[s];
                        dep[s] = old + dec;
                    }
                    const int32_t nr = (int32_t)(old >> 43) - 1;
                    const bool rdy = ok && nr == 0, cd = ok && nr == 1;
                    const uint64_t m1 = ballot(rdy), m2 = ballot(cd);
                    if (rdy) {
                        const int32_t pos = r + lanes_below(m1);
                        fbuf[pos] = s;
                        if (pos < kFC) fr0[pos] = s;
                    }
                    if (cd) {
                        const int32_t pos = nc + lanes_below(m2);
                        if (pos < kCC) {
                            cs[pos] = s;
                            cu[pos] = (int32_t)((old + dec) & M43);
                        } else {
                            fbuf[2 * n + pos] = s;
                        }
                    }
                    r += __popcll(m1);
                    nc += __popcll(m2);
                }
                if (r > r0) {
                    if (lane == 0) seg[nseg] = r;
                    nseg++;
                }
            }
        }
        PCLK(4);
        wg_fence();
        // successors left with one unfinished predecessor raise its IE (as in
        // the general loop)
        const bool single = ndone == 1;
        if (nc <= kWave && r <= kFC) {
            const bool hc = lane < nc;
            const int32_t s = hc ? cs[lane] : 0;
            int32_t u = hc ? cu[lane] : -1;
            staged = r <= kWave;
            const bool hf = staged && lane < r;
            const int32_t fv = hf ? fr0[lane] : 0;
            // a candidate made ready by a later completion of this event is none
            if (!single) {
                if (staged) {
                    for (int32_t k = 0; k < r; k++)
                        if (read_lane(fv, k) == s) u = -1;
                } else if (hc) {
                    for (int32_t k = 0; k < r; k++)
                        if (fr0[k] == s) {
                            u = -1;
                            break;
                        }
                }
            }
            // one wave owns the records, so plain vector loads see its stores
            TaskRec *ru = at(tr, max(u, 0));
            const int2 qs = *reinterpret_cast<const int2 *>(&ru->qpos);  // queue slot; push order and worker
            const int4 ux = *reinterpret_cast<const int4 *>(&ru->iev);   // IE, IA, tau, first edge
            const int32_t ts = at(tr, s)->tau;
            int2 fe = *at(est2, fv), fd = *at(dur2, fv);
            const int4 fx = *reinterpret_cast<const int4 *>(&at(tr, fv)->iev);
            int32_t fie = fx.x, fa = fx.y;
            const int32_t frs = fx.w;
            // fixed keys: the rank (low and high words), or the transitive attributes
            if (heft) {
                const int64_t rv = rk[fv];
                fa = (int32_t)(uint32_t)rv;
                fie = (int32_t)(uint32_t)((uint64_t)rv >> 32);
            } else if (tattr) {
                fa = tia[fv];
                fie = tie[fv];
            }
            const bool cond = u >= 0 && ux.z + ts <= U;
            int32_t mult = cond ? 1 : 0;
            bool lead = cond;
            if (nc > 1) {
                // several successors may name the same predecessor: the
                // first lane applies all of its increments
                lead = false;
                uint64_t left = ballot(cond);
                while (left) {
                    const int l = (int)__builtin_ctzll(left);
                    const uint64_t same = ballot(cond && u == read_lane(u, l));
                    left &= ~same;
                    if (lane == l) {
                        lead = true;
                        mult = __popcll(same);
                    }
                }
            }
            const int32_t nie = ux.x + mult;
            if (lead) ru->iev = nie;
            if constexpr (KK != kFixed) {
                const bool qd = lead && qs.x >= 0;
                if (ballot(qd)) raise(qd, qs.x, qs.y, ux.y, nie);
                // a raised IE of a task staged for this event's pushes goes into its key
                uint64_t lm = ballot(lead && qs.x == -1);
                while (lm) {
                    const int l = (int)__builtin_ctzll(lm);
                    lm &= lm - 1;
                    const int32_t uu = read_lane(u, l), kk = read_lane(mult, l);
                    if (hf && fv == uu) fie += kk;
                }
            }
            int32_t pos = lane;
            if (nseg > 1 && staged) {
                // rank in the merged ascending order (the event's ready ids are
                // distinct): how many of them are smaller
                int32_t rank = 0;
                for (int32_t k = 0; k < r; k++) rank += read_lane(fv, k) < fv ? 1 : 0;
                pos = rank;
            }
            if (!staged && nseg > 1) {
                for (int32_t i = lane; i < r; i += kWave) {
                    const int32_t x = fr0[i];
                    int32_t rank = 0, lo = 0;
                    for (int32_t g = 0; g < nseg; g++) {
                        const int32_t hi = seg[g];
                        if (i >= lo && i < hi) {
                            rank += i - lo;
                        } else {
                            int32_t a = lo, b = hi;
                            while (a < b) {
                                const int32_t mid = (a + b) >> 1;
                                if (fr0[mid] < x) a = mid + 1;
                                else b = mid;
                            }
                            rank += a - lo;
                        }
                        lo = hi;
                    }
                    fr1[rank] = x;
                }
                merged = true;
            }
            if (hf) {
                pre[pos] = fv;
                pre[64 + pos] = fe.x;
                pre[128 + pos] = fe.y;
                pre[192 + pos] = fd.x;
                pre[256 + pos] = fd.y;
                pre[320 + pos] = fa;
                pre[384 + pos] = frs;
                pre[448 + pos] = fie;
            }
        } else {
            for (int32_t i0 = 0; i0 < nc; i0 += kWave) {
                const int32_t i = i0 + lane;
                const int32_t s = i < nc ? (i < kCC ? cs[i] : wg_load(&fbuf[2 * n + i])) : 0;
                int32_t u = -1;
                if (i < nc) {
                    if (single && i < kCC) {
                        u = cu[i];
                    } else {
                        const uint64_t wd = wg_load(&dep[s]);
                        if ((wd >> 43) == 1) u = (int32_t)(wd & M43);
                    }
                }
                TaskRec *ru = at(tr, max(u, 0));
                const int2 qs = *reinterpret_cast<const int2 *>(&ru->qpos);
                const int4 ux = *reinterpret_cast<const int4 *>(&ru->iev);
                const bool cond = u >= 0 && ux.z + at(tr, s)->tau <= U;
                // the first lane that names a predecessor applies all of the chunk's increments
                uint64_t left = ballot(cond);
                bool lead = false;
                int32_t mult = 0;
                while (left) {
                    const int l = (int)__builtin_ctzll(left);
                    const uint64_t same = ballot(cond && u == read_lane(u, l));
                    left &= ~same;
                    if (lane == l) {
                        lead = true;
                        mult = __popcll(same);
                    }
                }
                const int32_t nie = ux.x + mult;
                if (lead) ru->iev = nie;
                if constexpr (KK != kFixed) {
                    const bool qd = lead && qs.x >= 0;
                    if (ballot(qd)) raise(qd, qs.x, qs.y, ux.y, nie);
                }
            }
            wg_fence();
            if (nseg > 1) {
                const bool in_lds = r <= kFC;
                for (int32_t i0 = 0; i0 < r; i0 += kWave) {
                    const int32_t i = i0 + lane;
                    if (i < r) {
                        const int32_t x = in_lds ? fr0[i] : fbuf[i];
                        int32_t rank = 0, lo = 0;
                        for (int32_t g = 0; g < nseg; g++) {
                            const int32_t hi = seg[g];
                            if (i >= lo && i < hi) {
                                rank += i - lo;
                            } else {
                                int32_t a = lo, b = hi;
                                while (a < b) {
                                    const int32_t mid = (a + b) >> 1;
                                    const int32_t y = in_lds ? fr0[mid] : fbuf[mid];
                                    if (y < x) a = mid + 1;
                                    else b = mid;
                                }
                                rank += a - lo;
                            }
                            lo = hi;
                        }
                        if (in_lds) fr1[rank] = x;
                        else fbuf[n + rank] = x;
                    }
                }
                merged = true;
            }
        }
        PCLK(7);
        wg_fence();
        PCLK(8);
    }
#ifdef INSP_PHASE_CLOCKS
    if (lane == 0 && d.id < 8192)
        for (int i = 0; i < 32; i++) g_phase_clk[d.id * 32 + i] = pc[i];
#endif
    if (lane == 0) {
        A.makespan[di] = (status & ST_HANG) ? -1 : t;
        if (A.n_events) A.n_events[di] = events;
        if (status) atomicOr(&A.stat[2 * d.id], status);
        A.stat[2 * d.id + 1] = events;
    }
}

// The work-group's LDS, carved in the order lds_bytes() counts it.
__device__ __forceinline__ Lds carve_lds(const SimArgs &A) {
    extern __shared__ int64_t lds64[];
    const int32_t MW = A.max_w;
    Lds L;
    L.fin = lds64;
    L.expend = lds64 + MW;
    L.qest = lds64 + 2 * MW;
    L.sum = reinterpret_cast<unsigned long long *>(lds64 + 3 * MW);
    L.sk = L.sum + 2 * A.sum_cap;
    L.sx = L.sk + 64 * A.key_cap;
    int32_t *l32 = reinterpret_cast<int32_t *>(L.sx + 64 * A.slot_cap);
    L.run = l32;
    L.len = l32 + MW;
    L.nb = l32 + 2 * MW;
    L.last = l32 + 3 * MW;
    L.seg = l32 + 4 * MW;
    L.rsr = l32 + 5 * MW;
    L.dgr = l32 + 6 * MW;
    L.blist = l32 + 7 * MW;
    L.fr0 = L.blist + MW * A.lb;
    L.fr1 = L.fr0 + kFC;
    L.cs = L.fr1 + kFC;
    L.cu = L.cs + kCC;
    L.pre = L.cu + kCC;
    L.srs = L.pre + 8 * kWave;
    L.hs = L.srs + 64 * A.slot_cap;
    return L;
}

// The work-group's third wave, while the first simulates DAG di: it reads
// ahead for the running tasks that finish first -- their successor lists,
// the successors' dependency words, and the records and estimate rows the
// release of those tasks will read (of successors about to become ready,
// and of the remaining predecessor of those about to have one left) -- so
// that the simulating wave finds them in the caches.  It only reads, and it
// stops when the simulating wave marks the DAG finished.
constexpr int kAhead = 4;          // running tasks read ahead for, earliest finish first
constexpr int kAheadEdges = 16;    // successors read per task

template <int WPL>
__device__ void read_ahead(const SimArgs &A, int32_t di) {
    using LL = LaneLds<WPL>;
    const uint64_t *lrun = LL::template arr<uint64_t>(LL::kRun);
    int32_t *hs = LL::template arr<int32_t>(LL::kHs);
    const DagDesc d = A.desc[di];
    const int lane = lane_id();
    const int64_t ub = d.toff - A.base;
    const int32_t *col = A.col + d.eoff;
    const TaskRec *tr = A.tr + d.toff;
    const unsigned long long *dep = A.dep + d.toff;
    const int2 *est2 = reinterpret_cast<const int2 *>(A.est) + ub;
    const int2 *dur2 = reinterpret_cast<const int2 *>(A.dur) + ub;
    int32_t pref[WPL];  // the last task read ahead for each of this lane's workers
#pragma unroll
    for (int k = 0; k < WPL; k++) pref[k] = -1;
    uint32_t sink = 0;
    for (int64_t it = 0; it < kHelperSpin; it++) {
        if (lds_load(&hs[1])) break;
        // the lane's next task to read ahead for: of two workers' the one that ends first
        int32_t c = -1, kc = 0;
        int64_t f = INT64_MAX;
#pragma unroll
        for (int k = 0; k < WPL; k++) {
            const uint64_t rf = lds_load(&lrun[lane + k * kWave]);
            const int32_t ck = (int32_t)(uint32_t)rf;
            const int64_t fk = (int64_t)(rf >> 32);  // low 32 bits: good for an order of finishes, which is all it is for
            if (ck >= 0 && (WPL == 1 || ck != pref[k]) && fk < f) {
                f = fk;
                c = ck;
                kc = k;
            }
        }
        // the kAhead-th earliest finish among the running tasks
        uint64_t thr = 0;
        {
            uint64_t prev = 0;
            bool first = true;
            for (int k = 0; k < kAhead; k++) {
                const uint64_t m = wave_min_u64f(first || (uint64_t)f > prev ? (uint64_t)f : ~0ull);
                if (m == ~0ull) break;
                thr = m;
                prev = m;
                first = false;
            }
        }
        const bool go = c >= 0 && c != (kc == 0 ? pref[0] : pref[WPL - 1]) && c < d.n && (uint64_t)f <= thr;
        if (!ballot(go)) {
            __builtin_amdgcn_s_sleep(4);
            continue;
        }
        if (go) {
#pragma unroll
            for (int k = 0; k < WPL; k++)
                if (k == kc) pref[k] = c;
            const int4 fx = *reinterpret_cast<const int4 *>(&tr[c].iev);  // IE, IA, tau, first edge
            const int32_t deg = min(fx.y, kAheadEdges), rs = fx.w;
            int32_t sv[kAheadEdges];
            unsigned long long dw[kAheadEdges];
#pragma unroll
            for (int j = 0; j < kAheadEdges; j++) sv[j] = deg > 0 ? col[rs + min(j, deg - 1)] : c;
#pragma unroll
            for (int j = 0; j < kAheadEdges; j++) dw[j] = dep[sv[j]];
#pragma unroll
            for (int j = 0; j < kAheadEdges; j++) {
                if (j >= deg) break;
                const uint32_t rem = (uint32_t)(dw[j] >> 43);
                if (rem == 1) {
                    const int2 e = est2[sv[j]], u = dur2[sv[j]];
                    const int4 q = *reinterpret_cast<const int4 *>(&tr[sv[j]].iev);
                    const int2 qs = *reinterpret_cast<const int2 *>(&tr[sv[j]].qpos);
                    sink ^= (uint32_t)(e.x ^ u.y ^ q.x ^ qs.x);
                } else if (rem == 2) {
                    const int32_t pu = (int32_t)((dw[j] & ((1ull << 43) - 1)) - (unsigned long long)c);
                    if (pu >= 0 && pu < d.n) {
                        const int4 q = *reinterpret_cast<const int4 *>(&tr[pu].iev);
                        const int2 qs = *reinterpret_cast<const int2 *>(&tr[pu].qpos);
                        sink ^= (uint32_t)(q.x ^ qs.y);
                    }
                    sink ^= (uint32_t)tr[sv[j]].tau;
                }
            }
        }
    }
    hs[2] = (int32_t)sink;  // keeps the reads
}

// The event loop for machines of at most 128 workers (WPL = 1: 64), one
// kernel per key kind with and without the data model, so that each gets its
// own register allocation.  Three waves per work-group: one simulates, one
// keeps the workers' best queue entries, one reads ahead.
template <int WPL, int KK, bool DATA>
__global__ __launch_bounds__(3 * kWave, WPL == 1 ? 3 : 1) void k_sim(SimArgs A) {
    using LL = LaneLds<WPL>;
    int32_t *hs = LL::template arr<int32_t>(LL::kHs);
    int2 *lrun = LL::template arr<int2>(LL::kRun);
    const int wave = uniform(threadIdx.x / kWave);
    for (;;) {
        if (threadIdx.x == 0) {
            hs[0] = dev_fetch_add(A.counter, 1);
            hs[1] = 0;
            hs[3] = 0;
        }
        for (int32_t w = threadIdx.x; w < LL::kMW; w += 3 * kWave) lrun[w] = make_int2(-1, 0);
        __syncthreads();
        const int32_t i = uniform(hs[0]);
        if (i >= A.count) break;
        const int32_t di = uniform(A.order[i]);
        if (wave == 0) {
            // the largest DAGs (dispensed first) set the batch's critical path:
            // their waves win instruction issue over co-resident waves
            if (i < A.prio_top) __builtin_amdgcn_s_setprio(3);
            else __builtin_amdgcn_s_setprio(0);
            sim_lane<WPL, KK, DATA>(A, di);
            wg_fence();
            if (threadIdx.x == 0) lds_store(&hs[1], 1);
        } else if (wave == 1) {
            keep_best<WPL, KK>(A, di);
        } else {
            read_ahead<WPL>(A, di);
        }
        __syncthreads();
    }
}

// The general event loop, for larger machines: one wave per work-group.
__global__ __launch_bounds__(kWave) void k_sim_general(SimArgs A) {
    const Lds L = carve_lds(A);
    for (;;) {
        if (threadIdx.x == 0) L.hs[0] = dev_fetch_add(A.counter, 1);
        __syncthreads();
        const int32_t i = L.hs[0];
        if (i >= A.count) break;
        if (i < A.prio_top) __builtin_amdgcn_s_setprio(3);
        else __builtin_amdgcn_s_setprio(0);
        sim_dag(A, A.order[i], L);
        __syncthreads();
    }
}

__global__ void k_counter_reset(int32_t *c) {
    if (threadIdx.x < 4) c[threadIdx.x] = 0;
}

// Unpack the schedules the simulation left in the task records into the
// caller's arrays (tasks never popped -- a failed DAG -- are left alone).
__global__ __launch_bounds__(256) void k_records(const TaskRec *tr, int64_t n, int32_t *worker, int64_t *start,
                                                 int64_t *finish, int32_t *ie_at_pop, int8_t *mode_at_pop) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int4 q = *reinterpret_cast<const int4 *>(tr + i);
    if (q.z > -2) return;
    const uint64_t wd = (uint64_t)(uint32_t)q.x | (uint64_t)(uint32_t)q.y << 32;
    const int64_t s = (int64_t)(wd & ((1ull << 42) - 1));
    worker[i] = -2 - q.z;
    start[i] = s;
    finish[i] = s + (int64_t)(wd >> 42);
    if (ie_at_pop) ie_at_pop[i] = q.w & ((1 << 22) - 1);
    if (mode_at_pop) mode_at_pop[i] = (int8_t)(q.w >> 22);
}

// The kernel of a launch and the LDS it needs for a given shape.
struct SimKernel {
    void (*run)(SimArgs);
    size_t (*lds)(int mw, int sc, int lb, int slc, int slk);
    int threads;
};

template <int WPL, int KK>
static SimKernel lane_kernel(bool data) {
    return {data ? k_sim<WPL, KK, true> : k_sim<WPL, KK, false>, LaneLds<WPL>::bytes, 3 * kWave};
}
template <int WPL>
static SimKernel lane_kernel(int kk, bool data) {
    return kk == kNarrow ? lane_kernel<WPL, kNarrow>(data)
         : kk == kFixed ? lane_kernel<WPL, kFixed>(data) : lane_kernel<WPL, kWide>(data);
}

// The one-wave loop up to 128 workers (two per lane above 64), on 32-bit keys
// where those of every DAG of the launch fit; the general loop above.
static SimKernel pick_kernel(const insp_dag *dag, const Workspace *ws, const insp_params &p) {
    if (ws->max_w > 2 * kWave) return {k_sim_general, lds_bytes, kWave};
    int kk = kNarrow;
    if (p.policy == INSP_POLICY_HEFT || p.attr_mode == INSP_ATTR_TRANSITIVE) {
        kk = kFixed;
    } else {
        for (int32_t b = ws->first; b < ws->first + ws->count; b++) {
            const int64_t n = dag->toff[b + 1] - dag->toff[b];
            if (n > 0 && 1 + 2 * field_bits((uint32_t)dag->maxdeg[b]) + field_bits((uint32_t)(n - 1)) > 32) kk = kWide;
        }
    }
    return ws->max_w <= kWave ? lane_kernel<1>(kk, p.data_bw > 0) : lane_kernel<2>(kk, p.data_bw > 0);
}

int launch_sim(insp_dag *dag, Workspace *ws, const insp_params &p, const int32_t *dur, const int32_t *est,
               int32_t *worker, int64_t *start, int64_t *finish, int64_t *makespan, int32_t *ie_at_pop,
               int8_t *mode_at_pop, insp_trace_rec *trace, int32_t *n_events, int grid, int sum_cap, int slot_cap,
               int key_cap, hipStream_t st, int prio_top, int per_cu) {
    SimArgs A;
    memset(&A, 0, sizeof A);
    A.desc = ws->desc.as<DagDesc>();
    A.order = ws->order.as<int32_t>();
    A.count = ws->count;
    A.max_w = ws->max_w;
    A.col = dag->col.as<int32_t>();
    A.dur = dur;
    A.est = est;
    A.base = ws->base;
    A.tr = ws->tr;
    A.dep = ws->dep;
    A.fbuf = ws->fbuf;
    A.slots = SlotPool::over(ws->slots.p, ws->slots.bytes);
    A.sums = ws->sums.as<unsigned long long>();
    A.paux = ws->paux.as<int32_t>();
    A.freeb_base = ws->total_wl;
    A.dag_u = ws->dag_u;
    A.dag_taubar = ws->dag_taubar;
    A.stat = dag->dag_stat.as<int32_t>();
    A.rank = dag->rank.as<int64_t>();
    A.tia = dag->tia.as<int32_t>();
    A.tie = dag->tie.as<int32_t>();
    A.attr_mode = p.attr_mode;
    A.data_bw = p.data_bw;
    A.dkib = dag->dkib.as<int32_t>();
    A.pprp = dag->pprp.as<int32_t>();
    A.ppred = dag->ppred.as<int32_t>();
    A.barr = ws->barr.as<long long>();
    A.dxc = dag->dxc.as<int32_t>();
    A.counter = ws->counter.as<int32_t>();
    A.makespan = makespan;
    A.trace = trace;
    A.n_events = n_events;
    A.policy = p.policy;
    A.s_inc = p.s_inc;
    A.s_dec = p.s_dec;
    A.dec_step = p.dec_step;
    A.c = p.c;
    A.k_num = p.k_num;
    A.k_den = p.k_den;
    A.max_events = p.max_events;
    A.prio_top = prio_top;
    // LDS: block maxima, block lists and the slots of the low blocks -- as
    // many as fit where one or two work-groups have the CU to themselves, a
    // few blocks per DAG for a larger batch (tunable)
    const SimKernel kern = pick_kernel(dag, ws, p);
    const bool one = ws->count == 1, fill = one || per_cu < 3;
    const int64_t budget = (one || per_cu == 1 ? 140 : per_cu == 2 ? 78 : 150) * 1024;
    auto need = [&](int64_t sc, int64_t lb, int64_t slc, int64_t slk) {
        return (int64_t)kern.lds(ws->max_w, (int)sc, (int)lb, (int)slc, (int)slk);
    };
    int64_t sc = std::min<int64_t>(ws->max_nblk, one ? 2048 : fill ? 512 : sum_cap);
    int64_t lb = std::min<int64_t>(ws->max_nblk, one ? 64 : fill ? 32 : 16);
    // machines of hundreds of workers: shorter LDS block lists, then fewer
    // LDS block maxima, until the per-worker state fits (the rest lives in
    // global memory)
    while (lb > 1 && need(sc, lb, 0, 0) > budget) lb /= 2;
    while (sc > 0 && need(sc, lb, 0, 0) > budget) sc /= 2;
    int64_t slc = slot_cap;
    if (fill) slc = (budget - need(sc, lb, 0, 0)) / (64 * 20);
    slc = std::max<int64_t>(0, std::min<int64_t>(ws->max_nblk, slc));
    while (slc > 0 && need(sc, lb, slc, slc) > budget) slc--;
    // keys of further blocks in what LDS is left (a rescan reads only keys)
    int64_t slk = std::max<int64_t>(slc, std::min<int64_t>(ws->max_nblk, key_cap));
    while (slk > slc && need(sc, lb, slc, slk) > budget) slk--;
    A.sum_cap = (int32_t)sc;
    A.lb = (int32_t)lb;
    A.slot_cap = (int32_t)slc;
    A.key_cap = (int32_t)slk;
    const size_t lds = (size_t)need(sc, lb, slc, slk);
    if (lds > 160 * 1024) return set_error(INSP_E_RANGE, "simulation state of %d workers exceeds LDS", ws->max_w);
    grid = std::max(1, std::min(grid, ws->count));
    if (int rc = set_lds_limit((const void *)kern.run, lds)) return rc;
    hipLaunchKernelGGL(k_counter_reset, dim3(1), dim3(64), 0, st, A.counter);
    {
        ProfScope ps(st, "sim");
        hipLaunchKernelGGL(kern.run, dim3(grid), dim3(kern.threads), lds, st, A);
    }
    INSP_HIP(hipGetLastError());
    if (ws->tasks > 0) {
        ProfScope pr(st, "rec");
        hipLaunchKernelGGL(k_records, dim3((unsigned)((ws->tasks + 255) / 256)), dim3(256), 0, st,
                           ws->tr + ws->base, ws->tasks, worker, start, finish, ie_at_pop, mode_at_pop);
    }
    INSP_HIP(hipGetLastError());
    return INSP_OK;
}

}  // namespace insp

using namespace insp;

// Transitive attributes of the range into the handle's arrays, read by the
// simulation as fixed keys.
static int run_sim_transitive(insp_dag *dag, Workspace *ws, const int32_t *est, int32_t unit_time, hipStream_t st) {
    const int64_t N = std::max<int64_t>(dag->N, 1);
    int rc;
    if ((!dag->tia.p && (rc = dag->tia.alloc(sizeof(int32_t) * N))) ||
        (!dag->tie.p && (rc = dag->tie.alloc(sizeof(int32_t) * N))))
        return rc;
    return run_transitive(dag, ws, est, unit_time, dag->tia.as<int32_t>() + ws->base,
                          dag->tie.as<int32_t>() + ws->base, false, st);
}

static int check_params(const insp_params *p) {
    if (!p) return set_error(INSP_E_INVAL, "null params");
    if (p->attr_mode < 0 || p->attr_mode > INSP_ATTR_TRANSITIVE)
        return set_error(INSP_E_INVAL, "unknown attr_mode %d", p->attr_mode);
    if (p->data_bw < 0) return set_error(INSP_E_INVAL, "negative data_bw");
    if (p->policy < 0 || p->policy > INSP_POLICY_LOCALITY) return set_error(INSP_E_INVAL, "unknown policy %d", p->policy);
    if (p->unit_time < 0 || p->max_events < 0) return set_error(INSP_E_INVAL, "negative unit_time/max_events");
    if (p->k_num > INSP_MAX_TICK || p->k_den > INSP_MAX_TICK) return set_error(INSP_E_RANGE, "k_num/k_den > 2^20");
    return INSP_OK;
}

static int check_workers(const insp_workers *w, int32_t count) {
    for (int32_t i = 0; i < count; i++) {
        if (w[i].n_cpu < 0 || w[i].n_gpu < 0) return set_error(INSP_E_INVAL, "negative worker count");
        int32_t W = w[i].n_cpu + w[i].n_gpu;
        if (W < 1 || W > INSP_MAX_WORKERS) return set_error(INSP_E_RANGE, "worker count %d outside [1, 1024]", W);
    }
    return INSP_OK;
}

static int cu_count() {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess) cus = n;
    }
    return cus;
}

// Work-groups per CU of a batch: three, which is what the default LDS shape
// (128 block maxima, 24 blocks of full entries, keys of 40) leaves room for on
// machines of up to 20 workers, and fewer, with more of each queue in LDS,
// where each DAG has a work-group of its own or the batch still ends with its
// largest DAG: a work-group's share of all tasks stays below three quarters of
// that DAG's.
// Measured, layered DAGs on 20 workers: 600 of 200-5,000 tasks with the data
// model 16.3 ms with three, 15.2 with one; 256 of 20,000 tasks 42.5 with three,
// 34.6 with one, 512 of them 51.1 and 47.1 (two); 4,096 of 200-20,000 tasks 66
// with two, 52.7 with three.
static int groups_per_cu(const insp_dag *dag, int cus) {
    int64_t most = 0;
    for (int32_t b = 0; b < dag->B; b++) most = std::max(most, dag->toff[b + 1] - dag->toff[b]);
    int k = 1;
    while (k < 3 && dag->B > cus * k && 4 * dag->N > 3 * most * cus * k) k++;
    return k;
}

extern "C" int insp_schedule(const insp_dag *cdag, int32_t index, const insp_workers *workers, const int32_t *dur,
                             const int32_t *est, const insp_params *params, int32_t *worker, int64_t *start,
                             int64_t *finish, int64_t *makespan, int32_t *ie_at_pop, int8_t *mode_at_pop,
                             insp_trace_rec *trace, int32_t *n_events, void *stream) {
    insp_dag *dag = const_cast<insp_dag *>(cdag);
    if (!dag || !workers || !makespan) return set_error(INSP_E_INVAL, "null argument");
    if (index < 0 || index >= dag->B) return set_error(INSP_E_INVAL, "dag index %d out of range", index);
    int rc;
    if ((rc = check_params(params)) || (rc = check_workers(workers, 1))) return rc;
    if (params->data_bw > 0 && !dag->dkib.p) return set_error(INSP_E_INVAL, "data_bw > 0 needs insp_set_task_data");
    const int64_t n = dag->toff[index + 1] - dag->toff[index];
    if (n > 0 && (!dur || !est || !worker || !start || !finish)) return set_error(INSP_E_INVAL, "null array");
    if ((((uintptr_t)dur | (uintptr_t)est) & 7) != 0) return set_error(INSP_E_INVAL, "dur/est rows must be 8-byte aligned");
    hipStream_t st = (hipStream_t)stream;
    INSP_HIP(hipSetDevice(dag->device));
    if ((rc = ensure_state(dag, st))) return rc;
    Workspace *ws;
    if ((rc = get_workspace(dag, index, 1, workers, true, &ws)) || (rc = ensure_sim(dag, ws))) return rc;
    if ((rc = run_attributes(dag, ws, est, params->unit_time, nullptr, nullptr, nullptr, true, st))) return rc;
    if (params->policy == INSP_POLICY_HEFT && (rc = run_rank(dag, ws, est, st))) return rc;
    if (params->attr_mode == INSP_ATTR_TRANSITIVE && (rc = run_sim_transitive(dag, ws, est, params->unit_time, st)))
        return rc;
    if (params->data_bw > 0 && (rc = ensure_preds(dag, st))) return rc;
    if (params->data_bw > 0 && !dag->dxc.p && (rc = dag->dxc.alloc(sizeof(int32_t) * std::max<int64_t>(dag->N, 1))))
        return rc;
    return launch_sim(dag, ws, *params, dur, est, worker, start, finish, makespan, ie_at_pop, mode_at_pop, trace,
                      n_events, 1, 4096, 0, 0, st, 0, 1);
}

static void parse_tune(const char *key, int *waves, int *grid, int *sum_cap, int *slot_cap, int *key_cap, int *prio,
                       int *scan) {
    if (!key) return;
    std::string s(key);
    size_t a = s.find("waves="), b = s.find("grid="), c = s.find("lds_blocks="), d = s.find("lds_slots=");
    size_t e = s.find("prio="), f = s.find("scan="), g = s.find("lds_keys=");
    if (g != std::string::npos) *key_cap = atoi(s.c_str() + g + 9);
    if (e != std::string::npos) *prio = atoi(s.c_str() + e + 5);
    if (f != std::string::npos) *scan = atoi(s.c_str() + f + 5);
    if (a != std::string::npos) *waves = atoi(s.c_str() + a + 6);
    if (b != std::string::npos) *grid = atoi(s.c_str() + b + 5);
    if (c != std::string::npos) *sum_cap = atoi(s.c_str() + c + 11);
    if (d != std::string::npos) *slot_cap = atoi(s.c_str() + d + 10);
}

namespace insp {

int batch_prologue(insp_dag *dag, const insp_workers *workers, const int32_t *dur, const int32_t *est,
                   const insp_params *params, const int32_t *worker, const int64_t *start, const int64_t *finish,
                   const int64_t *makespan, const char *tune_key, BatchLaunch *launch) {
    if (!dag || !workers || !makespan) return set_error(INSP_E_INVAL, "null argument");
    int rc;
    if ((rc = check_params(params)) || (rc = check_workers(workers, dag->B))) return rc;
    if (params->data_bw > 0 && !dag->dkib.p) return set_error(INSP_E_INVAL, "data_bw > 0 needs insp_set_task_data");
    if (dag->N > 0 && (!dur || !est || !worker || !start || !finish)) return set_error(INSP_E_INVAL, "null array");
    if ((((uintptr_t)dur | (uintptr_t)est) & 7) != 0) return set_error(INSP_E_INVAL, "dur/est rows must be 8-byte aligned");
    INSP_HIP(hipSetDevice(dag->device));
    const int cus = cu_count();
    int waves = 1, grid = std::max(1, std::min(dag->B, 3 * cus)), sum_cap = 128, slot_cap = 24, key_cap = 40, prio = 0,
        scan = kScan;
    // a key that shapes the launch has its own way
    launch->per_cu = tune_key && (strstr(tune_key, "grid=") || strstr(tune_key, "lds_")) ? 3 : groups_per_cu(dag, cus);
    if (launch->per_cu < 3) grid = std::max(1, std::min(dag->B, launch->per_cu * cus));
    parse_tune(tune_key, &waves, &grid, &sum_cap, &slot_cap, &key_cap, &prio, &scan);
    // (what a key may ask for: the general loop's LDS, and five bytes a maximum
    // that it once took besides, so that the line stays where callers know it)
    if (grid < 1 || sum_cap < 0 || sum_cap > 8192 || slot_cap < 0 || key_cap < 0 || prio < 0 || scan < 0 ||
        scan > kScan || lds_bytes(1, sum_cap, 16, slot_cap, std::max(slot_cap, key_cap)) + 5 * sum_cap > 150 * 1024)
        return set_error(INSP_E_INVAL, "bad tune key '%s'", tune_key);
    // one wave simulates one DAG; no other shape is implemented
    if (waves != 1) return set_error(INSP_E_INVAL, "tune key '%s': only waves=1 is supported", tune_key);
    launch->grid = grid;
    launch->sum_cap = sum_cap;
    launch->slot_cap = slot_cap;
    launch->key_cap = key_cap;
    launch->prio = prio;
    return INSP_OK;
}

}  // namespace insp

static int schedule_batch(const insp_dag *cdag, const insp_workers *workers, const int32_t *dur, const int32_t *est,
                          const insp_params *params, int32_t *worker, int64_t *start, int64_t *finish,
                          int64_t *makespan, int32_t *ie_at_pop, int8_t *mode_at_pop, insp_trace_rec *trace,
                          int32_t *n_events, const char *tune_key, void *stream) {
    insp_dag *dag = const_cast<insp_dag *>(cdag);
    BatchLaunch bl;
    int rc;
    if ((rc = batch_prologue(dag, workers, dur, est, params, worker, start, finish, makespan, tune_key, &bl)))
        return rc;
    hipStream_t st = (hipStream_t)stream;
    if ((rc = ensure_state(dag, st))) return rc;
    Workspace *ws;
    if ((rc = get_workspace(dag, 0, dag->B, workers, true, &ws)) || (rc = ensure_sim(dag, ws))) return rc;
    if ((rc = run_attributes(dag, ws, est, params->unit_time, nullptr, nullptr, nullptr, true, st))) return rc;
    if (params->policy == INSP_POLICY_HEFT && (rc = run_rank(dag, ws, est, st))) return rc;
    if (params->attr_mode == INSP_ATTR_TRANSITIVE && (rc = run_sim_transitive(dag, ws, est, params->unit_time, st)))
        return rc;
    if (params->data_bw > 0 && (rc = ensure_preds(dag, st))) return rc;
    if (params->data_bw > 0 && !dag->dxc.p && (rc = dag->dxc.alloc(sizeof(int32_t) * std::max<int64_t>(dag->N, 1))))
        return rc;
    return launch_sim(dag, ws, *params, dur, est, worker, start, finish, makespan, ie_at_pop, mode_at_pop, trace,
                      n_events, bl.grid, bl.sum_cap, bl.slot_cap, bl.key_cap, st, bl.prio, bl.per_cu);
}

extern "C" int insp_schedule_batch(const insp_dag *cdag, const insp_workers *workers, const int32_t *dur,
                                   const int32_t *est, const insp_params *params, int32_t *worker, int64_t *start,
                                   int64_t *finish, int64_t *makespan, int32_t *ie_at_pop, int8_t *mode_at_pop,
                                   const char *tune_key, void *stream) {
    return schedule_batch(cdag, workers, dur, est, params, worker, start, finish, makespan, ie_at_pop, mode_at_pop,
                          nullptr, nullptr, tune_key, stream);
}

extern "C" int insp_schedule_batch_trace(const insp_dag *cdag, const insp_workers *workers, const int32_t *dur,
                                         const int32_t *est, const insp_params *params, int32_t *worker,
                                         int64_t *start, int64_t *finish, int64_t *makespan, int32_t *ie_at_pop,
                                         int8_t *mode_at_pop, insp_trace_rec *trace, int32_t *n_events,
                                         const char *tune_key, void *stream) {
    if (!trace || !n_events) return set_error(INSP_E_INVAL, "insp_schedule_batch_trace: null trace or n_events");
    return schedule_batch(cdag, workers, dur, est, params, worker, start, finish, makespan, ie_at_pop, mode_at_pop,
                          trace, n_events, tune_key, stream);
}

// A batch step captured in a HIP graph owned by the library.
struct insp_graph {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    int device = 0;
};

extern "C" void insp_batch_graph_free(insp_graph *g) {
    if (!g) return;
    if (g->exec) (void)hipGraphExecDestroy(g->exec);
    if (g->graph) (void)hipGraphDestroy(g->graph);
    delete g;
}

extern "C" int insp_batch_graph_create(const insp_dag *cdag, const insp_workers *workers, const int32_t *dur,
                                       const int32_t *est, const insp_params *params, int32_t *worker,
                                       int64_t *start, int64_t *finish, int64_t *makespan, int32_t *ie_at_pop,
                                       int8_t *mode_at_pop, const char *tune_key, void *stream, insp_graph **out) {
    if (!out) return set_error(INSP_E_INVAL, "null out");
    *out = nullptr;
    // an eager step first: it builds every buffer made on first use and sets
    // the kernels' attributes, so that the captured step only launches kernels
    int rc = insp_schedule_batch(cdag, workers, dur, est, params, worker, start, finish, makespan, ie_at_pop,
                                 mode_at_pop, tune_key, stream);
    if (rc) return rc;
    INSP_HIP(hipStreamSynchronize((hipStream_t)stream));
    std::unique_ptr<insp_graph> g(new insp_graph());
    g->device = cdag->device;
    hipStream_t cs = nullptr;
    INSP_HIP(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
        prof_suspend(true);
        rc = insp_schedule_batch(cdag, workers, dur, est, params, worker, start, finish, makespan, ie_at_pop,
                                 mode_at_pop, tune_key, cs);
        prof_suspend(false);
        e = hipStreamEndCapture(cs, &g->graph);
    }
    (void)hipStreamDestroy(cs);
    if (rc) return rc;
    if (e != hipSuccess) return set_error(INSP_E_DEVICE, "graph capture failed: %s", hipGetErrorString(e));
    INSP_HIP(hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0));
    *out = g.release();
    return INSP_OK;
}

extern "C" int insp_batch_graph_launch(insp_graph *g, void *stream) {
    if (!g || !g->exec) return set_error(INSP_E_INVAL, "null graph");
    INSP_HIP(hipSetDevice(g->device));
    INSP_HIP(hipGraphLaunch(g->exec, (hipStream_t)stream));
    return INSP_OK;
}

#ifdef INSP_PHASE_CLOCKS
extern "C" int insp_debug_phase_clocks(unsigned long long *host, int count) {
    INSP_HIP(hipMemcpyFromSymbol(host, HIP_SYMBOL(g_phase_clk), sizeof(unsigned long long) * 32 * count));
    return INSP_OK;
}
#endif

extern "C" int insp_sync_status(const insp_dag *cdag, void *stream) {
    if (!cdag) return set_error(INSP_E_INVAL, "null handle");
    insp_dag *dag = const_cast<insp_dag *>(cdag);
    hipStream_t st = (hipStream_t)stream;
    INSP_HIP(hipSetDevice(dag->device));
    INSP_HIP(hipStreamSynchronize(st));
    if (!dag->dag_stat.p) return INSP_OK;
    // the latest schedule's status words and the failures of earlier calls
    // not yet reported; both are cleared once read
    std::vector<int32_t> stat(2 * dag->B), sticky(dag->B);
    INSP_HIP(hipMemcpyAsync(stat.data(), dag->dag_stat.p, sizeof(int32_t) * 2 * dag->B, hipMemcpyDeviceToHost, st));
    INSP_HIP(hipMemcpyAsync(sticky.data(), dag->dag_sticky.p, sizeof(int32_t) * dag->B, hipMemcpyDeviceToHost, st));
    INSP_HIP(hipStreamSynchronize(st));
    bool any = false;
    for (int32_t b = 0; b < dag->B; b++) {
        any |= (stat[2 * b] | sticky[b]) != 0;
        stat[2 * b] |= sticky[b];
    }
    if (any) {
        std::vector<int32_t> zero(2 * dag->B, 0);
        for (int32_t b = 0; b < dag->B; b++) zero[2 * b + 1] = stat[2 * b + 1];  // event counts stay
        INSP_HIP(hipMemcpyAsync(dag->dag_stat.p, zero.data(), sizeof(int32_t) * 2 * dag->B, hipMemcpyHostToDevice, st));
        INSP_HIP(hipMemsetAsync(dag->dag_sticky.p, 0, sizeof(int32_t) * dag->B, st));
        INSP_HIP(hipStreamSynchronize(st));
    }
    for (int32_t b = 0; b < dag->B; b++) {
        if (stat[2 * b] & ST_EST) return set_error(INSP_E_RANGE, "estimate outside [1, 2^20] in DAG %d", b);
        if (stat[2 * b] & ST_DUR) return set_error(INSP_E_RANGE, "duration outside [1, 2^20] in DAG %d", b);
        if (stat[2 * b] & ST_RANK) return set_error(INSP_E_RANGE, "HEFT rank of DAG %d reaches 2^42", b);
        if (stat[2 * b] & ST_PATH) return set_error(INSP_E_RANGE, "longest path of DAG %d reaches 2^30 ticks", b);
        if (stat[2 * b] & ST_XFER)
            return set_error(INSP_E_RANGE, "input transfers of a task of DAG %d exceed 2^20 ticks", b);
        if (stat[2 * b] & ST_HANG)
            return set_error(INSP_E_HANG, "DAG %d needed more than max_events events", b);
    }
    return INSP_OK;
}
