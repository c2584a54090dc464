// Transitive reading of the inspiring attributes (Section 4.3: the source of
// a fully connected DAG scores the number of its tasks; Section 4.2: with a
// large unit time IE converges to IA; Section 7: IE looks at a time window
// after the task), computed on the whole graph:
//   D(v)       = v and every task reachable from v,
//   IA_T(v)    = |D(v)|,
//   EF_v(d)    = the longest tau-weighted path from v to d, both ends
//                included (d's earliest finish with v starting at 0 and
//                unlimited workers),
//   IE_T(v; U) = #{d in D(v) : EF_v(d) <= U}.
//
// The forward pass over D(v) keeps EF in LDS by position in a level order of
// the DAG, so the descendants of a level sit behind it and are final once the
// level is reached.  Each source leaves IA_T, and either its count within an
// explicit U or its cumulative counts per ladder rung 2^j; a per-DAG pass then
// scores the rungs and picks U.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "common.hpp"
#include "internal.hpp"

namespace insp {

constexpr int kTT = 512;                 // threads per work-group of the per-DAG pass
constexpr uint32_t kPathCap = 1u << 30;  // paths saturate here (out of range)

// Forms of the forward pass.  A source runs in the one that its window (the
// positions behind it) and its DAG select, in a launch for windows of about
// its size, as LDS is what limits the sources in flight:
//   kSmall  one wave, EF in 32 bits with LDS atomicMax: windows up to kSmallMax;
//   kHalf   one wave, EF in 16 bits: up to kHalfMax, in DAGs whose paths stay below 2^16;
//   kTeam   eight waves, EF in 32 bits: the others up to kTeamMax (two or more a CU);
//   kCrew   sixteen waves: those of which a CU holds one.
// The lines, on the batch of 768 layered DAGs (200-20,000 tasks): 16 bits take
// twice the sources and twice the instructions, so that up to 2,500 both forms
// are even (58.4 and 58.6 ms with the line at 500 and at 2,500; a chain of
// 2,000 tasks takes 2.57 ms in 16 bits and 1.70 in 32).  With teams from
// 5,200, 6,600, 8,600, 10,000, 14,600 and 18,700 on the batch takes 50.4, 48.7, 48.0,
// 48.1, 51.7 and 55.8 ms: larger windows leave too few single waves on a CU.
// A crew takes 2.39 ms for one DAG of 32,768 tasks, a team 2.84.
enum { kSmall, kHalf, kTeam, kCrew };
constexpr int32_t kSmallMax = 2500, kHalfMax = 8600, kTeamMax = 19900;
// Largest windows of the launches (those of one that would not fill the chip
// four times over go to the next larger one).
constexpr int32_t kCaps[] = {600, 1200, 2500, 3500, 5200, 6600, 8600, 10000, 12000, 14600, 19900, INSP_MAX_TRANSITIVE_TASKS};
constexpr int kReachCounters = 8;
constexpr int kReachMax = 2 * sizeof(kCaps) / sizeof(kCaps[0]);
struct ReachList {
    int32_t count;
    int32_t form[kReachMax], lo[kReachMax], hi[kReachMax];  // windows lo < n - position <= hi
};

struct TransArgs {
    const DagDesc *desc;
    int32_t count;
    int64_t base, items;
    const int32_t *topo, *lvl, *nlev;
    const uint4 *rec;         // per position: its successors' positions
    const uint4 *more;        // ... those of tasks with more than eight
    int32_t *ptau;
    int32_t clear_status;
    const int32_t *est;
    int32_t unit_time;
    int32_t *ia, *ie;         // outputs by task, relative to base
    int32_t *cum;             // [items][kTRungs]: members with EF <= 2^j (automatic U)
    unsigned int *longest;    // [count]: longest path of each DAG
    unsigned int *maxtau;     // [count]: its largest tau
    int32_t *pre;             // [kReachMax][count + 1]: sources of a launch before each DAG
    int32_t *next;            // [kReachMax][kReachCounters], 32 words apart: chunks taken
    int32_t *score;           // [count][kTRungs]: sources of a DAG with 0 < count < IA at a rung
    int32_t *stat;
};

// Workspace DAG holding item `item` (its tasks are items toff - base ...).
__device__ __forceinline__ int32_t desc_of(const DagDesc *desc, int32_t count, int64_t base, int64_t item) {
    int32_t lo = 0, hi = count - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (desc[mid].toff - base <= item) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ int32_t dag_of_off(const int64_t *off, int32_t B, int64_t x) {
    int32_t lo = 0, hi = B - 1;  // last b with off[b] <= x
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (off[mid] <= x) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// ---------------------------------------------------------------------------
// Per handle: successors' positions in level order.

__global__ __launch_bounds__(256) void k_positions(int32_t B, const int64_t *toff, const int32_t *topo, int32_t *ppos) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= toff[B]) return;
    const int64_t t0 = toff[dag_of_off(toff, B, t)];
    ppos[t0 + topo[t]] = (int32_t)(t - t0);
}

// A task's record: eight 16-bit positions of successors, the last of them
// first and n behind the others; a task with more has four, then where its
// further records of eight start, how many they are, and 0xFFFF.
__global__ __launch_bounds__(256) void k_reach_rec(int32_t B, const int64_t *toff, const int64_t *eoff,
                                                    const int32_t *rp, const int32_t *col, const int32_t *ppos,
                                                    uint4 *rec, uint4 *more, int32_t *used) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= toff[B]) return;
    const int32_t b = dag_of_off(toff, B, t);
    const int64_t t0 = toff[b];
    const int32_t n = (int32_t)(toff[b + 1] - t0);
    if (n > INSP_MAX_TRANSITIVE_TASKS) return;  // refused
    const int32_t *r = rp + t0 + b + (t - t0);
    const int32_t *c = col + eoff[b];
    const int32_t e0 = r[0], deg = r[1] - e0;
    int32_t last = 0, at = 0;
    for (int32_t k = 0; k < deg; k++) {
        const int32_t q = ppos[t0 + c[e0 + k]];
        if (q > last) {
            last = q;
            at = k;
        }
    }
    // successor k with the last one moved to the front
    auto pos = [&](int32_t k) -> uint32_t {
        if (k >= deg) return (uint32_t)n;
        return (uint32_t)(k == 0 ? last : ppos[t0 + c[e0 + (k == at ? 0 : k)]]);
    };
    auto eight = [&](int32_t k) {
        return make_uint4(pos(k) | pos(k + 1) << 16, pos(k + 2) | pos(k + 3) << 16, pos(k + 4) | pos(k + 5) << 16,
                          pos(k + 6) | pos(k + 7) << 16);
    };
    uint4 x = eight(0);
    if (deg > 8) {
        const int32_t cnt = (deg - 4 + 7) / 8;
        const int32_t off = dev_fetch_add(used, cnt);
        for (int32_t j = 0; j < cnt; j++) more[off + j] = eight(4 + 8 * j);
        x.z = (uint32_t)off;
        x.w = (uint32_t)cnt | 0xFFFF0000u;
    }
    rec[t0 + ppos[t]] = x;
}

// ---------------------------------------------------------------------------
// Per call.

// tau by position (the GPU estimate when the machine has GPU workers, else
// the CPU one) and its maximum; estimates outside [1, 2^20] flag the DAG.
__global__ __launch_bounds__(256) void k_position_tau(TransArgs A) {
    const int64_t item = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool on = item < A.items;
    const int32_t d = desc_of(A.desc, A.count, A.base, on ? item : A.items - 1);
    uint32_t tau = 0;
    if (on) {
        const DagDesc D = A.desc[d];
        const int64_t u0 = D.toff - A.base;
        const int32_t i = (int32_t)(item - u0);
        const int32_t v = A.topo[D.toff + i];
        const int2 e = reinterpret_cast<const int2 *>(A.est)[u0 + v];
        if (e.x < 1 || e.x > INSP_MAX_TICK || e.y < 1 || e.y > INSP_MAX_TICK) atomicOr(&A.stat[2 * D.id], ST_EST);
        // clamped, so that paths stay in 32 bits even for a DAG already flagged
        tau = (uint32_t)min(max(D.n_gpu > 0 ? e.y : e.x, 1), INSP_MAX_TICK);
        A.ptau[D.toff + i] = (int32_t)tau;
    }
    // the maximum: one atomic a wave for the DAG of its first lane
    const int32_t d0 = uniform(d);
    const uint32_t m = wave_max_u32f(d == d0 ? tau : 0u);
    if (d != d0) atomicMax(&A.maxtau[d], tau);
    else if ((threadIdx.x & 63) == 0) atomicMax(&A.maxtau[d], m);
}

__global__ void k_trans_clear(TransArgs A) {
    const int32_t d = blockIdx.x * 256 + threadIdx.x;
    if (d < A.count) {
        A.longest[d] = A.maxtau[d] = 0;
        for (int j = 0; j < kTRungs; j++) A.score[d * kTRungs + j] = 0;
        if (A.clear_status) A.stat[2 * A.desc[d].id] = 0;
    }
    if (d < kReachMax * kReachCounters) A.next[d * 32] = 0;
}

// Sources of launch blockIdx.x before each DAG.
__global__ __launch_bounds__(1024) void k_reach_lists(TransArgs A, ReachList R) {
    __shared__ int32_t part[16];
    const int32_t form = R.form[blockIdx.x], wlo = R.lo[blockIdx.x], whi = R.hi[blockIdx.x];
    int32_t *pre = A.pre + (int64_t)blockIdx.x * (A.count + 1);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int32_t sum = 0;
    for (int32_t d0 = 0; d0 < A.count; d0 += 1024) {
        const int32_t d = d0 + tid;
        int32_t c = 0;
        if (d < A.count) {
            const int32_t n = A.desc[d].n;
            c = max(0, n - wlo) - max(0, n - whi);
            if (c > 0 && form != kSmall && wlo < kHalfMax) {
                // no path is longer than its levels at the largest tau
                const bool half = (uint64_t)A.nlev[A.desc[d].id] * A.maxtau[d] < 65535;
                if (half != (form == kHalf)) c = 0;
            }
        }
        const int32_t inc = wave_incl_scan(c);
        __syncthreads();
        if (lane == 63) part[wv] = inc;
        __syncthreads();
        int32_t off = sum;
        for (int w = 0; w < 16; w++) {
            if (w < wv) off += part[w];
            sum += part[w];
        }
        if (d < A.count) pre[d] = off + inc - c;
    }
    if (tid == 0) pre[A.count] = sum;
}

typedef uint16_t __attribute__((may_alias)) u16a;
typedef uint32_t __attribute__((may_alias)) u32a;
typedef uint2 __attribute__((may_alias)) uint2a;
typedef uint4 __attribute__((may_alias)) uint4a;

// Order LDS accesses of the wave's lanes (which execute in step).
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// EF of up to eight successors raised to v (positions n are none): win holds
// EF by position less `b0`.  `meanwhile` runs while the first readings are on
// their way.
template <bool HALF, typename F>
__device__ __forceinline__ void reach_push(uint8_t *win, int32_t b0, uint32_t n, u16a *spare, uint4 r, uint32_t v, F &&meanwhile) {
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
    if constexpr (!HALF) {
        u32a *ef = reinterpret_cast<u32a *>(win) - b0;
#pragma unroll
        for (int j = 0; j < 8; j++) {
            // (lanes without a successor stay out: atomics on one address take turns)
            const uint32_t p = j & 1 ? w[j >> 1] >> 16 : w[j >> 1] & 0xFFFFu;
            if (p != n) (void)__hip_atomic_fetch_max(&ef[p], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        meanwhile();
    } else {
        // LDS has no 16-bit maximum: written where v is larger (elsewhere to
        // a slot of the lane's own), and again where another lane's smaller
        // value has gone over it
        u16a *at[8];
        uint32_t c[8];
#pragma unroll
        for (int j = 0; j < 8; j++) {
            at[j] = reinterpret_cast<u16a *>(win) + ((j & 1 ? w[j >> 1] >> 16 : w[j >> 1] & 0xFFFFu) - (uint32_t)b0);
            c[j] = *at[j];
        }
        meanwhile();
        bool again;
        do {
            wave_order();
#pragma unroll
            for (int j = 0; j < 8; j++) *(v > c[j] ? at[j] : spare) = (uint16_t)v;
            wave_order();
#pragma unroll
            for (int j = 0; j < 8; j++) c[j] = *at[j];
            again = false;
#pragma unroll
            for (int j = 0; j < 8; j++) again |= v > c[j];
        } while (again);
        wave_order();
    }
}

// The forward pass of one source after another: a wave (or NW waves) walks
// the levels behind the source, collects the tasks reached (EF not zero),
// counts them by ladder rung, and raises the EF of their successors.
//
// What bounds it is LDS space and the chain per level: few waves fit a CU
// beside their windows, and each level takes two or three LDS trips and one to
// the L2.  So a window holds no more than the positions behind the source; a
// single wave first collects a level's tasks (46 of 400 are reached, in a
// layered DAG of 13,000), so that one step over full lanes serves them, while
// a team takes a position per lane and skips 64 at a time; and a task's
// successors are one 16-byte load.  What goes to a DAG as a whole (longest
// path, scores) is kept in registers until the DAG changes: one atomic per
// source on the same words took 100 us each.
// Measured on the batch of 768 layered DAGs (3.2 M sources, 69 M levels):
// 48 ms, against 184 in a work-group of 512 threads per source that read one
// edge at a time; one DAG of 1,000 tasks 0.12 ms against 0.23, of 20,000 0.96
// against 1.83.
template <bool HALF>
using reach_entry = std::conditional_t<HALF, uint32_t, uint2>;
constexpr int kReachList = 384, kReachCols = 8;

template <bool HALF, int NW>
__global__ __launch_bounds__(NW *kWave) void k_reach(TransArgs A, int32_t cls, int32_t wmax, int32_t chunk, int32_t entries) {
    static_assert(!HALF || NW == 1, "16-bit windows belong to one wave");
    constexpr uint32_t kFull = HALF ? 0xFFFFu : 0xFFFFFFFFu;
    constexpr int kES = HALF ? 2 : 4;
    extern __shared__ __align__(16) uint8_t win[];  // EF [entries]
    // one wave's tasks reached in a level: position, largest EF of the predecessors
    __shared__ reach_entry<HALF> list[NW == 1 ? kReachList + kWave : 1];
    __shared__ __align__(16) uint32_t hist[kTRungs * kReachCols];
    __shared__ uint32_t s_spare[kWave];
    __shared__ int32_t s_id, s_hi;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = NW == 1 ? 0 : uniform(tid >> 6);
    const uint32_t ut = (uint32_t)A.unit_time;
    const int32_t *pre = A.pre + (int64_t)cls * (A.count + 1);
    const int32_t total = pre[A.count];
    u16a *spare = reinterpret_cast<u16a *>(&s_spare[lane]);
    auto sync = [&] {
        if constexpr (NW > 1) __syncthreads();
        else wave_order();
    };
    for (int32_t k = tid * 16; k < entries * kES; k += NW * kWave * 16) *reinterpret_cast<uint4a *>(win + k) = make_uint4(0, 0, 0, 0);
    for (int k = tid; k < kTRungs * kReachCols; k += NW * kWave) hist[k] = 0;
    int32_t d = 0;
    // of DAG d so far: longest path, and scores (odd lanes, a rung each)
    uint32_t longest = 0;
    int32_t scored = 0;
    auto flush = [&] {
        longest = wave_max_u32f(longest);
        if (lane == 0 && longest) atomicMax(&A.longest[d], longest);
        if (ut == 0 && (lane & 1) && scored) atomicAdd(&A.score[d * kTRungs + (lane >> 1)], scored);
        longest = 0;
        scored = 0;
    };
    // every eighth chunk belongs to one counter (a single one would hand out
    // no more than 30 a microsecond), and a group's first goes by its index
    const int32_t q = (int32_t)blockIdx.x % kReachCounters;
    for (int32_t id = (int32_t)blockIdx.x * chunk; id < total;) {
        const int32_t id_end = min(id + chunk, total);
        while (id < id_end) {
            // the DAG of source id: the last whose sources start at or before it
            if (pre[d + 1] <= id) {
                flush();
                int32_t lo = d + 1, hi = A.count - 1;
                while (lo < hi) {
                    const int32_t mid = (lo + hi + 1) >> 1;
                    if (pre[mid] <= id) lo = mid;
                    else hi = mid - 1;
                }
                d = uniform(lo);
            }
            const DagDesc D = A.desc[d];
            const int32_t n = D.n;
            const int32_t *ls = A.lvl + D.toff + D.id;
            const int32_t nl = uniform(A.nlev[D.id]);
            const uint4 *rec = A.rec + D.toff;
            const int32_t *ptau = A.ptau + D.toff;
            const int64_t u0 = D.toff - A.base;
            const int32_t i0 = max(0, n - wmax) + (id - pre[d]);
            const int32_t i1 = i0 + min(id_end, pre[d + 1]) - id;
            id += i1 - i0;
            // ends of 64 levels at a time, in the lanes
            int32_t Lb = 0, ends = ls[min(1 + lane, nl)];
            auto end_of = [&](int32_t L) {
                if ((uint32_t)(L - Lb) >= 64u) {
                    Lb = L;
                    ends = ls[min(L + 1 + lane, nl)];
                }
                return __builtin_amdgcn_readlane(ends, L - Lb);
            };
            int32_t L0 = 0;
            while (end_of(L0) <= i0) L0 += __popcll(ballot(Lb + lane < nl && ends <= i0)) - (L0 - Lb);
            for (int32_t i = i0; i < i1; i++) {
                while (end_of(L0) <= i) L0++;
                const int32_t b0 = (i + 1) & ~3;
                int32_t hi = 0;  // last position reached
                const uint32_t none = (uint32_t)n << 16 | (uint32_t)n;
                // a task per lane, its record and EF: counted by rung, its successors raised
                auto step = [&](bool on, uint4 cur, uint32_t v) {
                    if (!HALF) v = min(v, kPathCap);
                    const bool ext = cur.w >= 0xFFFF0000u;
                    const uint32_t off = cur.z, more = ext ? cur.w & 0xFFFFu : 0u;
                    if (ext) cur.z = cur.w = none;
                    reach_push<HALF>(win, b0, (uint32_t)n, spare, cur, v, [&] {
                        const uint32_t to = cur.x & 0xFFFFu;
                        hi = max(hi, (int32_t)wave_max_u32f(to == (uint32_t)n ? 0u : to));
                        longest = max(longest, v);
                        // smallest j with v <= 2^j, or within / past the unit time
                        const uint32_t j = ut ? (v <= ut ? 0u : 1u) : v <= 1 ? 0u : 32u - (uint32_t)__clz(v - 1);
                        (void)__hip_atomic_fetch_add(on ? &hist[j * kReachCols + (lane & (kReachCols - 1))] : &s_spare[lane],
                                                     1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    });
                    // further records: up to eight lane by lane, longer rows by the whole wave
                    if (ballot(ext)) {
                        for (uint32_t q = 0; ballot(q < more && more <= 8); q++)
                            if (q < more && more <= 8) reach_push<HALF>(win, b0, (uint32_t)n, spare, A.more[off + q], v, [] {});
                        for (uint64_t rows = ballot(more > 8); rows; rows &= rows - 1) {
                            const int l = __builtin_ctzll(rows);
                            const uint32_t ro = (uint32_t)__builtin_amdgcn_readlane((int)off, l);
                            const uint32_t rc = (uint32_t)__builtin_amdgcn_readlane((int)more, l);
                            const uint32_t rv = (uint32_t)__builtin_amdgcn_readlane((int)v, l);
                            for (uint32_t q = (uint32_t)lane; q < rc; q += kWave)
                                reach_push<HALF>(win, b0, (uint32_t)n, spare, A.more[ro + q], rv, [] {});
                        }
                    }
                };
                // a task's record and tau
                auto fetch = [&](bool on, uint32_t pos, uint4 &r, uint32_t &t) {
                    r = make_uint4(none, none, none, none);
                    t = 0;
                    if (on) {
                        r = rec[pos];
                        t = (uint32_t)ptau[pos];
                    }
                };
                // the slot behind the last task takes what records hold too much
                if (tid == 0) {
                    if constexpr (HALF) reinterpret_cast<u16a *>(win)[n - b0] = (uint16_t)kFull;
                    else reinterpret_cast<u32a *>(win)[n - b0] = kFull;
                    if (NW > 1) s_hi = 0;
                }
                sync();
                uint4 r;
                uint32_t t;
                if (wv == 0) {
                    fetch(lane == 0, (uint32_t)i, r, t);
                    step(lane == 0, r, t);
                }
                int32_t a = end_of(L0);
                for (int32_t L = L0 + 1;; L++) {
                    // (a team's waves read s_hi before any goes on to raise it)
                    if constexpr (NW > 1) {
                        if (lane == 0) atomicMax(&s_hi, hi);
                        __syncthreads();
                        hi = uniform(s_hi);
                    }
                    if (a > hi) break;
                    const int32_t z = end_of(L);
                    if constexpr (NW > 1) {
                        u32a *ef = reinterpret_cast<u32a *>(win) - b0;
                        for (int32_t g = a + kWave * wv; g < z; g += kWave * NW) {
                            const int32_t p = g + lane;
                            const uint32_t x = p < z ? ef[p] : 0u;
                            if (!ballot(x != 0)) continue;
                            fetch(x != 0, (uint32_t)p, r, t);
                            if (x) ef[p] = 0;
                            step(x != 0, r, x ? x + t : 0u);
                        }
                    } else {
                        uint32_t cnt = 0;
                        for (int32_t g = a & ~3; g < z; g += 256) {
                            const int32_t p = g + 4 * lane;
                            // read and cleared, up to the level's end
                            uint32_t x[4];
                            if constexpr (HALF) {
                                uint2a *w = reinterpret_cast<uint2a *>(win + (size_t)(p - b0) * 2);
                                uint2 y = make_uint2(0, 0);
                                if (p < z) y = *w;
                                x[0] = p < z ? y.x & 0xFFFFu : 0u;
                                x[1] = p + 1 < z ? y.x >> 16 : 0u;
                                x[2] = p + 2 < z ? y.y & 0xFFFFu : 0u;
                                x[3] = p + 3 < z ? y.y >> 16 : 0u;
                                if (p < z) *w = make_uint2(y.x ^ (x[0] | x[1] << 16), y.y ^ (x[2] | x[3] << 16));
                            } else {
                                uint4a *w = reinterpret_cast<uint4a *>(win + (size_t)(p - b0) * 4);
                                uint4 y = make_uint4(0, 0, 0, 0);
                                if (p < z) y = *w;
                                x[0] = p < z ? y.x : 0u;
                                x[1] = p + 1 < z ? y.y : 0u;
                                x[2] = p + 2 < z ? y.z : 0u;
                                x[3] = p + 3 < z ? y.w : 0u;
                                if (p < z) *w = make_uint4(y.x ^ x[0], y.y ^ x[1], y.z ^ x[2], y.w ^ x[3]);
                            }
                            // appended to the list, lane by lane
                            const uint32_t c = (x[0] != 0) + (x[1] != 0) + (x[2] != 0) + (x[3] != 0);
                            const uint32_t inc = (uint32_t)wave_incl_scan((int32_t)c);
                            uint32_t at = cnt + inc - c;
#pragma unroll
                            for (int j = 0; j < 4; j++) {
                                const uint32_t k = x[j] ? at : (uint32_t)(kReachList + lane);
                                if constexpr (HALF) list[k] = (uint32_t)(p + j) | x[j] << 16;
                                else list[k] = make_uint2((uint32_t)(p + j), x[j]);
                                at += x[j] ? 1u : 0u;
                            }
                            cnt += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
                            if (g + 256 < z && cnt <= kReachList - 256) continue;  // room for the next 256 positions
                            wave_order();
                            // served 64 at a time, the next ones' records on their way
                            auto entry = [&](uint32_t k) {
                                const auto e = list[min(k, (uint32_t)kReachList - 1)];
                                if constexpr (HALF) return make_uint2(e & 0xFFFFu, e >> 16);
                                else return e;
                            };
                            uint2 e = entry((uint32_t)lane);
                            fetch((uint32_t)lane < cnt, e.x, r, t);
                            for (uint32_t k = 0; k < cnt; k += kWave) {
                                const uint4 cur = r;
                                const uint32_t v = k + lane < cnt ? e.y + t : 0u;
                                if (k + kWave < cnt) {
                                    e = entry(k + kWave + lane);
                                    fetch(k + kWave + lane < cnt, e.x, r, t);
                                }
                                step(k + lane < cnt, cur, v);
                            }
                            wave_order();
                            cnt = 0;
                        }
                    }
                    a = z;
                }
                sync();
                if (tid == 0) {
                    if constexpr (HALF) reinterpret_cast<u16a *>(win)[n - b0] = 0;
                    else reinterpret_cast<u32a *>(win)[n - b0] = 0;
                }
                if (wv == 0) {
                    // two lanes a rung
                    uint4a *h = reinterpret_cast<uint4a *>(hist) + lane;
                    const uint4 x = *h;
                    *h = make_uint4(0, 0, 0, 0);
                    const int32_t c = wave_incl_scan((int32_t)(x.x + x.y + x.z + x.w));
                    const int64_t v = u0 + A.topo[D.toff + i];
                    const int32_t members = __builtin_amdgcn_readlane(c, 63);
                    scored += c > 0 && c < members ? 1 : 0;
                    if (ut == 0 && (lane & 1)) A.cum[v * kTRungs + (lane >> 1)] = c;
                    if (lane == 63) A.ia[v] = c;
                    if (ut != 0 && lane == 1) A.ie[v] = c;
                }
                sync();
            }
        }
        if ((int64_t)gridDim.x * chunk >= total) break;
        if (NW > 1) __syncthreads();
        if (tid == 0) {
            const int32_t k = dev_fetch_add(&A.next[(cls * kReachCounters + q) * 32], 1);
            id = ((k + ((int32_t)gridDim.x - q + kReachCounters - 1) / kReachCounters) * kReachCounters + q) * chunk;
        }
        if constexpr (NW > 1) {
            if (tid == 0) s_id = id;
            __syncthreads();
            id = s_id;
        }
        id = uniform(id);
    }
    flush();
}

// Per DAG: the range check on the longest path, and with an automatic U the
// ladder U = 2^j, j = 0..J (2^J the first power of two at least the longest
// path), scored by #{v : 0 < IE_T < IA_T}, the larger U on a tie.
__global__ __launch_bounds__(kTT) void k_trans_select(TransArgs A, int32_t *u_out) {
    __shared__ int32_t s_best;
    const int tid = threadIdx.x;
    const DagDesc D = A.desc[blockIdx.x];
    const int64_t u0 = D.toff - A.base;
    const uint32_t cp = A.longest[blockIdx.x];
    if (cp >= kPathCap) {
        if (tid == 0) {
            atomicOr(&A.stat[2 * D.id], ST_PATH);
            u_out[blockIdx.x] = 0;
        }
        return;
    }
    if (A.unit_time > 0 || D.n == 0) {
        if (tid == 0) u_out[blockIdx.x] = A.unit_time > 0 ? A.unit_time : 1;
        return;
    }
    int J = 0;
    while ((1u << J) < cp) J++;
    // the best rung of 0..J, the larger on a tie
    int32_t best = 0;
    if (tid < kWave)
        best = (int32_t)(wave_max_u64f(tid <= J ? (uint64_t)(uint32_t)A.score[blockIdx.x * kTRungs + tid] << 32 | (uint32_t)tid : 0ull) & 0xFFu);
    if (tid == 0) {
        s_best = best;
        u_out[blockIdx.x] = 1 << best;
    }
    __syncthreads();
#pragma unroll 4
    for (int32_t v = tid; v < D.n; v += kTT) A.ie[u0 + v] = A.cum[(u0 + v) * kTRungs + s_best];
}

// Successor records by position, built once.
static int ensure_records(insp_dag *dag, hipStream_t st) {
    int rc;
    if ((rc = ensure_levels(dag, st))) return rc;
    if (dag->rrec.p) return INSP_OK;
    const int64_t N = std::max<int64_t>(dag->N, 1);
    DevBuf ppos, rec, used;
    // (a task of more than eight successors has at most a sixth as many further records)
    if ((rc = ppos.alloc(sizeof(int32_t) * N)) || (rc = used.alloc(sizeof(int32_t))) ||
        (rc = rec.alloc(sizeof(uint4) * N)) || (rc = dag->rmore.alloc(sizeof(uint4) * (dag->M / 6 + 1))))
        return rc;
    INSP_HIP(hipMemsetAsync(used.p, 0, sizeof(int32_t), st));
    if (dag->N > 0) {
        const dim3 grid((unsigned)((dag->N + 255) / 256));
        hipLaunchKernelGGL(k_positions, grid, dim3(256), 0, st, dag->B, dag->d_toff.as<int64_t>(),
                           dag->topo.as<int32_t>(), ppos.as<int32_t>());
        hipLaunchKernelGGL(k_reach_rec, grid, dim3(256), 0, st, dag->B, dag->d_toff.as<int64_t>(),
                           dag->d_eoff.as<int64_t>(), dag->rp.as<int32_t>(), dag->col.as<int32_t>(),
                           ppos.as<int32_t>(), rec.as<uint4>(), dag->rmore.as<uint4>(), used.as<int32_t>());
    }
    INSP_HIP(hipGetLastError());
    INSP_HIP(hipStreamSynchronize(st));  // before the scratch is freed
    std::swap(dag->rrec.p, rec.p);
    std::swap(dag->rrec.bytes, rec.bytes);
    return INSP_OK;
}

// Work-groups of a launch that a CU holds.
static int64_t reach_groups(int form, int32_t entries) {
    const int64_t word = form == kHalf ? 2 : 4, list = form == kSmall ? 8 : form == kHalf ? 4 : 0;
    const int64_t lds = entries * word + (kReachList + kWave) * list + 4 * kTRungs * kReachCols + 768;
    const int64_t most = form == kCrew ? 2 : form == kTeam ? 4 : 28;  // (by registers)
    return std::max<int64_t>(1, std::min<int64_t>(most, 160 * 1024 / lds));
}
// A window, the slot behind it, and whole groups of four.
static int32_t reach_entries(int32_t window) { return (window + 5 + 7) & ~7; }

template <bool HALF, int NW>
static int launch_reach(const TransArgs &A, int cls, int32_t window, int64_t sources, int64_t groups, hipStream_t st) {
    const int32_t entries = reach_entries(window);
    const size_t lds = (size_t)entries * (HALF ? 2 : 4);
    if (int rc = set_lds_limit((const void *)&k_reach<HALF, NW>, lds)) return rc;
    const int32_t chunk = (int32_t)std::min<int64_t>(8, std::max<int64_t>(1, sources / (8 * groups)));
    hipLaunchKernelGGL((k_reach<HALF, NW>), dim3((unsigned)std::min<int64_t>((sources + chunk - 1) / chunk, groups)), dim3(NW * kWave), lds, st,
                       A, (int32_t)cls, window, chunk, entries);
    return INSP_OK;
}

int run_transitive(insp_dag *dag, Workspace *ws, const int32_t *est, int32_t unit_time, int32_t *ia, int32_t *ie,
                   bool clear_status, hipStream_t st) {
    int rc;
    int32_t maxn = 0;
    for (int32_t i = 0; i < ws->count; i++) {
        const int32_t b = ws->first + i;
        maxn = std::max<int32_t>(maxn, (int32_t)(dag->toff[b + 1] - dag->toff[b]));
    }
    if (maxn > INSP_MAX_TRANSITIVE_TASKS)
        return set_error(INSP_E_RANGE, "transitive attributes need DAGs of at most %d tasks (got %d)",
                         INSP_MAX_TRANSITIVE_TASKS, maxn);
    if ((rc = ensure_records(dag, st))) return rc;
    const int64_t N = std::max<int64_t>(dag->N, 1);
    if (!dag->ptau.p && (rc = dag->ptau.alloc(sizeof(int32_t) * N))) return rc;
    if (unit_time == 0 && dag->tcum.bytes < sizeof(int32_t) * kTRungs * (size_t)std::max<int64_t>(ws->tasks, 1) &&
        (rc = dag->tcum.alloc(sizeof(int32_t) * kTRungs * (size_t)std::max<int64_t>(ws->tasks, 1))))
        return rc;
    // longest path and largest tau per DAG, the launches' lists and counters
    const size_t words = 2 * (size_t)std::max(ws->count, 1) + kReachMax * ((size_t)ws->count + 1 + 32 * kReachCounters) + (size_t)kTRungs * ws->count;
    if (ws->tlong.bytes < sizeof(uint32_t) * words && (rc = ws->tlong.alloc(sizeof(uint32_t) * words))) return rc;
    if (ws->tu.bytes < sizeof(int32_t) * (size_t)std::max(ws->count, 1) &&
        (rc = ws->tu.alloc(sizeof(int32_t) * (size_t)std::max(ws->count, 1))))
        return rc;
    TransArgs A;
    A.desc = ws->desc.as<DagDesc>();
    A.count = ws->count;
    A.base = ws->base;
    A.items = ws->tasks;
    A.topo = dag->topo.as<int32_t>();
    A.lvl = dag->lvl.as<int32_t>();
    A.nlev = dag->nlev.as<int32_t>();
    A.rec = dag->rrec.as<uint4>();
    A.more = dag->rmore.as<uint4>();
    A.ptau = dag->ptau.as<int32_t>();
    A.est = est;
    A.clear_status = clear_status ? 1 : 0;
    A.unit_time = unit_time;
    A.ia = ia;
    A.ie = ie;
    A.cum = unit_time == 0 ? dag->tcum.as<int32_t>() : nullptr;
    A.longest = ws->tlong.as<unsigned int>();
    A.maxtau = A.longest + ws->count;
    A.pre = reinterpret_cast<int32_t *>(A.maxtau + ws->count);
    A.next = A.pre + (int64_t)kReachMax * (ws->count + 1);
    A.score = A.next + kReachMax * kReachCounters * 32;
    // a standalone call has status words of its own (it neither clears nor
    // reports a schedule's pending failures)
    A.stat = clear_status ? dag->dag_astat.as<int32_t>() : dag->dag_stat.as<int32_t>();
    hipLaunchKernelGGL(k_trans_clear, dim3((unsigned)((std::max<int64_t>(ws->count, kReachMax * kReachCounters) + 255) / 256)), dim3(256), 0, st, A);
    if (ws->tasks > 0) {
        hipLaunchKernelGGL(k_position_tau, dim3((unsigned)((ws->tasks + 255) / 256)), dim3(256), 0, st, A);
        int dev = 0, cus = 256;
        INSP_HIP(hipGetDevice(&dev));
        INSP_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        // sources by window: at most this many in a launch
        auto sources = [&](int32_t lo, int32_t hi) {
            int64_t c = 0;
            for (int32_t b = ws->first; b < ws->first + ws->count; b++) {
                const int64_t n = dag->toff[b + 1] - dag->toff[b];
                c += std::max<int64_t>(0, n - lo) - std::max<int64_t>(0, n - hi);
            }
            return c;
        };
        ReachList R;
        R.count = 0;
        int64_t src[kReachMax], groups[kReachMax];
        const struct {
            int form;
            int32_t lo, hi;
        } ranges[] = {{kCrew, kTeamMax, INSP_MAX_TRANSITIVE_TASKS}, {kTeam, kHalfMax, kTeamMax}, {kTeam, kSmallMax, kHalfMax},
                      {kHalf, kSmallMax, kHalfMax}, {kSmall, 0, kSmallMax}};
        for (const auto &g : ranges) {
            const int form = g.form;
            const int32_t least = g.lo;
            int32_t hi = std::min(maxn, g.hi);
            while (hi > least) {
                const int c = R.count++;
                groups[c] = cus * reach_groups(form, reach_entries(hi));
                // down to the next cap below which the launch is full
                int32_t lo = least;
                for (int k = kReachMax / 2 - 1; k >= 0; k--)
                    if (kCaps[k] < hi && kCaps[k] > least && sources(kCaps[k], hi) >= 4 * groups[c]) {
                        lo = kCaps[k];
                        break;
                    }
                R.form[c] = form;
                R.lo[c] = lo;
                R.hi[c] = hi;
                src[c] = sources(lo, hi);
                hi = lo;
            }
        }
        ProfScope ps(st, "trans");
        hipLaunchKernelGGL(k_reach_lists, dim3((unsigned)R.count), dim3(1024), 0, st, A, R);
        for (int c = 0; c < R.count; c++)
            if ((rc = R.form[c] == kSmall  ? launch_reach<false, 1>(A, c, R.hi[c], src[c], groups[c], st)
                      : R.form[c] == kHalf ? launch_reach<true, 1>(A, c, R.hi[c], src[c], groups[c], st)
                      : R.form[c] == kTeam ? launch_reach<false, 8>(A, c, R.hi[c], src[c], groups[c], st)
                                           : launch_reach<false, 16>(A, c, R.hi[c], src[c], groups[c], st)))
                return rc;
    }
    hipLaunchKernelGGL(k_trans_select, dim3((unsigned)std::max(ws->count, 1)), dim3(kTT), 0, st, A,
                       ws->tu.as<int32_t>());
    INSP_HIP(hipGetLastError());
    return INSP_OK;
}

}  // namespace insp

using namespace insp;

extern "C" int insp_transitive_attributes(const insp_dag *cdag, int32_t dag_index, const int32_t *est,
                                          const insp_workers *workers, int32_t unit_time, int32_t *ia, int32_t *ie,
                                          int32_t *unit_time_used, int64_t *longest_path, void *stream) {
    insp_dag *dag = const_cast<insp_dag *>(cdag);
    if (!dag || !workers || !unit_time_used) return set_error(INSP_E_INVAL, "null argument");
    if (unit_time < 0) return set_error(INSP_E_INVAL, "negative unit_time");
    if (dag_index != INSP_ALL_DAGS && (dag_index < 0 || dag_index >= dag->B))
        return set_error(INSP_E_INVAL, "dag index %d out of range", dag_index);
    const int32_t first = dag_index == INSP_ALL_DAGS ? 0 : dag_index;
    const int32_t count = dag_index == INSP_ALL_DAGS ? dag->B : 1;
    const int64_t n = dag->toff[first + count] - dag->toff[first];
    if (n > 0 && (!est || !ia || !ie)) return set_error(INSP_E_INVAL, "null est/ia/ie");
    hipStream_t st = (hipStream_t)stream;
    INSP_HIP(hipSetDevice(dag->device));
    int rc;
    if ((rc = ensure_state(dag, st))) return rc;
    Workspace *ws;
    if ((rc = get_workspace(dag, first, count, workers, true, &ws))) return rc;
    // computed into the handle's arrays and copied out once the call is known
    // to succeed, so that a failing call leaves ia and ie untouched
    const int64_t NN = std::max<int64_t>(dag->N, 1);
    if ((!dag->tia.p && (rc = dag->tia.alloc(sizeof(int32_t) * NN))) ||
        (!dag->tie.p && (rc = dag->tie.alloc(sizeof(int32_t) * NN))))
        return rc;
    int32_t *tia = dag->tia.as<int32_t>() + ws->base, *tie = dag->tie.as<int32_t>() + ws->base;
    if ((rc = run_transitive(dag, ws, est, unit_time, tia, tie, true, st))) return rc;
    std::vector<int32_t> stat(2 * dag->B);
    std::vector<uint32_t> lp(count);
    std::vector<int32_t> uu(count);
    INSP_HIP(hipMemcpyAsync(uu.data(), ws->tu.p, sizeof(int32_t) * count, hipMemcpyDeviceToHost, st));
    INSP_HIP(hipMemcpyAsync(lp.data(), ws->tlong.p, sizeof(uint32_t) * count, hipMemcpyDeviceToHost, st));
    INSP_HIP(hipMemcpyAsync(stat.data(), dag->dag_astat.p, sizeof(int32_t) * 2 * dag->B, hipMemcpyDeviceToHost, st));
    INSP_HIP(hipStreamSynchronize(st));
    for (int32_t i = first; i < first + count; i++) {
        if (stat[2 * i] & ST_EST) return set_error(INSP_E_RANGE, "estimate outside [1, 2^20] in DAG %d", i);
        if (stat[2 * i] & ST_PATH) return set_error(INSP_E_RANGE, "longest path of DAG %d reaches 2^30 ticks", i);
    }
    if (n > 0) {
        INSP_HIP(hipMemcpyAsync(ia, tia, sizeof(int32_t) * n, hipMemcpyDeviceToDevice, st));
        INSP_HIP(hipMemcpyAsync(ie, tie, sizeof(int32_t) * n, hipMemcpyDeviceToDevice, st));
        INSP_HIP(hipStreamSynchronize(st));
    }
    for (int32_t i = 0; i < count; i++) unit_time_used[i] = uu[i];
    if (longest_path)
        for (int32_t i = 0; i < count; i++) longest_path[i] = lp[i];
    return INSP_OK;
}
