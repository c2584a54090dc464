// Queue keys of the simulation: their layouts and orders.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace insp {

constexpr uint64_t M21 = (1ull << 21) - 1;
constexpr uint64_t BIT63 = 1ull << 63;

// Sort key of a queue entry under rule `ord`: 0 ability, 1 efficiency,
// 2 FIFO, 3 HEFT (whose entries hold rank << 21 | (2^21-1-seq) instead).
__host__ __device__ __forceinline__ uint64_t key_of(uint64_t k, int ord) {
    if (ord == 0 || ord == 3) return k | BIT63;
    if (ord == 1) return ((k >> 21) & M21) << 42 | (k >> 42 & M21) << 21 | (k & M21) | BIT63;
    return (k & M21) | BIT63;
}

// Bits of a key field that holds values up to `most`.
__host__ __device__ constexpr uint32_t field_bits(uint32_t most) { return most == 0 ? 1 : 32 - __builtin_clz(most); }

// Key layout of one DAG.
struct KeyFmt {
    uint32_t sa, sb;    // shifts of the second and first key fields (s, a + s)
    uint32_t smask;     // 2^s - 1
    uint32_t amask;     // 2^a - 1
    bool fifo;          // kA holds the FIFO key
    __host__ __device__ __forceinline__ uint32_t ka(uint32_t ia, uint32_t ie, uint32_t seq) const {
        return 0x80000000u | (fifo ? 0u : ia << sb | ie << sa) | (smask - seq);
    }
    __host__ __device__ __forceinline__ uint32_t ke(uint32_t ia, uint32_t ie, uint32_t seq) const {
        return 0x80000000u | ie << sb | ia << sa | (smask - seq);
    }
};

// Queue keys of the one-wave loop.
//   kNarrow  direct attributes, two 32-bit rule keys per entry (kA, kE), each
//            raised in place when the task's IE grows; block and worker maxima
//            hold key << 32 | slot.
//   kFixed   HEFT ranks or transitive attributes, fixed while queued: one
//            64-bit key per entry in the general loop's format under a valid
//            bit, from which key_of derives the rule keys when an entry is read
//            (zero stays zero: an empty slot).
//   kWide    direct attributes in that format, raised in place.
// With 64-bit keys the maxima hold rule keys alone: the second wave leaves
// the slot of a worker's best beside it, and the simulating wave keeps the
// best entry it pushed or raised since the worker's last pop, with its slot,
// in the worker's lane.
enum KeyKind { kNarrow = 0, kFixed = 1, kWide = 2 };

template <int KK>
struct Keys {
    static constexpr bool kBig = KK != kNarrow;
    using T = typename std::conditional<kBig, unsigned long long, uint32_t>::type;
    T *ka, *ke;  // LDS keys [64 * key_cap]: kA and kE, or ka the 64-bit key
    int o0;      // 64-bit keys: the rule of maximum 0 (0 ability, 2 FIFO, 3 rank)
    __host__ __device__ __forceinline__ T rule(uint64_t raw, int r) const {
        if constexpr (kBig) return raw ? key_of(raw, r ? 1 : o0) : 0ull;
        else return (uint32_t)(raw >> (r ? 32 : 0));
    }
    // 64-bit keys: the word of an entry with `top` (rank, or IA << 21 | IE) over
    // its push order, under a valid bit: the last of 2^21 tasks to be pushed has
    // no successors, so that without it all bits of its word would be zero
    __host__ __device__ __forceinline__ static uint64_t big(uint64_t top, uint32_t seq) {
        return BIT63 | top << 21 | (M21 - (uint64_t)seq);
    }
    // rule-r key of the entry in LDS slot p
    __host__ __device__ __forceinline__ T lds(int32_t p, int r) const {
        if constexpr (kBig) return rule(ka[p], r);
        else return (r ? ke : ka)[p];
    }
    // the entry's key word (the two 32-bit keys, kE above kA, or the 64-bit key)
    __host__ __device__ __forceinline__ uint64_t word(int32_t p) const {
        if constexpr (kBig) return ka[p];
        else return (uint64_t)ke[p] << 32 | ka[p];
    }
    __host__ __device__ __forceinline__ void put(int32_t p, uint64_t w) const {
        if constexpr (kBig) {
            ka[p] = w;
        } else {
            ka[p] = (uint32_t)w;
            ke[p] = (uint32_t)(w >> 32);
        }
    }
    // the key of a block or worker maximum
    __host__ __device__ __forceinline__ static T of_max(unsigned long long m) {
        if constexpr (kBig) return m;
        else return (uint32_t)(m >> 32);
    }
};

}  // namespace insp
