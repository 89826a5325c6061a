// Parallel CF splitting of the PMIS type (De Sterck, Yang and Heys, 2006):
// the device alternative to the sequential Ruge-Stueben first pass of
// Sec. 4.  Weight of point i: the number of points that strongly depend on
// it, then fmix32(i) (MurmurHash3's 32-bit finalizer), then i.  Points on
// which nothing strongly depends are F.  A round: every undecided point that
// beats every undecided point it is strongly connected to (either
// direction) becomes C, then every undecided point that strongly depends on
// a C-point becomes F.
//
// The rounds decide every point from the points of larger weight that it
// strongly depends on: a C-point has beaten every undecided point connected
// to it, so a point becomes F only through a C-point of larger weight, and a
// point whose larger neighbours are all decided, none of those it depends on
// C, becomes C.  Hence i is F if one of the larger points it depends on is C
// and C if all of them are F; that is what a thread asks here, again and
// again, of whatever states it finds.  States only ever go from undecided to
// decided and a decision needs no undecided point, so the result is that of
// the rounds whatever the order, without their three launches each and
// without the other direction's connections.
#include <hip/hip_runtime.h>

#include "k_common.hpp"
#include "lair_internal.hpp"

namespace lair {

constexpr int SPLIT_BS = 256;
constexpr int8_t ST_U = -1, ST_F = 0, ST_C = 1;

__device__ __forceinline__ uint32_t fmix32(uint32_t h) {
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h;
}

// cnt[i] += 1 for every strong entry (j, i), j != i
__global__ void __launch_bounds__(SPLIT_BS)
k_pmis_count(int32_t n, const int32_t *rp, const int32_t *cj, const uint8_t *smask,
             int32_t *cnt) {
    const int32_t j = blockIdx.x * SPLIT_BS + threadIdx.x;
    if (j >= n) return;
    for (int32_t p = rp[j]; p < rp[j + 1]; ++p)
        if (smask[p] && cj[p] != j) atomicAdd(&cnt[cj[p]], 1);
}

// weights and the first states
__global__ void __launch_bounds__(SPLIT_BS)
k_pmis_init(int32_t n, const int32_t *cnt, uint64_t *key, int8_t *state) {
    const int32_t i = blockIdx.x * SPLIT_BS + threadIdx.x;
    if (i >= n) return;
    key[i] = ((uint64_t)(uint32_t)cnt[i] << 32) | fmix32((uint32_t)i);
    state[i] = cnt[i] == 0 ? ST_F : ST_U;
}

// States move between the chip's L2s within a launch: device-scope accesses.
__device__ __forceinline__ int8_t state_of(const int8_t *state, int32_t i) {
    return __hip_atomic_load(state + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Each thread looks at its point up to PMIS_TRIES times (then a later launch
// does): an undecided larger point may be decided meanwhile by its own thread.
// The points left undecided are counted, one atomic per wavefront.  What
// bounds it is the chain of decisions, each a round trip through memory: 16 us
// a launch on average over the levels of 24 systems in one union, 21 launches,
// 0.34 ms; the rounds, three launches of up to 11 us each and eight of them
// before a readback, took 1.8 ms there.
constexpr int PMIS_TRIES = 12;

__global__ void __launch_bounds__(SPLIT_BS)
k_pmis_decide(int32_t n, const int32_t *rp, const int32_t *cj, const uint8_t *smask,
              const uint64_t *key, int8_t *state, int32_t *left) {
    const int32_t j = blockIdx.x * SPLIT_BS + threadIdx.x;
    bool und = j < n && state_of(state, j) == ST_U;
    if (und) {
        const int32_t lo = rp[j], hi = rp[j + 1];
        const uint64_t kj = key[j];
        int32_t p0 = lo;                   // entries before p0 cannot hold j up
        for (int t = 0; t < PMIS_TRIES && und; ++t) {
            bool wait = false, to_f = false;
            int32_t first = hi;
            for (int32_t p = p0; p < hi && !to_f; ++p) {
                const int32_t i = cj[p];
                if (!smask[p] || i == j) continue;
                const uint64_t ki = key[i];
                if (ki < kj || (ki == kj && i < j)) continue;
                const int8_t st = state_of(state, i);
                if (st == ST_C) to_f = true;
                else if (st == ST_U && !wait) {
                    wait = true;
                    first = p;
                }
            }
            p0 = first;
            if (to_f || !wait) {
                __hip_atomic_store(state + j, to_f ? ST_F : ST_C, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
                und = false;
            }
        }
    }
    const unsigned long long m = __ballot(und);
    if ((threadIdx.x & 63) == 0 && m != 0ull) atomicAdd(left, (int32_t)__popcll(m));
}

void launch_pmis_split(int32_t n, const int32_t *rp, const int32_t *cj, const uint8_t *smask,
                       int8_t *cf, hipStream_t s) {
    if (n == 0) return;
    const dim3 grid(blocks_for(n, SPLIT_BS)), blk(SPLIT_BS);
    DevArr<int32_t> cnt, left;
    DevArr<uint64_t> key;
    cnt.alloc((size_t)n, s);
    key.alloc((size_t)n, s);
    // one counter per launch of a group of launches
    constexpr int LAUNCHES = 3;
    left.alloc(LAUNCHES, s);
    LAIR_HIP(hipMemsetAsync(cnt.get(), 0, sizeof(int32_t) * n, s));
    LAIR_LAUNCH(k_pmis_count, grid, blk, 0, s, n, rp, cj, smask, cnt.get());
    LAIR_LAUNCH_CHECK();
    LAIR_LAUNCH(k_pmis_init, grid, blk, 0, s, n, cnt.get(), key.get(), cf);
    LAIR_LAUNCH_CHECK();
    // every launch decides at least the undecided point of largest weight, so
    // n launches always suffice; they go out in groups and the number of
    // undecided points is read after each group
    for (int64_t done = 0; done < n; done += LAUNCHES) {
        LAIR_HIP(hipMemsetAsync(left.get(), 0, sizeof(int32_t) * LAUNCHES, s));
        for (int r = 0; r < LAUNCHES; ++r) {
            LAIR_LAUNCH(k_pmis_decide, grid, blk, 0, s, n, rp, cj, smask, key.get(), cf,
                        left.get() + r);
            LAIR_LAUNCH_CHECK();
        }
        int32_t hl[LAUNCHES];
        Readback rb(s);
        rb.add(hl, left.get(), sizeof(hl));
        rb.run();
        if (hl[LAUNCHES - 1] == 0) return;
    }
    fail(LAIR_EDEVICE, "parallel splitting did not finish");
}

}  // namespace lair
