// Selection of the smallest (key, index) pairs of a stream by one wave.
#pragma once
#include "internal.h"

namespace lnbnn {

// Orders a wave's LDS writes before its later reads by other lanes (a wave's
// LDS operations complete in order; this keeps the compiler from moving them).
static __device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A pair as one unsigned 64-bit number that orders like (key, index): the
// key's bits made monotonic (both zeros the same) above the index (>= 0).
static __device__ __forceinline__ uint64_t pair_of(float key, int index)
{
    const uint32_t b = __builtin_bit_cast(uint32_t, key + 0.0f);
    const uint32_t m = b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
    return (uint64_t)m << 32 | (uint32_t)index;
}
static __device__ __forceinline__ float pair_key(uint64_t p)
{
    const uint32_t m = (uint32_t)(p >> 32);
    return __builtin_bit_cast(float, m ^ ((uint32_t)((int32_t)~m >> 31) | 0x80000000u));
}
static __device__ __forceinline__ int pair_index(uint64_t p) { return (int)(uint32_t)p; }

// The `need` smallest pairs of a stream, 64 pairs (one per lane) at a time:
// pairs that may still be among them are appended to an LDS buffer; a full
// buffer is ranked and cut to `need`, which tightens the bound that later pairs
// must beat.  need + 64 <= CAP; the buffer holds CAP + 4 pairs.
template <int CAP>
struct WaveSelect {
    static_assert(CAP % 64 == 0, "whole waves of pairs");
    static constexpr int kSize = CAP + 4;
    uint64_t *buf;
    int need;
    int n;              // pairs held
    uint64_t bound;     // only pairs below it can be among the needed ones

    __device__ __forceinline__ WaveSelect(uint64_t *b, int need_, uint64_t bound_)
        : buf(b), need(need_), n(0), bound(bound_) {}

    // Ranks the first OWN * 64 pairs held (each lane OWN of them, against all):
    // two vector instructions and half a (broadcast) LDS read per pair and OWN.
    template <int OWN>
    __device__ __forceinline__ void rank_cut(int lane)
    {
        uint64_t own[OWN];
        int rank[OWN];
#pragma unroll
        for (int c = 0; c < OWN; ++c) {
            own[c] = buf[lane + 64 * c];
            rank[c] = 0;
        }
        for (int i = 0; i < n; i += 4) {
            uint64_t e[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) e[u] = buf[i + u];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int c = 0; c < OWN; ++c) rank[c] += e[u] < own[c] ? 1 : 0;
        }
        wave_lds_fence();
#pragma unroll
        for (int c = 0; c < OWN; ++c)
            if (lane + 64 * c < n && rank[c] < need) buf[rank[c]] = own[c];
        wave_lds_fence();
    }

    // keep the `need` first pairs, in order
    __device__ __forceinline__ void cut(int lane)
    {
        wave_lds_fence();
        if (lane < 4) buf[n + lane] = ~0ull;          // the last step's pairs past the end
        wave_lds_fence();
        if (n <= 64)
            rank_cut<1>(lane);
        else
            rank_cut<CAP / 64>(lane);
        if (n >= need) {
            n = need;
            bound = min(bound, buf[need - 1]);
        }
    }

    // false: no lane's pair passed the bound
    __device__ __forceinline__ bool add(uint64_t pair, bool ok, int lane)
    {
        bool pass = ok && pair < bound;
        unsigned long long m = __builtin_amdgcn_ballot_w64(pass);
        if (m == 0) return false;
        if (n + (int)__builtin_popcountll(m) > CAP) {
            cut(lane);
            pass = pass && pair < bound;
            m = __builtin_amdgcn_ballot_w64(pass);
        }
        const int at = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
        if (pass) buf[at] = pair;
        n += (int)__builtin_popcountll(m);
        return true;
    }
};

}  // namespace lnbnn
