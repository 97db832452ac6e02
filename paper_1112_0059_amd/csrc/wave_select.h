// Selection of the smallest (key, index) pairs of a stream by one wave.
#pragma once
#include "internal.h"

namespace lnbnn {

static __device__ __forceinline__ bool pair_less(float d0, int i0, float d1, int i1)
{
    return d0 < d1 || (d0 == d1 && i0 < i1);
}

// Orders a wave's LDS writes before its later reads by other lanes (a wave's
// LDS operations complete in order; this keeps the compiler from moving them).
static __device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The `need` smallest (key, pos) pairs of a stream, 64 pairs (one per lane) at
// a time: pairs that may still be among them are appended to an LDS buffer;
// a full buffer is sorted and cut to `need`, which tightens the bound that
// later pairs must beat.  need + 64 <= CAP.
template <int CAP>
struct WaveSelect {
    static constexpr int kOwn = CAP / 64;
    uint2 *buf;
    int need;
    int n;              // pairs held
    float bk;           // only pairs before (bk, bp) can be among the needed ones
    int bp;

    __device__ __forceinline__ WaveSelect(uint2 *b, int need_, float bk_) : buf(b), need(need_), n(0), bk(bk_), bp(0x7fffffff) {}

    // rank every held pair, keep the `need` first, in order
    __device__ __forceinline__ void cut(int lane)
    {
        wave_lds_fence();
        float k[kOwn];
        int p[kOwn], rank[kOwn];
#pragma unroll
        for (int c = 0; c < kOwn; ++c) {
            const uint2 e = buf[min(lane + 64 * c, CAP - 1)];
            k[c] = __builtin_bit_cast(float, e.x);
            p[c] = (int)e.y;
            rank[c] = 0;
        }
        for (int i = 0; i < n; ++i) {
            const uint2 e = buf[i];
            const float ek = __builtin_bit_cast(float, e.x);
#pragma unroll
            for (int c = 0; c < kOwn; ++c) rank[c] += pair_less(ek, (int)e.y, k[c], p[c]) ? 1 : 0;
        }
        wave_lds_fence();
#pragma unroll
        for (int c = 0; c < kOwn; ++c)
            if (lane + 64 * c < n && rank[c] < need) buf[rank[c]] = make_uint2(__builtin_bit_cast(uint32_t, k[c]), (uint32_t)p[c]);
        wave_lds_fence();
        if (n >= need) {
            n = need;
            const uint2 e = buf[need - 1];
            bk = __builtin_bit_cast(float, e.x);
            bp = (int)e.y;
        }
    }

    // false: no lane's pair passed the bound
    __device__ __forceinline__ bool add(float key, int pos, bool ok, int lane)
    {
        bool pass = ok && pair_less(key, pos, bk, bp);
        unsigned long long m = __builtin_amdgcn_ballot_w64(pass);
        if (m == 0) return false;
        if (n + (int)__builtin_popcountll(m) > CAP) {
            cut(lane);
            pass = pass && pair_less(key, pos, bk, bp);
            m = __builtin_amdgcn_ballot_w64(pass);
        }
        const int at = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
        if (pass) buf[at] = make_uint2(__builtin_bit_cast(uint32_t, key), (uint32_t)pos);
        n += (int)__builtin_popcountll(m);
        return true;
    }
};

}  // namespace lnbnn
