// planes.h -- bit-sliced reach counters of a workgroup slot, shared by the LDS-claim and the
// forest kernel: plane p of slot s holds bit p of the number of the slot's samples that reached
// each vertex (by reach id).
#pragma once

#include "imin_internal.h"

namespace imin {
namespace planes {

// Add the set bits of bm[0..n) into the words of the slot's bit-sliced counters from w0 on.
template <int B>
__device__ __forceinline__ void plane_add(uint32_t *planes, int64_t words, int64_t w0,
                                          const uint32_t *bm, int n)
{
    for (int w = threadIdx.x; w < n; w += 4 * B) {
        uint32_t x[4], o[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            x[u] = w + u * B < n ? bm[w + u * B] : 0u;
            o[u] = x[u] ? planes[w0 + w + u * B] : 0u;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (!x[u]) continue;
            uint32_t *at = planes + w0 + w + u * B;
            *at = o[u] ^ x[u];
            uint32_t carry = o[u] & x[u];
            for (int p = 1; p < kTreePlanes && carry; ++p) {
                at += words;
                const uint32_t v = *at;
                *at = v ^ carry;
                carry &= v;
            }
        }
    }
}

// The slot's counters into D (by reach id) with atomics, and back to zero: a slot that has
// counted as many samples as its planes hold.
template <int B>
__device__ __forceinline__ void planes_drain(uint32_t *planes, int64_t words, unsigned long long *D)
{
    for (int64_t w = threadIdx.x; w < words; w += B) {
        uint32_t p[kTreePlanes], any = 0;
#pragma unroll
        for (int i = 0; i < kTreePlanes; ++i) {
            p[i] = planes[i * words + w];
            any |= p[i];
        }
        if (!any) continue;
#pragma unroll
        for (int i = 0; i < kTreePlanes; ++i) planes[i * words + w] = 0u;
        while (any) {
            const int b = __builtin_ctz(any);
            any &= any - 1;
            uint32_t v = 0;
#pragma unroll
            for (int i = 0; i < kTreePlanes; ++i) v |= ((p[i] >> b) & 1u) << i;
            atomicAdd(&D[w * 32 + b], (unsigned long long)v);
        }
    }
}

}  // namespace planes
}  // namespace imin
