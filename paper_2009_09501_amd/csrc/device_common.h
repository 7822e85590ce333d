// Device helpers shared by the gfx950 kernels of the pseudo-stereo pipeline.
#pragma once

#include <hip/hip_runtime.h>

#include "pstereo_internal.h"

namespace pstereo {

// Range weights of the cross-bilateral filter: round(255 exp(-d^2 / (2 * 12^2)))
// for a luma difference d = 0..42, zero for larger d (range sigma 12).
__host__ __device__ constexpr uint32_t range_w(int d) {
    constexpr uint16_t t[43] = {255, 254, 251, 247, 241, 234, 225, 215, 204, 192, 180, 168, 155, 142, 129,
                                117, 105, 93,  83,  73,  64,  55,  47,  41,  35,  29,  24,  20,  17,  14,
                                11,  9,   7,   6,   5,   4,   3,   2,   2,   1,   1,   1,   1};
    return d < 43 ? t[d] : 0u;
}

// Spatial weights round(255 exp(-k / (2 * 1.5^2))) by squared distance k.
__host__ __device__ constexpr uint32_t spatial_w(int k) {
    return k == 0 ? 255 : k == 1 ? 204 : k == 2 ? 164 : k == 3 ? 131 : k == 4 ? 105
         : k == 5 ? 84 : k == 6 ? 67 : k == 7 ? 54 : k == 8 ? 43 : k == 9 ? 35
         : k == 10 ? 28 : k == 11 ? 22 : k == 12 ? 18 : k == 13 ? 14 : k == 14 ? 11
         : k == 15 ? 9 : k == 16 ? 7 : k == 17 ? 6 : 5;
}

// Luma guide: Q8 BT.601 weights summing to 256, rounded half up.
__device__ __forceinline__ int luma(int r, int g, int b) {
    return (77 * r + 150 * g + 29 * b + 128) >> 8;
}

// Exact floor(num / den) for num < 2^31, 0 < den < 2^22 and a quotient below
// 2^8: a single-precision reciprocal estimate is within 1 of the quotient,
// and one integer correction step makes it exact.  (The estimate and den fit
// 24 bits, whose product is a quarter of the cost of the 32-bit one.)
__device__ __forceinline__ uint32_t div_small_quotient(uint32_t num, uint32_t den) {
    const float qf = (float)num * __builtin_amdgcn_rcpf((float)den);
    int q = (int)qf;
    const int rem = (int)num - (int)__umul24((unsigned)q, den);
    if (rem < 0) --q;
    else if (rem >= (int)den) ++q;
    return (uint32_t)q;
}

// Row ramp of the region depth: 0 (far) at block row 0, 255 (near) at the
// bottom block row, rounded half up (quotient <= 255, so the reciprocal
// division above is exact).
__device__ __forceinline__ int ramp(int row, int gh) {
    return gh > 1 ? (int)div_small_quotient((uint32_t)(255 * row + (gh - 1) / 2), (uint32_t)(gh - 1)) : 0;
}

__device__ __forceinline__ int iabs(int v) { return v < 0 ? -v : v; }

// Loads and stores of dwords at any byte address: the hardware takes
// unaligned global accesses, and the compiler forms one instruction for each.
struct __attribute__((packed)) Bytes12 { uint32_t x, y, z; };

__device__ __forceinline__ uint3 load_96(const uint8_t* p) {
    Bytes12 v;
    __builtin_memcpy(&v, p, 12);
    return make_uint3(v.x, v.y, v.z);
}
__device__ __forceinline__ void store_96(uint8_t* p, uint3 q) {
    const Bytes12 v = {q.x, q.y, q.z};
    __builtin_memcpy(p, &v, 12);
}
__device__ __forceinline__ uint32_t load_32(const uint8_t* p) {
    uint32_t v;
    __builtin_memcpy(&v, p, 4);
    return v;
}
__device__ __forceinline__ void store_32(uint8_t* p, uint32_t v) { __builtin_memcpy(p, &v, 4); }

// The n (1..4) pixels of a quad starting at p as three dwords of RGB24 bytes,
// zero past the n-th pixel.  ALIGNED: a whole quad at a 4-byte aligned
// address; otherwise a whole quad is one load too, and the quad a row of
// another width ends with (n < 4) is read bytewise.
template <bool ALIGNED>
__device__ __forceinline__ uint3 load_quad_words(const uint8_t* p, int n) {
    if constexpr (ALIGNED) {
        return *reinterpret_cast<const uint3*>(p);
    } else {
        if (n >= 4) return load_96(p);
        uint32_t w[3] = {0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < 9; ++i)
            if (i < 3 * n) w[i >> 2] |= (uint32_t)p[i] << (8 * (i & 3));
        return make_uint3(w[0], w[1], w[2]);
    }
}

// The n (1..4) bytes at p, zero past the n-th; the same rule.
template <bool ALIGNED>
__device__ __forceinline__ uint32_t load_quad_bytes(const uint8_t* p, int n) {
    if constexpr (ALIGNED) {
        return *reinterpret_cast<const uint32_t*>(p);
    } else {
        if (n >= 4) return load_32(p);
        uint32_t w = 0;
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (i < n) w |= (uint32_t)p[i] << (8 * i);
        return w;
    }
}

// The low n (1..4) bytes of v to p; the same rule.
template <bool ALIGNED>
__device__ __forceinline__ void store_quad_bytes(uint8_t* p, uint32_t v, int n) {
    if constexpr (ALIGNED) {
        *reinterpret_cast<uint32_t*>(p) = v;
    } else {
        if (n >= 4) {
            store_32(p, v);
            return;
        }
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (i < n) p[i] = (uint8_t)(v >> (8 * i));
    }
}

// Second word of a block's table entry: its region depth with this flag, or
// (without it) the slot its component has in the merge's table.
constexpr uint32_t kResolved = 1u << 31;

// Lanes of the wave below this one whose bit is set in m.
__device__ __forceinline__ uint32_t lanes_below(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

constexpr size_t kMaxLds = 160 * 1024;

// The value of v, opaque to the optimiser: indices derived from it are
// recomputed where they are used (or in each loop iteration) instead of being
// held in registers across the whole kernel.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Workgroups are dispatched to the 8 XCDs round-robin by linear workgroup id.
// Tile for workgroup bid of n: each XCD gets one contiguous run of tiles in
// raster order, so neighbouring tiles -- sharing halo rows and the 128-byte
// lines across tile borders -- meet in the same L2.  A bijection on [0, n).
__device__ __forceinline__ int xcd_tile(int bid, int n) {
    constexpr int X = 8;
    const int q = n / X, r = n - q * X;
    const int xcd = bid % X, idx = bid / X;
    return xcd * q + min(xcd, r) + idx;
}

}  // namespace pstereo
