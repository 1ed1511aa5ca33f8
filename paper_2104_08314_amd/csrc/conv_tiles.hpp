// What the matrix-core convolutions share: exact division, range-checked loads, tile numbering, windows.
#pragma once

#include "common.hpp"

#include <algorithm>

namespace cpoconv {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kXcds = 8;               // accelerator dies, each with an L2 of its own

// Exact division of 0 <= x < 2^31 by a divisor the host knows: multiply and shift.
struct Divisor {
    uint32_t m, s;
};
__device__ __forceinline__ int quotient(int x, const Divisor &d)
{
    return static_cast<int>(__umulhi(static_cast<uint32_t>(x) << 1, d.m) >> d.s);
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kLanes - 1); }
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint3v __attribute__((ext_vector_type(3)));
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));

// Loads through a buffer descriptor: a 32-bit offset per lane and one per wavefront, no address
// arithmetic in the vector ALU, and an offset past the end reads zero.
template <bool kFar>
struct Buffer {
    typedef uint32_t Offset;
    static constexpr Offset kNothing = ~Offset{0};   // past the end of every buffer
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ Buffer(const void *p, int64_t bytes)
    {
        const int64_t limit = 0xFFFFFFF0ll;
        rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, static_cast<uint32_t>(bytes < limit ? bytes : limit), 0x00027000);
    }
    __device__ __forceinline__ float load1(Offset lane_offset, Offset offset) const
    {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, lane_offset, offset, 0));
    }
    __device__ __forceinline__ uint4v load4(Offset lane_offset, Offset offset) const
    {
        return __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_offset, offset, 0);
    }
    __device__ __forceinline__ uint3v load3(Offset lane_offset, Offset offset) const
    {
        return __builtin_amdgcn_raw_buffer_load_b96(rsrc, lane_offset, offset, 0);
    }
    template <int N> __device__ __forceinline__ void load(float *f, Offset lane_offset, Offset offset) const
    {
        if constexpr (N == 1) {
            f[0] = load1(lane_offset, offset);
        } else if constexpr (N == 2) {
            const uint2v v = __builtin_amdgcn_raw_buffer_load_b64(rsrc, lane_offset, offset, 0);
#pragma unroll
            for (int i = 0; i < N; ++i) f[i] = __uint_as_float(v[i]);
        } else {
#pragma unroll
            for (int i0 = 0; i0 < N; i0 += 4) {
                const uint4v v = load4(lane_offset + 4 * i0, offset);
#pragma unroll
                for (int i = 0; i < 4; ++i) f[i0 + i] = __uint_as_float(v[i]);
            }
        }
    }
};

// The same for arrays that 32-bit offsets do not reach: 64-bit addresses, the range checked here.
template <>
struct Buffer<true> {
    typedef uint64_t Offset;
    static constexpr Offset kNothing = ~Offset{0};
    const char *base;
    uint64_t bytes;
    __device__ __forceinline__ Buffer(const void *p, int64_t n) : base(static_cast<const char *>(p)), bytes(n < 0 ? 0 : n) {}
    __device__ __forceinline__ float load1(Offset lane_offset, Offset offset) const
    {
        const bool inside = lane_offset < bytes && lane_offset + offset + 4 <= bytes;
        return inside ? *reinterpret_cast<const float *>(base + lane_offset + offset) : 0.0f;
    }
    __device__ __forceinline__ uint4v load4(Offset lane_offset, Offset offset) const
    {
        uint4v v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = __float_as_uint(load1(lane_offset, offset + 4 * i));
        return v;
    }
    __device__ __forceinline__ uint3v load3(Offset lane_offset, Offset offset) const
    {
        uint3v v;
#pragma unroll
        for (int i = 0; i < 3; ++i) v[i] = __float_as_uint(load1(lane_offset, offset + 4 * i));
        return v;
    }
    template <int N> __device__ __forceinline__ void load(float *f, Offset lane_offset, Offset offset) const
    {
#pragma unroll
        for (int i = 0; i < N; ++i) f[i] = load1(lane_offset, offset + 4 * i);
    }
};

// Tile of the i-th of `total` workgroups.  Workgroups go to the XCDs in turn: the tile numbers (kernel block
// outermost) are dealt so that an XCD holds a contiguous range of them - its L2 then fetches one stretch of
// the map and, with eight kernel blocks or more, its share of the weights only.
__device__ __forceinline__ int dealt(int i, int total)
{
    const int xcd = i % kXcds;
    return xcd * (total / kXcds) + min(xcd, total % kXcds) + i / kXcds;
}

constexpr int kComputeUnits = 256;
constexpr int kLdsLimit = 160 * 1024;

// window rows behind nb positions of strips sw wide, over all tiles
inline int window_rows(const Geometry &g, int nb, int sw)
{
    const int out_rows = std::min(nb % sw == 0 ? nb / sw : (nb - 2) / sw + 2, g.N * g.Oh);   // tiles start at multiples of nb
    int rows = (out_rows - 1) * g.stride + g.kh;
    // a tile that runs into the next image also spans the rows between the images' windows
    const bool may_cross = g.N > 1 && (static_cast<int64_t>(g.Oh) * sw) % nb != 0;
    if (may_cross) rows += ((out_rows + g.Oh - 2) / g.Oh) * std::max(0, g.Ih - g.Oh * g.stride);
    return rows;
}

inline Divisor divisor(int d)
{
    Divisor r;
    r.s = 0;
    while ((1ll << r.s) < d) ++r.s;
    r.m = static_cast<uint32_t>(((1ull << (31 + r.s)) + d - 1) / d);
    return r;
}

}  // namespace cpoconv
