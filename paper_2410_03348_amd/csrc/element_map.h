// One thread per (sample, element) of a [batch, n] space, consecutive lanes on consecutive elements of one row:
// a workgroup owns a chunk of whole rows and splits its flat element index into (row, column) with a float reciprocal,
// which is exact for such small indices.  A row wider than a chunk is cut into chunks of its own, one workgroup each, so
// that a small batch of wide rows still fills the chip.  A chunk has 2 048 elements where the space gives 512 workgroups or
// more of that size, fewer (down to one per thread) where it does not: a Filter of 64 rows of 14 symbols ran as one
// workgroup of eight elements per thread, 2-3 us against 1.8.
#pragma once

#include "internal.h"

#include <algorithm>

namespace dol {

constexpr int kThreads = 256;
constexpr int kChunk = 2048;            // most elements per workgroup (whole rows)
constexpr int kChunkGrid = 512;         // workgroups below which chunks get smaller

struct Rows {                           // how a [batch, n] element space is cut into workgroup chunks
    int32_t batch, n, rpb;
    int32_t chunk;                      // elements per workgroup
    int32_t cpr;                        // rpb == 1: chunks (workgroups) per row
    float inv_n;
    unsigned grid;
};

static inline Rows rows_of(int32_t batch, int32_t n)
{
    Rows r;
    r.batch = batch;
    r.n = n;
    const int64_t share = static_cast<int64_t>(batch) * n / kChunkGrid;
    r.chunk = static_cast<int32_t>(std::min<int64_t>(kChunk, std::max<int64_t>(kThreads, share / kThreads * kThreads)));
    r.rpb = n >= r.chunk ? 1 : r.chunk / n;
    r.cpr = r.rpb == 1 ? (n + r.chunk - 1) / r.chunk : 1;
    r.inv_n = 1.0f / static_cast<float>(n);
    r.grid = static_cast<unsigned>((static_cast<int64_t>(batch) + r.rpb - 1) / r.rpb * r.cpr);
    return r;
}

typedef float __attribute__((ext_vector_type(4), aligned(4))) f32x4_u;   // (global accesses may be unaligned)

// Calls f(sample, column) for every element of this workgroup's chunk.
template <typename F>
__device__ __forceinline__ void for_each_element(const Rows &R, F f)
{
    if (R.rpb == 1) {
        const int64_t s = blockIdx.x / static_cast<unsigned>(R.cpr);
        const int c0 = static_cast<int>(blockIdx.x - s * R.cpr) * R.chunk, c1 = min(R.n, c0 + R.chunk);
        for (int c = c0 + threadIdx.x; c < c1; c += kThreads) f(s, c);
        return;
    }
    const int64_t s0 = static_cast<int64_t>(blockIdx.x) * R.rpb;
    const int rows = static_cast<int>(min(static_cast<int64_t>(R.rpb), R.batch - s0));
    const int total = rows * R.n;
#pragma unroll 4
    for (int e = threadIdx.x; e < total; e += kThreads) {
        int r = static_cast<int>(static_cast<float>(e) * R.inv_n);
        int c = e - r * R.n;
        if (c < 0) { c += R.n; --r; } else if (c >= R.n) { c -= R.n; ++r; }
        f(s0 + r, c);
    }
}

// pre[c] = sum over the tuples of column c, ascending (i, j), one fma each.  This order is part of the
// operator's contract: the backward pass re-derives the clamp decision [pre <= 1] from it.
// The loads of kGather tuples are issued together (index words first, then the tags they name) so that a column
// costs a few memory round trips rather than two per tuple; the adds keep their order.
constexpr int kGather = 4;

__device__ __forceinline__ float column_sum(const float *__restrict__ ar, const float *__restrict__ br,
                                            const uint32_t *__restrict__ col_ij, uint32_t q0, uint32_t q1)
{
    float acc = 0.0f;
    for (uint32_t q = q0; q < q1; q += kGather) {
        uint32_t ij[kGather];
        float x[kGather], y[kGather];
#pragma unroll
        for (int u = 0; u < kGather; ++u) ij[u] = col_ij[min(q + u, q1 - 1)];
#pragma unroll
        for (int u = 0; u < kGather; ++u) {
            x[u] = ar[ij[u] & 0xffffu];
            y[u] = br[ij[u] >> 16];
        }
#pragma unroll
        for (int u = 0; u < kGather; ++u)
            if (q + u < q1) acc = __builtin_fmaf(x[u], y[u], acc);
    }
    return acc;
}

// Four neighbouring floats at a 4-byte aligned address, of which the first n exist.
__device__ __forceinline__ float4 load4(const float *__restrict__ p, int n)
{
    if (n >= 4) {
        const f32x4_u v = *reinterpret_cast<const f32x4_u *>(p);
        return make_float4(v.x, v.y, v.z, v.w);
    }
    return make_float4(p[0], n > 1 ? p[1] : 0.0f, n > 2 ? p[2] : 0.0f, 0.0f);
}

__device__ __forceinline__ void store4(float *__restrict__ p, const float (&v)[4], int n, uint32_t skip = 0)
{
    if (n >= 4 && skip == 0) {
        f32x4_u w;
        w.x = v[0], w.y = v[1], w.z = v[2], w.w = v[3];
        *reinterpret_cast<f32x4_u *>(p) = w;
        return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (k < n && !((skip >> k) & 1u)) p[k] = v[k];
}

}  // namespace dol
