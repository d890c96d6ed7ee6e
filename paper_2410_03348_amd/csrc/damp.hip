// DAMP provenance kernels (Sec. 3.2, Table 1: conjunction t*t', disjunction min(1, t+t')) for gfx950:
// Apply with an arbitrary function table and its vector-Jacobian products, for what no other form takes (operand or result
// rows beyond LDS); the entry points of Apply, which try those forms first: sums of digits (damp_conv.hip), code generated
// for small tables (damp_table.hip), tiles of samples (damp_lds.hip), a workgroup per sample (damp_sample.hip).  Filter and
// Union are in damp_rows.hip.
//
// Thread mapping: one thread per (sample, output element), consecutive lanes on consecutive elements of one
// row, so that every store is coalesced and, for tables with regular structure (grids), lane-adjacent gathers
// touch adjacent addresses.  A workgroup owns a chunk of whole rows (about 2048 elements) and splits its
// flat element index into (row, column) with a float reciprocal, which is exact for such small indices.
#include "element_map.h"
#include "internal.h"
#include "wave_util.h"

namespace dol {

// ---------------------------------------------------------------- apply2 forward

// One thread per (sample, column).  The column's first four tuples come with one 16-byte load of col_head; only a
// column with more tuples goes on through its list (same order).
__global__ void __launch_bounds__(kThreads)
damp_apply2_fwd_kernel(Rows R, const uint32_t *__restrict__ col_ptr, const uint32_t *__restrict__ col_ij,
                       const uint4 *__restrict__ col_head, const float *__restrict__ a, int64_t lda,
                       const float *__restrict__ b, int64_t ldb, float *__restrict__ out, int64_t ldo)
{
    for_each_element(R, [&](int64_t s, int c) {
        const float *ar = a + s * lda, *br = b + s * ldb;
        const uint4 h = col_head[c];
        const uint32_t t[4] = {h.x, h.y, h.z, h.w};
        float x[4], y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool there = t[u] != 0xFFFFFFFFu;
            x[u] = there ? ar[t[u] & 0xffffu] : 0.0f;
            y[u] = there ? br[t[u] >> 16] : 0.0f;
        }
        float acc = 0.0f;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (t[u] != 0xFFFFFFFFu) acc = __builtin_fmaf(x[u], y[u], acc);
        if (t[3] != 0xFFFFFFFFu) {                                         // four or more tuples: the rest of the list
            const uint32_t q0 = col_ptr[c], q1 = col_ptr[c + 1];
            if (q1 - q0 > static_cast<uint32_t>(kLongTableCol)) return;    // left to the wavefront-per-column kernel
            for (uint32_t q = q0 + 4; q < q1; q += kGather) {
                uint32_t ij[kGather];
                float xs[kGather], ys[kGather];
#pragma unroll
                for (int u = 0; u < kGather; ++u) ij[u] = col_ij[min(q + u, q1 - 1)];
#pragma unroll
                for (int u = 0; u < kGather; ++u) {
                    xs[u] = ar[ij[u] & 0xffffu];
                    ys[u] = br[ij[u] >> 16];
                }
#pragma unroll
                for (int u = 0; u < kGather; ++u)
                    if (q + u < q1) acc = __builtin_fmaf(xs[u], ys[u], acc);
            }
        }
        out[s * ldo + c] = fminf(acc, 1.0f);
    });
}

// One workgroup of 1, 4 or 16 wavefronts (by the table's longest column) per (sample, long column).  The lanes stride
// over the column's tuples and their partial sums meet by shuffles and, between wavefronts, through LDS; this is not the order the clamp decision is defined in, so alongside the sum the lanes add up the
// terms' magnitudes, which bounds how far the two orders can lie apart (n roundings of relative size 2^-24 each
// way).  Only a sum within that distance of 1 is taken again in the defining order, by every lane alike.
__global__ void __launch_bounds__(1024)
damp_apply2_fwd_long_kernel(int32_t n_long, const uint32_t *__restrict__ long_cols,
                            const uint32_t *__restrict__ col_ptr, const uint32_t *__restrict__ col_ij,
                            const float *__restrict__ a, int64_t lda, const float *__restrict__ b, int64_t ldb,
                            float *__restrict__ out, int64_t ldo)
{
    const int64_t s = blockIdx.x / n_long;
    const uint32_t c = long_cols[blockIdx.x - s * n_long];
    const float *ar = a + s * lda, *br = b + s * ldb;
    const uint32_t q0 = col_ptr[c], q1 = col_ptr[c + 1];
    __shared__ float part[2][16];
    const uint32_t step = blockDim.x;
    float acc = 0.0f, mag = 0.0f;
    for (uint32_t q = q0 + threadIdx.x; q < q1; q += kGather * step) {
        uint32_t ij[kGather];
        float x[kGather], y[kGather];
#pragma unroll
        for (int u = 0; u < kGather; ++u) ij[u] = col_ij[min(q + u * step, q1 - 1)];
#pragma unroll
        for (int u = 0; u < kGather; ++u) {
            x[u] = ar[ij[u] & 0xffffu];
            y[u] = br[ij[u] >> 16];
        }
#pragma unroll
        for (int u = 0; u < kGather; ++u)
            if (q + u * step < q1) {
                acc = __builtin_fmaf(x[u], y[u], acc);
                mag = __builtin_fmaf(fabsf(x[u]), fabsf(y[u]), mag);
            }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        acc += __shfl_xor(acc, d, kWave);
        mag += __shfl_xor(mag, d, kWave);
    }
    if (step > kWave) {                             // uniform: the wavefronts' sums, added in wavefront order
        const int wave = threadIdx.x / kWave, n_waves = step / kWave;
        if ((threadIdx.x & (kWave - 1)) == 0) { part[0][wave] = acc; part[1][wave] = mag; }
        __syncthreads();
        if (wave != 0) return;
        acc = 0.0f, mag = 0.0f;
        for (int w = 0; w < n_waves; ++w) { acc += part[0][w]; mag += part[1][w]; }
    }
    const float slack = mag * (static_cast<float>(q1 - q0 + step) * 1.1920929e-7f);
    float pre = acc;
    if (fabsf(acc - 1.0f) <= slack) pre = column_sum(ar, br, col_ij, q0, q1);
    if (threadIdx.x == 0) out[s * ldo + c] = fminf(pre, 1.0f);
}

static dol_status launch_fwd_waves(const dol_fn_table *f, const DevArray<uint32_t> &cols, int32_t n_huge, int32_t batch,
                                   const float *a, int64_t lda, const float *b, int64_t ldb, float *out, int64_t ldo,
                                   hipStream_t st)
{
    const int64_t n_long = static_cast<int64_t>(cols.n);
    if (n_long == 0) return DOL_OK;
    if (batch * n_long > 0x7fffffffLL)
        return fail(DOL_EUNSUPPORTED, "batch x long table columns = %lld exceeds 2^31", static_cast<long long>(batch * n_long));
    if (n_huge > 0)                                  // the list's first n_huge columns: 16 wavefronts each
        hipLaunchKernelGGL(damp_apply2_fwd_long_kernel, dim3(static_cast<unsigned>(batch) * n_huge), dim3(1024), 0, st, n_huge,
                           cols.ptr, f->col_ptr.ptr, f->col_ij.ptr, a, lda, b, ldb, out, ldo);
    if (n_long > n_huge)
        hipLaunchKernelGGL(damp_apply2_fwd_long_kernel, dim3(static_cast<unsigned>(batch * (n_long - n_huge))), dim3(kWave), 0,
                           st, static_cast<int32_t>(n_long - n_huge), cols.ptr + n_huge, f->col_ptr.ptr, f->col_ij.ptr, a, lda,
                           b, ldb, out, ldo);
    DOL_HIP(hipGetLastError());
    return DOL_OK;
}

dol_status launch_damp_apply2_fwd(const dol_fn_table *f, int32_t batch, const float *a, int64_t lda, const float *b,
                                  int64_t ldb, float *out, int64_t ldo, hipStream_t st)
{
    if (batch == 0 || f->n_out == 0) return DOL_OK;
    {   // shape limits before anything is launched (a failing call leaves the outputs untouched)
        const int64_t most = static_cast<int64_t>(f->long_cols.n);
        if (batch * most > 0x7fffffffLL)
            return fail(DOL_EUNSUPPORTED, "batch x long table columns = %lld exceeds 2^31", static_cast<long long>(batch * most));
    }
    if (conv_path_ok(f)) return launch_damp_conv_fwd(f, batch, a, lda, b, ldb, out, ldo, st);
    bool done = false;
    if (dol_status s2 = launch_damp_table_fwd(f, batch, a, lda, b, ldb, out, ldo, st, &done)) return s2;
    if (done) return DOL_OK;
    if (dol_status s2 = launch_damp_lds_fwd(f, batch, a, lda, b, ldb, out, ldo, st, &done)) return s2;
    if (done) return DOL_OK;
    if (dol_status s2 = launch_sample_fwd(f, batch, a, lda, b, ldb, out, ldo, st, &done)) return s2;
    if (done) return DOL_OK;
    const Rows R = rows_of(batch, f->n_out);
    hipLaunchKernelGGL(damp_apply2_fwd_kernel, dim3(R.grid), dim3(kThreads), 0, st, R, f->col_ptr.ptr, f->col_ij.ptr,
                       reinterpret_cast<const uint4 *>(f->col_head.ptr), a, lda, b, ldb, out, ldo);
    DOL_HIP(hipGetLastError());
    return launch_fwd_waves(f, f->long_cols, f->n_huge_cols, batch, a, lda, b, ldb, out, ldo, st);
}

// ---------------------------------------------------------------- apply2 backward

// Gradient reaching the unclamped sum of column c.  out < 1 means the clamp did not act (pre = out);
// out == 1 leaves pre == 1 (passes) and pre > 1 (blocks) apart only by recomputing pre.
__device__ __forceinline__ float gated_grad(float g, float out_c, const float *__restrict__ ar,
                                            const float *__restrict__ br, const uint32_t *__restrict__ col_ptr,
                                            const uint32_t *__restrict__ col_ij, uint32_t c)
{
    if (out_c >= 1.0f) {
        const float pre = column_sum(ar, br, col_ij, col_ptr[c], col_ptr[c + 1]);
        if (!(pre <= 1.0f)) g = 0.0f;
    }
    return g;
}

// acc += sum over entries q0 + k * stride < q1 of gated gradient of the entry's column times the other operand's
// tag, in entry order; the loads of kGather entries are issued together.
__device__ __forceinline__ float row_sum(float acc, const uint32_t *__restrict__ ent, uint32_t q0, uint32_t q1,
                                         uint32_t stride, const float *__restrict__ gr, const float *__restrict__ outr,
                                         const float *__restrict__ other, const float *__restrict__ ar,
                                         const float *__restrict__ br, const uint32_t *__restrict__ col_ptr,
                                         const uint32_t *__restrict__ col_ij)
{
    for (uint32_t q = q0; q < q1; q += kGather * stride) {
        uint32_t e[kGather];
        float gv[kGather], ov[kGather], xv[kGather];
#pragma unroll
        for (int u = 0; u < kGather; ++u) e[u] = ent[min(q + u * stride, q1 - 1)];
#pragma unroll
        for (int u = 0; u < kGather; ++u) {
            gv[u] = gr[e[u] >> 16];
            ov[u] = outr[e[u] >> 16];
            xv[u] = other[e[u] & 0xffffu];
        }
#pragma unroll
        for (int u = 0; u < kGather; ++u)
            if (q + u * stride < q1)
                acc = __builtin_fmaf(gated_grad(gv[u], ov[u], ar, br, col_ptr, col_ij, e[u] >> 16), xv[u], acc);
    }
    return acc;
}

struct BwdTable {
    const uint32_t *col_ptr, *col_ij, *rowa_ptr, *rowa_jc, *rowb_ptr, *rowb_ic;
    int32_t na, nb;
};

// Element x of a sample is position x of a (x < na) or x - na of b.  Rows of the table with more than
// kLongTableRow tuples are left to damp_apply2_bwd_long_kernel.
__global__ void __launch_bounds__(kThreads)
damp_apply2_bwd_kernel(Rows R, BwdTable T, const float *__restrict__ a, int64_t lda, const float *__restrict__ b,
                       int64_t ldb, const float *__restrict__ out, int64_t ldo, const float *__restrict__ g,
                       int64_t ldg, float *__restrict__ ga, float *__restrict__ gb, int32_t accumulate)
{
    for_each_element(R, [&](int64_t s, int x) {
        const float *ar = a + s * lda, *br = b + s * ldb, *outr = out + s * ldo, *gr = g + s * ldg;
        const bool is_a = x < T.na;
        if (is_a ? !ga : !gb) return;
        const int r = is_a ? x : x - T.na;
        const uint32_t *ptr = is_a ? T.rowa_ptr : T.rowb_ptr;
        const uint32_t *ent = is_a ? T.rowa_jc : T.rowb_ic;
        const float *other = is_a ? br : ar;
        const uint32_t q0 = ptr[r], q1 = ptr[r + 1];
        if (q1 - q0 > kLongTableRow) return;
        const float acc = row_sum(0.0f, ent, q0, q1, 1, gr, outr, other, ar, br, T.col_ptr, T.col_ij);
        float *dst = is_a ? ga + s * lda + r : gb + s * ldb + r;
        const bool add = is_a ? (accumulate & 1) : (accumulate & 2);
        *dst = add ? *dst + acc : acc;
    });
}

// One wavefront per (sample, long row): lanes stride over the row's tuples, the partial sums meet by shuffles.
__global__ void __launch_bounds__(kWave)
damp_apply2_bwd_long_kernel(int32_t n_long, const uint32_t *__restrict__ long_rows, BwdTable T,
                            const float *__restrict__ a, int64_t lda, const float *__restrict__ b, int64_t ldb,
                            const float *__restrict__ out, int64_t ldo, const float *__restrict__ g, int64_t ldg,
                            float *__restrict__ ga, float *__restrict__ gb, int32_t accumulate)
{
    const int64_t s = blockIdx.x / n_long;
    const int x = static_cast<int>(long_rows[blockIdx.x - s * n_long]);
    const float *ar = a + s * lda, *br = b + s * ldb, *outr = out + s * ldo, *gr = g + s * ldg;
    const bool is_a = x < T.na;
    if (is_a ? !ga : !gb) return;
    const int r = is_a ? x : x - T.na;
    const uint32_t *ptr = is_a ? T.rowa_ptr : T.rowb_ptr;
    const uint32_t *ent = is_a ? T.rowa_jc : T.rowb_ic;
    const float *other = is_a ? br : ar;
    float acc = row_sum(0.0f, ent, ptr[r] + threadIdx.x, ptr[r + 1], kWave, gr, outr, other, ar, br, T.col_ptr, T.col_ij);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, kWave);
    if (threadIdx.x == 0) {
        float *dst = is_a ? ga + s * lda + r : gb + s * ldb + r;
        const bool add = is_a ? (accumulate & 1) : (accumulate & 2);
        *dst = add ? *dst + acc : acc;
    }
}

dol_status launch_damp_apply2_bwd(const dol_fn_table *f, int32_t batch, const float *a, int64_t lda, const float *b,
                                  int64_t ldb, const float *out, int64_t ldo, const float *g, int64_t ldg, float *ga,
                                  float *gb, int32_t accumulate, hipStream_t st)
{
    if (batch == 0 || f->na + f->nb == 0 || (!ga && !gb)) return DOL_OK;
    if (batch * static_cast<int64_t>(f->long_rows.n) > 0x7fffffffLL)      // before anything is launched
        return fail(DOL_EUNSUPPORTED, "batch x long table rows = %lld exceeds 2^31",
                    static_cast<long long>(batch * static_cast<int64_t>(f->long_rows.n)));
    if (conv_path_ok(f)) return launch_damp_conv_bwd(f, batch, a, lda, b, ldb, g, ldg, ga, gb, accumulate, st);
    bool done = false;
    if (dol_status s2 = launch_damp_table_bwd(f, batch, a, lda, b, ldb, g, ldg, ga, gb, accumulate, st, &done)) return s2;
    if (done) return DOL_OK;
    if (dol_status s2 = launch_damp_lds_bwd(f, batch, a, lda, b, ldb, out, ldo, g, ldg, ga, gb, accumulate, st, &done)) return s2;
    if (done) return DOL_OK;
    if (dol_status s2 = launch_sample_bwd(f, batch, a, lda, b, ldb, out, ldo, g, ldg, ga, gb, accumulate, st, &done)) return s2;
    if (done) return DOL_OK;
    const BwdTable T{f->col_ptr.ptr, f->col_ij.ptr, f->rowa_ptr.ptr, f->rowa_jc.ptr, f->rowb_ptr.ptr, f->rowb_ic.ptr,
                     f->na, f->nb};
    const Rows R = rows_of(batch, f->na + f->nb);
    hipLaunchKernelGGL(damp_apply2_bwd_kernel, dim3(R.grid), dim3(kThreads), 0, st, R, T, a, lda, b, ldb, out, ldo, g, ldg, ga, gb,
                       accumulate);
    DOL_HIP(hipGetLastError());
    const int64_t n_long = static_cast<int64_t>(f->long_rows.n);
    if (n_long > 0) {
        if (batch * n_long > 0x7fffffffLL)
            return fail(DOL_EUNSUPPORTED, "batch x long table rows = %lld exceeds 2^31", static_cast<long long>(batch * n_long));
        hipLaunchKernelGGL(damp_apply2_bwd_long_kernel, dim3(static_cast<unsigned>(batch * n_long)), dim3(kWave), 0, st,
                           static_cast<int32_t>(n_long), f->long_rows.ptr, T, a, lda, b, ldb, out, ldo, g, ldg, ga, gb,
                           accumulate);
        DOL_HIP(hipGetLastError());
    }
    return DOL_OK;
}

// ---------------------------------------------------------------- filter

// x[s, 0..n) = 0 (a fill kernel rather than a memset node, so that callers may capture the stream)
__global__ void __launch_bounds__(kThreads)
zero_rows_kernel(Rows R, float *__restrict__ x, int64_t ld)
{
    for_each_element(R, [&](int64_t s, int c) { x[s * ld + c] = 0.0f; });
}

dol_status launch_zero_rows(int32_t batch, int32_t n, float *x, int64_t ld, hipStream_t st)
{
    if (batch == 0 || n == 0) return DOL_OK;
    const Rows R = rows_of(batch, n);
    hipLaunchKernelGGL(zero_rows_kernel, dim3(R.grid), dim3(kThreads), 0, st, R, x, ld);
    DOL_HIP(hipGetLastError());
    return DOL_OK;
}

// ---------------------------------------------------------------- harness helper: gradient of -log p[target]

__global__ void __launch_bounds__(kThreads)
nll_grad_kernel(Rows R, const float *__restrict__ p, int64_t ld, const int32_t *__restrict__ target,
                float *__restrict__ grad)
{
    for_each_element(R, [&](int64_t s, int c) {
        grad[s * ld + c] = c == target[s] ? -1.0f / fmaxf(p[s * ld + c], 1.17549435e-38f) : 0.0f;
    });
}

// The same for wide rows, any row stride: a workgroup owns kThreads * kNllWide neighbouring columns of one row, whose
// target and value are the same for all its threads (23 410 columns at B=256: 42 us with whole rows to a workgroup).
constexpr int kNllWide = 8;

__global__ void __launch_bounds__(kThreads)
nll_grad_wide_kernel(int32_t n, int32_t cpr, const float *__restrict__ p, int64_t ld, const int32_t *__restrict__ target,
                     float *__restrict__ grad)
{
    const int64_t s = blockIdx.x / static_cast<unsigned>(cpr);
    const int32_t c0 = static_cast<int32_t>(blockIdx.x - s * cpr) * (kThreads * kNllWide);
    const int32_t t = target[s];
    const float val = t >= 0 && t < n ? -1.0f / fmaxf(p[s * ld + t], 1.17549435e-38f) : 0.0f;
    float *gr = grad + s * ld;
#pragma unroll
    for (int x = 0; x < kNllWide / 4; ++x) {
        const int32_t c = c0 + 4 * (static_cast<int32_t>(threadIdx.x) + x * kThreads);
        f32x4_u v;
        v.x = c == t ? val : 0.0f, v.y = c + 1 == t ? val : 0.0f, v.z = c + 2 == t ? val : 0.0f, v.w = c + 3 == t ? val : 0.0f;
        if (c + 3 < n) *reinterpret_cast<f32x4_u *>(gr + c) = v;
        else
            for (int k = 0; c + k < n; ++k) gr[c + k] = c + k == t ? val : 0.0f;
    }
}

// The same over a contiguous [batch, n] gradient, 16 bytes per store: a workgroup owns `rows` whole rows (a multiple of
// four, so its piece starts on a 16-byte boundary; at most kNllRows), first puts every row's target and value in LDS
// and then walks its piece without a division and without a load between the stores (a load's wait would also wait for
// the stores before it).
constexpr int kNllRows = 2048;

__global__ void __launch_bounds__(kThreads)
nll_grad_flat_kernel(int32_t batch, int32_t n, int32_t rows, const float *__restrict__ p, const int32_t *__restrict__ target,
                     float *__restrict__ grad)
{
    __shared__ int32_t tg[kNllRows];
    __shared__ float val[kNllRows];
    const int64_t s0 = static_cast<int64_t>(blockIdx.x) * rows;
    const int32_t rows_here = static_cast<int32_t>(min(static_cast<int64_t>(rows), batch - s0));
    const int32_t n_here = rows_here * n;           // floats of this piece
    const float *pp = p + s0 * n;
    float *gg = grad + s0 * n;
    for (int r = threadIdx.x; r < rows_here; r += kThreads) {
        const int32_t t = target[s0 + r];
        tg[r] = t;
        val[r] = t >= 0 && t < n ? -1.0f / fmaxf(pp[static_cast<int64_t>(r) * n + t], 1.17549435e-38f) : 0.0f;
    }
    __syncthreads();
    constexpr int kStep = 4 * kThreads;
    const int32_t dr = kStep / n, dc = kStep - dr * n;
    int32_t e = 4 * static_cast<int32_t>(threadIdx.x);
    int32_t r = e / n, c = e - r * n;
    for (; e < n_here; e += kStep) {
        int32_t rr = r, cc = c;
        float v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            while (cc >= n) { cc -= n; ++rr; }      // (once at most per element, n >= 1)
            v[k] = e + k < n_here && cc == tg[rr] ? val[rr] : 0.0f;
            ++cc;
        }
        if (e + 3 < n_here) *reinterpret_cast<float4 *>(gg + e) = make_float4(v[0], v[1], v[2], v[3]);
        else
            for (int k = 0; e + k < n_here; ++k) gg[e + k] = v[k];
        r += dr; c += dc;
        if (c >= n) { c -= n; ++r; }
    }
}

dol_status launch_nll_grad(int32_t batch, int32_t n, const float *p, int64_t ld, const int32_t *target, float *grad,
                           hipStream_t st)
{
    if (batch == 0 || n == 0) return DOL_OK;
    if (n >= kThreads * kNllWide / 2) {             // at least half a workgroup's columns
        const int32_t cpr = (n + kThreads * kNllWide - 1) / (kThreads * kNllWide);
        if (static_cast<int64_t>(batch) * cpr <= 0x7fffffffLL) {
            hipLaunchKernelGGL(nll_grad_wide_kernel, dim3(static_cast<unsigned>(batch) * cpr), dim3(kThreads), 0, st, n, cpr, p, ld, target, grad);
            DOL_HIP(hipGetLastError());
            return DOL_OK;
        }
    }
    if (ld == n && reinterpret_cast<uintptr_t>(grad) % 16 == 0) {
        const int32_t rows = std::min(kNllRows, std::max(4, (8192 / n + 3) / 4 * 4));
        if (static_cast<int64_t>(rows) * n < (int64_t{1} << 30)) {
            const unsigned grid = static_cast<unsigned>((static_cast<int64_t>(batch) + rows - 1) / rows);
            hipLaunchKernelGGL(nll_grad_flat_kernel, dim3(grid), dim3(kThreads), 0, st, batch, n, rows, p, target, grad);
            DOL_HIP(hipGetLastError());
            return DOL_OK;
        }
    }
    const Rows R = rows_of(batch, n);
    hipLaunchKernelGGL(nll_grad_kernel, dim3(R.grid), dim3(kThreads), 0, st, R, p, ld, target, grad);
    DOL_HIP(hipGetLastError());
    return DOL_OK;
}

}  // namespace dol
