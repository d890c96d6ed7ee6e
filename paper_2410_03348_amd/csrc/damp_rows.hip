// DAMP Filter and Union (Sec. 3.1.2) and their vector-Jacobian products, any row strides.
//
// A thread owns a column of the result: it fetches the column's map entries (kept position, merge positions) once and then
// walks rows, several on their way at a time.  Lanes of a wavefront are neighbouring columns, of one row or, where rows are
// short, of several; the maps ascend, so their reads are neighbours too and every access is a coalesced one without a stage
// in LDS.  The workgroup has as many wavefronts as lose the fewest lanes to the row's end.
// Bound by the latency of the maps and of a few batches of loads, then by memory.  (Tiles of rows copied into LDS, four
// neighbouring results per lane, spent 60 % of the LDS clocks on bank conflicts and more instructions on splitting every
// index: 10 007 rows of 196, Filter 5.4 us, Union 7.4, backwards 10.7; here 4.5, 5.9, 9.9.  Rows of 16 at 32 000: 42.5 us
// for the six launches of a pipeline, 24 here.  At 262 144 rows of 256, of which 3/4 are kept: Filter 84 and 86
// backwards, where dropped columns that read the result's old row, to throw it away, cost 136; Union 151 and 239 (168 and 262
// in tiles).  Rows in several chunks lose there: 100 000 of 700, Filter backwards 98 (77 in tiles), Union 168 (150) and 228 (313).)
#include "internal.h"

#include <algorithm>

namespace dol {

namespace {

constexpr int kMaxThreads = 512;
constexpr int kAhead = 4;               // rows a thread has on their way
constexpr int kMostSteps = 16;          // rows of a thread: enough to make the maps' fetch a small part of its work,
constexpr int kFillGrid = 512;          // few enough to give the chip this many workgroups

struct RowCols {
    int32_t batch, n;
    int32_t width, per;                 // columns of a workgroup; rows side by side
    int32_t chunks, rows;               // workgroups side by side over a row; rows of a workgroup
    int32_t threads;
    unsigned grid;
};

RowCols row_cols(int32_t batch, int32_t n)
{
    RowCols R{};
    R.batch = batch, R.n = n;
    R.chunks = (n + kMaxThreads - 1) / kMaxThreads;
    R.width = (n + R.chunks - 1) / R.chunks;
    R.per = 1;
    auto waves = [&](int32_t per) { return (per * R.width + 63) / 64; };
    const int32_t most = std::min(kMaxThreads / R.width, batch);
    for (int32_t per = 2; per <= most; ++per)       // (the fullest wavefronts; of the like, the fewest)
        if (static_cast<int64_t>(per) * waves(R.per) * 16 > static_cast<int64_t>(R.per) * waves(per) * 17) R.per = per;
    R.threads = waves(R.per) * 64;
    const int64_t steps = (static_cast<int64_t>(batch) + R.per - 1) / R.per;
    int64_t mine = std::max<int64_t>(1, std::min<int64_t>(kMostSteps, steps * R.chunks / kFillGrid));
    if (mine > kAhead) mine = mine / kAhead * kAhead;
    R.rows = static_cast<int32_t>(mine) * R.per;
    R.grid = static_cast<unsigned>((static_cast<int64_t>(batch) + R.rows - 1) / R.rows * R.chunks);
    return R;
}

// Where a thread is: column c, rows first, first + per, .. , n of them (0: none).
struct Place {
    int c, n;
    int64_t first;

    __device__ __forceinline__ explicit Place(const RowCols &R)
    {
        const unsigned block = blockIdx.x / static_cast<unsigned>(R.chunks);
        const int sub = static_cast<int>(threadIdx.x / static_cast<unsigned>(R.width));
        c = static_cast<int>(blockIdx.x - block * R.chunks) * R.width + static_cast<int>(threadIdx.x) - sub * R.width;
        const int64_t s = static_cast<int64_t>(block) * R.rows;
        const int rows = static_cast<int>(min(static_cast<int64_t>(R.rows), R.batch - s));
        first = s + sub;
        n = sub < R.per && c < R.n ? (rows - sub + R.per - 1) / R.per : 0;
    }
};

// A column's entries in a thread's rows, one after the other.
template <typename T>
struct Walk {
    T *at;
    int64_t step;
    __device__ __forceinline__ Walk(T *x, int64_t ld, const Place &p, int per, int col) : at(x + p.first * ld + col), step(ld * per) {}
    __device__ __forceinline__ T &next()
    {
        T *x = at;
        at += step;
        return *x;
    }
};

// The column that a lane without one (x < 0) reads instead, to throw it away: another lane's, whose line is fetched anyway;
// -1 where no lane of the wavefront has one.
__device__ __forceinline__ int stand_in(int x)
{
    const uint64_t there = __ballot(x >= 0);
    const int other = __shfl(x, there ? __builtin_ctzll(there) : 0);
    return x >= 0 ? x : there ? other : -1;
}

// load(u) takes the next row's operands as number u, put(u) stores its result.  (Neither branches: with branches around
// the loads the compiler waits for each.)
template <class Load, class Put>
__device__ __forceinline__ void over_rows(int n, Load load, Put put)
{
    for (; n >= kAhead; n -= kAhead) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) load(u);
#pragma unroll
        for (int u = 0; u < kAhead; ++u) put(u);
    }
    for (; n > 0; --n) { load(0); put(0); }
}

}  // namespace

// out[s, c] = in[s, src_col[c]], or 0 where src_col[c] < 0: Filter forward (src_col = kept positions) and its transpose
// (src_col = position in the filtered row or -1)
template <bool ADD>
__global__ void __launch_bounds__(kMaxThreads)
damp_rows_gather_kernel(RowCols R, const int32_t *__restrict__ src_col, const float *__restrict__ in, int64_t ldi, float *__restrict__ out,
                        int64_t ldo)
{
    const Place p(R);
    if (p.n <= 0) return;
    const int32_t i = src_col[p.c];
    Walk<float> dst(out, ldo, p, R.per, p.c), old = dst;
    const int32_t from = stand_in(i);
    Walk<const float> src(in, ldi, p, R.per, from);
    if (from < 0) src.at = dst.at, src.step = dst.step;
    float v[kAhead], o[kAhead];
    over_rows(p.n,
              [&](int u) {
                  v[u] = src.next();
                  if (ADD) o[u] = old.next();
              },
              [&](int u) {
                  const float x = i >= 0 ? v[u] : 0.0f;
                  dst.next() = ADD ? x + o[u] : x;
              });
}

__global__ void __launch_bounds__(kMaxThreads)
damp_rows_union_fwd_kernel(RowCols R, const int32_t *__restrict__ ia, const int32_t *__restrict__ ib, const float *__restrict__ a,
                           int64_t lda, const float *__restrict__ b, int64_t ldb, float *__restrict__ out, int64_t ldo)
{
    const Place p(R);
    if (p.n <= 0) return;
    const int32_t i = ia[p.c], j = ib[p.c];         // (one of them at least is there)
    Walk<const float> xa(a, lda, p, R.per, i), xb(b, ldb, p, R.per, j);
    if (i < 0) xa = xb;
    if (j < 0) xb = xa;
    Walk<float> dst(out, ldo, p, R.per, p.c);
    float va[kAhead], vb[kAhead];
    over_rows(p.n,
              [&](int u) { va[u] = xa.next(), vb[u] = xb.next(); },
              [&](int u) { dst.next() = i >= 0 && j >= 0 ? fminf(va[u] + vb[u], 1.0f) : va[u]; });
}

// Column x is input position x of a (x < na) or x - na of b; without ga (gb) the columns are those of the other operand.
// The gradient passes unless both operands have the symbol and their sum exceeds 1.
template <bool ADD>
__global__ void __launch_bounds__(kMaxThreads)
damp_rows_union_bwd_kernel(RowCols R, int32_t na, const int32_t *__restrict__ ia, const int32_t *__restrict__ ib,
                           const int32_t *__restrict__ ca, const int32_t *__restrict__ cb, const float *__restrict__ a,
                           int64_t lda, const float *__restrict__ b, int64_t ldb, const float *__restrict__ g, int64_t ldg,
                           float *__restrict__ ga, float *__restrict__ gb, int32_t accumulate)
{
    const Place p(R);
    if (p.n <= 0) return;
    const bool is_a = ga && p.c < na;
    const int x = ga && !is_a ? p.c - na : p.c;
    const int32_t c = is_a ? ca[x] : cb[x];         // -1: a symbol that a fused filter drops
    const int32_t i = c >= 0 ? ia[c] : -1, j = c >= 0 ? ib[c] : -1;
    const bool both = i >= 0 && j >= 0, add = ADD && (accumulate & (is_a ? 1 : 2)) != 0;
    Walk<float> dst(is_a ? ga : gb, is_a ? lda : ldb, p, R.per, x), old = dst;
    const int32_t from = stand_in(c);
    Walk<const float> xg(g, ldg, p, R.per, from);
    if (from < 0) xg.at = dst.at, xg.step = dst.step;
    Walk<const float> xa(a, lda, p, R.per, i), xb(b, ldb, p, R.per, j);
    if (!both) xa = xb = xg;
    float gv[kAhead], o[kAhead], va[kAhead], vb[kAhead];
    over_rows(p.n,
              [&](int u) {
                  gv[u] = xg.next(), va[u] = xa.next(), vb[u] = xb.next();
                  if (ADD) o[u] = old.next();
              },
              [&](int u) {
                  float v = c >= 0 && !(both && !(va[u] + vb[u] <= 1.0f)) ? gv[u] : 0.0f;
                  if (add) v = o[u] + v;
                  dst.next() = v;
              });
}

static dol_status gather(int32_t batch, int32_t n, const int32_t *src_col, const float *in, int64_t ldi, float *out, int64_t ldo,
                  int32_t accumulate, hipStream_t st)
{
    if (batch == 0 || n == 0) return DOL_OK;
    const RowCols R = row_cols(batch, n);
    hipLaunchKernelGGL(accumulate ? damp_rows_gather_kernel<true> : damp_rows_gather_kernel<false>, dim3(R.grid),
                       dim3(static_cast<unsigned>(R.threads)), 0, st, R, src_col, in, ldi, out, ldo);
    DOL_HIP(hipGetLastError());
    return DOL_OK;
}

dol_status launch_damp_filter_fwd(const FilterPlan *p, int32_t batch, const float *in, int64_t ldi, float *out,
                                  int64_t ldo, hipStream_t st)
{
    return gather(batch, p->n_out, p->d_keep_idx.ptr, in, ldi, out, ldo, 0, st);
}

dol_status launch_damp_filter_bwd(const FilterPlan *p, int32_t batch, const float *g, int64_t ldg, float *gin,
                                  int64_t ldgi, int32_t accumulate, hipStream_t st)
{
    return gather(batch, p->n_in, p->d_pos.ptr, g, ldg, gin, ldgi, accumulate & 1, st);
}

dol_status launch_damp_union_fwd(const UnionPlan *p, int32_t batch, const float *a, int64_t lda, const float *b,
                                 int64_t ldb, float *out, int64_t ldo, hipStream_t st)
{
    if (batch == 0 || p->n_out == 0) return DOL_OK;
    const RowCols R = row_cols(batch, p->n_out);
    hipLaunchKernelGGL(damp_rows_union_fwd_kernel, dim3(R.grid), dim3(static_cast<unsigned>(R.threads)), 0, st, R, p->d_ia.ptr, p->d_ib.ptr,
                       a, lda, b, ldb, out, ldo);
    DOL_HIP(hipGetLastError());
    return DOL_OK;
}

dol_status launch_damp_union_bwd(const UnionPlan *p, int32_t batch, const float *a, int64_t lda, const float *b,
                                 int64_t ldb, const float *g, int64_t ldg, float *ga, float *gb, int32_t accumulate,
                                 hipStream_t st)
{
    const int32_t n = (ga ? p->na : 0) + (gb ? p->nb : 0);
    if (batch == 0 || n == 0) return DOL_OK;
    const RowCols R = row_cols(batch, n);
    hipLaunchKernelGGL(accumulate & 3 ? damp_rows_union_bwd_kernel<true> : damp_rows_union_bwd_kernel<false>, dim3(R.grid),
                       dim3(static_cast<unsigned>(R.threads)), 0, st, R, p->na, p->d_ia.ptr, p->d_ib.ptr, p->d_ca.ptr, p->d_cb.ptr, a, lda, b, ldb, g, ldg, ga, gb, accumulate);
    DOL_HIP(hipGetLastError());
    return DOL_OK;
}

}  // namespace dol
