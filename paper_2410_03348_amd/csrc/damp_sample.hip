// DAMP apply2 with a workgroup per sample (or per sample and part of its output row), for any function table whose rows
// fit in LDS: Apply forward and its vector-Jacobian products.
//
//     out[s, c] = min(1, sum over the tuples (i, j) of column c, ascending (i, j), of a[s, i] * b[s, j])
//     ga[s, i]  = sum_j gh[s, col(i, j)] * b[s, j],    gb[s, j] = sum_i gh[s, col(i, j)] * a[s, i]
//
// The rows a sample's tuples gather from are copied into LDS first (a cached gather from a row of thousands of tags touches
// another cache line on every lane, and a compute unit looks up about one line a clock); everything else is read and
// written coalesced:
//   * second operands of at most 16 symbols: dense maps, one j at a time, four columns (rows) a thread, 64 apart, so that a
//     map entry costs two bytes of an 8-byte load and the lanes of a gather are neighbours, whose tags lie in other banks;
//   * other tables: tuple lists of columns (rows) sorted by length inside blocks of 4 096 and interleaved in chunks of 64
//     (struct ListPlan), so that a wavefront's tuples are one 256-byte load and its lanes end together; the forward results
//     of a block meet in LDS and leave in column order.
// Lists longer than 64 tuples are summed by 16 lanes, those above 512 by a wavefront or the workgroup (struct ListPlan), in the
// same launch; forward, where tiles of samples serve the table in large batches, in the order of definition (ChainColumns).
// Empty map entries and the words past a list's end name one slot past the row, which holds 0.
#include "element_map.h"
#include "internal.h"
#include "wave_util.h"

#include <cmath>
#include <type_traits>

namespace dol {

constexpr int kSmallThreads = 256;      // workgroups of the kernels over rows of fewer than kStageMinRow tags
constexpr int kSampleThreads = 1024;
constexpr int kUnits = 256;             // compute units

constexpr int kLateMax = 64;            // long columns at the clamp that a workgroup lists

struct Lists {                          // struct ListPlan (internal.h) on the device
    const uint32_t *order, *ptr, *words, *longer;
    int32_t n_huge, n_wave, n_mid;
};

struct SampleFwd {
    int32_t na, nb, S, parts;
    int32_t map_ld, long_weight;        // dense maps
    int32_t huge;                       // dense maps: the one column that a workgroup sums (else -1), and its tuples
    uint32_t huge_q0, huge_q1;
    int32_t exact;                      // every column in its tuples' order (lists only)
    uint32_t shared;                    // see xcd_shared
    const uint16_t *map;
    Lists lists;                        // of the columns
    const uint32_t *col_ptr, *col_ij;   // a column's tuples in their order
    const float *a, *b;
    int64_t lda, ldb, ldo;
    float *out;
};

struct SampleBwd {
    int32_t na, nb, S, accumulate;
    int32_t map_ld;                     // dense maps
    const uint16_t *map;
    Lists lists;                        // of the symbols of a, then of b
    const uint32_t *rowa_ptr, *rowa_jc, *rowb_ptr, *rowb_ic;
    const uint32_t *col_ptr, *col_ij;
    const float *a, *b, *out, *g;
    int64_t lda, ldb, ldo, ldg;
    float *ga, *gb;
};

// ---------------------------------------------------------------- device helpers

// Copies n floats into LDS (16-byte aligned there) with every thread of the workgroup, and puts a 0 behind them.
__device__ __forceinline__ void copy_row(float *__restrict__ dst, const float *__restrict__ src, int n)
{
    const int n4 = n >> 2, step = blockDim.x;
#pragma unroll 4
    for (int e = threadIdx.x; e < n4; e += step) {
        const f32x4_u v = reinterpret_cast<const f32x4_u *>(src)[e];
        reinterpret_cast<float4 *>(dst)[e] = make_float4(v.x, v.y, v.z, v.w);
    }
    for (int e = (n4 << 2) + threadIdx.x; e < n; e += step) dst[e] = src[e];
    if (threadIdx.x == 0) dst[n] = 0.0f;
}

// The sum of x * y over the tuples [q0, q1) in list order, one fused multiply-add each, worked out by a whole wavefront
// (every lane gets it).  The order is serial by definition, but a term t changes nothing once s + t rounds to s, and for
// terms >= 0 the sum only grows, so a term whose DOUBLE rounds away against the sum so far (then t is at most a quarter of
// the sum's last place) is out whatever the sum becomes: 64 terms are tested at a time and only the others are added.
// A column of tens of thousands of small probabilities behind a few large ones costs a test per 64 terms; one lane adding
// them up took 0.77 ms for 18 506 terms.
__device__ __forceinline__ float serial_sum(const float *ar, const float *br, const uint32_t *__restrict__ ij_of, uint32_t q0, uint32_t q1)
{
    constexpr int kAhead = 8;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    float s = 0.0f;
    for (uint32_t q = q0; q < q1; q += kAhead * kWave) {
        uint32_t ij[kAhead];
        float x[kAhead], y[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) ij[u] = ij_of[min(q + u * kWave + lane, q1 - 1)];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            x[u] = q + u * kWave + lane < q1 ? ar[ij[u] & 0xffffu] : 0.0f;
            y[u] = br[ij[u] >> 16];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const bool quiet = x[u] * y[u] >= 0.0f && s >= 0.0f && __builtin_fmaf(x[u] + x[u], y[u], s) == s;
            uint64_t todo = __ballot(!quiet);
            if (__ballot(!(x[u] * y[u] >= 0.0f))) todo = ~uint64_t(0);      // a negative term (or none): every term counts
            for (; todo; todo &= todo - 1) {
                const int k = __builtin_ctzll(todo);
                const float xk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[u]), k));
                const float yk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(y[u]), k));
                s = __builtin_fmaf(xk, yk, s);
            }
        }
    }
    return s;
}

__device__ __forceinline__ int wave_number() { return __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave); }

__device__ __forceinline__ float wave_sum(float x)
{
    return with_lane32<AddOp>(reduce32<AddOp>(x));
}

// The wavefront's sums of each of N values, as wave_sum's bit for bit; put(k, sum) is called by the first lane of a row of 16.  Across
// rows two values share an exchange, across halves two pairs.  (At the end of every backward launch over a dense map, ten values: 16-digit
// product, 256 samples, one value after the other through LDS 279.9 us a pass, by swaps 274.0, two at a time 270.4, and the
// workgroup's shares read at once 269.8; formula of seven symbols, 200 samples 168.3, 166.7, 165.9, 164.6.)
template <int N, typename Put>
__device__ __forceinline__ void wave_sums(const float (&x)[N], Put put)
{
    constexpr int M = (N + 1) / 2, Q = (M + 1) / 2;
    const int lane = threadIdx.x & (kWave - 1), kept = (lane >> 4 & 1) + 2 * (lane >> 5);      // which of a quad's four this lane ends with
    float row[2 * M], pair[2 * Q];
#pragma unroll
    for (int k = 0; k < 2 * M; ++k) row[k] = k < N ? reduce16<AddOp>(x[k < N ? k : 0]) : row[k - 1];
#pragma unroll
    for (int k = 0; k < 2 * Q; ++k) {
        if (k >= M) { pair[k] = pair[k - 1]; continue; }
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(row[2 * k]), __float_as_uint(row[2 * k + 1]), false, false);
        pair[k] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(pair[2 * k]), __float_as_uint(pair[2 * k + 1]), false, false);
        const float sum = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        if ((lane & 15) == 0 && 4 * k + kept < N) put(4 * k + kept, sum);
    }
}

// Whether the sum `acc` of n terms, added up by `lanes` lanes, is so close to 1 that only the defining order can tell on which
// side it lies.  How far the two can lie apart: a step of the serial sum errs by at most half a unit in the last place of a
// partial sum, and by at most the term itself (s is one of the two neighbours of s + t), so by err = the sum of
// min(|t|, 2^-23) while the terms' magnitudes sum to mag <= 2; the sum over lanes errs by a rounding per step.
__device__ __forceinline__ bool order_matters(float acc, float mag, float err, uint32_t n, uint32_t lanes)
{
    const float parallel = mag * (static_cast<float>(n / lanes + 40) * 1.1920929e-7f);
    const float serial = mag <= 2.0f ? 1.01f * err : mag * (static_cast<float>(n) * 1.1920929e-7f);
    return !(fabsf(acc - 1.0f) > parallel + serial);
}

// A long column's sum: the lanes of a wavefront (WG: of the workgroup) stride over its tuples; whole wavefronts call this.
// That is not the order the clamp decision is defined in: only a sum within rounding of 1 is taken again in that order.
template <bool WG>
__device__ __forceinline__ float long_sum(const float *ar, const float *br, const uint32_t *__restrict__ ij_of, uint32_t q0, uint32_t q1,
                                          float *scratch)
{
    constexpr int kAhead = 4;
    const uint32_t step = WG ? blockDim.x : kWave, me = WG ? threadIdx.x : threadIdx.x & (kWave - 1);
    float acc = 0.0f, mag = 0.0f, err = 0.0f;
    for (uint32_t q = q0 + me; q < q1; q += kAhead * step) {
        uint32_t ij[kAhead];
        float x[kAhead], y[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) ij[u] = ij_of[min(q + u * step, q1 - 1)];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            x[u] = q + u * step < q1 ? ar[ij[u] & 0xffffu] : 0.0f;
            y[u] = br[ij[u] >> 16];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            acc = __builtin_fmaf(x[u], y[u], acc);
            mag = __builtin_fmaf(fabsf(x[u]), fabsf(y[u]), mag);
            err += fminf(fabsf(x[u] * y[u]), 1.1920929e-7f);
        }
    }
    acc = wave_sum(acc), mag = wave_sum(mag), err = wave_sum(err);
    if (WG && step > kWave) {
        const int wave = threadIdx.x / kWave, n_waves = step / kWave;
        __syncthreads();                            // the scratch of an earlier column has been read
        if ((threadIdx.x & (kWave - 1)) == 0) { scratch[wave] = acc; scratch[16 + wave] = mag; scratch[32 + wave] = err; }
        __syncthreads();
        acc = mag = err = 0.0f;
        for (int w = 0; w < n_waves; ++w) { acc += scratch[w]; mag += scratch[16 + w]; err += scratch[32 + w]; }
    }
    if (WG && threadIdx.x >= kWave) return acc;     // (the first wavefront's answer is the one that counts)
    if (order_matters(acc, mag, err, q1 - q0, step)) acc = serial_sum(ar, br, ij_of, q0, q1);
    return acc;
}

// Columns of up to kMidList words of ListPlan, four to a wavefront, 16 lanes each, the same way: put(c, sum) is called by one lane.
// A lane keeps four sums, so that a column is 64 partial sums as in a wavefront of its own and has no more roundings (one sum a
// lane: 1 000 tags 0.50e-7 off, root mean square, 0.43e-7 so).  `first`: this wavefront's first four, `step` wavefronts share them.
template <typename F>
__device__ __forceinline__ void mid_columns(const float *ar, const float *br, const uint32_t *__restrict__ col_ptr,
                                            const uint32_t *__restrict__ ij_of, const uint32_t *__restrict__ cols, int n, int first, int step, F put)
{
    constexpr int kAhead = 4, kLanes = 16;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t me = lane % kLanes;
    for (int l0 = 4 * first; l0 < n; l0 += 4 * step) {
        const int l = l0 + lane / kLanes;
        const int c = static_cast<int>(cols[min(l, n - 1)]);
        const uint32_t q0 = col_ptr[c], q1 = col_ptr[c + 1];
        float part[kAhead] = {}, mag = 0.0f, err = 0.0f;
        for (uint32_t q = q0 + me; q < q1; q += kAhead * kLanes) {
            uint32_t ij[kAhead];
            float x[kAhead], y[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) ij[u] = ij_of[min(q + u * kLanes, q1 - 1)];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                x[u] = q + u * kLanes < q1 ? ar[ij[u] & 0xffffu] : 0.0f;
                y[u] = br[ij[u] >> 16];
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                part[u] = __builtin_fmaf(x[u], y[u], part[u]);
                mag = __builtin_fmaf(fabsf(x[u]), fabsf(y[u]), mag);
                err += fminf(fabsf(x[u] * y[u]), 1.1920929e-7f);
            }
        }
        float acc = reduce16<AddOp>((part[0] + part[1]) + (part[2] + part[3]));
        mag = reduce16<AddOp>(mag), err = reduce16<AddOp>(err);
        const bool near = order_matters(acc, mag, err, q1 - q0, kLanes) && l < n && me == 0;
        for (uint64_t todo = __ballot(near); todo; todo &= todo - 1) {
            const int from = __builtin_ctzll(todo);
            const uint32_t p0 = __builtin_amdgcn_readlane(q0, from), p1 = __builtin_amdgcn_readlane(q1, from);
            const float exact = serial_sum(ar, br, ij_of, p0, p1);
            if (lane == from) acc = exact;
        }
        if (l < n && me == 0) put(c, acc);
    }
}

// s + x * y of this lane and the 15 behind it in the row of 16, one after the other, for a row's first lane: two instructions
// a term, the multiply-add takes x from the other lane by itself.  (Left to the compiler x is moved as well, into one register
// for all terms, and a term takes 29 clocks.)
__device__ __forceinline__ float chain16(float x, float y, float s)
{
    float t0, t1, t2;
#define DOL_Y(t, k) "v_mov_b32_dpp " t ", %5 row_shl:" #k " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
#define DOL_S(t, k) "v_fmac_f32_dpp %0, %4, " t " row_shl:" #k " row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
    asm("s_nop 1\n\t"                          // (x and y may have been written just now)
        DOL_Y("%1", 1) DOL_Y("%2", 2) "v_fmac_f32 %0, %4, %5\n\t"
        DOL_Y("%3", 3) DOL_S("%1", 1) DOL_Y("%1", 4) DOL_S("%2", 2) DOL_Y("%2", 5) DOL_S("%3", 3)
        DOL_Y("%3", 6) DOL_S("%1", 4) DOL_Y("%1", 7) DOL_S("%2", 5) DOL_Y("%2", 8) DOL_S("%3", 6)
        DOL_Y("%3", 9) DOL_S("%1", 7) DOL_Y("%1", 10) DOL_S("%2", 8) DOL_Y("%2", 11) DOL_S("%3", 9)
        DOL_Y("%3", 12) DOL_S("%1", 10) DOL_Y("%1", 13) DOL_S("%2", 11) DOL_Y("%2", 14) DOL_S("%3", 12)
        DOL_Y("%3", 15) DOL_S("%1", 13) DOL_S("%2", 14) DOL_S("%3", 15)
        : "+v"(s), "=&v"(t0), "=&v"(t1), "=&v"(t2)
        : "v"(x), "v"(y));
#undef DOL_Y
#undef DOL_S
    return s;
}

// The columns cols[0 .. n) in the order of their tuples, 16 lanes each, four to a wavefront: the lanes fetch 64 tuples' tags,
// the first one adds them up.  `first`, `step` as for mid_columns; the first columns' words are asked for when the object is
// made, which needs no rows yet.
struct ChainColumns {
    static constexpr uint32_t kLanes = 16;
    static constexpr int kSteps = 4;
    const uint32_t *col_ptr, *ij_of, *cols;
    int n, l0, step, c;
    uint32_t me, q0, q1, ij[kSteps];

    __device__ __forceinline__ ChainColumns(const SampleFwd &A, int first, int wavefronts)
        : col_ptr(A.col_ptr), ij_of(A.col_ij), cols(A.lists.longer), n(A.lists.n_huge + A.lists.n_wave + A.lists.n_mid), l0(4 * first),
          step(4 * wavefronts), me(threadIdx.x % kLanes)
    {
        if (l0 < n) fetch();
    }
    __device__ __forceinline__ int which() const { return l0 + static_cast<int>(threadIdx.x & (kWave - 1)) / static_cast<int>(kLanes); }
    __device__ __forceinline__ void fetch()
    {
        c = static_cast<int>(cols[min(which(), n - 1)]);
        q0 = col_ptr[c], q1 = col_ptr[c + 1];
        words(q0);
    }
    __device__ __forceinline__ void words(uint32_t q)
    {
#pragma unroll
        for (int u = 0; u < kSteps; ++u) ij[u] = ij_of[min(q + u * kLanes + me, q1 - 1)];
    }
    // put(c, sum) is called by one lane
    template <typename F>
    __device__ __forceinline__ void run(const float *ar, const float *br, F put)
    {
        while (l0 < n) {
            float s = 0.0f;
            for (uint32_t q = q0; q < q1; q += kSteps * kLanes) {
                float x[kSteps], y[kSteps];
#pragma unroll
                for (int u = 0; u < kSteps; ++u) {
                    const bool there = q + u * kLanes + me < q1;
                    x[u] = there ? ar[ij[u] & 0xffffu] : 0.0f, y[u] = there ? br[ij[u] >> 16] : 0.0f;   // (the filling adds 0 * 0)
                }
                words(q + kSteps * kLanes);                 // (on their way meanwhile)
#pragma unroll
                for (int u = 0; u < kSteps; ++u)
                    if (u == 0 || q + u * kLanes < q1) s = chain16(x[u], y[u], s);
            }
            if (which() < n && me == 0) put(c, s);
            l0 += step;
            if (l0 < n) fetch();
        }
    }
};

// The columns of more than kLaneList tuples (from the `first` on), part `part` of `parts` (the last one gets the longest): put(c, sum)
// is called by one lane.
template <typename F>
__device__ __forceinline__ void long_columns(const SampleFwd &A, int first, const float *ar, const float *br, int part, float *scratch, F put)
{
    const Lists &L = A.lists;
    for (int l = first + A.parts - 1 - part; l < L.n_huge; l += A.parts) {
        const int c = static_cast<int>(L.longer[l]);
        const float v = long_sum<true>(ar, br, A.col_ij, A.col_ptr[c], A.col_ptr[c + 1], scratch);
        if (threadIdx.x == 0) put(c, v);
    }
    const int lane = threadIdx.x & (kWave - 1), n_waves = blockDim.x / kWave, wave = part * n_waves + wave_number(), step = A.parts * n_waves;
    for (int l = L.n_huge + wave; l < L.n_huge + L.n_wave; l += step) {
        const int c = __builtin_amdgcn_readfirstlane(static_cast<int>(L.longer[l]));
        const float v = long_sum<false>(ar, br, A.col_ij, A.col_ptr[c], A.col_ptr[c + 1], scratch);
        if (lane == 0) put(c, v);
    }
    mid_columns(ar, br, A.col_ptr, A.col_ij, L.longer + L.n_huge + L.n_wave, L.n_mid, wave, step, put);
}

// ---------------------------------------------------------------- forward, dense maps

typedef __attribute__((address_space(3))) float lds_float;

__device__ __forceinline__ uint32_t lds_address(float *p) { return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_float *)p)); }

// The row's entry that half H of two map entries names; the row lies at `base` in LDS.  One instruction makes the address (the
// compiler takes the half out and adds it shifted, two of the five that a tuple cost).
template <int H>
__device__ __forceinline__ float entry_of(uint32_t base, uint32_t two)
{
    uint32_t at;
    if constexpr (H == 0) asm("v_mad_u32_u16 %0, %1, 4, %2" : "=v"(at) : "v"(two), "s"(base));
    else asm("v_mad_u32_u16 %0, %1, 4, %2 op_sel:[1,0,0,0]" : "=v"(at) : "v"(two), "s"(base));
    return *reinterpret_cast<const lds_float *>(at);
}

// The one column of a dense-map table that a workgroup sums, the last part's (in a product's table that of 0: as many tuples
// as the first operand has symbols).  Its words are on their way while the row is copied and while the words before them
// are used; the wavefronts' shares of the sum wait in LDS until the other columns are done.  A step takes four tuples a thread, as in
// long_sum: of 8 195 and 1 024 threads eight at a time make 16 of 8, and cost as much.  A step of its own for every word asked
// for at the end / so, us at 256 samples: 6 085 x 10 -> 8 282 11.3 / 9.9, 18 497 x 10 -> 23 410 19.0 / 17.7; at 16 6.0 / 5.5, 6.9 / 7.0.
// Tables with several such columns share them out over the parts instead (long_columns): one part for the first and the
// others too took 1.5 times as long, two columns of 8 193 at 16 samples 5.3 / 7.9.
struct HugeColumn {
    static constexpr int kAhead = 12, kStep = 4;
    uint32_t ij[kAhead], q, q1;

    __device__ __forceinline__ void words(const SampleFwd &A, int of, uint32_t from)
    {
#pragma unroll
        for (int u = of; u < of + kStep; ++u) ij[u] = A.col_ij[min(from + (u - of) * blockDim.x, q1 - 1)];
    }
    __device__ __forceinline__ void ask(const SampleFwd &A)
    {
        q = A.huge_q0 + threadIdx.x, q1 = A.huge_q1;
#pragma unroll
        for (int of = 0; of < kAhead; of += kStep) words(A, of, q + of * blockDim.x);
    }
    // br: the second operand's tags, in LDS
    __device__ __forceinline__ void run(const SampleFwd &A, const float *ar, const float *br, float *shares)
    {
        const uint32_t T = blockDim.x;
        float acc = 0.0f, mag = 0.0f, err = 0.0f;
        while (q - threadIdx.x < q1) {                      // (the same for all threads)
#pragma unroll
            for (int of = 0; of < kAhead; of += kStep) {
                if (q - threadIdx.x >= q1) break;
                float x[kStep], y[kStep];
#pragma unroll
                for (int u = 0; u < kStep; ++u) {
                    x[u] = q + u * T < q1 ? ar[ij[of + u] & 0xffffu] : 0.0f;
                    y[u] = q + u * T < q1 ? br[ij[of + u] >> 16] : 0.0f;
                }
                if (q + kAhead * T - threadIdx.x < q1) words(A, of, q + kAhead * T);
                q += kStep * T;
#pragma unroll
                for (int u = 0; u < kStep; ++u) {
                    acc = __builtin_fmaf(x[u], y[u], acc);
                    mag = __builtin_fmaf(fabsf(x[u]), fabsf(y[u]), mag);
                    err += fminf(fabsf(x[u] * y[u]), 1.1920929e-7f);
                }
            }
        }
        acc = wave_sum(acc), mag = wave_sum(mag), err = wave_sum(err);
        const int wave = wave_number();
        if ((threadIdx.x & (kWave - 1)) == 0) shares[wave] = acc, shares[16 + wave] = mag, shares[32 + wave] = err;
    }
    // The sum, by a whole wavefront after a barrier.
    static __device__ __forceinline__ float finish(const SampleFwd &A, const float *ar, const float *br, const float *shares)
    {
        float acc = 0.0f, mag = 0.0f, err = 0.0f;
        const int n_waves = blockDim.x / kWave;
        for (int w = 0; w < n_waves; ++w) acc += shares[w], mag += shares[16 + w], err += shares[32 + w];
        if (order_matters(acc, mag, err, A.huge_q1 - A.huge_q0, blockDim.x)) acc = serial_sum(ar, br, A.col_ij, A.huge_q0, A.huge_q1);
        return acc;
    }
};

// A column's tuples are defined to be added up in the order of i.  FALLING: in every column j falls as i rises (any function that
// grows with both operands), and one j at a time, the last one first, is that order: 18 497 x 10 -> 23 410, B=256 20.2 us, 19.7 so.
// Else the terms' magnitudes bound how far the two sums can lie apart, and only a sum within that distance of 1 is taken again
// in the defining order.  With one instruction to an address and the longest column's words ahead 17.7 us, of which an empty launch
// takes 3.6, the row's copy 2 and the columns 11 (60 M gathers of 4 bytes and 0.5 MB of map a sample, from L2).  Two samples to a
// workgroup, side by side in LDS and a map entry read once for both: 17.8, but nothing gained at 100 samples and below.
template <int NBP, bool FALLING, bool HUGE>
__device__ __forceinline__ void byj_fwd(const SampleFwd &A, float *ar)
{
    __shared__ float shares[48], yl[HUGE ? kByJMax : 1];
    __shared__ int some;
    const unsigned id = xcd_shared(blockIdx.x, A.shared);
    const int64_t s = id / static_cast<unsigned>(A.parts);
    const int part = static_cast<int>(id - s * A.parts);
    // the last part also sums the longest column: it weighs as much as `long_weight` columns
    const int per = ((A.S + A.long_weight + A.parts - 1) / A.parts + kByJBlock - 1) & ~(kByJBlock - 1);
    const int c0 = min(A.S, part * per), c1 = part == A.parts - 1 ? A.S : min(A.S, c0 + per);
    const float *br = A.b + s * A.ldb;
    float *out = A.out + s * A.ldo;
    const bool sums_huge = HUGE && part == A.parts - 1;
    HugeColumn huge;
    if (sums_huge) huge.ask(A);
    if (threadIdx.x == 0) some = 0;
    copy_row(ar, A.a + s * A.lda, A.na);
    if (HUGE && static_cast<int>(threadIdx.x) < A.nb) yl[threadIdx.x] = br[threadIdx.x];
    float y[NBP];
#pragma unroll
    for (int j = 0; j < NBP; ++j) y[j] = br[j < A.nb ? j : 0];      // (the maps' extra rows are empty)
    __syncthreads();
    if (sums_huge) huge.run(A, ar, yl, shares);
    bool again = false;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t base = lds_address(ar);
    // (Neighbouring lanes take neighbouring columns: their tags are mostly neighbours too, and lie in other banks.  With four
    // neighbours to a lane the gathers of a 16-digit product's tables met 1.6 times as many bank conflicts; its pass at 256 samples
    // 300 us, 296 with the forward maps so, 293 with the backward ones as well.)
    for (int block = c0 + kByJBlock * wave_number(); block < c1; block += 4 * static_cast<int>(blockDim.x)) {
        const int c = block + lane;                     // and 64, 128, 192 further
        uint2 m[NBP];                                   // four entries each
#pragma unroll
        for (int j = 0; j < NBP; ++j) m[j] = *reinterpret_cast<const uint2 *>(A.map + static_cast<size_t>(j) * A.map_ld + block + 4 * lane);
        const uint32_t mark[4] = {m[0].x & 0xffffu, m[0].x >> 16, m[0].y & 0xffffu, m[0].y >> 16};
        const uint32_t none = static_cast<uint32_t>(A.na);
        m[0].x = min(mark[0], none) | min(mark[1], none) << 16, m[0].y = min(mark[2], none) | min(mark[3], none) << 16;
        float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f}, mag[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int jj = 0; jj < NBP; ++jj) {
            const int j = FALLING ? NBP - 1 - jj : jj;
            const float x[4] = {entry_of<0>(base, m[j].x), entry_of<1>(base, m[j].x), entry_of<0>(base, m[j].y), entry_of<1>(base, m[j].y)};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                acc[k] = __builtin_fmaf(x[k], y[j], acc[k]);
                if (!FALLING) mag[k] = __builtin_fmaf(fabsf(x[k]), fabsf(y[j]), mag[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool there = c + kWave * k < c1 && mark[k] != kByJWave;           // (kByJWave: many tuples, summed apart)
            const bool near = FALLING ? acc[k] != acc[k]                            // (0 for no tuple, times an infinity)
                                      : !(fabsf(acc[k] - 1.0f) > mag[k] * (static_cast<float>(NBP + 2) * 1.1920929e-7f));
            const bool list = (near || mark[k] == kByJList) && there;               // (kByJList: some j twice)
            again |= list;
            if (there) out[c + kWave * k] = list ? __builtin_nanf("") : fminf(acc[k], 1.0f);
        }
    }
    if (again) some = 1;
    lds_barrier();                          // (does not wait for the results to be in memory)
    if (some) {                             // columns marked by a NaN, which no result is: neighbouring lanes, neighbouring columns
        __syncthreads();
        for (int c = c0 + static_cast<int>(threadIdx.x); c < c1; c += static_cast<int>(blockDim.x)) {
            const float v = out[c];
            if (v == v) continue;
            const uint32_t q0 = A.col_ptr[c], q1 = A.col_ptr[c + 1];
            if (q1 - q0 <= static_cast<uint32_t>(kLaneList)) out[c] = fminf(column_sum(ar, br, A.col_ij, q0, q1), 1.0f);
        }
    }
    if (sums_huge && wave_number() == 0) {
        const float v = HugeColumn::finish(A, ar, br, shares);
        if (lane == 0) out[A.huge] = fminf(v, 1.0f);
    }
    long_columns(A, HUGE ? 1 : 0, ar, br, part, shares, [&](int c, float v) { out[c] = fminf(v, 1.0f); });
}

template <int NBP, bool FALLING, bool HUGE>
__global__ void __launch_bounds__(kSmallThreads)
damp_byj_fwd_kernel(const SampleFwd A)
{
    extern __shared__ __align__(16) float lds[];
    byj_fwd<NBP, FALLING, HUGE>(A, lds);
}

// (64 registers, for two workgroups of 1 024 threads to a unit)
template <int NBP, bool FALLING, bool HUGE>
__global__ void __launch_bounds__(kSampleThreads, 8)
damp_byj_fwd_staged_kernel(const SampleFwd A)
{
    extern __shared__ __align__(16) float lds[];
    byj_fwd<NBP, FALLING, HUGE>(A, lds);
}

// ---------------------------------------------------------------- forward, tuple lists

// A wavefront walks one chunk of 64 lists at a time, N words of each per step; a step's words, and the first ones of the
// next chunk, are read while the step before is worked on (they come from L2, whose latency is what this would cost).
// Columns: N = 4 (most are short); rows, of as many tuples as the other operand has symbols: N = 8.
template <int N>
struct Chunk {
    uint32_t e, w0, len, t[N];
};

template <int N>
__device__ __forceinline__ void read_words(uint32_t (&t)[N], const Lists &L, uint32_t w)
{
    const uint32_t *__restrict__ p = L.words + static_cast<size_t>(w) * kWave + (threadIdx.x & (kWave - 1));
#pragma unroll
    for (int u = 0; u < N; ++u) t[u] = p[u * kWave];
}

template <int N>
__device__ __forceinline__ Chunk<N> read_chunk(const Lists &L, int ch)
{
    Chunk<N> c;
    c.w0 = L.ptr[ch], c.len = L.ptr[ch + 1] - c.w0;
    c.e = L.order[ch * kWave + (threadIdx.x & (kWave - 1))];
    read_words(c.t, L, c.w0);
    return c;
}

// Walks the chunks [ch0, ch1), a wavefront every blockDim.x / 64th: term(word, sum) takes a tuple into a list's sum, in list
// order, and done(list, sum) is called for every list that is walked here, elsewhere(list) for the longer ones.  `now`: this
// wavefront's first chunk.
template <int N, typename T, typename D, typename E>
__device__ __forceinline__ void walk_lists(const Lists &L, int ch0, int ch1, Chunk<N> now, T term, D done, E elsewhere)
{
    const int n_waves = blockDim.x / kWave;
    for (int ch = ch0 + wave_number(); ch < ch1; ch += n_waves) {
        const Chunk<N> next = read_chunk<N>(L, min(ch + n_waves, ch1 - 1));
        float acc = 0.0f;
        for (uint32_t w = 0; w < now.len; w += N) {
            uint32_t t[N];
#pragma unroll
            for (int u = 0; u < N; ++u) t[u] = now.t[u];
            if (w + N < now.len) read_words<N>(now.t, L, now.w0 + w + N);
            const uint32_t left = now.len - w;              // (the same for all lanes)
            if (left >= static_cast<uint32_t>(N)) {
#pragma unroll
                for (int u = 0; u < N; ++u) acc = term(t[u], acc);
            } else {
#pragma unroll
                for (int u = 0; u < N - 1; ++u)
                    if (static_cast<uint32_t>(u) < left) acc = term(t[u], acc);
            }
        }
        if (!(now.e & kListElsewhere)) done(static_cast<int>(now.e), acc);
        else if (now.e != kNoList) elsewhere(static_cast<int>(now.e & ~kListElsewhere));
        now = next;
    }
}

// RES: a block of results meets in LDS and leaves in column order; without it they are stored where they fall.  Longer columns
// are shared out over all parts and stored apart.
template <bool RES>
__global__ void __launch_bounds__(kSampleThreads)
damp_apply2_fwd_staged_kernel(const SampleFwd A)
{
    extern __shared__ __align__(16) float lds[];            // a's row and a 0, b's and a 0 [a block of results]
    __shared__ float scratch[48];
    float *ar = lds, *br = lds + ((A.na + 4) & ~3), *res = br + ((A.nb + 4) & ~3);
    const unsigned id = xcd_shared(blockIdx.x, A.shared);
    const int64_t s = id / static_cast<unsigned>(A.parts);
    const int part = static_cast<int>(id - s * A.parts);
    constexpr int kBlockChunks = kOrderBlock / kWave;
    const int n_chunks = (A.S + kWave - 1) / kWave;
    Chunk<4> now = read_chunk<4>(A.lists, min(part * kBlockChunks + wave_number(), n_chunks - 1));
    const int n_waves = blockDim.x / kWave;                 // (the last wavefronts have the fewest lists)
    ChainColumns chain(A, A.exact ? part + A.parts * (n_waves - 1 - wave_number()) : INT32_MAX / 4, A.parts * n_waves);
    copy_row(ar, A.a + s * A.lda, A.na);
    copy_row(br, A.b + s * A.ldb, A.nb);
    __syncthreads();
    float *out = A.out + s * A.ldo;
    auto put_long = [&](int c, float v) { out[c] = fminf(v, 1.0f); };
    chain.run(ar, br, put_long);
    for (int b0 = part * kOrderBlock; b0 < A.S; b0 += A.parts * kOrderBlock) {
        const int b1 = min(A.S, b0 + kOrderBlock);
        walk_lists<4>(A.lists, b0 / kWave, (b1 + kWave - 1) / kWave, now,
                   [&](uint32_t t, float acc) { return __builtin_fmaf(ar[t & 0xffffu], br[t >> 16], acc); },
                   [&](int c, float v) { (RES ? res - b0 : out)[c] = fminf(v, 1.0f); },
                   [&](int c) { if (RES) res[c - b0] = __builtin_nanf(""); });      // (a result is never a NaN: the clamp makes it 1)
        const int next = b0 + A.parts * kOrderBlock;
        if (next < A.S) now = read_chunk<4>(A.lists, min(next / kWave + wave_number(), n_chunks - 1));
        if (!RES) continue;
        __syncthreads();
        for (int c = 4 * static_cast<int>(threadIdx.x); c < b1 - b0; c += 4 * static_cast<int>(blockDim.x)) {
            const float4 v = *reinterpret_cast<const float4 *>(res + c);
            const float r[4] = {v.x, v.y, v.z, v.w};
            uint32_t skip = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) skip |= (r[k] == r[k] ? 0u : 1u) << k;
            store4(out + b0 + c, r, b1 - b0 - c, skip);
        }
        __syncthreads();
    }
    if (!A.exact) long_columns(A, 0, ar, br, part, scratch, put_long);
}

// Unary Apply over wide rows: out[c] = min(1, sum of the tags of column c's symbols).  The lists hold two symbols to a word.  A
// wavefront walks C chunks of them at a time, N words of each per step, so that short lists have as much on the way as long
// ones; all parts' wavefronts share the chunks out, each every parts * wavefronts-th, which get shorter by steps.  38 400 -> 8 333 (a seven-symbol formula's value), us,
// with the first eight symbols of a column in a 16-byte word, the others four at a time out of the column's list and
// the columns above 64 in a launch of their own: B=16 11.6, 64 19.4, 200 27.4; so 5.9, 8.8, 14.9.  Bound by the row's way into LDS.
// Every list is added up in its defining order, which the clamp decides by.  BLOCKS: where a chunk has lists of more than 64 symbols the
// lanes add up blocks of 16 to 24 as well, and below 1 their sum is the result: one after the other, 128 tags end 1.6e-7 off (root
// mean square), as 64 lanes' shares 0.42e-7, so 0.42e-7.
constexpr uint32_t kPlainWords = kLaneList / 2;     // (two symbols each)
template <int C, int N>
struct Walk {
    uint32_t e[C], w0[C], len[C], t[C][N];

    __device__ __forceinline__ void start(const Lists &L, int ch, int step, int n_chunks)
    {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int at = min(ch + c * step, n_chunks - 1);
            w0[c] = L.ptr[at], len[c] = ch + c * step < n_chunks ? L.ptr[at + 1] - w0[c] : 0u;
            e[c] = ch + c * step < n_chunks ? L.order[at * kWave + (threadIdx.x & (kWave - 1))] : kNoList;
            read_words(t[c], L, w0[c]);
        }
    }
};

template <int C, int N, bool BLOCKS>
__global__ void __launch_bounds__(kSampleThreads)
damp_apply1_fwd_staged_kernel(const SampleFwd A)
{
    extern __shared__ __align__(16) float lds[];            // the row and a 0
    __shared__ float scratch[48], one;
    const unsigned id = xcd_shared(blockIdx.x, A.shared);
    const int64_t s = id / static_cast<unsigned>(A.parts);
    const int part = static_cast<int>(id - s * A.parts);
    const int n_chunks = (A.S + kWave - 1) / kWave, step = A.parts * (blockDim.x / kWave);
    int ch = part + A.parts * wave_number();
    Walk<C, N> now, next;
    now.start(A.lists, ch, step, n_chunks);
    copy_row(lds, A.a + s * A.lda, A.na);
    if (threadIdx.x == 0) one = 1.0f;
    __syncthreads();
    float *out = A.out + s * A.ldo;
    auto put = [&](int c, float v) { out[c] = fminf(v, 1.0f); };
    for (; ch < n_chunks; ch += C * step) {
        const bool more = ch + C * step < n_chunks;
        if (more) next.start(A.lists, ch + C * step, step, n_chunks);
        float acc[C] = {};
        uint32_t most = 0;
#pragma unroll
        for (int c = 0; c < C; ++c) most = max(most, now.len[c]);
        float total[C][4] = {}, block[C] = {};              // (blocks go to the four totals in turn)
        auto walk = [&](auto blocks) {
            for (uint32_t w = 0; w < most; w += N) {
                float v[C][N][2];                           // (a word past a list's end is another's: read, not added)
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int u = 0; u < N; ++u) v[c][u][0] = lds[now.t[c][u] & 0xffffu], v[c][u][1] = lds[now.t[c][u] >> 16];
#pragma unroll
                for (int c = 0; c < C; ++c)
                    if (w + N < now.len[c]) read_words(now.t[c], A.lists, now.w0[c] + w + N);
#pragma unroll
                for (int c = 0; c < C; ++c) {
#pragma unroll
                    for (int u = 0; u < N; ++u) acc[c] = w + u < now.len[c] ? acc[c] + v[c][u][0] + v[c][u][1] : acc[c];
                    if constexpr (blocks) {
                        float pair[N];
#pragma unroll
                        for (int u = 0; u < N; ++u) pair[u] = w + u < now.len[c] ? v[c][u][0] + v[c][u][1] : 0.0f;
#pragma unroll
                        for (int d = 1; d < N; d *= 2)
#pragma unroll
                            for (int u = 0; u + d < N; u += 2 * d) pair[u] += pair[u + d];
                        block[c] += pair[0];
                        if (N >= 8 || (w / N) % 4 == 3) {
                            const float t = total[c][0] + block[c];
                            total[c][0] = total[c][1], total[c][1] = total[c][2], total[c][2] = total[c][3], total[c][3] = t, block[c] = 0.0f;
                        }
                    }
                }
            }
        };
        if (!BLOCKS || most <= kPlainWords) {
            walk(std::false_type{});
        } else {
            walk(std::true_type{});
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float sum = ((total[c][0] + block[c]) + total[c][1]) + (total[c][2] + total[c][3]);
                acc[c] = acc[c] < 1.0f ? fminf(sum, 0x1.fffffep-1f) : acc[c];
            }
        }
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (!(now.e[c] & kListElsewhere)) put(static_cast<int>(now.e[c]), acc[c]);
        if (!more) break;
        now = next;
    }
    long_columns(A, 0, lds, &one, part, scratch, put);         // (a tuple's word: the symbol, times symbol 0 of `one`)
}

// ---------------------------------------------------------------- backward

// The long columns at the clamp, n of them, by a wavefront each: close(c), by one lane, where it acted.
template <typename F>
__device__ __forceinline__ void late_columns(const SampleBwd &A, const float *ar, const float *br, const float *outr, int n, const int *late, F close)
{
    const int lane = threadIdx.x & (kWave - 1), wave = wave_number(), n_waves = blockDim.x / kWave;
    auto decide = [&](int c) {              // by a whole wavefront
        const float pre = long_sum<false>(ar, br, A.col_ij, A.col_ptr[c], A.col_ptr[c + 1], nullptr);
        if (!(pre <= 1.0f) && lane == 0) close(c);
    };
    if (n <= kLateMax) {
        for (int l = wave; l < n; l += n_waves) decide(__builtin_amdgcn_readfirstlane(late[l]));
    } else {                                // more than the list holds: every wavefront looks through its share of the columns
        for (int c0 = wave; c0 < A.S; c0 += kWave * n_waves) {
            const int c = c0 + lane * n_waves;
            const bool mine = c < A.S && outr[c] >= 1.0f && A.col_ptr[c + 1] - A.col_ptr[c] > static_cast<uint32_t>(kLongTableCol);
            for (uint64_t todo = __ballot(mine); todo; todo &= todo - 1) decide(c0 + __builtin_ctzll(todo) * n_waves);
        }
    }
}

// gh[c] = g[c] where the clamp did not act, else 0, for the whole row, and a 0 behind it.  out < 1: it did not act;
// out == 1 leaves pre == 1 (passes) and pre > 1 (blocks) apart only by pre itself, taken again: by the thread at hand, long
// columns by a wavefront each after the others.  (45 000 x 10 -> 300, every column of 1 500 tuples clamped, B=256: 2.8 ms with
// the columns beyond the list summed by the thread that met them, a tuple at a time, and the others in their order of
// definition.)  STAGED: gh is filled with that row; else `closed` gets a bit per
// column the clamp acted on, and the answer is whether there are any.
template <bool STAGED>
__device__ __forceinline__ bool gated_row(const SampleBwd &A, int64_t s, float *gh, uint32_t *closed, int *n_late, int *late)
{
    const float *ar = A.a + s * A.lda, *br = A.b + s * A.ldb, *outr = A.out + s * A.ldo, *gr = A.g + s * A.ldg;
    int any = 0;
    auto close = [&](int c) {
        if (STAGED) gh[c] = 0.0f;
        else atomicOr(closed + (c >> 5), 1u << (c & 31));
        any = 1;
    };
    if (threadIdx.x == 0) { *n_late = 0; if (STAGED) gh[A.S] = 0.0f; }
    if (!STAGED)
        for (int w = threadIdx.x; w < (A.S + 31) / 32; w += blockDim.x) closed[w] = 0u;
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1), wave = wave_number(), n_waves = blockDim.x / kWave;
    constexpr int U = 2;                    // pieces of both rows that a lane asks for before it waits
    for (int first = 4 * kWave * wave; first < A.S; first += U * 4 * kWave * n_waves) {
        float4 o4[U], g4[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c0 = first + u * 4 * kWave * n_waves, c = c0 + 4 * lane;
            if (c0 >= A.S) break;           // (uniform)
            o4[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (c >= A.S) continue;
            o4[u] = load4(outr + c, A.S - c);
            if (STAGED) g4[u] = load4(gr + c, A.S - c);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c0 = first + u * 4 * kWave * n_waves, c = c0 + 4 * lane;
            if (c0 >= A.S) break;
            if (STAGED && c + 4 <= A.S) {
                *reinterpret_cast<float4 *>(gh + c) = g4[u];
            } else if (STAGED) {
                const float g[4] = {g4[u].x, g4[u].y, g4[u].z, g4[u].w};
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (c + k < A.S) gh[c + k] = g[k];
            }
            if (!__ballot(o4[u].x >= 1.0f || o4[u].y >= 1.0f || o4[u].z >= 1.0f || o4[u].w >= 1.0f)) continue;
            for (int cc = c0 + lane; cc < min(A.S, c0 + 4 * kWave); cc += kWave) {      // (neighbouring lanes, neighbouring columns)
                if (!(outr[cc] >= 1.0f)) continue;
                const uint32_t q0 = A.col_ptr[cc], q1 = A.col_ptr[cc + 1];
                if (q1 - q0 > static_cast<uint32_t>(kLongTableCol)) {
                    const int slot = atomicAdd(n_late, 1);
                    if (slot < kLateMax) late[slot] = cc;
                } else if (!(column_sum(ar, br, A.col_ij, q0, q1) <= 1.0f)) close(cc);
            }
        }
    }
    __syncthreads();
    const int n = *n_late;
    late_columns(A, ar, br, outr, n, late, close);
    if (!STAGED) return __syncthreads_or(any) != 0;
    if (n) __syncthreads();
    return false;
}

// Unary Apply over wide rows: every operand symbol picks its column's entry of the gated gradient row, four neighbours a thread.
// 38 400 symbols -> 8 333: us, a symbol at a time by a 32-bit column number B=16 5.3, 64 6.9, 200 15.7; so 4.1, 5.4, 9.7 (with two
// workgroups to a unit 4.5, 7.0, 10.6).  Columns at the clamp: one to a thread, neighbouring ones to neighbouring lanes, those of more
// than 64 symbols to a wavefront.  (By the thread that meets them, four neighbours each, 40 400 -> 242, one to 1 300 symbols to a column,
// B=16 470 us, one each 157; so 16.  That somebody has to look costs rows of 5 000 0.8 us of 12 at 2 000 samples.)
__global__ void __launch_bounds__(kSampleThreads, 8)
damp_apply1_bwd_staged_kernel(const SampleBwd A, int32_t parts, uint32_t shared)
{
    extern __shared__ __align__(16) float gh[];             // the gated row and a 0
    __shared__ int n_late, late[kLateMax];
    __shared__ bool acted[kSampleThreads / kWave];
    constexpr int kAhead = 2;
    const unsigned id = xcd_shared(blockIdx.x, shared);
    const int64_t s = id / static_cast<unsigned>(parts);
    const int part = static_cast<int>(id - s * parts), per = ((A.na + parts - 1) / parts + 3) & ~3, T = blockDim.x;
    const int i0 = part * per, i1 = min(A.na, i0 + per);
    ushort4 c[kAhead];
    auto columns = [&](int i) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u)                    // (the map is padded to whole fours)
            if (i + 4 * T * u < i1) c[u] = *reinterpret_cast<const ushort4 *>(A.map + i + 4 * T * u);
    };
    columns(i0 + 4 * static_cast<int>(threadIdx.x));
    const float *gr = A.g + s * A.ldg, *outr = A.out + s * A.ldo;
    bool at_one = false;
    for (int k0 = 4 * static_cast<int>(threadIdx.x); k0 < A.S; k0 += 8 * T) {
        float4 v[2], o[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int k = k0 + 4 * T * u;
            if (k < A.S) v[u] = load4(gr + k, A.S - k), o[u] = load4(outr + k, A.S - k);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int k = k0 + 4 * T * u;
            if (k >= A.S) continue;
            at_one |= o[u].x >= 1.0f || o[u].y >= 1.0f || o[u].z >= 1.0f || o[u].w >= 1.0f;
            *reinterpret_cast<float4 *>(gh + k) = v[u];     // (words past the row are 0)
        }
    }
    const int lane = threadIdx.x & (kWave - 1);
    const bool some = __ballot(at_one) != 0;
    if (lane == 0) acted[wave_number()] = some;
    if (threadIdx.x == 0) n_late = 0;
    if (threadIdx.x == 0 && (A.S & 3) == 0) gh[A.S] = 0.0f;
    __syncthreads();
    if (__ballot(lane < T / kWave && acted[lane & 15]) != 0) {      // (the same for all wavefronts)
        const float *ar = A.a + s * A.lda;
        for (int k = threadIdx.x; k < A.S; k += T) {        // (neighbouring lanes, neighbouring columns)
            if (!(outr[k] >= 1.0f)) continue;
            const uint32_t q0 = A.col_ptr[k], q1 = A.col_ptr[k + 1];
            if (q1 - q0 > static_cast<uint32_t>(kLongTableCol)) {
                const int slot = atomicAdd(&n_late, 1);
                if (slot < kLateMax) late[slot] = k;
            } else if (!(column_sum(ar, A.b, A.col_ij, q0, q1) <= 1.0f)) gh[k] = 0.0f;
        }
        __syncthreads();
        late_columns(A, ar, A.b, outr, n_late, late, [&](int k) { gh[k] = 0.0f; });
        __syncthreads();
    }
    float *dst = A.ga + s * A.lda;
    for (int i = i0 + 4 * static_cast<int>(threadIdx.x); i < i1; i += 4 * T * kAhead) {
        float v[kAhead][4];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (i + 4 * T * u >= i1) continue;
            v[u][0] = gh[c[u].x], v[u][1] = gh[c[u].y], v[u][2] = gh[c[u].z], v[u][3] = gh[c[u].w];
        }
        columns(i + 4 * T * kAhead);
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (i + 4 * T * u < i1) store4(dst + i + 4 * T * u, v[u], i1 - (i + 4 * T * u));
    }
}

// Dense maps: a thread owns four rows of a, 64 apart (see byj_fwd), and adds their shares of gb up in registers; the workgroup's
// shares meet at the end (so the long rows of b need no launch of their own).  STAGED: the gated gradient row is in LDS.
// Result rows that do not fit there (more than 40 447 symbols) are gathered from memory, and from LDS a bit per column where
// the clamp acted, if it acted anywhere in the sample: B=256, 41 000 x 4 -> 41 000 234 us, element by element with a look at
// every column's clamp 2 335; all columns clamped 2 865 and 6 763.
template <int NBP, int T, bool STAGED>
__device__ __forceinline__ void byj_bwd(const SampleBwd &A, float *lds)
{
    __shared__ __align__(16) float red[NBP][T / kWave];
    __shared__ int n_late, late[kLateMax];
    const int64_t s = blockIdx.x;
    const float *ar = A.a + s * A.lda, *br = A.b + s * A.ldb, *gr = A.g + s * A.ldg;
    float *gh = lds;
    uint32_t *closed = reinterpret_cast<uint32_t *>(lds);
    const bool gates = gated_row<STAGED>(A, s, gh, closed, &n_late, late);
    float bj[NBP], pb[NBP];
#pragma unroll
    for (int j = 0; j < NBP; ++j) {
        bj[j] = j < A.nb ? br[j] : 0.0f;
        pb[j] = 0.0f;
    }
    constexpr int R = STAGED || NBP < 10 ? 4 : 2;       // rows at a time (gathers from memory: as many as registers hold)
    typedef uint16_t __attribute__((ext_vector_type(R))) entries;
    const int last = A.S - 1;
    const uint32_t base = lds_address(gh);
    const int lane = threadIdx.x & (kWave - 1), wave = wave_number(), n_waves = blockDim.x / kWave;
    for (int i0 = R * kWave * wave; i0 < A.na; i0 += R * kWave * n_waves) {
        const int i = i0 + lane, at = (i0 & ~(kByJBlock - 1)) + 4 * lane + ((i0 / kWave) & 3);      // rows i, i + 64 ..; where their entries lie
        entries m[NBP];
#pragma unroll
        for (int j = 0; j < NBP; ++j) m[j] = *reinterpret_cast<const entries *>(A.map + static_cast<size_t>(j) * A.map_ld + at);
        float av[4];
#pragma unroll
        for (int k = 0; k < R; ++k) av[k] = i + kWave * k < A.na ? ar[i + kWave * k] : 0.0f;
        float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int j = 0; j < NBP; ++j) {
            int col[R];
            float v[R];
            if constexpr (STAGED) {
                const uint2 two = __builtin_bit_cast(uint2, m[j]);
                v[0] = entry_of<0>(base, two.x), v[1] = entry_of<1>(base, two.x), v[2] = entry_of<0>(base, two.y), v[3] = entry_of<1>(base, two.y);
            } else {
#pragma unroll
                for (int k = 0; k < R; ++k) col[k] = m[j][k];
                uint32_t shut[R];
#pragma unroll
                for (int k = 0; k < R; ++k) shut[k] = gates ? closed[min(col[k], last) >> 5] >> (col[k] & 31) : 0u;
#pragma unroll
                for (int k = 0; k < R; ++k) v[k] = gr[min(col[k], last)];
#pragma unroll
                for (int k = 0; k < R; ++k) v[k] = col[k] > last || (shut[k] & 1u) ? 0.0f : v[k];
            }
#pragma unroll
            for (int k = 0; k < R; ++k) {
                acc[k] = __builtin_fmaf(v[k], bj[j], acc[k]);
                pb[j] = __builtin_fmaf(v[k], av[k], pb[j]);
            }
        }
        if (A.ga) {
            float *dst = A.ga + s * A.lda + i;
            if (A.accumulate & 1) {
#pragma unroll
                for (int k = 0; k < R; ++k)
                    if (i + kWave * k < A.na) acc[k] += dst[kWave * k];
            }
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (i + kWave * k < A.na) dst[kWave * k] = acc[k];
        }
    }
    if (!A.gb) return;
    wave_sums<NBP>(pb, [&](int j, float v) { red[j][wave] = v; });
    __syncthreads();
    if (threadIdx.x < static_cast<unsigned>(A.nb)) {
        float share[T / kWave], tot = 0.0f;             // (read at once, added in order)
#pragma unroll
        for (int w = 0; w < T / kWave; ++w) share[w] = red[threadIdx.x][w];
#pragma unroll
        for (int w = 0; w < T / kWave; ++w) tot = w < n_waves ? tot + share[w] : tot;
        float *dst = A.gb + s * A.ldb + threadIdx.x;
        *dst = (A.accumulate & 2) ? *dst + tot : tot;
    }
}

template <int NBP>
__global__ void __launch_bounds__(kSmallThreads)
damp_byj_bwd_kernel(const SampleBwd A)
{
    extern __shared__ __align__(16) float lds[];
    byj_bwd<NBP, kSmallThreads, true>(A, lds);
}

// (at least six wavefronts to a SIMD where the maps of ten j leave 81 registers: two workgroups of twelve share a unit)
template <int NBP>
__global__ void __launch_bounds__(kSampleThreads, NBP == 10 ? 6 : 4)
damp_byj_bwd_row_kernel(const SampleBwd A)
{
    extern __shared__ __align__(16) float lds[];
    byj_bwd<NBP, kSampleThreads, true>(A, lds);
}

template <int NBP>
__global__ void __launch_bounds__(kSampleThreads)
damp_byj_bwd_global_kernel(const SampleBwd A)
{
    extern __shared__ __align__(16) float lds[];
    byj_bwd<NBP, kSampleThreads, false>(A, lds);
}

// Tuple lists: a lane owns a symbol of a or b (element x: symbol x of a, or x - na of b) and adds up its tuples from the
// gated gradient row, in list order; longer lists are summed by 16 lanes or the workgroup, strided partial sums in list order
// that meet in a fixed order.  ROWS: the operand rows fit in LDS as well.
template <bool ROWS>
__global__ void __launch_bounds__(kSampleThreads)
damp_apply2_bwd_staged_kernel(const SampleBwd A)
{
    extern __shared__ __align__(16) float lds[];            // gated gradient row and a 0 [a and b behind each other, a 0]
    __shared__ float scratch[kSampleThreads / kWave];
    __shared__ int n_late, late[kLateMax];
    const int64_t s = blockIdx.x;
    float *gh = lds, *rows = lds + ((A.S + 4) & ~3);
    const float *ar = A.a + s * A.lda, *br = A.b + s * A.ldb;
    const int n = A.na + A.nb;
    const int n_chunks = (n + kWave - 1) / kWave;
    const Chunk<8> now = read_chunk<8>(A.lists, min(wave_number(), n_chunks - 1));
    if (ROWS) {
        for (int e = threadIdx.x; e < A.na; e += blockDim.x) rows[e] = ar[e];
        for (int e = threadIdx.x; e < A.nb; e += blockDim.x) rows[A.na + e] = br[e];
        if (threadIdx.x == 0) rows[n] = 0.0f;
    }
    gated_row<true>(A, s, gh, nullptr, &n_late, late);      // (ends after a barrier)
    // a list's word: the other operand's symbol, counted from a's first one (b's from na on; na + nb: none), and the column
    auto other = [&](uint32_t x) {
        if (ROWS) return rows[x];
        const uint32_t na = A.na, end = A.na + A.nb;
        return x < na ? ar[x] : x < end ? br[x - na] : 0.0f;
    };
    auto term = [&](uint32_t t, float acc) { return __builtin_fmaf(gh[t >> 16], other(t & 0xffffu), acc); };
    auto put = [&](int x, float v) {
        const bool is_a = x < A.na;
        if (is_a ? !A.ga : !A.gb) return;
        float *dst = is_a ? A.ga + s * A.lda + x : A.gb + s * A.ldb + (x - A.na);
        *dst = (A.accumulate & (is_a ? 1 : 2)) ? *dst + v : v;
    };
    walk_lists<8>(A.lists, 0, n_chunks, now, term, put, [](int) {});
    const Lists &L = A.lists;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, n_waves = blockDim.x / kWave;
    // the partial sum of this lane, one of `step` lanes, over the list of element x
    auto partial = [&](int x, uint32_t me, uint32_t step) {
        const bool is_a = x < A.na;
        const uint32_t *__restrict__ ent = is_a ? A.rowa_jc : A.rowb_ic;
        const uint32_t q0 = is_a ? A.rowa_ptr[x] : A.rowb_ptr[x - A.na], q1 = is_a ? A.rowa_ptr[x + 1] : A.rowb_ptr[x - A.na + 1];
        const uint32_t base = is_a ? A.na : 0;
        float acc = 0.0f;
        for (uint32_t q = q0 + me; q < q1; q += 4 * step) {
            uint32_t t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] = ent[min(q + u * step, q1 - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float x4 = other(base + (t[u] & 0xffffu)), g4 = gh[t[u] >> 16];
                acc = __builtin_fmaf(q + u * step < q1 ? g4 : 0.0f, x4, acc);
            }
        }
        return acc;
    };
    for (int l0 = 4 * wave; l0 < L.n_mid; l0 += 4 * n_waves) {
        const int l = l0 + lane / 16;
        const int x = static_cast<int>(L.longer[L.n_huge + min(l, L.n_mid - 1)]);
        const float v = reduce16<AddOp>(partial(x, lane & 15, 16));
        if (l < L.n_mid && (lane & 15) == 0) put(x, v);
    }
    for (int l = 0; l < L.n_huge; ++l) {
        const int x = static_cast<int>(L.longer[l]);
        const float v = wave_sum(partial(x, threadIdx.x, blockDim.x));
        __syncthreads();                                    // (the last list's totals have been read)
        if (lane == 0) scratch[wave] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            float tot = 0.0f;
            for (int w = 0; w < n_waves; ++w) tot += scratch[w];
            put(x, tot);
        }
    }
}

// ---------------------------------------------------------------- Apply + Filter + Union, forward, backward or both

struct SampleMerge {
    int32_t na, nb, S, nc, n3, accumulate;
    Lists cols, rows;
    const int32_t *ia, *ib, *ca, *cb;   // struct UnionPlan
    const float *a, *b, *c, *g;
    float *out, *ga, *gb, *gc;
    int32_t *saved;
};

// The merged calls (api.hip) for small batches and tables of columns and rows of at most 64 tuples: contiguous tensors, all
// of a sample's rows in LDS, nothing intermediate anywhere else.  What counts is the chain of latencies: the rows and the
// first words of both sweeps' lists are requested together, and the only other memory the kernel waits for are the lists'
// further words.
template <bool FWD, bool BWD>
__global__ void __launch_bounds__(512)
damp_merge_sample_kernel(SampleMerge A)
{
    extern __shared__ __align__(16) float lds[];            // [a][b][0], [a][0], sums of the Apply, c's row, gated gradient and 0
    const int n = A.na + A.nb;
    // (a again, with a 0 behind it, for the columns: their lists' filling must not multiply a tag, which may be no number)
    float *rows = lds, *ar = rows + n + 1, *pre = lds + ((n + A.na + 5) & ~3), *cr = pre + A.S, *gh = cr + A.nc;
    const int64_t s = blockIdx.x;
    const int T = blockDim.x, tid = threadIdx.x, wave = wave_number();
    const int col_chunks = (A.S + kWave - 1) / kWave, row_chunks = (n + kWave - 1) / kWave;
    Chunk<4> first_cols = read_chunk<4>(A.cols, min(wave, col_chunks - 1));
    Chunk<8> first_rows{};
    if (BWD) first_rows = read_chunk<8>(A.rows, min(wave, row_chunks - 1));
    int acted = BWD && !FWD && A.saved ? A.saved[s] : 1;
    for (int e = tid; e < n; e += T) {
        const float v = e < A.na ? A.a[s * A.na + e] : A.b[s * A.nb + (e - A.na)];
        rows[e] = v;
        if (e < A.na) ar[e] = v;
    }
    for (int e = tid; e < A.nc; e += T) cr[e] = A.c[s * A.nc + e];
    if (tid == 0) { rows[n] = ar[A.na] = 0.0f; if (BWD) gh[A.S] = 0.0f; }
    __syncthreads();
    if (FWD || acted) {                     // (the same for the whole workgroup)
        int over = 0;
        walk_lists<4>(A.cols, 0, col_chunks, first_cols,
                      [&](uint32_t t, float acc) { return __builtin_fmaf(ar[t & 0xffffu], rows[A.na + (t >> 16)], acc); },
                      [&](int c, float v) { pre[c] = v; over |= !(v <= 1.0f); }, [](int) {});
        __syncthreads();
        if (FWD) {
            for (int u = tid; u < A.n3; u += T) {
                const int i = A.ia[u], j = A.ib[u];
                const float x = i >= 0 ? fminf(pre[i], 1.0f) : 0.0f, y = j >= 0 ? cr[j] : 0.0f;
                float v = i >= 0 ? x : y;
                if (i >= 0 && j >= 0) {
                    v = x + y;
                    over |= !(v <= 1.0f);
                    v = fminf(v, 1.0f);
                }
                A.out[s * A.n3 + u] = v;
            }
            acted = __syncthreads_or(over);
            if (A.saved && tid == 0) A.saved[s] = acted ? 1 : 0;
        }
    }
    if (!BWD) return;
    const float *gr = A.g + s * A.n3;
    for (int x = tid; x < A.S; x += T) {    // the gradient that reaches each of the Apply's sums
        const int oc = A.ca[x];
        float v = oc >= 0 ? gr[oc] : 0.0f;
        if (acted && oc >= 0) {
            const int j = A.ib[oc];
            if (!(pre[x] <= 1.0f) || (j >= 0 && !(fminf(pre[x], 1.0f) + cr[j] <= 1.0f))) v = 0.0f;
        }
        gh[x] = v;
    }
    if (A.gc)
        for (int j = tid; j < A.nc; j += T) {
            const int oc = A.cb[j];
            float v = oc >= 0 ? gr[oc] : 0.0f;
            if (acted && oc >= 0) {
                const int i = A.ia[oc];
                if (i >= 0 && !(fminf(pre[i], 1.0f) + cr[j] <= 1.0f)) v = 0.0f;
            }
            float *dst = A.gc + s * A.nc + j;
            *dst = (A.accumulate & 4) ? *dst + v : v;
        }
    __syncthreads();
    walk_lists<8>(A.rows, 0, row_chunks, first_rows, [&](uint32_t t, float acc) { return __builtin_fmaf(gh[t >> 16], rows[t & 0xffffu], acc); },
                  [&](int x, float v) {
                      const bool is_a = x < A.na;
                      if (is_a ? !A.ga : !A.gb) return;
                      float *dst = is_a ? A.ga + s * A.na + x : A.gb + s * A.nb + (x - A.na);
                      *dst = (A.accumulate & (is_a ? 1 : 2)) ? *dst + v : v;
                  }, [](int) {});
}

// ---------------------------------------------------------------- which tables, which launch

static unsigned threads_for(int64_t work, int most)
{
    const int64_t t = (work + kWave - 1) / kWave * kWave;
    return static_cast<unsigned>(std::max<int64_t>(kWave, std::min<int64_t>(most, t)));
}

// The same for `work` steps that a workgroup takes `most` at a time, shared out evenly.
static unsigned even_threads(int64_t work, int most)
{
    const int64_t turns = std::max<int64_t>(1, (work + most - 1) / most);
    return threads_for((work + turns - 1) / turns, most);
}

static Lists lists_of(const ListPlan &p)
{
    return Lists{p.order.ptr, p.ptr.ptr, p.words.ptr, p.longer.ptr, p.n_huge, p.n_wave, p.n_mid};
}

// Workgroups of one launch: it may have 2^32 - 1 threads.  Larger batches go in several.
constexpr int32_t kMostGroups = 0xffffffffu / kSampleThreads;

// Threads for n lists (a lane each, eight for one that 16 lanes sum) beside the copying of a row: 2 048 for all the workgroups
// that a unit gets of the launch, or has LDS for.  A workgroup's phases run one after the other, those of several side by
// side, so more than one to a unit shall mean smaller ones, down to `least` threads.  (B=4 000, us, with 1 024 / 512 / 256 / 128
// threads, LDS for 14 workgroups, rows of 40 and of 700 tuples: backward 356 / 196 / 131 / 139, forward 47 / 41 / 41 / 49;
// 1 200 x 7 -> 6 500, LDS for seven: forward 60 / 49 / 50 / 75; 9 000 x 20 -> 9 000, LDS for two: backward 627 / 755 / 1 189.)
static unsigned list_threads(const ListPlan &p, int32_t n, int32_t row, int64_t groups, size_t lds, int least)
{
    const int64_t held = std::max<int64_t>(1, std::min<int64_t>((groups + kUnits - 1) / kUnits, static_cast<int64_t>(160 * 1024 / (lds + 1024))));
    const int64_t share = held >= 16 ? 128 : held >= 8 ? 256 : held >= 4 ? 512 : kSampleThreads;
    return threads_for(std::max<int64_t>(n + 8 * static_cast<int64_t>(p.n_mid), row / 4),
                       static_cast<int>(std::min<int64_t>(kSampleThreads, std::max<int64_t>(least, share))));
}

// Parts of a sample's output row, at most `most`: a workgroup copies `row` floats and then does work(p) floats' worth of
// gathers when there are p of them; the grid runs in rounds of what the chip holds at once (256 compute units, 2 048 threads
// and 160 KB of LDS each), and a round that is nearly empty costs as much as a full one.
template <typename Work>
static int32_t best_parts(int64_t batch, int most, double row, Work work, unsigned threads, size_t lds)
{
    const int64_t held = kUnits * std::max<int64_t>(1, std::min<int64_t>(2048 / threads, static_cast<int64_t>(160 * 1024 / (lds + 1024))));
    int32_t best = 1;
    double best_cost = 0.0;
    for (int p = 1; p <= most && batch * p <= kMostGroups; ++p) {
        const double cost = static_cast<double>((batch * p + held - 1) / held) * (row + 1500.0 + work(p));
        if (p == 1 || cost < 0.97 * best_cost) { best = p; best_cost = cost; }
    }
    return best;
}

// As many parts as the longer columns keep busy (64 of 16 lanes each, or 16 of a wavefront, to a part), at least `least`.
static int long_parts(const ListPlan &p, int least) { return std::max(least, std::min(64, p.n_mid / 64 + p.n_wave / 16)); }

static size_t list_fwd_bytes(const dol_fn_table *f, bool results)
{
    return sizeof(float) * (static_cast<size_t>((f->na + 4) & ~3) + ((f->nb + 4) & ~3) + (results ? std::min((f->n_out + 3) & ~3, kOrderBlock) : 0));
}

static size_t gated_bytes(const dol_fn_table *f) { return sizeof(float) * static_cast<size_t>((f->n_out + 4) & ~3); }

// Tables that tiles of samples serve as well (damp_lds.hip, damp_table.hip) have every column added up in the order of its
// tuples, as the tiles do, so that a sample's result does not depend on the batch it is in: through the lists, long columns by
// a chain.  (The map goes one j at a time.)
static bool exact_fwd(const dol_fn_table *f) { return f->lds_fwd_ok || table_code_ok(f); }

bool byj_fwd_sample_ok(const dol_fn_table *f)
{
    return f->byj_fwd && !exact_fwd(f) && sizeof(float) * static_cast<size_t>(f->na + 4) <= kStageMaxBytes;
}

bool list_fwd_sample_ok(const dol_fn_table *f) { return f->lists_ok && list_fwd_bytes(f, false) <= kStageMaxBytes; }

// (without the maps' long rows of b the lists have a lane for every row: 16 x 16 -> 32, B=4 096, 7.5 us through the map, 5.0
// through the lists; 101 x 10 6.5 and 8.3)
bool byj_bwd_sample_ok(const dol_fn_table *f) { return f->byj_ok && (f->byj_nbp <= 4 || f->row_lists.longer.n > 0); }

bool byj_bwd_staged(const dol_fn_table *f) { return gated_bytes(f) <= kStageMaxBytes; }

bool list_bwd_sample_ok(const dol_fn_table *f) { return f->lists_ok && gated_bytes(f) <= kStageMaxBytes; }

#define DOL_DISPATCH_NBP(nbp, CALL) \
    switch (nbp) {                  \
    case 4: CALL(4); break;         \
    case 8: CALL(8); break;         \
    case 10: CALL(10); break;       \
    default: CALL(16); break;       \
    }

// The launch of the dense-map kernels over rows of at least kStageMinRow tags takes up to 1 024 threads, over shorter
// rows up to 256 (two or more workgroups share a compute unit then).
bool byj_fwd_wide(const dol_fn_table *f) { return f->na >= kStageMinRow; }
bool byj_bwd_wide(const dol_fn_table *f) { return f->na + f->nb > 1024; }

template <int NBP, bool FALLING>
static void (*byj_fwd_kernel(bool wide, bool huge))(SampleFwd)
{
    if (wide) return huge ? &damp_byj_fwd_staged_kernel<NBP, FALLING, true> : &damp_byj_fwd_staged_kernel<NBP, FALLING, false>;
    return huge ? &damp_byj_fwd_kernel<NBP, FALLING, true> : &damp_byj_fwd_kernel<NBP, FALLING, false>;
}

dol_status launch_sample_fwd(const dol_fn_table *f, int32_t batch, const float *a, int64_t lda, const float *b, int64_t ldb, float *out,
                             int64_t ldo, hipStream_t st, bool *done)
{
    *done = false;
    const bool byj = byj_fwd_sample_ok(f);
    if (!byj && !list_fwd_sample_ok(f)) return DOL_OK;
    for (; batch > kMostGroups; batch -= kMostGroups, a += kMostGroups * lda, b += kMostGroups * ldb, out += kMostGroups * ldo)
        if (dol_status s = launch_sample_fwd(f, kMostGroups, a, lda, b, ldb, out, ldo, st, done)) return s;
    SampleFwd A{};
    A.na = f->na, A.nb = f->nb, A.S = f->n_out;
    A.a = a, A.lda = lda, A.b = b, A.ldb = ldb, A.out = out, A.ldo = ldo;
    A.col_ptr = f->col_ptr.ptr, A.col_ij = f->col_ij.ptr;
    A.lists = lists_of(f->col_lists);
    if (byj) {
        A.map = f->byj_src.ptr, A.map_ld = f->byj_src_ld;
        A.long_weight = static_cast<int32_t>(std::min<int64_t>(f->col_lists.huge_words / f->byj_nbp, f->n_out));
        const size_t lds = sizeof(float) * static_cast<size_t>(f->na + 4);
        A.parts = best_parts(batch, long_parts(f->col_lists, std::min(16, (f->n_out + 4 * kSmallThreads - 1) / (4 * kSmallThreads))), f->na,
                             [&](int p) { return (static_cast<double>(f->n_out + A.long_weight) * f->byj_nbp + 4.0 * f->col_lists.mid_words) / p; },
                             byj_fwd_wide(f) ? kSampleThreads : kSmallThreads, lds);
        A.shared = shared_ranges(batch, A.parts, f->na);
        const dim3 grid(static_cast<unsigned>(batch) * A.parts);
        const dim3 block(threads_for(std::max<int64_t>(f->n_out / A.parts + 3, f->na) / 4, byj_fwd_wide(f) ? kSampleThreads : kSmallThreads));
        // (a column that long_sum would take in one step has nothing to ask for ahead: 785 x 10 -> 1 297 4.9 us, 4.7 without)
        const int32_t huge_col = f->col_lists.only_huge;
        A.huge = huge_col >= 0 && f->h_col_ptr[huge_col + 1] - f->h_col_ptr[huge_col] > 4 * block.x ? huge_col : -1;
        if (A.huge >= 0) A.huge_q0 = f->h_col_ptr[A.huge], A.huge_q1 = f->h_col_ptr[A.huge + 1];
#define CALL(N)                                                                                                                \
    {                                                                                                                          \
        const bool wide = byj_fwd_wide(f), huge = A.huge >= 0;                                                                 \
        const auto kernel = f->byj_falling ? byj_fwd_kernel<N, true>(wide, huge) : byj_fwd_kernel<N, false>(wide, huge);       \
        if (lds > 48 * 1024) DOL_HIP(allow_dynamic_lds(reinterpret_cast<const void *>(kernel), kStageMaxBytes));               \
        hipLaunchKernelGGL(kernel, grid, block, lds, st, A);                                                                   \
    }
        DOL_DISPATCH_NBP(f->byj_nbp, CALL)
#undef CALL
    } else {
        // (stored where they fall the results of lists of many lengths dirty every line many times over: 1 200 x 30 -> 6 500,
        // 5.5 words to a list, B=4 000 79 us against 63.  Lists of one or two words are in column order but for a few: 1 200 x 7
        // -> 6 500 44 against 49, 800 x 3 -> 2 400 21 against 24.  Nor is there room beside rows of more than 36 000 symbols.)
        const bool results = list_fwd_bytes(f, true) <= kStageMaxBytes && f->col_lists.n_words >= 3 * static_cast<size_t>(f->n_out);
        A.exact = exact_fwd(f) ? 1 : 0;
        const size_t lds = list_fwd_bytes(f, results);
        const int blocks = (f->n_out + kOrderBlock - 1) / kOrderBlock;
        A.parts = best_parts(batch, long_parts(f->col_lists, blocks), f->na + f->nb, [&](int p) {
            return (2.0 * f->col_lists.n_words + f->n_out) / std::min(p, blocks) + 4.0 * f->col_lists.mid_words / p + 2.0 * f->col_lists.huge_words;
        }, kSampleThreads, lds);
        unsigned threads = list_threads(f->col_lists, f->n_out, f->na, batch * static_cast<int64_t>(A.parts), lds, 512);
        if (A.exact && f->col_lists.longer.n && threads < kSampleThreads) threads += kWave;        // (the chain runs beside the lists)
        A.shared = shared_ranges(batch, A.parts, f->na);
        const dim3 grid(static_cast<unsigned>(batch) * A.parts), block(threads);
        if (results) {
            if (lds > 48 * 1024) DOL_HIP(allow_dynamic_lds(reinterpret_cast<const void *>(damp_apply2_fwd_staged_kernel<true>), kStageMaxBytes));
            hipLaunchKernelGGL(damp_apply2_fwd_staged_kernel<true>, grid, block, lds, st, A);
        } else {
            DOL_HIP(allow_dynamic_lds(reinterpret_cast<const void *>(damp_apply2_fwd_staged_kernel<false>), kStageMaxBytes));
            hipLaunchKernelGGL(damp_apply2_fwd_staged_kernel<false>, grid, block, lds, st, A);
        }
    }
    DOL_HIP(hipGetLastError());
    *done = true;
    return DOL_OK;
}

template <int C, int N>
static void (*apply1_fwd_kernel(const ListPlan &lists))(SampleFwd)
{
    return lists.lane_words > static_cast<int32_t>(kPlainWords) ? &damp_apply1_fwd_staged_kernel<C, N, true> : &damp_apply1_fwd_staged_kernel<C, N, false>;
}

dol_status launch_unary_fwd(int32_t n_in, int32_t S, const ListPlan &lists, const uint32_t *col_ptr, const uint32_t *col_ij, int32_t batch,
                            const float *x, int64_t ldx, float *out, int64_t ldo, hipStream_t st)
{
    for (; batch > kMostGroups; batch -= kMostGroups, x += kMostGroups * ldx, out += kMostGroups * ldo)
        if (dol_status s = launch_unary_fwd(n_in, S, lists, col_ptr, col_ij, kMostGroups, x, ldx, out, ldo, st)) return s;
    SampleFwd A{};
    A.na = n_in, A.nb = 1, A.S = S, A.a = x, A.lda = ldx, A.out = out, A.ldo = ldo;
    A.col_ptr = col_ptr, A.col_ij = col_ij, A.lists = lists_of(lists);
    const size_t lds = sizeof(float) * static_cast<size_t>((n_in + 4) & ~3);
    // (more parts than their lists fill, for lists that take several lanes most of all, only while each has a unit to itself: one sample
    // of 24 000 -> 16 24.8 / 10.1 us, 40 400 -> 68 10.3 / 8.1; 12 000 -> 11 995 16 samples in 16 parts 4.0, in 24 4.7)
    const int halves = (2 * S + kSampleThreads - 1) / kSampleThreads, few = lists.n_mid / 16 + lists.n_wave / 4 + lists.n_huge;
    const int most = std::max(long_parts(lists, std::min(16, halves)), std::min(std::min(40, kUnits / batch), std::max(halves, few)));
    A.parts = best_parts(batch, most, n_in, [&](int p) {
        const double huge = lists.n_huge > 0 ? static_cast<double>((lists.n_huge + p - 1) / p) / lists.n_huge : 0.0;     // one part's share
        return (2.0 * lists.n_words + S + 4.0 * lists.mid_words) / p + 2.0 * lists.huge_words * huge;
    }, kSampleThreads, lds);
    A.shared = shared_ranges(batch, A.parts, n_in);
    const unsigned threads = list_threads(lists, S, n_in, batch * static_cast<int64_t>(A.parts), lds, 512);
    // (us, two chunks of two words a step, one of three, one of eight: a permutation of 38 400, one word to a list, B=200 26.1, 32.1, 42.0;
    // 38 400 -> 7 679, three words to every list, B=16 5.0, 4.6, 5.0, B=600 33.0, 32.2, 39.3; -> 4 267, five, B=600 28.4, 30.0, 30.1,
    // B=16 5.1, 4.7, 4.9; -> 2 743, seven, B=600 27.6, 28.9, 25.7; -> 8 333, one to 47 words and three on average, B=200 20.6, 17.1, 14.9)
    const int64_t words = static_cast<int64_t>(lists.n_words), n = S;
    const auto kernel = lists.lane_words < 6 ? (2 * words < 5 * n ? apply1_fwd_kernel<2, 2>(lists) : apply1_fwd_kernel<1, 3>(lists))
                                             : words < 2 * n ? apply1_fwd_kernel<2, 2>(lists) : apply1_fwd_kernel<1, 8>(lists);
    if (lds > 48 * 1024) DOL_HIP(allow_dynamic_lds(reinterpret_cast<const void *>(kernel), kStageMaxBytes + 16));
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(batch) * A.parts), dim3(threads), lds, st, A);
    DOL_HIP(hipGetLastError());
    return DOL_OK;
}

dol_status launch_unary_bwd(int32_t n_in, int32_t S, const uint16_t *pick, const uint32_t *col_ptr, const uint32_t *col_ij, const float *one, int32_t batch,
                            const float *x, int64_t ldx, const float *out, int64_t ldo, const float *g, int64_t ldg, float *gx, hipStream_t st)
{
    for (; batch > kMostGroups; batch -= kMostGroups, x += kMostGroups * ldx, out += kMostGroups * ldo, g += kMostGroups * ldg, gx += kMostGroups * ldx)
        if (dol_status s = launch_unary_bwd(n_in, S, pick, col_ptr, col_ij, one, kMostGroups, x, ldx, out, ldo, g, ldg, gx, st)) return s;
    SampleBwd A{};
    A.na = n_in, A.nb = 1, A.S = S, A.map = pick, A.col_ptr = col_ptr, A.col_ij = col_ij;
    A.a = x, A.lda = ldx, A.b = one, A.out = out, A.ldo = ldo, A.g = g, A.ldg = ldg, A.ga = gx;
    // (while each part has a unit to itself: one sample of 38 400 -> 8 333 in parts of 4 096 symbols 3.9 us, of 1 024 3.8; -> 26 3.3 and 3.0)
    const int32_t parts = std::max(1, std::min((n_in + kSampleThreads - 1) / kSampleThreads, kUnits / batch)), fours = (std::max((n_in + parts - 1) / parts, S) + 3) / 4;
    const size_t lds = sizeof(float) * static_cast<size_t>((S + 4) & ~3);
    DOL_HIP(allow_dynamic_lds(reinterpret_cast<const void *>(damp_apply1_bwd_staged_kernel), kStageMaxBytes + 16));
    hipLaunchKernelGGL(damp_apply1_bwd_staged_kernel, dim3(static_cast<unsigned>(batch) * parts), dim3(threads_for(fours, kSampleThreads)), lds, st, A, parts,
                       shared_ranges(batch, parts, S));
    DOL_HIP(hipGetLastError());
    return DOL_OK;
}

dol_status launch_sample_bwd(const dol_fn_table *f, int32_t batch, const float *a, int64_t lda, const float *b, int64_t ldb,
                             const float *out, int64_t ldo, const float *g, int64_t ldg, float *ga, float *gb, int32_t accumulate,
                             hipStream_t st, bool *done)
{
    *done = false;
    const bool byj = byj_bwd_sample_ok(f);
    if (!byj && !list_bwd_sample_ok(f)) return DOL_OK;
    for (; batch > kMostGroups; batch -= kMostGroups) {
        if (dol_status s = launch_sample_bwd(f, kMostGroups, a, lda, b, ldb, out, ldo, g, ldg, ga, gb, accumulate, st, done)) return s;
        a += kMostGroups * lda, b += kMostGroups * ldb, out += kMostGroups * ldo, g += kMostGroups * ldg;
        if (ga) ga += kMostGroups * lda;
        if (gb) gb += kMostGroups * ldb;
    }
    SampleBwd A{};
    A.na = f->na, A.nb = f->nb, A.S = f->n_out;
    A.a = a, A.lda = lda, A.b = b, A.ldb = ldb, A.out = out, A.ldo = ldo, A.g = g, A.ldg = ldg, A.ga = ga, A.gb = gb;
    A.accumulate = accumulate;
    A.col_ptr = f->col_ptr.ptr, A.col_ij = f->col_ij.ptr;
    A.lists = lists_of(f->row_lists);
    size_t lds = gated_bytes(f);
    const dim3 grid(static_cast<unsigned>(batch));
    if (byj) {
        A.map = f->byj_col.ptr, A.map_ld = f->byj_col_ld;
        const int64_t work = std::max(f->na, f->n_out) / 4 + 1;
        if (!byj_bwd_staged(f)) {
            lds = sizeof(uint32_t) * static_cast<size_t>((f->n_out + 31) / 32);
#define CALL(N) hipLaunchKernelGGL(damp_byj_bwd_global_kernel<N>, grid, dim3(threads_for(work, kSampleThreads)), lds, st, A)
            DOL_DISPATCH_NBP(f->byj_nbp, CALL)
#undef CALL
        } else if (byj_bwd_wide(f)) {
            const bool shared = batch > kUnits && 2 * (lds + 2048) <= 160 * 1024;
            const int most = !shared || f->byj_nbp <= 4 ? kSampleThreads : f->byj_nbp <= 10 ? 768 : 512;
#define CALL(N)                                                                                                                \
    {                                                                                                                          \
        if (lds > 48 * 1024) DOL_HIP(allow_dynamic_lds(reinterpret_cast<const void *>(damp_byj_bwd_row_kernel<N>), kStageMaxBytes));   \
        hipLaunchKernelGGL(damp_byj_bwd_row_kernel<N>, grid, dim3(even_threads(work, most)), lds, st, A);                      \
    }
            DOL_DISPATCH_NBP(f->byj_nbp, CALL)
#undef CALL
        } else {
#define CALL(N)                                                                                                                \
    {                                                                                                                          \
        if (lds > 48 * 1024) DOL_HIP(allow_dynamic_lds(reinterpret_cast<const void *>(damp_byj_bwd_kernel<N>), kStageMaxBytes));   \
        hipLaunchKernelGGL(damp_byj_bwd_kernel<N>, grid, dim3(threads_for(work, kSmallThreads)), lds, st, A);                  \
    }
            DOL_DISPATCH_NBP(f->byj_nbp, CALL)
#undef CALL
        }
    } else {
        A.rowa_ptr = f->rowa_ptr.ptr, A.rowa_jc = f->rowa_jc.ptr, A.rowb_ptr = f->rowb_ptr.ptr, A.rowb_ic = f->rowb_ic.ptr;
        const size_t with_rows = lds + sizeof(float) * static_cast<size_t>(f->na + f->nb + 1);
        const dim3 block(list_threads(f->row_lists, f->na + f->nb, f->n_out, batch, with_rows <= kStageMaxBytes ? with_rows : lds, 128));
        if (with_rows <= kStageMaxBytes) {
            if (with_rows > 48 * 1024) DOL_HIP(allow_dynamic_lds(reinterpret_cast<const void *>(damp_apply2_bwd_staged_kernel<true>), kStageMaxBytes));
            hipLaunchKernelGGL(damp_apply2_bwd_staged_kernel<true>, grid, block, with_rows, st, A);
        } else {
            if (lds > 48 * 1024) DOL_HIP(allow_dynamic_lds(reinterpret_cast<const void *>(damp_apply2_bwd_staged_kernel<false>), kStageMaxBytes));
            hipLaunchKernelGGL(damp_apply2_bwd_staged_kernel<false>, grid, block, lds, st, A);
        }
    }
    DOL_HIP(hipGetLastError());
    *done = true;
    return DOL_OK;
}

// What a launch with a workgroup per sample takes, in us, for the choice against tiles of 64 samples, whose time does not
// depend on how many tiles there are until each compute unit has one (struct dol_fn_table: tile_fwd_us, tile_bwd_us).  Wavefronts
// come and go at a rate, lists cost by their words, long ones more: fitted to 36 tables from 4 x 4 -> 4 to 442 x 10 -> 785 at 16
// to 8 192 samples, most within 20 %; dense maps' rows come out up to 1.6 times too long, far from the tiles' time.
static double sample_fwd_us(const dol_fn_table *f, int64_t batch)
{
    const ListPlan &p = f->col_lists;
    const double waves = list_threads(p, f->n_out, f->na, batch, list_fwd_bytes(f, true), 512) / static_cast<double>(kWave);
    const double n_long = static_cast<double>(p.longer.n), longer = p.huge_words + p.mid_words + 48.0 * n_long;   // (in 64s)
    const double chain = n_long > 0 ? std::ceil(n_long / (4.0 * waves)) * longer / n_long : 0.0;                    // one wavefront's
    return 3.4 + 7.5e-3 * chain + 0.18e-3 * p.n_words + 0.31e-3 * std::max(0.0, batch * waves - 1500.0) +
           batch * (0.86e-6 * longer + 0.18e-6 * p.n_words);
}

static double sample_bwd_us(const dol_fn_table *f, int64_t batch)
{
    const ListPlan &p = f->row_lists;
    const double waves = list_threads(p, f->na + f->nb, f->n_out, batch, gated_bytes(f), 128) / static_cast<double>(kWave);
    return 3.8 + 0.11e-3 * p.n_words + 0.21e-3 * std::max(0.0, batch * waves - 1500.0) +
           batch * (0.44e-6 * (p.huge_words + p.mid_words) + 0.13e-6 * p.n_words);
}

// Tables that damp_lds.hip tiles: a workgroup per sample where that is faster.  (Tiles against samples, us: 50 x 37 -> 201
// forward B=64 10.3 / 4.3, 4 096 11.0 / 10.2, 8 192 11.4 / 18.2, backward 4 096 15.1 / 8.8, 8 192 15.3 / 15.3; 128 x 128 -> 200
// forward B=64 33 / 9, 1 024 34 / 34, 4 096 33 / 134; 300 x 8 -> 20 forward 2 048 23 / 11, 8 192 23 / 32; 13 x 12 -> 30 backward
// 4 096 7.5 / 5.1.  Above 8 192 samples, or 4 096 without a dense map, tiles: from there each sample costs more than its share.)
bool lds_small_batch(const dol_fn_table *f, int64_t batch, bool backward)
{
    if (batch < 1 || !(backward ? byj_bwd_sample_ok(f) || list_bwd_sample_ok(f) : list_fwd_sample_ok(f))) return false;
    if (batch > (f->byj_ok ? 8192 : 4096)) return false;
    return backward ? sample_bwd_us(f, batch) < f->tile_bwd_us : sample_fwd_us(f, batch) < f->tile_fwd_us;
}

// Tables with generated code (damp_table.hip): whether another kernel takes the call.  Rows of whole 16-byte pieces (64 x 64 -> 256
// forward 4.3 us and a workgroup per sample 4.1 to 4.6 up to 512 samples, smaller tables 2.8 and 3.5): forward never, backward while
// a workgroup per sample is estimated below a time of tiles of 64 samples.  With eight wavefronts to a tile, or 32 samples, tiles
// are faster than that time, and the kernels break even earlier than the line, us, samples / tiles: 64 x 64 -> 256 B=256 4.7 / 8.6,
// 2 048 8.0 / 8.7, 3 072 10.8 / 8.8, 4 096 13.3 / 8.8; 48 x 48 -> 512 2 048 7.9 / 9.7, 4 096 12.1 / 10.2; 32 x 40 -> 128 1 024 4.6 / 5.2,
// 2 048 5.6 / 5.3, 4 096 7.9 / 5.4; 16 x 16 -> 32 3.2 / 2.7.  Up to the line a backward call has no compiler to wait for.
// Other rows, gathers / generated code, forward and backward: from 2^24 multiply-adds a pass on, 50 x 37 -> 201 B=9 069 12.0 / 5.6
// and 15.8 / 9.4, 72 552 57 / 22 and 65 / 33; 61 x 5 -> 76 55 008 19 / 10 and 55 / 14; an eighth of 63 x 61 -> 216 35 621 22.9 / 14.5 and
// 33 / 21; 33 x 47 -> 784 10 818 20 / 9.4 and 25 / 15.7.  The first pass of a direction and a range of batches (of two or three, build_for)
// waits for the compiler, 0.11 to 0.37 s forward, 0.16 to 1.4 backward: at the line the gain of 20 000 to 200 000 passes, as for
// whole pieces, where it is so at any size.  The line leaves calls of less work to kernels that need no compiler.
bool table_small_batch(const dol_fn_table *f, int64_t batch, bool backward)
{
    const bool whole = whole_pieces(f);
    if (!whole && batch < (int64_t{1} << 24) / std::max<int64_t>(1, f->n_tuples)) return true;
    if (!backward || batch < 1 || batch > (whole ? 4096 : 8192) || !(byj_bwd_sample_ok(f) || list_bwd_sample_ok(f))) return false;
    if (!whole && f->lds_bwd_ok) return false;                      // (tiles of damp_lds.hip would take it)
    const double tiles = 3.0 + 2.5e-3 * static_cast<double>(f->n_tuples) + 6e-3 * f->n_out;
    return sample_bwd_us(f, batch) < tiles;
}

// What damp_merge_sample_kernel keeps in LDS: besides the table's rows the whole second Distribution, of up to 65 535 symbols.
static size_t merge_bytes(const dol_fn_table *f, const UnionPlan *p)
{
    return sizeof(float) * (static_cast<size_t>((2 * f->na + f->nb + 5) & ~3) + f->n_out + p->nb + f->n_out + 1);
}

// Apply + Filter + Union, a workgroup per sample / tiles, us, forward, backward, both in one launch.  64 x 64 -> 256 B=512 4.3 / 8.3, 5.8 / 12.1,
// 7.9 / 15.9, 2 048 6.5 / 8.5, 8.8 / 12.5, 14.1 / 16.9, 3 072 8.5 / 8.6, 12.9 / 12.7, 19.0 / 17.5, 4 096 10.8 / 9.1, 16.0 / 13.2, 24.4 / 18.0
// (where the plan is not aligned, 4 096 10.6 / 9.3, 15.9 / 13.6, 24.5 / 22.5); 32 x 40 -> 128 2 048 4.6 / 5.5, 6.0 / 6.7, 7.9 / 8.6, 3 072 5.3 / 5.6,
// 7.2 / 6.8, 9.5 / 8.8.  So the line of two calls; one call breaks even from 2 048 samples on, the soonest with a wide result (16 x 64 -> 400 1 024
// 10.5 / 15.7, 2 048 19.0 / 16.7, 3 072 26.0 / 17.3; 48 x 48 -> 512 20.5 / 21.1, 28.4 / 22.0), but up to the line waits for no compiler.
// Only tables of which a lane walks every list: their sums are then the tiles' bit for bit.  What does not fit LDS is left to the
// tiles, which read the second Distribution from memory; where only one workgroup fits a unit its turns end the gain earlier
// (32 x 40 -> 128 and 40 000 symbols: tiles / samples, B=2 048 1 017 / 943, 3 072 1 079 / 1 409).
bool merge_small_batch(const dol_fn_table *f, const UnionPlan *p, int64_t batch)
{
    const size_t bytes = merge_bytes(f, p);
    return f->lists_ok && f->col_lists.longer.n == 0 && f->row_lists.longer.n == 0 && bytes <= kStageMaxBytes &&
           batch <= (2 * bytes <= 160 * 1024 ? 3072 : 2048);
}

dol_status launch_sample_merge(const dol_fn_table *f, const UnionPlan *p, int32_t batch, const float *a, const float *b, const float *c,
                               float *out, int32_t *saved, const float *g, float *ga, float *gb, float *gc, int32_t accumulate, hipStream_t st)
{
    SampleMerge A{};
    A.na = f->na, A.nb = f->nb, A.S = f->n_out, A.nc = p->nb, A.n3 = p->n_out, A.accumulate = accumulate;
    A.cols = lists_of(f->col_lists), A.rows = lists_of(f->row_lists);
    A.ia = p->d_ia.ptr, A.ib = p->d_ib.ptr, A.ca = p->d_ca.ptr, A.cb = p->d_cb.ptr;
    A.a = a, A.b = b, A.c = c, A.g = g, A.out = out, A.ga = ga, A.gb = gb, A.gc = gc, A.saved = saved;
    const size_t lds = merge_bytes(f, p);
    const dim3 grid(static_cast<unsigned>(batch)), block(threads_for(std::max(std::max(f->n_out, f->na + f->nb), p->n_out / 2), 512));
    auto launch = [&](void (*kernel)(SampleMerge)) -> dol_status {
        if (lds > 48 * 1024) DOL_HIP(allow_dynamic_lds(reinterpret_cast<const void *>(kernel), kStageMaxBytes));
        hipLaunchKernelGGL(kernel, grid, block, lds, st, A);
        DOL_HIP(hipGetLastError());
        return DOL_OK;
    };
    if (out && g) return launch(damp_merge_sample_kernel<true, true>);
    if (out) return launch(damp_merge_sample_kernel<true, false>);
    return launch(damp_merge_sample_kernel<false, true>);
}

}  // namespace dol
