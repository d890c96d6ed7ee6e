// The iteration kernels (iterate.hip) for tables shaped like a grid: node c of a grid w wide takes part in the tuples of its
// column with itself and with each of its neighbours c - w, c - 1, c + 1, c + w, and in no others, as one round of
// reachability with a "stay" symbol does.
//
// A workgroup owns a sample, a lane a strip of R nodes, one above the other; as many bands of strips as fit lie side by side
// in a wavefront, and no band is cut.  The general kernels read a node's five operands from LDS, with a barrier after every
// round: two serial phases of that much, LDS and arithmetic, and the barrier's own time.  Here a lane keeps its nodes' tags
// (the gradients that reach them, in the reverse rounds) in registers: within the strip a node's upper and lower neighbour
// are the lane's own, left and right come from the lanes beside it (a shift of the wavefront inside the instruction), and
// only the strip's two ends are exchanged through LDS.  What the reverse sweep needs of the rounds, the lane's own tags, lies
// in LDS as one vector per lane and round.
//
// A neighbour that is not there is an exact 0 (masked), so the sums, in ascending order of the operand's symbol, are those of
// the general kernels bit for bit.  Nodes past the grid (the last strips' ends, lanes without a strip) have the tag 1 and a
// product of 2 with themselves: they are clamped in every round, no gradient leaves them.
//
// Bound by the chain of a round - ends from LDS, five sums one after the other, ends to LDS, barrier: 0.17 us in a
// forward round and 0.18 to 0.20 in a reverse round at 32 x 32 (what 8 to 64 rounds take more), where the arithmetic alone would
// take 0.07 and 0.12 - up to one sample per unit, then by the arithmetic.  Flags in the exchanged words instead of barriers were slower (polling takes more
// instructions than it saves waits), and so were the shares added up a round late.
// Both sweeps of 64 rounds, general kernels and these: 8 x 8 grid, B = 256 33.2 and 15.8 us; 16 x 16 27.2 and 21.2;
// 32 x 32 39.3 and 30.1; B = 1024 8 x 8 78 and 18, 16 x 16 74 and 29, 32 x 32 134 and 83.
// (32 x 32: LDS holds the tags of half the rounds.  With one sample to a unit the registers hold the other half, and no round
// is run forward twice: 35.3 us with 32 rounds replayed from a checkpoint, 30.1 so.)
#include "iterate.h"

namespace dol {

namespace {

// Operand slots of a node in ascending symbol order.
enum { kUp, kLeft, kSelf, kRight, kDown, kSlots };

constexpr int kMaxWaves = 8;
constexpr int kUnits = 256;             // compute units

// How a grid lies in a workgroup.
struct GridLayout {
    int32_t w, h;
    int32_t per_wave;                   // bands side by side in a wavefront
    int32_t bands;                      // of R rows each
    __host__ __device__ int strips() const { return bands * w; }
};

// LDS, in floats: two rows of strip ends, a word per thread that goes down and one that goes up; then a row of tags per
// round, R per strip (and R for the lanes without one).
template <int R>
struct Rows {
    static __host__ __device__ int tags(int threads) { return 4 * threads; }                                // where the first row of tags is
    static __host__ __device__ int tag_row(const GridLayout &g) { return (g.strips() + 1) * R; }
};

// Where a lane's strip is: byte addresses of the words it exchanges, in even or in odd rounds.
struct Ends {
    uint32_t up, down;                  // what the strips above and below have to say (its own, where there is none)
    uint32_t top, bottom;               // where this strip says it
};

template <int R>
struct Strip {
    int node, w, n_valid;               // first node; how many of the R are nodes of the grid
    uint32_t from_left, from_right, from_up, from_down;     // bits of a neighbour's value that count: all or none
    Ends ends[2];
    uint32_t tags, tag_row;

    __device__ __forceinline__ Strip(const GridLayout &g, const float *lds)
    {
        const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, T = blockDim.x;
        const int in_wave = lane / g.w, col = lane - in_wave * g.w, band = wave * g.per_wave + in_wave;
        const bool there = in_wave < g.per_wave && band < g.bands, above = there && band > 0, below = there && band + 1 < g.bands;
        w = g.w;
        node = band * R * w + col;
        n_valid = there ? min(R, g.h - band * R) : 0;
        // (opaque: the shift and the mask are one instruction)
        from_left = fixed_offset(there && col > 0 ? 0xFFFFFFFFu : 0u);
        from_right = fixed_offset(there && col + 1 < w ? 0xFFFFFFFFu : 0u);
        from_up = above ? 0xFFFFFFFFu : 0u;
        from_down = below ? 0xFFFFFFFFu : 0u;
        const int over = in_wave > 0 ? lane - w : (g.per_wave - 1) * w + col - kWave;       // the strip above, relative to the wavefront
        const int under = in_wave + 1 < g.per_wave ? lane + w : col + kWave;
        const uint32_t lds0 = lds_address(lds);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const uint32_t goes_down = lds0 + p * 2 * T * 4u, goes_up = goes_down + T * 4u;
            ends[p].top = goes_up + threadIdx.x * 4u;
            ends[p].bottom = goes_down + threadIdx.x * 4u;
            ends[p].up = above ? goes_down + (wave * kWave + over) * 4u : ends[p].top;
            ends[p].down = below ? goes_up + (wave * kWave + under) * 4u : ends[p].bottom;
        }
        tags = lds0 + (Rows<R>::tags(T) + (there ? band * w + col : g.strips()) * R) * 4u;
        tag_row = Rows<R>::tag_row(g) * 4u;
    }
};

template <int R>
__device__ __forceinline__ void put_ends(const Ends &e, const float (&x)[R])
{
    lds_put(e.bottom, x[R - 1]);
    lds_put(e.top, x[0]);
}

__device__ __forceinline__ float masked(float x, uint32_t mask) { return __uint_as_float(__float_as_uint(x) & mask); }

// A phase begins with x.
template <int R>
__device__ __forceinline__ void begin_phase(const Strip<R> &s, const float (&x)[R])
{
    put_ends(s.ends[0], x);
    lds_barrier();
}

template <int R>
using vec = float __attribute__((ext_vector_type(R)));

template <int R>
__device__ __forceinline__ void put_tags(uint32_t at, const float (&x)[R])
{
    if constexpr (R == 1) lds_put(at, x[0]);
    else {
        vec<R> t;
#pragma unroll
        for (int r = 0; r < R; ++r) t[r] = x[r];
        *reinterpret_cast<__attribute__((address_space(3))) vec<R> *>(static_cast<uintptr_t>(at)) = t;
    }
}

template <int R>
__device__ __forceinline__ void get_tags(uint32_t at, float (&x)[R])
{
    if constexpr (R == 1) x[0] = lds_at(at);
    else {
        const vec<R> t = *reinterpret_cast<const __attribute__((address_space(3))) vec<R> *>(static_cast<uintptr_t>(at));
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = t[r];
    }
}

// x of the lane to the left (right), as far as `mask` lets it through
__device__ __forceinline__ float left_of(float x, uint32_t mask)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x138, 0xF, 0xF, true) & static_cast<int>(mask));    // wave_shr:1
}

__device__ __forceinline__ float right_of(float x, uint32_t mask)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130, 0xF, 0xF, true) & static_cast<int>(mask));    // wave_shl:1
}

// The unclamped sum of the strip's node r, from its tags x and its neighbours' ends.
template <int R>
__device__ __forceinline__ float row_sum(const Strip<R> &s, int r, float up, float down, const float (&x)[R], const float (&k)[R][kSlots])
{
    const float l = left_of(x[r], s.from_left), t = right_of(x[r], s.from_right);
    float acc = __builtin_fmaf(fabsf(r ? x[r ? r - 1 : 0] : up), k[r][kUp], 0.0f);
    acc = __builtin_fmaf(fabsf(l), k[r][kLeft], acc);
    acc = __builtin_fmaf(fabsf(x[r]), k[r][kSelf], acc);
    acc = __builtin_fmaf(fabsf(t), k[r][kRight], acc);
    return __builtin_fmaf(fabsf(r + 1 < R ? x[r + 1 < R ? r + 1 : r] : down), k[r][kDown], acc);
}

// `len` rounds from the tags x, whose ends are in s.ends[0]; KEEP: rows 1, 2, .. of tags (`row`: address of row 1).  At the
// end s.ends[0] is where the last round's ends lie; pre: its unclamped sums.
template <int R, bool KEEP>
__device__ __forceinline__ void rounds(Strip<R> &s, int len, const float (&k)[R][kSlots], float (&x)[R], float (&pre)[R], uint32_t row)
{
    auto one = [&](const Ends &from, const Ends &to) {
        const float up = masked(lds_at(from.up), s.from_up), down = masked(lds_at(from.down), s.from_down);
#pragma unroll
        for (int r = 0; r < R; ++r) pre[r] = row_sum(s, r, up, down, x, k);
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = signed_tag(pre[r]);
        put_ends(to, x);
        if constexpr (KEEP) { put_tags(row, x); row += s.tag_row; }
        lds_barrier();
    };
    for (int t = 0; t + 1 < len; t += 2) {
        one(s.ends[0], s.ends[1]);
        one(s.ends[1], s.ends[0]);
    }
    if (len & 1) {
        one(s.ends[0], s.ends[1]);
        const Ends sw = s.ends[0]; s.ends[0] = s.ends[1]; s.ends[1] = sw;
    }
}

// Rounds whose tags a lane can keep in registers (at one or two wavefronts to a SIMD there are 256 of them).
template <int R>
constexpr int kept_rounds = 68 / R;

template <int R>
using Kept = float[kept_rounds<R>][R];

// (a scalar to compare with here and now: all comparisons of an unrolled loop made ahead fill the scalar registers)
__device__ __forceinline__ int compared(int x)
{
    asm volatile("" : "+s"(x));
    return x;
}

// `len` rounds as rounds() runs them, len <= kept_rounds; the tags that round t starts from are left in kept[t].
template <int R>
__device__ __forceinline__ void rounds_kept(Strip<R> &s, int len, const float (&k)[R][kSlots], float (&x)[R], float (&pre)[R], Kept<R> &kept)
{
#pragma unroll
    for (int t = 0; t < kept_rounds<R>; ++t) {
        if (t >= compared(len)) break;
        const Ends &from = s.ends[t & 1], &to = s.ends[(t + 1) & 1];
        const float up = masked(lds_at(from.up), s.from_up), down = masked(lds_at(from.down), s.from_down);
#pragma unroll
        for (int r = 0; r < R; ++r) kept[t][r] = x[r];
#pragma unroll
        for (int r = 0; r < R; ++r) pre[r] = row_sum(s, r, up, down, x, k);
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = signed_tag(pre[r]);
        put_ends(to, x);
        lds_barrier();
    }
    if (len & 1) { const Ends sw = s.ends[0]; s.ends[0] = s.ends[1]; s.ends[1] = sw; }
}

// A strip's entries in the row of node `first`; past the grid: `else_`.
template <int R>
__device__ __forceinline__ void load_nodes(const Strip<R> &s, const float *__restrict__ row, float else_, float (&x)[R])
{
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = r < s.n_valid ? row[s.node + r * s.w] : else_;
}

// The second operand's symbols in the slots of the strip's nodes (none: where there is none).
template <int R>
__device__ __forceinline__ void load_slots(const Strip<R> &s, const uint32_t *__restrict__ slots, int na, int none, int (&second)[R][kSlots])
{
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int y = 0; y < kSlots; ++y) second[r][y] = r < s.n_valid ? static_cast<int>(slots[y * na + s.node + r * s.w]) : none;
}

template <int R>
__device__ __forceinline__ void take_values(const float *le, const int (&second)[R][kSlots], float (&k)[R][kSlots])
{
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int y = 0; y < kSlots; ++y) k[r][y] = le[second[r][y]];
}

__device__ __forceinline__ void stage(float *le, const float *__restrict__ e, int nb)
{
    for (int j = threadIdx.x; j <= nb; j += blockDim.x) le[j] = j < nb ? e[j] : 0.0f;
}

// Forward sweep.  PRE (both sweeps in one launch): the rounds of the last segment are left in the rows of tags; KEEP: those of
// the segment before it in registers.
template <int R, bool PRE, bool KEEP>
__device__ __forceinline__ void grid_forward(const ItFwdArgs &A, Strip<R> &s, const float (&k)[R][kSlots], Kept<R> &kept)
{
    const int na = A.na;
    const int64_t b = blockIdx.x, plane = static_cast<int64_t>(A.batch) * na;
    auto store = [&](float *row, const float (&v)[R]) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (r < s.n_valid) row[s.node + r * s.w] = v[r];
    };
    float x[R], pre[R];
    load_nodes(s, A.r0 + b * A.ldr, 1.0f, x);
    if (A.hist) store(A.hist + b * na, x);
    if (A.rounds == 0 && A.out) store(A.out + b * A.ldo, x);
    begin_phase(s, x);
    const int stride = A.hist ? 1 : A.every;
    const int t_keep = PRE && A.rounds > 0 ? (A.rounds - 1) / A.every * A.every : A.rounds;    // first round of the kept segment
    const int t_reg = KEEP ? max(0, t_keep - A.every) : t_keep;
    int t = 0, n_ckpt = 0;
    auto leave = [&]() {
        float v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = fminf(pre[r], 1.0f);
        if (A.hist) store(A.hist + t * plane + b * na, v);
        else if (t < A.rounds && A.ckpt) store(A.ckpt + (n_ckpt++) * plane + b * na, v);
        if (t == A.rounds && A.out) store(A.out + b * A.ldo, v);
    };
    while (t < t_reg) {
        const int stop = min(A.rounds, (t / stride + 1) * stride);
        rounds<R, false>(s, stop - t, k, x, pre, 0u);
        t = stop;
        leave();
    }
    if (KEEP && t < t_keep) {
        rounds_kept<R>(s, t_keep - t, k, x, pre, kept);
        t = t_keep;
        leave();
    }
    if constexpr (PRE) {
        if (A.rounds > 0) {
            put_tags(s.tags, x);
            rounds<R, true>(s, A.rounds - t, k, x, pre, s.tags + s.tag_row);
#pragma unroll
            for (int r = 0; r < R; ++r) pre[r] = fminf(pre[r], 1.0f);
            if (A.out) store(A.out + b * A.ldo, pre);
        }
    }
}

// How the shares meet: GridPlan's brief, longer and pos.
struct GridSums {
    const uint2 *brief;
    const uint32_t *longer, *pos;
    int32_t n_longer;
};

// Reverse sweep, a segment of `every` rounds at a time: its rounds forward into the rows of tags, then backwards (the general
// kernel's comment in iterate.hip tells the arithmetic).  KEEP: the last segment but one's tags wait in `kept`, and it is not
// run forward again.
template <int R, bool PRE, bool KEEP>
__device__ __forceinline__ void grid_backward(const ItBwdArgs &A, const GridSums &S, Strip<R> &s, const float (&kc)[R][kSlots],
                                              const float (&kr)[R][kSlots], const Kept<R> &kept, float *share_buf)
{
    const int na = A.na, nb = A.nb, T = blockDim.x;
    const int64_t b = blockIdx.x, plane = static_cast<int64_t>(A.batch) * na;
    float g[R];                                     // the gradient handed over to the segment at hand, not yet gated
    if (!A.target) load_nodes(s, A.gout + b * A.ldg, 0.0f, g);
    else {
        const int target = A.target[b];
        const float at = -1.0f / fmaxf(A.out[b * A.ldo + target], 1.17549435e-38f);
#pragma unroll
        for (int r = 0; r < R; ++r) g[r] = r < s.n_valid && s.node + r * s.w == target ? at : 0.0f;
    }
    float share[R][kSlots];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int y = 0; y < kSlots; ++y) share[r][y] = 0.0f;
    // One round backwards: gh, whose ends are in `from`, to the next one's ends in `to`; xi: the tags it started from.
    auto reverse_round = [&](const Ends &from, const Ends &to, float (&gh)[R], const float (&xi)[R], auto fetch) {
        const float up = lds_at(from.up), down = lds_at(from.down);
        float v[R][kSlots];
        fetch();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            v[r][kUp] = r ? gh[r ? r - 1 : 0] : masked(up, s.from_up);
            v[r][kLeft] = left_of(gh[r], s.from_left);
            v[r][kSelf] = gh[r];
            v[r][kRight] = right_of(gh[r], s.from_right);
            v[r][kDown] = r + 1 < R ? gh[r + 1 < R ? r + 1 : r] : masked(down, s.from_down);
            float acc = kr[r][kSelf] * v[r][kSelf];
            acc = __builtin_fmaf(kr[r][kLeft], v[r][kLeft], acc);
            acc = __builtin_fmaf(kr[r][kRight], v[r][kRight], acc);
            acc = __builtin_fmaf(kr[r][kUp], v[r][kUp], acc);
            g[r] = __builtin_fmaf(kr[r][kDown], v[r][kDown], acc);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) gh[r] = xi[r] < 0.0f ? 0.0f : g[r];
        put_ends(to, gh);
        __builtin_amdgcn_sched_barrier(0);      // (the ends first, the shares while they are written)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int y = 0; y < kSlots; ++y) share[r][y] = __builtin_fmaf(fabsf(xi[r]), v[r][y], share[r][y]);
        lds_barrier();
    };
    const int n_seg = (A.rounds + A.every - 1) / A.every;
    // ready: the forward sweep has left the segment's rounds in the rows of tags
    auto segment = [&](int sg, bool ready) {
        const int t0 = sg * A.every, len = min(A.every, A.rounds - t0);
        float x[R], pre[R];
        // ---- the rounds of this segment into the rows 0 .. len
        if (ready) {
            get_tags(s.tags + len * s.tag_row, x);
        } else {
            const float *first = A.hist ? A.hist + t0 * plane + b * na : sg == 0 ? A.r0 + b * A.ldr : A.ckpt + (sg - 1) * plane + b * na;
            load_nodes(s, first, 1.0f, x);
            put_tags(s.tags, x);
            begin_phase(s, x);
            if (A.hist) {
                // a stored 1 may be a clamped sum: it gets the sign of the decision (the magnitude others read stays 1)
                for (int t = 1; t <= len; ++t) {
                    const float up = masked(lds_at(s.ends[0].up), s.from_up), down = masked(lds_at(s.ends[0].down), s.from_down);
#pragma unroll
                    for (int r = 0; r < R; ++r) pre[r] = row_sum(s, r, up, down, x, kc);
                    load_nodes(s, A.hist + (t0 + t) * plane + b * na, 1.0f, x);
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        if (x[r] >= 1.0f) x[r] = signed_tag(pre[r]) < 0.0f ? -1.0f : 1.0f;
                    put_ends(s.ends[1], x);
                    put_tags(s.tags + t * s.tag_row, x);
                    lds_barrier();
                    const Ends sw = s.ends[0]; s.ends[0] = s.ends[1]; s.ends[1] = sw;
                }
            } else {
                rounds<R, true>(s, len, kc, x, pre, s.tags + s.tag_row);
            }
        }
        // ---- the gradient handed over meets the decision of this segment's last round
        float gh[R];
#pragma unroll
        for (int r = 0; r < R; ++r) gh[r] = x[r] < 0.0f ? 0.0f : g[r];
        begin_phase(s, gh);
        // ---- walk the segment backwards; xi: the tags of the round at hand, fetched a round ahead
        uint32_t row = s.tags + (len - 1) * s.tag_row;
        float xi[R];
        get_tags(row, xi);
        auto one = [&](const Ends &from, const Ends &to, bool last) {
            float next[R];
            row -= last ? 0u : s.tag_row;
            reverse_round(from, to, gh, xi, [&] { get_tags(row, next); });
#pragma unroll
            for (int r = 0; r < R; ++r) xi[r] = next[r];
        };
        int left = len;
        for (; left > 1; left -= 2) {
            one(s.ends[0], s.ends[1], false);
            one(s.ends[1], s.ends[0], left == 2);
        }
        if (left) {
            one(s.ends[0], s.ends[1], true);
            const Ends sw = s.ends[0]; s.ends[0] = s.ends[1]; s.ends[1] = sw;
        }
    };
    int sg = n_seg - 1;
    if constexpr (PRE) {
        if (sg >= 0) segment(sg--, true);
    }
    if constexpr (KEEP) {
        if (sg >= 0) {
            const int len = A.every;
            float x[R], gh[R];
            get_tags(s.tags, x);                // (those after the segment's last round; the last segment began with them)
#pragma unroll
            for (int r = 0; r < R; ++r) gh[r] = x[r] < 0.0f ? 0.0f : g[r];
            if (len & 1) put_ends(s.ends[0], gh);
            else put_ends(s.ends[1], gh);
            lds_barrier();
            // (short segments skip eight rounds at a time: 8 x 8, segments of 4 rounds where 68 fit, 10 rounds 10.9 us one by one both ways, 9.1 so)
#pragma unroll
            for (int t8 = (kept_rounds<R> - 1) & ~7; t8 >= 0; t8 -= 8) {
                if (t8 >= compared(len)) continue;
#pragma unroll
                for (int t = t8 + 7; t >= t8; --t)
                    if (t < kept_rounds<R> && t < compared(len)) reverse_round(s.ends[t & 1], s.ends[(t + 1) & 1], gh, kept[t < kept_rounds<R> ? t : 0], [] {});
            }
            --sg;
        }
    }
    for (; sg >= 0; --sg) segment(sg, false);
    if (A.grad_r0) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (r < s.n_valid) A.grad_r0[b * na + s.node + r * s.w] = g[r];
    }
    if (!A.grad_e) return;
    // ---- the tuples' shares meet per symbol of e, in the order of the symbol's row (ascending first operand): a row of up to
    // four tuples by a thread, a longer one - the "stay" symbol's has one per node - by a wavefront
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int y = 0; y < kSlots; ++y)
            if (r < s.n_valid) share_buf[y * na + s.node + r * s.w] = share[r][y];
    if (threadIdx.x == 0) share_buf[kSlots * na] = 0.0f;
    lds_barrier();
    constexpr int J = 8;                            // symbols of a thread at a time
    for (int j0 = threadIdx.x; j0 < nb; j0 += J * T) {
        uint2 p[J];
#pragma unroll
        for (int x = 0; x < J; ++x) p[x] = S.brief[min(j0 + x * T, nb - 1)];
#pragma unroll
        for (int x = 0; x < J; ++x) {
            float tot = share_buf[p[x].x & 0xFFFFu] + share_buf[p[x].x >> 16];
            tot += share_buf[p[x].y & 0xFFFFu];
            tot += share_buf[p[x].y >> 16];
            if (j0 + x * T < nb) A.grad_e[b * A.ldge + j0 + x * T] = tot;
        }
    }
    if (S.n_longer == 0) return;
    __syncthreads();                                // (those rows' entries are written twice)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x & (kWave - 1);
    for (int l = wave; l < S.n_longer; l += T / kWave) {
        const uint32_t *row = S.longer + 3 * l;
        const uint32_t b0 = row[1], b1 = row[2];
        float tot = 0.0f;
        for (uint32_t p = b0 + lane; p < b1; p += 8 * kWave) {
            uint32_t pos[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) pos[u] = S.pos[min(p + u * kWave, b1 - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float v = share_buf[pos[u]];
                tot += p + u * kWave < b1 ? v : 0.0f;
            }
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) tot += __shfl_xor(tot, d, kWave);
        if (lane == 0) A.grad_e[b * A.ldge + row[0]] = tot;
    }
}

template <int R>
__global__ void __launch_bounds__(kMaxWaves * kWave)
damp_iterate_grid_fwd_kernel(const ItFwdArgs A, const GridLayout L, const uint32_t *__restrict__ slots)
{
    extern __shared__ float lds[];
    Strip<R> s(L, lds);
    int second[R][kSlots];
    load_slots(s, slots, A.na, A.nb, second);
    float *le = lds + Rows<R>::tags(blockDim.x);    // (no rows of tags)
    stage(le, A.e + blockIdx.x * A.lde, A.nb);
    lds_barrier();
    float k[R][kSlots];
    take_values(le, second, k);
#pragma unroll
    for (int r = 0; r < R; ++r) k[r][kSelf] = r < s.n_valid ? k[r][kSelf] : 2.0f;
    Kept<R> none;
    grid_forward<R, false, false>(A, s, k, none);
}

// The kernels with a reverse sweep.
template <int R, bool PRE, bool KEEP>
__device__ __forceinline__ void grid_reverse(const ItFwdArgs *F, const ItBwdArgs &B, const GridLayout &L, const uint32_t *__restrict__ slots,
                                             const GridSums &S, float *lds)
{
    Strip<R> s(L, lds);
    int as_column[R][kSlots], as_row[R][kSlots];
    load_slots(s, slots, B.na, B.nb, as_column);
    load_slots(s, slots + kSlots * B.na, B.na, B.nb, as_row);
    float *tags = lds + Rows<R>::tags(blockDim.x), *le = tags + (B.every + 1) * Rows<R>::tag_row(L);
    stage(le, B.e + blockIdx.x * B.lde, B.nb);
    lds_barrier();
    float kc[R][kSlots], kr[R][kSlots];
    take_values(le, as_column, kc);
    take_values(le, as_row, kr);
#pragma unroll
    for (int r = 0; r < R; ++r) kc[r][kSelf] = r < s.n_valid ? kc[r][kSelf] : 2.0f;
    Kept<R> kept;
    if constexpr (PRE) {
        grid_forward<R, true, KEEP>(*F, s, kc, kept);
        __syncthreads();                            // (the result is read back where the loss is taken from it)
    }
    grid_backward<R, PRE, KEEP>(B, S, s, kc, kr, kept, B.shares_in_seg ? tags : le + B.nb + 1);
}

template <int R>
__global__ void __launch_bounds__(kMaxWaves * kWave, 4)
damp_iterate_grid_bwd_kernel(const ItBwdArgs B, const GridLayout L, const uint32_t *__restrict__ slots, const GridSums S)
{
    extern __shared__ float lds[];
    grid_reverse<R, false, false>(nullptr, B, L, slots, S, lds);
}

template <int R>
__global__ void __launch_bounds__(kMaxWaves * kWave, 4)
damp_iterate_grid_fwd_bwd_kernel(const ItFwdArgs F, const ItBwdArgs B, const GridLayout L, const uint32_t *__restrict__ slots, const GridSums S)
{
    extern __shared__ float lds[];
    grid_reverse<R, true, false>(&F, B, L, slots, S, lds);
}

// The last segment's rounds in LDS, those of the segment before it in registers: up to twice as many rounds in all are run
// forward once only.
template <int R>
__global__ void __launch_bounds__(kMaxWaves * kWave, 2)
damp_iterate_grid_fwd_bwd_kept_kernel(const ItFwdArgs F, const ItBwdArgs B, const GridLayout L, const uint32_t *__restrict__ slots, const GridSums S)
{
    extern __shared__ float lds[];
    grid_reverse<R, true, true>(&F, B, L, slots, S, lds);
}

GridLayout layout_of(const dol_fn_table *f, int R)
{
    GridLayout g;
    g.w = f->grid.width, g.h = f->na / g.w;
    g.per_wave = kWave / g.w;
    g.bands = (g.h + R - 1) / R;
    return g;
}

int waves_of(const dol_fn_table *f, int R)
{
    const GridLayout g = layout_of(f, R);
    return (g.bands + g.per_wave - 1) / g.per_wave;
}

// Rows of a strip.  While a unit has at most two of the batch's samples, the fewest with which a sample takes no more than
// eight wavefronts: with one wavefront on a SIMD the arithmetic of a taller strip has nothing to hide behind, with more than
// two the barriers cost more than they hide.  With more samples to a unit they hide each other's waits, and fewer, taller
// strips exchange less: up to twelve wavefronts on the unit then.  (B = 256, both sweeps, 1, 2 and 4 rows: 16 x 16 grid 21.2,
// 22.5, 25.8 us; 32 x 32 grid -, 35.6, 38.6; B = 1024: 12 x 12 34.3, 36.4, 42.2; 16 x 16 41.0, 36.5, 43.0; 32 x 32 -, 110, 91)
int strip_rows(const dol_fn_table *f, int32_t batch)
{
    const int samples = (std::max(batch, 1) + kUnits - 1) / kUnits;
    const int waves = samples <= 2 ? kMaxWaves : std::min(kMaxWaves, 12 / std::min(samples, 4));
    return waves_of(f, 1) <= waves ? 1 : waves_of(f, 2) <= waves ? 2 : 4;
}

template <typename Fn>
auto with_rows(const dol_fn_table *f, int32_t batch, Fn fn)
{
    switch (strip_rows(f, batch)) {
    case 1: return fn(std::integral_constant<int, 1>{});
    case 2: return fn(std::integral_constant<int, 2>{});
    default: return fn(std::integral_constant<int, 4>{});
    }
}

template <class... Args>
dol_status launch(const dol_fn_table *f, int32_t batch, const void *kern, int R, size_t lds, hipStream_t st, const Args &...args)
{
    if (lds > 64 * 1024) DOL_HIP(allow_dynamic_lds(kern, kItLdsMax));
    void *argv[] = {const_cast<void *>(static_cast<const void *>(&args))...};
    DOL_HIP(hipLaunchKernel(kern, dim3(static_cast<unsigned>(batch)), dim3(static_cast<unsigned>(waves_of(f, R) * kWave)), argv, lds, st));
    return DOL_OK;
}

const uint32_t *slots_of(const dol_fn_table *f) { return f->grid.slots.ptr; }

GridSums sums_of(const dol_fn_table *f)
{
    return {reinterpret_cast<const uint2 *>(f->grid.brief.ptr), f->grid.longer.ptr, f->grid.pos.ptr, f->grid.n_longer};
}

// words for the shares: [5][na] and a 0
size_t share_words(const dol_fn_table *f) { return static_cast<size_t>(kSlots) * f->na + 1; }

}  // namespace

dol_status grid_plan_build(dol_fn_table *f, const std::vector<uint32_t> &col_ptr, const std::vector<uint32_t> &col_ij,
                           const std::vector<uint32_t> &rowb_ptr, const std::vector<uint32_t> &rowb_ic)
{
    const int32_t na = f->na, nb = f->nb;
    if (f->n_out != na || na < 4 || kSlots * na >= 0xFFFF) return DOL_OK;
    int32_t w = 0;
    for (int32_t c = 0; c < na && w <= 1; ++c)
        for (uint32_t q = col_ptr[c]; q < col_ptr[c + 1] && w <= 1; ++q) w = std::abs(static_cast<int32_t>(col_ij[q] & 0xFFFFu) - c);
    if (w <= 1 || w >= na || na % w != 0) return DOL_OK;
    const int64_t h = na / w;
    if (static_cast<int64_t>(col_ij.size()) != na + 2 * (na - w) + 2 * h * (w - 1)) return DOL_OK;
    const int32_t off[kSlots] = {-w, -1, 0, 1, w};
    auto slot = [&](int32_t from, int32_t to) {     // -1: no neighbours
        for (int y = 0; y < kSlots; ++y)
            if (to - from == off[y]) return std::abs(off[y]) == 1 && from / w != to / w ? -1 : y;
        return -1;
    };
    std::vector<uint32_t> slots(2 * static_cast<size_t>(kSlots) * na, static_cast<uint32_t>(nb));
    std::vector<uint8_t> seen(static_cast<size_t>(kSlots) * na, 0);
    for (int32_t c = 0; c < na; ++c)
        for (uint32_t q = col_ptr[c]; q < col_ptr[c + 1]; ++q) {
            const int32_t i = col_ij[q] & 0xFFFFu, j = col_ij[q] >> 16;
            const int y = slot(c, i);
            if (y < 0 || seen[static_cast<size_t>(y) * na + c]) return DOL_OK;
            seen[static_cast<size_t>(y) * na + c] = 1;
            slots[static_cast<size_t>(y) * na + c] = j;
            slots[static_cast<size_t>(kSlots + slot(i, c)) * na + i] = j;
        }
    const uint32_t none = kSlots * na;
    std::vector<uint32_t> brief(2 * static_cast<size_t>(nb)), longer, pos;
    for (int32_t j = 0; j < nb; ++j) {
        uint32_t p[4] = {none, none, none, none};
        const uint32_t q0 = rowb_ptr[j], q1 = rowb_ptr[j + 1];
        const uint32_t first = static_cast<uint32_t>(pos.size());
        for (uint32_t q = q0; q < q1; ++q) {
            const int32_t i = rowb_ic[q] & 0xFFFFu, c = rowb_ic[q] >> 16;
            const uint32_t at = static_cast<uint32_t>(slot(i, c)) * na + i;
            if (q1 - q0 <= 4) p[q - q0] = at;
            else pos.push_back(at);
        }
        if (q1 - q0 > 4) longer.insert(longer.end(), {static_cast<uint32_t>(j), first, static_cast<uint32_t>(pos.size())});
        brief[2 * j] = pack16(p[0], p[1]), brief[2 * j + 1] = pack16(p[2], p[3]);
    }
    hipError_t e;
    if ((e = f->grid.slots.upload(slots)) != hipSuccess || (e = f->grid.brief.upload(brief)) != hipSuccess ||
        (e = f->grid.longer.upload(longer)) != hipSuccess || (e = f->grid.pos.upload(pos)) != hipSuccess)
        return hip_fail(e, "uploading the function table");
    f->grid.n_longer = static_cast<int32_t>(longer.size() / 3);
    f->grid.width = w;
    return DOL_OK;
}

bool grid_table(const dol_fn_table *f) { return f->grid.width > 0 && f->grid.width <= kWave && waves_of(f, 4) <= kMaxWaves; }

int grid_waves(const dol_fn_table *f, int32_t batch) { return waves_of(f, strip_rows(f, batch)); }

bool grid_shares_in_seg(const dol_fn_table *f, int32_t batch, int32_t every)
{
    return with_rows(f, batch, [&](auto R) { return share_words(f) <= (static_cast<size_t>(every) + 1) * Rows<R()>::tag_row(layout_of(f, R())); });
}

size_t grid_bwd_lds(const dol_fn_table *f, int32_t batch, int32_t every)
{
    const size_t shares = grid_shares_in_seg(f, batch, every) ? 0 : share_words(f);
    return with_rows(f, batch, [&](auto R) {
        return sizeof(float) * (Rows<R()>::tags(grid_waves(f, batch) * kWave) + (static_cast<size_t>(every) + 1) * Rows<R()>::tag_row(layout_of(f, R())) +
                                f->nb + 1 + shares);
    });
}

dol_status launch_grid_fwd(const dol_fn_table *f, const ItFwdArgs &A, hipStream_t st)
{
    return with_rows(f, A.batch, [&](auto R) {
        const size_t lds = sizeof(float) * (static_cast<size_t>(Rows<R()>::tags(grid_waves(f, A.batch) * kWave)) + f->nb + 1);
        return launch(f, A.batch, reinterpret_cast<const void *>(&damp_iterate_grid_fwd_kernel<R()>), R(), lds, st, A, layout_of(f, R()), slots_of(f));
    });
}

dol_status launch_grid_bwd(const dol_fn_table *f, const ItBwdArgs &A, size_t lds, hipStream_t st)
{
    return with_rows(f, A.batch, [&](auto R) {
        return launch(f, A.batch, reinterpret_cast<const void *>(&damp_iterate_grid_bwd_kernel<R()>), R(), lds, st, A, layout_of(f, R()), slots_of(f),
                      sums_of(f));
    });
}

template <int R>
static bool keeps(int32_t batch, int32_t rounds, int32_t every) { return batch <= kUnits && every < rounds && every <= kept_rounds<R>; }

const char *grid_fwd_bwd_kernel(const dol_fn_table *f, int32_t batch, int32_t rounds, int32_t every)
{
    return with_rows(f, batch, [&](auto R) { return keeps<R()>(batch, rounds, every) ? "damp_iterate_grid_fwd_bwd_kept_kernel" : "damp_iterate_grid_fwd_bwd_kernel"; });
}

dol_status launch_grid_fwd_bwd(const dol_fn_table *f, const ItFwdArgs &F, const ItBwdArgs &B, size_t lds, hipStream_t st)
{
    return with_rows(f, F.batch, [&](auto R) {
        const auto kernel = keeps<R()>(F.batch, B.rounds, B.every) ? &damp_iterate_grid_fwd_bwd_kept_kernel<R()> : &damp_iterate_grid_fwd_bwd_kernel<R()>;
        return launch(f, F.batch, reinterpret_cast<const void *>(kernel), R(), lds, st, F, B, layout_of(f, R()), slots_of(f), sums_of(f));
    });
}

}  // namespace dol
