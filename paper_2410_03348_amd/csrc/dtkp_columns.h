// The columns of a function table under DTKP, in one launch (dtkp.hip, applyk.hip): one lane per (sample, column) for
// columns of up to kLongDtkpCol tuples, 4 lanes, 16, a wavefront or a workgroup for the longer ones.
//
// The workgroups of the longest columns come first, those of the short ones run beside them: as launches of their own, one
// after the other, they took 40 of the 103 us of a table of 38 400 columns (64 samples, k = 3: 77 us in one launch).  A lane
// waits for every tuple of its column, 0.8 us each, so it gets few: with up to 16 tuples to a lane that table took 77 us and
// one of 758 columns 16, with up to 8 (then 16 lanes) 79 and 11, with up to 4 and four lanes up to 16, as here, 75 and 8.
// Results gathered in LDS and stored as whole lines were slower (106 us): a workgroup of neighbours waits for its longest
// column.
// With lists ranked by keys that table took 61 us (73 before), k = 3, then 57: a tuple waits for its lists only (its word is read
// one tuple ahead, the first with the column's length, its fact lies in LDS), where the fact is new to all proofs one look at them
// says so and the lists meet as two lanes' do, columns of one tuple go from the operand's list to the result; and 52 now that facts
// and lists have a kernel each and LDS is read as LDS (dtkp.hip).  Not bound by issue (347 -> 308 vector instructions a wavefront
// between the first of these and the second, no time) but by what a wavefront waits for: of the 57, 14 us were its way to the first
// tuple, 21 the short columns, 13 those of 5 to 16 tuples, 10 the longer ones.  Those by a quarter of the lanes: a third fewer
// instructions, 68 us.  147 MB leave for 98 MB of results, whose order is that of the columns' lengths.  Lengths sorted inside
// fewer than 4 096 columns leave fewer bytes (129 MB) but unequal lanes: the pass of that expression took 206 us and more instead
// of 204 (passes in this file repeat the same inputs; where these change from pass to pass they take some ten us more).  Lists read
// four tuples ahead: 80 us, for want of wavefronts.
#pragma once

#include "dtkp_util.h"
#include "wave_util.h"

#include <algorithm>

namespace dol {

// Workgroups of the columns of 16 lanes, four and one in a set of samples (multiples of eight: the XCDs' turns stay the same).
struct SetBlocks {
    uint32_t mid, quad, lane;
};

struct ColumnArgs {
    int32_t batch, S, n_in;                 // n_in: the operands' symbols, of lists of their own
    int32_t n_huge, n_wave, n_mid, n_quad;  // `longer`: columns of a workgroup each, of a wavefront, of 16 lanes, of four
    uint32_t b_huge, b_wave;                // workgroups of these kinds, all samples'
    int32_t set, sets;                      // the other columns: samples of a set (the last one holds the remainder too), sets
    SetBlocks full, last;
    const uint32_t *longer;
    const uint32_t *col_ptr;                // tuples of a column
    const uint32_t *order, *len;            // short columns: the r-th one and its length (0: among the longer ones)
    uint64_t per_S;                         // 2^64 / S, rounded up (0: S = 1)
    uint64_t *om;
    float *op, *oprob;
    int64_t ldo;
};

inline void set_columns(ColumnArgs &A, const DtkpColumns &D)
{
    A.n_huge = D.n_huge, A.n_wave = D.n_wave, A.n_mid = D.n_mid, A.n_quad = D.n_quad;
    A.longer = D.longer.ptr, A.order = D.order.ptr, A.len = D.len.ptr;
}

// Threads of a workgroup: more for the sake of huge columns (last table of the seven-symbol expression: 100, 79, 77, 83 us
// with 64, 128, 256, 512; tables without huge columns: 128 or fewer).
constexpr int kColumnThreads = 128, kHugeThreads = 256;
inline int column_threads(const ColumnArgs &A) { return A.n_huge > 0 ? kHugeThreads : kColumnThreads; }

// How the columns go into workgroups; returns how many there are.
//
// Where the lists of all samples exceed the L2s, the samples go in sets, one sample's columns of all lengths (the very long
// ones apart: they start first) close together: a line of results holds columns of several lengths and leaves the L2 whole, and
// its lists are read once.  A set is eight samples, one for each XCD, or more where they are small, so that a set has work for the
// whole chip.
// (Seven-symbol expression, k = 3: with 64 samples the last table writes 116 instead of 149 MB and the unary Apply
// behind it takes 26.6 instead of 29.1 us, the pass 177 instead of 180; with 128 samples 288 instead of 311 us, with 1 024 2 186
// instead of 2 668.  Sets of 16 or 32: 178 and 179, 2 237 and 2 252.  With 16 samples, 27 MB, two sets cost 2 %.  The very long
// columns in their sets: 185, the last set's workgroup columns ending late.)
constexpr int64_t kL2Bytes = int64_t(32) << 20, kSetBytes = int64_t(8) << 20;
template <int K>
inline unsigned column_launch(ColumnArgs &A)
{
    const int threads = column_threads(A);
    const int64_t sample = (static_cast<int64_t>(A.S) + A.n_in) * (K * (sizeof(uint64_t) + sizeof(float)));
    A.set = A.batch, A.sets = 1;
    if (A.batch * sample > kL2Bytes) {
        const int64_t set = std::max<int64_t>(8, kSetBytes / sample / 8 * 8);
        if (A.batch >= 2 * set) A.set = static_cast<int32_t>(set), A.sets = static_cast<int32_t>(A.batch / set);
    }
    A.per_S = A.S > 1 ? ~uint64_t(0) / static_cast<uint32_t>(A.S) + 1 : 0;
    auto eight = [](int64_t n) { return static_cast<uint32_t>((n + 7) / 8 * 8); };
    auto groups = [&](int32_t samples, int32_t n, int lanes) {
        const int per = threads / lanes;
        return eight(static_cast<int64_t>(samples) * ((n + per - 1) / per));
    };
    auto blocks = [&](int32_t samples) {
        return SetBlocks{groups(samples, A.n_mid, 16), groups(samples, A.n_quad, 4),
                         eight((static_cast<int64_t>(samples) * A.S + threads - 1) / threads)};
    };
    auto all = [](const SetBlocks &b) { return b.mid + b.quad + b.lane; };
    A.b_huge = eight(static_cast<int64_t>(A.batch) * A.n_huge);
    A.b_wave = groups(A.batch, A.n_wave, kWave);
    A.full = blocks(A.set), A.last = blocks(A.batch - (A.sets - 1) * A.set);
    return A.b_huge + A.b_wave + (A.sets - 1) * all(A.full) + all(A.last);
}

// Offer: ask() and share() - what all threads of a workgroup need is on its way, is there; begin(s) - the sample; ahead(r) - the
// first tuple of the r-th short column, asked for before anything is known about it; listed(top, q, q1, step) - offers the
// tuples q, q + step, .. below q1 of col_ptr's lists; laned(top, len, r, c) - those of column c, the r-th in order; where it
// has_short(), short_listed and short_laned offer the same, of at most kLongDtkpCol tuples a lane, to a list of keys, and
// short_take() finds the proofs of the list, the same of `lanes` lanes, or says that it cannot (to each of them); kOneWay - how
// lists take in candidates (TopK::insert).
// (A candidate's way into a list of probabilities and masks takes some thirty
// instructions, most of them choices, and so does each entry of another lane's list; into a list of keys seven, and a whole list of
// three twelve and the lane shifts.)
constexpr int kKeyProofs = 4;           // longest lists ranked by keys

// Are two neighbours among the first facts of this wavefront's (first) sample equally probable?  Then proofs are too, most columns
// would be ranked in vain, and the general way is taken at once.  (Seven-symbol expression, k = 3, 64 samples, us, without / with
// this look: facts of one probability 267 / 229, one certain fact to a position 442 / 390; softmax 177.9 / 179.3.  Where only
// products that underflow are equal, as of logits twelve times as far apart, columns are ranked in vain: 275, by insertion 247.)
__device__ __forceinline__ bool equal_facts(const float *fact_prob, int n_facts, int32_t sample)
{
    constexpr int kLook = 8;
    if (n_facts < kLook || !fact_prob) return false;
    // (read as constants, by scalar loads: vector loads of all facts cost the passes of the seven-symbol expression 2 to 3 %)
    const auto *p = reinterpret_cast<const __attribute__((address_space(4))) uint32_t *>(
        reinterpret_cast<uintptr_t>(fact_prob + static_cast<int64_t>(__builtin_amdgcn_readfirstlane(sample)) * n_facts));
    bool same = false;
#pragma unroll
    for (int f = 0; f + 1 < kLook; ++f) same |= p[f] == p[f + 1];
    return same;
}

static_assert(kMidDtkpCol <= 4 * kLongDtkpCol && kWaveDtkpCol <= 16 * kLongDtkpCol, "a lane's tuples");

template <int K, class Offer>
__device__ __forceinline__ void dtkp_columns(const ColumnArgs &A, Offer offer)
{
    const int T = blockDim.x, t = threadIdx.x;
    offer.ask();
    TopK<K> top;
    top.clear();
    uint32_t b = blockIdx.x;
    int32_t s0 = 0, samples = A.batch;
    SetBlocks B{0, 0, 0};
    const uint32_t very_long = A.b_huge + A.b_wave;
    if (b >= very_long) {
        const uint32_t per_set = A.full.mid + A.full.quad + A.full.lane, set = min((b - very_long) / per_set, static_cast<uint32_t>(A.sets - 1));
        const bool last = set == static_cast<uint32_t>(A.sets - 1);
        B = last ? A.last : A.full;
        s0 = set * A.set, samples = last ? A.batch - s0 : A.set;
        b -= set * per_set;
    }
    const uint32_t first = very_long + B.mid + B.quad;
    if (b < first) {
        // ---- a longer column: every lane streams a share of its tuples through a list of its own; the lists of a group of
        // lanes meet by exchange rounds in which each lane offers its partner's entries to its own list.  (The list order is
        // total on distinct proofs and repeated proofs are one proof: the result does not depend on the split.)
        int lanes = T;
        int32_t n = A.n_huge, from = 0;
        uint32_t blocks = A.b_huge;
        auto next = [&](int l, int32_t count, uint32_t its) {       // uniform
            if (b < blocks) return;
            b -= blocks, from += n;
            lanes = l, n = count, blocks = its;
        };
        next(kWave, A.n_wave, A.b_wave);
        next(16, A.n_mid, B.mid);
        next(4, A.n_quad, B.quad);
        const bool huge = lanes == T;
        const int per = T / lanes, groups = (n + per - 1) / per;
        const int32_t id = xcd_contiguous(b, blocks);               // (a sample's columns on one XCD: its lists fill one L2)
        const int32_t in_set = id / groups, ci = (id - in_set * groups) * per + t / lanes, s = s0 + in_set;
        if (in_set >= samples) return;
        const uint32_t c = A.longer[from + min(ci, n - 1)];
        offer.share();
        if (ci >= n) return;                        // (all lanes of a group; never a huge column's)
        offer.begin(s);
        if constexpr (K <= kKeyProofs) {
            // (at most kLongDtkpCol tuples a lane)
            if (lanes <= 16 && offer.has_short() && !equal_facts(offer.A.fact_prob, offer.A.n_facts, s)) {
                TopKeys<K> keys;
                offer.short_listed(keys, A.col_ptr[c] + t % lanes, A.col_ptr[c + 1], lanes);
                keys.merge(lanes);
                if (!keys.unclear() && offer.short_take(top, keys, lanes)) {       // (the same for all lanes of the group)
                    if (t % lanes != 0) return;
                    const int64_t o = static_cast<int64_t>(s) * A.S + c;
                    A.oprob[s * A.ldo + c] = top.store(A.om + o * K, A.op + o * K);
                    return;
                }
                top.clear();
            }
        }
        offer.listed(top, A.col_ptr[c] + t % lanes, A.col_ptr[c + 1], lanes);
        if (lanes == 4) merge_lists<K, 4, Offer::kOneWay>(top);
        else if (lanes == 16) merge_lists<K, 16, Offer::kOneWay>(top);
        else merge_lists<K, kWave, Offer::kOneWay>(top);
        if (huge) {                                 // uniform: the wavefronts' lists meet in the first wavefront
            __shared__ uint64_t lm[kHugeThreads / kWave * K];
            __shared__ float lp[kHugeThreads / kWave * K];
            const int lane = t & (kWave - 1), w = t / kWave, n_waves = T / kWave;
            if (lane == 0) {
#pragma unroll
                for (int x = 0; x < K; ++x) { lm[w * K + x] = top.m[x]; lp[w * K + x] = top.p[x]; }
            }
            __syncthreads();
            if (w != 0) return;
            top.clear();
            if (lane < n_waves) {
#pragma unroll
                for (int x = 0; x < K; ++x) { top.m[x] = lm[lane * K + x]; top.p[x] = lp[lane * K + x]; }
            }
            merge_lists<K, kHugeThreads / kWave, Offer::kOneWay>(top);
        }
        if (t % lanes == 0) {
            const int64_t o = static_cast<int64_t>(s) * A.S + c;
            A.oprob[s * A.ldo + c] = top.store(A.om + o * K, A.op + o * K);
        }
        return;
    }
    const int32_t id = xcd_contiguous(b - first, B.lane);
    // the workgroup's first (sample, column), by a multiplication (a division of 64 bits by each lane took a tenth of a short
    // column's instructions); a lane's from there
    const uint32_t S = static_cast<uint32_t>(A.S);
    const uint64_t from = static_cast<uint64_t>(static_cast<uint32_t>(id)) * T, total = static_cast<uint64_t>(samples) * S;
    if (from >= total) return;
    uint32_t q0 = static_cast<uint32_t>(from);
    if (from >> 32) q0 = static_cast<uint32_t>(from / S);
    else if (S > 1) q0 = static_cast<uint32_t>((from * (A.per_S >> 32) + __umulhi(q0, static_cast<uint32_t>(A.per_S))) >> 32);
    uint32_t r = static_cast<uint32_t>(from - static_cast<uint64_t>(q0) * S) + t;
    const uint32_t over = S >= static_cast<uint32_t>(T) ? (r >= S ? 1u : 0u) : r / S;
    r -= over * S;
    const bool live = from + t < total;
    r = live ? r : 0;
    const int32_t s = s0 + static_cast<int32_t>(q0 + (live ? over : 0));
    // lanes of a wavefront: columns of like length
    const uint32_t len = A.len[r], c = A.order[r];
    offer.ahead(r);
    offer.share();
    if (!live) return;
    offer.begin(s);
    bool keys_ok = false;
    if constexpr (K <= kKeyProofs) keys_ok = offer.has_short() && !equal_facts(offer.A.fact_prob, offer.A.n_facts, s);     // (for all)
    if (len == 0) return;
    bool todo = true;
    if constexpr (K <= kKeyProofs) {
        if (keys_ok && len == 1) todo = !offer.single(top);
        if (keys_ok && todo) {
            TopKeys<K> keys;
            top.clear();
            offer.short_laned(keys, len, r);
            todo = keys.unclear() || !offer.short_take(top, keys, 1);
        }
    }
    if (__builtin_expect(todo, 0)) {
        top.clear();
        offer.laned(top, len, r, c);
    }
    const int64_t o = static_cast<int64_t>(s) * A.S + c;
    A.oprob[s * A.ldo + c] = top.store(A.om + o * K, A.op + o * K);
}

}  // namespace dol
