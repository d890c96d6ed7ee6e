// Fused left fold of Apply under DTKP-AM (the loop of Fig. 2 with the top-k proofs provenance of Sec. 3.2 /
// App. A) over naturally initialised inputs: symbol i of input t carries the single proof {fact_of_sym[t][i]}.
// One wavefront owns a sample: the fact probabilities and the running Distribution's proofs (S x k masks and
// probabilities) live in LDS, a lane (two where the wavefront has them to spare) owns an output symbol, streams the candidates of
// its tuples through a k-entry sorted list in registers and writes the list back to LDS for the next stage.  Up to four wavefronts
// form a workgroup and share one copy of the symbol side.  HBM sees the fact probabilities once and the final Distribution once.
// Optionally the gradient of the final tag probabilities w.r.t. the fact probabilities follows in the same launch (lane f owns fact
// f).
// Candidate order, proof probabilities, exclusion test and list order are those of dol_apply2, so the result is the
// same bit for bit.  The sorted list of a column carries probabilities and the origin of each proof; masks are built
// for the k winners only, and a stage whose input brings only new, higher facts (fresh_t below) never reads one.
#include "dtkp_util.h"
#include "plan_cache.h"
#include "wave_util.h"

#include <cfloat>
#include <cstdio>
#include <vector>

namespace dol {

constexpr int kDfMax = 32;              // most inputs of one fold
constexpr int kDfWaves = 4;             // most wavefronts (samples) of one workgroup

// The symbol side of the whole fold as one array of words, copied into LDS at the start of the kernel:
//   [0] number of inputs n, then for t = 0 .. n-1 four words: S_t, p_t, r_t, fresh_t
//   t = 0:  S_0 words at p_0: the facts of the first input's symbols
//   t >= 1: S_t + 1 words at p_t: where each output column's tuples start and end inside the stage's records;
//           the records at r_t, one per tuple in column order: the first operand's list, counted in bytes of
//           probabilities, | 4 x the second operand's FACT << 16 (spare records at the end so that the read-ahead
//           stays inside)
//   fresh_t, bit 0: every fact of input t lies above every fact of the inputs before it and shares no exclusion group
//           with any of them.  A proof of the running Distribution then never holds the new fact or a rival of it, and
//           the product over ascending facts is the proof's stored probability times the new fact's: the stage needs
//           no mask at all until its k winners are known.  Bit 1: and each input so far gives every symbol a fact of its own, none
//           of them known before: a proof says which symbols it is of, and no two symbols of a Distribution have one in common.
//           Bits 2 and 3: lanes help (dtkp_fold_stage), from bit 4 on: the stage's shares are the so many-th 64 words behind the
//           others.
enum Kind : int32_t { kFresh = 1, kDistinct = 2, kTwins = 4, kHelped = 8 };
constexpr int kShareShift = 4;
struct DtkpFoldArgs {
    int32_t n, batch, n_facts, max_s, n_words, wave_bytes;
    const int32_t *words;
    const uint64_t *rival;              // device [n_facts]: the other facts of each fact's exclusion group
    const float *fact_prob;
    uint64_t *om;
    float *op, *oprob;
    int64_t ldo;
    const int32_t *target;
    const float *gout;
    int64_t ldg;
    float *gfact;
    int32_t n_shares;
};

// The K best distinct proofs of one column, by the whole wavefront: lane y < K ends with the y-th (id -1: none).  Lanes K .. 63
// take the candidates as they come, the first K lanes keep the best so far; K times the best of all is taken, the smallest mask
// among equal probabilities, and with it whatever has its mask.  For probabilities that are finite and not below 0.
// (Two facts of one probability, in one of a thousand samples of softmax outputs, make tens of such columns.  By its lane, a
// candidate at a time, through code that no wavefront had fetched yet, a column took 4 us (k = 3) to 60 (k = 7) and the others of
// the stage with it: Sum-6, k = 5, 2 048 samples 50 us with one such sample and 17.7 without any, k = 7 83 and 22.6, Sum-5, k = 3,
// 1 024 12.9 and 9.1; so 28 and 17.8, 51 and 22.6, 9.5 and 9.1.)
// One column after the other, though, where a lane each does all of a stage's at once: where more than kManyTies of them are to be
// ranked they are exact_column's.  Logits twelve and thirty times as far apart, whose products underflow, us, columns by the
// wavefront up to 2, 4, 8, 16, all: Sum-5, k = 3, 1 024 samples 20.2 20.4 23.8 27.4 27.3 and 63 63 69 144 217; Sum-6, k = 5,
// 12 000 153 145 169 225 224 and 504 507 516 1 027 2 069; k = 7, 6 000 248 248 239 337 337 and 657 658 666 1 308 3 465; one sample
// with two equal facts, k = 5, 2 048 28 28 25 25 25.
template <int K>
constexpr int kManyTies = K <= 5 ? 4 : 8;

struct Ranked {
    float p;
    int id;
};

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x)
{
    x = max(x, static_cast<uint32_t>(dpp_i<0xB1>(static_cast<int>(x))));
    x = max(x, static_cast<uint32_t>(dpp_i<0x4E>(static_cast<int>(x))));
    x = max(x, static_cast<uint32_t>(dpp_i<0x141>(static_cast<int>(x))));
    x = max(x, static_cast<uint32_t>(dpp_i<0x140>(static_cast<int>(x))));
    const uint32_t a = __builtin_amdgcn_readlane(static_cast<int>(x), 0), b = __builtin_amdgcn_readlane(static_cast<int>(x), 16);
    const uint32_t c = __builtin_amdgcn_readlane(static_cast<int>(x), 32), d = __builtin_amdgcn_readlane(static_cast<int>(x), 48);
    return max(max(a, b), max(c, d));
}

template <int K, int KA>
__device__ __forceinline__ Ranked rank_column(uint32_t q0, uint32_t q1, const uint32_t *l_rec, const uint64_t *cm,
                                              const float *cp, const float *fp)
{
    const int lane = threadIdx.x & (kWave - 1);
    Ranked best{-1.0f, -1};
    uint64_t best_mask = kAbsent;
    const int total = static_cast<int>(q1 - q0) * KA;
#pragma unroll 1
    for (int first = 0; first < total; first += kWave - K) {
        float p = best.p;
        int id = best.id;
        uint64_t mask = best_mask;
        const int k = first + lane - K;
        if (lane >= K) {
            p = -1.0f, id = -1, mask = kAbsent;
            if (k < total) {
                const uint32_t q = q0 + static_cast<uint32_t>(k) / KA, x = static_cast<uint32_t>(k) % KA, r = l_rec[q];
                const int at = static_cast<int>((r & 0xffffu) >> 2) + static_cast<int>(x);
                const float pa = cp[at];
                if (pa >= 0.0f) p = pa * fp[r >> 18], id = static_cast<int>(q << 3 | x), mask = cm[at] | (uint64_t(1) << (r >> 18));
            }
        }
        best = Ranked{-1.0f, -1}, best_mask = kAbsent;
#pragma unroll 1
        for (int y = 0; y < K; ++y) {
            const uint32_t key = p >= 0.0f ? __float_as_uint(p) + 1 : 0, top = wave_max_u32(key);
            if (top == 0) break;
            const uint32_t lo = static_cast<uint32_t>(mask), hi = static_cast<uint32_t>(mask >> 32);
            int from = -1;
            uint64_t least = kAbsent;
            for (uint64_t equal = __ballot(key == top); equal; equal &= equal - 1) {
                const int at = __builtin_ctzll(equal);
                const uint32_t m_hi = __builtin_amdgcn_readlane(static_cast<int>(hi), at);
                const uint32_t m_lo = __builtin_amdgcn_readlane(static_cast<int>(lo), at);
                const uint64_t m = static_cast<uint64_t>(m_hi) << 32 | m_lo;
                if (from < 0 || m < least) from = at, least = m;
            }
            if (lane == y) best.p = __uint_as_float(top - 1), best_mask = least;
            const int id_from = __builtin_amdgcn_readlane(id, from);
            if (lane == y) best.id = id_from;
            if (mask == least) p = -1.0f;
        }
    }
    return best;
}

// One stage of the fold for this wavefront's sample: the columns of the stage's table, a lane each.  KA: slots of the
// first operand's lists that can hold a proof (1 right after the natural initialisation); FRESH: see fresh_t above.
// Absent slots carry the probability -1 in LDS (0 in the result tensors).
// The list keeps, per rank, the probability and where the proof came from (record, slot of the first operand's list);
// the masks are put together for the k winners only.  In a FRESH stage a tuple's k candidates are the first operand's
// list times one factor, i.e. in descending order already: the k + 1 best of both lists are the elementwise maxima of one
// and the other reversed, sorted again by a short network.  Masks matter only where probabilities are equal: two of the kept
// ones, or the last one and the best that dropped out, which is what the list's entry behind the k-th holds (of all that
// dropped out on the way none is larger).  Such a column is ranked again by the whole wavefront (rank_column), or where there are
// many candidate by candidate (exact_column), as is every column of a sample (plain = false) with a fact whose probability is
// negative, -0 or no finite number, or where an eighth of the facts have the probability of their neighbours: most columns would
// have ties and be done twice (Sum-5, k = 3, B=1 024, facts of one probability: 65 us, 58.4 so; facts in steps of 1/16 64 and 58.2;
// Sum-6, k = 5, B=12 000 560 and 516).
// (Bound by the vector ALUs.  k = 5 costs 33 instructions a tuple by the compiled code, none of them a choice; 65 with
// probabilities and origins exchanged by compare and select, which the units take 1.9 ns a piece for, and repeated choices by one
// condition longer.  Of the 33, 19 are the list's maxima and minima in twice the time of the others, and 14 the products, the
// origins, the addresses and the loop.  What a stage does besides is half as much again: a rank without a proof keeps an origin
// that can be read and a word of ones for its mask and probability to be put together with, and only the last stage adds
// probabilities up: Sum-6, k = 5, 12 000 samples 56.5 us, 55.6 so; k = 7, 1 024 samples 16.8 and 16.5.  The code lies in the order
// it is run in, with what is seldom run behind: Sum-5, k = 3, 1 024 samples 8.1 us so, 8.4 with the first stage's behind the
// others' and the seldom run between them.  Where the compiled code lies moves small batches by some 2 % either way.)
// Where a stage has fewer columns than the wavefront has lanes the others help (FRESH stages): a helper works on the second half of
// a column's tuples, and the two lists become one as a tuple's and the running one do, which costs up to two tuples' worth.
//   few samples: stages of at most 32 columns are worked on by twins, the wavefront's halves have the same columns.  Of Sum-6's
//   five stages two have 19 and 28 columns of up to 10 tuples: k = 5, 12 000 samples 55.6 us, 52.7 so, 1 024 13.4 and 12.7; Sum-5,
//   k = 3, 1 024 samples 8.1 and 7.4, 4 096 13.1 and 12.3.
//   MANY: a lane looks its share up (Share), and of more columns the longest are helped with (of 37 all 27 of more than five
//   tuples).  That takes a trip to LDS for the share and one for the lists, which several wavefronts on a SIMD hide: Sum-6, k = 5,
//   12 000 samples 52.5 and 50.0, k = 7 73.0 and 68.6, Sum-5, k = 3, 12 000 28.0 and 26.6, 4 096 12.3 and 12.0, but 2 048 8.6 and
//   8.7, 1 024 7.4 and 7.7; Sum-3, k = 5, 2 048 7.7 and 8.0.  (Both ways in one kernel take 76 registers, one wavefront less to a
//   SIMD: 52.6.)
constexpr int kListCost = 2;            // tuples saved that two lists are worth
constexpr int kManySamples = 3072;      // three to a SIMD (and see share_lookup_pays)

struct Share {                          // a lane's, in one word
    enum Role : uint32_t { kWhole, kFirstHalf, kHelper, kIdle };
    uint32_t word;
    static __host__ __device__ uint32_t pack(uint32_t col, uint32_t partner, Role role) { return col | partner << 8 | role << 16; }
    __device__ __forceinline__ int col() const { return word & 0xff; }
    __device__ __forceinline__ int partner() const { return word >> 8 & 0xff; }
    __device__ __forceinline__ uint32_t role() const { return word >> 16; }
};

__device__ __forceinline__ double key_of_lane(double x, int lane)
{
    const int hi = __builtin_amdgcn_ds_bpermute(4 * lane, __double2hiint(x)), lo = __builtin_amdgcn_ds_bpermute(4 * lane, __double2loint(x));
    return __hiloint2double(hi, lo);
}

// x of the lane in the lower (upper) half of the wavefront that has this lane's place there
__device__ __forceinline__ double key_of_half(double x, int upper)
{
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(x), false, false);
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(x), false, false);
    return __hiloint2double(static_cast<int>(hi[upper]), static_cast<int>(lo[upper]));
}

template <int K, int KA, bool FRESH, bool MANY>
__device__ __forceinline__ void dtkp_fold_stage(const DtkpFoldArgs &A, int64_t s, int S, bool last, const uint32_t *l_ptr,
                                                const uint32_t *l_rec, const uint64_t *cm, const float *cp, uint64_t *nm,
                                                float *np, const uint64_t *rival, const float *fp, float *gh, bool plain, int kind,
                                                const uint32_t *shares)
{
    const bool distinct = kind & kDistinct, helped = FRESH && (kind & (MANY ? kHelped : kTwins));
    const int lane = threadIdx.x & (kWave - 1);
    for (int base = 0; base < S; base += kWave) {
        const Share mine{MANY && helped ? shares[lane] : Share::pack(lane, 0, Share::kWhole)};
        const int c = base + (MANY ? mine.col() : helped ? lane % (kWave / 2) : lane);
        // (all help where a column has ties)
        const bool there = c < S && (MANY ? mine.role() < Share::kHelper : !(helped && lane >= kWave / 2));
        float tp[K];
        int tid_[K];
        int gone[K];                                        // all bits: no proof
#pragma unroll
        for (int x = 0; x < K; ++x) { tp[x] = -1.0f - x; tid_[x] = -1; }
        auto by_origin = [&]() {
#pragma unroll
            for (int x = 0; x < K; ++x) gone[x] = tid_[x] >> 31, tid_[x] &= ~gone[x];
        };
        auto mask_of = [&](int id) -> uint64_t {            // id = record << 3 | slot (at most DOL_MAX_K = 8 slots)
            const uint32_t r = l_rec[id >> 3];
            return cm[static_cast<int>((r & 0xffffu) >> 2) + (id & 7)] | (uint64_t(1) << (r >> 18));
        };
        // the full comparison: equal masks are one proof, order by probability, then by mask
        auto insert_tied = [&](uint64_t mask, float pr, int id) {
            uint64_t tm[K];
            bool dup = false;
#pragma unroll
            for (int y = 0; y < K; ++y) {
                tm[y] = tid_[y] >= 0 ? mask_of(tid_[y]) : kAbsent;
                dup |= tm[y] == mask;
            }
            if (dup || !TopK<K>::before(mask, pr, tm[K - 1], tp[K - 1])) return;
#pragma unroll
            for (int y = K - 1; y >= 0; --y) {
                const bool here = TopK<K>::before(mask, pr, tm[y], tp[y]);
                const bool above = y > 0 ? TopK<K>::before(mask, pr, tm[y - 1], tp[y - 1]) : false;
                if (above) { tp[y] = tp[y - 1]; tid_[y] = tid_[y - 1]; }
                else if (here) { tp[y] = pr; tid_[y] = id; }
            }
        };
        // offer = kNone: nothing to offer (below every slot, absent ones included)
        // (the kept probabilities are in descending order and the offer equals none of them: the new list is the larger
        // of the first and the offer, then the median of each neighbouring pair and the offer)
        constexpr float kNone = -32.0f;
        auto insert_untied = [&](float offer, int id) {
            bool gt[K];
#pragma unroll
            for (int y = 0; y < K; ++y) gt[y] = offer > tp[y];
#pragma unroll
            for (int y = K - 1; y >= 0; --y) {
                const bool above = y > 0 ? gt[y - 1] : false;
                tp[y] = y > 0 ? __builtin_amdgcn_fmed3f(tp[y - 1], tp[y], offer) : fmaxf(tp[0], offer);
                tid_[y] = above ? tid_[y - 1] : gt[y] ? id : tid_[y];
            }
        };
        const int like = min(c, S - 1);                     // lanes without a column go along with the last one
        const uint32_t q0 = l_ptr[like], q1 = l_ptr[like + 1];
        auto list_of = [&](uint32_t r) { return reinterpret_cast<const float *>(reinterpret_cast<const char *>(cp) + (r & 0xffffu)); };
        auto fact_of = [&](uint32_t r) { return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(fp) + (r >> 16)); };
        if constexpr (FRESH) {
            auto exact_column = [&]() {
#pragma unroll
                for (int x = 0; x < K; ++x) { tp[x] = -1.0f - x; tid_[x] = -1; }
                for (uint32_t q = q0; q < q1; ++q) {
                    const uint32_t cur = l_rec[q];
                    const float *pa = list_of(cur);
                    const float pb = fact_of(cur);
#pragma unroll
                    for (int x = 0; x < KA; ++x) {
                        if (!(pa[x] >= 0.0f)) continue;
                        const float offer = pa[x] * pb;
                        const int id = static_cast<int>(q) << 3 | x;
                        bool tie = false;
#pragma unroll
                        for (int y = 0; y < K; ++y) tie |= offer == tp[y];
                        if (tie) insert_tied(mask_of(id), offer, id);
                        else insert_untied(offer, id);
                    }
                }
            };
            if (__builtin_expect(!plain, 0)) {
                if (there) exact_column();
                by_origin();
            } else {
                // The next tuple's record is on its way while this one is worked on; past the last one lies the next column's or a
                // spare one.  (Read where it is used: Sum-5, k = 3, 1 024 samples 9.1 us, 8.2 so; Sum-6, k = 5, 12 000 57.2 and
                // 56.5.  Operands read a tuple ahead as well cost moves and registers: 8.4, and 58.5.)
                double top[K + 1];
#pragma unroll
                for (int x = 0; x <= K; ++x) top[x] = -1.0;
                uint32_t from = q0, to = q1;
                if (helped) {
                    const uint32_t mid = (q0 + q1 + 1) / 2;
                    if constexpr (MANY) {
                        to = mine.role() == Share::kFirstHalf ? mid : mine.role() == Share::kIdle ? q0 : q1;
                        from = mine.role() == Share::kHelper ? mid : q0;
                    } else {
                        (lane < kWave / 2 ? to : from) = mid;
                    }
                }
                uint32_t rec = l_rec[from];
                asm volatile("" : "+v"(rec));       // (or the compiler folds this read and the loop's into one before its use)
                int id = static_cast<int>(from) << 3;
                for (const uint32_t *next = l_rec + from + 1, *const end = l_rec + to; next <= end; ++next, id += 8) {
                    const float *list = list_of(rec);
                    const float pb = fact_of(rec);
                    float pa[KA];
#pragma unroll
                    for (int x = 0; x < KA; ++x) pa[x] = list[x];
                    rec = *next;
                    double offer[KA];       // (an absent proof's is negative or -0: below every proof)
#pragma unroll
                    for (int x = 0; x < KA; ++x) offer[x] = key_of(pa[x] * pb, id + x);
                    if constexpr (KA == K && K > 1) {
                        double best[K + 1];
                        best[0] = top[0];
#pragma unroll
                        for (int x = 1; x <= K; ++x) best[x] = key_max(top[x], offer[K - x]);
                        sort_valley<K + 1, K + 1>(best, 0);
#pragma unroll
                        for (int x = 0; x <= K; ++x) top[x] = best[x];
                    } else {
                        double o = offer[0];
#pragma unroll
                        for (int x = 0; x <= K; ++x) {
                            const double t = top[x];
                            top[x] = key_max(t, o);
                            if (x < K) o = key_min(t, o);
                        }
                    }
                }
                if (helped) {
                    auto join = [&](auto of_first, auto of_helper) {
                        double best[K + 1];
#pragma unroll
                        for (int x = 0; x <= K; ++x) best[x] = key_max(of_first(x), of_helper(K - x));
                        sort_valley<K + 1, K + 1>(best, 0);
#pragma unroll
                        for (int x = 0; x <= K; ++x) top[x] = best[x];
                    };
                    if constexpr (MANY) {
                        double other[K + 1];
#pragma unroll
                        for (int x = 0; x <= K; ++x) other[x] = key_of_lane(top[x], mine.partner());
                        if (mine.role() == Share::kFirstHalf) join([&](int x) { return top[x]; }, [&](int x) { return other[x]; });
                    } else {
                        join([&](int x) { return key_of_half(top[x], 0); }, [&](int x) { return key_of_half(top[x], 1); });
                    }
                }
                bool inner = false, again = false;
#pragma unroll
                for (int x = 0; x < K; ++x) {
                    const int hi = __double2hiint(top[x]), next = __double2hiint(top[x + 1]);
                    tp[x] = __int_as_float(hi);
                    tid_[x] = __double2loint(top[x]);       // (0, or that of an absent proof, where there is none)
                    (x + 1 < K ? inner : again) |= hi == next && hi >= 0;
                }
                // Equal probabilities among the kept ones: the masks' order, which only the result shows, unless a proof may be
                // there twice.  The last of them as probable as the best that dropped out: the kept ones may be others.
                again |= inner && (last || !distinct);
                uint64_t todo = __ballot(again && there);
                if (__builtin_expect(__builtin_popcountll(todo) > kManyTies<K>, 0)) {
                    todo = 0;
                    if (again && there) {
                        exact_column();
#pragma unroll
                        for (int x = 0; x < K; ++x) tp[x] = tid_[x] < 0 ? -1.0f : tp[x], tid_[x] = max(tid_[x], 0);
                    }
                }
                for (; __builtin_expect(todo != 0, 0); todo &= todo - 1) {
                    const int from = __builtin_ctzll(todo);
                    const uint32_t its_q0 = __builtin_amdgcn_readlane(static_cast<int>(q0), from);
                    const uint32_t its_q1 = __builtin_amdgcn_readlane(static_cast<int>(q1), from);
                    const Ranked r = rank_column<K, KA>(its_q0, its_q1, l_rec, cm, cp, fp);
#pragma unroll
                    for (int x = 0; x < K; ++x) {
                        const float p = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r.p), x));
                        const int id = __builtin_amdgcn_readlane(r.id, x);
                        if (lane == from) tp[x] = p, tid_[x] = max(id, 0);
                    }
                }
#pragma unroll
                for (int x = 0; x < K; ++x) gone[x] = __float_as_int(tp[x]) >> 31;
            }
        } else {
            uint32_t rec = l_rec[q0];
            for (uint32_t q = q0; q < (there ? q1 : q0); ++q) {
                const int i = static_cast<int>((rec & 0xffffu) >> 2), fb = static_cast<int>(rec >> 18);
                rec = l_rec[q + 1];                 // the next tuple's record is on its way while this one is worked on
                const float pb = fp[fb];
                uint64_t ma[KA];
                float pa[KA];
#pragma unroll
                for (int x = 0; x < KA; ++x) { ma[x] = cm[i + x]; pa[x] = cp[i + x]; }
                const uint64_t mb = uint64_t(1) << fb, bad = rival[fb];
                // kept proofs hold at most one fact per exclusion group, so the union is inconsistent exactly when
                // the first operand's proof holds a rival of the one fact the second brings.  The product over
                // ascending facts is unchanged when the fact is already there, takes one more factor when it lies
                // above every fact of the proof (ma < mb as integers), and is redone from scratch otherwise.
#pragma unroll
                for (int x = 0; x < KA; ++x) {
                    const bool ok = ma[x] != kAbsent && !(ma[x] & bad);
                    const bool plain = (ma[x] & mb) || ma[x] < mb;
                    float pr = (ma[x] & mb) ? pa[x] : pa[x] * pb;
                    if (ok && !plain) pr = proof_prob(ma[x] | mb, fp);
                    const int id = static_cast<int>(q) << 3 | x;
                    bool tie = false;
#pragma unroll
                    for (int y = 0; y < K; ++y) tie |= pr == tp[y];
                    if (ok && tie) insert_tied(ma[x] | mb, pr, id);
                    else insert_untied(ok ? pr : kNone, id);
                }
            }
            by_origin();
        }
        uint64_t wm[K];
#pragma unroll
        for (int x = 0; x < K; ++x) wm[x] = mask_of(tid_[x]) | static_cast<uint64_t>(static_cast<int64_t>(gone[x]));
        // a Distribution of at most 64 symbols is replaced in place: every lane has read what it needs by now
        wave_lds_fence();
        if (!there) continue;
#pragma unroll
        for (int x = 0; x < K; ++x) {
            nm[c * K + x] = wm[x];
            np[c * K + x] = __int_as_float((gone[x] & __float_as_int(-1.0f)) | (~gone[x] & __float_as_int(tp[x])));
        }
        if (last) {
            float sum = 0.0f;
#pragma unroll
            for (int x = 0; x < K; ++x) sum = gone[x] ? sum : sum + tp[x];
            const float pr = fminf(sum, 1.0f);
            A.oprob[s * A.ldo + c] = pr;
            if (A.gfact) {                      // upstream gradient, gated by the clamp (passes on sum <= 1)
                float g;
                if (A.target) g = c == A.target[s] ? -1.0f / fmaxf(pr, FLT_MIN) : 0.0f;
                else g = A.gout[s * A.ldg + c];
                gh[c] = sum <= 1.0f ? g : 0.0f;
            }
        }
    }
}

template <int K, bool MANY>
__global__ void __launch_bounds__(kDfWaves * kWave)
dtkp_fold_kernel(const DtkpFoldArgs A)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    // shared by the workgroup: rivals, symbol side; then per wavefront: masks and probabilities (two buffers where a
    // Distribution has more than 64 symbols, else one), fact probabilities, gated gradients
    uint64_t *rival = reinterpret_cast<uint64_t *>(lds_raw);
    uint32_t *const wl = reinterpret_cast<uint32_t *>(rival + 64);
    const uint32_t *w = wl;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int bufs = A.max_s > kWave ? 2 : 1, flip = (bufs - 1) * A.max_s * K;
    const int n_words = A.n_words + (MANY ? A.n_shares : 0);
    unsigned char *mine_lds = lds_raw + 64 * sizeof(uint64_t) + sizeof(uint32_t) * n_words +
                              static_cast<size_t>(wave) * A.wave_bytes;
    uint64_t *bufm = reinterpret_cast<uint64_t *>(mine_lds);
    float *bufp = reinterpret_cast<float *>(bufm + bufs * A.max_s * K);
    float *fp = bufp + bufs * A.max_s * K;
    float *gh = fp + 64;
    const int64_t s = static_cast<int64_t>(blockIdx.x) * (blockDim.x / kWave) + wave;
    const bool live = s < A.batch;
    const float my_fp = live && lane < A.n_facts ? A.fact_prob[s * A.n_facts + lane] : 1.0f;
    {   // 16 bytes per lane and two loads in flight: the words are the same for every sample and sit in L2, so what
        // this costs is round trips
        uint4 *dst = reinterpret_cast<uint4 *>(wl);
        const uint4 *src = reinterpret_cast<const uint4 *>(A.words);
        const int n4 = n_words / 4, step = blockDim.x;      // the host pads the array to whole 16-byte pieces
        for (int base = threadIdx.x; base < n4; base += 2 * step) {
            const uint4 v0 = src[base], v1 = src[min(base + step, n4 - 1)];
            dst[base] = v0;
            if (base + step < n4) dst[base + step] = v1;
        }
        if (threadIdx.x < 64) rival[threadIdx.x] = static_cast<int>(threadIdx.x) < A.n_facts ? A.rival[threadIdx.x] : 0;
    }
    fp[lane] = my_fp;
    const float next_fp = dpp<0x101>(my_fp);                                // row_shl:1
    const bool equal = lane + 1 < A.n_facts && (lane & 15) != 15 && my_fp == next_fp;
    const bool plain = __ballot(__float_as_uint(my_fp) >= 0x7f800000u) == 0 && 8 * __builtin_popcountll(__ballot(equal)) <= A.n_facts;
    __syncthreads();
    if (!live) return;                          // no barrier of the workgroup follows
    {   // natural initialisation (App. A.1)
        const int S0 = static_cast<int>(w[1]);
        const uint32_t *fact0 = w + w[2];
        for (int i = lane; i < S0; i += kWave) {
            const int f = static_cast<int>(fact0[i]);
            bufm[i * K] = uint64_t(1) << f;
            bufp[i * K] = 1.0f * fp[f];
            // (one proof to a symbol, and the first stage reads no more)
        }
    }
    wave_lds_fence();
    int S = 0;
    auto stage = [&](int t, auto slots) {
        constexpr int KA = decltype(slots)::value;
        const uint64_t *cm = bufm + ((t - 1) & 1) * flip;
        const float *cp = bufp + ((t - 1) & 1) * flip;
        uint64_t *nm = bufm + (t & 1) * flip;
        float *np = bufp + (t & 1) * flip;
        S = __builtin_amdgcn_readfirstlane(static_cast<int>(w[1 + 4 * t]));
        const uint32_t *l_ptr = w + w[2 + 4 * t], *l_rec = w + w[3 + 4 * t];
        const int kind = __builtin_amdgcn_readfirstlane(static_cast<int>(w[4 + 4 * t]));
        const bool last = t == A.n - 1;
        const uint32_t *shares = w + A.n_words + kWave * (kind >> kShareShift);
        if (__builtin_expect(kind & kFresh, kFresh))
            dtkp_fold_stage<K, KA, true, MANY>(A, s, S, last, l_ptr, l_rec, cm, cp, nm, np, rival, fp, gh, plain, kind, shares);
        else
            dtkp_fold_stage<K, KA, false, MANY>(A, s, S, last, l_ptr, l_rec, cm, cp, nm, np, rival, fp, gh, plain, kind, shares);
        wave_lds_fence();
    };
    stage(1, std::integral_constant<int, 1>{});         // the first operand is naturally initialised: one proof per symbol
    for (int t = 2; t < A.n; ++t) stage(t, std::integral_constant<int, K>{});
    // the proofs leave as one contiguous run per sample, in the order they have in LDS
    const uint64_t *fm = bufm + ((A.n - 1) & 1) * flip;
    {
        const float *fq = bufp + ((A.n - 1) & 1) * flip;
        const int64_t o = s * S * K;
        for (int e = lane; e < S * K; e += kWave) {
            A.om[o + e] = fm[e];
            A.op[o + e] = fmaxf(fq[e], 0.0f);
        }
    }
    if (!A.gfact) return;
    // d Pr / d p_f = sum over the kept proofs holding f of the product of their other facts (ascending symbol, rank).
    // Lane f owns fact f and holds its probability; a proof is the same for all lanes, so its facts are walked with
    // scalar instructions and their probabilities read from the lanes that own them.  Columns without a gradient
    // (all but one under a target) are passed over.
    const uint64_t mine = uint64_t(1) << lane;
    float acc = 0.0f;
    for (int base = 0; base < S; base += kWave) {
        const int c = base + lane;
        const float g_l = c < S ? gh[c] : 0.0f;
        for (uint64_t todo = __ballot(g_l != 0.0f); todo; todo &= todo - 1) {
            const int cl = __builtin_ctzll(todo);
            const float g = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g_l), cl));
#pragma unroll
            for (int x = 0; x < K; ++x) {
                const uint64_t raw = fm[(base + cl) * K + x];
                const uint32_t mm_lo = __builtin_amdgcn_readfirstlane(static_cast<int>(raw));
                const uint32_t mm_hi = __builtin_amdgcn_readfirstlane(static_cast<int>(raw >> 32));
                const uint64_t mm = static_cast<uint64_t>(mm_hi) << 32 | mm_lo;
                if (mm == kAbsent) continue;
                float others = 1.0f;
                for (uint64_t r = mm; r; r &= r - 1) {
                    const int j = __builtin_ctzll(r);
                    const float pj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_fp), j));
                    // (1 to the lane whose fact it is)
                    others = others * (__builtin_amdgcn_inverse_ballot_w64(r & -r) ? 1.0f : pj);
                }
                if (mm & mine) acc = __builtin_fmaf(g, others, acc);
            }
        }
    }
    if (lane < A.n_facts) A.gfact[s * A.n_facts + lane] = acc;
}

}  // namespace dol

using namespace dol;

namespace {

// The symbol side of a fold: a function of the tables, the facts of the inputs' symbols and the exclusion groups, kept by
// content (building it takes as long as the launch itself).
struct DtkpFoldPlan {
    DevArray<int32_t> words;
    DevArray<uint64_t> rival;
    int32_t n_words = 0, n_shares = 0, max_s = 0, s_last = 0;
    int waves = 0;                      // wavefronts (samples) of a workgroup
    size_t wave_bytes = 0, lds = 0;     // LDS of one, and of the workgroup
    bool wide = false;                  // lanes help in a stage of more than 32 columns
    bool looked_up = false;             // many samples take the build whose lanes look their shares up (share_lookup_pays)

    size_t share_bytes() const { return sizeof(uint32_t) * static_cast<size_t>(n_shares); }
    bool many(int32_t batch) const { return looked_up && batch > kManySamples; }
};

Cache<DtkpFoldPlan> &g_fold_plans = *new Cache<DtkpFoldPlan>;      // never destroyed, as the other plan caches

// How a stage's lanes help (Kind), and their shares where they do: the columns in their order, and the other lanes help with those
// of more than `most` tuples, which is the smallest number so that all of these get one.
int32_t add_shares(const dol_fn_table *f, std::vector<int32_t> &shares)
{
    const int S = f->n_out;
    if (S > kWave) return 0;
    auto length = [&](int c) { return static_cast<int>(f->h_col_ptr[c + 1] - f->h_col_ptr[c]); };
    auto above = [&](int most) {
        int count = 0;
        for (int c = 0; c < S; ++c) count += length(c) > most;
        return count;
    };
    int longest = 0;
    for (int c = 0; c < S; ++c) longest = std::max(longest, length(c));
    int most = (longest + 1) / 2;
    while (S + above(most) > kWave) ++most;
    if (longest - most < kListCost) return 0;
    const size_t at = shares.size();
    shares.resize(at + kWave, static_cast<int32_t>(Share::pack(S - 1, 0, Share::kIdle)));
    for (int c = 0, helper = S; c < S; ++c) {
        const bool two = length(c) > most;
        shares[at + c] = static_cast<int32_t>(Share::pack(c, two ? helper : c, two ? Share::kFirstHalf : Share::kWhole));
        if (two) shares[at + helper++] = static_cast<int32_t>(Share::pack(c, c, Share::kHelper));
    }
    return S <= kWave / 2 ? kHelped | kTwins : kHelped;
}

using FoldKernel = void (*)(const DtkpFoldArgs);

template <bool MANY>
FoldKernel fold_kernel(int k)
{
    static const FoldKernel of_k[DOL_MAX_K] = {
        dtkp_fold_kernel<1, MANY>, dtkp_fold_kernel<2, MANY>, dtkp_fold_kernel<3, MANY>, dtkp_fold_kernel<4, MANY>,
        dtkp_fold_kernel<5, MANY>, dtkp_fold_kernel<6, MANY>, dtkp_fold_kernel<7, MANY>, dtkp_fold_kernel<8, MANY>};
    return of_k[k - 1];
}

constexpr size_t kDfLds = 64 * 1024;    // most LDS of a workgroup

// The workgroup's wavefronts: as many as fit (the symbol side is a third of a lone wavefront's LDS for Sum-6 at k = 5, so four of
// them together fit a compute unit 28 times over instead of 11).
void set_workgroup(DtkpFoldPlan *p, int K)
{
    const size_t bufs = p->max_s > kWave ? 2 : 1;
    const size_t shared = 64 * sizeof(uint64_t) + sizeof(uint32_t) * static_cast<size_t>(p->n_words);
    p->wave_bytes = (bufs * p->max_s * K * (sizeof(uint64_t) + sizeof(float)) + sizeof(float) * (64 + p->max_s) + 15) & ~size_t(15);
    p->waves = kDfWaves;
    while (p->waves > 1 && shared + p->waves * p->wave_bytes > kDfLds) p->waves /= 2;
    p->lds = shared + p->waves * p->wave_bytes;
}

// Whether many samples (kManySamples) take the build whose lanes look their shares up: where a stage of more than 32 columns
// gets help, which twins cannot give, and a unit holds as many workgroups as without.  12 000 samples, us, twins / looked up:
//   Sum-6, k = 5, 20 000 samples 82.0 / 76.8; sums of six digits modulo 40, k = 5 47.9 / 45.2; products of three digits, k = 3
//   43.4 / 40.9
//   no such stage: sums of six digits modulo 30, 120 columns at last, k = 3 40.5 / 42.0; modulo 20, 300 at last, k = 5 140 / 145;
//   modulo 12, k = 5 61.3 / 64.3; without a last one modulo 32, k = 5 42.2 / 41.3; Sum-3, k = 5, 20 000 samples 30.6 / 29.9
//   a workgroup less for want of registers, k = 8 (four wavefronts to a SIMD instead of five): Sum-6, 20 000 samples 166 / 174,
//   modulo 40 93 / 97; modulo 36 with 100 columns at last, whose LDS leaves three workgroups either way, 149 / 145
//   a workgroup less for want of LDS: five digits modulo 50, 300 columns at last, k = 1, 40.6 KB or 41.4: 4 096 samples 12.4 / 16.3
// (How few wavefronts a SIMD holds does not decide: with one of them modulo 40, 200 columns at last, k = 5 159 / 157 and modulo 50,
// 300 at last, k = 4 131 / 134.)
bool share_lookup_pays(const DtkpFoldPlan &p, int K)
{
    if (!p.wide || p.lds + p.share_bytes() > kDfLds) return false;
    auto workgroups = [&](FoldKernel kernel, size_t lds) {
        int n = 0;
        const void *const entry = reinterpret_cast<const void *>(kernel);
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, entry, p.waves * kWave, lds);
        if (e != hipSuccess) (void)hipGetLastError();
        return e == hipSuccess ? n : 0;
    };
    const int own = workgroups(fold_kernel<false>(K), p.lds);
    return own > 0 && workgroups(fold_kernel<true>(K), p.lds + p.share_bytes()) >= own;
}

dol_status build_plan(const dol_dtkp_fold *fold, const dol_prov *prov, DtkpFoldPlan *p)
{
    const int n = fold->n_inputs, K = prov->k;
    std::vector<int32_t> words(1 + 4 * static_cast<size_t>(n), 0);
    words[0] = n;
    std::vector<int32_t> shares;
    int32_t s_prev = 0;
    int32_t fact_hi = -1;                   // highest fact of the inputs so far
    bool distinct = true;                   // see fresh_t, bit 1
    uint64_t facts_seen = 0;
    for (int t = 0; t < n; ++t) {
        const dol_dist *d = fold->inputs[t];
        const int32_t *fos = fold->fact_of_sym[t];
        for (int32_t i = 0; i < d->n_sym; ++i)
            if (fos[i] < 0 || fos[i] >= prov->n_facts)
                return fail(DOL_EINVAL, "fact_of_sym[%d][%d] = %d outside 0..%d", t, i, fos[i], prov->n_facts - 1);
        {   // fresh_t: this input's facts lie above every earlier fact and share no exclusion group with one
            bool fresh = true;
            uint64_t mine = 0;
            for (int32_t i = 0; i < d->n_sym; ++i) {
                fresh = fresh && fos[i] > fact_hi;
                mine |= uint64_t(1) << fos[i];
            }
            for (int f = 0; f < prov->n_facts && prov->fact_group && fresh; ++f)
                for (int h = 0; h < prov->n_facts && ((mine >> f) & 1); ++h)
                    if (((facts_seen >> h) & 1) && prov->fact_group[h] == prov->fact_group[f]) fresh = false;
            distinct = distinct && fresh && __builtin_popcountll(mine) == d->n_sym;
            words[4 + 4 * t] = (fresh ? kFresh : 0) | (distinct ? kDistinct : 0);
            for (int32_t i = 0; i < d->n_sym; ++i) fact_hi = std::max(fact_hi, fos[i]);
            facts_seen |= mine;
        }
        if (t == 0) {
            words[1] = d->n_sym;
            words[2] = static_cast<int32_t>(words.size());
            words.insert(words.end(), fos, fos + d->n_sym);
            s_prev = p->s_last = p->max_s = d->n_sym;
            continue;
        }
        const dol_fn_table *f = fold->tables[t - 1];
        if (f->na != s_prev || f->nb != d->n_sym)
            return fail(DOL_ESHAPE, "tables[%d] is %d x %d, its operands have %d and %d symbols", t - 1, f->na, f->nb, s_prev, d->n_sym);
        if (f->n_out < 1) return fail(DOL_EUNSUPPORTED, "tables[%d] produces no symbol", t - 1);
        // (a list's place in 16 bits; wider Distributions' lists do not fit in LDS either)
        if (4 * static_cast<int64_t>(K) * s_prev > 0xffff) return fail(DOL_EUNSUPPORTED, "the proofs of the fold do not fit in LDS");
        if (words.size() + static_cast<size_t>(f->n_out) + static_cast<size_t>(f->n_tuples) + 3 > 16000)
            return fail(DOL_EUNSUPPORTED, "the tables of the fold do not fit in LDS");
        words[1 + 4 * t] = f->n_out;
        words[2 + 4 * t] = static_cast<int32_t>(words.size());
        words.insert(words.end(), f->h_col_ptr.begin(), f->h_col_ptr.begin() + f->n_out + 1);
        words[3 + 4 * t] = static_cast<int32_t>(words.size());
        for (int64_t q = 0; q < f->n_tuples; ++q) {
            const uint32_t ij = f->h_col_ij[static_cast<size_t>(q)];
            words.push_back(static_cast<int32_t>((4u * K * (ij & 0xffffu)) | (static_cast<uint32_t>(fos[ij >> 16]) << 18)));
        }
        words.insert(words.end(), 2, 0);
        if (words[4 + 4 * t] & kFresh) {
            words[4 + 4 * t] |= static_cast<int32_t>(shares.size() / kWave) << kShareShift;
            const int32_t help = add_shares(f, shares);
            words[4 + 4 * t] |= help;
            p->wide |= help == kHelped;
        }
        s_prev = p->s_last = f->n_out;
        p->max_s = std::max(p->max_s, f->n_out);
    }
    while (words.size() % 4) words.push_back(0);
    p->n_words = static_cast<int32_t>(words.size());
    p->n_shares = static_cast<int32_t>(shares.size());
    words.insert(words.end(), shares.begin(), shares.end());
    std::vector<uint64_t> rival(static_cast<size_t>(prov->n_facts), 0);      // the other facts of each fact's exclusion group
    for (int f = 0; f < prov->n_facts && prov->fact_group; ++f)
        for (int h = 0; h < prov->n_facts; ++h)
            if (h != f && prov->fact_group[h] == prov->fact_group[f]) rival[f] |= uint64_t(1) << h;
    hipError_t e;
    if ((e = p->words.upload(words)) != hipSuccess || (e = p->rival.upload(rival)) != hipSuccess)
        return hip_fail(e, "uploading the fold's tables");
    set_workgroup(p, K);
    p->looked_up = share_lookup_pays(*p, K);
    return DOL_OK;
}

dol_status get_plan(const dol_dtkp_fold *fold, const dol_prov *prov, const DtkpFoldPlan **plan)
{
    int device = 0;
    (void)hipGetDevice(&device);
    const int n = fold->n_inputs;
    std::vector<int32_t> desc{n, prov->k, prov->n_facts, prov->fact_group ? 1 : 0};
    desc.reserve(4 + static_cast<size_t>(prov->n_facts) + 24 * static_cast<size_t>(n));
    if (prov->fact_group) desc.insert(desc.end(), prov->fact_group, prov->fact_group + prov->n_facts);
    for (int t = 0; t < n; ++t) {
        const uint64_t uid = t ? fold->tables[t - 1]->uid : 0;
        desc.insert(desc.end(), {static_cast<int32_t>(uid), static_cast<int32_t>(uid >> 32), fold->inputs[t]->n_sym});
        desc.insert(desc.end(), fold->fact_of_sym[t], fold->fact_of_sym[t] + fold->inputs[t]->n_sym);
    }
    std::vector<unsigned char> key = make_key(device, {{desc.data(), sizeof(int32_t) * desc.size()}});
    const uint64_t h = hash_bytes(key.data(), key.size());
    std::lock_guard<std::mutex> lock(g_fold_plans.mu);
    if ((*plan = g_fold_plans.find(h, key)) != nullptr) return DOL_OK;
    std::unique_ptr<DtkpFoldPlan> p(new (std::nothrow) DtkpFoldPlan);
    if (!p) return fail(DOL_ENOMEM, "out of host memory");
    if (dol_status st = build_plan(fold, prov, p.get())) return st;
    *plan = g_fold_plans.insert(h, std::move(key), std::move(p));
    return DOL_OK;
}

}  // namespace

// Checks the call's description as far as its shapes; the fold's plan.
static dol_status fold_checked(const dol_dtkp_fold *fold, const dol_prov *prov, const DtkpFoldPlan **plan)
{
    if (!fold || !prov) return fail(DOL_EINVAL, "NULL argument");
    if (prov->kind != DOL_DTKP) return fail(DOL_EINVAL, "dol_dtkp_fold_apply2 needs a DTKP provenance");
    const int n = fold->n_inputs, K = prov->k;
    if (n < 2 || n > kDfMax) return fail(n < 2 ? DOL_EINVAL : DOL_EUNSUPPORTED, "n_inputs = %d outside 2..%d", n, kDfMax);
    if (K < 1 || K > DOL_MAX_K) return fail(DOL_EINVAL, "k = %d outside 1..%d", K, DOL_MAX_K);
    if (prov->n_facts < 1 || prov->n_facts > 63) return fail(DOL_EINVAL, "n_facts = %d outside 1..63", prov->n_facts);
    if (!fold->inputs || !fold->tables || !fold->fact_of_sym || !fold->out) return fail(DOL_EINVAL, "inputs, tables, fact_of_sym or out is NULL");
    for (int t = 0; t < n; ++t) {
        const dol_dist *d = fold->inputs[t], *d0 = fold->inputs[0];
        if (!d) return fail(DOL_EINVAL, "inputs[%d] is NULL", t);
        if (d->batch < 0 || d->n_sym < 1) return fail(DOL_ESHAPE, "inputs[%d] has a bad shape", t);
        if (d->batch != d0->batch) return fail(DOL_ESHAPE, "inputs[%d].batch = %d, inputs[0].batch = %d", t, d->batch, d0->batch);
        if (!fold->fact_of_sym[t]) return fail(DOL_EINVAL, "fact_of_sym[%d] is NULL", t);
        if (t && !fold->tables[t - 1]) return fail(DOL_EINVAL, "tables[%d] is NULL", t - 1);
    }
    if (dol_status st = get_plan(fold, prov, plan)) return st;
    const dol_dist *o = fold->out;
    const int32_t batch = fold->inputs[0]->batch, s_last = (*plan)->s_last;
    if (o->batch != batch || o->n_sym != s_last || o->ld < o->n_sym)
        return fail(DOL_ESHAPE, "out has %d x %d, the fold produces %d x %d", o->batch, o->n_sym, batch, s_last);
    if ((*plan)->lds > kDfLds)
        return fail(DOL_EUNSUPPORTED, "the fold needs %zu bytes of LDS per sample, more than %zu", (*plan)->lds, kDfLds);
    return DOL_OK;
}

extern "C" const char *dol_dtkp_fold_kernel(const dol_dtkp_fold *fold, const dol_prov *prov)
{
    static thread_local char name[64];
    const DtkpFoldPlan *plan = nullptr;
    if (fold_checked(fold, prov, &plan) != DOL_OK) return "";
    snprintf(name, sizeof name, "dtkp_fold_kernel<%d, %s>", prov->k, plan->many(fold->inputs[0]->batch) ? "true" : "false");
    return name;
}

extern "C" dol_status dol_dtkp_fold_apply2(const dol_dtkp_fold *fold, const dol_prov *prov, void *hip_stream)
{
    const DtkpFoldPlan *plan = nullptr;
    if (dol_status st = fold_checked(fold, prov, &plan)) return st;
    const int K = prov->k;
    const int32_t s_last = plan->s_last;
    const dol_dist *o = fold->out;
    DtkpFoldArgs A{};
    A.n = fold->n_inputs;
    A.batch = fold->inputs[0]->batch;
    A.n_facts = prov->n_facts;
    A.max_s = plan->max_s;
    A.n_words = plan->n_words;
    A.n_shares = plan->n_shares;
    A.words = plan->words.ptr;
    A.rival = plan->rival.ptr;
    const bool many = plan->many(A.batch);
    const int waves = plan->waves;
    const size_t lds = plan->lds + (many ? plan->share_bytes() : 0);
    A.wave_bytes = static_cast<int32_t>(plan->wave_bytes);
    if (A.batch == 0) return DOL_OK;
    if (!o->proof_mask || !o->proof_prob || !o->prob) return fail(DOL_EINVAL, "out.proof_mask, out.proof_prob or out.prob is NULL");
    if (!prov->fact_prob) return fail(DOL_EINVAL, "prov.fact_prob is NULL");
    A.fact_prob = prov->fact_prob;
    A.om = o->proof_mask;
    A.op = o->proof_prob;
    A.oprob = o->prob;
    A.ldo = o->ld;
    A.gfact = fold->grad_fact_prob;
    A.target = fold->target_col;
    A.gout = fold->grad_out;
    A.ldg = fold->grad_out_ld;
    if (A.gfact && !A.target) {
        if (!A.gout) return fail(DOL_EINVAL, "grad_fact_prob needs target_col or grad_out");
        if (A.ldg < s_last) return fail(DOL_ESHAPE, "grad_out_ld = %lld is smaller than %d", static_cast<long long>(A.ldg), s_last);
    }
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const dim3 grid(static_cast<unsigned>((static_cast<int64_t>(A.batch) + waves - 1) / waves));
    const dim3 block(static_cast<unsigned>(waves * kWave));
    hipLaunchKernelGGL(many ? fold_kernel<true>(K) : fold_kernel<false>(K), grid, block, lds, st, A);
    DOL_HIP(hipGetLastError());
    return DOL_OK;
}
