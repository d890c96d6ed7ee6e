// DTKP-AM provenance kernels (Sec. 3.2, Table 1, App. A) for gfx950, on the bitmask encoding of proofs:
// a proof is the 64-bit set of input facts it uses; its probability is the float product of the facts'
// probabilities in ascending fact index starting from 1 (absent symbols contribute 1, Sec. 3.2).
// The set union of two proofs (the paper's element-wise minimum, App. A.1) is a bitwise OR.
//
// One thread owns one (sample, output symbol) and streams every candidate proof through a k-entry sorted
// list held in registers.  Repeated proofs are one proof, so insertion first looks the mask up; the list
// order (higher probability first, ties by smaller mask) is total on distinct masks, which makes the
// result independent of the order candidates arrive in.
#include "dtkp_columns.h"

#include <algorithm>

namespace dol {

constexpr int kThreadsT = 128;

static inline unsigned grid_t(int64_t work) { return static_cast<unsigned>((work + kThreadsT - 1) / kThreadsT); }

// ---------------------------------------------------------------- init

__global__ void __launch_bounds__(kThreadsT)
dtkp_init_kernel(int64_t total, int32_t n_sym, int32_t k, int32_t n_facts, const int32_t *__restrict__ fact_of_sym,
                 const float *__restrict__ fact_prob, uint64_t *__restrict__ mask, float *__restrict__ pprob,
                 float *__restrict__ prob, int64_t ld)
{
    const int64_t idx = static_cast<int64_t>(blockIdx.x) * kThreadsT + threadIdx.x;
    if (idx >= total) return;
    const int64_t s = idx / n_sym;
    const int32_t i = static_cast<int32_t>(idx - s * n_sym);
    const int32_t f = fact_of_sym[i];
    const float pr = 1.0f * fact_prob[s * n_facts + f];
    mask[idx * k] = uint64_t(1) << f;
    pprob[idx * k] = pr;
    for (int x = 1; x < k; ++x) { mask[idx * k + x] = kAbsent; pprob[idx * k + x] = 0.0f; }
    prob[s * ld + i] = fminf(pr, 1.0f);
}

dol_status launch_dtkp_init(int32_t batch, int32_t n_sym, int32_t k, int32_t n_facts, const int32_t *d_fact_of_sym,
                            const float *fact_prob, uint64_t *mask, float *pprob, float *prob, int64_t ld,
                            hipStream_t st)
{
    const int64_t total = static_cast<int64_t>(batch) * n_sym;
    if (total == 0) return DOL_OK;
    hipLaunchKernelGGL(dtkp_init_kernel, dim3(grid_t(total)), dim3(kThreadsT), 0, st, total, n_sym, k, n_facts,
                       d_fact_of_sym, fact_prob, mask, pprob, prob, ld);
    DOL_HIP(hipGetLastError());
    return DOL_OK;
}

// ---------------------------------------------------------------- apply2

struct PairArgs {
    int32_t S, na, nb, n_facts;
    const uint32_t *col_ij, *ord_tuples;
    const float *fact_prob;
    const uint64_t *am, *bm;
    const float *ap, *bp;
    // the second operand is an input Distribution under natural initialisation: its symbol is one fact, its tag the single
    // proof {that fact} (App. A.1); nothing of it is stored.  fact_b holds four words per symbol: the fact and the mask of
    // the other facts of its exclusion group (low, high word).
    const int32_t *fact_b;
    int32_t shared_facts;               // the second operand's symbols whose four words wait in LDS: all or none
};

constexpr int kSharedFacts = 64;        // most of them

// What a kernel takes as the second operand.  (Up to kKeyProofs proofs each has a kernel of its own: in one for both the lists'
// general union and the facts' keys share 70 registers at k = 3 and 75 at k = 4, apart 56 and 64, 60 and 72.  Tables as below, us,
// one kernel and two: lists 3 000 x 20 -> 6 000, k = 2 228 and 198, 3 000 x 10 -> 8 000, k = 3 40.6 and 39.2; facts, k = 4 23.5 and
// 21.4.  Longer lists have no keys, and their facts neither wait in LDS nor are their words read ahead: at k = 5 that took 83
// registers instead of 77, lists 54.0 us instead of 51.9, facts 28.3 instead of 27.2; facts in a kernel apart 29.0 with k = 5 and
// 385 instead of 361 with k = 6.)
enum class Second { kLists, kFacts, kEither };

// Offers every consistent union of a proof of a's symbol with a proof of b's symbol, tuple by tuple.
template <int K, Second SECOND>
struct PairOffer {
    static constexpr bool kShared = SECOND == Second::kFacts;
    // (facts of one probability, table 300 x 40 -> 700, 100 samples, us, two ways / one: k = 3 21.6 / 20.0, 4 34.0 / 32.9, 5 38.9 /
    // 40.4, 7 72.8 / 82.2; softmax k = 3 15.7 / 15.9, 5 27.3 / 32.3, 7 45.3 / 60.3)
    static constexpr bool kOneWay = SECOND != Second::kEither;
    const PairArgs &A;
    const GroupMasks &gm;
    const float *fp;
    int64_t a0, b0;
    uint4 mine;                         // what this thread brings to LDS
    uint32_t first;                     // the lane's first tuple

    // in LDS: the facts, then a lane's masks (run_short)
    static __device__ __forceinline__ uint4 *facts()
    {
        extern __shared__ __align__(16) uint64_t dtkp_lds[];
        return reinterpret_cast<uint4 *>(dtkp_lds);
    }
    __device__ __forceinline__ uint64_t *lane_masks() const { return reinterpret_cast<uint64_t *>(facts() + A.shared_facts); }
    __device__ __forceinline__ void ask()
    {
        if (kShared && static_cast<int>(threadIdx.x) < A.shared_facts)
            mine = reinterpret_cast<const uint4 *>(A.fact_b)[threadIdx.x];
    }
    __device__ __forceinline__ void share() const
    {
        if (!kShared || A.shared_facts == 0) return;
        if (static_cast<int>(threadIdx.x) < A.shared_facts) facts()[threadIdx.x] = mine;
        lds_barrier();
    }
    // (a tuple's fact is known before its probability can be asked for: from LDS that costs no round trip to memory)
    __device__ __forceinline__ uint4 fact_of(uint32_t j) const
    {
        uint4 f;
        if (kShared && A.shared_facts) {
            f = facts()[j];
            asm volatile("" : "+v"(f.x));       // (or both loads become one of either memory, which waits for the lists too)
        } else {
            f = reinterpret_cast<const uint4 *>(A.fact_b)[j];
        }
        return f;
    }
    __device__ __forceinline__ void ahead(uint32_t r) { first = A.ord_tuples[r]; }
    __device__ __forceinline__ void begin(int64_t s)
    {
        fp = A.fact_prob + s * A.n_facts;
        a0 = s * A.na * K, b0 = s * A.nb * K;
    }
    // The first operand's proofs hold at most one fact per exclusion group, so the union is inconsistent exactly when such a
    // proof holds a rival of the one fact the second operand brings.  The product over ascending facts is unchanged when the
    // fact is already there, takes one more factor when it lies above every fact of the proof (ma < bit as integers), and
    // is redone from scratch otherwise.
    __device__ __forceinline__ void with_fact(TopK<K> &top, const uint4 &f, const uint64_t (&ma)[K], const float (&pa)[K]) const
    {
        const uint64_t bit = uint64_t(1) << f.x, rival = (static_cast<uint64_t>(f.z) << 32) | f.y;
        const float pbit = 1.0f * fp[f.x];
#pragma unroll
        for (int x = 0; x < K; ++x) {
            if (ma[x] == kAbsent || (ma[x] & rival)) continue;
            const bool held = (ma[x] & bit) != 0;
            const float pr = A.ap && (held || ma[x] < bit) ? (held ? pa[x] : pa[x] * pbit) : proof_prob(ma[x] | bit, fp);
            top.template insert<kOneWay>(ma[x] | bit, pr);
        }
    }
    __device__ __forceinline__ void with_list(TopK<K> &top, uint32_t j, const uint64_t (&ma)[K], const float (&pa)[K]) const
    {
        const int64_t ib = b0 + static_cast<int64_t>(j) * K;
        uint64_t mb[K];
        float pb[K];
        load_masks<K>(A.bm + ib, mb);
#pragma unroll
        for (int x = 0; x < K; ++x) pb[x] = -1.0f;
        if (A.bp) load_probs<K>(A.bp + ib, pb);
#pragma unroll
        for (int x = 0; x < K; ++x) {
            if (ma[x] == kAbsent) continue;
#pragma unroll
            for (int y = 0; y < K; ++y) {
                if (mb[y] == kAbsent) continue;
                const uint64_t m = ma[x] | mb[y];
                if (proof_conflict(m, gm)) continue;
                top.template insert<kOneWay>(m, union_prob(ma[x], pa[x], mb[y], pb[y], fp));
            }
        }
    }
    // the tuples word(q), word(q + step), .. below q1 (a tuple's word is read while the one before it is worked on)
    template <class Word>
    __device__ __forceinline__ void run(TopK<K> &top, uint32_t q, uint32_t q1, uint32_t step, Word word) const
    {
        for (; q < q1; q += step) {
            const uint32_t ij = word(q), j = ij >> 16;
            const int64_t ia = a0 + static_cast<int64_t>(ij & 0xffffu) * K;
            uint64_t ma[K];
            float pa[K];
            load_masks<K>(A.am + ia, ma);
#pragma unroll
            for (int x = 0; x < K; ++x) pa[x] = -1.0f;
            if (A.ap) load_probs<K>(A.ap + ia, pa);
            if (SECOND == Second::kFacts || (SECOND == Second::kEither && A.fact_b)) with_fact(top, fact_of(j), ma, pa);
            else if constexpr (SECOND != Second::kFacts) with_list(top, j, ma, pa);
        }
    }
    __device__ __forceinline__ void listed(TopK<K> &top, uint32_t q, uint32_t q1, uint32_t step) const
    {
        run(top, q, q1, step, [&](uint32_t x) { return A.col_ij[x]; });
    }
    __device__ __forceinline__ bool has_short() const { return kShared && A.ap; }
    // One tuple's list and fact.
    struct Tuple {
        uint64_t ma[K], bit, rival;
        float pa[K], pbit;
        // the fact is above every fact of all proofs, and no rival of one: mostly so, and one look says it for all of them
        __device__ __forceinline__ bool fresh() const
        {
            uint64_t any = 0;
#pragma unroll
            for (int x = 0; x < K; ++x) any |= ma[x] != kAbsent ? ma[x] : 0;
            return !(any & rival) && any < bit;
        }
        // whether there is a proof of x and the fact, and its probability (see with_fact)
        __device__ __forceinline__ bool joins(int x) const { return ma[x] != kAbsent && !(ma[x] & rival); }
        __device__ __forceinline__ float joint(int x, const float *__restrict__ fp) const
        {
            const bool held = (ma[x] & bit) != 0;
            return held || ma[x] < bit ? (held ? pa[x] : pa[x] * pbit) : proof_prob(ma[x] | bit, fp);
        }
    };
    __device__ __forceinline__ Tuple tuple(uint32_t ij) const
    {
        Tuple t;
        const int64_t ia = a0 + static_cast<int64_t>(ij & 0xffffu) * K;
        const uint4 f = fact_of(ij >> 16);
        load_masks<K>(A.am + ia, t.ma);
        load_probs<K>(A.ap + ia, t.pa);
        t.pbit = 1.0f * fp[f.x];
        t.bit = uint64_t(1) << f.x, t.rival = (static_cast<uint64_t>(f.z) << 32) | f.y;
        return t;
    }
    // (the masks of a lane's few tuples wait in LDS for the winners; a key's id is the candidate's number in its lane, and the
    // lane's thread << 8.  Read again from memory once the winners are known: 192.6 us for the formula's pass, 184.2 so.)
    // ahead: word(q)
    template <class Word>
    __device__ __forceinline__ void run_short(TopKeys<K> &keys, uint32_t q, uint32_t q1, uint32_t step, uint32_t ahead,
                                              Word word) const
    {
        static_assert(K * kLongDtkpCol <= 256 || K > kKeyProofs, "a candidate's number");
        uint64_t *put = lane_masks() + threadIdx.x;
        int id = threadIdx.x << 8;
        for (; q < q1; q += step, id += K, put += K * blockDim.x) {
            const Tuple t = tuple(ahead);
            ahead = word(min(q + step, q1 - 1));
            // (uniform.  Where lanes took one way each, after both, facts that are held already, below others or rivals cost up to
            // a quarter of the launch; us, so and now: table 3 000 x 10 -> 3 000, 64 samples, k = 4 30.7 and 25.1, 3 000 x 20 ->
            // 6 000, 300 samples, k = 2 114 and 94, 300 x 40 -> 700 with 16 lanes to a column, 100 samples, k = 3 14.0 and 12.5.
            // One candidate after the other there too: 11.5, and where facts are new 16.7 instead of 15.7)
            if (__ballot(!t.fresh()) == 0) {
                float pr[K];
                bool ok[K], falls = true;
#pragma unroll
                for (int x = 0; x < K; ++x) {
                    ok[x] = t.ma[x] != kAbsent;
                    pr[x] = t.pa[x] * t.pbit;
                    put[x * blockDim.x] = t.ma[x] | t.bit;
                    falls &= x == 0 || !ok[x] || (ok[x > 0 ? x - 1 : 0] && pr[x > 0 ? x - 1 : 0] >= pr[x]);
                }
                if (__ballot(!falls) == 0) {
                    keys.offer_falling(ok, pr, id);
                } else {
#pragma unroll
                    for (int x = 0; x < K; ++x) keys.offer(ok[x], pr[x], id + x);
                }
            } else {
#pragma unroll
                for (int x = 0; x < K; ++x) {
                    if (!t.joins(x)) continue;
                    put[x * blockDim.x] = t.ma[x] | t.bit;
                    keys.offer(true, t.joint(x, fp), id + x);
                }
            }
        }
    }
    // A column of one tuple: its candidates are the result unless one before another is no proof, they do not fall, or one's
    // probability is no number to rank by; where that may be it says so.
    __device__ __forceinline__ bool single(TopK<K> &top) const
    {
        const Tuple t = tuple(first);
        bool clear = true;
        float before = __uint_as_float(0x7f800000u);
#pragma unroll
        for (int x = 0; x < K; ++x) {
            if (!t.joins(x)) {
                before = -1.0f;
                continue;
            }
            top.m[x] = t.ma[x] | t.bit, top.p[x] = t.joint(x, fp);
            clear &= __float_as_uint(top.p[x]) < 0x7f800000u && top.p[x] < before;
            before = top.p[x];
        }
        return clear;
    }
    __device__ __forceinline__ void short_listed(TopKeys<K> &keys, uint32_t q, uint32_t q1, uint32_t step) const
    {
        run_short(keys, q, q1, step, q < q1 ? A.col_ij[q] : 0, [&](uint32_t x) { return A.col_ij[x]; });
    }
    __device__ __forceinline__ void short_laned(TopKeys<K> &keys, uint32_t len, int32_t r) const
    {
        run_short(keys, 0, len, 1, first, [&](uint32_t k) { return A.ord_tuples[static_cast<size_t>(k) * A.S + r]; });
    }
    __device__ __forceinline__ bool short_take(TopK<K> &top, const TopKeys<K> &keys, int) const
    {
        const uint64_t *masks = lane_masks();
        wave_lds_fence();
#pragma unroll
        for (int x = 0; x < K; ++x) {
            if (!keys.present(x)) continue;
            top.m[x] = masks[(keys.id(x) & 255) * blockDim.x + (keys.id(x) >> 8)];
            top.p[x] = keys.prob(x);
        }
        return true;
    }
    __device__ __forceinline__ void laned(TopK<K> &top, uint32_t len, int32_t r, uint32_t) const
    {
        run(top, 0, len, 1, [&](uint32_t k) { return A.ord_tuples[static_cast<size_t>(k) * A.S + r]; });
    }
};

template <int K, Second SECOND>
__global__ void __launch_bounds__(kHugeThreads)
dtkp_apply2_kernel(ColumnArgs C, PairArgs A, GroupMasks gm)
{
    dtkp_columns<K>(C, PairOffer<K, SECOND>{A, gm, nullptr, 0, 0, {}, 0});
}

template <int K>
static void launch_apply2_k(ColumnArgs C, const PairArgs &A, const GroupMasks &gm, hipStream_t st)
{
    const dim3 grid(column_launch<K>(C)), block(column_threads(C));
    if constexpr (K > kKeyProofs) {
        hipLaunchKernelGGL((dtkp_apply2_kernel<K, Second::kEither>), grid, block, 0, st, C, A, gm);
    } else if (A.fact_b) {              // a lane's masks: 96 bytes at three proofs
        const size_t lds = sizeof(uint4) * A.shared_facts + sizeof(uint64_t) * block.x * kLongDtkpCol * K;
        hipLaunchKernelGGL((dtkp_apply2_kernel<K, Second::kFacts>), grid, block, lds, st, C, A, gm);
    } else {
        hipLaunchKernelGGL((dtkp_apply2_kernel<K, Second::kLists>), grid, block, 0, st, C, A, gm);
    }
}

#define DOL_DISPATCH_K(k, CALL)                                      \
    switch (k) {                                                     \
    case 1: CALL(1); break;                                          \
    case 2: CALL(2); break;                                          \
    case 3: CALL(3); break;                                          \
    case 4: CALL(4); break;                                          \
    case 5: CALL(5); break;                                          \
    case 6: CALL(6); break;                                          \
    case 7: CALL(7); break;                                          \
    case 8: CALL(8); break;                                          \
    default: return fail(DOL_EINVAL, "k = %d outside 1..%d", k, DOL_MAX_K); \
    }

dol_status launch_dtkp_apply2(const dol_fn_table *f, int32_t batch, int32_t k, int32_t n_facts, const GroupMasks &gm,
                              const float *fact_prob, const uint64_t *am, const float *ap, const uint64_t *bm,
                              const float *bp, const int32_t *fact_b, uint64_t *om, float *op, float *oprob, int64_t ldo,
                              hipStream_t st)
{
    const int64_t total = static_cast<int64_t>(batch) * f->n_out;
    if (total == 0) return DOL_OK;
    if (static_cast<int64_t>(batch) * static_cast<int64_t>(f->dtkp_cols.longer.n) > 0x7fffffffLL)
        return fail(DOL_EUNSUPPORTED, "batch x long table columns exceeds 2^31");
    ColumnArgs C{};
    C.batch = batch, C.S = f->n_out, C.n_in = f->na + (fact_b ? 0 : f->nb);
    C.col_ptr = f->col_ptr.ptr;
    set_columns(C, f->dtkp_cols);
    C.om = om, C.op = op, C.oprob = oprob, C.ldo = ldo;
    const PairArgs A{f->n_out, f->na, f->nb, n_facts, f->col_ij.ptr, f->dtkp_tuples.ptr, fact_prob, am, bm, ap, bp, fact_b,
                     fact_b && f->nb <= kSharedFacts ? f->nb : 0};
#define CALL(KK) launch_apply2_k<KK>(C, A, gm, st)
    DOL_DISPATCH_K(k, CALL)
#undef CALL
    DOL_HIP(hipGetLastError());
    return DOL_OK;
}

// ---------------------------------------------------------------- union

template <int K>
__global__ void __launch_bounds__(kThreadsT)
dtkp_union_kernel(int64_t total, int32_t S, int32_t na, int32_t nb, const int32_t *__restrict__ ia,
                  const int32_t *__restrict__ ib, const uint64_t *__restrict__ am, const float *__restrict__ ap,
                  const uint64_t *__restrict__ bm, const float *__restrict__ bp, uint64_t *__restrict__ om,
                  float *__restrict__ op, float *__restrict__ oprob, int64_t ldo)
{
    const int64_t idx = static_cast<int64_t>(blockIdx.x) * kThreadsT + threadIdx.x;
    if (idx >= total) return;
    const int64_t s = idx / S;
    const int32_t c = static_cast<int32_t>(idx - s * S);
    const int32_t i = ia[c], j = ib[c];
    TopK<K> top;
    top.clear();
    if (i >= 0) {
        const int64_t o = (s * na + i) * K;
#pragma unroll
        for (int x = 0; x < K; ++x)
            if (am[o + x] != kAbsent) top.insert(am[o + x], ap[o + x]);
    }
    if (j >= 0) {
        const int64_t o = (s * nb + j) * K;
#pragma unroll
        for (int x = 0; x < K; ++x)
            if (bm[o + x] != kAbsent) top.insert(bm[o + x], bp[o + x]);
    }
    oprob[s * ldo + c] = top.store(om + idx * K, op + idx * K);
}

dol_status launch_dtkp_union(const UnionPlan *p, int32_t batch, int32_t k, const uint64_t *am, const float *ap,
                             const uint64_t *bm, const float *bp, uint64_t *om, float *op, float *oprob, int64_t ldo,
                             hipStream_t st)
{
    const int64_t total = static_cast<int64_t>(batch) * p->n_out;
    if (total == 0) return DOL_OK;
#define CALL(KK)                                                                                                  \
    hipLaunchKernelGGL(dtkp_union_kernel<KK>, dim3(grid_t(total)), dim3(kThreadsT), 0, st, total, p->n_out, p->na, \
                       p->nb, p->d_ia.ptr, p->d_ib.ptr, am, ap, bm, bp, om, op, oprob, ldo)
    DOL_DISPATCH_K(k, CALL)
#undef CALL
    DOL_HIP(hipGetLastError());
    return DOL_OK;
}

// ---------------------------------------------------------------- filter

__global__ void __launch_bounds__(kThreadsT)
dtkp_filter_kernel(int64_t total, int32_t n_in, int32_t n_out, int32_t k, const int32_t *__restrict__ keep_idx,
                   const uint64_t *__restrict__ im, const float *__restrict__ ip, const float *__restrict__ iprob,
                   int64_t ldi, uint64_t *__restrict__ om, float *__restrict__ op, float *__restrict__ oprob,
                   int64_t ldo)
{
    const int64_t idx = static_cast<int64_t>(blockIdx.x) * kThreadsT + threadIdx.x;
    if (idx >= total) return;
    const int64_t s = idx / n_out;
    const int32_t c = static_cast<int32_t>(idx - s * n_out);
    const int64_t src = (s * n_in + keep_idx[c]) * k;
    for (int x = 0; x < k; ++x) { om[idx * k + x] = im[src + x]; op[idx * k + x] = ip[src + x]; }
    oprob[s * ldo + c] = iprob[s * ldi + keep_idx[c]];
}

dol_status launch_dtkp_filter(const FilterPlan *p, int32_t batch, int32_t k, const uint64_t *im, const float *ip,
                              const float *iprob, int64_t ldi, uint64_t *om, float *op, float *oprob, int64_t ldo,
                              hipStream_t st)
{
    const int64_t total = static_cast<int64_t>(batch) * p->n_out;
    if (total == 0) return DOL_OK;
    hipLaunchKernelGGL(dtkp_filter_kernel, dim3(grid_t(total)), dim3(kThreadsT), 0, st, total, p->n_in, p->n_out, k,
                       p->d_keep_idx.ptr, im, ip, iprob, ldi, om, op, oprob, ldo);
    DOL_HIP(hipGetLastError());
    return DOL_OK;
}

// ---------------------------------------------------------------- gradient of the tag probabilities

// Pr(symbol) = min(1, sum over its kept proofs of the product of their facts' probabilities) (Sec. 3.2); which
// proofs top-k kept is a constant of the differentiation and the clamp passes gradient inside and on its bound
// (App. A.2).  One workgroup per sample; its wavefronts take 64 symbols at a time, a lane per symbol (coalesced loads
// of the proof lists).  A lane folds the clamp's gate and the upstream gradient into one coefficient per proof,
// gradient * proof probability, and adds it to a register accumulator of every fact the proof holds (the loop over
// the facts is unrolled, so the accumulators are plain registers and a fact's test is a bit-field extract).  The
// product of a proof's other facts is its probability divided by the fact's: that division happens once, on the
// accumulator's total (one rounding more than multiplying the facts out, far inside the 1e-5 bar).  A fact of
// probability (nearly) 0 cannot be divided by: its accumulator takes gradient * (the other facts multiplied out, in
// ascending order) instead.  No atomics; the sums run over a lane's symbols in ascending order, then over the lanes
// (exchange tree), then over the wavefronts in order.
// The bit tests bound it (three instructions per proof and fact), and a small batch leaves most units idle: `parts` workgroups
// then share a sample, each for a stretch of the facts (it reads all lists: they come from its XCD's cache), which leaves
// every fact's sum as it is.  (64 samples of 8 334 symbols, k = 3, 49 facts: 33 us with one
// workgroup, 16 with four)
constexpr int kGradWaves = 16;

template <int K>
__global__ void __launch_bounds__(kGradWaves * 64)
dtkp_prob_bwd_kernel(int32_t parts, int32_t n_sym, int32_t n_facts, const uint64_t *__restrict__ mask,
                     const float *__restrict__ pprob, const float *__restrict__ fact_prob,
                     const float *__restrict__ g, int64_t ldg, float *__restrict__ gfact)
{
    __shared__ float part[kGradWaves][64];
    __shared__ float fp[64];
    const int id = xcd_contiguous(blockIdx.x, gridDim.x);
    const int64_t s = id / parts;
    const int octets = (n_facts + 7) / 8, lo = (id - static_cast<int>(s) * parts) * octets / parts * 8;      // this workgroup's facts
    const int hi = min(n_facts, ((id - static_cast<int>(s) * parts) + 1) * octets / parts * 8);
    const int lane = threadIdx.x & 63, n_waves = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));   // tells the compiler it is uniform
    if (wave == 0) fp[lane] = lane < n_facts ? fact_prob[s * n_facts + lane] : 1.0f;
    __syncthreads();
    const float pj = fp[lane];
    const uint64_t tiny = __ballot(!(pj > 1e-30f) && lane >= lo && lane < hi);
    float acc[64], mine_tiny = 0.0f;
#pragma unroll
    for (int j = 0; j < 64; ++j) acc[j] = 0.0f;
    for (int32_t i0 = wave * 64; i0 < n_sym; i0 += n_waves * 64) {
        const int32_t i = i0 + lane;
        uint64_t mm[K];                     // 0: absent, gated by the clamp, or past the last symbol
        float cf[K], gate_g = 0.0f;
#pragma unroll
        for (int x = 0; x < K; ++x) { mm[x] = 0; cf[x] = 0.0f; }
        if (i < n_sym) {
            const uint64_t *m = mask + (s * n_sym + i) * K;
            const float *pp = pprob + (s * n_sym + i) * K;
            uint64_t lm[K];
            float pv[K];
            load_masks<K>(m, lm);
            load_probs<K>(pp, pv);
            const float gi = g[s * ldg + i];
            float sum = 0.0f;               // the quantity the forward pass clamped: kept proofs in rank order
#pragma unroll
            for (int x = 0; x < K; ++x)
                if (lm[x] != kAbsent) sum = sum + pv[x];
            if (sum <= 1.0f) {
                gate_g = gi;
#pragma unroll
                for (int x = 0; x < K; ++x)
                    if (lm[x] != kAbsent) { mm[x] = lm[x]; cf[x] = gi * pv[x]; }
            }
        }
#pragma unroll
        for (int j0 = 0; j0 < 64; j0 += 8) {
            if (j0 < lo || j0 >= hi) continue;      // (uniform; facts past n_facts are in no proof)
#pragma unroll
            for (int j = j0; j < j0 + 8; ++j) {
#pragma unroll
                for (int x = 0; x < K; ++x) {
                    const int word = static_cast<int>(static_cast<uint32_t>(j < 32 ? mm[x] : mm[x] >> 32));
                    const int held = __builtin_amdgcn_sbfe(word, j & 31, 1);                    // all ones: the proof holds fact j
                    acc[j] = acc[j] + __builtin_bit_cast(float, held & __builtin_bit_cast(int, cf[x]));
                }
            }
        }
        for (uint64_t tm = tiny; tm; tm &= tm - 1) {                     // (uniform) facts that cannot be divided by
            const int j = __builtin_ctzll(tm);
            float t = 0.0f;
#pragma unroll
            for (int x = 0; x < K; ++x) {
                if (!((mm[x] >> j) & 1)) continue;
                float others = 1.0f;
                for (uint64_t r = mm[x] & ~(uint64_t(1) << j); r; r &= r - 1) others = others * fp[__builtin_ctzll(r)];
                t = __builtin_fmaf(gate_g, others, t);
            }
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) t += __shfl_xor(t, d, 64);
            if (lane == j) mine_tiny = mine_tiny + t;
        }
    }
    // The wavefront's totals, eight facts at a time: at each distance a lane gives away the half of its sums that the other one
    // keeps, and every sum meets the others in the order of an exchange of all of them, 20 instructions for eight facts instead of
    // 96, half of those through LDS (8 334 symbols, 49 facts, us: 64 samples k = 3 13.7, 12.5 so, k = 1 10.6 and 7.9; 300 samples
    // 65 and 56; 899 symbols, 38 facts, k = 5, 64 samples 8.2 and 5.7).
    const int kept = 4 * (lane >> 3 & 1) + 2 * (lane >> 4 & 1) + (lane >> 5);      // which of the eight this lane ends with
#pragma unroll
    for (int j0 = 0; j0 < 64; j0 += 8) {
        if (j0 < lo || j0 >= hi) continue;
        float u[4], t[2];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const uint32_t a = __float_as_uint(acc[j0 + 2 * x]), b = __float_as_uint(acc[j0 + 2 * x + 1]);
            const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
            u[x] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(u[2 * x]), __float_as_uint(u[2 * x + 1]), false, false);
            t[x] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
        const float mine = lane & 8 ? t[1] : t[0], other = lane & 8 ? t[0] : t[1];
        float v = mine + dpp<0x128>(other);                                 // row_ror:8
        v += __shfl_xor(v, 4, 64);
        v += dpp<0x4E>(v);
        v += dpp<0xB1>(v);
        if ((lane & 7) == 0) part[wave][j0 + kept] = v;
    }
    wave_lds_fence();
    const bool is_tiny = (tiny >> lane) & 1;
    if (is_tiny) part[wave][lane] = mine_tiny;
    __syncthreads();
    if (wave == 0 && lane >= lo && lane < hi) {
        const float per = is_tiny ? 1.0f : __builtin_amdgcn_rcpf(pj);
        float tot = 0.0f;
        for (int w = 0; w < n_waves; ++w) tot = tot + part[w][lane] * per;
        gfact[s * n_facts + lane] = tot;
    }
}

dol_status launch_dtkp_prob_bwd(int32_t batch, int32_t n_sym, int32_t k, int32_t n_facts, const uint64_t *mask,
                                const float *pprob, const float *fact_prob, const float *g, int64_t ldg, float *gfact,
                                hipStream_t st)
{
    if (batch == 0 || n_facts == 0) return DOL_OK;
    const int waves = std::max(1, std::min(kGradWaves, (n_sym + 63) / 64));
    // one workgroup per unit at most, and eight facts per workgroup at least
    const int parts = std::max(1, std::min((n_facts + 7) / 8, 256 / batch));
#define CALL(K)                                                                                                        \
    hipLaunchKernelGGL(dtkp_prob_bwd_kernel<K>, dim3(static_cast<unsigned>(batch) * parts), dim3(64 * waves), 0, st, parts, n_sym, \
                       n_facts, mask, pprob, fact_prob, g, ldg, gfact)
    DOL_DISPATCH_K(k, CALL)
#undef CALL
    DOL_HIP(hipGetLastError());
    return DOL_OK;
}

}  // namespace dol
