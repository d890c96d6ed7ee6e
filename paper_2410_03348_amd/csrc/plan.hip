// Symbol side of the operators (Sec. 3.1.2): everything that depends only on the symbols and the
// user function, computed once on the host for the whole batch and uploaded as index arrays.
#include "internal.h"
#include "plan_cache.h"

#include <algorithm>
#include <atomic>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <set>
#include <unordered_map>

namespace dol {

// ---------------------------------------------------------------- errors

static thread_local std::string g_last_error;

void set_error(const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
}

dol_status fail(dol_status st, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return st;
}

dol_status hip_fail(hipError_t e, const char *what)
{
    set_error("%s: %s", what, hipGetErrorString(e));
    return e == hipErrorOutOfMemory ? DOL_ENOMEM : DOL_EHIP;
}

hipError_t allow_dynamic_lds(const void *kernel, size_t bytes)
{
    static std::mutex mu;
    static std::set<std::pair<int, const void *>> *seen = new std::set<std::pair<int, const void *>>;   // never destroyed
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    if (seen->count({dev, kernel})) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes));
    if (e == hipSuccess) seen->insert({dev, kernel});
    return e;
}

// ---------------------------------------------------------------- function tables

struct Tuple {
    int32_t i, j, id;
};

// struct ListPlan from lists ptr[x] .. ptr[x + 1] of word(q).  by_workgroup(lengths): how many of the lists of more than kMidList
// words, whose lengths these are, the longest first, a workgroup sums.
template <typename F, typename G>
static hipError_t upload_lists(const std::vector<uint32_t> &ptr, int32_t n, F word, uint32_t filling, G by_workgroup, ListPlan *plan)
{
    std::vector<uint32_t> order = columns_by_length(ptr, n, kLaneList), start{0}, words, huge, wave, mid;
    auto length = [&](uint32_t x) { const uint32_t l = ptr[x + 1] - ptr[x]; return l > static_cast<uint32_t>(kLaneList) ? 0u : l; };
    for (int32_t r0 = 0; r0 < n; r0 += 64) {
        uint32_t most = 0;
        for (int32_t r = r0; r < std::min(n, r0 + 64); ++r) most = std::max(most, length(order[r]));
        const size_t at = words.size();
        words.resize(at + static_cast<size_t>(most) * 64, filling);
        for (int32_t r = r0; r < std::min(n, r0 + 64); ++r)
            for (uint32_t k = 0; k < length(order[r]); ++k) words[at + static_cast<size_t>(k) * 64 + (r - r0)] = word(ptr[order[r]] + k);
        start.push_back(start.back() + most);
        plan->lane_words = std::max(plan->lane_words, static_cast<int32_t>(most));
    }
    plan->n_words = words.size();
    words.resize(words.size() + 8 * 64, filling);           // up to eight words are read at a time
    for (uint32_t &x : order)
        if (ptr[x + 1] - ptr[x] > static_cast<uint32_t>(kLaneList)) x |= kListElsewhere;
    while (order.size() % 64) order.push_back(kNoList);
    auto words_of = [&](uint32_t x) { return static_cast<int64_t>(ptr[x + 1]) - ptr[x]; };
    std::vector<uint32_t> longest;          // the lists too long for 16 lanes
    for (int32_t x = 0; x < n; ++x) {
        if (words_of(x) > kMidList) longest.push_back(static_cast<uint32_t>(x));
        else if (words_of(x) > kLaneList) mid.push_back(static_cast<uint32_t>(x)), plan->mid_words += words_of(x);
    }
    std::stable_sort(longest.begin(), longest.end(), [&](uint32_t x, uint32_t y) { return words_of(x) > words_of(y); });
    std::vector<int64_t> lengths;
    for (uint32_t x : longest) lengths.push_back(words_of(x));
    const size_t whole = by_workgroup(lengths);
    for (size_t r = 0; r < longest.size(); ++r) {
        (r < whole ? plan->huge_words : plan->mid_words) += lengths[r];
        (r < whole ? huge : wave).push_back(longest[r]);
    }
    plan->n_huge = static_cast<int32_t>(huge.size()), plan->n_wave = static_cast<int32_t>(wave.size()), plan->n_mid = static_cast<int32_t>(mid.size());
    if (huge.size() == 1) plan->only_huge = static_cast<int32_t>(huge[0]);
    huge.insert(huge.end(), wave.begin(), wave.end());
    huge.insert(huge.end(), mid.begin(), mid.end());
    hipError_t e;
    if ((e = plan->order.upload(order)) != hipSuccess || (e = plan->ptr.upload(start)) != hipSuccess ||
        (e = plan->longer.upload(huge)) != hipSuccess) return e;
    return plan->words.upload(words);
}

// (two symbols to a word.  A wavefront takes 0.6 us for 256 symbols, a workgroup for 4 096 and another 0.8 for its barriers, but one
// list after the other, where sixteen wavefronts sum side by side: 24 000 symbols in 16 columns of 1 500, 64 samples, 25.6 us with a
// workgroup to each and 12.0 so; one column of 2 043 5.7 with a wavefront and 4.1 so)
static size_t pairs_by_workgroup(const std::vector<int64_t> &words)
{
    auto turns = [](int64_t l, int64_t at_once) { return 0.6 * static_cast<double>((2 * l + at_once - 1) / at_once); };
    double rest = 0.0, whole = 0.0, best_us = 0.0;
    for (int64_t l : words) rest += turns(l, 256);
    size_t best = 0;
    for (size_t m = 0; m <= words.size(); ++m) {
        const double us = whole + (m < words.size() ? std::max(turns(words[m], 256), rest / 16) : 0.0);
        if (m == 0 || us < best_us) best = m, best_us = us;
        if (m < words.size()) whole += 0.8 + turns(words[m], 4096), rest -= turns(words[m], 256);
    }
    return best;
}

hipError_t upload_pair_lists(const std::vector<uint32_t> &ptr, int32_t n, const std::vector<uint32_t> &pairs, uint32_t filling, ListPlan *plan)
{
    return upload_lists(ptr, n, [&](uint32_t q) { return pairs[q]; }, filling, pairs_by_workgroup, plan);
}

static size_t columns_by_workgroup(const std::vector<int64_t> &words)
{
    int64_t above = 0;
    for (int64_t l : words) above += l;
    return static_cast<size_t>(std::count_if(words.begin(), words.end(), [&](int64_t l) { return 16 * l > above; }));
}

static dol_status build_table(int32_t na, int32_t nb, std::vector<Tuple> &tup, dol_fn_table **out)
{
    // ascending (i, j); a function has one value per argument tuple
    std::sort(tup.begin(), tup.end(), [](const Tuple &x, const Tuple &y) { return x.i != y.i ? x.i < y.i : x.j < y.j; });
    for (size_t t = 1; t < tup.size(); ++t)
        if (tup[t].i == tup[t - 1].i && tup[t].j == tup[t - 1].j)
            return fail(DOL_EINVAL, "function table lists the tuple (%d, %d) twice", tup[t].i, tup[t].j);

    std::unique_ptr<dol_fn_table> tb(new (std::nothrow) dol_fn_table);
    if (!tb) return fail(DOL_ENOMEM, "out of host memory");
    static std::atomic<uint64_t> tables_made{0};
    tb->uid = ++tables_made;
    tb->na = na;
    tb->nb = nb;
    tb->n_tuples = static_cast<int64_t>(tup.size());

    // Eq. 2: the output symbols are the distinct produced ids, ascending
    tb->out_syms.reserve(tup.size());
    for (const Tuple &t : tup) tb->out_syms.push_back(t.id);
    std::sort(tb->out_syms.begin(), tb->out_syms.end());
    tb->out_syms.erase(std::unique(tb->out_syms.begin(), tb->out_syms.end()), tb->out_syms.end());
    if (tb->out_syms.size() > DOL_MAX_SYMBOLS)
        return fail(DOL_EUNSUPPORTED, "function table produces %zu symbols, more than %d", tb->out_syms.size(),
                    DOL_MAX_SYMBOLS);
    const int32_t S = tb->n_out = static_cast<int32_t>(tb->out_syms.size());

    std::vector<uint32_t> col(tup.size());
    for (size_t t = 0; t < tup.size(); ++t)
        col[t] = static_cast<uint32_t>(std::lower_bound(tb->out_syms.begin(), tb->out_syms.end(), tup[t].id) -
                                       tb->out_syms.begin());

    // counting sorts (stable, so each group keeps ascending (i, j))
    std::vector<uint32_t> col_ptr(S + 1, 0), rowa_ptr(na + 1, 0), rowb_ptr(nb + 1, 0);
    for (size_t t = 0; t < tup.size(); ++t) {
        col_ptr[col[t] + 1]++;
        rowa_ptr[tup[t].i + 1]++;
        rowb_ptr[tup[t].j + 1]++;
    }
    for (int32_t c = 0; c < S; ++c) {
        tb->max_col_len = std::max<int32_t>(tb->max_col_len, static_cast<int32_t>(col_ptr[c + 1]));
        col_ptr[c + 1] += col_ptr[c];
    }
    for (int32_t i = 0; i < na; ++i) rowa_ptr[i + 1] += rowa_ptr[i];
    for (int32_t j = 0; j < nb; ++j) rowb_ptr[j + 1] += rowb_ptr[j];
    std::vector<uint32_t> col_ij(tup.size()), rowa_jc(tup.size()), rowb_ic(tup.size());
    std::vector<uint32_t> rowb_pos(S == na ? tup.size() : 0);
    {
        std::vector<uint32_t> fc(col_ptr.begin(), col_ptr.end() - 1), fa(rowa_ptr.begin(), rowa_ptr.end() - 1),
            fb(rowb_ptr.begin(), rowb_ptr.end() - 1);
        for (size_t t = 0; t < tup.size(); ++t) {
            const uint32_t i = static_cast<uint32_t>(tup[t].i), j = static_cast<uint32_t>(tup[t].j);
            col_ij[fc[col[t]]++] = pack16(i, j);
            const uint32_t qa = fa[i]++, qb = fb[j]++;
            rowa_jc[qa] = pack16(j, col[t]);
            rowb_ic[qb] = pack16(i, col[t]);
            if (!rowb_pos.empty()) rowb_pos[qb] = qa;
        }
    }
    // sum-like: inside every column i rises by one and j falls by one (f(i,j) depends on i+j only and is injective in it)
    tb->sum_like = !tup.empty();
    for (int32_t c = 0; c < S && tb->sum_like; ++c)
        for (uint32_t q = col_ptr[c] + 1; q < col_ptr[c + 1]; ++q) {
            const uint32_t p0 = col_ij[q - 1], p1 = col_ij[q];
            if ((p1 & 0xffff) != (p0 & 0xffff) + 1 || (p1 >> 16) + 1 != (p0 >> 16)) { tb->sum_like = false; break; }
        }

    tb->conv_like = na > 0 && nb > 0 && tup.size() == static_cast<size_t>(na) * static_cast<size_t>(nb) && S == na + nb - 1;
    for (size_t t = 0; t < tup.size() && tb->conv_like; ++t)
        tb->conv_like = col[t] == static_cast<uint32_t>(tup[t].i + tup[t].j);

    std::vector<uint32_t> long_rows;
    for (int32_t i = 0; i < na; ++i) {
        if (rowa_ptr[i + 1] - rowa_ptr[i] > static_cast<uint32_t>(kLongTableRow)) { long_rows.push_back(static_cast<uint32_t>(i)); ++tb->n_long_rowa; }
        tb->max_rowa_len = std::max(tb->max_rowa_len, static_cast<int32_t>(rowa_ptr[i + 1] - rowa_ptr[i]));
    }
    for (int32_t j = 0; j < nb; ++j)
        if (rowb_ptr[j + 1] - rowb_ptr[j] > static_cast<uint32_t>(kLongTableRow)) long_rows.push_back(static_cast<uint32_t>(na + j));

    // long columns, the huge ones first
    std::vector<uint32_t> long_cols, less_long;
    for (int32_t c = 0; c < S; ++c) {
        const uint32_t len = col_ptr[c + 1] - col_ptr[c];
        if (len > static_cast<uint32_t>(kHugeTableCol)) long_cols.push_back(static_cast<uint32_t>(c));
        else if (len > static_cast<uint32_t>(kLongTableCol)) less_long.push_back(static_cast<uint32_t>(c));
    }
    tb->n_huge_cols = static_cast<int32_t>(long_cols.size());
    long_cols.insert(long_cols.end(), less_long.begin(), less_long.end());

    if (hipGetDevice(&tb->device) != hipSuccess) tb->device = 0;
    hipError_t e;
    if ((e = tb->long_rows.upload(long_rows)) != hipSuccess) return hip_fail(e, "uploading the function table");
    const std::vector<uint32_t> col_order = columns_by_length(col_ptr, S, kLongDtkpCol);
    std::vector<uint32_t> lengths;
    if ((e = tb->long_cols.upload(long_cols)) != hipSuccess || (e = tb->dtkp_cols.build(col_ptr, col_order, &lengths)) != hipSuccess)
        return hip_fail(e, "uploading the function table");
    std::vector<uint32_t> col_head(static_cast<size_t>(S) * 4, 0xFFFFFFFFu);
    for (int32_t c = 0; c < S; ++c)
        for (uint32_t q = col_ptr[c], u = 0; q < col_ptr[c + 1] && u < 4; ++q, ++u) col_head[static_cast<size_t>(c) * 4 + u] = col_ij[q];
    if ((e = tb->col_head.upload(col_head)) != hipSuccess) return hip_fail(e, "uploading the function table");
    {
        // (a row even where every column is a longer one: first words are asked for before lengths are known)
        const uint32_t longest = S ? std::max(1u, *std::max_element(lengths.begin(), lengths.end())) : 0;
        std::vector<uint32_t> tuples(static_cast<size_t>(longest) * S, 0);
        for (int32_t r = 0; r < S; ++r)
            for (uint32_t k = 0; k < lengths[r]; ++k) tuples[static_cast<size_t>(k) * S + r] = col_ij[col_ptr[col_order[r]] + k];
        if ((e = tb->dtkp_tuples.upload(tuples)) != hipSuccess) return hip_fail(e, "uploading the function table");
    }
    if ((e = tb->col_ptr.upload(col_ptr)) != hipSuccess || (e = tb->col_ij.upload(col_ij)) != hipSuccess ||
        (e = tb->rowa_ptr.upload(rowa_ptr)) != hipSuccess || (e = tb->rowa_jc.upload(rowa_jc)) != hipSuccess ||
        (e = tb->rowb_ptr.upload(rowb_ptr)) != hipSuccess || (e = tb->rowb_ic.upload(rowb_ic)) != hipSuccess ||
        (e = tb->rowb_pos.upload(rowb_pos)) != hipSuccess)
        return hip_fail(e, "uploading the function table");
    if (dol_status s2 = grid_plan_build(tb.get(), col_ptr, col_ij, rowb_ptr, rowb_ic)) return s2;
    if (!conv_path_ok(tb.get()))
        if (dol_status s2 = lds_plan_build(tb.get(), col_ptr, col_ij, rowa_ptr, rowa_jc, rowb_ptr, rowb_ic)) return s2;
    if (!conv_path_ok(tb.get()) && na >= 1 && nb >= 1 && S >= 1 && na + nb < 0xFFFF && S < 0xFFFF) {
        if ((e = upload_lists(col_ptr, S, [&](uint32_t q) { return col_ij[q]; }, pack16(na, nb), columns_by_workgroup, &tb->col_lists)) != hipSuccess)
            return hip_fail(e, "uploading the function table");
        std::vector<uint32_t> row_ptr(rowa_ptr);
        for (int32_t j = 0; j < nb; ++j) row_ptr.push_back(rowa_ptr[na] + rowb_ptr[j + 1]);
        const uint32_t n_a = rowa_ptr[na];
        auto word = [&](uint32_t q) {
            if (q < n_a) return pack16(na + (rowa_jc[q] & 0xffffu), rowa_jc[q] >> 16);
            return rowb_ic[q - n_a];
        };
        if ((e = upload_lists(row_ptr, na + nb, word, pack16(na + nb, S), [](const std::vector<int64_t> &words) { return words.size(); }, &tb->row_lists)) != hipSuccess)
            return hip_fail(e, "uploading the function table");
        tb->lists_ok = true;
    }
    if (!conv_path_ok(tb.get()) && nb >= 1 && nb <= kByJMax && na >= 1 && na <= kByJMaxNa && S >= 1 && S <= kByJMaxNa &&
        tb->lists_ok) {
        const int32_t nbp = nb <= 4 ? 4 : nb <= 8 ? 8 : nb <= 10 ? 10 : 16;
        const int32_t src_ld = (S + kByJBlock - 1) / kByJBlock * kByJBlock, col_ld = (na + kByJBlock - 1) / kByJBlock * kByJBlock;
        tb->byj_nbp = nbp, tb->byj_src_ld = src_ld, tb->byj_col_ld = col_ld;
        const uint16_t no_i = static_cast<uint16_t>(na), no_c = static_cast<uint16_t>(S);
        std::vector<uint16_t> src(static_cast<size_t>(nbp) * src_ld, no_i), colof(static_cast<size_t>(nbp) * col_ld, no_c);
        bool falling = true;
        for (int32_t c = 0; c < S; ++c) {
            const bool is_long = col_ptr[c + 1] - col_ptr[c] > static_cast<uint32_t>(kLaneList);
            bool regular = !is_long;
            for (uint32_t q = col_ptr[c] + 1; q < col_ptr[c + 1] && !is_long; ++q) falling &= col_ij[q] >> 16 < col_ij[q - 1] >> 16;
            for (uint32_t q = col_ptr[c]; q < col_ptr[c + 1] && regular; ++q) {
                uint16_t &slot = src[static_cast<size_t>(col_ij[q] >> 16) * src_ld + byj_place(c)];
                if (slot != no_i) regular = false;
                slot = static_cast<uint16_t>(col_ij[q] & 0xffffu);
            }
            if (!regular) {
                for (int32_t j = 0; j < nb; ++j) src[static_cast<size_t>(j) * src_ld + byj_place(c)] = no_i;
                src[byj_place(c)] = is_long ? kByJWave : kByJList;
            }
        }
        for (size_t t = 0; t < tup.size(); ++t) colof[static_cast<size_t>(tup[t].j) * col_ld + byj_place(tup[t].i)] = static_cast<uint16_t>(col[t]);
        if ((e = tb->byj_src.upload(src)) != hipSuccess || (e = tb->byj_col.upload(colof)) != hipSuccess)
            return hip_fail(e, "uploading the function table");
        tb->byj_ok = true;
        tb->byj_falling = falling;
        tb->byj_fwd = 2 * tup.size() >= static_cast<size_t>(nb) * static_cast<size_t>(S);
    }
    tb->h_col_ptr.swap(col_ptr);
    tb->h_col_ij.swap(col_ij);
    tb->kernel_fwd = damp_kernel_name(tb.get(), false);
    tb->kernel_bwd = damp_kernel_name(tb.get(), true);
    *out = tb.release();
    return DOL_OK;
}

static dol_status check_table_dims(int32_t na, int32_t nb, dol_fn_table **table)
{
    if (!table) return fail(DOL_EINVAL, "table output pointer is NULL");
    *table = nullptr;
    if (na < 0 || nb < 0 || na > DOL_MAX_SYMBOLS || nb > DOL_MAX_SYMBOLS)
        return fail(DOL_ESHAPE, "operand sizes %d x %d outside 0..%d", na, nb, DOL_MAX_SYMBOLS);
    return DOL_OK;
}

// ---------------------------------------------------------------- content-addressed plan caches

// (on the heap and never destroyed: no hipFree during static destruction, when the HIP runtime may already be down)
static Cache<FilterPlan> &g_filter_cache = *new Cache<FilterPlan>;
static Cache<UnionPlan> &g_union_cache = *new Cache<UnionPlan>;

dol_status get_filter_plan(int32_t n, const uint8_t *pred, const FilterPlan **plan)
{
    int device = 0;
    (void)hipGetDevice(&device);
    std::vector<uint8_t> norm(static_cast<size_t>(n));
    for (int32_t i = 0; i < n; ++i) norm[i] = pred[i] ? 1 : 0;
    std::vector<unsigned char> key = make_key(device, {{norm.data(), norm.size()}});
    const uint64_t h = hash_bytes(key.data(), key.size());
    std::lock_guard<std::mutex> lock(g_filter_cache.mu);
    if ((*plan = g_filter_cache.find(h, key)) != nullptr) return DOL_OK;

    std::unique_ptr<FilterPlan> p(new (std::nothrow) FilterPlan);
    if (!p) return fail(DOL_ENOMEM, "out of host memory");
    p->n_in = n;
    std::vector<int32_t> pos(static_cast<size_t>(n), -1);
    for (int32_t i = 0; i < n; ++i)
        if (norm[i]) {
            pos[i] = static_cast<int32_t>(p->keep_idx.size());
            p->keep_idx.push_back(i);
        }
    p->n_out = static_cast<int32_t>(p->keep_idx.size());
    hipError_t e;
    if ((e = p->d_keep_idx.upload(p->keep_idx)) != hipSuccess || (e = p->d_pos.upload(pos)) != hipSuccess)
        return hip_fail(e, "uploading the filter plan");
    *plan = g_filter_cache.insert(h, std::move(key), std::move(p));
    return DOL_OK;
}

dol_status get_union_plan(int32_t na, const int32_t *sa, int32_t nb, const int32_t *sb, const UnionPlan **plan)
{
    int device = 0;
    (void)hipGetDevice(&device);
    std::vector<unsigned char> key =
        make_key(device, {{sa, sizeof(int32_t) * static_cast<size_t>(na)}, {sb, sizeof(int32_t) * static_cast<size_t>(nb)}});
    const uint64_t h = hash_bytes(key.data(), key.size());
    std::lock_guard<std::mutex> lock(g_union_cache.mu);
    if ((*plan = g_union_cache.find(h, key)) != nullptr) return DOL_OK;

    std::unique_ptr<UnionPlan> p(new (std::nothrow) UnionPlan);
    if (!p) return fail(DOL_ENOMEM, "out of host memory");
    p->na = na;
    p->nb = nb;
    std::vector<int32_t> ia, ib, ca(static_cast<size_t>(na)), cb(static_cast<size_t>(nb));
    int32_t i = 0, j = 0;
    while (i < na || j < nb) {            // ascending merge of two ascending id lists
        const int32_t c = static_cast<int32_t>(ia.size());
        if (j >= nb || (i < na && sa[i] < sb[j])) {
            p->out_syms.push_back(sa[i]); ia.push_back(i); ib.push_back(-1); ca[i++] = c;
        } else if (i >= na || sb[j] < sa[i]) {
            p->out_syms.push_back(sb[j]); ia.push_back(-1); ib.push_back(j); cb[j++] = c;
        } else {
            p->out_syms.push_back(sa[i]); ia.push_back(i); ib.push_back(j); ca[i++] = c; cb[j++] = c;
        }
    }
    p->n_out = static_cast<int32_t>(ia.size());
    hipError_t e;
    if ((e = p->d_ia.upload(ia)) != hipSuccess || (e = p->d_ib.upload(ib)) != hipSuccess ||
        (e = p->d_ca.upload(ca)) != hipSuccess || (e = p->d_cb.upload(cb)) != hipSuccess)
        return hip_fail(e, "uploading the union plan");
    *plan = g_union_cache.insert(h, std::move(key), std::move(p));
    return DOL_OK;
}

static Cache<UnionPlan> &g_filter_union_cache = *new Cache<UnionPlan>;

// union(filter(d, pred), c) as ONE merge plan over the unfiltered operand: ia[u] is a position in d (of a kept
// symbol) or -1, ca[x] is the output column of d's symbol x or -1 when the predicate drops it.
dol_status get_filter_union_plan(int32_t n, const int32_t *sd, const uint8_t *pred, int32_t nc, const int32_t *sc,
                                 const UnionPlan **plan)
{
    int device = 0;
    (void)hipGetDevice(&device);
    std::vector<uint8_t> norm(static_cast<size_t>(n));
    for (int32_t i = 0; i < n; ++i) norm[i] = pred[i] ? 1 : 0;
    std::vector<unsigned char> key = make_key(device, {{norm.data(), norm.size()},
                                                       {sd, sizeof(int32_t) * static_cast<size_t>(n)},
                                                       {sc, sizeof(int32_t) * static_cast<size_t>(nc)}});
    const uint64_t h = hash_bytes(key.data(), key.size());
    std::lock_guard<std::mutex> lock(g_filter_union_cache.mu);
    if ((*plan = g_filter_union_cache.find(h, key)) != nullptr) return DOL_OK;

    std::unique_ptr<UnionPlan> p(new (std::nothrow) UnionPlan);
    if (!p) return fail(DOL_ENOMEM, "out of host memory");
    p->na = n;
    p->nb = nc;
    std::vector<int32_t> ia, ib, ca(static_cast<size_t>(n), -1), cb(static_cast<size_t>(nc));
    int32_t i = 0, j = 0;
    while (true) {                          // ascending merge of the kept ids of d with the ids of c
        while (i < n && !norm[i]) ++i;
        if (i >= n && j >= nc) break;
        const int32_t col = static_cast<int32_t>(ia.size());
        if (j >= nc || (i < n && sd[i] < sc[j])) {
            p->out_syms.push_back(sd[i]); ia.push_back(i); ib.push_back(-1); ca[i++] = col;
        } else if (i >= n || sc[j] < sd[i]) {
            p->out_syms.push_back(sc[j]); ia.push_back(-1); ib.push_back(j); cb[j++] = col;
        } else {
            p->out_syms.push_back(sd[i]); ia.push_back(i); ib.push_back(j); ca[i++] = col; cb[j++] = col;
        }
    }
    p->n_out = static_cast<int32_t>(ia.size());
    p->aligned = p->n_out == nc && n <= nc;
    for (int32_t c = 0; c < p->n_out && p->aligned; ++c) p->aligned = ib[c] == c && (ia[c] == c || ia[c] < 0);
    hipError_t e;
    if ((e = p->d_ia.upload(ia)) != hipSuccess || (e = p->d_ib.upload(ib)) != hipSuccess ||
        (e = p->d_ca.upload(ca)) != hipSuccess || (e = p->d_cb.upload(cb)) != hipSuccess)
        return hip_fail(e, "uploading the filter-union plan");
    *plan = g_filter_union_cache.insert(h, std::move(key), std::move(p));
    return DOL_OK;
}

struct I32Array {
    DevArray<int32_t> d;
};
static Cache<I32Array> &g_i32_cache = *new Cache<I32Array>;

// Device copy of a small host int32 array, cached by content.
dol_status get_i32_array(int32_t n, const int32_t *data, const int32_t **dptr)
{
    int device = 0;
    (void)hipGetDevice(&device);
    std::vector<unsigned char> key = make_key(device, {{data, sizeof(int32_t) * static_cast<size_t>(n)}});
    const uint64_t h = hash_bytes(key.data(), key.size());
    std::lock_guard<std::mutex> lock(g_i32_cache.mu);
    const I32Array *hit = g_i32_cache.find(h, key);
    if (!hit) {
        std::unique_ptr<I32Array> p(new (std::nothrow) I32Array);
        if (!p) return fail(DOL_ENOMEM, "out of host memory");
        hipError_t e = p->d.upload(std::vector<int32_t>(data, data + n));
        if (e != hipSuccess) return hip_fail(e, "uploading an index array");
        hit = g_i32_cache.insert(h, std::move(key), std::move(p));
    }
    *dptr = hit->d.ptr;
    return DOL_OK;
}

dol_status make_group_masks(const dol_prov *prov, GroupMasks *gm)
{
    gm->n = 0;
    if (!prov->fact_group) return DOL_OK;
    std::unordered_map<int32_t, uint64_t> by_group;
    for (int32_t f = 0; f < prov->n_facts; ++f) {
        if (prov->fact_group[f] < 0) return fail(DOL_EINVAL, "fact_group[%d] is negative", f);
        by_group[prov->fact_group[f]] |= uint64_t(1) << f;
    }
    std::vector<uint64_t> masks;
    for (const auto &kv : by_group)
        if (__builtin_popcountll(kv.second) >= 2) masks.push_back(kv.second);
    std::sort(masks.begin(), masks.end());
    if (masks.size() > 32) return fail(DOL_EUNSUPPORTED, "more than 32 exclusion groups with two or more facts");
    gm->n = static_cast<int32_t>(masks.size());
    for (size_t x = 0; x < masks.size(); ++x) gm->m[x] = masks[x];
    return DOL_OK;
}

}  // namespace dol

// ---------------------------------------------------------------- C ABI: tables and plans

extern "C" {

dol_status dol_fn_table_create_dense(int32_t na, int32_t nb, const int32_t *out_id, dol_fn_table **table)
{
    if (dol_status st = dol::check_table_dims(na, nb, table)) return st;
    if (!out_id && na > 0 && nb > 0) return dol::fail(DOL_EINVAL, "out_id is NULL");
    std::vector<dol::Tuple> tup;
    tup.reserve(static_cast<size_t>(na) * static_cast<size_t>(nb));
    for (int32_t i = 0; i < na; ++i)
        for (int32_t j = 0; j < nb; ++j) {
            const int32_t id = out_id[static_cast<size_t>(i) * nb + j];
            if (id < -1) return dol::fail(DOL_EINVAL, "out_id[%d,%d] = %d; ids are >= 0 or -1 for a rejected tuple", i, j, id);
            if (id >= 0) tup.push_back({i, j, id});
        }
    return dol::build_table(na, nb, tup, table);
}

dol_status dol_fn_table_create_if(int32_t na, int32_t nb, const int32_t *out_id, const uint8_t *cond,
                                  dol_fn_table **table)
{
    if (dol_status st = dol::check_table_dims(na, nb, table)) return st;
    if ((!out_id || !cond) && na > 0 && nb > 0) return dol::fail(DOL_EINVAL, "out_id or cond is NULL");
    std::vector<dol::Tuple> tup;
    for (int32_t i = 0; i < na; ++i)
        for (int32_t j = 0; j < nb; ++j) {
            const size_t e = static_cast<size_t>(i) * nb + j;
            if (!cond[e]) continue;
            if (out_id[e] < 0) return dol::fail(DOL_EINVAL, "out_id[%d,%d] = %d is negative where the condition holds", i, j, out_id[e]);
            tup.push_back({i, j, out_id[e]});
        }
    return dol::build_table(na, nb, tup, table);
}

dol_status dol_fn_table_create_sparse(int32_t na, int32_t nb, int64_t n, const int32_t *i, const int32_t *j,
                                      const int32_t *out_id, dol_fn_table **table)
{
    if (dol_status st = dol::check_table_dims(na, nb, table)) return st;
    if (n < 0) return dol::fail(DOL_EINVAL, "negative tuple count");
    if (n > 0 && (!i || !j || !out_id)) return dol::fail(DOL_EINVAL, "tuple arrays are NULL");
    std::vector<dol::Tuple> tup;
    tup.reserve(static_cast<size_t>(n));
    for (int64_t t = 0; t < n; ++t) {
        if (i[t] < 0 || i[t] >= na || j[t] < 0 || j[t] >= nb)
            return dol::fail(DOL_ESHAPE, "tuple %lld = (%d, %d) outside %d x %d", static_cast<long long>(t), i[t], j[t], na, nb);
        if (out_id[t] < 0) return dol::fail(DOL_EINVAL, "tuple %lld produces the negative id %d", static_cast<long long>(t), out_id[t]);
        tup.push_back({i[t], j[t], out_id[t]});
    }
    return dol::build_table(na, nb, tup, table);
}

int32_t dol_fn_table_n_out(const dol_fn_table *table) { return table ? table->n_out : 0; }

const int32_t *dol_fn_table_out_syms(const dol_fn_table *table) { return table ? table->out_syms.data() : nullptr; }

void dol_fn_table_destroy(dol_fn_table *table) { delete table; }

const char *dol_fn_table_kernel(const dol_fn_table *table, int32_t which)
{
    if (!table) return "";
    return which ? table->kernel_bwd.c_str() : table->kernel_fwd.c_str();
}

const char *dol_fn_table_kernel_at(const dol_fn_table *table, int32_t which, int64_t batch)
{
    static thread_local std::string name;
    if (!table) return "";
    name = dol::damp_kernel_name(table, which != 0, batch);
    return name.c_str();
}

dol_status dol_filter_plan(const dol_dist *d, const uint8_t *pred_mask, int32_t *n_out, int32_t *out_syms)
{
    if (!d || !n_out) return dol::fail(DOL_EINVAL, "NULL argument");
    if (d->n_sym < 0 || d->n_sym > DOL_MAX_SYMBOLS) return dol::fail(DOL_ESHAPE, "n_sym %d outside 0..%d", d->n_sym, DOL_MAX_SYMBOLS);
    if (d->n_sym > 0 && (!pred_mask || (out_syms && !d->sym_ids))) return dol::fail(DOL_EINVAL, "pred_mask or sym_ids is NULL");
    int32_t m = 0;
    for (int32_t i = 0; i < d->n_sym; ++i)
        if (pred_mask[i]) {
            if (out_syms) out_syms[m] = d->sym_ids[i];
            ++m;
        }
    *n_out = m;
    return DOL_OK;
}

dol_status dol_filter_union_plan(const dol_dist *d, const uint8_t *pred_mask, const dol_dist *c, int32_t *n_out,
                                 int32_t *out_syms)
{
    if (!d || !c || !n_out || !pred_mask) return dol::fail(DOL_EINVAL, "NULL argument");
    if (d->n_sym < 0 || c->n_sym < 0 || d->n_sym > DOL_MAX_SYMBOLS || c->n_sym > DOL_MAX_SYMBOLS)
        return dol::fail(DOL_ESHAPE, "n_sym outside 0..%d", DOL_MAX_SYMBOLS);
    if ((d->n_sym > 0 && !d->sym_ids) || (c->n_sym > 0 && !c->sym_ids)) return dol::fail(DOL_EINVAL, "sym_ids is NULL");
    for (int32_t i = 1; i < d->n_sym; ++i)
        if (d->sym_ids[i - 1] >= d->sym_ids[i]) return dol::fail(DOL_EINVAL, "d.sym_ids not strictly ascending at %d", i);
    for (int32_t j = 1; j < c->n_sym; ++j)
        if (c->sym_ids[j - 1] >= c->sym_ids[j]) return dol::fail(DOL_EINVAL, "c.sym_ids not strictly ascending at %d", j);
    int32_t i = 0, j = 0, m = 0;
    while (true) {
        while (i < d->n_sym && !pred_mask[i]) ++i;
        if (i >= d->n_sym && j >= c->n_sym) break;
        int32_t id;
        if (j >= c->n_sym || (i < d->n_sym && d->sym_ids[i] < c->sym_ids[j])) id = d->sym_ids[i++];
        else if (i >= d->n_sym || c->sym_ids[j] < d->sym_ids[i]) id = c->sym_ids[j++];
        else { id = d->sym_ids[i++]; ++j; }
        if (out_syms) out_syms[m] = id;
        ++m;
    }
    *n_out = m;
    return DOL_OK;
}

dol_status dol_union_plan(const dol_dist *a, const dol_dist *b, int32_t *n_out, int32_t *out_syms)
{
    if (!a || !b || !n_out) return dol::fail(DOL_EINVAL, "NULL argument");
    if (a->n_sym < 0 || b->n_sym < 0 || a->n_sym > DOL_MAX_SYMBOLS || b->n_sym > DOL_MAX_SYMBOLS)
        return dol::fail(DOL_ESHAPE, "n_sym outside 0..%d", DOL_MAX_SYMBOLS);
    if ((a->n_sym > 0 && !a->sym_ids) || (b->n_sym > 0 && !b->sym_ids)) return dol::fail(DOL_EINVAL, "sym_ids is NULL");
    for (int32_t i = 1; i < a->n_sym; ++i)
        if (a->sym_ids[i - 1] >= a->sym_ids[i]) return dol::fail(DOL_EINVAL, "a.sym_ids not strictly ascending at %d", i);
    for (int32_t j = 1; j < b->n_sym; ++j)
        if (b->sym_ids[j - 1] >= b->sym_ids[j]) return dol::fail(DOL_EINVAL, "b.sym_ids not strictly ascending at %d", j);
    int32_t i = 0, j = 0, m = 0;
    while (i < a->n_sym || j < b->n_sym) {
        int32_t id;
        if (j >= b->n_sym || (i < a->n_sym && a->sym_ids[i] < b->sym_ids[j])) id = a->sym_ids[i++];
        else if (i >= a->n_sym || b->sym_ids[j] < a->sym_ids[i]) id = b->sym_ids[j++];
        else { id = a->sym_ids[i++]; ++j; }
        if (out_syms) out_syms[m] = id;
        ++m;
    }
    *n_out = m;
    return DOL_OK;
}

const char *dol_last_error(void) { return dol::g_last_error.c_str(); }

const char *dol_version(void) { return "0.1.0"; }

}  // extern "C"
