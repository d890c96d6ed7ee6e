// The fused left fold of convolution-shaped DAMP applies (the loop of Fig. 2, forward + loss gradient + reverse sweep
// in one launch) as code written for the chain's shape.
//
// The symbol side of a fold is known before any tag is touched (Sec. 3.1.2): the number of inputs and the symbol
// counts of every stage.  With those as compile-time constants the whole sweep unrolls: 16 lanes own a sample, a
// wavefront four, and in every stage a lane owns a CONTIGUOUS block of w columns (rows, in the reverse sweep), which
// stays in its registers from the stage that makes it to the reverse sweep.
//
// A stage's columns need the nb - 1 entries before the lane's block as well.  Where two stages have the same width these
// are registers of the lanes before and come by lane shifts inside the sample's 16 lanes (a shift fills with the zeros that
// lie outside the row); where the width changes the row passes through LDS.  The widths are chosen for that (plan_widths):
// Sum-15 takes 1 2 2 3 3 5 5 5 7 7 7 7 9 9 9 columns a lane.  What bounds it is the issue of vector instructions; a lane
// shift costs two multiply-adds (1.8 and 1.0 ns a SIMD with four wavefronts of a test of its own on it), an LDS word 2 clocks of what four SIMDs
// share.  With every stage's row in LDS a wavefront used 2 556 LDS cycles and 2 806 vector instructions and held 13 KB, so
// that three shared a SIMD: B=524 288 802 us, B=4 096 11.8.  Now 1 262 cycles, 2 305 instructions and 7 KB: 493 and 9.2.
//
// A stage's result is kept as x = pre where pre <= 1 and -1 where the clamp acted: |x| is the tag and the sign is the clamp's
// decision, read by the reverse sweep with the operand it needs anyway - no stage is ever summed twice.  The tag is taken once
// an entry: as a modifier of every multiply-add the absolute value asks for the long encoding (Sum-15 with sums at the clamp,
// B=262 144, us, target / explicit gradient: 586 / 650 so, 293 / 338 once an entry).
//
// Under a target the gradient of a late stage is zero but for the few columns from which the remaining digits can reach
// the target: counted from the target these are the same for every sample, so the reverse sweep of the late stages holds
// S[x] = gradient of column (target - x), 1, 10, 19 ... entries for Sum-15 instead of 136, 127, 118 ..., and fetches the
// operand's row from LDS at the place the target says.  Half way through it turns to the columns themselves.
//
// Arithmetic is that of dol_apply2 / dol_backward: out[c] = min(1, sum over ascending i of a[i] * b[c - i]), one
// fused multiply-add per tuple from 0; gradients gated by [pre <= 1].  The gradient of a short operand is a sum over
// the sample's 16 lanes per symbol: the lanes share the symbols out while they exchange (emit_scattered_sums), and every
// total ends in the lanes that store it.
#include "internal.h"

#include <cstdarg>
#include <map>
#include <mutex>

namespace dol {

namespace {

constexpr int kL = 16;                  // lanes per sample
constexpr int kSP = 64 / kL;            // samples per wavefront
constexpr int kNBR = 16;                // most symbols of a short input
// Registers of a lane for the running Distributions and a stage's operands; what is too much, from the first Distribution on,
// waits in LDS, each lane's words apart.  (Sum-15 keeps all 75 words, in 140 registers and 7 KB of LDS.  A build of 128 registers
// and four wavefronts to a SIMD for large grids, with up to 27 KB of LDS, was no faster: Sum-15 B=524 288 488 us, 493 so; 64 and
// six of 16 symbols, B=262 144, 220 / 221; Sum-20 635 / 426; the most lost 100 and six of ten with an explicit gradient, 237 / 246;
// and every shape was compiled once for either.)
constexpr int kLaneRegs = 220;
constexpr size_t kChainLdsMax = 16 * 1024;   // per wavefront: ten to a compute unit

struct Src {
    std::string s;
    void operator()(const char *fmt, ...) __attribute__((format(printf, 2, 3)))
    {
        char buf[2048];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        s += buf;
    }
};

int ceil_div(int a, int b) { return (a + b - 1) / b; }

// LDS cycles per word of a 64-lane access whose lanes are w words apart, the samples 16 more than a multiple of 32 apart:
// odd widths meet every bank once.
int bank_ways(int w) { return w & 1 ? 1 : w & 2 ? 2 : w & 4 ? 4 : 8; }

// What a lane's share of a stage costs, in multiply-adds (which issue every 2 to 3 clocks, a lane shift every 4; an LDS word
// takes 2 clocks of what four SIMDs share).
constexpr double kShiftCost = 2.0, kWordCost = 1.2, kTurnCost = 10.0;

double turn_cost(int from, int to, int nb) { return kTurnCost + kWordCost * (from * bank_ways(from) + (to + nb - 1) * bank_ways(to)); }

// Columns of each row per lane: the narrowest that hold the row, or up to two more where a change of width costs more than
// the idle columns.  rows[0 .. n): symbols; nb[t]: symbols of the short operand between rows t - 1 and t; use[t]: multiply-adds
// per column of row t.
std::vector<int> plan_widths(const std::vector<int> &rows, const std::vector<int> &nb, const std::vector<double> &use)
{
    const int n = static_cast<int>(rows.size());
    std::vector<std::vector<double>> cost(n, std::vector<double>(3, 0.0));
    std::vector<std::vector<int>> from(n, std::vector<int>(3, 0));
    auto width = [&](int t, int x) { return ceil_div(rows[t], kL) + x; };
    for (int t = 0; t < n; ++t) {
        for (int x = 0; x < 3; ++x) {
            double best = 0.0;
            for (int y = 0; t > 0 && y < 3; ++y) {
                const int a = width(t - 1, y), b = width(t, x);
                const double c = cost[t - 1][y] + (a == b ? kShiftCost * (nb[t] - 1) : turn_cost(a, b, nb[t]));
                if (a <= b && (best == 0.0 || c < best)) { best = c; from[t][x] = y; }
            }
            cost[t][x] = (t > 0 && best == 0.0 ? 1e30 : best) + use[t] * width(t, x);
        }
    }
    std::vector<int> w(n);
    int x = 0;
    for (int y = 1; y < 3; ++y)
        if (cost[n - 1][y] < cost[n - 1][x]) x = y;
    for (int t = n - 1; t >= 0; --t) { w[t] = width(t, x); x = from[t][x]; }
    return w;
}

struct Layout {
    int n = 0;
    int m[kFoldChainMax] = {}, nb[kFoldChainMax] = {};
    int w[kFoldChainMax] = {};          // columns of acc_t per lane
    int ts = 0;                         // under a target: stages after ts count their gradient from the target
    int ws[kFoldChainMax] = {};         // entries of S_t per lane, ts <= t < n - 1
    int hist[kFoldChainMax] = {};       // acc_t's place in LDS for the reverse sweep (each lane its own words), or -1: registers
    int zero = 0, row = 0;              // words of a sample: the row buffer from here, zeros before it
    int row_len = 0;
    int off_d = 0, pitch = 0;           // the short input rows
    int stride = 0;
};

Layout lay_out(const std::vector<int> &shape)
{
    Layout Y;
    const int n = Y.n = shape[0], n1 = n - 1;
    Y.m[0] = shape[1];
    int nb_max = 1;
    for (int t = 1; t < n; ++t) {
        Y.nb[t] = shape[1 + t];
        Y.m[t] = Y.m[t - 1] + Y.nb[t] - 1;
        nb_max = std::max(nb_max, Y.nb[t]);
    }
    // symbols that S_t holds
    std::vector<int> reach(n, 1);
    for (int t = n1; t > 0; --t) reach[t - 1] = reach[t] + Y.nb[t] - 1;
    Y.ts = n1 - 1;
    while (Y.ts > 0) {
        const int t = Y.ts, nb = Y.nb[t], s = ceil_div(reach[t], kL), s1 = ceil_div(reach[t - 1], kL), w = ceil_div(Y.m[t - 1], kL);
        if (nb * (s + s1) + kWordCost * (w + s + nb) + kTurnCost >= 2.0 * nb * w) break;
        --Y.ts;
    }
    {
        std::vector<int> rows(Y.m, Y.m + n), nb(Y.nb, Y.nb + n);
        std::vector<double> use(n);
        for (int t = 0; t < n; ++t)
            use[t] = (t > 0 ? Y.nb[t] : 0) + (t == n1 ? 0.0 : t >= Y.ts ? kWordCost : 2.0 * Y.nb[t + 1]);
        const std::vector<int> w = plan_widths(rows, nb, use);
        std::copy(w.begin(), w.end(), Y.w);
    }
    if (Y.ts < n1) {                        // S_{n1 - 1} .. S_{ts}, in this order
        std::vector<int> rows, nb;
        std::vector<double> use;
        for (int t = n1 - 1; t >= Y.ts; --t) {
            rows.push_back(reach[t]);
            nb.push_back(Y.nb[t + 1]);
            use.push_back((t == n1 - 1 ? 1.0 : Y.nb[t + 1]) + (t > Y.ts ? Y.nb[t] + kWordCost : kWordCost));
        }
        const std::vector<int> w = plan_widths(rows, nb, use);
        for (size_t x = 0; x < w.size(); ++x) Y.ws[n1 - 1 - x] = w[x];
    }
    // in front of the row buffer: what windows reach before a row's first entry
    int halo = nb_max - 1, extent = kL * Y.w[n1] + nb_max;
    for (int t = Y.ts; t < n1; ++t) {
        halo = std::max(halo, kL * Y.ws[t] + nb_max);
        extent = std::max(extent, kL * Y.ws[t] + nb_max);
    }
    halo = std::max(halo, kL * Y.w[std::max(0, Y.ts - 1)] + nb_max);
    Y.row = (halo + 3) & ~3;
    Y.row_len = (std::max(extent, Y.m[n1]) + kL - 1) & ~(kL - 1);
    Y.off_d = Y.row + Y.row_len;
    Y.pitch = (nb_max + 3) & ~3;
    int pos = Y.off_d + n * Y.pitch, regs = 2 * Y.w[n1] + 3 * nb_max - 1;
    for (int t = n1 - 1; t >= 0; --t) {
        regs += Y.w[t];
        Y.hist[t] = -1;
        if (regs <= kLaneRegs) continue;
        Y.hist[t] = pos;
        pos += kL * Y.w[t];
    }
    Y.stride = (pos + 15) / 32 * 32 + 16;
    if (Y.stride < pos) Y.stride += 32;
    return Y;
}

// Sums of the n values s0 .. s<n-1> over the 16 lanes of a sample, each total ending in some lanes' s0: the four exchange
// steps pair a lane with the lane whose number differs by 15, 7, 2 and 1 (together these reach all 16), and in every step
// the two lanes of a pair share the values out - the one with the step's bit clear goes on with the first half, the other
// with the second half, an odd value out with both.  The first two steps' halves are whole groups of four lanes, which an
// instruction can write apart: two additions for two values.  which_sum(n) is the index of the total a lane ends up with.
void emit_scattered_sums(Src &o, int n)
{
    static const int which[4] = {3, 2, 1, 0}, bit[4] = {8, 4, 2, 1};
    static const char *const shift[2] = {"row_mirror", "row_half_mirror"};
    static const int clear[2] = {0x3, 0x5}, set[2] = {0xc, 0xa};
    for (int st = 0; st < 4; ++st) {
        const int h = n / 2;
        if (st < 2 && h > 0) {
            o("    asm volatile(\"s_nop 1\\n\\t\"\n");      // (values written just now)
            for (int k = 0; k < h; ++k)
                o("      \"v_add_f32_dpp %%%d, %%%d, %%%d %s row_mask:0xf bank_mask:0x%x\\n\\tv_add_f32_dpp %%%d, %%%d, %%%d %s row_mask:0xf bank_mask:0x%x\\n\\t\"\n",
                  k, k, k, shift[st], clear[st], k, k + h, k + h, shift[st], set[st]);
            o("      \"s_nop 1\" : ");
            for (int k = 0; k < h; ++k) o("%s\"+v\"(s%d)", k ? ", " : "", k);
            o(" : ");
            for (int k = 0; k < h; ++k) o("%s\"v\"(s%d)", k ? ", " : "", k + h);
            o(");\n");
        } else {
            for (int k = 0; k < h; ++k)
                o("    { const bool up = l & %d; const float mine = up ? s%d : s%d, other = up ? s%d : s%d; s%d = mine + dppx(other, %d); }\n", bit[st], k + h, k,
                  k, k + h, k, which[st]);
        }
        if (n & 1) {
            if (h > 0) o("    s%d = s%d + dppx(s%d, %d);\n", h, n - 1, n - 1, which[st]);
            else o("    s0 += dppx(s0, %d);\n", which[st]);
        }
        n = h + (n & 1);
    }
}

std::string which_sum(int n)
{
    static const int bit[4] = {8, 4, 2, 1};
    std::vector<std::string> e(n);
    for (int j = 0; j < n; ++j) e[j] = std::to_string(j);
    for (int st = 0; st < 4; ++st) {
        const int h = n / 2;
        std::vector<std::string> f;
        for (int k = 0; k < h; ++k) f.push_back("((l & " + std::to_string(bit[st]) + ") ? " + e[k + h] + " : " + e[k] + ")");
        if (n & 1) f.push_back(e[n - 1]);
        e = f;
        n = h + (n & 1);
    }
    return e[0];
}

// A wavefront's rows of an input: lane e takes word e of its four samples, lanes past the end the last word again, and samples
// past the batch the last sample again.  <p>_at<class>_<count>_<x>: where, in bytes from the first sample's row; <p>_w..: the
// word's place in LDS, <p>_r..: that of the sample which it is (to store from, the same word again too).
void emit_places(Src &o, const Layout &Y, const std::vector<int> &cls, const char *p, int first)
{
    std::vector<std::vector<int>> seen;
    auto fresh = [&](std::vector<int> key) {
        if (std::find(seen.begin(), seen.end(), key) != seen.end()) return false;
        seen.push_back(key);
        return true;
    };
    o("  int %s_lane = lane; asm volatile(\"\" : \"+v\"(%s_lane));\n", p, p);
    for (int t = first; t < Y.n; ++t) {
        const int cnt = t == 0 ? Y.m[0] : Y.nb[t];
        if (fresh({-1, cls[t]})) o("  const long long %s_first%d = wg * %d * A.ld[%d];\n", p, cls[t], 4 * kSP, t);
        const bool places = fresh({cnt}), at = fresh({cls[t], cnt});
        for (int x = 0; x < kSP * cnt; x += 64) {
            const std::string id = std::to_string(cnt) + "_" + std::to_string(x), e = std::string(p) + "_e" + id, q = std::string(p) + "_q" + id,
                              c = std::string(p) + "_c" + id, i = std::string(p) + "_i" + id;
            if (places) {
                o("  const int %s = %s_lane + %d < %d ? %s_lane + %d : %d, %s = %s / %d, %s = %s < n_live ? %s : n_live - 1, %s = %s - %s * %d;\n", e.c_str(), p, x,
                  kSP * cnt, p, x, kSP * cnt - 1, q.c_str(), e.c_str(), cnt, c.c_str(), q.c_str(), q.c_str(), i.c_str(), e.c_str(), q.c_str(), cnt);
                if (first == 0) o("  const int %s_w%s = %s * %d + %s;\n", p, id.c_str(), q.c_str(), Y.stride, i.c_str());
                else o("  const int %s_r%s = %s * %d + %s;\n", p, id.c_str(), c.c_str(), Y.stride, i.c_str());
            }
            if (at) o("  const unsigned %s_at%d_%s = 4u * ((unsigned)%s * (unsigned)A.ld[%d] + (unsigned)%s);\n", p, cls[t], id.c_str(), c.c_str(), t, i.c_str());
        }
    }
}

// Writes the code of one sweep (forward, result, reverse): calm where no sum can exceed 1.
struct Sweep {
    const Layout &Y;
    Src &o;
    const bool calm;
    const int n1;
    const std::vector<int> &cls;        // see chain_source
    int dirty = 0;                      // entries of the row buffer from here on are zeros

    Sweep(const Layout &y, Src &src, bool c, const std::vector<int> &classes) : Y(y), o(src), calm(c), n1(y.n - 1), cls(classes), dirty(y.m[0]) {}

    static std::string num(const char *name, int k) { return std::string(name) + std::to_string(k); }
    static std::string at(const char *name, int t, int k) { return std::string(name) + std::to_string(t) + "_" + std::to_string(k); }
    std::string tag(const std::string &x) const { return calm ? x : "__builtin_fabsf(" + x + ")"; }

    void fence() { o("  fence();\n"); }

    // `name`<t>_<j> = the short operand of stage t
    void load_d(const char *name, int t)
    {
        const int nb = Y.nb[t], at = Y.off_d + t * Y.pitch;
        int j = 0;
        for (; j + 4 <= nb; j += 4) {
            o("    const float4 %sq%d_%d = *reinterpret_cast<const float4 *>(base + %d);\n   ", name, t, j, at + j);
            for (int x = 0; x < 4; ++x) o(" const float %s%d_%d = %sq%d_%d.%c;", name, t, j + x, name, t, j, "xyzw"[x]);
            o("\n");
        }
        if (j + 2 <= nb) {
            o("    const float2 %sq%d_%d = *reinterpret_cast<const float2 *>(base + %d); const float %s%d_%d = %sq%d_%d.x, %s%d_%d = %sq%d_%d.y;\n", name, t, j, at + j,
              name, t, j, name, t, j, name, t, j + 1, name, t, j);
            j += 2;
        }
        if (j < nb) o("    const float %s%d_%d = base[%d];\n", name, t, j, at + j);
    }

    // a row of w entries per lane into the row buffer; zeros behind it up to `need`
    void put_row(const std::vector<std::string> &v, int need)
    {
        const int w = static_cast<int>(v.size());
        o("  { DOL_ROW(wp, %d, %d);\n", Y.row, w);
        for (int k = 0; k < w; ++k) o("    wp[%d] = %s;\n", k, v[k].c_str());
        o("  }\n");
        const int end = std::min(dirty, need);
        for (int x = kL * w; x < end; x += kL) o("  base[%d + l] = 0.0f;\n", Y.row + x);       // (the row buffer holds whole sixteens)
        dirty = end >= dirty ? kL * w : std::max(dirty, kL * w);
        fence();
    }

    // `name`<k> = the entry k + 1 places before (after) the lane's block, k < count, of a row whose block is v
    void shifted(const char *name, const std::vector<std::string> &v, int count, bool before)
    {
        const int w = static_cast<int>(v.size());
        for (int e = 0; e < count; ++e) {
            const int lanes = 1 + e / w, k = before ? w - 1 - e % w : e % w;
            if (lanes > kL - 1) o("    const float %s%d = 0.0f;\n", name, e);
            else o("    float %s%d = from_lane<%d>(%s); opaque(%s%d);\n", name, e, (before ? 0x110 : 0x100) + lanes, v[k].c_str(), name, e);
        }
    }

    std::vector<std::string> block(const char *name, int t, int w) const
    {
        std::vector<std::string> v(w);
        for (int k = 0; k < w; ++k) v[k] = at(name, t, k);
        return v;
    }

    // dst<k> = sum over j of the entries k - j of a row (of tags) with the short operand: descending j (forward) or ascending
    void convolve(const char *dst, int w, const char *d, int t, const std::vector<std::string> &own, const char *before, bool ascending)
    {
        const int nb = Y.nb[t];
        for (int k = 0; k < w; ++k) {
            o("    float %s%d = 0.0f;\n", dst, k);
            for (int x = 0; x < nb; ++x) {
                const int j = ascending ? x : nb - 1 - x, e = k - j;
                const std::string src = e >= 0 ? own[e] : num(before, -1 - e);
                o("    %s%d = __builtin_fmaf(%s, %s, %s%d);\n", dst, k, src.c_str(), at(d, t, j).c_str(), dst, k);
            }
        }
    }

    // v<t>_<k>: acc_t's block, signs and all; u<t>_<k>: its tags, where there can be signs
    void forward()
    {
        for (int k = 0; k < Y.w[0]; ++k) o("  const float v0_%d = base[%d + l * %d + %d];\n", k, Y.row, Y.w[0], k);
        if (Y.hist[0] >= 0) keep(0);
        for (int t = 1; t <= n1; ++t)
            for (int k = 0; k < Y.w[t]; ++k) o(calm ? "  float v%d_%d;\n" : "  float v%d_%d, u%d_%d;\n", t, k, t, k);
        for (int t = 1; t <= n1; ++t) {
            const int nb = Y.nb[t], w = Y.w[t], w1 = Y.w[t - 1];
            std::vector<std::string> own = block(calm || t == 1 ? "v" : "u", t - 1, w1);
            if (w != w1 && t > 1) put_row(own, kL * w);
            if (t == 1) load_d("f", 1);
            if (t < n1) load_d("f", t + 1);             // (on its way meanwhile)
            fence();
            o("  {\n");
            if (w == w1) {
                shifted("e", own, nb - 1, true);
            } else {
                o("    DOL_ROW(rp, %d, %d);\n", Y.row - (nb - 1), w);
                for (int e = nb - 2; e >= 0; --e) o("    const float e%d = rp[%d];\n", e, nb - 2 - e);
                own.resize(w);
                for (int k = 0; k < w; ++k) { o("    const float r%d = rp[%d];\n", k, nb - 1 + k); own[k] = num("r", k); }
            }
            convolve("p", w, "f", t, own, "e", false);
            for (int k = 0; k < w; ++k) {
                if (calm) o("    v%d_%d = p%d;\n", t, k, k);
                else o("    v%d_%d = p%d <= 1.0f ? p%d : -1.0f; u%d_%d = fminf(p%d, 1.0f);\n", t, k, k, k, t, k, k);
            }
            o("  }\n");
            fence();
            if (t < n1 && Y.hist[t] >= 0) keep(t);
        }
    }

    void keep(int t)
    {
        for (int k = 0; k < Y.w[t]; ++k) o("  base[%d + l] = v%d_%d;\n", Y.hist[t] + kL * k, t, k);
    }

    // acc_t's block again, in the registers x<t>_<k>
    std::vector<std::string> recall(int t)
    {
        if (Y.hist[t] < 0) return block("v", t, Y.w[t]);
        for (int k = 0; k < Y.w[t]; ++k) o("    const float x%d_%d = base[%d + l];\n", t, k, Y.hist[t] + kL * k);
        return block("x", t, Y.w[t]);
    }

    void result()
    {
        const int m = Y.m[n1];
        put_row(block("v", n1, Y.w[n1]), 0);
        o("  { SAMPLE(s); if (A.out && s < A.batch) { float *os = A.out + s * A.ldo;\n");
        for (int x = 0; x < m; x += kL)
            o("    %s os[%d + l] = %s;\n", m - x >= kL ? "" : (std::string("if (l < ") + std::to_string(m - x) + ")").c_str(), x,
              tag("base[" + std::to_string(Y.row + x) + " + l]").c_str());
        o("  } }\n  if (!A.backward) return;\n");
        fence();
    }

    // the short operand's gradient: sums of the lanes' shares s0 ..; it takes the place of the operand's row, which is spent
    void give_gb(int t)
    {
        emit_scattered_sums(o, Y.nb[t]);
        o("    base[%d + jl%d] = s0;\n", Y.off_d + t * Y.pitch, Y.nb[t]);
    }

    // gw<k> = the gradient of stage t's columns from the first row (of width w[t - 1]) that the lane will sum, out of g<t>_<k>
    void window(int t)
    {
        const int w = Y.w[t], w1 = Y.w[t - 1], nb = Y.nb[t];
        const std::vector<std::string> g = block("g", t, w);
        if (w == w1) {
            for (int k = 0; k < w; ++k) o("    gw%d = %s;\n", k, g[k].c_str());
            o("    {\n");
            shifted("e", g, nb - 1, false);
            for (int e = 0; e < nb - 1; ++e) o("    gw%d = e%d;\n", w + e, e);
            o("    }\n");
        } else {
            put_row(g, 0);
            o("  { DOL_ROW(rp, %d, %d);\n", Y.row, w1);
            for (int k = 0; k < w1 + nb - 1; ++k) o("    gw%d = rp[%d];\n", k, k);
            o("  }\n");
            fence();
        }
    }

    // stage t of the reverse sweep, columns counted from the row's first: gw -> g<t - 1>_<k> and the short operand's gradient
    // (first, last: the stages of this run of the code)
    void stage(int t, int first, int last)
    {
        const int nb = Y.nb[t], m = Y.m[t - 1], w = Y.w[t - 1];
        if (t == first) load_d("d", t);
        if (t > last) load_d("d", t - 1);
        o("  {\n");
        fence();
        const std::vector<std::string> x = recall(t - 1);
        for (int j = 0; j < nb; ++j) o("    float s%d = 0.0f;\n", j);
        for (int k = 0; k < w; ++k) {
            o("    { float acc = 0.0f;\n");
            for (int j = 0; j < nb; ++j) o("      acc = __builtin_fmaf(gw%d, d%d_%d, acc);\n", k + j, t, j);
            // rows past the operand's last symbol hold 0; a row whose own sum was clamped (sign) passes no gradient on
            // (only the last lanes' last rows can lie past the end: the test is written where that can happen)
            std::string cond;
            if ((kL - 1) * w + k >= m) cond = "l < " + std::to_string(ceil_div(m - k, w));
            if (t > 1 && !calm) cond += (cond.empty() ? "!(" : " && !(") + x[k] + " < 0.0f)";
            o("      g%d_%d = %s; }\n", t - 1, k, cond.empty() ? "acc" : (cond + " ? acc : 0.0f").c_str());
            std::string y = x[k];
            if (t > 1 && !calm) {
                o("    float y%d = __builtin_fabsf(%s); opaque(y%d);\n", k, x[k].c_str(), k);
                y = num("y", k);
            }
            for (int j = 0; j < nb; ++j) o("    s%d = __builtin_fmaf(gw%d, %s, s%d);\n", j, k + j, y.c_str(), j);
        }
        give_gb(t);
        o("  }\n");
    }

    // the late stages under a target (calm sweeps): S<t>_<k> = gradient of column target - (l * ws + k)
    void from_target()
    {
        const int m = Y.m[n1];
        o("    const bool in_row = target >= 0 && target < %d;\n    const int tgt = in_row ? target : 0;\n", m);
        o("    const float xv = base[%d + tgt], gv = in_row ? -1.0f / fmaxf(xv, 1.17549435e-38f) : 0.0f;\n", Y.row);
        fence();
        for (int t = n1 - 1; t >= Y.ts; --t)
            for (int k = 0; k < Y.ws[t]; ++k) o("    float S%d_%d;\n", t, k);
        // the last stage: one column
        {
            const int nb = Y.nb[n1], ws = Y.ws[n1 - 1];
            o("    {\n");
            put_row(recall(n1 - 1), m);
            o("    const float x = base[%d + tgt - l];\n", Y.row);
            for (int k = 0; k < ws; ++k) {
                o("    { const int j = l * %d + %d; const float v = base[%d + (j < %d ? j : %d)]; S%d_%d = j < %d ? gv * v : 0.0f; }\n", ws, k, Y.off_d + n1 * Y.pitch, nb,
                  nb - 1, n1 - 1, k, nb);
            }
            fence();
            o("    base[l < %d ? %d + l : %d] = gv * x;\n    }\n", nb, Y.off_d + n1 * Y.pitch, Y.off_d);       // (row 0 of the short inputs is free)
        }
        for (int t = n1 - 1; t > Y.ts; --t) {
            const int nb = Y.nb[t], ws = Y.ws[t], ws1 = Y.ws[t - 1], win = ws + nb - 1;
            if (t == n1 - 1) load_d("d", t);
            if (t - 1 > Y.ts) load_d("d", t - 1);
            o("  {\n");
            put_row(recall(t - 1), m);
            at_target("ap", ws, win);
            for (int e = 0; e < win; ++e) o("    const float a%d = ap[%d];\n", e, win - 1 - e);
            fence();
            const std::vector<std::string> S = block("S", t, ws);
            for (int j = 0; j < nb; ++j) {
                o("    float s%d = 0.0f;\n", j);
                for (int k = 0; k < ws; ++k) o("    s%d = __builtin_fmaf(%s, a%d, s%d);\n", j, S[k].c_str(), k + j, j);
            }
            std::vector<std::string> own = S;
            if (ws == ws1) {
                shifted("e", S, nb - 1, true);
            } else {
                put_row(S, kL * ws1);
                o("    DOL_ROW(rp, %d, %d);\n", Y.row - (nb - 1), ws1);
                for (int e = nb - 2; e >= 0; --e) o("    const float e%d = rp[%d];\n", e, nb - 2 - e);
                own.resize(ws1);
                for (int k = 0; k < ws1; ++k) { o("    const float r%d = rp[%d];\n", k, nb - 1 + k); own[k] = num("r", k); }
                fence();
            }
            convolve("p", ws1, "d", t, own, "e", true);
            for (int k = 0; k < ws1; ++k) o("    S%d_%d = p%d;\n", t - 1, k, k);
            give_gb(t);
            o("  }\n");
        }
        // back to columns
        put_row(block("S", Y.ts, Y.ws[Y.ts]), m);
        const int w = Y.w[std::max(0, Y.ts - 1)], win = Y.ts > 0 ? w + Y.nb[Y.ts] - 1 : w;
        o("  {\n");
        at_target("gp", w, win);
        for (int e = 0; e < win; ++e) {
            if (Y.ts > 0) o("    gw%d = gp[%d];\n", e, win - 1 - e);
            else o("    g0_%d = gp[%d];\n", e, win - 1 - e);
        }
        o("  }\n");
        fence();
    }

    // name[win - 1 - e] = the row buffer's entry at target - (l * w + e)
    void at_target(const char *name, int w, int win)
    {
        o("    int %s_i = qb + 4 * (%d + tgt) - l * %d; opaque(%s_i); const float *%s = reinterpret_cast<const float *>(reinterpret_cast<const char *>(lds) + %s_i);\n",
          name, Y.row - (win - 1), 4 * w, name, name, name);
    }

    // the gradient that comes in, from the row's first column: g<n1 - 1>_<k> (target) or g<n1>_<k>
    void from_row()
    {
        const int t = n1, nb = Y.nb[t], m = Y.m[t - 1], w = Y.w[t - 1];
        // a target: the last stage's gradient row is zero but for one entry G, so the first operand's gradient is
        // G * d[target - i] (nb entries) and the short operand's G * a[target - j]; a lane per entry
        o("  if (A.target) {\n    float gv = 0.0f;\n");
        o("    if (target >= 0 && target < %d) { const float xv = base[%d + target]; gv = xv < 0.0f ? 0.0f : -1.0f / fmaxf(xv, 1.17549435e-38f); }\n", Y.m[n1], Y.row);
        fence();
        const int was = dirty;
        put_row(recall(t - 1), 0);
        o("    const int i = target - l;\n    const bool has = target >= 0 && target < %d && l < %d && i >= 0 && i < %d;\n", Y.m[n1], nb, m);
        o("    float x = 0.0f;\n    if (has) x = base[%d + i];\n", Y.row);
        fence();
        for (int x = 0; x < w; ++x) o("    base[%d + l] = 0.0f;\n", Y.row + kL * x);
        fence();
        o("    if (has) base[%d + i] = %sgv * base[%d + l];\n", Y.row, t > 1 ? "x < 0.0f ? 0.0f : " : "", Y.off_d + t * Y.pitch);
        fence();
        o("    { DOL_ROW(rp, %d, %d);\n", Y.row, w);
        for (int k = 0; k < w; ++k) o("      g%d_%d = rp[%d];\n", t - 1, k, k);
        o("    }\n    if (l < %d) base[%d + l] = has ? gv * __builtin_fabsf(x) : 0.0f;\n", nb, Y.off_d + t * Y.pitch);
        fence();
        o("  } else {\n    SAMPLE(s);\n    const float *gs = A.gout + (s < A.batch ? s : A.batch - 1) * A.ldg;\n");
        dirty = was;
        for (int x = 0; x < Y.w[t]; ++x)
            o("    { const int c = %d + l; float v = 0.0f; if (c < %d) v = gs[c]; base[%d + c] = v; }\n", kL * x, Y.m[t], Y.row);
        fence();
        o("    { DOL_ROW(rp, %d, %d);\n", Y.row, Y.w[t]);
        for (int k = 0; k < Y.w[t]; ++k) {
            if (calm) o("      g%d_%d = rp[%d];\n", t, k, k);
            else o("      g%d_%d = v%d_%d < 0.0f ? 0.0f : rp[%d];\n", t, k, t, k, k);
        }
        o("    }\n");
        fence();
        window(t);
        stage(t, t, t);
        o("  }\n");
    }

    void reverse()
    {
        int win = 0;
        for (int t = 1; t <= n1; ++t) win = std::max(win, Y.w[t - 1] + Y.nb[t] - 1);
        for (int k = 0; k < win; ++k) o("  float gw%d;\n", k);
        for (int t = 0; t <= n1; ++t)
            for (int k = 0; k < Y.w[t]; ++k) o("  float g%d_%d;\n", t, k);
        int from = n1;
        if (calm) {
            const int was = dirty;
            o("  if (bounded && A.target) {\n");
            from_target();
            dirty = was;
            o("  } else {\n");
            from_row();
            for (int t = n1 - 1; t > Y.ts; --t) { window(t); stage(t, n1 - 1, Y.ts + 1); }
            if (Y.ts > 0) window(Y.ts);
            o("  }\n");
            if (Y.ts > 0) stage(Y.ts, Y.ts, 1);
            from = Y.ts;
        } else {
            from_row();
        }
        for (int t = from - 1; t > 0; --t) { window(t); stage(t, calm ? Y.ts : n1 - 1, 1); }
        fence();
        emit_places(o, Y, cls, "z", 1);
        for (int t = 1; t <= n1; ++t)
            for (int x = 0; x < kSP * Y.nb[t]; x += 64)
                o("  const float out%d_%d = lds[z_r%d_%d + %d];\n", t, x, Y.nb[t], x, Y.off_d + t * Y.pitch);
        for (int t = 1; t <= n1; ++t) {
            o("  if (A.gin[%d]) { char *dst = reinterpret_cast<char *>(A.gin[%d]) + z_first%d;", t, t, cls[t]);
            for (int x = 0; x < kSP * Y.nb[t]; x += 64) o(" *reinterpret_cast<float *>(dst + z_at%d_%d_%d) = out%d_%d;", cls[t], Y.nb[t], x, t, x);
            o(" }\n");
        }
        o("  SAMPLE(s);\n  if (s < A.batch && A.gin[0]) { float *dst = A.gin[0] + s * A.ld[0] + l * %d;\n", Y.w[0]);
        for (int k = 0; k < Y.w[0]; ++k) o("    if (l * %d + %d < %d) dst[%d] = g0_%d;\n", Y.w[0], k, Y.m[0], k, k);
        o("  }\n");
    }
};

// cls[t]: the first input that shares the registers of its rows' addresses with input t (see launch_fold_chain).
std::string chain_source(const std::vector<int> &shape, const std::vector<int> &cls)
{
    const Layout Y = lay_out(shape);
    const int n = Y.n;
    Src o;
    // (leading dimensions as 32-bit words: a row's offset is then one 32 x 32 -> 64 bit multiply-add)
    o("struct Args { int batch; int backward; const float *in[%d]; int ld[%d]; float *gin[%d]; float *out; int ldo; "
      "const int *target; const float *gout; int ldg; };\n", kFoldChainMax, kFoldChainMax, kFoldChainMax);
    o("__device__ __forceinline__ void fence() { __builtin_amdgcn_fence(__ATOMIC_RELEASE, \"wavefront\"); __builtin_amdgcn_wave_barrier(); "
      "__builtin_amdgcn_fence(__ATOMIC_ACQUIRE, \"wavefront\"); }\n");
    o("__device__ __forceinline__ float dppx(float x, int which) {\n"
      "  switch (which) {\n"
      "  case 0: return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, false));\n"
      "  case 1: return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xF, 0xF, false));\n"
      "  case 2: return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xF, 0xF, false));\n"
      "  default: return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x140, 0xF, 0xF, false)); } }\n");
    // another lane's value (zero where there is none in the sample's 16); opaque: the shift stays an instruction of its own,
    // a multiply-add that shifts its operand takes twice as long and there are up to 16 of them to a shift
    o("template <int CTRL> __device__ __forceinline__ float from_lane(float x) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true)); }\n"
      "#define opaque(x) asm(\"\" : \"+v\"(x))\n");
    o("extern \"C\" __global__ void __launch_bounds__(64, 2) damp_fold_chain_kernel(const Args A)\n{\n");
    o("  __shared__ __align__(16) float lds[%d];\n", kSP * Y.stride);
    o("  const int lane = threadIdx.x, l = lane & %d, q = lane >> 4;\n", kL - 1);
    // workgroups are dealt round-robin to the 8 XCDs: give every XCD a contiguous range of samples
    o("  const unsigned id = blockIdx.x, nwg = gridDim.x, xcd = id & 7u, per = nwg >> 3, rem = nwg & 7u;\n");
    o("  const long long wg = (long long)(xcd * per + (xcd < rem ? xcd : rem) + (id >> 3));\n");
    // a lane's sample, worked out again where it is needed (kept all along it is spilled)
    o("#define SAMPLE(name) int name##_z = lane; asm volatile(\"\" : \"+v\"(name##_z)); const long long name = wg * %d + (name##_z >> 4)\n", kSP);
    o("  float *base = lds + q * %d;\n", Y.stride);
    // A row is addressed through an index the compiler cannot see through: every access of a stage is then that register
    // plus a small immediate (one instruction), where a folded constant beyond the reach of the two-word LDS instructions'
    // offset field would cost an address addition per access.
    o("  const int qb = q * %d;\n", 4 * Y.stride);
    {
        bool len[kNBR + 1] = {};
        for (int t = 1; t < n; ++t)     // which of a short operand's gradient sums a lane ends up with (see emit_scattered_sums)
            if (!len[Y.nb[t]]) { len[Y.nb[t]] = true; o("  const int jl%d = %s;\n", Y.nb[t], which_sum(Y.nb[t]).c_str()); }
    }
    // (volatile: not worked out once and kept in a register for every width)
    o("#define DOL_ROW(name, start, step) int name##_i; asm volatile(\"v_mad_u32_u24 %%0, %%1, %%2, %%3\" : \"=v\"(name##_i) : \"v\"(l), \"v\"(4 * step), \"v\"(qb)); "
      "name##_i += 4 * (start); opaque(name##_i); float *name = reinterpret_cast<float *>(reinterpret_cast<char *>(lds) + name##_i)\n");
    // ---- inputs: all loads first, then the LDS writes
    o("  const int n_live = A.batch - (int)(wg * %d) < %d ? A.batch - (int)(wg * %d) : %d;\n", kSP, kSP, kSP, kSP);
    o("  int target = -1;\n  if (A.target) target = A.target[wg * %d + (q < n_live ? q : n_live - 1)];\n", kSP);
    emit_places(o, Y, cls, "a", 0);
    {
        for (int t = 0; t < n; ++t) {
            const int cnt = t == 0 ? Y.m[0] : Y.nb[t];
            for (int x = 0; x < kSP * cnt; x += 64)
                o("  const float in%d_%d = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(A.in[%d]) + a_first%d + a_at%d_%d_%d);\n", t, x, t, cls[t],
                  cls[t], cnt, x);
        }
        // the row buffer starts as zeros
        for (int x = 0; x < Y.off_d; x += 4 * kL)
            o("  %s*reinterpret_cast<float4 *>(base + %d + 4 * l) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);\n",
              Y.off_d - x >= 4 * kL ? "" : (std::string("if (l < ") + std::to_string((Y.off_d - x) / 4) + ") ").c_str(), x);
        o("  fence();\n");
        for (int t = 0; t < n; ++t) {
            const int cnt = t == 0 ? Y.m[0] : Y.nb[t], dst = t == 0 ? Y.row : Y.off_d + t * Y.pitch;
            for (int x = 0; x < kSP * cnt; x += 64) o("  lds[a_w%d_%d + %d] = in%d_%d;\n", cnt, x, dst, t, x);
        }
    }
    o("  fence();\n");
    // ---- can any sum of this wavefront's samples exceed 1?  max(acc_t) <= max(acc_0) * product of the sums of the first t
    // short rows.  A later row with a small sum must not make up for an earlier one with a large sum: with every factor taken
    // as at least 1 the product over all rows bounds that over any first few.  What rounding adds is far below the distance to
    // 1 that is asked for.  Where no sum can exceed 1, and no tag is negative, the sweeps below run without a clamp, a sign
    // or a gate.  bounded: nor can a product of short rows with the loss's gradient overflow, so that entries outside a row,
    // which the late stages carry along, are numbers.
    o("  bool calm, bounded;\n  { float top = 0.0f, prod = 1.0f, least = 0.0f; bool bad = false;\n");
    for (int x = 0; x < Y.m[0]; x += kL)
        o("    if (l + %d < %d) { const float v = base[%d + l]; top = fmaxf(top, v); bad |= !(v >= 0.0f); }\n", x, Y.m[0], Y.row + x);
    for (int t0 = 1; t0 < n; t0 += kL) {
        o("    if (l + %d < %d) { const float *row = base + %d + l * %d; float sum = 0.0f;\n", t0, n, Y.off_d + t0 * Y.pitch, Y.pitch);
        // (rows of different lengths: entries past a row's end were never written and count as 0)
        int nb_max = 0;
        bool same = true;
        for (int t = t0; t < std::min(n, t0 + kL); ++t) { nb_max = std::max(nb_max, Y.nb[t]); same = same && Y.nb[t] == Y.nb[t0]; }
        if (!same) {
            o("      int len = 0;\n");
            for (int t = t0; t < std::min(n, t0 + kL); ++t) o("      len = l == %d ? %d : len;\n", t - t0, Y.nb[t]);
        }
        for (int j = 0; j < nb_max; ++j)
            o("      { const float v = %srow[%d]%s; sum += v; least = fminf(least, v); }\n", same ? "" : (std::to_string(j) + " < len ? ").c_str(), j, same ? "" : " : 0.0f");
        o("      bad |= !(sum >= 0.0f); prod *= fmaxf(sum, 1.0f); }\n");        // (a sum with a NaN in it is one)
    }
    for (int st = 0; st < 4; ++st) o("    top = fmaxf(top, dppx(top, %d)); prod *= dppx(prod, %d);\n", st, st);
    o("    calm = __ballot(bad || least < 0.0f || !(top * prod <= 0.999f)) == 0;\n    bounded = __ballot(!(prod <= 2.0f)) == 0; }\n");
    for (int calm = 1; calm >= 0; --calm) {
        o(calm ? "  if (calm) {\n" : "  } else {\n");
        Sweep sweep(Y, o, calm != 0, cls);
        sweep.forward();
        sweep.result();
        sweep.reverse();
    }
    o("  }\n}\n");

    return o.s;
}

struct ChainKernel {
    hipModule_t mod = nullptr;
    hipFunction_t fn = nullptr;
    dol_status status = DOL_OK;
};

struct ChainArgs {
    int32_t batch, backward;
    const float *in[kFoldChainMax];
    int32_t ld[kFoldChainMax];
    float *gin[kFoldChainMax];
    float *out;
    int32_t ldo;
    const int32_t *target;
    const float *gout;
    int32_t ldg;
};

}  // namespace

bool fold_chain_ok(int n, const int32_t *m, const int32_t *nb, const int64_t *ld, int64_t ldo, int64_t ldg)
{
    if (n < 2 || n > kFoldChainMax) return false;
    for (int t = 0; t < n; ++t)
        if (ld[t] > (1 << 28)) return false;            // (four rows' bytes in 32 bits)
    if (ldo > INT32_MAX || ldg > INT32_MAX) return false;
    std::vector<int> shape{n, m[0]};
    for (int t = 1; t < n; ++t) {
        if (nb[t] < 1 || nb[t] > kNBR) return false;
        shape.push_back(nb[t]);
    }
    if (m[0] < 1 || m[0] > 256) return false;
    static std::mutex mu;
    static std::map<std::vector<int>, bool> known;          // (laying a chain out takes 70 us)
    std::lock_guard<std::mutex> lock(mu);
    auto it = known.find(shape);
    if (it == known.end()) {
        const Layout Y = lay_out(shape);
        if (known.size() >= 4096) known.clear();
        it = known.emplace(std::move(shape), sizeof(float) * kSP * static_cast<size_t>(Y.stride) <= kChainLdsMax).first;
    }
    return it->second;
}

dol_status launch_fold_chain(int n, const int32_t *m, const int32_t *nb, int32_t batch, const float *const *in, const int64_t *ld,
                             float *const *gin, float *out, int64_t ldo, const int32_t *target, const float *gout, int64_t ldg,
                             int32_t backward, hipStream_t st, bool *done)
{
    *done = false;
    static std::mutex mu;
    static std::map<std::pair<int, std::vector<int>>, ChainKernel> cache;    // per device, shape and kind of strides; lives until the process ends
    std::vector<int> shape{n, m[0]};
    for (int t = 1; t < n; ++t) shape.push_back(nb[t]);
    const unsigned grid = static_cast<unsigned>((static_cast<int64_t>(batch) + kSP - 1) / kSP);
    int dev = 0;
    DOL_HIP(hipGetDevice(&dev));
    hipFunction_t fn = nullptr;
    {
        std::lock_guard<std::mutex> lock(mu);
        // Inputs of one number of symbols mostly lie one row length apart and then share their addresses; where any two of them
        // do not, every input has its own, in a build that serves all strides.  (Sum-15, us, shared / not: B=64 8.0 / 8.55,
        // 4 096 9.2 / 9.9, 524 288 493 / 507; to compile takes 0.45 s, and 0.15 to 1 s for other chains.)
        std::vector<int> cls(n), keyed(shape);
        bool shared = true;
        for (int t = 0; t < n; ++t) {
            const auto width = [&](int u) { return u ? nb[u] : m[0]; };
            cls[t] = 0;
            while (width(cls[t]) != width(t)) ++cls[t];
            shared = shared && ld[cls[t]] == ld[t];
        }
        if (!shared)
            for (int t = 0; t < n; ++t) cls[t] = t;
        keyed.push_back(shared);
        auto key = std::make_pair(dev, keyed);
        auto it = cache.find(key);
        if (it == cache.end()) {
            ChainKernel k;
            k.status = jit_compile(chain_source(shape, cls), "damp_fold_chain_kernel", &k.mod, &k.fn);
            it = cache.emplace(key, k).first;
        }
        if (it->second.status != DOL_OK) return DOL_OK;         // code that does not build leaves the call to the kernels of fold.hip
        fn = it->second.fn;
    }
    ChainArgs A{};
    A.batch = batch, A.backward = backward;
    for (int t = 0; t < n; ++t) { A.in[t] = in[t]; A.ld[t] = static_cast<int32_t>(ld[t]); A.gin[t] = gin ? gin[t] : nullptr; }
    A.out = out, A.ldo = static_cast<int32_t>(ldo), A.target = target, A.gout = gout, A.ldg = static_cast<int32_t>(ldg);
    void *args[] = {&A};
    DOL_HIP(hipModuleLaunchKernel(fn, grid, 1, 1, 64, 1, 1, 0, st, args, nullptr));
    *done = true;
    return DOL_OK;
}

}  // namespace dol
