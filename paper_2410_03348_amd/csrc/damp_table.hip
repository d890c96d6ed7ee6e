// DAMP apply2 for small arbitrary (hashed, dense or sparse) function tables, as code written for the table.
//
//     out[s, c] = min(1, sum over the tuples (i, j) of column c, ascending (i, j), of a[s, i] * b[s, j])
//     ga[s, i]  = sum_j gh[s, col(i, j)] * b[s, j],    gb[s, j] = sum_i gh[s, col(i, j)] * a[s, i]
//
// The symbol side is batch-invariant (Sec. 3.1.2: the user function is evaluated once, before any tag is touched),
// so with one sample per lane every tuple index is the same for all 64 lanes of a wavefront.  A table whose operand
// rows fit in registers (at most 64 symbols each) is therefore compiled, once per table and on its first use, into
// straight-line code: the operand rows of a lane's sample sit in registers and every tuple is ONE fused multiply-add
// on named registers - no index loads, no operand gathers.  (A generic kernel has to fetch both operands of every
// tuple from LDS, 8 bytes per multiply-add, and stops at the rate of the LDS pipe; see damp_lds.hip, which still
// serves larger tables and padded or unaligned tensors.)  A column's tuples keep their ascending (i, j) order and
// start from 0, so the sum is bit for bit the one dol_apply2 defines and the clamp decisions agree.
//
// Layout of a launch: a workgroup of four wavefronts owns a tile of 64 samples (batches too small to give every compute
// unit two such tiles: eight wavefronts, or tiles of 32 samples; see build_for).  The tile's operand rows travel
// HBM -> LDS with flat 16-byte loads (rows of whole 16-byte pieces an odd number of them apart, which keeps a lane's
// 16-byte reads of its own row off its neighbours' banks; rows of any other length as they lie in memory, read word by word),
// each lane pulls its sample's rows into registers, the wavefronts split the work (forward: 64 output columns at a time each;
// backward: half of the rows of one operand each), results go back through LDS and leave as flat 16-byte stores.
// Symbol counts that are no multiples of four came here late: 50 x 37 -> 201, us forward / backward, B=10 007 11.7 / 15.4 through
// the gathers of damp_lds.hip, 5.3 / 9.2 here, B=100 000 74.5 / 87.1 and 27.2 / 41.8; 61 x 5 -> 77 at 100 000 38 / 88, 18 / 24.
//
// Backward needs gh = g * [pre <= 1].  For tags in [0, 1] a column's sum is bounded by max(a) * sum(b) * M, M = the
// most tuples of one column that share a second-operand symbol (and the same with the operands' roles swapped): a
// tile whose samples all stay below 0.9999 by that bound cannot hold a clamped column and passes g through without
// ever reading the forward result; any other tile recomputes pre with the forward code and gates with it.
//
// Merged forms (dol_apply2_filter_union and its reverse): the same kernels with Filter and Union folded into their
// epilogues, so the Apply's result never leaves the chip; the forward pass leaves one word per sample saying whether
// any clamp acted, and the reverse pass re-derives decisions only for tiles that hold such a sample.  The two merged
// bodies are also emitted one after the other into one kernel (dol_apply2_filter_union_forward_backward): the operands' rows stay
// in registers (see keeps_rows) and the clamp words in LDS.  Where the result has the third Distribution's symbols in its order (an aligned plan)
// the first pieces of that operand and of the gradient are asked for together with a's and b's, the kept columns are bits in
// LDS, and where no clamp acted the third gradient leaves from the registers that bring the gradient in.  One tile to a unit,
// its phases one after the other, bounds it: 64 x 64 -> 256 at B = 16 384 (84 MB) took 27.6 us with the bodies apart, each staging
// a and b and the second reading the gradient twice; 20.5 so, where a copy takes 16.7.  (Two groups of the gradient on their way
// instead of one: 24.4.)
#include "internal.h"

#include <hip/hiprtc.h>

#include <cstdarg>
#include <mutex>

namespace dol {

constexpr int kJitTile = 64;            // samples per tile = lanes per wavefront
constexpr int kJitWavesLarge = 4;       // wavefronts per workgroup: four, or eight in the builds for small batches
constexpr int kJitGroup = 64;           // output columns a wavefront takes at a time
constexpr int kJitMaxSym = 64;          // operand rows live in registers
constexpr int kJitMaxOut = 1024;
constexpr int kJitMaxMergeOut = 512;   // merged launches keep the Apply's whole result tile in LDS
constexpr int64_t kJitMaxTuples = 16384;

// (the last two: merged launches whose filter-union plan is `aligned`, see UnionPlan)
enum { kSlotFwd = 0, kSlotBwd = 1, kSlotMergeFwd = 2, kSlotMergeBwd = 3, kSlotMergeFwdAligned = 4, kSlotMergeBwdAligned = 5, kSlotMergeBoth = 6,
       kSlotMergeBothAligned = 7, kSlots = 8 };

struct JitState {
    std::mutex mu;
    hipModule_t mod[3 * kSlots] = {};        // (a table has up to three builds of each kernel, see build_for)
    hipFunction_t fn[3 * kSlots] = {};
    dol_status status[3 * kSlots] = {};
    bool tried[3 * kSlots] = {};
    ~JitState()
    {
        for (hipModule_t m : mod)
            if (m) (void)hipModuleUnload(m);
    }
};

void JitDeleter::operator()(JitState *p) const { delete p; }

bool table_code_ok(const dol_fn_table *f)
{
    return f->na >= 4 && f->nb >= 4 && f->n_out >= 4 && f->na <= kJitMaxSym && f->nb <= kJitMaxSym && f->n_out <= kJitMaxOut &&
           f->n_tuples > 0 && f->n_tuples <= kJitMaxTuples && !f->h_col_ptr.empty();
}

bool whole_pieces(const dol_fn_table *f) { return !((f->na | f->nb | f->n_out) & 3); }

namespace {

struct Src {
    std::string s;
    void operator()(const char *fmt, ...) __attribute__((format(printf, 2, 3)))
    {
        char buf[768];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        s += buf;
    }
};

// Wavefronts per workgroup and samples per tile of the source being written.
thread_local int t_waves = kJitWavesLarge, t_tile_rows = kJitTile;
#define kJitWaves t_waves
#define kThreads (kJitTile * t_waves)

// Floats from one sample's row to the next in LDS: an odd number of 16-byte pieces where it is whole pieces, which are then
// read and written by their lanes as such (an even number puts lanes on one another's banks: 60 x 60 -> 64 both ways in one launch with
// rows 16 pieces apart 22.4 us at B = 8 192, 15 apart 16.3); any other row has its own length, so that the tile is the block of memory it came
// from (and an odd length keeps the lanes' words off one another's banks).
int pitch_of(int n) { return n & 3 || n & 4 ? n : n + 4; }

// Declares r0 .. r{n-1} and fills them from the lane's row of the staged tile.
void emit_row_to_regs(Src &o, const char *r, const char *tile, int n)
{
    if (n & 3) {
        for (int i = 0; i < n; ++i) o("  const float %s%d = %s[lane * %d + %d];\n", r, i, tile, n, i);
        return;
    }
    for (int i = 0; i < n; i += 4)
        o("  float %s%d, %s%d, %s%d, %s%d; { const float4 t = *reinterpret_cast<const float4 *>(%s + lane * %d + %d); %s%d = t.x; %s%d = t.y; "
          "%s%d = t.z; %s%d = t.w; }\n", r, i, r, i + 1, r, i + 2, r, i + 3, tile, pitch_of(n), i, r, i, r, i + 1, r, i + 2, r, i + 3);
}

// Flat copy of a tile of `valid` rows of n floats from memory into LDS rows (pitch_of): the loads of all pieces
// of a thread first (into t<tag>_*), the LDS writes in a second step so that several tiles' loads can be in flight.
void emit_stage_load(Src &o, const char *tag, const char *src_ptr, int n)
{
    const int per_thread = (kJitTile * n / 4 + kThreads - 1) / kThreads;
    for (int x = 0; x < per_thread; ++x) o("  float4 ld%s%d;\n", tag, x);
    if (n & 3) {            // (the last tile's words need not be whole pieces: the rest one by one)
        o("  const int whole%s = valid * %d >> 2, rest%s = valid * %d & 3;\n  float one%s = 0.0f;\n", tag, n, tag, n, tag);
        o("  { const float *g1 = %s + s0 * %d; const float4 *g4 = reinterpret_cast<const float4 *>(g1);\n", src_ptr, n);
        for (int x = 0; x < per_thread; ++x) o("    { const int q = tid + %d; ld%s%d = g4[q < whole%s ? q : whole%s - 1]; }\n", kThreads * x, tag, x, tag, tag);
        o("    if (tid < rest%s) one%s = g1[4 * whole%s + tid];\n  }\n", tag, tag, tag);
        return;
    }
    o("  { const float4 *g4 = reinterpret_cast<const float4 *>(%s + s0 * %d);\n", src_ptr, n);
    for (int x = 0; x < per_thread; ++x)
        o("    { const int q = tid + %d; ld%s%d = g4[q < valid * %d ? q : valid * %d - 1]; }\n", kThreads * x, tag, x, n / 4, n / 4);
    o("  }\n");
}

void emit_stage_store(Src &o, const char *tag, const char *dst, int n)
{
    const int per_thread = (kJitTile * n / 4 + kThreads - 1) / kThreads;
    if (n & 3) {
        for (int x = 0; x < per_thread; ++x)
            o("  { const int q = tid + %d; if (q < whole%s) reinterpret_cast<float4 *>(%s)[q] = ld%s%d; }\n", kThreads * x, tag, dst, tag, x);
        o("  if (tid < rest%s) %s[4 * whole%s + tid] = one%s;\n", tag, dst, tag, tag);
        return;
    }
    for (int x = 0; x < per_thread; ++x)
        o("  { const int q = tid + %d; %s{ const int s = q / %d, k = q - s * %d; *reinterpret_cast<float4 *>(%s + s * %d + 4 * k) = ld%s%d; } }\n",
          kThreads * x, kThreads * (x + 1) <= kJitTile * n / 4 ? "" : (std::string("if (q < ") + std::to_string(kJitTile * n / 4) + ") ").c_str(), n / 4, n / 4,
          dst, pitch_of(n), tag, x);
}

// The forward sums of the columns [c0, c1): declares p<c> and leaves the unclamped sum in it.
void emit_columns(Src &o, const dol_fn_table *f, int c0, int c1, const char *indent)
{
    for (int c = c0; c < c1; ++c) {
        o("%sfloat p%d = 0.0f;\n", indent, c);
        for (uint32_t q = f->h_col_ptr[c]; q < f->h_col_ptr[c + 1]; ++q)
            o("%sp%d = __builtin_fmaf(a%u, b%u, p%d);\n", indent, c, f->h_col_ij[q] & 0xffffu, f->h_col_ij[q] >> 16, c);
    }
}

const char *kPrologue =
    "typedef unsigned int u32;\n"
    "typedef float __attribute__((ext_vector_type(4), aligned(4))) float4u;\n"
    "__device__ __forceinline__ void wave_lds_fence() {\n"
    "  __builtin_amdgcn_fence(__ATOMIC_RELEASE, \"wavefront\"); __builtin_amdgcn_wave_barrier(); __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, \"wavefront\"); }\n";

void emit_tile_head(Src &o)
{
    // (one tile per workgroup: inside a loop over tiles the compiler keeps every thread-constant offset of the body alive
    // across it, in registers the body needs)
    o("  {\n  const int tile = blockIdx.x;\n");
    o("  const long long s0 = (long long)tile * %d;\n  const int valid = batch - s0 < %d ? (int)(batch - s0) : %d;\n", t_tile_rows, t_tile_rows, t_tile_rows);
}

// Loads of one group of the gradient reaching the Apply's columns [c0, c1) into registers (th[]), and their way
// into the LDS stage.  merged: column c of the Apply is column ca[c] of the upstream gradient (or dropped).
// (raw: the gradient as it is; the dropped columns, of an aligned plan, are taken out on the way into the stage)
void emit_gh_regs(Src &o)
{
    for (int x = 0; x < (kJitTile * (kJitGroup / 4) + kThreads - 1) / kThreads; ++x) o("  float4 th%d;\n", x);
}

void emit_gh_load(Src &o, int S, int c0, int c1, bool merged, bool aligned, const char *ind, bool raw)
{
    const int chunks = (c1 - c0 + 3) / 4, per_thread = (kJitTile * chunks + kThreads - 1) / kThreads, over = 4 * chunks - (c1 - c0);
    for (int x = 0; x < per_thread; ++x) {
        // (no branches: a conditional block here would invite the compiler to sink the multiply-adds before it past it)
        o("%s{ int q = tid + %d; q = q < valid * %d ? q : valid * %d - 1; const int s = q / %d, k = q - s * %d;\n", ind, kThreads * x, chunks, chunks,
          chunks, chunks);
        if (raw) {
            o("%s  th%d = *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(g + s0 * n3) + (u32)(s * (4 * n3) + (%d + 16 * k))); }\n", ind, x, 4 * c0);
        } else if (merged) {
            o("%s  const int4 oc = reinterpret_cast<const int4 *>(ca)[%d + k]; const float *gr = g + (s0 + s) * n3;\n", ind, c0 / 4);
            if (aligned)    // a kept column of the Apply is the same column of the result: one 16-byte load
                o("%s  const float4 t = *reinterpret_cast<const float4 *>(gr + %d + 4 * k);\n", ind, c0);
            else
                o("%s  const float4 t = make_float4(gr[oc.x > 0 ? oc.x : 0], gr[oc.y > 0 ? oc.y : 0], gr[oc.z > 0 ? oc.z : 0], gr[oc.w > 0 ? oc.w : 0]);\n", ind);
            o("%s  th%d = make_float4(oc.x >= 0 ? t.x : 0.0f, oc.y >= 0 ? t.y : 0.0f, oc.z >= 0 ? t.z : 0.0f, oc.w >= 0 ? t.w : 0.0f); }\n", ind, x);
        } else if (S & 3) {
            // (a row's last piece is the one that ends with the row, moved down in registers)
            o("%s  const float4u t = *reinterpret_cast<const float4u *>(g + (s0 + s) * %d + %d + 4 * k%s);\n", ind, S, c0,
              over ? (" - (k == " + std::to_string(chunks - 1) + " ? " + std::to_string(over) + " : 0)").c_str() : "");
            static const char *const down[4] = {"make_float4(t.x, t.y, t.z, t.w)", "make_float4(t.y, t.z, t.w, 0.0f)", "make_float4(t.z, t.w, 0.0f, 0.0f)",
                                                "make_float4(t.w, 0.0f, 0.0f, 0.0f)"};
            if (over) o("%s  th%d = k == %d ? %s : %s; }\n", ind, x, chunks - 1, down[over], down[0]);
            else o("%s  th%d = %s; }\n", ind, x, down[0]);
        } else {
            o("%s  th%d = reinterpret_cast<const float4 *>(g)[((s0 + s) * %d + %d) / 4 + k]; }\n", ind, x, S, c0);
        }
    }
}

// The group's way from registers into its LDS stage, gated on the way by the words of sm (all ones where no clamp acted).
// raw: where no clamp acted the pieces are c's gradient as well, and leave from here.
void emit_gh_store(Src &o, int c0, int c1, int g, int n_groups, const char *dst, bool masked, const char *ind, bool raw)
{
    const int chunks = (c1 - c0 + 3) / 4, per_thread = (kJitTile * chunks + kThreads - 1) / kThreads;
    for (int x = 0; x < per_thread; ++x) {
        const bool whole = kThreads * (x + 1) <= kJitTile * chunks;
        o("%s{ const int q = tid + %d; %s{ const int s = q / %d, k = q - s * %d;\n", ind, kThreads * x,
          whole ? "" : (std::string("if (q < ") + std::to_string(kJitTile * chunks) + ") ").c_str(), chunks, chunks);
        if (raw) {
            o("%s    if (gc_here && s < valid) { float4 *d4 = reinterpret_cast<float4 *>(reinterpret_cast<char *>(gc + s0 * n3) + (u32)(s * (4 * n3) + (%d + 16 * k))); float4 v = th%d;\n", ind, 4 * c0, x);
            o("%s      if (accumulate & 4) { const float4 old = *d4; v.x += old.x; v.y += old.y; v.z += old.z; v.w += old.w; }\n%s      *d4 = v; }\n", ind, ind);
            o("%s    const u32 kw = s_keep[%d + k];\n", ind, c0 / 4);
            o("%s    th%d = make_float4(kw & 1u ? th%d.x : 0.0f, kw & 2u ? th%d.y : 0.0f, kw & 4u ? th%d.z : 0.0f, kw & 8u ? th%d.w : 0.0f);\n", ind, x, x, x, x, x);
        }
        if (masked) {
            o("%s    const u32 mw = sm[(s * %d + %d) * 2 + (k >> 3)] >> ((4 * k) & 31);\n", ind, n_groups, g);
            o("%s    th%d = make_float4(mw & 1u ? th%d.x : 0.0f, mw & 2u ? th%d.y : 0.0f, mw & 4u ? th%d.z : 0.0f, mw & 8u ? th%d.w : 0.0f);\n", ind, x, x, x, x, x);
        }
        o("%s    *reinterpret_cast<float4 *>(%s + s * %d + 4 * k) = th%d; } }\n", ind, dst, kJitGroup + 4, x);
    }
}

// The next four pieces of c (of an aligned plan: its columns are the result's) of a thread, pieces qb, qb + threads, ..
void emit_union_load(Src &o, const char *qb, const char *ind)
{
    for (int u = 0; u < 4; ++u)
        o("%s{ int q = %s + %d; q = q < total3 ? q : total3 - 1; y%d = *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(c + s0 * n3) + 16u * (u32)q); }\n", ind, qb, kThreads * u, u);
}

// What a source is written for: a kernel of its own, one half of the kernel that runs both passes with the operands' rows kept in
// registers (both_source has its head), or a device function over an LDS array handed in, of the kernel that runs two such.
enum class Form { kernel, half, body };

// Forward.  merged: the kept symbols of the result are merged with a third Distribution c in the same launch
// (out = union(filter(apply2(a, b)), c)); the Apply's own result then lives in LDS only.
std::string forward_source(const dol_fn_table *f, bool merged, bool aligned = false, Form form = Form::kernel, int *lds_floats = nullptr)
{
    const bool both = form == Form::half, body = form == Form::body;
    const int na = f->na, nb = f->nb, S = f->n_out;
    const bool ahead = both && aligned;
    const int pa = pitch_of(na), pb = pitch_of(nb);
    const int fcols = kJitGroup * kJitWavesLarge / kJitWaves;       // columns a wavefront takes at a time: 64, or 32 of eight wavefronts
    const int po = merged ? pitch_of(S) : fcols + 4;         // pitch of the result stage: the whole tile, or a wavefront's columns
    const int in_floats = kJitTile * (pa + pb), out_floats = merged ? kJitTile * po : kJitWaves * kJitTile * po;
    const int stage_floats = std::max(in_floats, out_floats);
    Src o;
    if (form == Form::kernel) o.s = kPrologue;
    if (lds_floats) *lds_floats = stage_floats + kJitTile;
    if (both)
        ;
    else if (body)
        o("static __device__ __forceinline__ void damp_table_merge_fwd_body(float *lds, const float *__restrict__ a, const float *__restrict__ b, "
          "const float *__restrict__ c, float *__restrict__ out, const int *__restrict__ ia, const int *__restrict__ ib, int *saved, "
          "int batch, int n_tiles, int nc, int n3)\n{\n");
    else if (merged)
        o("extern \"C\" __global__ void __launch_bounds__(%d) __attribute__((amdgpu_waves_per_eu(2, 2))) damp_table_merge_fwd_kernel(const float *__restrict__ a, const float *__restrict__ b, "
          "const float *__restrict__ c, float *__restrict__ out, const int *__restrict__ ia, const int *__restrict__ ib, int *__restrict__ saved, "
          "int batch, int n_tiles, int nc, int n3)\n{\n", kThreads);
    else
        o("extern \"C\" __global__ void __launch_bounds__(%d) __attribute__((amdgpu_waves_per_eu(2, 2))) damp_table_fwd_kernel(const float *__restrict__ a, const float *__restrict__ b, "
          "float *__restrict__ out, int batch, int n_tiles)\n{\n", kThreads);
    if (!both) {
        if (!body) o("  __shared__ __align__(16) float lds[%d];\n", stage_floats + (merged ? kJitTile : 0));
        o("  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // (a scalar: branches on it are uniform)\n");
        if (merged) o("  int *sflag = reinterpret_cast<int *>(lds + %d);\n", stage_floats);
        emit_tile_head(o);
        o("  __syncthreads();\n");
    }
    o("  float *sa = lds, *sb = lds + %d, *so = lds + wave * %d;\n", kJitTile * pa, merged ? 0 : kJitTile * po);
    if (merged) o("  if (tid < 64) sflag[tid] = 0;\n");
    emit_stage_load(o, "a", "a", na);
    emit_stage_load(o, "b", "b", nb);
    // What both passes want next, c's first pieces and the gradient's first group, is asked for behind the operands, or, where a
    // wavefront has 64 columns to sum and long rows in its registers, behind the sums.  (Four wavefronts, behind the operands / the sums, us
    // at 40 000 and 131 072 samples: 56 x 56 -> 200 59.0 / 58.0, 140.6 / 136.6, 60 x 60 -> 64 42.3 / 41.1, 94.7 / 92.5, 64 x 56 -> 256 81.0 both,
    // 182.3 / 177.8; shorter rows go either way, 48 x 48 -> 256 54.2 / 55.8, 128.6 / 131.0, 32 x 32 -> 128 29.5 both, 69.4 / 70.3,
    // 48 x 44 -> 160 40.3 / 39.9, 93.8 / 89.5, 64 x 32 -> 400 85.8 / 82.7, 228 / 221.)
    constexpr int kEarlySyms = 96;
    auto ask_ahead = [&](bool now) {
        if (!now) return;
        emit_union_load(o, "tid", "  ");
        emit_gh_load(o, S, 0, std::min(S, kJitGroup), true, true, "  ", true);
    };
    const bool early = kJitWaves > kJitWavesLarge || na + nb <= kEarlySyms;
    if (ahead) {
        o("  const int4 kept4 = reinterpret_cast<const int4 *>(ia)[tid < %d ? tid : %d];\n", S / 4, S / 4 - 1);
        o("  const int chunks3 = n3 >> 2, total3 = valid * chunks3;\n  float4 y0, y1, y2, y3;\n");
        emit_gh_regs(o);
        ask_ahead(early);
    }
    emit_stage_store(o, "a", "sa", na);
    emit_stage_store(o, "b", "sb", nb);
    if (ahead)
        o("  if (tid < %d) s_keep[tid] = (kept4.x >= 0 ? 1u : 0u) | (kept4.y >= 0 ? 2u : 0u) | (kept4.z >= 0 ? 4u : 0u) | (kept4.w >= 0 ? 8u : 0u);\n", S / 4);
    o("  __syncthreads();\n");
    emit_row_to_regs(o, "a", "sa", na);
    emit_row_to_regs(o, "b", "sb", nb);
    o("  __syncthreads();\n");                  // the staged rows are spent: their LDS becomes the result stage
    for (int g = 0; g * fcols < S; ++g) {
        const int c0 = g * fcols, c1 = std::min(S, c0 + fcols);
        o("  if (wave == %d) {\n", g % kJitWaves);
        emit_columns(o, f, c0, c1, "    ");
        auto clamped = [&](int c) { return c < c1 ? "fminf(p" + std::to_string(c) + ", 1.0f)" : std::string("0.0f"); };
        for (int c = c0; c < c1; c += 4)
            o("    *reinterpret_cast<float4 *>(so + lane * %d + %d) = make_float4(%s, %s, %s, %s);\n", po, merged ? c : c - c0, clamped(c).c_str(),
              clamped(c + 1).c_str(), clamped(c + 2).c_str(), clamped(c + 3).c_str());
        if (merged) {
            o("    { bool over = false;\n");
            for (int c = c0; c < c1; ++c) o("      over |= !(p%d <= 1.0f);\n", c);
            o("      if (over) atomicOr(&sflag[lane], 1); }\n");
        } else {
            // the wavefront's own stage: program order within the wavefront is all the ordering it needs
            o("    wave_lds_fence();\n");
            const int chunks = (c1 - c0) / 4, rest = (c1 - c0) & 3;     // 16-byte pieces per sample (S & 3: at any 4-byte boundary)
            if (chunks && (S & 3)) {
                o("    for (int q = lane; q < valid * %d; q += 64) { const int s = q / %d, k = q - s * %d;\n", chunks, chunks, chunks);
                o("      const float4 t = *reinterpret_cast<const float4 *>(so + s * %d + 4 * k); float4u v; v.x = t.x; v.y = t.y; v.z = t.z; v.w = t.w;\n", po);
                o("      *reinterpret_cast<float4u *>(out + (s0 + s) * %d + %d + 4 * k) = v; }\n", S, c0);
            }
            if (rest) {
                o("    for (int q = lane; q < valid * %d; q += 64) { const int s = q / %d, k = q - s * %d;\n", rest, rest, rest);
                o("      out[(s0 + s) * %d + %d + k] = so[s * %d + %d + k]; }\n", S, c0 + 4 * chunks, po, 4 * chunks);
            }
            if (!(S & 3)) o("    for (int q = lane; q < valid * %d; q += 64) { const int s = q / %d, k = q - s * %d;\n", chunks, chunks, chunks);
            if (!(S & 3)) o("      *reinterpret_cast<float4 *>(out + (s0 + s) * %d + %d + 4 * k) = *reinterpret_cast<const float4 *>(so + s * %d + 4 * k); }\n", S, c0, po);
            o("    wave_lds_fence();\n");
        }
        o("  }\n");
    }
    if (ahead) {
        // out[s, c] from the Apply's column c, where it is kept (in LDS), and c's column c: 16-byte pieces of the result tile, four
        // per thread and pass, the next pass's loads on their way
        ask_ahead(!early);
        o("  __syncthreads();\n");
        o("  const int dq = %d / chunks3, dr = %d - dq * chunks3;\n  int ps = tid / chunks3, pk = tid - ps * chunks3;\n", kThreads, kThreads);
        o("  for (int qb = tid; qb < total3; qb += %d) {\n", 4 * kThreads);
        o("    const float4 z0 = y0, z1 = y1, z2 = y2, z3 = y3;\n");
        o("    if (qb + %d < total3) {\n", 4 * kThreads);
        emit_union_load(o, ("qb + " + std::to_string(4 * kThreads)).c_str(), "      ");
        o("    }\n");
        for (int u = 0; u < 4; ++u) {
            o("    { const int pq = qb + %d;\n", kThreads * u);
            o("      if (pq < total3) { const u32 kw = pk < %d ? s_keep[pk] : 0u; float4 x4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);\n", S / 4);
            o("        if (pk < %d) x4 = *reinterpret_cast<const float4 *>(so + ps * %d + 4 * pk);\n", S / 4, po);
            o("        const float xx[4] = {x4.x, x4.y, x4.z, x4.w}, yy[4] = {z%d.x, z%d.y, z%d.z, z%d.w}; float v[4]; bool over = false;\n", u, u, u, u);
            o("        for (int e = 0; e < 4; ++e) { const float t = xx[e] + yy[e]; const bool two = (kw >> e) & 1u; over |= two && !(t <= 1.0f); v[e] = two ? fminf(t, 1.0f) : yy[e]; }\n");
            o("        *reinterpret_cast<float4 *>(reinterpret_cast<char *>(out + s0 * n3) + 16u * (u32)pq) = make_float4(v[0], v[1], v[2], v[3]);\n");
            o("        if (over) atomicOr(&sflag[ps], 1); }\n");
            o("      ps += dq; pk += dr; if (pk >= chunks3) { pk -= chunks3; ++ps; } }\n");
        }
        o("  }\n  __syncthreads();\n  if (saved && tid < valid) saved[s0 + tid] = sflag[tid];\n");
    } else if (merged) {
        // out[s, oc] from the Apply's column ia[oc] (in LDS) and c's column ib[oc]: 16-byte pieces of the result tile, four
        // per thread and pass with their loads in flight together; a piece whose four columns of c are neighbours comes
        // with one 16-byte load
        o("  __syncthreads();\n");
        o("  { const int chunks = n3 >> 2, total = valid * chunks;\n");
        o("    for (int qb = tid; qb < total; qb += %d) {\n", 4 * kThreads);
        for (int u = 0; u < 4; ++u) {
            o("      int pq%d = qb + %d; pq%d = pq%d < total ? pq%d : total - 1; const int ps%d = pq%d / chunks, pk%d = pq%d - ps%d * chunks;\n", u, kThreads * u, u, u, u, u,
              u, u, u, u);
            o("      const int4 ja%d = reinterpret_cast<const int4 *>(ia)[pk%d], jb%d = reinterpret_cast<const int4 *>(ib)[pk%d];\n", u, u, u, u);
        }
        for (int u = 0; u < 4; ++u) {
            o("      float4 y%d; { const float *cr = c + (s0 + ps%d) * nc;\n", u, u);
            if (aligned) {          // the result has c's symbols in c's order: one 16-byte load
                o("        y%d = *reinterpret_cast<const float4 *>(cr + 4 * pk%d); }\n", u, u);
                continue;
            }
            o("        if (jb%d.x >= 0 && !(jb%d.x & 3) && jb%d.y == jb%d.x + 1 && jb%d.z == jb%d.x + 2 && jb%d.w == jb%d.x + 3) y%d = *reinterpret_cast<const float4 *>(cr + jb%d.x);\n",
              u, u, u, u, u, u, u, u, u, u);
            o("        else y%d = make_float4(cr[jb%d.x > 0 ? jb%d.x : 0], cr[jb%d.y > 0 ? jb%d.y : 0], cr[jb%d.z > 0 ? jb%d.z : 0], cr[jb%d.w > 0 ? jb%d.w : 0]); }\n",
              u, u, u, u, u, u, u, u, u);
        }
        for (int u = 0; u < 4; ++u) {
            o("      { const float *xr = so + ps%d * %d; bool over = false; float v[4];\n", u, po);
            o("        const int ja[4] = {ja%d.x, ja%d.y, ja%d.z, ja%d.w}, jb[4] = {jb%d.x, jb%d.y, jb%d.z, jb%d.w}; const float yy[4] = {y%d.x, y%d.y, y%d.z, y%d.w};\n",
              u, u, u, u, u, u, u, u, u, u, u, u);
            if (aligned) {          // a kept column of the Apply sits at its own position in the result
                o("        const float4 x4 = 4 * pk%d < %d ? *reinterpret_cast<const float4 *>(xr + 4 * pk%d) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);\n", u, S, u);
                o("        const float xx[4] = {x4.x, x4.y, x4.z, x4.w};\n");
                o("        for (int e = 0; e < 4; ++e) { const float x = xx[e], t = x + yy[e];\n");
            } else {
                o("        for (int e = 0; e < 4; ++e) { const float x = xr[ja[e] > 0 ? ja[e] : 0], t = x + yy[e];\n");
            }
            o("          if (ja[e] >= 0 && jb[e] >= 0) { over |= !(t <= 1.0f); v[e] = fminf(t, 1.0f); } else v[e] = ja[e] >= 0 ? x : yy[e]; }\n");
            o("        if (qb + %d < total) { *reinterpret_cast<float4 *>(out + (s0 + ps%d) * n3 + 4 * pk%d) = make_float4(v[0], v[1], v[2], v[3]);\n", kThreads * u, u, u);
            o("          if (over) atomicOr(&sflag[ps%d], 1); } }\n", u);
        }
        o("    } }\n");
        o("  __syncthreads();\n  if (saved && tid < valid) saved[s0 + tid] = sflag[tid];\n");
    }
    if (!both) o("  }\n}\n");
    return o.s;
}

// Most tuples of one column that share a symbol of the second (by_b) or first operand.
int max_multiplicity(const dol_fn_table *f, bool by_b)
{
    int best = 1;
    std::vector<int> cnt(static_cast<size_t>(by_b ? f->nb : f->na));
    for (int c = 0; c < f->n_out; ++c) {
        std::fill(cnt.begin(), cnt.end(), 0);
        for (uint32_t q = f->h_col_ptr[c]; q < f->h_col_ptr[c + 1]; ++q) {
            const uint32_t x = by_b ? f->h_col_ij[q] >> 16 : f->h_col_ij[q] & 0xffffu;
            best = std::max(best, ++cnt[x]);
        }
    }
    return best;
}

// (as a half: the operands' rows are in registers, sflag says which samples a clamp acted in, and of an aligned plan th<x> holds the
// first group)
std::string backward_source(const dol_fn_table *f, bool merged, bool aligned = false, Form form = Form::kernel, int *lds_floats = nullptr)
{
    const bool both = form == Form::half, body = form == Form::body;
    const bool ahead = both && aligned;
    const int na = f->na, nb = f->nb, S = f->n_out;
    const int pa = pitch_of(na), pb = pitch_of(nb), pg = kJitGroup + 4;
    const int n_groups = (S + kJitGroup - 1) / kJitGroup;
    // LDS: a tile, b tile, two stages for one group of gh each (the first re-used as the result stage), gate words
    const int off_b = kJitTile * pa, off_g = both ? 0 : off_b + kJitTile * pb;
    const int stage = std::max(kJitTile * pg, kJitTile * std::max(pa, pb));
    const int off_m = off_g + 2 * stage, off_u = off_m + kJitTile * n_groups * 2;
    const int off_x = off_u + (merged ? kJitTile * n_groups * 2 : 0), off_f = off_x + (merged ? 2 * S : 0);
    // the first half of the wavefronts share out the rows of a (they keep b), the second half those of b: two or four
    // parts each, multiples of four rows
    const int parts = kJitWaves / 2;
    const int ha = std::min(na, std::max(4, (na / parts + 3) & ~3)), hb = std::min(nb, std::max(4, (nb / parts + 3) & ~3));
    Src o;
    if (form == Form::kernel) o.s = kPrologue;
    if (lds_floats) *lds_floats = off_f + 4;
    if (both)
        ;
    else if (body)
        o("static __device__ __forceinline__ void damp_table_merge_bwd_body(float *lds, const float *__restrict__ a, const float *__restrict__ b, "
          "const float *__restrict__ c, const float *__restrict__ g, float *__restrict__ ga, float *__restrict__ gb, float *__restrict__ gc, "
          "const int *__restrict__ ia, const int *__restrict__ ib, const int *__restrict__ ca, const int *__restrict__ cb, "
          "const int *saved, int batch, int n_tiles, int nc, int n3, int accumulate)\n{\n");
    else if (merged)
        o("extern \"C\" __global__ void __launch_bounds__(%d) __attribute__((amdgpu_waves_per_eu(2, 2))) damp_table_merge_bwd_kernel(const float *__restrict__ a, const float *__restrict__ b, "
          "const float *__restrict__ c, const float *__restrict__ g, float *__restrict__ ga, float *__restrict__ gb, float *__restrict__ gc, "
          "const int *__restrict__ ia, const int *__restrict__ ib, const int *__restrict__ ca, const int *__restrict__ cb, "
          "const int *__restrict__ saved, int batch, int n_tiles, int nc, int n3, int accumulate)\n{\n", kThreads);
    else
        o("extern \"C\" __global__ void __launch_bounds__(%d) __attribute__((amdgpu_waves_per_eu(2, 2))) damp_table_bwd_kernel(const float *__restrict__ a, const float *__restrict__ b, "
          "const float *__restrict__ g, float *__restrict__ ga, float *__restrict__ gb, int batch, int n_tiles, int accumulate)\n{\n", kThreads);
    if (!both) {
        if (!body) o("  __shared__ __align__(16) float lds[%d];\n", off_f + 4);
        o("  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // (a scalar: branches on it are uniform)\n");
        o("  float *sa = lds, *sb = lds + %d;\n  int *flag = reinterpret_cast<int *>(lds + %d);\n", off_b, off_f);
    }
    o("  float *sg0 = lds + %d, *sg1 = lds + %d;\n  u32 *sm = reinterpret_cast<u32 *>(lds + %d);\n", off_g, off_g + stage, off_m);
    if (merged) {
        // where each column of the Apply lands in the result (-1: dropped), and which column of c it meets there (-1: none)
        o("  u32 *su = reinterpret_cast<u32 *>(lds + %d);\n  int *s_oc = reinterpret_cast<int *>(lds + %d), *s_jc = s_oc + %d;\n", off_u, off_x, S);
    }
    if (!both) {
        emit_tile_head(o);
        o("  __syncthreads();\n  if (tid == 0) *flag = 0;\n");
        emit_stage_load(o, "a", "a", na);
        emit_stage_load(o, "b", "b", nb);
    }
    if (!ahead) {
        emit_gh_regs(o);
        emit_gh_load(o, S, 0, std::min(S, kJitGroup), merged, aligned, "  ", false);
    }
    if (both) {
        // (the same in every wavefront)
        o("  const bool gate = __ballot(lane < valid && sflag[lane] != 0) != 0;\n");
        if (ahead) o("  const bool gc_here = gc && !gate;\n");
    } else {
        if (merged) o("  int was_clamped = 1; if (saved) was_clamped = lane < valid ? saved[s0 + lane] : 0;\n");
        emit_stage_store(o, "a", "sa", na);
        emit_stage_store(o, "b", "sb", nb);
    }
    emit_gh_store(o, 0, std::min(S, kJitGroup), 0, n_groups, "sg0", false, "  ", ahead);
    if (!both) {
        o("  __syncthreads();\n");
        emit_row_to_regs(o, "a", "sa", na);
        emit_row_to_regs(o, "b", "sb", nb);
    }
    if (both) {
    } else if (merged) {
        // the forward launch left word: did any clamp act in this sample?
        o("  if (was_clamped && lane < valid) *flag = 1;\n");
    } else {
        // can any column of this lane's sample exceed 1?
        o("  { float ma = a0, mb = b0, ta = a0, tb = b0;\n");
        for (int i = 1; i < na; ++i) o("    ma = fmaxf(ma, a%d); ta += a%d;\n", i, i);
        for (int j = 1; j < nb; ++j) o("    mb = fmaxf(mb, b%d); tb += b%d;\n", j, j);
        o("    const float bound = fminf(ma * tb * %d.0f, mb * ta * %d.0f);\n", max_multiplicity(f, true), max_multiplicity(f, false));
        o("    if (lane < valid && !(bound <= 0.9999f)) *flag = 1; }\n");
    }
    if (!both) o("  __syncthreads();\n  const bool gate = *flag != 0;\n");
    // rare: recompute pre, one group of columns per wavefront, and leave one bit per (sample, column)
    o("  if (gate) {\n");
    if (merged) o("    for (int x = tid; x < %d; x += %d) { const int oc = ca[x]; s_oc[x] = oc; s_jc[x] = oc >= 0 ? ib[oc] : -1; }\n    __syncthreads();\n", S, kThreads);
    if (merged) o("    const long long sr = s0 + (lane < valid ? lane : 0);\n");
    for (int g = 0; g < n_groups; ++g) {
        const int c0 = g * kJitGroup, c1 = std::min(S, c0 + kJitGroup);
        o("    if (wave == %d) {\n", g % kJitWaves);
        o("      u32 m0 = 0, m1 = 0;\n");
        if (merged) o("      u32 u0 = 0, u1 = 0;\n");
        for (int d0 = c0; d0 < c1; d0 += 16) {
            const int d1 = std::min(c1, d0 + 16);
            o("      {\n");
            emit_columns(o, f, d0, d1, "        ");
            for (int c = d0; c < d1; ++c) {
                if (merged) {
                    o("        { const int oc = s_oc[%d], jc = s_jc[%d];\n", c, c);
                    o("          bool open = true; if (jc >= 0) open = fminf(p%d, 1.0f) + c[sr * nc + jc] <= 1.0f;\n", c);
                    o("          if (open) u%d |= %uu; if (open && oc >= 0 && p%d <= 1.0f) m%d |= %uu; }\n", (c - c0) / 32, 1u << ((c - c0) & 31), c,
                      (c - c0) / 32, 1u << ((c - c0) & 31));
                } else {
                    o("        m%d |= p%d <= 1.0f ? %uu : 0u;\n", (c - c0) / 32, c, 1u << ((c - c0) & 31));
                }
            }
            o("      }\n      __builtin_amdgcn_sched_barrier(0);\n");
        }
        if (merged) o("      su[(lane * %d + %d) * 2] = u0; su[(lane * %d + %d) * 2 + 1] = u1;\n", n_groups, g, n_groups, g);
        o("      sm[(lane * %d + %d) * 2] = m0; sm[(lane * %d + %d) * 2 + 1] = m1;\n    }\n", n_groups, g, n_groups, g);
    }
    o("    __syncthreads();\n");
    {   // the first group is already staged: gate it in place
        const int c1 = std::min(S, kJitGroup), chunks = (c1 + 3) / 4;
        o("    for (int q = tid; q < %d; q += %d) { const int s = q / %d, k = q - s * %d;\n", kJitTile * chunks, kThreads, chunks, chunks);
        o("      const u32 mw = sm[(s * %d) * 2 + (k >> 3)] >> ((4 * k) & 31); float4 *p4 = reinterpret_cast<float4 *>(sg0 + s * %d + 4 * k);\n", n_groups, pg);
        o("      const float4 t = *p4; *p4 = make_float4(mw & 1u ? t.x : 0.0f, mw & 2u ? t.y : 0.0f, mw & 4u ? t.z : 0.0f, mw & 8u ? t.w : 0.0f); }\n");
    }
    o("  } else {\n    for (int x = tid; x < %d; x += %d) sm[x] = 0xffffffffu;\n  }\n  __syncthreads();\n", kJitTile * n_groups * 2, kThreads);
    // The four roles.  Every role runs the same sequence of workgroup barriers and takes part in the same flat
    // copies; only the multiply-adds differ.  While a group's multiply-adds run, the next group's loads are in flight.
    for (int w = 0; w < kJitWaves; ++w) {
        const bool is_a = w < parts;
        const int n = is_a ? na : nb, h = is_a ? ha : hb, part = w % parts;
        const int r0 = std::min(n, part * h), r1 = part + 1 == parts ? n : std::min(n, (part + 1) * h);
        const char *acc = is_a ? "x" : "y";
        o("  %sif (wave == %d) {\n", w ? "else " : "", w);
        for (int r = r0; r < r1; ++r) o("    float %s%d = 0.0f;\n", acc, r);
        for (int g = 0; g < n_groups; ++g) {
            const int c0 = g * kJitGroup, c1 = std::min(S, c0 + kJitGroup);
            const char *cur = g & 1 ? "sg1" : "sg0", *nxt = g & 1 ? "sg0" : "sg1";
            if (g + 1 < n_groups) emit_gh_load(o, S, c1, std::min(S, c1 + kJitGroup), merged, aligned, "    ", ahead);
            // 16 columns at a time, fenced for the instruction scheduler: it would otherwise fetch the whole group first and
            // run out of registers
            o("    {\n");
            for (int d0 = c0; d0 < c1; d0 += 16) {
                const int d1 = std::min(c1, d0 + 16);
                o("    {\n");
                for (int c = d0; c < d1; c += 4)
                    o("      float h%d, h%d, h%d, h%d; { const float4 t = *reinterpret_cast<const float4 *>(%s + lane * %d + %d); h%d = t.x; h%d = t.y; h%d = t.z; h%d = t.w; }\n",
                      c, c + 1, c + 2, c + 3, cur, pg, c - c0, c, c + 1, c + 2, c + 3);
                // the tuples of these columns whose row belongs to this role
                for (int c = d0; c < d1; ++c)
                    for (uint32_t q = f->h_col_ptr[c]; q < f->h_col_ptr[c + 1]; ++q) {
                        const int i = static_cast<int>(f->h_col_ij[q] & 0xffffu), j = static_cast<int>(f->h_col_ij[q] >> 16);
                        const int r = is_a ? i : j;
                        if (r < r0 || r >= r1) continue;
                        if (is_a) o("      x%d = __builtin_fmaf(h%d, b%d, x%d);\n", i, c, j, i);
                        else o("      y%d = __builtin_fmaf(h%d, a%d, y%d);\n", j, c, i, j);
                    }
                o("    }\n    __builtin_amdgcn_sched_barrier(0);\n");
            }
            o("    }\n");
            if (g + 1 < n_groups) emit_gh_store(o, c1, std::min(S, c1 + kJitGroup), g + 1, n_groups, nxt, true, "    ", ahead);
            o("    __syncthreads();\n");
        }
        // results: through LDS (a's in the first stage, b's in the second)
        const char *dst = is_a ? "sg0" : "sg1";
        const int pp = pitch_of(n);
        if (n & 3)
            for (int r = r0; r < r1; ++r) o("    %s[lane * %d + %d] = %s%d;\n", dst, pp, r, acc, r);
        else
            for (int r = r0; r < r1; r += 4)
                o("    *reinterpret_cast<float4 *>(%s + lane * %d + %d) = make_float4(%s%d, %s%d, %s%d, %s%d);\n", dst, pp, r, acc, r, acc, r + 1, acc, r + 2, acc,
                  r + 3);
        o("  }\n");
    }
    // .. out with flat 16-byte accesses
    o("  __syncthreads();\n");
    for (int pass = 0; pass < 2; ++pass) {
        const char *src = pass ? "sg1" : "sg0", *to = pass ? "gb" : "ga";
        const int pn = pass ? nb : na, pp = pitch_of(pn), bit = pass ? 2 : 1;
        o("  if (%s) { float4 *d4 = reinterpret_cast<float4 *>(%s + s0 * %d);\n", to, to, pn);
        if (pn & 3) {
            o("    const int whole = valid * %d >> 2, rest = valid * %d & 3;\n", pn, pn);
            o("    for (int q = tid; q < whole; q += %d) { float4 v = reinterpret_cast<const float4 *>(%s)[q];\n", kThreads, src);
            o("      if (accumulate & %d) { const float4 old = d4[q]; v.x += old.x; v.y += old.y; v.z += old.z; v.w += old.w; }\n      d4[q] = v; }\n", bit);
            o("    if (tid < rest) { float *d1 = reinterpret_cast<float *>(d4 + whole) + tid; const float v = %s[4 * whole + tid]; *d1 = accumulate & %d ? v + *d1 : v; } }\n",
              src, bit);
            continue;
        }
        o("    for (int q = tid; q < valid * %d; q += %d) { const int s = q / %d, k = q - s * %d;\n", pn / 4, kThreads, pn / 4, pn / 4);
        o("      float4 v = *reinterpret_cast<const float4 *>(%s + s * %d + 4 * k);\n", src, pp);
        o("      if (accumulate & %d) { const float4 old = d4[q]; v.x += old.x; v.y += old.y; v.z += old.z; v.w += old.w; }\n", bit);
        o("      d4[q] = v; } }\n");
    }
    if (merged) {
        // gradient of c: column jc of c is column cb[jc] of the result; a symbol of both sides is gated by the union's clamp.
        // 16-byte pieces, four per thread and pass, one 16-byte load where the four columns are neighbours in the result.
        // (ahead: where no clamp acted the columns that the Apply has are written)
        o("  if (gc) { const int from = %s, chunks = (nc >> 2) - from, total = valid * chunks;\n", ahead ? ("gc_here ? " + std::to_string(S / 4) + " : 0").c_str() : "0");
        o("    for (int qb = tid; qb < total; qb += %d) {\n", 4 * kThreads);
        for (int u = 0; u < 4; ++u) {
            o("      int pq%d = qb + %d; pq%d = pq%d < total ? pq%d : total - 1; const int ps%d = pq%d / chunks, pk%d = pq%d - ps%d * chunks + from;\n", u, kThreads * u, u, u, u, u,
              u, u, u, u);
            o("      const int4 oc%d = reinterpret_cast<const int4 *>(cb)[pk%d];\n", u, u);
        }
        for (int u = 0; u < 4; ++u) {
            o("      float4 v%d; { const float *gr = g + (s0 + ps%d) * n3;\n", u, u);
            o("        if (!(oc%d.x & 3) && oc%d.y == oc%d.x + 1 && oc%d.z == oc%d.x + 2 && oc%d.w == oc%d.x + 3) v%d = *reinterpret_cast<const float4 *>(gr + oc%d.x);\n",
              u, u, u, u, u, u, u, u, u);
            o("        else v%d = make_float4(gr[oc%d.x], gr[oc%d.y], gr[oc%d.z], gr[oc%d.w]); }\n", u, u, u, u, u);
        }
        for (int u = 0; u < 4; ++u) {
            o("      if (qb + %d < total) {\n", kThreads * u);
            o("        if (gate) { const int oc[4] = {oc%d.x, oc%d.y, oc%d.z, oc%d.w}; float w[4] = {v%d.x, v%d.y, v%d.z, v%d.w};\n", u, u, u, u, u, u, u, u);
            o("          for (int e = 0; e < 4; ++e) { const int col = ia[oc[e]];\n");
            o("            if (col >= 0 && !((su[(ps%d * %d + (col >> 6)) * 2 + ((col >> 5) & 1)] >> (col & 31)) & 1u)) w[e] = 0.0f; }\n", u, n_groups);
            o("          v%d = make_float4(w[0], w[1], w[2], w[3]); }\n", u);
            o("        float4 *d4 = reinterpret_cast<float4 *>(gc + (s0 + ps%d) * nc) + pk%d;\n", u, u);
            o("        if (accumulate & 4) { const float4 old = *d4; v%d.x += old.x; v%d.y += old.y; v%d.z += old.z; v%d.w += old.w; }\n        *d4 = v%d; }\n", u, u, u, u, u);
        }
        o("    } }\n");
    }
    o("  }\n}\n");
    return o.s;
}

// Whether the result's tile leaves room for one workgroup to a unit only.
bool wide_result(const dol_fn_table *f) { return 4 * kJitTile * pitch_of(f->n_out) > 80 * 1024; }

// Whether the kernel that runs both passes keeps the operands' rows in registers from one to the other, and the clamp words in LDS.
// Long rows are staged again, by two bodies, where registers are short: beside the Union of a plan that is not aligned, which takes
// most of a wavefront's by itself (64 x 64 -> 256 and 256 symbols, 192 of them the same, kept / so, us at B = 32 000 41.8 / 40.6, at 6 000
// 25.7 / 24.1), and in the four wavefronts of a tile, where two tiles share a unit (64 x 64 -> 256 aligned, at 32 000 and 131 072
// 45.9 / 42.9 and 208 / 170, eight wavefronts and rows kept 48.0 and 185; 64 x 64 -> 64 at 32 000 29.4 / 27.0).
constexpr int kKeptSyms = 120;
bool keeps_rows(const dol_fn_table *f, bool aligned, int waves)
{
    return f->na + f->nb <= kKeptSyms || (aligned && (waves > kJitWavesLarge || wide_result(f)));
}

// Apply + Filter + Union forward and backward in one launch.  (As bodies the second reads the clamp words that the first has just written,
// other threads' words: the workgroup's barrier between the two orders them.)
std::string both_source(const dol_fn_table *f, bool aligned)
{
    const bool kept = keeps_rows(f, aligned, kJitWaves);
    const Form form = kept ? Form::half : Form::body;
    int lf = 0, lb = 0;
    const std::string fwd = forward_source(f, true, aligned, form, &lf), bwd = backward_source(f, true, aligned, form, &lb);
    Src o;
    o.s = kPrologue;
    if (!kept) o.s += fwd + bwd;
    o("extern \"C\" __global__ void __launch_bounds__(%d) __attribute__((amdgpu_waves_per_eu(2, 2))) damp_table_merge_fwd_bwd_kernel("
      "const float *__restrict__ a, const float *__restrict__ b, const float *__restrict__ c, float *__restrict__ out, "
      "const float *__restrict__ g, float *__restrict__ ga, float *__restrict__ gb, float *__restrict__ gc, const int *__restrict__ ia, "
      "const int *__restrict__ ib, const int *__restrict__ ca, const int *__restrict__ cb, int *saved, int batch, int n_tiles, int nc, int n3, "
      "int accumulate)\n{\n", kThreads);
    const int floats = std::max(lf, lb);
    o("  __shared__ __align__(16) float lds[%d];\n", floats + (kept ? kJitTile + f->n_out / 4 : 0));
    if (!kept) {
        o("  damp_table_merge_fwd_body(lds, a, b, c, out, ia, ib, saved, batch, n_tiles, nc, n3);\n  __syncthreads();\n");
        o("  damp_table_merge_bwd_body(lds, a, b, c, g, ga, gb, gc, ia, ib, ca, cb, saved, batch, n_tiles, nc, n3, accumulate);\n}\n");
        return o.s;
    }
    o("  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // (a scalar: branches on it are uniform)\n");
    o("  int *sflag = reinterpret_cast<int *>(lds + %d);\n", floats);
    if (aligned) o("  u32 *s_keep = reinterpret_cast<u32 *>(lds + %d);\n", floats + kJitTile);
    emit_tile_head(o);
    o.s += fwd + bwd;
    return o.s;
}

}  // namespace

dol_status jit_compile(const std::string &src, const char *name, hipModule_t *mod, hipFunction_t *fn)
{
    // DOL_JIT_DUMP_DIR names a folder that receives the source of every kernel generated in this process, so that
    // the code written for a table or a chain can be read and compiled by hand.
    if (const char *dump = getenv("DOL_JIT_DUMP_DIR")) {
        const std::string path = std::string(dump) + "/" + name + ".hip";
        if (FILE *fh = fopen(path.c_str(), "w")) { fputs(src.c_str(), fh); fclose(fh); }
    }
    hiprtcProgram prog = nullptr;
    if (hiprtcCreateProgram(&prog, src.c_str(), "dol_table.hip", 0, nullptr, nullptr) != HIPRTC_SUCCESS)
        return fail(DOL_EHIP, "hiprtcCreateProgram failed");
    const char *opts[] = {"--offload-arch=gfx950", "-O3", "-ffp-contract=off", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"};
    const hiprtcResult rc = hiprtcCompileProgram(prog, static_cast<int>(sizeof opts / sizeof *opts), opts);
    if (rc != HIPRTC_SUCCESS) {
        size_t n = 0;
        std::string log;
        if (hiprtcGetProgramLogSize(prog, &n) == HIPRTC_SUCCESS && n > 1) {
            log.resize(n);
            (void)hiprtcGetProgramLog(prog, &log[0]);
        }
        (void)hiprtcDestroyProgram(&prog);
        return fail(DOL_EHIP, "compiling the table's code failed (%s): %.300s", hiprtcGetErrorString(rc), log.c_str());
    }
    size_t size = 0;
    std::vector<char> code;
    if (hiprtcGetCodeSize(prog, &size) != HIPRTC_SUCCESS || size == 0) {
        (void)hiprtcDestroyProgram(&prog);
        return fail(DOL_EHIP, "hiprtcGetCodeSize failed");
    }
    code.resize(size);
    const hiprtcResult rc2 = hiprtcGetCode(prog, code.data());
    (void)hiprtcDestroyProgram(&prog);
    if (rc2 != HIPRTC_SUCCESS) return fail(DOL_EHIP, "hiprtcGetCode failed");
    DOL_HIP(hipModuleLoadData(mod, code.data()));
    DOL_HIP(hipModuleGetFunction(fn, *mod, name));
    return DOL_OK;
}

namespace {

unsigned tile_grid(int n_tiles) { return static_cast<unsigned>(n_tiles); }

// How a batch is cut up.  The registers of these kernels allow two wavefronts on a SIMD, and the chip has 256 compute
// units.  With tiles of 64 samples and four wavefronts to a tile, a batch of up to 256 tiles leaves every unit with one
// wavefront per SIMD and the tile's loads, arithmetic and stores one after the other.  Such a batch gets a build of its
// own, of eight wavefronts, which share the tile's columns (rows, in the reverse pass) out finer, and one of up to 128 tiles may
// be cut into tiles of 32 samples instead: half of the lanes idle, but all units at work.
struct JitBuild {
    int rows, waves;        // samples per tile, wavefronts per workgroup
    int variant;            // which of the table's builds
};
constexpr JitBuild kFourWaves = {kJitTile, kJitWavesLarge, 0}, kEightWaves = {kJitTile, 2 * kJitWavesLarge, 1},
                   kHalfTiles = {kJitTile / 2, kJitWavesLarge, 2};

// Tiles of 32 samples or eight wavefronts, up to 8 192 samples (us at 6 000, eight / tiles of 32).  By tuples an output symbol has:
// the more, the longer a wavefront's arithmetic, which eight of them halve.
//   Apply forward: eight, but for the smallest tables.  32 x 40 -> 128 4.2 / 4.7, 24 x 24 -> 100 3.7 / 4.1, 16 x 64 -> 400 5.5 / 5.8,
//     64 x 64 -> 64 7.0 / 10.2; 20 x 20 -> 20 3.6 / 3.5, 16 x 16 -> 32 3.5 / 3.3.
//   Apply backward: each wavefront reads the gradient that its rows need from LDS.  With many tuples to a symbol the arithmetic hides
//     that, with few most of it is not needed: eight, 64 x 64 -> 256 (16) 9.4 / 10.4, 63 x 61 -> 216 8.8 / 10.4, 60 x 60 -> 64 6.6 / 7.6;
//     36 x 36 -> 300 (4.3) 7.3 / 7.9, 64 x 32 -> 1 000 13.8 / 15.6.  In between tiles of 32: 32 x 40 -> 128 (10) 6.1 / 5.9,
//     64 x 32 -> 256 8.3 / 8.0, 32 x 16 -> 64 4.3 / 4.1, 48 x 48 -> 512 (4.5) 12.3 / 10.4.
//   Apply + Filter + Union, which stages the union's operand and result besides, and moves more bytes to a tuple: forward
//     36 x 36 -> 300 11.2 / 10.1, 56 x 56 -> 200 (15.7) 10.4 / 9.7, 64 x 64 -> 256 9.7 / 9.5; 40 x 64 -> 64 (40) 8.1 / 9.6,
//     60 x 60 -> 64 9.4 / 11.6; up to 128 symbols, two of four wavefronts' columns, 32 x 40 -> 128 6.2 / 6.5 where the plan is
//     aligned, 6.9 / 6.8 where not.  Backward 16 x 64 -> 400 16.8 / 15.4, 56 x 56 -> 200 12.3 / 11.8, 60 x 60 -> 64 8.3 / 8.9.
JitBuild build_for(const dol_fn_table *f, int kind, int32_t batch)
{
    if (batch > 256 * kJitTile) return kFourWaves;
    if (batch > 128 * kJitTile) return kEightWaves;
    const int64_t tuples = f->n_tuples, symbols = f->n_out;
    if (kind == kSlotFwd) return tuples <= 400 ? kHalfTiles : kEightWaves;
    if (kind == kSlotBwd) return 10 * tuples >= 44 * symbols && tuples <= 12 * symbols ? kHalfTiles : kEightWaves;
    return tuples >= (kind == kSlotMergeFwdAligned && symbols <= 128 ? 10 : 20) * symbols ? kEightWaves : kHalfTiles;
}

// Both passes in one launch, us.  Of a plan that is not aligned as above (at 6 000, eight / tiles of 32: 48 x 48 -> 512 38.4 / 33.4,
// 64 x 64 -> 256 24.1 / 22.7, 32 x 40 -> 128 13.3 / 12.2; 60 x 60 -> 64 15.7 / 18.4).  Of an aligned one eight up to 16 384 samples: what
// both passes want is on its way at once, and tiles of 32 would ask for half as much (64 x 64 -> 256 20.2 / 27.9, 32 x 40 -> 128 9.8 /
// 10.0, 24 x 24 -> 100 8.7 / 8.0).  But eight wavefronts have 256 registers each also where LDS has room for one workgroup only
// and four have 512: with a wide result (48 x 48 -> 512, at 6 000 36.9 / 23.7, and at 16 384, eight / four 42.5 / 32.2) the rows of both
// operands and the pieces on their way are too much for 256, up to 229 of them spilled; shorter rows are not (16 x 64 -> 400,
// at 16 384 28.8 / 25.3, where clamps act 60.7 / 71.3).
// Above 16 384 samples two tiles of four wavefronts share a unit.  Long rows, which are staged again there (keeps_rows), keep eight
// wavefronts while few units get a second tile, us with eight / four, and where clamps act: 64 x 64 -> 256 at 17 000 35.7 / 39.8 and 61.6 / 71.3,
// at 20 000 37.7 / 40.6 and 64.3 / 75.1, 22 000 40.1 / 41.0 and 70.3 / 75.9, 24 000 41.4 / 41.7 and 85.0 / 76.9, 30 000 45.5 / 44.4 and 91.4 / 79.6.
// Not with many tuples to a symbol: 64 x 60 -> 64 (60) at 20 000 27.0 / 31.4, but 63.0 / 50.5.
constexpr int kShortRows = 88;
JitBuild build_for_both(const dol_fn_table *f, bool aligned, int32_t batch)
{
    const JitBuild b = build_for(f, aligned ? kSlotMergeBothAligned : kSlotMergeBoth, batch);
    if (!aligned) return b;
    if (batch > 256 * kJitTile) {
        const bool few_second = batch <= 352 * kJitTile && static_cast<int64_t>(f->n_tuples) <= 20 * static_cast<int64_t>(f->n_out);
        return few_second && f->na + f->nb > kKeptSyms && !wide_result(f) ? kEightWaves : b;
    }
    if (!wide_result(f)) return kEightWaves;
    return batch <= 128 * kJitTile ? kHalfTiles : f->na + f->nb <= kShortRows ? kEightWaves : kFourWaves;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

JitState *state_of(const dol_fn_table *f)
{
    static std::mutex mu;
    std::lock_guard<std::mutex> lock(mu);
    if (!f->jit) f->jit.reset(new JitState);
    return f->jit.get();
}

}  // namespace

// The kernel of `slot` for this table, built on first use.
static dol_status kernel_of(const dol_fn_table *f, int kind, const JitBuild &bd, hipFunction_t *fn)
{
    const int slot = kind + bd.variant * kSlots;
    static const char *const names[kSlots] = {"damp_table_fwd_kernel", "damp_table_bwd_kernel", "damp_table_merge_fwd_kernel",
                                              "damp_table_merge_bwd_kernel", "damp_table_merge_fwd_kernel", "damp_table_merge_bwd_kernel",
                                              "damp_table_merge_fwd_bwd_kernel", "damp_table_merge_fwd_bwd_kernel"};
    JitState *js = state_of(f);
    std::lock_guard<std::mutex> lock(js->mu);
    if (!js->tried[slot]) {
        js->tried[slot] = true;
        t_tile_rows = bd.rows, t_waves = bd.waves;
        const std::string src = kind == kSlotFwd ? forward_source(f, false) : kind == kSlotBwd ? backward_source(f, false) :
                                kind == kSlotMergeFwd ? forward_source(f, true) : kind == kSlotMergeBwd ? backward_source(f, true) :
                                kind == kSlotMergeFwdAligned ? forward_source(f, true, true) :
                                kind == kSlotMergeBwdAligned ? backward_source(f, true, true) : both_source(f, kind == kSlotMergeBothAligned);
        t_tile_rows = kJitTile, t_waves = kJitWavesLarge;
        js->status[slot] = jit_compile(src, names[kind], &js->mod[slot], &js->fn[slot]);
        if (js->status[slot] != DOL_OK) return js->status[slot];      // with the compiler's message
    } else if (js->status[slot] != DOL_OK) {
        return fail(js->status[slot], "the code of this function table did not build (see the first call's message)");
    }
    *fn = js->fn[slot];
    return DOL_OK;
}

// *done = the call was taken (otherwise the caller uses the generic kernels).
dol_status launch_damp_table_fwd(const dol_fn_table *f, int32_t batch, const float *a, int64_t lda, const float *b,
                                 int64_t ldb, float *out, int64_t ldo, hipStream_t st, bool *done)
{
    *done = false;
    if (!table_code_ok(f) || batch < 1 || table_small_batch(f, batch, false)) return DOL_OK;
    if (lda != f->na || ldb != f->nb || ldo != f->n_out || !aligned16(a) || !aligned16(b) || !aligned16(out)) return DOL_OK;
    hipFunction_t fn = nullptr;
    const JitBuild bd = build_for(f, kSlotFwd, batch);
    if (dol_status s = kernel_of(f, kSlotFwd, bd, &fn)) return whole_pieces(f) ? s : DOL_OK;      // (the others have kernels that need no compiler)
    int n_tiles = (batch + bd.rows - 1) / bd.rows;
    void *args[] = {&a, &b, &out, &batch, &n_tiles};
    DOL_HIP(hipModuleLaunchKernel(fn, tile_grid(n_tiles), 1, 1, kJitTile * bd.waves, 1, 1, 0, st, args, nullptr));
    *done = true;
    return DOL_OK;
}

dol_status launch_damp_table_bwd(const dol_fn_table *f, int32_t batch, const float *a, int64_t lda, const float *b,
                                 int64_t ldb, const float *g, int64_t ldg, float *ga, float *gb, int32_t accumulate,
                                 hipStream_t st, bool *done)
{
    *done = false;
    if (!table_code_ok(f) || batch < 1 || (ga && ga == gb) || table_small_batch(f, batch, true)) return DOL_OK;
    if (lda != f->na || ldb != f->nb || ldg != f->n_out || !aligned16(a) || !aligned16(b) || !aligned16(g) || !aligned16(ga) ||
        !aligned16(gb))
        return DOL_OK;
    hipFunction_t fn = nullptr;
    const JitBuild bd = build_for(f, kSlotBwd, batch);
    if (dol_status s = kernel_of(f, kSlotBwd, bd, &fn)) return whole_pieces(f) ? s : DOL_OK;
    int n_tiles = (batch + bd.rows - 1) / bd.rows;
    void *args[] = {&a, &b, &g, &ga, &gb, &batch, &n_tiles, &accumulate};
    DOL_HIP(hipModuleLaunchKernel(fn, tile_grid(n_tiles), 1, 1, kJitTile * bd.waves, 1, 1, 0, st, args, nullptr));
    *done = true;
    return DOL_OK;
}

bool table_merge_ok(const dol_fn_table *f) { return table_code_ok(f) && whole_pieces(f) && f->n_out <= kJitMaxMergeOut; }

dol_status launch_damp_table_merge_fwd(const dol_fn_table *f, const UnionPlan *p, int32_t batch, const float *a, const float *b,
                                       const float *c, float *out, int32_t *saved, hipStream_t st)
{
    if (merge_small_batch(f, p, batch)) return launch_sample_merge(f, p, batch, a, b, c, out, saved, nullptr, nullptr, nullptr, nullptr, 0, st);
    hipFunction_t fn = nullptr;
    const int kind = p->aligned ? kSlotMergeFwdAligned : kSlotMergeFwd;
    const JitBuild bd = build_for(f, kind, batch);
    if (dol_status s = kernel_of(f, kind, bd, &fn)) return s;
    int n_tiles = (batch + bd.rows - 1) / bd.rows, nc = p->nb, n3 = p->n_out;
    const int32_t *ia = p->d_ia.ptr, *ib = p->d_ib.ptr;
    void *args[] = {&a, &b, &c, &out, &ia, &ib, &saved, &batch, &n_tiles, &nc, &n3};
    DOL_HIP(hipModuleLaunchKernel(fn, tile_grid(n_tiles), 1, 1, kJitTile * bd.waves, 1, 1, 0, st, args, nullptr));
    return DOL_OK;
}

dol_status launch_damp_table_merge_bwd(const dol_fn_table *f, const UnionPlan *p, int32_t batch, const float *a, const float *b,
                                       const float *c, const float *g, float *ga, float *gb, float *gc, const int32_t *saved,
                                       int32_t accumulate, hipStream_t st)
{
    if (merge_small_batch(f, p, batch)) return launch_sample_merge(f, p, batch, a, b, c, nullptr, const_cast<int32_t *>(saved), g, ga, gb, gc, accumulate, st);
    hipFunction_t fn = nullptr;
    const int kind = p->aligned ? kSlotMergeBwdAligned : kSlotMergeBwd;
    const JitBuild bd = build_for(f, kind, batch);
    if (dol_status s = kernel_of(f, kind, bd, &fn)) return s;
    int n_tiles = (batch + bd.rows - 1) / bd.rows, nc = p->nb, n3 = p->n_out;
    const int32_t *ia = p->d_ia.ptr, *ib = p->d_ib.ptr, *ca = p->d_ca.ptr, *cb = p->d_cb.ptr;
    void *args[] = {&a, &b, &c, &g, &ga, &gb, &gc, &ia, &ib, &ca, &cb, &saved, &batch, &n_tiles, &nc, &n3, &accumulate};
    DOL_HIP(hipModuleLaunchKernel(fn, tile_grid(n_tiles), 1, 1, kJitTile * bd.waves, 1, 1, 0, st, args, nullptr));
    return DOL_OK;
}

dol_status launch_damp_table_merge_both(const dol_fn_table *f, const UnionPlan *p, int32_t batch, const float *a, const float *b,
                                        const float *c, float *out, int32_t *saved, const float *g, float *ga, float *gb, float *gc,
                                        int32_t accumulate, hipStream_t st)
{
    if (merge_small_batch(f, p, batch)) return launch_sample_merge(f, p, batch, a, b, c, out, saved, g, ga, gb, gc, accumulate, st);
    hipFunction_t fn = nullptr;
    const JitBuild bd = build_for_both(f, p->aligned, batch);
    if (dol_status s = kernel_of(f, p->aligned ? kSlotMergeBothAligned : kSlotMergeBoth, bd, &fn)) return s;
    int n_tiles = (batch + bd.rows - 1) / bd.rows, nc = p->nb, n3 = p->n_out;
    const int32_t *ia = p->d_ia.ptr, *ib = p->d_ib.ptr, *ca = p->d_ca.ptr, *cb = p->d_cb.ptr;
    void *args[] = {&a, &b, &c, &out, &g, &ga, &gb, &gc, &ia, &ib, &ca, &cb, &saved, &batch, &n_tiles, &nc, &n3, &accumulate};
    DOL_HIP(hipModuleLaunchKernel(fn, tile_grid(n_tiles), 1, 1, kJitTile * bd.waves, 1, 1, 0, st, args, nullptr));
    return DOL_OK;
}

}  // namespace dol
