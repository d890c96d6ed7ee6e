// What the two families of iteration kernels share (iterate.hip, iterate_grid.hip): arguments, LDS addressing, the clamp
// decision in the sign.
#pragma once

#include "internal.h"
#include "wave_util.h"

namespace dol {

constexpr size_t kItLdsMax = 160 * 1024;

__device__ __forceinline__ float signed_tag(float pre) { return pre <= 1.0f ? pre : -1.0f; }

struct ItFwdArgs {
    int32_t batch, na, nb, rounds;
    const uint32_t *col_ptr, *col_ij;
    const float *r0;
    int64_t ldr;
    const float *e;
    int64_t lde;
    float *hist;                        // [rounds + 1, batch, na] or nullptr
    float *ckpt;                        // [n_ckpt, batch, na] or nullptr: r_every, r_2*every, ... (those before r_rounds)
    int32_t every;
    float *out;                         // [batch, ldo] or nullptr: r_rounds
    int64_t ldo;
};

struct ItBwdArgs {
    int32_t batch, na, nb, rounds, every;   // every: rounds per segment (the checkpoint interval)
    int32_t n_tuples, n_long;
    int32_t shares_in_seg;                  // every tuple's share lives in a register during the sweep: the LDS words they
                                            // are gathered through at the end take the place of the (then spent) segment
    const uint32_t *col_ptr, *col_ij, *rowa_ptr, *rowa_jc, *rowb_ptr, *rowb_pos, *long_rows;
    const float *e;
    int64_t lde;
    const float *hist;                      // full history, or nullptr: then r0 and ckpt
    const float *r0;
    int64_t ldr;
    const float *ckpt;
    const float *gout;                      // upstream gradient w.r.t. r_rounds, or
    int64_t ldg;
    const int32_t *target;                  // [batch]: the loss is -log r_rounds[target], read from `out`
    const float *out;
    int64_t ldo;
    float *grad_r0;                         // [batch, na] or nullptr
    float *grad_e;                          // [batch, ldge] or nullptr
    int64_t ldge;
};

// LDS addresses as 32-bit numbers: what a thread keeps in a register is the address of its element in the first row.
typedef __attribute__((address_space(3))) float lds_float;

__device__ __forceinline__ uint32_t lds_address(const float *p)
{
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const lds_float *)p));
}

__device__ __forceinline__ float lds_at(uint32_t address) { return *reinterpret_cast<const lds_float *>(static_cast<uintptr_t>(address)); }

__device__ __forceinline__ void lds_put(uint32_t address, float v) { *reinterpret_cast<lds_float *>(static_cast<uintptr_t>(address)) = v; }

// (an address the compiler must take as it is: what is added to it afterwards stays a constant on the instruction)
__device__ __forceinline__ uint32_t fixed_offset(uint32_t x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// ---------------------------------------------------------------- tables shaped like a grid (iterate_grid.hip)

bool grid_table(const dol_fn_table *f);
int grid_waves(const dol_fn_table *f, int32_t batch);                  // wavefronts of a workgroup
size_t grid_bwd_lds(const dol_fn_table *f, int32_t batch, int32_t every);
bool grid_shares_in_seg(const dol_fn_table *f, int32_t batch, int32_t every);
dol_status launch_grid_fwd(const dol_fn_table *f, const ItFwdArgs &A, hipStream_t st);
dol_status launch_grid_bwd(const dol_fn_table *f, const ItBwdArgs &A, size_t lds, hipStream_t st);
const char *grid_fwd_bwd_kernel(const dol_fn_table *f, int32_t batch, int32_t rounds, int32_t every);      // the name of what this launches:
dol_status launch_grid_fwd_bwd(const dol_fn_table *f, const ItFwdArgs &F, const ItBwdArgs &B, size_t lds, hipStream_t st);

}  // namespace dol
