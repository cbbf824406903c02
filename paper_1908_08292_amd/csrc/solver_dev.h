// solver_dev.h -- device-side data structures of the batched RVE solver.
#pragma once
#include <cstdint>

#include "plan.h"

namespace fehmm {

struct DevFront {
    int32_t m, p, parent, child_begin, child_end, asm_begin, asm_end, u_lds, wave, pad;
    int64_t rows_off, relind_off, L_off, D_off, y_off, U_off, ea_off;
};

// a front's child as its parent reads it, in the order of children[]
struct DevChild {
    int32_t mc, npre;  // update rows; update entries (a prefix) that go to the parent's panel
    int32_t u_lds, pad;
    int64_t ea_off, inv_off, U_off;
};

// a wave front as the backward substitution reads it, in the order of wave_list
struct BackRec {
    int32_t m, p, rows_off, L_off, D_off, y_off;
};

struct DevPlan {
    int32_t d, n, nnode, nelem, nfront, lds_ok;  // lds_ok: every front's panel fits LDS
    const DevFront* fronts;
    const int32_t* rows;
    const int32_t* relind;
    const int32_t* children;
    const int32_t* asm_dst;
    const int32_t* asm_src;
    const int32_t* ea_dst;
    const int32_t* inv;
    const DevChild* childrec;
    const BackRec* back;
    const int32_t* wave_hbeg;
    int32_t nwave_h;       // number of heights in the wave phase
    int32_t wave_slice;    // LDS elements per wave slice
    const int32_t* wg_steps;  // [nwg_steps][kStepFronts] workgroup-front steps (-1 padded)
    int32_t nwg_steps;
    const int32_t* task;      // wave phase: first and last front of every task
    const int32_t* task_beg;  // [ntask_lev + 1] tasks of each level
    int32_t ntask_lev;
    int32_t ul_base, ul_stride;  // LDS update matrices: first element of wave 0's, elements from wave to wave
    int32_t wide_rhs;         // panels in LDS, FP32 factors: pivots and right-hand sides in FP64 all the same
    int32_t cls;              // launch of the batch that solves the plan's RVEs (set per batch)
    int32_t bc;               // micro boundary conditions: 0 periodic, 1 linear displacements
};

// offsets (in doubles) of the per-slot workspace regions
struct SlotLayout {
    int64_t w, wt, R, rhs, x, fe, ke, re, L, U, S, ir1, ir2, stride;
};

struct SolveArgs {
    const DevPlan* plans;        // [nplan]
    const int32_t* rve_plan;     // [B]
    const int64_t* rve_phase;    // [B] offset into phase_pool
    const uint8_t* phase_pool;
    const int32_t* rve_lame;     // [B] offset (in doubles) into lame_pool
    const int32_t* rve_kind;     // [B] RVE_LAW_* | RVE_ELEM_* << 8 of each RVE's mesh
    const double* lame_pool;
    const int64_t* state_off;    // [B+1]
    const double* rve_atol;      // [B] default absolute tolerance
    const int32_t* order;        // [B] queue order (longest first), or a subset list
    const int32_t* count_dev;    // length of a subset list (device), or null for the whole batch
    const int* skip;             // device flag: when set, the launch solves nothing (graph-captured steps)
    int64_t B;
    int64_t nq;                  // queue entries (without a subset list)
    int32_t cls;                 // >= 0: only the RVEs of plans with this cls
    double* ws;
    SlotLayout lay;
    unsigned int* counter;
    const double* F;
    double* P;
    double* A;
    double* wstate;
    int32_t* status;
    int32_t* iters;
    double rtol, atol;
    int32_t max_iter, backtrack, want_A, dim;
    int32_t lds_elems;           // elements (of the front type) of the dynamic LDS
    int32_t bs_slice;            // FP64 scratch per wave of the LDS plans' backward substitution
    int32_t flags;               // RVE_FLAG_* of the options
    int32_t ir_max;              // refinement sweeps per Newton step (FP32 factors)
    int32_t ir_max_tan;          // refinement sweeps of the tangent solves
    int32_t tan64;               // FP32 factors: the condensation factorization of LDS plans in FP64
    int32_t reuse_tan;           // 2D LDS plans: the condensation from the last Newton factorization
    double ir_eta;               // stop refining when ||b - K x|| <= ir_eta ||R||
    double ir_eta_tan;           // same for the d^2 tangent columns (Frobenius)
};

// LDS of a CU
constexpr int kLdsBytesMax = 160 * 1024;

// tiles of the global-front updates: kTileM rows x (64 or 128) columns per
// pass; two LDS buffers of a 16-column slab of A (kTileM rows) and B (up to
// 128 rows), row stride 144 elements (= 16 mod 32: the four lane groups of an
// MFMA operand read hit distinct LDS banks)
constexpr int kTileM = 128, kTileSlab = 16, kTileStride = 144;
constexpr int kTileLdsElems = 2 * kTileSlab * 2 * kTileStride;

}  // namespace fehmm
