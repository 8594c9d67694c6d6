// Arguments of the polyphase kernels (wtconv_phase.h) and their launchers.
// Internal; not part of the public ABI.
#pragma once

#include "wtconv_internal.h"

namespace wtc {

// ----------------------------------------------------------------------------
// Polyphase kernels on the matrix cores (wtconv_phase.h, wtconv_phase_fwd.hip).
//
// One Haar level of the branch together with the base path is, per output
// phase (row and column parity), a plain correlation of the input with a
// (2k) x (2k) kernel: E_ab = 1/4 (LL +- LH +- HL +- HH) of the folded subband
// kernels spread over the 2 x 2 phases, plus the base kernel. Stage s (level
// s + 1) applies it to X_s, the 2^s x 2^s block means of the input, and the
// stages add up: y = Op_0(X_0) + up(Op_1(X_1) + up(...)), up() repeating every
// value 2 x 2. A 2 x 8 pixel tile of one stage is a 16 x (16 k) matrix (its
// 2k x 16 input window) times the window, so 16 tiles are one chain of k
// v_mfma_f32_16x16x32 per pair of operand pieces.
// ----------------------------------------------------------------------------
constexpr int kPhaseMaxStages = 5;
// Row pairs of one vertical segment a lane keeps sums for: eight would spill
// next to one block round's loads at three wavefronts per SIMD.
__host__ __device__ constexpr int phase_max_js(int block_rounds) { return block_rounds > 1 ? 8 : 7; }
constexpr int kPhaseMargin = 4;  // zero rows above and columns left of a stage's pixels in LDS (2 (k / 2) <= 4)
constexpr int kPhaseTabPitch = 24;  // 16-bit elements per row of a weight table

struct PhaseStage {
    int h, w;    // grid of X_s
    int ct;      // 8-column tiles per row
    int pitch;   // 16-bit elements per LDS row (multiple of 8)
    int poff;    // byte offset of piece 0 in a plane's region; pixel (y, x) at row y + margin, column x + margin
    int psz;     // bytes per piece
    int V, js;   // vertical segments and row pairs per segment: V * js >= ceil(h / 2)
    int roff;    // s >= 1: byte offset of the stage's float32 result in a plane's region
    int rpitch;  // floats per row of it
    int mf;      // s >= 2, when a deeper stage reads it: byte offset of X_s in float32 (w floats per row)
    int tab;     // s >= 1: byte offset of the stage's weight table in LDS
    float r_ct, r_vct;  // 1 / ct, 1 / (V * ct)
};

struct PhaseArgs {
    const void* in;
    void* out;
    ParamPtrs p;
    int B, C;
    int nb, PP;         // batch planes per workgroup, resident planes
    int L;              // stages 0 .. max(L, 1) - 1 (L >= 1)
    int skip_base;
    int fine_waves;     // wavefronts that run stage 0: 4 (L = 1), 3 (the fourth runs the deeper stages) or 2
                        // (the third runs stage 1, the fourth the stages from 2 on; L >= 3)
    int planes_off;     // byte offset of the first plane's region in LDS
    int plane_bytes;    // bytes per plane's region
    int mark_off;       // byte offset of the marks of non-finite pixels (and one of infinities)
    int lds_bytes;
    int bx, by;         // 4 x 4 pixel blocks per row / column of the loaded area
    float r_bx, r_bxy;  // 1 / bx, 1 / (bx * by)
    // Region mode (rg_ntx > 0, L = 1): workgroup (chunk, tile) covers the
    // rg_th x rg_tw output tile at (ty * rg_th, tx * rg_tw) of the H x W plane.
    int rg_ntx, rg_nty, rg_th, rg_tw;
    int H, W;           // the real plane
    // region mode only: the contribution of the levels above the first on the
    // level-1 grid ([B][C][carry_H][carry_W], storage type; nullable)
    const void* carry;
    int carry_H, carry_W;
    // the launch also runs the finalize `fin`: in fin_blocks workgroups at the
    // head of the grid (see FusedArgs), or its fin_tasks tasks in the plane
    // workgroups
    int fin_blocks, fin_tasks;
    ReduceArgs fin;
    PhaseStage st[kPhaseMaxStages];
};

// Kernel gradients in the polyphase formulation (wtconv_phase_grad.hip): the
// gradient of stage s's 16 x 16 k weight matrix is the product of its output
// gradients' tiles (the block means D_s of dy) with the windows of X_s.
// One operand side (x or dy) of every stage in LDS, per plane:
struct PhaseSide {
    int margin;  // zero rows and columns before the first pixel
    int off[kPhaseMaxStages];    // byte offset of piece 0 in the plane's region
    int pitch[kPhaseMaxStages];  // 16-bit elements per row (multiple of 8)
    int psz[kPhaseMaxStages];    // bytes per piece
    int mf[kPhaseMaxStages];     // s >= 2, when a deeper stage reads it: the means in float32 (w floats per row)
};

struct PhaseGradArgs {
    const void* x;
    const void* dy;
    float* partial;  // [nchunks (* tiles)][C][NP] kernel-gradient partials
    int B, C, H, W;
    int nb, PP, L;
    int skip_base;
    int fine_waves;   // wavefronts on stage 0: 4 (L = 1), 3 (L = 2), 2 (L = 3) or 1; then one per deeper stage
                      // (the fourth takes stages 3 and 4)
    int plane_bytes, lds_bytes;
    int xbx, xby;     // 4 x 4 blocks of x per row / column of the loaded area
    int dbx, dby;     // of dy
    float r_xbx, r_xb, r_dbx, r_db;  // 1 / xbx, 1 / (xbx xby), 1 / dbx, 1 / (dbx dby)
    int h[kPhaseMaxStages], w[kPhaseMaxStages];   // grids
    int ct[kPhaseMaxStages];                      // 8-column tiles per row
    int V[kPhaseMaxStages], js[kPhaseMaxStages];  // vertical segments, row pairs each
    float r_ct[kPhaseMaxStages], r_vct[kPhaseMaxStages];
    PhaseSide sx, sd;
    // Region mode (rg_ntx > 0, L = 1): rg_T x rg_T tiles; x is loaded with one
    // block of halo, dy without. cx, cdy (nullable): the level-1 carriers of x
    // and dy of the tile's own pixels, [B][C][cH][cW].
    int rg_ntx, rg_nty, rg_T;
    void* cx;
    void* cdy;
    int cH, cW;
};

// Weak: the planner's host tests link without the kernels; the phase route is
// then not offered.
hipError_t launch_phase_forward(int k, wtconv_dtype dt, const PhaseArgs& a, int grid, int block_rounds,
                                hipStream_t s) __attribute__((weak));
hipError_t launch_phase_grad(int k, wtconv_dtype dt, const PhaseGradArgs& a, int grid, int block_rounds,
                             hipStream_t s) __attribute__((weak));

}  // namespace wtc
