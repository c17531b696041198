// Internal declarations shared by the host driver and the HIP kernels of the
// gradient-domain fusion library.  Not part of the public ABI.
#pragma once

#include "device.h"
#include "smooth.h"

namespace gdf {

// One multigrid level of one slice.  Arrays are row-major with row pitch
// `pitch` (elements, even, >= W + 1 for odd W) so that a lane's two-column
// vector access never leaves the allocation.  Exception: the iterate of
// level 0 (outside the periodic multigrid) stores each row by colour, pixel
// (x, y) at element x / 2 of the half (x + y) & 1 of row y, each half pitch / 2
// elements long: a red-black sweep pass then reads the one colour it needs as
// contiguous runs.
struct LevelDesc {
    void *u[2];      // iterate ping-pong buffers at this level
    void *b;         // right-hand side at this level (scaled units, see below)
    void *ec;        // coarse correction to prolongate (level+1 iterate), or null
    void *bc;        // coarse right-hand side to restrict into (level+1), or null
    int H, W, pitch;
    int Hc, Wc, pitch_c;
    double sigma;    // alpha * h^2 with h = 2^level: the level's scaled screening term
    double wxL, wyL; // width of the last column / height of the last row relative to a full
                     // cell (ceil-halving leaves a partial last cell when a side is odd)
    const double *bshift;  // level 0: per-slice mean of b subtracted on load (null: none)
    int slice;       // slice index (flags, partial sums)
    int pad_;
    // level 1: the level-0 mean; a right-hand side restricted from the unshifted
    // level-0 one (BlockLaunch::raw_rhs) has each cell's children's share of it
    // subtracted on load on the way down
    const double *bshift_fine;
};

// A strip work item: one wave processes columns [x0 - G, x0 - G + 128) of
// rows [y0 - G, y1 + G) and owns output columns [x0, x0 + 128 - 2G) x rows [y0, y1).
struct Item {
    int lev;   // index into the LevelDesc table
    int x0;
    int y0;
    int y1;
    int pidx;  // slot of this item's partial sums (a slice's slots are contiguous)
};

enum ResidMode { RES_NONE = 0, RES_NORM = 1, RES_RESTRICT = 2, RES_BOTH = 3 };

// Launch parameters of one strip pass.
struct StripLaunch {
    const LevelDesc *levs;
    const Item *items;
    int n_items;
    int n_fast;              // items [0, n_fast) run the interior variant
    int n_rows_in;           // items [n_fast, n_rows_in) the column-edge variant, the rest the guarded one
    int in_sel, out_sel;     // which u buffer is read / written
    const int *cycles;       // if non-null: read buffer (cycles[slice] & 1), write the other
    int cycles_stride;       // ints between consecutive slices' counters
    const int *active;       // per-slice "still iterating" flags
    const int *done;         // if non-null and set: no slice is iterating (every wave exits at once)
    float2 *partials;        // per-item partial sums (r^2, r) (RES_NORM / RES_BOTH)
};

// Strip kernel variants (template instances live in mg_kernels.hip).
enum StripKind {
    SK_FIRST_RESTRICT,  // finest, first pass of a solve from zero: restrict b (no sweeps)
    SK_FINE,         // prolongate, fsw sweeps, residual -> norm + restrict (finest, fused up+down)
    SK_SINGLE_ZERO,  // zero start, 2 sweeps, residual -> norm (single-level slices)
    SK_SINGLE,       // 2 sweeps, residual -> norm
    SK_FINE_ZERO,    // as SK_FINE from a zero iterate (the first cycle after SK_FIRST_RESTRICT)
    SK_COUNT
};

// Halo (G) of a strip kind: stages after the load, plus one for prolongation,
// rounded up to even.  Valid output width per strip is 128 - 2G.
int strip_halo(StripKind k, int fsw);

// Enqueue one strip pass (one launch).  Items [0, a.n_fast) stay clear of
// the slice's edges (rows y0 - G .. y1 + G in [1, H - 2], columns x0 - G ..
// x0 - G + 127 in [1, W - 2]) and run the code without row guards and edge
// masks; items [a.n_fast, a.n_rows_in) have such rows but touch a column edge
// (no row guards, per-lane masks); the others run the guarded code.  fsw: sweeps of the fused finest
// pass (SK_FINE).  fp64 selects double precision.  persistent: the grid is capped
// at the workgroups resident on the device at once and each wave loops over
// the list's items; otherwise one wave per item.  sor: the over-relaxed
// instances of SK_FINE / SK_FINE_ZERO (FP32, fsw 4 or 5; any other pass or
// setting is an error).
hipError_t launch_strip(StripKind k, int fsw, bool fp64, bool persistent, const StripLaunch &a, hipStream_t s,
                        bool sor = false);

// Waves of a strip kernel variant that the device holds at once (occupancy x
// SIMDs); 0 if the runtime cannot tell (no device).
int strip_resident_waves(StripKind k, int fsw, bool fp64);

// Resolves the persistent grid sizes of every strip kernel variant for
// fsw and the precision (device queries; call before a stream capture begins).
void strip_prepare(int fsw, bool fp64);

// ---- per-slice reductions and flags ------------------------------------

struct SliceState {
    double bb;          // ||b||^2 of Eq. (1) (f-form right-hand side)
    double rr;          // ||r||^2 at the last check
    double rel;         // sqrt(rr / bb)
    double rel_init;    // residual of f = g_o relative to b
    double aux;         // FIN_SUM result
    double npx;         // pixels in the slice (set by the host)
    double alpha;       // screening weight (set by the host)
    double shift;       // constant-mode correction mean(r) / alpha of the last check
    double bmean;       // mean of the level-0 right-hand side (subtracted on load)
    double uoff;        // bmean / alpha: the solution's mean, added back at the end
    int cycles;         // coarse-grid corrections applied
    int status;         // 0 ok / iterating, GDF_ENONFINITE ...
    int stalled;        // 1: stopped because a cycle no longer reduced the residual
    int pad_;
};

enum FinishMode {
    FIN_BB = 0,       // store the sum as ||b||^2
    FIN_CHECK = 1,    // in-loop residual: store rr/rel, count the cycle, clear `active` when done
    FIN_FINAL = 2,    // residual of the returned f: store rr/rel (count_cycle: not of slices still active)
    FIN_INIT = 3,     // ||b_u||^2: rel_init = sqrt(sum / bb)
    FIN_SUM = 4,      // plain sum into state.aux (e.g. dLoss/dalpha)
    FIN_MEAN = 5      // sum of b: bmean = sum / npx, uoff = bmean / alpha
};

// Sum the partials of each slice over [range[2s], range[2s+1]) in a fixed
// order (deterministic) and update the slice state and flags.  max_slots: the
// longest of these ranges (sizes the blocks; any value is correct).
// partials_f: strip partials (r^2, r); partials_d: FP64 tile partials.
// FIN_CHECK with strip partials also records the constant-mode correction.
// FIN_CHECK with stall_ratio > 0: from the second counted cycle on, a slice
// whose residual shrank by less than that factor in one cycle (while still
// above tol) stops with state.stalled = 1 (the working precision's floor).
// partials_d2 (with partials_d, FIN_CHECK): FP64 partial sums of r, giving
// the constant-mode correction as the strip partials do.
// host_flags (FIN_CHECK, may be null): host memory the device writes; slice s's
// entry becomes 2 seq + its flag.
hipError_t launch_finish(int n_slices, int max_slots, const int *range, const float2 *partials_f,
                         const double *partials_d, const double *partials_d2, int mode, double tol,
                         int max_cycles, int count_cycle, double stall_ratio, SliceState *state, int *active,
                         unsigned *host_flags, unsigned seq, hipStream_t s);

// FIN_BB, FIN_INIT and FIN_MEAN of one right-hand side in one launch.
hipError_t launch_finish_rhs(int n_slices, int max_slots, const int *range, const double *pbb, const double *pb0,
                             const double *pbs, SliceState *state, hipStream_t s);

// After the exact residual of the output (FIN_FINAL): slices whose FP64
// relative residual still exceeds tol, with cycles left and finite state,
// get active = only = 1 (resume iterating, re-form f); others get 0.
// done = 1 when no slice's active flag is set, else 0 (one workgroup).  Lets
// the passes of a captured schedule that outlast the last active slice exit
// at their first instruction.
hipError_t launch_done(int n_slices, const int *active, int *done, hipStream_t s);

hipError_t launch_resume_flags(int n_slices, const SliceState *state, double tol, int max_cycles,
                               int *active, int *only, hipStream_t s);

// ---- elementwise / simple stencil kernels --------------------------------

struct SliceIO {        // per-slice user-buffer view (element offsets/pitches)
    long long off_gs, pitch_gs;
    long long off_go, pitch_go;
    long long off_f, pitch_f;
    double alpha;
    int H, W;
    int lev0;           // LevelDesc index of the slice's finest level
    int tiles_x;        // 64-wide tiles per row (for the simple 2D kernels)
    long long tile_begin;  // first tile index of this slice
    int ftiles_x;       // blocks per row of the row-marching output pass
    int pad_;
    long long ftile_begin;  // first such block of this slice
};

// b_u = alpha (g_s - g_o) into level 0 b, and FP64 partials of
// ||alpha g_s + L g_o||^2, ||b_u||^2 and sum(b_u) per tile (rows: per block, as
// in launch_finalize).
hipError_t launch_prep(bool fp64, bool rows, int gs_dtype, const void *gs, int go_dtype, const void *go,
                       const SliceIO *io_dev, int n_slices, long long n_tiles,
                       const LevelDesc *levs, double *part_bb, double *part_b0, double *part_bs,
                       hipStream_t s);

// f = g_o + u (out dtype), FP64 partials of ||b_u - A u||^2 per tile.  The
// level-0 iterate of slice s is buffer (state[s].cycles & 1).
// With `only` non-null, tiles of slices with only[s] == 0 are skipped.
// rows: the row-marching kernel over blocks of kFinCols x kFinRows (n_tiles
// of those; every width at least 4), else the quad kernel over 64 x 16 tiles.
constexpr int kFinCols = 256, kFinRows = 64;
hipError_t launch_finalize(bool fp64, bool rows, int go_dtype, const void *go, int out_dtype, void *f,
                           const SliceIO *io_dev, int n_slices, long long n_tiles,
                           const LevelDesc *levs, const SliceState *state, const int *only,
                           double *part_rr, hipStream_t s);

// Adjoint right-hand side: b = grad_f (converted), partials of ||grad_f||^2 and sum(grad_f).
hipError_t launch_prep_adjoint(bool fp64, const void *grad_f, const SliceIO *io_dev, int n_slices,
                               long long n_tiles, const LevelDesc *levs, double *part_bb,
                               double *part_bs, hipStream_t s);

// From lambda (level-0 iterate): grad_gs = alpha lambda, grad_go = L lambda,
// partials of lambda . (g_s - f) (part_da null: not formed, g_s and f not read).
// Buffers share the dtype of the solve.
// With u64 non-null, lambda is the FP64 iterate of the mixed solve (buffer
// state[s].cycles & 1) instead of the level-0 working-precision iterate.
hipError_t launch_adjoint_assemble(bool fp64, const void *gs, const void *f, void *grad_gs,
                                   void *grad_go, const SliceIO *io_dev, int n_slices,
                                   long long n_tiles, const LevelDesc *levs,
                                   const SliceState *state, double *const *u64, double *part_da,
                                   hipStream_t s);

// Mixed precision refinement step: u64_out = u64_in + e (e = level-0 FP32
// iterate, buffer e_sel; u64_in zero and not read when first), r = alpha (g_s - g_o) - A u64_out
// in FP64, written as FP32 into level-0 b, partials of ||r||^2.
struct RefineArgs {
    int gs_dtype, go_dtype;
    const void *gs, *go;
    const void *rhs;         // if non-null: b = rhs (dtype gs_dtype, indexed like f) instead of
                             // alpha (g_s - g_o) -- the adjoint system A lambda = grad_f
    const SliceIO *io;
    int n_slices;
    bool rows;               // by row marching (as in launch_finalize); then r is restricted
                             // to level 1's right-hand side as well
    long long n_tiles;
    const LevelDesc *levs;   // FP32 hierarchy
    double *const *u64;      // [2][n_slices] device table of FP64 iterates (pitch = level-0 pitch)
    int in_sel, e_sel;       // which FP64 buffer is read; which FP32 level-0 buffer holds e
    int first;               // 1: u64_in = 0, not read
    const int *active;
    double *part_rr;
};
hipError_t launch_refine(const RefineArgs &a, hipStream_t s);

// Mixed precision output: f = g_o + u64 (buffer state[s].cycles & 1).
hipError_t launch_finalize64(int go_dtype, const void *go, int out_dtype, void *f,
                             const SliceIO *io_dev, int n_slices, long long n_tiles,
                             double *const *u64, const SliceState *state, const LevelDesc *levs,
                             hipStream_t s);

// ---- register-block passes ---------------------------------------------------
//
// Passes over the coarse levels, over the finest level of small batches and over
// every level of a periodic hierarchy (block_kernels.hip): one workgroup per kBlockCols x kBlockRows region.  Along
// a side of n cells with a halo of G, tile t of a Neumann level covers cells
// [t (len - 2 G), + len) and owns those at least G from the region's ends, an
// end on the slice's edge excepted; a periodic tile owns cells
// [t (len - 2 G), (t + 1) (len - 2 G)) and its halo wraps.
constexpr int kBlockCols = 2 * kWave, kBlockRows = 64, kBlockWaves = 8;
struct BItem {
    int lev;     // LevelDesc index
    int tx, ty;  // tile along the columns and the rows
};
// tiles along a side of n cells
constexpr int block_tiles(int n, int len, int G, bool periodic)
{
    return periodic ? (n + len - 2 * G - 1) / (len - 2 * G)
                    : (n <= len ? 1 : 1 + (n - len + len - 2 * G - 1) / (len - 2 * G));
}
struct BlockLaunch {
    const LevelDesc *levs;
    const BItem *items;
    int n_items;
    int G;                 // halo of the list's tiles
    int in_sel, out_sel;   // u buffers read and written
    const int *active;
    const int *done;       // as in StripLaunch
    int raw_rhs;           // level 1: b holds sums of unshifted level-0 values (see LevelDesc)
    double *part_rr, *part_r;   // level-0 residual: per-item sums of r^2 and r
    // fused finest pass of the Neumann hierarchy: as in StripLaunch
    const int *cycles;
    int cycles_stride;
    float2 *partials;
};
// Sweeps per smoothing step is `sweeps` (two half-sweeps each).  Level 0 (periodic
// only) has the arithmetic type and forms the residual norms on the way up;
// coarse levels are stored as LevelDesc says.
enum BlockKind {
    BK_DOWN_ZERO,   // zero start, sweeps, restriction of the residual
    BK_DOWN,        // sweeps, restriction (periodic level 0 after the first cycle)
    BK_UP,          // prolongation, sweeps (level 0: residual norms)
    BK_LAST_ZERO,   // coarsest level: zero start, sweeps (Neumann: 2 sweeps)
    BK_LAST_MID,    // coarsest level that is level 0: sweeps
    BK_LAST         // coarsest level: sweeps (level 0: residual norms)
};
// halo of a pass: cells that go stale per pass, rounded up to even
constexpr int block_halo(int sweeps) { return 2 * sweeps + 2; }
// The coarse levels of a slice from the first that is at most kTailSide a side, in
// one workgroup (Neumann; at least two levels).  Items: lev the first level's
// descriptor, tx its number, ty how many levels; sweeps per level number.
constexpr int kTailSide = 128;
static_assert(kTailSide <= kBlockCols && kTailSide <= 2 * kBlockRows, "a tail level is one region");
struct TailLaunch {
    BlockLaunch a;
    int sweeps[kMaxLevels];
};
hipError_t launch_tail(bool fp64, const TailLaunch &t, hipStream_t s);
// The fused finest pass (SK_FINE, SK_FINE_ZERO when zero) as blocks; halo
// block_halo(sweeps).
hipError_t launch_block_fine(bool zero, int sweeps, bool sor, bool fp64, const BlockLaunch &a, hipStream_t s);
hipError_t launch_block(BlockKind k, bool periodic, bool level0, int sweeps, bool fp64, const BlockLaunch &a,
                        hipStream_t s);

// ---- periodic boundaries ---------------------------------------------------
//
// Slices with wrap-around (periodic) boundaries run the levels and finite-volume
// operators of the Neumann hierarchy with the neighbours of the first and last
// row and column taken across the wrap (the passes above).  Level-0 iterates
// are row-major, in buffer 0 between cycles (a constant index: a runtime one into a
// descriptor copy sends it to scratch memory).  The per-pixel kernels (periodic_kernels.hip) run one workgroup
// per 64 x 16 pixel tile (SliceIO::tile_begin counts them slice by slice, so
// per-slice partial sums occupy contiguous slots).
struct PLaunch {
    const LevelDesc *levs;
    const int *slice_of;   // the slice of each tile
    int n_items;           // tiles
    double *part_rr;       // per-item sums of r^2
};
// Buffer element types (gdf_dtype values of the public header).
enum { GDF_DT_U8 = 0, GDF_DT_F32 = 1, GDF_DT_F64 = 2 };
// b_u = alpha (g_s - g_o) into level-0 b, partials of ||alpha g_s + L g_o||^2,
// ||b_u||^2, sum(b_u), with the periodic L; items of level 0
hipError_t launch_pprep(bool fp64, int gs_dtype, const void *gs, int go_dtype, const void *go, const SliceIO *io,
                        const PLaunch &a, double *part_bb, double *part_b0, double *part_bs, hipStream_t s);
// f = g_o + u (+ uoff + shift) from the level-0 buffer 0, FP64 partials
// of the residual ||b_u - A u||^2; slices with only[s] == 0 skipped (only non-null)
hipError_t launch_pfinalize(bool fp64, int go_dtype, const void *go, int out_dtype, void *f, const SliceIO *io,
                            const PLaunch &a, const SliceState *st, const int *only, hipStream_t s);
// mixed refinement step with the periodic operator (as launch_refine; the
// FP32 correction is in level-0 buffer e_sel)
hipError_t launch_prefine(const RefineArgs &r, const PLaunch &a, hipStream_t s);
// adjoint assembly with the periodic L (as launch_adjoint_assemble; lambda in
// level-0 buffer a.in_sel, or the FP64 iterate u64[(cycles & 1) * n + s] when
// u64 is non-null)
hipError_t launch_padjoint(bool fp64, const void *gs, const void *f, void *grad_gs, void *grad_go,
                           const SliceIO *io, int n_slices, const PLaunch &a, const SliceState *st,
                           double *const *u64, double *part_da, hipStream_t s);

// Transpose of the smoothing for FP32 gradients: out = K (g / D) (see
// smooth_transpose.hip); tmp holds S H W floats, inv_d the tables 1 / Dz (S),
// 1 / Dy (H), 1 / Dx (W) in that order; wxy[0..7] and wz[0..15] the taps.
// 1 / D tables of the smoothing transpose (W + H + S floats at inv_d), from
// the in-plane (radius rxy <= 7) and cross-slice (rz <= 15) taps in FP64.
hipError_t launch_transpose_tables(float *inv_d, int S, int H, int W, int rxy, int rz, const double *wxy,
                                   const double *wz, hipStream_t s);
// add (nullable, may be out itself): out = K (g / D) + add.  tmp2: a second
// S H W buffer for the one-voxel passes.
hipError_t launch_smooth_transpose(const float *g, float *out, const float *add, float *tmp, float *tmp2,
                                   const float *inv_d, int S, int H, int W, int rxy, int rz, const float *wxy,
                                   const float *wz, hipStream_t s);
// dst[0] = sum of state[i].aux over the slices, in slice order (one thread)
hipError_t launch_sum_aux(int n_slices, const SliceState *state, double *dst, hipStream_t s);

}  // namespace gdf
