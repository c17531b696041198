// Per-pixel kernels around the multigrid solve of Eq. (1): right-hand side
// formation, output formation with the FP64 residual of the returned f, the
// adjoint assembly, the FP64 refinement step of the mixed-precision solve,
// and the fixed-order per-slice reductions.
//
// All of them walk 64 x 16 pixel tiles with 256 threads; each thread handles
// four consecutive pixels of one tile row (vector loads and stores), so rows
// are read coalesced; horizontal stencil neighbours come from the adjacent
// threads by DPP row shifts, vertical ones from the adjacent rows (L2 hits).
// Partial sums are reduced per tile in FP64 and written to a per-tile slot; a
// second kernel sums each slice's slots in a fixed order.
#include "internal.h"

namespace gdf {

constexpr int kTileW = 64, kTileH = 16;

__device__ __forceinline__ int find_slice(const SliceIO *io, int n, long long tile)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (io[mid].tile_begin <= tile) lo = mid; else hi = mid - 1;
    }
    return lo;
}

template <typename TV> __device__ __forceinline__ double ldv(const TV *p, long long i) { return (double)p[i]; }

// Sum over a 256-thread block in a fixed order (butterfly within each wave,
// then the four wave sums in order), so results do not depend on scheduling.
__device__ double block_sum(double v, double *red)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    const double r = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
    return r;
}

// ---- quad mapping: thread t of a tile handles the four pixels x .. x + 3 of
// one row, x = tile_x0 + 4 (t & 15), y = ty0 + (t >> 4).  The 16 threads of a
// tile row form one DPP row, so horizontal neighbours across threads come from
// row shifts; the tile's two outer neighbours are loaded.

template <typename T> struct Vec4 { typedef T type __attribute__((ext_vector_type(4))); };

// p[i .. i + 3] as doubles; elements at or past nvalid read as 0
template <typename TV>
__device__ __forceinline__ void load4(const TV *p, long long i, int nvalid, double v[4])
{
    using V = typename Vec4<TV>::type;
    if (nvalid >= 4 && (reinterpret_cast<uintptr_t>(p + i) & (sizeof(V) - 1)) == 0) {
        const V q = *reinterpret_cast<const V *>(p + i);
        v[0] = (double)q.x;
        v[1] = (double)q.y;
        v[2] = (double)q.z;
        v[3] = (double)q.w;
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = k < nvalid ? (double)p[i + k] : 0.0;
    }
}

template <typename T> struct Vec2 { typedef T type __attribute__((ext_vector_type(2))); };

// Level-0 iterates store each row by colour (see LevelDesc): pixel (x, y) at
// element x / 2 of the half (x + y) & 1 of row y, the halves pitch / 2 long.
template <typename S> struct RBView {
    const S *u;
    long long pitch, half;
    __device__ RBView(const S *u_, long long pitch_) : u(u_), pitch(pitch_), half(pitch_ >> 1) {}
    __device__ double at(int x, int y) const
    {
        return (double)u[(long long)y * pitch + ((x + y) & 1) * half + (x >> 1)];
    }
    // pixels x .. x + 3 of row y (x a multiple of 4); past nvalid: 0
    __device__ void quad(int x, int y, int nvalid, double v[4]) const
    {
        using V2 = typename Vec2<S>::type;
        if (nvalid <= 0) {
            v[0] = v[1] = v[2] = v[3] = 0.0;
            return;
        }
        const S *r0 = u + (long long)y * pitch + (x >> 1), *r1 = r0 + half;
        const S *re = (y & 1) ? r1 : r0, *ro = (y & 1) ? r0 : r1;   // colours of pixels x and x + 1
        if (nvalid >= 4) {
            const V2 a = *reinterpret_cast<const V2 *>(re), b = *reinterpret_cast<const V2 *>(ro);
            v[0] = (double)a.x;
            v[1] = (double)b.x;
            v[2] = (double)a.y;
            v[3] = (double)b.y;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = k < nvalid ? (double)((k & 1) ? ro : re)[k >> 1] : 0.0;
        }
    }
};
// A row-major array (the FP64 iterates of the mixed scheme), same interface.
template <typename S> struct RowView {
    const S *u;
    long long pitch;
    __device__ RowView(const S *u_, long long pitch_) : u(u_), pitch(pitch_) {}   // u null: all zero
    __device__ double at(int x, int y) const { return u ? (double)u[(long long)y * pitch + x] : 0.0; }
    __device__ void quad(int x, int y, int nvalid, double v[4]) const
    {
        load4(u, (long long)y * pitch + x, u ? nvalid : 0, v);
    }
};

template <typename TV>
__device__ __forceinline__ void store4(TV *p, long long i, int nvalid, const double v[4])
{
    using V = typename Vec4<TV>::type;
    if (nvalid >= 4 && (reinterpret_cast<uintptr_t>(p + i) & (sizeof(V) - 1)) == 0) {
        V q;
        q.x = (TV)v[0];
        q.y = (TV)v[1];
        q.z = (TV)v[2];
        q.w = (TV)v[3];
        *reinterpret_cast<V *>(p + i) = q;
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < nvalid) p[i + k] = (TV)v[k];
    }
}

// value of the previous / next thread in the 16-lane DPP row (0 at the row ends)
__device__ __forceinline__ double row_prev(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), 0x111, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x111, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double row_next(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), 0x101, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x101, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

struct QuadCtx {
    long long tile;         // logical tile index (also the slot of its partial sums)
    int si, x, y, nvalid;   // nvalid: pixels of the quad inside the row (<= 0: none)
    bool row_in;
    SliceIO P;
};

__device__ __forceinline__ bool quad_ctx(const SliceIO *io, int n, long long n_tiles, QuadCtx &c)
{
    const long long tile = xcd_tile(blockIdx.x, gridDim.x);
    c.tile = tile;
    if (tile >= n_tiles) return false;
    c.si = find_slice(io, n, tile);
    c.P = io[c.si];
    const long long lt = tile - c.P.tile_begin;
    c.x = (int)(lt % c.P.tiles_x) * 64 + 4 * (threadIdx.x & 15);
    c.y = (int)(lt / c.P.tiles_x) * 16 + (threadIdx.x >> 4);
    c.nvalid = min(4, c.P.W - c.x);
    c.row_in = c.y < c.P.H && c.nvalid > 0;
    return true;
}

// ------------------------------------------------------------- finish ---

// One block per slice; fixed-order strided sum then a fixed tree, so the
// result does not depend on scheduling.  The kernels are a chain of dependent
// loads on as many CUs as there are slices: each thread keeps kFinLoads
// independent loads in flight, and slices with many partial sums take NT =
// 1024 threads (launch_finish*).  2 slices of 559104 partials: 0.93 ms
// with 256 threads and one load in flight each, 0.10 ms now.
constexpr int kFinLoads = 8;

// Sum over an NT-thread block in a fixed order (butterfly within each wave,
// then the wave sums in order).
template <int NT> __device__ double block_sum_n(double v, double *red)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) r += red[w];
    __syncthreads();
    return r;
}

// sum over i in [b0, b1) of get(i) by the block's threads: thread-strided
// elements, kFinLoads accumulators per thread added in order
template <int NT, class Get> __device__ __forceinline__ double strided_sum(int b0, int b1, Get get)
{
    double acc[kFinLoads];
#pragma unroll
    for (int k = 0; k < kFinLoads; ++k) acc[k] = 0.0;
    for (long long i = (long long)b0 + threadIdx.x; i < b1; i += kFinLoads * NT)
#pragma unroll
        for (int k = 0; k < kFinLoads; ++k) {
            // (clamped, unconditional loads: they all start before the first is waited for)
            const long long j = i + (long long)k * NT;
            const double x = get((int)(j < b1 ? j : i));
            acc[k] += j < b1 ? x : 0.0;
        }
    double v = acc[0];
#pragma unroll
    for (int k = 1; k < kFinLoads; ++k) v += acc[k];
    return v;
}

template <int NT>
__global__ __launch_bounds__(NT) void finish_kernel(int n_slices, const int *range,
                                                    const float2 *pf, const double *pd, const double *pd2,
                                                    int mode, double tol, int max_cycles, int count_cycle,
                                                    double stall_ratio, SliceState *st, int *active,
                                                    unsigned *host_flags, unsigned seq)
{
    __shared__ double red[NT / 64];
    const int sidx = blockIdx.x;
    if (sidx >= n_slices) return;
    const int b0 = range[2 * sidx], b1 = range[2 * sidx + 1];
    double v = 0.0, w = 0.0;
    if (pf) {
        v = strided_sum<NT>(b0, b1, [=](int i) { return (double)pf[i].x; });
        w = strided_sum<NT>(b0, b1, [=](int i) { return (double)pf[i].y; });
    } else {
        v = strided_sum<NT>(b0, b1, [=](int i) { return pd[i]; });
        if (pd2) w = strided_sum<NT>(b0, b1, [=](int i) { return pd2[i]; });
    }
    const bool has_r = pf || pd2;   // (uniform)
    const double sum = block_sum_n<NT>(v, red);
    const double rsum = has_r ? block_sum_n<NT>(w, red) : 0.0;
    if (threadIdx.x != 0) return;
    SliceState &S = st[sidx];
    switch (mode) {
    case FIN_BB: S.bb = sum; break;
    case FIN_INIT: S.rel_init = S.bb > 0.0 ? sqrt(sum / S.bb) : sqrt(sum); break;
    case FIN_SUM: S.aux = sum; break;
    case FIN_MEAN:
        S.bmean = sum / S.npx;
        S.uoff = S.bmean / S.alpha;
        break;
    case FIN_FINAL:
        if (count_cycle && active[sidx]) return;   // still iterating: its state stays the in-loop one
        S.rr = sum;
        S.rel = S.bb > 0.0 ? sqrt(sum / S.bb) : sqrt(sum);
        if (!isfinite(sum)) S.status = 6;  // GDF_ENONFINITE
        break;
    case FIN_CHECK:
    default:
        // the flag for the host: one posted write, tagged with the check's number
        auto tell = [&](unsigned v) {
            if (host_flags)
                __hip_atomic_store(host_flags + sidx, seq * 2u + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        };
        if (!active[sidx]) {   // frozen slice keeps its last state
            tell(0u);
            return;
        }
        const double prev = S.rel;   // the previous check's (0 before the first)
        S.rr = sum;
        S.rel = S.bb > 0.0 ? sqrt(sum / S.bb) : sqrt(sum);
        if (count_cycle) S.cycles += 1;
        if (stall_ratio > 0.0 && count_cycle && S.cycles >= 2 && prev > 0.0 && S.rel > tol &&
            S.rel > stall_ratio * prev) {
            S.stalled = 1;
            active[sidx] = 0;
        }
        // Neumann: 1^T A = alpha 1^T, so the constant-mode error of the iterate is
        // exactly -mean(r) / alpha; adding it back removes mean(r) from the residual
        S.shift = has_r ? rsum / (S.npx * S.alpha) : 0.0;
        if (!isfinite(sum)) S.status = 6;
        if (!isfinite(sum) || S.rel <= tol || S.cycles >= max_cycles) active[sidx] = 0;
        tell(active[sidx] ? 1u : 0u);
        break;
    }
}

// The three sums after right-hand-side formation in one launch: ||b||^2,
// rel_init = sqrt(||b_u||^2 / ||b||^2), and the mean of b_u (bmean, uoff).
template <int NT>
__global__ __launch_bounds__(NT) void finish_rhs_kernel(int n_slices, const int *range, const double *pbb,
                                                        const double *pb0, const double *pbs, SliceState *st)
{
    __shared__ double red[NT / 64];
    const int sidx = blockIdx.x;
    if (sidx >= n_slices) return;
    const int b0 = range[2 * sidx], b1 = range[2 * sidx + 1];
    const double v = strided_sum<NT>(b0, b1, [=](int i) { return pbb[i]; });
    const double w = strided_sum<NT>(b0, b1, [=](int i) { return pb0[i]; });
    const double x = strided_sum<NT>(b0, b1, [=](int i) { return pbs[i]; });
    const double sbb = block_sum_n<NT>(v, red), sb0 = block_sum_n<NT>(w, red), sbs = block_sum_n<NT>(x, red);
    if (threadIdx.x != 0) return;
    SliceState &S = st[sidx];
    S.bb = sbb;
    S.rel_init = sbb > 0.0 ? sqrt(sb0 / sbb) : sqrt(sb0);
    S.bmean = sbs / S.npx;
    S.uoff = S.bmean / S.alpha;
}

// A slice with more partial sums than this takes a 1024-thread block: 256
// threads then need more than one trip of kFinLoads loads.
constexpr int kFinWide = 256 * kFinLoads;

hipError_t launch_finish_rhs(int n_slices, int max_slots, const int *range, const double *pbb, const double *pb0,
                             const double *pbs, SliceState *state, hipStream_t s)
{
    if (n_slices <= 0) return hipSuccess;
    if (max_slots > kFinWide)
        hipLaunchKernelGGL(finish_rhs_kernel<1024>, dim3(n_slices), dim3(1024), 0, s, n_slices, range, pbb, pb0, pbs, state);
    else
        hipLaunchKernelGGL(finish_rhs_kernel<256>, dim3(n_slices), dim3(256), 0, s, n_slices, range, pbb, pb0, pbs, state);
    return hipGetLastError();
}

hipError_t launch_finish(int n_slices, int max_slots, const int *range, const float2 *partials_f,
                         const double *partials_d, const double *partials_d2, int mode, double tol,
                         int max_cycles, int count_cycle, double stall_ratio, SliceState *state, int *active,
                         unsigned *host_flags, unsigned seq, hipStream_t s)
{
    if (n_slices <= 0) return hipSuccess;
    if (max_slots > kFinWide)
        hipLaunchKernelGGL(finish_kernel<1024>, dim3(n_slices), dim3(1024), 0, s, n_slices, range, partials_f,
                           partials_d, partials_d2, mode, tol, max_cycles, count_cycle, stall_ratio, state, active,
                           host_flags, seq);
    else
        hipLaunchKernelGGL(finish_kernel<256>, dim3(n_slices), dim3(256), 0, s, n_slices, range, partials_f,
                           partials_d, partials_d2, mode, tol, max_cycles, count_cycle, stall_ratio, state, active,
                           host_flags, seq);
    return hipGetLastError();
}

__global__ __launch_bounds__(64) void sum_aux_kernel(int n_slices, const SliceState *st, double *dst)
{
    if (threadIdx.x != 0) return;
    double v = 0.0;
    for (int i = 0; i < n_slices; ++i) v += st[i].aux;   // fixed order
    *dst = v;
}

hipError_t launch_sum_aux(int n_slices, const SliceState *state, double *dst, hipStream_t s)
{
    hipLaunchKernelGGL(sum_aux_kernel, dim3(1), dim3(64), 0, s, n_slices, state, dst);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void done_kernel(int n_slices, const int *active, int *done)
{
    __shared__ int any;
    if (threadIdx.x == 0) any = 0;
    __syncthreads();
    int a = 0;
    for (int i = threadIdx.x; i < n_slices; i += blockDim.x) a |= active[i];
    if (a) any = 1;   // benign race: every writer stores 1
    __syncthreads();
    if (threadIdx.x == 0) *done = any ? 0 : 1;
}

hipError_t launch_done(int n_slices, const int *active, int *done, hipStream_t s)
{
    hipLaunchKernelGGL(done_kernel, dim3(1), dim3(256), 0, s, n_slices, active, done);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void resume_flags_kernel(int n_slices, const SliceState *st, double tol,
                                                          int max_cycles, int *active, int *only)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_slices) return;
    const SliceState &S = st[i];
    const int again = S.status == 0 && !S.stalled && isfinite(S.rel) && S.rel > tol && S.cycles < max_cycles;
    active[i] = again;
    only[i] = again;
}

hipError_t launch_resume_flags(int n_slices, const SliceState *state, double tol, int max_cycles,
                               int *active, int *only, hipStream_t s)
{
    if (n_slices <= 0) return hipSuccess;
    hipLaunchKernelGGL(resume_flags_kernel, dim3((n_slices + 255) / 256), dim3(256), 0, s, n_slices, state,
                       tol, max_cycles, active, only);
    return hipGetLastError();
}

// -------------------------------------------------------- row marching ---

constexpr int kFinQ = 4;   // rows of loads in flight

__device__ __forceinline__ int find_fslice(const SliceIO *io, int n, long long t)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (io[mid].ftile_begin <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// lane i receives lane i - 1's / i + 1's value (0 at the wave's ends)
__device__ __forceinline__ double wave_prev(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), 0x138, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x138, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double wave_next(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), 0x130, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x130, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

template <typename V> __device__ __forceinline__ void v4_to_d(const V &q, double v[4])
{
    v[0] = (double)q.x;
    v[1] = (double)q.y;
    v[2] = (double)q.z;
    v[3] = (double)q.w;
}

#define GDF_GLOBAL __attribute__((address_space(1)))

// four elements starting on any element
template <typename T> struct Vec4U { typedef T type __attribute__((ext_vector_type(4), aligned(sizeof(T)))); };

// q[d], q[d + 1], ... at the front (d in 0 .. 3; what is behind them repeats q[3])
template <typename V> __device__ __forceinline__ V shift_down(const V &q, int d)
{
    V r;
    r.x = d == 0 ? q.x : d == 1 ? q.y : d == 2 ? q.z : q.w;
    r.y = d == 0 ? q.y : d == 1 ? q.z : q.w;
    r.z = d == 0 ? q.z : q.w;
    r.w = q.w;
    return r;
}

// A row block of the marching passes: this wave's columns and rows.
struct RowBlock {
    int si, H, W, X0, Y0, Y1;
    int x, nv;      // the lane's first pixel and the pixels of its quad inside the row (<= 0: none)
    int xa, xo, d;  // quad in padded arena rows; quad in caller rows, and its shift
    bool in, tail;  // the lane has pixels; (uniform) the row ends inside some lane's quad
};
__device__ __forceinline__ RowBlock row_block(const SliceIO *io, int si, long long ft)
{
    RowBlock b;
    b.si = si;
    b.H = __builtin_amdgcn_readfirstlane(io[si].H);
    b.W = __builtin_amdgcn_readfirstlane(io[si].W);
    const int ftx = __builtin_amdgcn_readfirstlane(io[si].ftiles_x);
    const int lt = __builtin_amdgcn_readfirstlane((int)(ft - io[si].ftile_begin));
    b.X0 = lt % ftx * kFinCols;
    b.Y0 = lt / ftx * kFinRows;
    b.Y1 = min(b.Y0 + kFinRows, b.H);
    b.x = b.X0 + 4 * (int)threadIdx.x;
    b.nv = min(4, b.W - b.x);
    b.in = b.nv > 0;
    b.tail = (b.W & 3) && b.W - b.X0 <= kFinCols;
    b.xa = min(b.x, (b.W - 1) & ~3);
    b.xo = min(b.x, b.W - 4);
    b.d = min(b.x - b.xo, 3);
    return b;
}
// a partial quad's missing pixels repeat its last one
__device__ __forceinline__ void fill_quad(int nv, double v[4])
{
    v[1] = nv > 1 ? v[1] : v[0];
    v[2] = nv > 2 ? v[2] : v[1];
    v[3] = nv > 3 ? v[3] : v[2];
}

// --------------------------------------------------------------- prep ---

// b_u = alpha (g_s - g_o) and partial sums of ||alpha g_s + L g_o||^2, ||b_u||^2
// and sum(b_u).  Quad mapping.
template <typename T, typename TS, typename TO>
__global__ __launch_bounds__(256) void prep_kernel(const TS *gs, const TO *go, const SliceIO *io,
                                                   int n_slices, long long n_tiles,
                                                   const LevelDesc *levs, double *part_bb,
                                                   double *part_b0, double *part_bs)
{
    __shared__ double red[4];
    QuadCtx c;
    if (!quad_ctx(io, n_slices, n_tiles, c)) return;
    const SliceIO &P = c.P;
    const LevelDesc &L = levs[P.lev0];
    const int x = c.x, y = c.y, nv = c.row_in ? c.nvalid : 0;
    const double al = P.alpha;
    const long long go_row = P.off_go + (long long)min(y, P.H - 1) * P.pitch_go;
    double o[4], on[4], os[4], sv[4];
    load4(go, go_row + x, nv, o);
    load4(go, go_row - P.pitch_go + x, (y > 0) ? nv : 0, on);
    load4(go, go_row + P.pitch_go + x, (y < P.H - 1) ? nv : 0, os);
    load4(gs, P.off_gs + (long long)min(y, P.H - 1) * P.pitch_gs + x, nv, sv);
    double ol = row_prev(o[3]), orr = row_next(o[0]);
    const int g = threadIdx.x & 15;
    if (nv > 0 && g == 0 && x > 0) ol = (double)go[go_row + x - 1];
    if (nv > 0 && g == 15 && x + nv < P.W) orr = (double)go[go_row + x + nv];
    double sbb = 0.0, sb0 = 0.0, sbs = 0.0, bq[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double l = k == 0 ? ol : o[k - 1], r = k == 3 ? orr : o[k + 1];
        double lap = 0.0;   // (L g_o)_p over in-slice neighbours
        if (x + k > 0) lap += o[k] - l;
        if (x + k < P.W - 1) lap += o[k] - r;
        if (y > 0) lap += o[k] - on[k];
        if (y < P.H - 1) lap += o[k] - os[k];
        const double bf = al * sv[k] + lap;
        const T bu = (T)(al * (sv[k] - o[k]));
        bq[k] = (double)bu;
        if (k < nv) {
            sbb += bf * bf;
            sb0 += (double)bu * (double)bu;
            sbs += (double)bu;
        }
    }
    store4(static_cast<T *>(L.b), (long long)min(y, P.H - 1) * L.pitch + x, nv, bq);
    const double tbb = block_sum(sbb, red);
    const double tb0 = block_sum(sb0, red);
    const double tbs = block_sum(sbs, red);
    if (threadIdx.x == 0) {
        part_bb[c.tile] = tbb;
        part_b0[c.tile] = tb0;
        part_bs[c.tile] = tbs;
    }
}

// The same by row marching (see finalize_kernel): one wave per kFinCols x kFinRows
// block holds g_o's rows y - 1, y, y + 1, so each is read once, and the slice
// lookup and the block's sums are paid once per 16384 pixels instead of per 1024.
// 96 slices of 512 to 4096 a side (510 Mpx, 9 B per pixel): 1.90 ms as quads, 0.85 ms
// (5.4 TB/s) marched.
template <typename T, typename TS, typename TO>
__global__ __launch_bounds__(64) void prep_rows_kernel(const TS *gs_, const TO *go_, const SliceIO *io, int n_slices,
                                                       long long n_ft, const LevelDesc *levs, double *part_bb,
                                                       double *part_b0, double *part_bs)
{
    using VT = typename Vec4<T>::type;
    using VS = typename Vec4U<TS>::type;
    using VO = typename Vec4U<TO>::type;
    constexpr int Q = kFinQ;
    const long long ft = xcd_tile(blockIdx.x, gridDim.x);
    if (ft >= n_ft) return;
    const int si = find_fslice(io, n_slices, ft);
    const RowBlock B = row_block(io, si, ft);
    const int H = B.H, W = B.W, X0 = B.X0, Y0 = B.Y0, Y1 = B.Y1, xa = B.xa, xo = B.xo;
    const bool tail = B.tail;
    const double al = io[si].alpha;
    const long long pb = levs[io[si].lev0].pitch;
    GDF_GLOBAL T *b = (GDF_GLOBAL T *)levs[io[si].lev0].b;
    const long long pitch_gs = io[si].pitch_gs, pitch_go = io[si].pitch_go;
    const GDF_GLOBAL TS *gs = (const GDF_GLOBAL TS *)gs_ + io[si].off_gs;
    const GDF_GLOBAL TO *go = (const GDF_GLOBAL TO *)go_ + io[si].off_go;
    const int lane = threadIdx.x;
    // the wave's outer neighbour columns (lane 0: left, lane 63: right), clamped
    const int xe = min(max(lane == 0 ? X0 - 1 : X0 + kFinCols, 0), W - 1);
    const double ml = B.x > 0 ? 1.0 : 0.0, mr = B.x + 3 < W - 1 ? 1.0 : 0.0;
    auto oquad = [&](int y) -> VO {
        return *reinterpret_cast<const GDF_GLOBAL VO *>(go + (long long)min(max(y, 0), H - 1) * pitch_go + xo);
    };
    auto quad_d = [&](const VO &q, double v[4]) {
        v4_to_d(tail ? shift_down(q, B.d) : q, v);
        if (tail) fill_quad(B.nv, v);
    };
    double on[4], oc[4], os[4];
    quad_d(oquad(Y0 - 1), on);   // (row -1: masked below)
    quad_d(oquad(Y0), oc);
    double oe = (double)go[(long long)Y0 * pitch_go + xe];
    // queue: g_o of row y + 1 (and its outer element), g_s of row y; past the
    // block's last row it re-reads that row
    VO qo[Q];
    VS qs[Q];
    TO qe[Q];
    auto issue = [&](int t, int slot) {
        const int y = min(Y0 + t, Y1 - 1), yn = min(y + 1, H - 1);
        qo[slot] = oquad(yn);
        qe[slot] = go[(long long)yn * pitch_go + xe];
        qs[slot] = *reinterpret_cast<const GDF_GLOBAL VS *>(gs + (long long)y * pitch_gs + xo);
    };
#pragma unroll
    for (int q = 0; q < Q - 1; ++q) issue(q, q);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0) (see finalize_kernel)
    double sbb = 0.0, sb0 = 0.0, sbs = 0.0;
    const int n_rows = Y1 - Y0;
    for (int tb = 0; tb < n_rows; tb += Q) {
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const int t = tb + k;
            issue(t + Q - 1, (k + Q - 1) % Q);
            const int y = Y0 + t;
            const double mu = y > 0 ? 1.0 : 0.0, md = y < H - 1 ? 1.0 : 0.0;   // uniform
            const bool keep = t < n_rows && B.in;
            double sv[4];
            quad_d(qo[k], os);
            v4_to_d(tail ? shift_down(qs[k], B.d) : qs[k], sv);
            const double oe_next = (double)qe[k];
            double ol = wave_prev(oc[3]), orr = wave_next(oc[0]);
            ol = lane == 0 ? oe : ol;
            orr = lane == 63 ? oe : orr;
            VT bv;
            double rbb = 0.0, rb0 = 0.0, rbs = 0.0;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const double l = m == 0 ? ol : oc[m - 1], r = m == 3 ? orr : oc[m + 1];
                double lap = (m == 0 ? ml : 1.0) * (oc[m] - l);   // (L g_o)_p over in-slice neighbours
                lap = fma(m == 3 ? mr : 1.0, oc[m] - r, lap);
                lap = fma(mu, oc[m] - on[m], lap);
                lap = fma(md, oc[m] - os[m], lap);
                const double bf = al * sv[m] + lap;
                const T bu = (T)(al * (sv[m] - oc[m]));
                bv[m] = bu;
                const bool w = !tail || m < B.nv;
                const double bd = w ? (double)bu : 0.0, bfw = w ? bf : 0.0;
                rbb = fma(bfw, bfw, rbb);
                rb0 = fma(bd, bd, rb0);
                rbs += bd;
            }
            sbb += keep ? rbb : 0.0;
            sb0 += keep ? rb0 : 0.0;
            sbs += keep ? rbs : 0.0;
            // (arena rows are padded: a whole quad may be stored past the row's end)
            if (keep) *reinterpret_cast<GDF_GLOBAL VT *>(b + (long long)y * pb + xa) = bv;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                on[m] = oc[m];
                oc[m] = os[m];
            }
            oe = oe_next;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        sbb += __shfl_xor(sbb, off);
        sb0 += __shfl_xor(sb0, off);
        sbs += __shfl_xor(sbs, off);
    }
    if (lane == 0) {
        part_bb[ft] = sbb;
        part_b0[ft] = sb0;
        part_bs[ft] = sbs;
    }
}

template <typename T, typename TS, typename TO>
static hipError_t prep_launch(bool rows, const void *gs, const void *go, const SliceIO *io, int n, long long nt,
                              const LevelDesc *levs, double *pbb, double *pb0, double *pbs, hipStream_t s)
{
    const dim3 g((unsigned)nt);
    if (rows)
        hipLaunchKernelGGL((prep_rows_kernel<T, TS, TO>), g, dim3(64), 0, s, (const TS *)gs, (const TO *)go, io, n, nt,
                           levs, pbb, pb0, pbs);
    else
        hipLaunchKernelGGL((prep_kernel<T, TS, TO>), g, dim3(256), 0, s, (const TS *)gs, (const TO *)go, io, n, nt, levs,
                           pbb, pb0, pbs);
    return hipGetLastError();
}
template <typename T, typename TS>
static hipError_t prep_go(bool rows, int go_dtype, const void *gs, const void *go, const SliceIO *io, int n,
                          long long nt, const LevelDesc *levs, double *pbb, double *pb0, double *pbs, hipStream_t s)
{
    if (go_dtype == 0) return prep_launch<T, TS, uint8_t>(rows, gs, go, io, n, nt, levs, pbb, pb0, pbs, s);
    if (go_dtype == 1) return prep_launch<T, TS, float>(rows, gs, go, io, n, nt, levs, pbb, pb0, pbs, s);
    return prep_launch<T, TS, double>(rows, gs, go, io, n, nt, levs, pbb, pb0, pbs, s);
}

hipError_t launch_prep(bool fp64, bool rows, int gs_dtype, const void *gs, int go_dtype, const void *go,
                       const SliceIO *io_dev, int n_slices, long long n_tiles,
                       const LevelDesc *levs, double *part_bb, double *part_b0, double *part_bs,
                       hipStream_t s)
{
    if (n_tiles <= 0) return hipSuccess;
    if (fp64)
        return gs_dtype == 2 ? prep_go<double, double>(rows, go_dtype, gs, go, io_dev, n_slices, n_tiles, levs, part_bb, part_b0, part_bs, s)
                             : prep_go<double, float>(rows, go_dtype, gs, go, io_dev, n_slices, n_tiles, levs, part_bb, part_b0, part_bs, s);
    return gs_dtype == 2 ? prep_go<float, double>(rows, go_dtype, gs, go, io_dev, n_slices, n_tiles, levs, part_bb, part_b0, part_bs, s)
                         : prep_go<float, float>(rows, go_dtype, gs, go, io_dev, n_slices, n_tiles, levs, part_bb, part_b0, part_bs, s);
}

// ----------------------------------------------------------- finalize ---

// f = g_o + u, and partial sums of the FP64 residual ||b_u - A u||^2 of the
// unrounded g_o + u (A(g_o + u) - (alpha g_s + L g_o) = A u - b_u).  Quad
// mapping: one tile row of four-pixel vectors per thread.
template <typename T, typename TO, typename TF>
__global__ __launch_bounds__(256) void finalize_quad_kernel(const TO *go, TF *f, const SliceIO *io,
                                                       int n_slices, long long n_tiles,
                                                       const LevelDesc *levs,
                                                       const SliceState *st, const int *only,
                                                       double *part_rr)
{
    __shared__ double red[4];
    QuadCtx c;
    if (!quad_ctx(io, n_slices, n_tiles, c)) return;
    if (only && !only[c.si]) return;   // uniform per block: keeps this slice's partial sum
    const SliceIO &P = c.P;
    const LevelDesc &L = levs[P.lev0];
    const int x = c.x, y = c.y, nv = c.row_in ? c.nvalid : 0;
    const double sg = P.alpha;
    const RBView<T> u(static_cast<const T *>(L.u[st[c.si].cycles & 1]), L.pitch);
    const T *bu = static_cast<const T *>(L.b);
    // full correction = uoff (mean removed on load) + u + shift (constant-mode
    // correction); constants cancel in L, and b is used as stored
    const double shift = st[c.si].shift + st[c.si].uoff;
    const long long pu = L.pitch;
    const int yc = min(y, P.H - 1);   // clamped row: loads stay in the slice
    const long long p = (long long)yc * pu + x;
    double uc[4], un[4], us[4], bb[4];
    u.quad(x, yc, nv, uc);
    load4(bu, p, nv, bb);
    u.quad(x, yc - 1, (y > 0) ? nv : 0, un);
    u.quad(x, yc + 1, (y < P.H - 1) ? nv : 0, us);
    // horizontal neighbours of the quad's first and last pixel
    double ul = row_prev(uc[3]), ur = row_next(uc[0]);
    const int g = threadIdx.x & 15;
    if (nv > 0 && g == 0 && x > 0) ul = u.at(x - 1, yc);
    if (nv > 0 && (g == 15 || nv < 4) && x + nv < P.W) ur = u.at(x + nv, yc);
    double srr = 0.0, o[4], fo[4];
    load4(go, P.off_go + (long long)y * P.pitch_go + x, nv, o);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double l = k == 0 ? ul : uc[k - 1], r = k == 3 ? ur : uc[k + 1];
        double acc = 0.0;
        if (x + k > 0) acc += uc[k] - l;
        if (x + k < P.W - 1) acc += uc[k] - r;
        if (y > 0) acc += uc[k] - un[k];
        if (y < P.H - 1) acc += uc[k] - us[k];
        const double res = bb[k] - sg * (uc[k] + shift) - acc;
        if (k < nv) srr += res * res;
        fo[k] = o[k] + (uc[k] + shift);
    }
    store4(f, P.off_f + (long long)y * P.pitch_f + x, nv, fo);
    const double t = block_sum(srr, red);
    if (threadIdx.x == 0) part_rr[c.tile] = t;
}

// Row-marching passes (every width at least 4).  g_o, g_s and f rows may start
// on any element: their quads are moved with accesses that need no more than
// element alignment (one instruction either way), and where a row ends inside a
// lane's quad (nv < 4 pixels) the lane loads the row's last four pixels and
// shifts them down.  33 x 1021 x 1531 (nothing aligned): the quad pass took 254 us, this 148.
//
// The output pass.  One wave owns a block of kFinCols columns (four
// per lane) by kFinRows rows and walks down it holding the iterate's rows
// y - 1, y, y + 1, so every row is read once; the loads of the next rows are
// in flight kFinQ - 1 rows ahead.  The wave's two outer horizontal neighbours
// come from one extra element per row; the others cross lanes by DPP.
template <typename T, typename TO, typename TF>
__global__ __launch_bounds__(64) void finalize_kernel(const TO *go_, TF *f_, const SliceIO *io, int n_slices,
                                                      long long n_ft, const LevelDesc *levs,
                                                      const SliceState *st, const int *only, double *part_rr)
{
    using VT = typename Vec4<T>::type;
    using VO = typename Vec4U<TO>::type;
    using VF = typename Vec4U<TF>::type;
    constexpr int Q = kFinQ;
    const long long ft = xcd_tile(blockIdx.x, gridDim.x);
    if (ft >= n_ft) return;
    const int si = find_fslice(io, n_slices, ft);
    if (only && !only[si]) return;   // uniform per wave: keeps this slice's partial sum
    // the slice's fields as wave-uniform scalars (stores to f cannot alias them)
    const RowBlock B = row_block(io, si, ft);
    const int H = B.H, W = B.W, X0 = B.X0, Y0 = B.Y0, Y1 = B.Y1, x = B.x, xa = B.xa, xo = B.xo;
    const bool in = B.in, tail = B.tail;
    const long long off_go = io[si].off_go, pitch_go = io[si].pitch_go;
    const long long off_f = io[si].off_f, pitch_f = io[si].pitch_f;
    const double sg = io[si].alpha;
    const LevelDesc &L = levs[io[si].lev0];
    const long long pu = L.pitch;
    const GDF_GLOBAL T *u = (const GDF_GLOBAL T *)L.u[st[si].cycles & 1];
    const GDF_GLOBAL T *bu = (const GDF_GLOBAL T *)L.b;
    const GDF_GLOBAL TO *go = (const GDF_GLOBAL TO *)go_;
    GDF_GLOBAL TF *f = (GDF_GLOBAL TF *)f_;
    // full correction = uoff (mean removed on load) + u + shift (constant-mode
    // correction); constants cancel in L, and b is used as stored
    const double shift = st[si].shift + st[si].uoff;

    const int lane = threadIdx.x;
    // the wave's outer neighbour columns (lane 0: left, lane 63: right), clamped
    const int xe = min(max(lane == 0 ? X0 - 1 : X0 + kFinCols, 0), W - 1);
    // horizontal neighbour masks of the quad's first and last pixel
    const double ml = x > 0 ? 1.0 : 0.0, mr = x + 3 < W - 1 ? 1.0 : 0.0;
    // The iterate stores each row by colour (LevelDesc): pixel (x, y) at
    // element x / 2 of the half (x + y) & 1 of row y (halves pu / 2 long).  A
    // lane's quad (xa a multiple of 4) is two pairs: pixels xa, xa + 2 of one
    // colour and xa + 1, xa + 3 of the other.  Rows are clamped into the slice;
    // arena rows are multiples of 64 elements, so a pair never leaves its half.
    using VT2 = typename Vec2<T>::type;
    const long long pu2 = pu >> 1;
    auto uat = [&](int x, int y) -> T {
        const int yc = min(max(y, 0), H - 1);
        return u[(long long)yc * pu + ((x + yc) & 1) * pu2 + (x >> 1)];
    };
    auto uquad = [&](int y, VT2 &ev, VT2 &od) {   // the colours of pixels xa (ev) and xa + 1 (od)
        const int yc = min(max(y, 0), H - 1);
        const GDF_GLOBAL T *r0 = u + (long long)yc * pu + (xa >> 1);
        ev = *reinterpret_cast<const GDF_GLOBAL VT2 *>((yc & 1) ? r0 + pu2 : r0);
        od = *reinterpret_cast<const GDF_GLOBAL VT2 *>((yc & 1) ? r0 : r0 + pu2);
    };
    auto quad_d = [&](const VT2 &ev, const VT2 &od, double v[4]) {
        v[0] = (double)ev.x;
        v[1] = (double)od.x;
        v[2] = (double)ev.y;
        v[3] = (double)od.y;
        // (past the row's end: the last pixel again, so its difference is zero)
        if (tail) fill_quad(B.nv, v);
    };

    double un[4], uc[4], us[4];
    {
        VT2 ev, od;
        uquad(Y0 - 1, ev, od);   // (row -1: masked below)
        quad_d(ev, od, un);
        uquad(Y0, ev, od);
        quad_d(ev, od, uc);
    }
    double ue = (double)uat(xe, Y0);

    // queue: u of row y + 1 (and its outer element), b and g_o of row y; past
    // the block's last row the queue re-reads that row (cache hits, unused)
    VT2 qev[Q], qod[Q];
    VT qb[Q];
    VO qo[Q];
    T qe[Q];
    auto issue = [&](int t, int slot) {
        const int y = min(Y0 + t, Y1 - 1);
        uquad(y + 1, qev[slot], qod[slot]);
        qe[slot] = uat(xe, y + 1);
        qb[slot] = *reinterpret_cast<const GDF_GLOBAL VT *>(bu + (long long)y * pu + xa);
        qo[slot] = *reinterpret_cast<const GDF_GLOBAL VO *>(go + off_go + (long long)y * pitch_go + xo);
    };
#pragma unroll
    for (int q = 0; q < Q - 1; ++q) issue(q, q);
    // one full wait here, so the wait at the head of the row loop (which merges
    // the entry with the back edge) stays partial
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)

    double srr = 0.0;
    const int n_rows = Y1 - Y0;
    for (int tb = 0; tb < n_rows; tb += Q) {
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const int t = tb + k;
            issue(t + Q - 1, (k + Q - 1) % Q);
            const int y = Y0 + t;
            const double mu = y > 0 ? 1.0 : 0.0, md = y < H - 1 ? 1.0 : 0.0;   // uniform
            const bool keep = t < n_rows && in;
            double bb[4], o[4];
            quad_d(qev[k], qod[k], us);
            v4_to_d(qb[k], bb);
            v4_to_d(tail ? shift_down(qo[k], B.d) : qo[k], o);
            const double ue_next = (double)qe[k];
            double ul = wave_prev(uc[3]), ur = wave_next(uc[0]);
            ul = lane == 0 ? ue : ul;
            ur = lane == 63 ? ue : ur;
            VF fv;
            double rr = 0.0;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const double l = m == 0 ? ul : uc[m - 1], r = m == 3 ? ur : uc[m + 1];
                const double kl = m == 0 ? ml : 1.0, kr = m == 3 ? mr : 1.0;
                double acc = kl * (uc[m] - l);
                acc = fma(kr, uc[m] - r, acc);
                acc = fma(mu, uc[m] - un[m], acc);
                acc = fma(md, uc[m] - us[m], acc);
                // (past the row's end b is row padding, which may hold anything, NaN too:
                // taken out by selection, here and for lanes past it, not by a factor zero)
                const double res = tail && m >= B.nv ? 0.0 : bb[m] - sg * (uc[m] + shift) - acc;
                rr = fma(res, res, rr);
                fv[m] = (TF)(o[m] + (uc[m] + shift));
            }
            srr += keep ? rr : 0.0;
            if (keep) {
                GDF_GLOBAL TF *fp = f + off_f + (long long)y * pitch_f + x;
                if (!tail || B.nv == 4) {
                    *reinterpret_cast<GDF_GLOBAL VF *>(fp) = fv;
                } else {
                    fp[0] = fv.x;
                    if (B.nv > 1) fp[1] = fv.y;
                    if (B.nv > 2) fp[2] = fv.z;
                }
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                un[m] = uc[m];
                uc[m] = us[m];
            }
            ue = ue_next;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) srr += __shfl_xor(srr, off);
    if (lane == 0) part_rr[ft] = srr;
}

template <typename T, typename TO>
static hipError_t fin_go(bool rows, int out_dtype, const void *go, void *f, const SliceIO *io, int n,
                         long long nt, const LevelDesc *levs, const SliceState *st, const int *only,
                         double *prr, hipStream_t s)
{
    if (rows) {
        const dim3 g((unsigned)nt), blk(64);
        if (out_dtype == 2)
            hipLaunchKernelGGL((finalize_kernel<T, TO, double>), g, blk, 0, s, (const TO *)go, (double *)f, io, n, nt, levs, st, only, prr);
        else
            hipLaunchKernelGGL((finalize_kernel<T, TO, float>), g, blk, 0, s, (const TO *)go, (float *)f, io, n, nt, levs, st, only, prr);
    } else {
        const dim3 g((unsigned)nt), blk(256);
        if (out_dtype == 2)
            hipLaunchKernelGGL((finalize_quad_kernel<T, TO, double>), g, blk, 0, s, (const TO *)go, (double *)f, io, n, nt, levs, st, only, prr);
        else
            hipLaunchKernelGGL((finalize_quad_kernel<T, TO, float>), g, blk, 0, s, (const TO *)go, (float *)f, io, n, nt, levs, st, only, prr);
    }
    return hipGetLastError();
}

hipError_t launch_finalize(bool fp64, bool rows, int go_dtype, const void *go, int out_dtype, void *f,
                           const SliceIO *io_dev, int n, long long n_tiles,
                           const LevelDesc *levs, const SliceState *st, const int *only,
                           double *part_rr, hipStream_t s)
{
    if (n_tiles <= 0) return hipSuccess;
    if (fp64) {
        if (go_dtype == 0) return fin_go<double, uint8_t>(rows, out_dtype, go, f, io_dev, n, n_tiles, levs, st, only, part_rr, s);
        if (go_dtype == 1) return fin_go<double, float>(rows, out_dtype, go, f, io_dev, n, n_tiles, levs, st, only, part_rr, s);
        return fin_go<double, double>(rows, out_dtype, go, f, io_dev, n, n_tiles, levs, st, only, part_rr, s);
    }
    if (go_dtype == 0) return fin_go<float, uint8_t>(rows, out_dtype, go, f, io_dev, n, n_tiles, levs, st, only, part_rr, s);
    if (go_dtype == 1) return fin_go<float, float>(rows, out_dtype, go, f, io_dev, n, n_tiles, levs, st, only, part_rr, s);
    return fin_go<float, double>(rows, out_dtype, go, f, io_dev, n, n_tiles, levs, st, only, part_rr, s);
}

// ------------------------------------------------------------ adjoint ---
//
// These kernels use the quad mapping (four pixels of one tile row per thread).

template <typename T>
__global__ __launch_bounds__(256) void prep_adjoint_kernel(const T *gf, const SliceIO *io, int n,
                                                           long long n_tiles, const LevelDesc *levs,
                                                           double *part_bb, double *part_bs)
{
    __shared__ double red[4];
    QuadCtx c;
    if (!quad_ctx(io, n, n_tiles, c)) return;
    const SliceIO &P = c.P;
    const LevelDesc &L = levs[P.lev0];
    const int y = min(c.y, P.H - 1), nv = c.row_in ? c.nvalid : 0;
    double v[4];
    load4(gf, P.off_f + (long long)y * P.pitch_f + c.x, nv, v);
    store4(static_cast<T *>(L.b), (long long)y * L.pitch + c.x, nv, v);
    double sbb = 0.0, sbs = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {   // elements past nv are 0
        sbb += v[k] * v[k];
        sbs += v[k];
    }
    const double t = block_sum(sbb, red);
    const double t2 = block_sum(sbs, red);
    if (threadIdx.x == 0) {
        part_bb[c.tile] = t;
        part_bs[c.tile] = t2;
    }
}

hipError_t launch_prep_adjoint(bool fp64, const void *grad_f, const SliceIO *io_dev, int n,
                               long long n_tiles, const LevelDesc *levs, double *part_bb,
                               double *part_bs, hipStream_t s)
{
    if (n_tiles <= 0) return hipSuccess;
    if (fp64)
        hipLaunchKernelGGL(prep_adjoint_kernel<double>, dim3((unsigned)n_tiles), dim3(256), 0, s, (const double *)grad_f, io_dev, n, n_tiles, levs, part_bb, part_bs);
    else
        hipLaunchKernelGGL(prep_adjoint_kernel<float>, dim3((unsigned)n_tiles), dim3(256), 0, s, (const float *)grad_f, io_dev, n, n_tiles, levs, part_bb, part_bs);
    return hipGetLastError();
}

// The quad of level-0 values at row y and its four-neighbour sums: c (the
// quad), and sum over in-slice neighbours q of (c_k - v_q).
template <typename View>
__device__ __forceinline__ void quad_lap(const View &v, const QuadCtx &q, int nv, double c[4], double lap[4])
{
    const int x = q.x, y = min(q.y, q.P.H - 1), H = q.P.H, W = q.P.W;
    double n[4], s[4];
    v.quad(x, y, nv, c);
    v.quad(x, y - 1, y > 0 ? nv : 0, n);
    v.quad(x, y + 1, y < H - 1 ? nv : 0, s);
    double l = row_prev(c[3]), r = row_next(c[0]);
    const int g = threadIdx.x & 15;
    if (nv > 0 && g == 0 && x > 0) l = v.at(x - 1, y);
    if (nv > 0 && g == 15 && x + nv < W) r = v.at(x + nv, y);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double vl = k == 0 ? l : c[k - 1], vr = k == 3 ? r : c[k + 1];
        double acc = 0.0;
        if (x + k > 0) acc += c[k] - vl;
        if (x + k < W - 1) acc += c[k] - vr;
        if (y > 0) acc += c[k] - n[k];
        if (y < H - 1) acc += c[k] - s[k];
        lap[k] = acc;
    }
}

// lambda = A^{-1} grad_f (level-0 iterate): grad_gs = alpha lambda,
// grad_go = L lambda, partials of lambda . (g_s - f).
template <typename T, typename View>
__device__ __forceinline__ void adjoint_quad(const View &lam, double shift, const T *gs, const T *f, T *ggs,
                                             T *ggo, const QuadCtx &q, bool need_da, double &sda)
{
    const SliceIO &P = q.P;
    const int nv = q.row_in ? q.nvalid : 0;
    const int y = min(q.y, P.H - 1);
    double lc[4], lap[4], g[4], fv[4], og[4], oo[4];
    quad_lap(lam, q, nv, lc, lap);   // L is blind to the constant shift
    const long long fo = P.off_f + (long long)y * P.pitch_f + q.x;
    load4(gs, P.off_gs + (long long)y * P.pitch_gs + q.x, need_da ? nv : 0, g);   // (zeros unless read)
    load4(f, fo, need_da ? nv : 0, fv);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double l = lc[k] + shift;
        og[k] = P.alpha * l;
        oo[k] = lap[k];
        if (k < nv) sda += l * (g[k] - fv[k]);
    }
    if (ggs) store4(ggs, fo, nv, og);
    if (ggo) store4(ggo, fo, nv, oo);
}

template <typename T>
__global__ __launch_bounds__(256) void adjoint_kernel(const T *gs, const T *f, T *ggs, T *ggo,
                                                      const SliceIO *io, int n, long long n_tiles,
                                                      const LevelDesc *levs, const SliceState *st,
                                                      double *const *u64, double *part_da)
{
    __shared__ double red[4];
    QuadCtx c;
    if (!quad_ctx(io, n, n_tiles, c)) return;
    const SliceIO &P = c.P;
    const LevelDesc &L = levs[P.lev0];
    const int cycles = st[c.si].cycles, par = cycles & 1;
    const bool need_da = part_da != nullptr;
    double sda = 0.0;
    if (u64) {   // (no refinement step: still zero, and never written)
        adjoint_quad<T>(RowView<double>(cycles ? u64[par * n + c.si] : nullptr, L.pitch), 0.0, gs, f, ggs, ggo, c,
                        need_da, sda);
    } else {
        const RBView<T> lam(static_cast<const T *>(L.u[par]), L.pitch);
        const double shift = st[c.si].shift + st[c.si].uoff;   // constant parts of lambda
        adjoint_quad<T>(lam, shift, gs, f, ggs, ggo, c, need_da, sda);
    }
    if (!need_da) return;
    const double t = block_sum(sda, red);
    if (threadIdx.x == 0) part_da[c.tile] = t;
}

hipError_t launch_adjoint_assemble(bool fp64, const void *gs, const void *f, void *ggs, void *ggo,
                                   const SliceIO *io_dev, int n, long long n_tiles,
                                   const LevelDesc *levs, const SliceState *st, double *const *u64,
                                   double *part_da, hipStream_t s)
{
    if (n_tiles <= 0) return hipSuccess;
    if (fp64)
        hipLaunchKernelGGL(adjoint_kernel<double>, dim3((unsigned)n_tiles), dim3(256), 0, s, (const double *)gs, (const double *)f, (double *)ggs, (double *)ggo, io_dev, n, n_tiles, levs, st, u64, part_da);
    else
        hipLaunchKernelGGL(adjoint_kernel<float>, dim3((unsigned)n_tiles), dim3(256), 0, s, (const float *)gs, (const float *)f, (float *)ggs, (float *)ggo, io_dev, n, n_tiles, levs, st, u64, part_da);
    return hipGetLastError();
}

// ---------------------------------------------------- mixed refinement ---

// u64_out = u64_in + e (e: the FP32 correction of the last inner solve; u64_in is
// zero in the first step, and not read), then the FP64 residual of u64_out stored as
// the FP32 right-hand side of the next inner solve, and its squared norm.
template <typename TS, typename TO>
__global__ __launch_bounds__(256) void refine_kernel(RefineArgs a)
{
    __shared__ double red[4];
    QuadCtx c;
    if (!quad_ctx(a.io, a.n_slices, a.n_tiles, c)) return;
    const SliceIO &P = c.P;
    double srr = 0.0;
    if (a.active[c.si]) {   // uniform per block
        const LevelDesc &L = a.levs[P.lev0];
        const long long pl = L.pitch;
        const int x = c.x, y = min(c.y, P.H - 1), H = P.H, W = P.W;
        const int nv = c.row_in ? c.nvalid : 0;
        const double *uin = a.u64[a.in_sel * a.n_slices + c.si];
        double *uout = a.u64[(a.in_sel ^ 1) * a.n_slices + c.si];
        const RBView<float> e(static_cast<const float *>(L.u[a.e_sel]), pl);
        const long long p = (long long)y * pl + x;
        // new iterate on the quad and its four neighbour rows / columns
        double uc[4], un[4], us[4], t0[4], t1[4];
        double ul = 0.0, ur = 0.0;
        const RowView<double> u0(a.first ? nullptr : uin, pl);
        u0.quad(x, y, nv, uc);
        e.quad(x, y, nv, t0);
        u0.quad(x, y - 1, y > 0 ? nv : 0, un);
        e.quad(x, y - 1, y > 0 ? nv : 0, t1);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uc[k] += t0[k];
            un[k] += t1[k];
        }
        u0.quad(x, y + 1, y < H - 1 ? nv : 0, us);
        e.quad(x, y + 1, y < H - 1 ? nv : 0, t1);
#pragma unroll
        for (int k = 0; k < 4; ++k) us[k] += t1[k];
        ul = row_prev(uc[3]);
        ur = row_next(uc[0]);
        const int g = threadIdx.x & 15;
        if (nv > 0 && g == 0 && x > 0) ul = u0.at(x - 1, y) + e.at(x - 1, y);
        if (nv > 0 && g == 15 && x + nv < W) ur = u0.at(x + nv, y) + e.at(x + nv, y);
        double bv[4];
        if (a.rhs) {
            load4(static_cast<const TS *>(a.rhs), P.off_f + (long long)y * P.pitch_f + x, nv, bv);
        } else {
            double sv[4], o[4];
            load4(static_cast<const TS *>(a.gs), P.off_gs + (long long)y * P.pitch_gs + x, nv, sv);
            load4(static_cast<const TO *>(a.go), P.off_go + (long long)y * P.pitch_go + x, nv, o);
#pragma unroll
            for (int k = 0; k < 4; ++k) bv[k] = P.alpha * (sv[k] - o[k]);
        }
        double res[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double vl = k == 0 ? ul : uc[k - 1], vr = k == 3 ? ur : uc[k + 1];
            double acc = 0.0;
            if (x + k > 0) acc += uc[k] - vl;
            if (x + k < W - 1) acc += uc[k] - vr;
            if (y > 0) acc += uc[k] - un[k];
            if (y < H - 1) acc += uc[k] - us[k];
            res[k] = bv[k] - P.alpha * uc[k] - acc;
            if (k < nv) srr += res[k] * res[k];
        }
        store4(uout, p, nv, uc);
        store4(static_cast<float *>(L.b), p, nv, res);
    }
    const double t = block_sum(srr, red);
    if (threadIdx.x == 0) a.part_rr[c.tile] = t;
}

// The same by row marching (see finalize_kernel): the new iterate's rows y - 1, y,
// y + 1 are held in registers, so every row of u64 and e is read once.  The quad
// kernel reads each three times, from L2 where it is still there: 2 x 21504 x
// 26624, 29 bytes per pixel (21 in the first step): 8.3 + 7.1 ms as quads, 6.8 + 5.0
// (4.9 TB/s) marched.  It also restricts the residual to level 1, whose cells are
// two columns of a lane by two consecutive rows: the solve's own restriction pass
// read it again (4.5 bytes per pixel, 1.1 ms there).  FIRST: u64_in is zero.  RHS: the
// right-hand side is a.rhs.
template <typename TS, typename TO, bool RHS, bool FIRST>
__global__ __launch_bounds__(64) void refine_rows_kernel(RefineArgs a)
{
    using VD = typename Vec4<double>::type;
    using VF = typename Vec4<float>::type;
    using V2 = typename Vec2<float>::type;
    using VS = typename Vec4U<TS>::type;
    using VO = typename Vec4U<TO>::type;
    constexpr int Q = kFinQ;
    const long long ft = xcd_tile(blockIdx.x, gridDim.x);
    if (ft >= a.n_tiles) return;
    const int si = find_fslice(a.io, a.n_slices, ft), lane = threadIdx.x;
    if (!a.active[si]) {   // uniform
        if (lane == 0) a.part_rr[ft] = 0.0;
        return;
    }
    const RowBlock B = row_block(a.io, si, ft);
    const SliceIO &P = a.io[si];
    const int H = B.H, W = B.W, X0 = B.X0, Y0 = B.Y0, Y1 = B.Y1, x = B.x, xa = B.xa, xo = B.xo;
    const bool tail = B.tail;
    const double al = P.alpha;
    const LevelDesc &L = a.levs[P.lev0];
    const long long pl = L.pitch, pl2 = pl >> 1;
    const GDF_GLOBAL float *e = (const GDF_GLOBAL float *)(a.e_sel ? L.u[1] : L.u[0]);
    GDF_GLOBAL float *b = (GDF_GLOBAL float *)L.b;
    const GDF_GLOBAL double *uin = (const GDF_GLOBAL double *)a.u64[a.in_sel * a.n_slices + si];
    GDF_GLOBAL double *uout = (GDF_GLOBAL double *)a.u64[(a.in_sel ^ 1) * a.n_slices + si];
    const long long pitch_s = RHS ? P.pitch_f : P.pitch_gs, pitch_go = P.pitch_go;
    const GDF_GLOBAL TS *src = (const GDF_GLOBAL TS *)(RHS ? a.rhs : a.gs) + (RHS ? P.off_f : P.off_gs);
    const GDF_GLOBAL TO *go = (const GDF_GLOBAL TO *)a.go + P.off_go;
    // the wave's outer neighbour columns (lane 0: left, lane 63: right), clamped
    const int xe = min(max(lane == 0 ? X0 - 1 : X0 + kFinCols, 0), W - 1);
    const double ml = x > 0 ? 1.0 : 0.0, mr = x + 3 < W - 1 ? 1.0 : 0.0;
    // raw loads of one row of the iterate (rows clamped into the slice; e is stored
    // by colour, see finalize_kernel), and the new iterate's values from them
    struct Row {
        VD u;
        V2 ev, od;
        double ue;
        float ee;
    };
    auto load_row = [&](int y, Row &q) {
        const int yc = min(max(y, 0), H - 1);
        const GDF_GLOBAL float *r0 = e + (long long)yc * pl;
        q.ev = *reinterpret_cast<const GDF_GLOBAL V2 *>(r0 + ((yc & 1) ? pl2 : 0) + (xa >> 1));
        q.od = *reinterpret_cast<const GDF_GLOBAL V2 *>(r0 + ((yc & 1) ? 0 : pl2) + (xa >> 1));
        q.ee = r0[((xe + yc) & 1) * pl2 + (xe >> 1)];
        if constexpr (!FIRST) {
            q.u = *reinterpret_cast<const GDF_GLOBAL VD *>(uin + (long long)yc * pl + xa);
            q.ue = uin[(long long)yc * pl + xe];
        }
    };
    auto row_values = [&](const Row &q, double v[4], double &ve) {
        v[0] = (double)q.ev.x;
        v[1] = (double)q.od.x;
        v[2] = (double)q.ev.y;
        v[3] = (double)q.od.y;
        ve = (double)q.ee;
        if constexpr (!FIRST) {
            v[0] += q.u.x;
            v[1] += q.u.y;
            v[2] += q.u.z;
            v[3] += q.u.w;
            ve += q.ue;
        }
        if (tail) fill_quad(B.nv, v);   // (past the row's end: its last pixel, so their difference is zero)
    };
    double un[4], uc[4], us[4], ue, t;
    {
        Row q;
        load_row(Y0 - 1, q);   // (row -1: masked below)
        row_values(q, un, t);
        load_row(Y0, q);
        row_values(q, uc, ue);
    }
    Row qr[Q];
    VS qs[Q];
    VO qo[Q];
    auto issue = [&](int t, int slot) {
        const int y = min(Y0 + t, Y1 - 1);
        load_row(y + 1, qr[slot]);
        qs[slot] = *reinterpret_cast<const GDF_GLOBAL VS *>(src + (long long)y * pitch_s + xo);
        if constexpr (!RHS) qo[slot] = *reinterpret_cast<const GDF_GLOBAL VO *>(go + (long long)y * pitch_go + xo);
    };
#pragma unroll
    for (int q = 0; q < Q - 1; ++q) issue(q, q);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0) (see finalize_kernel)
    double srr = 0.0;
    const int n_rows = Y1 - Y0;
    // level 1's right-hand side (null without one): the sums of each cell's children
    GDF_GLOBAL unsigned short *bc = (GDF_GLOBAL unsigned short *)L.bc;
    const long long pc = L.pitch_c;
    static_assert(kFinRows % 2 == 0 && Q % 2 == 0, "a block starts on an even row; row parities are static");
    float c0 = 0.f, c1 = 0.f;   // the cells' first rows
    typedef float F2 __attribute__((ext_vector_type(2)));
    typedef __bf16 BF2 __attribute__((ext_vector_type(2)));
    for (int tb = 0; tb < n_rows; tb += Q) {
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const int r = tb + k;
            issue(r + Q - 1, (k + Q - 1) % Q);
            const int y = Y0 + r;
            const double mu = y > 0 ? 1.0 : 0.0, md = y < H - 1 ? 1.0 : 0.0;   // uniform
            const bool keep = r < n_rows && B.in;
            double ue_next, bv[4];
            row_values(qr[k], us, ue_next);
            v4_to_d(tail ? shift_down(qs[k], B.d) : qs[k], bv);
            if constexpr (!RHS) {
                double o[4];
                v4_to_d(tail ? shift_down(qo[k], B.d) : qo[k], o);
#pragma unroll
                for (int m = 0; m < 4; ++m) bv[m] = al * (bv[m] - o[m]);
            }
            double ul = wave_prev(uc[3]), ur = wave_next(uc[0]);
            ul = lane == 0 ? ue : ul;
            ur = lane == 63 ? ue : ur;
            VF rv;
            double rr = 0.0;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const double l = m == 0 ? ul : uc[m - 1], rt = m == 3 ? ur : uc[m + 1];
                double acc = (m == 0 ? ml : 1.0) * (uc[m] - l);
                acc = fma(m == 3 ? mr : 1.0, uc[m] - rt, acc);
                acc = fma(mu, uc[m] - un[m], acc);
                acc = fma(md, uc[m] - us[m], acc);
                const double res = bv[m] - al * uc[m] - acc;
                rv[m] = (float)res;
                const double rs = tail && m >= B.nv ? 0.0 : res;
                rr = fma(rs, rs, rr);
            }
            srr += keep ? rr : 0.0;
            if (keep) {   // (arena rows are padded: whole quads may be stored past the row's end)
                *reinterpret_cast<GDF_GLOBAL VD *>(uout + (long long)y * pl + xa) = VD{uc[0], uc[1], uc[2], uc[3]};
                *reinterpret_cast<GDF_GLOBAL VF *>(b + (long long)y * pl + xa) = rv;
                // (pixels past the row's end add nothing)
                const float s0 = rv.x + (tail && B.nv < 2 ? 0.f : rv.y);
                const float s1 = (tail && B.nv < 3 ? 0.f : rv.z) + (tail && B.nv < 4 ? 0.f : rv.w);
                c0 = (k & 1) ? c0 + s0 : s0;
                c1 = (k & 1) ? c1 + s1 : s1;
                // (the last row may be the only one of its cells; rows of level 1 are padded)
                if (bc && ((k & 1) || y == H - 1))
                    *reinterpret_cast<GDF_GLOBAL unsigned *>(bc + (long long)(y >> 1) * pc + (xa >> 1)) =
                        __builtin_bit_cast(unsigned, __builtin_convertvector((F2{c0, c1}), BF2));
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                un[m] = uc[m];
                uc[m] = us[m];
            }
            ue = ue_next;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) srr += __shfl_xor(srr, off);
    if (lane == 0) a.part_rr[ft] = srr;
}

template <typename TS, typename TO, bool RHS>
static hipError_t refine_rows(const RefineArgs &a, hipStream_t s)
{
    const dim3 g((unsigned)a.n_tiles);
    if (a.first) hipLaunchKernelGGL((refine_rows_kernel<TS, TO, RHS, true>), g, dim3(64), 0, s, a);
    else hipLaunchKernelGGL((refine_rows_kernel<TS, TO, RHS, false>), g, dim3(64), 0, s, a);
    return hipGetLastError();
}
template <typename TS> static hipError_t refine_rows_t(const RefineArgs &a, hipStream_t s)
{
    if (a.rhs) return refine_rows<TS, uint8_t, true>(a, s);   // (g_o is not read)
    return a.go_dtype == 0 ? refine_rows<TS, uint8_t, false>(a, s)
         : a.go_dtype == 1 ? refine_rows<TS, float, false>(a, s) : refine_rows<TS, double, false>(a, s);
}

hipError_t launch_refine(const RefineArgs &a, hipStream_t s)
{
    if (a.n_tiles <= 0) return hipSuccess;
    if (a.rows) return a.gs_dtype == 2 ? refine_rows_t<double>(a, s) : refine_rows_t<float>(a, s);
    const dim3 g((unsigned)a.n_tiles), b(256);
    const bool s64 = a.gs_dtype == 2;
    switch (a.go_dtype) {
    case 0:
        if (s64) hipLaunchKernelGGL((refine_kernel<double, uint8_t>), g, b, 0, s, a);
        else hipLaunchKernelGGL((refine_kernel<float, uint8_t>), g, b, 0, s, a);
        break;
    case 1:
        if (s64) hipLaunchKernelGGL((refine_kernel<double, float>), g, b, 0, s, a);
        else hipLaunchKernelGGL((refine_kernel<float, float>), g, b, 0, s, a);
        break;
    default:
        if (s64) hipLaunchKernelGGL((refine_kernel<double, double>), g, b, 0, s, a);
        else hipLaunchKernelGGL((refine_kernel<float, double>), g, b, 0, s, a);
        break;
    }
    return hipGetLastError();
}

template <typename TO, typename TF>
__global__ __launch_bounds__(256) void finalize64_kernel(const TO *go, TF *f, const SliceIO *io,
                                                         int n, long long n_tiles,
                                                         double *const *u64, const SliceState *st,
                                                         const LevelDesc *levs)
{
    QuadCtx c;
    if (!quad_ctx(io, n, n_tiles, c)) return;
    const SliceIO &P = c.P;
    // latest FP64 iterate (no refinement step: still zero, and never written)
    const int cycles = st[c.si].cycles;
    const RowView<double> u(cycles ? u64[(cycles & 1) * n + c.si] : nullptr, levs[P.lev0].pitch);
    const int y = min(c.y, P.H - 1), nv = c.row_in ? c.nvalid : 0;
    double o[4], uv[4];
    load4(go, P.off_go + (long long)y * P.pitch_go + c.x, nv, o);
    u.quad(c.x, y, nv, uv);
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] += uv[k];
    store4(f, P.off_f + (long long)y * P.pitch_f + c.x, nv, o);
}

hipError_t launch_finalize64(int go_dtype, const void *go, int out_dtype, void *f,
                             const SliceIO *io, int n, long long nt, double *const *u64,
                             const SliceState *st, const LevelDesc *levs, hipStream_t s)
{
    if (nt <= 0) return hipSuccess;
    const dim3 g((unsigned)nt), b(256);
#define GDF_F64(TO, TF) hipLaunchKernelGGL((finalize64_kernel<TO, TF>), g, b, 0, s, (const TO *)go, (TF *)f, io, n, nt, u64, st, levs)
    if (out_dtype == 2) {
        if (go_dtype == 0) GDF_F64(uint8_t, double); else if (go_dtype == 1) GDF_F64(float, double); else GDF_F64(double, double);
    } else {
        if (go_dtype == 0) GDF_F64(uint8_t, float); else if (go_dtype == 1) GDF_F64(float, float); else GDF_F64(double, float);
    }
#undef GDF_F64
    return hipGetLastError();
}

}  // namespace gdf
