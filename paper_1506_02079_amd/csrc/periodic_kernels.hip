// Kernels around the per-slice screened-Poisson solve of Eq. (1) with periodic
// (wrap-around) boundaries: the paper's own Fourier basis (Section III-B,
// frequency-space interpretation), where the grid Laplacian couples the
// first and last row and column of a slice.
//
// These are the per-pixel passes around the multigrid, whose own passes are in
// block_kernels.hip: right-hand side, output with its FP64 residual, mixed
// refinement and adjoint assembly.  Every kernel walks 64 x 16 tiles
// of level 0 with 256 threads, one column each, four rows per thread;
// per-tile partial sums are FP64.
#include "internal.h"

namespace gdf {

namespace {

__device__ double pblock_sum(double v, double *red)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    const double r = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
    return r;
}

constexpr int kPTileW = 64, kPTileH = 16, kPRows = kPTileH / 4;   // tile, rows per thread

// the tile of this workgroup: its slice and origin
struct PTile {
    int slice, x0, y0;
};
__device__ __forceinline__ PTile ptile(const PLaunch &a, const SliceIO *io)
{
    const int slice = a.slice_of[blockIdx.x];
    const int lt = (int)(blockIdx.x - io[slice].tile_begin), nx = io[slice].tiles_x;
    return PTile{slice, lt % nx * kPTileW, lt / nx * kPTileH};
}

// ---------------------------------------------------------------- kernels

template <typename V> __device__ __forceinline__ double ldd(const V *p, long long i) { return (double)p[i]; }

// (L v)_p with the periodic pixel graph (level 0: unit couplings; a side of
// one pixel has none, a side of two couples across both faces)
template <typename V>
__device__ __forceinline__ double plap(const V *v, long long off, long long pitch, int H, int W, int y, int x)
{
    const double c = ldd(v, off + (long long)y * pitch + x);
    double s = 0.0;
    if (W > 1) {
        const int xl = x == 0 ? W - 1 : x - 1, xr = x == W - 1 ? 0 : x + 1;
        s += (c - ldd(v, off + (long long)y * pitch + xl)) + (c - ldd(v, off + (long long)y * pitch + xr));
    }
    if (H > 1) {
        const int yu = y == 0 ? H - 1 : y - 1, yd = y == H - 1 ? 0 : y + 1;
        s += (c - ldd(v, off + (long long)yu * pitch + x)) + (c - ldd(v, off + (long long)yd * pitch + x));
    }
    return s;
}

// b_u = alpha (g_s - g_o) into level-0 b, partials of ||alpha g_s + L g_o||^2,
// ||b_u||^2 and sum(b_u).  With gs null, g_s is taken as b_u / alpha + g_o from
// the b_u already in level-0 b (written by the smoothing), which is then kept.
template <typename T, typename TS, typename TO>
__global__ __launch_bounds__(256) void pprep_kernel(const TS *gs, const TO *go, const SliceIO *io, PLaunch a,
                                                    double *pbb, double *pb0, double *pbs)
{
    __shared__ double red[4];
    if (blockIdx.x >= (unsigned)a.n_items) return;
    const PTile it = ptile(a, io);
    const SliceIO P = io[it.slice];
    const LevelDesc L = a.levs[P.lev0];
    T *b = static_cast<T *>(L.b);
    const int x = it.x0 + (threadIdx.x & 63);
    double sbb = 0.0, sb0 = 0.0, sbs = 0.0;
    if (x < P.W) {
#pragma unroll
        for (int i = 0; i < kPRows; ++i) {
            const int y = it.y0 + (threadIdx.x >> 6) + 4 * i;
            if (y >= P.H) break;
            const double o = ldd(go, P.off_go + (long long)y * P.pitch_go + x);
            const size_t pb = (size_t)y * L.pitch + x;
            T bu;
            double bf;
            if (gs) {
                const double sv = ldd(gs, P.off_gs + (long long)y * P.pitch_gs + x);
                bu = (T)(P.alpha * (sv - o));
                bf = P.alpha * sv + plap(go, P.off_go, P.pitch_go, P.H, P.W, y, x);
                b[pb] = bu;
            } else {
                bu = b[pb];
                bf = (double)bu + P.alpha * o + plap(go, P.off_go, P.pitch_go, P.H, P.W, y, x);
            }
            sbb += bf * bf;
            sb0 += (double)bu * (double)bu;
            sbs += (double)bu;
        }
    }
    const double t1 = pblock_sum(sbb, red), t2 = pblock_sum(sb0, red), t3 = pblock_sum(sbs, red);
    if (threadIdx.x == 0) {
        pbb[blockIdx.x] = t1;
        pb0[blockIdx.x] = t2;
        pbs[blockIdx.x] = t3;
    }
}

// f = g_o + (u + uoff + shift) and the FP64 residual b_u - A (u + uoff + shift)
// of the returned correction (constants cancel in L).
template <typename T, typename TO, typename TF>
__global__ __launch_bounds__(256) void pfinalize_kernel(const TO *go, TF *f, const SliceIO *io, PLaunch a,
                                                        const SliceState *st, const int *only)
{
    __shared__ double red[4];
    if (blockIdx.x >= (unsigned)a.n_items) return;
    const PTile it = ptile(a, io);
    if (only && !only[it.slice]) return;   // uniform per block: keeps this slice's partial sum
    const SliceIO P = io[it.slice];
    const LevelDesc L = a.levs[P.lev0];
    const T *u = static_cast<const T *>(L.u[0]);
    const T *b = static_cast<const T *>(L.b);
    const double shift = st[it.slice].shift + st[it.slice].uoff;
    const int x = it.x0 + (threadIdx.x & 63);
    double srr = 0.0;
    if (x < P.W) {
#pragma unroll
        for (int i = 0; i < kPRows; ++i) {
            const int y = it.y0 + (threadIdx.x >> 6) + 4 * i;
            if (y >= P.H) break;
            const double uc = (double)u[(size_t)y * L.pitch + x];
            const double res = (double)b[(size_t)y * L.pitch + x] - P.alpha * (uc + shift) -
                               plap(u, 0, L.pitch, P.H, P.W, y, x);
            srr += res * res;
            f[P.off_f + (long long)y * P.pitch_f + x] =
                (TF)(ldd(go, P.off_go + (long long)y * P.pitch_go + x) + (uc + shift));
        }
    }
    const double t = pblock_sum(srr, red);
    if (threadIdx.x == 0) a.part_rr[blockIdx.x] = t;
}

// Mixed refinement: u64_out = u64_in + e (e = level-0 FP32 iterate, buffer
// r.e_sel; u64_in is zero, and not read, on the first step), r = rhs - A u64_out in FP64 with
// rhs = alpha (g_s - g_o) or r.rhs, stored as FP32 into level-0 b; ||r||^2.
template <typename TS, typename TO>
__global__ __launch_bounds__(256) void prefine_kernel(RefineArgs r, PLaunch a)
{
    __shared__ double red[4];
    if (blockIdx.x >= (unsigned)a.n_items) return;
    const PTile it = ptile(a, r.io);
    double srr = 0.0;
    if (r.active[it.slice]) {   // uniform per block
        const SliceIO P = r.io[it.slice];
        const LevelDesc L = a.levs[P.lev0];
        const long long pl = L.pitch;
        const double *uin = r.u64[r.in_sel * r.n_slices + it.slice];
        double *uout = r.u64[(r.in_sel ^ 1) * r.n_slices + it.slice];
        const float *e = static_cast<const float *>(L.u[0]);
        float *b = static_cast<float *>(L.b);
        const int x = it.x0 + (threadIdx.x & 63);
        auto unew = [&](int y, int xx) -> double {
            const long long q = (long long)y * pl + xx;
            return (r.first ? 0.0 : uin[q]) + (double)e[q];
        };
        if (x < P.W) {
#pragma unroll
            for (int i = 0; i < kPRows; ++i) {
                const int y = it.y0 + (threadIdx.x >> 6) + 4 * i;
                if (y >= P.H) break;
                const double uc = unew(y, x);
                double lap = 0.0;
                if (P.W > 1) {
                    const int xl = x == 0 ? P.W - 1 : x - 1, xr = x == P.W - 1 ? 0 : x + 1;
                    lap += (uc - unew(y, xl)) + (uc - unew(y, xr));
                }
                if (P.H > 1) {
                    const int yu = y == 0 ? P.H - 1 : y - 1, yd = y == P.H - 1 ? 0 : y + 1;
                    lap += (uc - unew(yu, x)) + (uc - unew(yd, x));
                }
                double bv;
                if (r.rhs)
                    bv = ldd(static_cast<const TS *>(r.rhs), P.off_f + (long long)y * P.pitch_f + x);
                else
                    bv = P.alpha * (ldd(static_cast<const TS *>(r.gs), P.off_gs + (long long)y * P.pitch_gs + x) -
                                    ldd(static_cast<const TO *>(r.go), P.off_go + (long long)y * P.pitch_go + x));
                const double res = bv - P.alpha * uc - lap;
                srr += res * res;
                uout[(long long)y * pl + x] = uc;
                b[(long long)y * pl + x] = (float)res;
            }
        }
    }
    const double t = pblock_sum(srr, red);
    if (threadIdx.x == 0) r.part_rr[blockIdx.x] = t;
}

// lambda = A^-1 grad_f: grad_gs = alpha lambda, grad_go = L lambda, partials
// of lambda . (g_s - f).
template <typename T, typename TL>
__global__ __launch_bounds__(256) void padjoint_kernel(const T *gs, const T *f, T *ggs, T *ggo, const SliceIO *io,
                                                       int n, PLaunch a, const SliceState *st,
                                                       double *const *u64, double *part_da)
{
    __shared__ double red[4];
    if (blockIdx.x >= (unsigned)a.n_items) return;
    const PTile it = ptile(a, io);
    const SliceIO P = io[it.slice];
    const LevelDesc L = a.levs[P.lev0];
    const int cycles = st[it.slice].cycles;
    const TL *lam = u64 ? reinterpret_cast<const TL *>(u64[(cycles & 1) * n + it.slice])
                        : static_cast<const TL *>(L.u[0]);
    const bool zero = u64 && cycles == 0;   // no refinement step: still zero, and never written
    const double shift = u64 ? 0.0 : st[it.slice].shift + st[it.slice].uoff;   // constant parts of lambda
    const int x = it.x0 + (threadIdx.x & 63);
    double sda = 0.0;
    if (x < P.W) {
#pragma unroll
        for (int i = 0; i < kPRows; ++i) {
            const int y = it.y0 + (threadIdx.x >> 6) + 4 * i;
            if (y >= P.H) break;
            const double l = zero ? 0.0 : ldd(lam, (long long)y * L.pitch + x) + shift;
            const long long fo = P.off_f + (long long)y * P.pitch_f + x;
            if (ggs) ggs[fo] = (T)(P.alpha * l);
            if (ggo) ggo[fo] = zero ? T(0) : (T)plap(lam, 0, L.pitch, P.H, P.W, y, x);   // L is blind to the shift
            if (part_da) sda += l * (ldd(gs, P.off_gs + (long long)y * P.pitch_gs + x) - ldd(f, fo));
        }
    }
    if (!part_da) return;
    const double t = pblock_sum(sda, red);
    if (threadIdx.x == 0) part_da[blockIdx.x] = t;
}

}  // namespace

// ------------------------------------------------------------------- launch

hipError_t launch_pprep(bool fp64, int gs_dtype, const void *gs, int go_dtype, const void *go, const SliceIO *io,
                        const PLaunch &a, double *pbb, double *pb0, double *pbs, hipStream_t s)
{
    if (a.n_items <= 0) return hipSuccess;
    const dim3 g((unsigned)a.n_items), blk(256);
#define GDF_PP(T, TS, TO)                                                                                       \
    hipLaunchKernelGGL((pprep_kernel<T, TS, TO>), g, blk, 0, s, (const TS *)gs, (const TO *)go, io, a, pbb, pb0, pbs)
#define GDF_PPO(T, TS)                                   \
    do {                                                 \
        if (go_dtype == GDF_DT_U8) GDF_PP(T, TS, uint8_t); \
        else if (go_dtype == GDF_DT_F32) GDF_PP(T, TS, float); \
        else GDF_PP(T, TS, double);                      \
    } while (0)
    if (fp64) {
        if (gs_dtype == GDF_DT_F64) GDF_PPO(double, double); else GDF_PPO(double, float);
    } else {
        if (gs_dtype == GDF_DT_F64) GDF_PPO(float, double); else GDF_PPO(float, float);
    }
#undef GDF_PPO
#undef GDF_PP
    return hipGetLastError();
}

hipError_t launch_pfinalize(bool fp64, int go_dtype, const void *go, int out_dtype, void *f, const SliceIO *io,
                            const PLaunch &a, const SliceState *st, const int *only, hipStream_t s)
{
    if (a.n_items <= 0) return hipSuccess;
    const dim3 g((unsigned)a.n_items), blk(256);
#define GDF_PF(T, TO, TF) hipLaunchKernelGGL((pfinalize_kernel<T, TO, TF>), g, blk, 0, s, (const TO *)go, (TF *)f, io, a, st, only)
#define GDF_PFO(T, TF)                                   \
    do {                                                 \
        if (go_dtype == GDF_DT_U8) GDF_PF(T, uint8_t, TF); \
        else if (go_dtype == GDF_DT_F32) GDF_PF(T, float, TF); \
        else GDF_PF(T, double, TF);                      \
    } while (0)
    if (fp64) {
        if (out_dtype == GDF_DT_F64) GDF_PFO(double, double); else GDF_PFO(double, float);
    } else {
        if (out_dtype == GDF_DT_F64) GDF_PFO(float, double); else GDF_PFO(float, float);
    }
#undef GDF_PFO
#undef GDF_PF
    return hipGetLastError();
}

hipError_t launch_prefine(const RefineArgs &r, const PLaunch &a, hipStream_t s)
{
    if (a.n_items <= 0) return hipSuccess;
    const dim3 g((unsigned)a.n_items), blk(256);
    const bool s64 = r.gs_dtype == GDF_DT_F64;
    switch (r.go_dtype) {
    case GDF_DT_U8:
        if (s64) hipLaunchKernelGGL((prefine_kernel<double, uint8_t>), g, blk, 0, s, r, a);
        else hipLaunchKernelGGL((prefine_kernel<float, uint8_t>), g, blk, 0, s, r, a);
        break;
    case GDF_DT_F32:
        if (s64) hipLaunchKernelGGL((prefine_kernel<double, float>), g, blk, 0, s, r, a);
        else hipLaunchKernelGGL((prefine_kernel<float, float>), g, blk, 0, s, r, a);
        break;
    default:
        if (s64) hipLaunchKernelGGL((prefine_kernel<double, double>), g, blk, 0, s, r, a);
        else hipLaunchKernelGGL((prefine_kernel<float, double>), g, blk, 0, s, r, a);
        break;
    }
    return hipGetLastError();
}

hipError_t launch_padjoint(bool fp64, const void *gs, const void *f, void *ggs, void *ggo, const SliceIO *io, int n,
                           const PLaunch &a, const SliceState *st, double *const *u64, double *part_da,
                           hipStream_t s)
{
    if (a.n_items <= 0) return hipSuccess;
    const dim3 g((unsigned)a.n_items), blk(256);
    if (fp64)
        hipLaunchKernelGGL((padjoint_kernel<double, double>), g, blk, 0, s, (const double *)gs, (const double *)f,
                           (double *)ggs, (double *)ggo, io, n, a, st, u64, part_da);
    else if (u64)
        hipLaunchKernelGGL((padjoint_kernel<float, double>), g, blk, 0, s, (const float *)gs, (const float *)f,
                           (float *)ggs, (float *)ggo, io, n, a, st, u64, part_da);
    else
        hipLaunchKernelGGL((padjoint_kernel<float, float>), g, blk, 0, s, (const float *)gs, (const float *)f,
                           (float *)ggs, (float *)ggo, io, n, a, st, u64, part_da);
    return hipGetLastError();
}

}  // namespace gdf
