// Register-block multigrid passes: the coarse levels of the Neumann hierarchy,
// its finest level for small batches, and every level of the periodic one.
//
// A workgroup of 8 waves holds a region of 128 columns x 64 rows of one level
// of one slice in registers: two adjacent columns per lane, 8 consecutive rows
// per wave.  All loads of the region are issued at once; then red-black
// half-sweeps run one after the other, horizontal neighbours coming from DPP
// wave shifts, vertical ones from the lane's own registers, and only each
// wave's first and last row through LDS (one barrier per half-sweep).  The
// region carries a halo of G cells on the sides where the slice goes on, so a
// pass applies several sweeps, the residual and its restriction (or the
// prolongation before them) in one trip over memory, and the owned cells come
// out as if the half-sweeps had run one by one over the whole level.
//
// What bounds it: a coarse level is small, so a pass is a chain of latencies
// rather than a stream.  Marching a strip row by row pays one dependent step
// per row (about 0.4 us a row on a nearly idle chip); a block pays one load
// latency plus one short exchange per half-sweep.  Measurements are at
// launch_block.
//
// Levels follow the finite-volume operators described in mg_kernels.hip.  On
// the torus (periodic boundaries) a cell's neighbours are taken modulo the
// side, and the coupling across a face is 2 / (width left + width right), so
// the faces on either side of the narrower last cell carry 2 / (1 + wL).  A
// side of one cell has no couplings; a side of two couples the two cells
// across both faces.  Where an odd side brings two cells of one colour
// together across the wrap, each reads the other's previous value.
#include "internal.h"
#include "wave.h"

#include <type_traits>

namespace gdf {

namespace {

#define GDF_G __attribute__((address_space(1)))

constexpr int kR = kBlockRows / kBlockWaves;   // rows per wave

template <typename T> struct Quad { typedef T type __attribute__((ext_vector_type(4))); };

template <typename T> struct BlockShared {
    // first / last rows of each wave, by half-sweep parity: [parity][first, last][column][wave][lane]
    T x[2][2][2][kBlockWaves][kWave];
    // stencils by row class: couplings (left, right, up, down) over the diagonal,
    // the diagonal and its inverse: [class][column][lane]
    typename Quad<T>::type cf[4][2][kWave];
    T dg[4][2][kWave], iv[4][2][kWave];
    double red[kBlockWaves][2];
};

// The part of one side of a level (n cells) that tile t covers: region cells
// [r0, r0 + len), owned cells [o0, o1); see BItem.  plain: the coefficients in
// the region are those of full cells with both neighbours, and colours
// alternate along it (the outermost halo cell may be any).
struct Seg {
    int r0, o0, o1;
    bool plain;
};
__device__ __forceinline__ Seg segment(bool per, int t, int n, int len, int G, double wl)
{
    Seg g;
    if (per) {
        g.o0 = t * (len - 2 * G);
        g.r0 = g.o0 - G;
        g.o1 = min(g.o0 + len - 2 * G, n);
    } else {
        g.r0 = t * (len - 2 * G);
        g.o0 = t == 0 ? 0 : g.r0 + G;
        g.o1 = g.r0 + len >= n ? n : g.r0 + len - G;
    }
    g.plain = (g.r0 >= 1 && g.r0 + len - 1 <= n - 2) || (per && !(n & 1) && wl == 1.0);
    return g;
}

__device__ __forceinline__ int wrap_idx(int i, int n)
{
    const int m = i % n;
    return m < 0 ? m + n : m;
}

// element i of the row starting at element `row` of p (a wave-uniform base plus a
// 32-bit lane offset; V: the element type, or a pair of it)
template <typename V, typename S> __device__ __forceinline__ V ld(const GDF_G S *p, size_t row, unsigned i)
{
    return *reinterpret_cast<const GDF_G V *>(reinterpret_cast<const GDF_G char *>(p + row) + i * (unsigned)sizeof(S));
}
template <typename V, typename S> __device__ __forceinline__ void st(V v, GDF_G S *p, size_t row, unsigned i)
{
    *reinterpret_cast<GDF_G V *>(reinterpret_cast<GDF_G char *>(p + row) + i * (unsigned)sizeof(S)) = v;
}

// couplings (left, right) and relative width of cell i of a side of n cells
// whose last cell has relative width wl (ke = 2 / (1 + wl))
template <typename T, bool PER>
__device__ __forceinline__ void side_coef(int i, int n, T wl, T ke, T &w, T &kl, T &kr)
{
    w = i == n - 1 ? wl : T(1);
    if constexpr (PER) {
        // face f lies between cells f and f + 1 (mod n)
        const int fl = i == 0 ? n - 1 : i - 1;
        kl = n > 1 ? (fl >= n - 2 ? ke : T(1)) : T(0);
        kr = n > 1 ? (i >= n - 2 ? ke : T(1)) : T(0);
    } else {
        kl = i > 0 ? (i == n - 1 ? ke : T(1)) : T(0);
        kr = i < n - 1 ? (i == n - 2 ? ke : T(1)) : T(0);
    }
}

// PLAIN: both segments are plain (one stencil for every cell); otherwise
// coefficients are per lane and per row.
// R: rows per wave.  NHS: half-sweeps (0: 2 `sweeps`, a run-time count).
template <int R, typename T, typename SO, typename SC, bool PER, bool RB, bool PROLONG, bool ZERO, int NHS, int RMODE,
          bool SOR, bool PLAIN>
__device__ __forceinline__ void block_item(const BlockLaunch &a, const LevelDesc &L, const Seg &sx, const Seg &sy, int slot,
                                           int in_sel, int out_sel, int sweeps, BlockShared<T> &sh)
{
    static_assert(R % 2 == 0 && NHS % 2 == 0, "a wave's first row is even and sweeps are whole: static parities");
    using SOt = Stor<SO>;
    using SCt = Stor<SC>;
    using PO = typename SOt::Pair;
    const int lane = threadIdx.x & (kWave - 1), wv = uniform(threadIdx.x >> 6);
    const int H = L.H, W = L.W, pitch = L.pitch, Hc = L.Hc, Wc = L.Wc;
    const T sig = (T)L.sigma;
    const T dg = sig + T(4), ivs = T(1) / dg;

    // ---- columns (c0 even) and rows of the lane, in the region and in the slice
    const int c0 = sx.r0 + 2 * lane;
    const int y0 = sy.r0 + wv * R;   // even
    const bool dead = !PER && y0 >= H;        // (uniform) no row of this wave lies in the slice
    const bool below = wv < kBlockWaves - 1 && (PER || y0 + R < H);   // (uniform) the next wave has some
    int x0, x1;
    bool in0 = true, in1 = true;       // Neumann: the column lies in the slice
    // colours alternate along the region's rows and columns (no wrap across an odd side)
    const bool regular = !PER || PLAIN || !((W | H) & 1);
    if constexpr (PER) {
        x0 = wrap_idx(c0, W);
        x1 = x0 + 1 == W ? 0 : x0 + 1;
    } else {
        in0 = c0 < W;
        in1 = c0 + 1 < W;
        x0 = min(c0, (W - 1) & ~1);
        x1 = x0 + 1;
    }
    int yw[R];   // the row in the slice (uniform; Neumann: clamped)
    {
        int y = PER ? wrap_idx(y0, H) : 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (PER) {
                yw[r] = uniform(y);
                y = y + 1 == H ? 0 : y + 1;
            } else {
                yw[r] = min(y0 + r, H - 1);
            }
        }
    }

    // ---- loads: all rows at once
    const GDF_G SO *gb = (const GDF_G SO *)L.b;
    if constexpr (RB) {   // per-slice parity: the latest iterate sits in buffer cycles & 1
        if (a.cycles) {
            in_sel = uniform(a.cycles[(size_t)L.slice * a.cycles_stride]) & 1;
            out_sel = in_sel ^ 1;
        }
    }
    const GDF_G SO *gu = (const GDF_G SO *)(in_sel ? L.u[1] : L.u[0]);
    const bool pairs = regular || !(W & 1);   // the two columns are adjacent and start even
    auto load_rows = [&](const GDF_G SO *g, T v[R][2]) {
        if (pairs) {
            PO q[R];
#pragma unroll
            for (int r = 0; r < R; ++r) q[r] = ld<PO>(g, (size_t)yw[r] * pitch, (unsigned)x0);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                v[r][0] = (T)SOt::lo(q[r]);
                v[r][1] = (T)SOt::hi(q[r]);
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                v[r][0] = (T)SOt::get(ld<SO>(g, (size_t)yw[r] * pitch, (unsigned)x0));
                v[r][1] = (T)SOt::get(ld<SO>(g, (size_t)yw[r] * pitch, (unsigned)x1));
            }
        }
    };
    T b[R][2], u[R][2];
    if (!dead) {
        load_rows(gb, b);
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) b[r][0] = b[r][1] = T(0);
    }
    if (ZERO || dead) {
#pragma unroll
        for (int r = 0; r < R; ++r) u[r][0] = u[r][1] = T(0);
    } else if constexpr (RB) {
        // rows stored by colour (LevelDesc): the lane's black pixel is element
        // x0 / 2 of half 1; the red one is dead (the first half-sweep overwrites it)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            u[r][(r & 1) ^ 1] = (T)ld<SO>(gu, (size_t)yw[r] * pitch + (pitch >> 1), (unsigned)x0 >> 1);
            u[r][r & 1] = T(0);
        }
    } else {
        load_rows(gu, u);
    }

    // ---- prolongation: cell-centred bilinear, 3/4 of the parent row plus 1/4 of
    // the next coarse row towards the fine row, then the same in x
    if (PROLONG && !dead) {
        const GDF_G SC *ge = (const GDF_G SC *)L.ec;
        const int pc = L.pitch_c;
        if (regular) {
            const int lc = min(x0 >> 1, Wc - 1);
            const bool ledge = !PER && lc == 0, redge = !PER && lc == Wc - 1;
            // coarse rows (y0 >> 1) - 1 .. (y0 >> 1) + R / 2, clamped (mirrored) or wrapped
            T e[R / 2 + 2];
            int m = PER ? (yw[0] >> 1) : 0;
            m = PER ? (m == 0 ? Hc - 1 : m - 1) : 0;
#pragma unroll
            for (int k = 0; k < R / 2 + 2; ++k) {
                const int mk = PER ? m : min(max((y0 >> 1) - 1 + k, 0), Hc - 1);
                e[k] = (T)SCt::get(ld<SC>(ge, (size_t)mk * pc, (unsigned)lc));
                m = m + 1 == Hc ? 0 : m + 1;
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const T V = T(0.75) * e[r / 2 + 1] + T(0.25) * ((r & 1) ? e[r / 2 + 2] : e[r / 2]);
                T VL = wave_shr1(V), VR = wave_shl1(V);
                if constexpr (!PER && !PLAIN) {
                    VL = ledge ? V : VL;
                    VR = redge ? V : VR;
                }
                u[r][0] += T(0.75) * V + T(0.25) * VL;
                u[r][1] += T(0.75) * V + T(0.25) * VR;
            }
        } else {
            const int X0 = x0 >> 1, X1 = x1 >> 1;
            const int N0 = wrap_idx((x0 & 1) ? X0 + 1 : X0 - 1, Wc), N1 = wrap_idx((x1 & 1) ? X1 + 1 : X1 - 1, Wc);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int Y = yw[r] >> 1;
                const int N = (yw[r] & 1) ? (Y + 1 == Hc ? 0 : Y + 1) : (Y == 0 ? Hc - 1 : Y - 1);
                const GDF_G SC *e0 = ge + (size_t)Y * pc, *e1 = ge + (size_t)N * pc;
                const T p0 = T(0.75) * (T)SCt::get(e0[X0]) + T(0.25) * (T)SCt::get(e1[X0]);
                const T q0 = T(0.75) * (T)SCt::get(e0[N0]) + T(0.25) * (T)SCt::get(e1[N0]);
                const T p1 = T(0.75) * (T)SCt::get(e0[X1]) + T(0.25) * (T)SCt::get(e1[X1]);
                const T q1 = T(0.75) * (T)SCt::get(e0[N1]) + T(0.25) * (T)SCt::get(e1[N1]);
                u[r][0] += T(0.75) * p0 + T(0.25) * q0;
                u[r][1] += T(0.75) * p1 + T(0.25) * q1;
                __builtin_amdgcn_sched_barrier(0);   // (row by row: all rows' loads at once would not fit the registers)
            }
        }
    }

    // ---- coefficients.  Rows: recomputed from the row index where needed (scalars)
    const T wxL = (T)L.wxL, wyL = (T)L.wyL;
    const T kxe = T(2) / (T(1) + wxL), kye = T(2) / (T(1) + wyL);
    T wx0 = T(1), kl0 = T(1), kr0 = T(1), wx1 = T(1), kl1 = T(1), kr1 = T(1);
    // Stencils differ by column, and among rows only in the first, the
    // second-to-last and the last (class 1, 2, 3; 0 the others).  Columns outside
    // the slice have none; rows outside repeat the last one's and are never read
    // by a row inside (no coupling leads there).
    using T4 = typename Quad<T>::type;
    auto row_class = [&](int r) -> int { return yw[r] == H - 1 ? 3 : yw[r] == 0 ? 1 : yw[r] == H - 2 ? 2 : 0; };
    bool rows0 = true;   // every row of this wave is of class 0 (uniform)
    T4 q0{}, q1{};       // the stencils of class 0
    T iv0 = ivs, iv1 = ivs;
    if constexpr (!PLAIN) {
        side_coef<T, PER>(PER ? x0 : c0, W, wxL, kxe, wx0, kl0, kr0);
        side_coef<T, PER>(PER ? x1 : c0 + 1, W, wxL, kxe, wx1, kl1, kr1);
        auto stencil = [&](bool in, T wx, T kl, T kr, T wy, T ku, T kd, T &d, T &i) -> T4 {
            // (a full cell with every neighbour takes the diagonal of PLAIN tiles to the
            // last bit: the mean is removed alike in every tile, see below)
            const bool full = wx == T(1) && wy == T(1) && kl == T(1) && kr == T(1) && ku == T(1) && kd == T(1);
            d = full ? dg : sig * wx * wy + wy * (kl + kr) + wx * (ku + kd);
            i = in ? T(1) / d : T(0);
            return T4{wy * kl * i, wy * kr * i, wx * ku * i, wx * kd * i};
        };
        T d, i;
        if (wv < 4) {   // wave w: class w (a side without that class's row never reads it)
            T wy = T(1), ku = T(1), kd = T(1);
            if (wv > 0) side_coef<T, PER>(wv == 1 ? 0 : max(H - 4 + wv, 0), H, wyL, kye, wy, ku, kd);
            sh.cf[wv][0][lane] = stencil(in0, wx0, kl0, kr0, wy, ku, kd, d, i);
            sh.dg[wv][0][lane] = d;
            sh.iv[wv][0][lane] = i;
            sh.cf[wv][1][lane] = stencil(in1, wx1, kl1, kr1, wy, ku, kd, d, i);
            sh.dg[wv][1][lane] = d;
            sh.iv[wv][1][lane] = i;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) rows0 = rows0 && row_class(r) == 0;
        q0 = stencil(in0, wx0, kl0, kr0, T(1), T(1), T(1), d, iv0);
        q1 = stencil(in1, wx1, kl1, kr1, T(1), T(1), T(1), d, iv1);
        __syncthreads();
    }
    // the level-0 mean is removed from the right-hand side (level 0), or its
    // children's share of it (a level 1 restricted from unshifted values, on the way
    // down)
    if (!dead) {
        const T bsh = L.bshift ? (T)uniform_d(*L.bshift) : T(0);
        const T bsc = (!PROLONG && a.raw_rhs && L.bshift_fine) ? T(4) * (T)uniform_d(*L.bshift_fine) : T(0);
        const T bsg = (bsh + bsc) * ivs;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            // the right-hand side is held over the diagonal (and the mean over it
            // subtracted, as the strips do: its FP32 rounding is a constant of the
            // whole slice)
            if constexpr (PLAIN) {
                b[r][0] = fma(b[r][0], ivs, -bsg);
                b[r][1] = fma(b[r][1], ivs, -bsg);
            } else {
                const T wy = yw[r] == H - 1 ? wyL : T(1);
                T i0 = iv0, i1 = iv1;
                if (!rows0) {
                    i0 = sh.iv[row_class(r)][0][lane];
                    i1 = sh.iv[row_class(r)][1][lane];
                }
                // (outside the slice: zero, whatever was loaded)
                b[r][0] = in0 ? fma(b[r][0], i0, -(fma(bsc * wx0, wy, bsh) * i0)) : T(0);
                b[r][1] = in1 ? fma(b[r][1], i1, -(fma(bsc * wx1, wy, bsh) * i1)) : T(0);
                u[r][0] = in0 ? u[r][0] : T(0);
                u[r][1] = in1 ? u[r][1] : T(0);
            }
        }
    }

    // ---- half-sweeps (red first)
    // exchange of the waves' first and last rows: up[j] / dn[j] are column j of
    // the rows above and below the wave's (zero past the region's edge: only
    // halo rows, or rows without that coupling, read them).  Parity halves
    // alternate with the colour, so one barrier separates the writes of one half-sweep from
    // its reads and from the next writes to the same half.
    auto exchange = [&](int p, bool both, int jf, int jl, T up[2], T dn[2]) {
        // jf: the column of the first row that the wave above reads; jl: of the last row
        if (dead) {
        } else if (both) {
            sh.x[p][0][0][wv][lane] = u[0][0];
            sh.x[p][0][1][wv][lane] = u[0][1];
            sh.x[p][1][0][wv][lane] = u[R - 1][0];
            sh.x[p][1][1][wv][lane] = u[R - 1][1];
        } else {
            sh.x[p][0][0][wv][lane] = u[0][jf];
            sh.x[p][1][0][wv][lane] = u[R - 1][jl];
        }
        __syncthreads();
        if (dead) {
        } else if (both) {
            up[0] = wv > 0 ? sh.x[p][1][0][wv - 1][lane] : T(0);
            up[1] = wv > 0 ? sh.x[p][1][1][wv - 1][lane] : T(0);
            dn[0] = below ? sh.x[p][0][0][wv + 1][lane] : T(0);
            dn[1] = below ? sh.x[p][0][1][wv + 1][lane] : T(0);
        } else {
            up[jl] = wv > 0 ? sh.x[p][1][0][wv - 1][lane] : T(0);
            dn[jf] = below ? sh.x[p][0][0][wv + 1][lane] : T(0);
        }
    };
    auto apply = [](const T4 &q, T vl, T vr, T vu, T vd, T bb) -> T {
        return fma(q.x, vl, fma(q.y, vr, fma(q.z, vu, fma(q.w, vd, bb))));
    };
    // (a regular half-sweep of colour c updates column (r & 1) ^ c of row r;
    // the first row is even, the last odd)
    auto half_sweep = [&](const int c, const bool first) __attribute__((always_inline)) {
        T up[2] = {T(0), T(0)}, dn[2] = {T(0), T(0)};
        if (PLAIN || regular) {
            if (ZERO && !PROLONG && first) {   // from zero: no neighbours yet
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int j = (r & 1) ^ c;
                    u[r][j] = b[r][j];
                }
                return;
            }
            exchange(c, false, 1 ^ c, c, up, dn);
            if (dead) return;
            auto sweep = [&](auto row) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int j = (r & 1) ^ c;
                    const T vu = r > 0 ? u[r > 0 ? r - 1 : 0][j] : up[j];
                    const T vd = r < R - 1 ? u[r < R - 1 ? r + 1 : r][j] : dn[j];
                    const T vl = j == 0 ? wave_shr1(u[r][1]) : u[r][0];
                    const T vr = j == 0 ? u[r][1] : wave_shl1(u[r][0]);
                    const T v = row(r, j, vl, vr, vu, vd);
                    // SOR: every half-sweep after the first moves its cells by kOmega
                    // times the Gauss-Seidel step (the first overwrites dead values)
                    u[r][j] = SOR && !first ? fma(T(kOmega), v - u[r][j], u[r][j]) : v;
                }
            };
            if constexpr (PLAIN) {
                sweep([&](int r, int j, T vl, T vr, T vu, T vd) { return fma((vl + vr) + (vu + vd), ivs, b[r][j]); });
            } else if (rows0) {
                sweep([&](int r, int j, T vl, T vr, T vu, T vd) { return apply(j ? q1 : q0, vl, vr, vu, vd, b[r][j]); });
            } else {
                sweep([&](int r, int j, T vl, T vr, T vu, T vd) {
                    return apply(sh.cf[row_class(r)][j][lane], vl, vr, vu, vd, b[r][j]);
                });
            }
        } else if constexpr (!PLAIN) {
            // an odd side wraps inside the region: colours per cell, all cells of
            // the colour updated from the values before the half-sweep
            exchange(c, true, 0, 0, up, dn);
            T p0 = up[0], p1 = up[1];   // the row above, before the half-sweep
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const T o0 = u[r][0], o1 = u[r][1];
                const T d0 = r < R - 1 ? u[r < R - 1 ? r + 1 : r][0] : dn[0];
                const T d1 = r < R - 1 ? u[r < R - 1 ? r + 1 : r][1] : dn[1];
                const T l = wave_shr1(o1), rr = wave_shl1(o0);
                const int k = row_class(r);
                const T n0 = apply(sh.cf[k][0][lane], l, o1, p0, d0, b[r][0]);
                const T n1 = apply(sh.cf[k][1][lane], o0, rr, p1, d1, b[r][1]);
                u[r][0] = ((x0 + yw[r]) & 1) == c ? n0 : o0;
                u[r][1] = ((x1 + yw[r]) & 1) == c ? n1 : o1;
                p0 = o0;
                p1 = o1;
            }
        }
    };
    if constexpr (NHS > 0) {
#pragma unroll
        for (int s = 0; s < NHS; ++s) half_sweep(s & 1, s == 0);
    } else {
        half_sweep(0, true);
        half_sweep(1, false);
        for (int s = 1; s < sweeps; ++s) {
            half_sweep(0, false);
            half_sweep(1, false);
        }
    }

    // ---- store the owned cells
    const bool own = c0 >= sx.o0 && c0 < sx.o1;
    {
        GDF_G SO *go = (GDF_G SO *)(out_sel ? L.u[1] : L.u[0]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int y = y0 + r;
            // (the pair's second column may lie in the row padding)
            if constexpr (RB) {
                if (y >= sy.o0 && y < sy.o1 && own) {   // column c0 has colour y & 1 = r & 1
                    st<SO>(u[r][r & 1], go, (size_t)y * pitch, (unsigned)c0 >> 1);
                    st<SO>(u[r][(r & 1) ^ 1], go, (size_t)y * pitch + (pitch >> 1), (unsigned)c0 >> 1);
                }
            } else if (y >= sy.o0 && y < sy.o1 && own)
                st<PO>(SOt::pair(u[r][0], u[r][1]), go, (size_t)y * pitch, (unsigned)c0);
        }
    }

    // ---- residual r = b - sigma u - sum_q k_q (u - u_q) (neighbour differences
    // are nearly exact), its norm and its restriction.  The last half-sweep
    // solved every black cell's equation for the cell, so with regular colours
    // only red cells have a residual to restrict; the norms take every cell
    // (rounding is part of them).
    if constexpr (RMODE != RES_NONE) {
        T up[2] = {T(0), T(0)}, dn[2] = {T(0), T(0)};
        const bool all = (RMODE & RES_NORM) != 0 || !(PLAIN || regular);
        exchange(0, all, 1, 0, up, dn);
        if (dead && !(RMODE & RES_NORM)) return;   // (with norms there is a barrier below)
        double s2 = 0.0, s1 = 0.0;
        T prow = T(0);
        GDF_G SC *gc = (GDF_G SC *)L.bc;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const T v0 = u[r][0], v1 = u[r][1];
            const T u0 = r > 0 ? u[r > 0 ? r - 1 : 0][0] : up[0], u1 = r > 0 ? u[r > 0 ? r - 1 : 0][1] : up[1];
            const T d0 = r < R - 1 ? u[r < R - 1 ? r + 1 : r][0] : dn[0];
            const T d1 = r < R - 1 ? u[r < R - 1 ? r + 1 : r][1] : dn[1];
            const T l0 = wave_shr1(v1), r1 = wave_shl1(v0);
            const T dd = v0 - v1;
            T r0 = T(0), rr1 = T(0);
            const bool f0 = all || !(r & 1), f1 = all || (r & 1);   // red: column r & 1
            if constexpr (PLAIN) {
                // b = (sigma + 4) x the scaled value, exact inside the fma
                if (f0) r0 = fma(dg, b[r][0], -fma(sig, v0, (((v0 - l0) + dd) + (v0 - u0)) + (v0 - d0)));
                if (f1) rr1 = fma(dg, b[r][1], -fma(sig, v1, (((v1 - r1) - dd) + (v1 - u1)) + (v1 - d1)));
            } else {
                T wy, ku, kd;
                side_coef<T, PER>(yw[r], H, wyL, kye, wy, ku, kd);
                const int k = row_class(r);
                if (f0) {
                    const T h = fma(kl0, v0 - l0, kr0 * dd), w = fma(ku, v0 - u0, kd * (v0 - d0));
                    r0 = fma(sh.dg[k][0][lane], b[r][0], -fma(sig * wx0 * wy, v0, fma(wy, h, wx0 * w)));
                }
                if (f1) {
                    const T h = fma(kr1, v1 - r1, -(kl1 * dd)), w = fma(ku, v1 - u1, kd * (v1 - d1));
                    rr1 = fma(sh.dg[k][1][lane], b[r][1], -fma(sig * wx1 * wy, v1, fma(wy, h, wx1 * w)));
                }
            }
            const int y = y0 + r;
            const bool orow = y >= sy.o0 && y < sy.o1;   // uniform
            // (children outside the slice contribute nothing)
            if constexpr (!PLAIN) rr1 = c0 + 1 < W ? rr1 : T(0);
            if constexpr ((RMODE & RES_NORM) != 0) {
                if (orow && own) {
                    s2 += (double)r0 * (double)r0 + (double)rr1 * (double)rr1;
                    s1 += (double)r0 + (double)rr1;
                }
            }
            if constexpr ((RMODE & RES_RESTRICT) != 0) {
                const T pr = r0 + rr1;
                if ((r & 1) == 0) {
                    prow = pr;
                } else {
                    // (owned rows start even; the last may be the first of its pair)
                    const bool o0 = y - 1 >= sy.o0 && y - 1 < sy.o1;   // uniform
                    const T sum = PLAIN || y < H ? prow + pr : prow;
                    if (o0 && own) st<SC>(SCt::put(sum), gc, (size_t)(y >> 1) * L.pitch_c, (unsigned)(c0 >> 1));
                }
            }
        }
        if constexpr ((RMODE & RES_NORM) != 0) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                s2 += __shfl_xor(s2, off);
                s1 += __shfl_xor(s1, off);
            }
            if (lane == 0) {
                sh.red[wv][0] = s2;
                sh.red[wv][1] = s1;
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                double t2 = 0.0, t1 = 0.0;
#pragma unroll
                for (int w = 0; w < kBlockWaves; ++w) {
                    t2 += sh.red[w][0];
                    t1 += sh.red[w][1];
                }
                if constexpr (RB) {
                    a.partials[slot] = make_float2((float)t2, (float)t1);
                } else {
                    a.part_rr[slot] = t2;
                    a.part_r[slot] = t1;
                }
            }
        }
    }
}

template <typename T, typename SO, typename SC, bool PER, bool RB, bool PROLONG, bool ZERO, int NHS, int RMODE,
          bool SOR = false>
__global__ __launch_bounds__(kBlockWaves *kWave, sizeof(T) == 4 ? 4 : 2) void block_kernel(BlockLaunch a)
{
    __shared__ BlockShared<T> sh;
    if (a.done && uniform(*a.done)) return;   // a captured pass after the last active slice
    const int slot = uniform((int)xcd_tile(blockIdx.x, gridDim.x));
    const BItem &g = a.items[slot];
    const LevelDesc L = uniform_level(a.levs[uniform(g.lev)]);
    if (!uniform(a.active[L.slice])) {
        if ((RMODE & RES_NORM) && threadIdx.x == 0) {
            if constexpr (RB) a.partials[slot] = make_float2(0.f, 0.f);
            else a.part_rr[slot] = a.part_r[slot] = 0.0;
        }
        return;
    }
    const Seg sx = segment(PER, uniform(g.tx), L.W, kBlockCols, a.G, L.wxL);
    const Seg sy = segment(PER, uniform(g.ty), L.H, kBlockRows, a.G, L.wyL);
    if (sx.plain && sy.plain)
        block_item<kR, T, SO, SC, PER, RB, PROLONG, ZERO, NHS, RMODE, SOR, true>(a, L, sx, sy, slot, a.in_sel, a.out_sel, 0,
                                                                                 sh);
    else
        block_item<kR, T, SO, SC, PER, RB, PROLONG, ZERO, NHS, RMODE, SOR, false>(a, L, sx, sy, slot, a.in_sel, a.out_sel, 0,
                                                                                  sh);
}

// The coarse end of a Neumann V-cycle in one launch, one workgroup per slice: from
// the first level that fits one region (kTailSide a side) down to the coarsest
// and back up.  Each level is the pass above over its one tile; what one wave
// writes and another reads goes through memory with a barrier between (the
// workgroup's own CU, so no further fence).  A launch per pass costs 6.5 us on
// levels this small, of which 3 are the launch and the item's table look-ups; the
// seven passes of 6 x 96 x 80 take 41 us in one, 5.8 each: dependent loads, LDS
// reads and barriers.
template <typename T>
__global__ __launch_bounds__(kBlockWaves *kWave, sizeof(T) == 4 ? 4 : 2) void tail_kernel(TailLaunch t)
{
    typedef typename LevelStor<T>::Coarse S;
    __shared__ BlockShared<T> sh;
    const BlockLaunch &a = t.a;
    if (a.done && uniform(*a.done)) return;
    const BItem &g = a.items[blockIdx.x];
    const int lev = uniform(g.lev), l0 = uniform(g.tx), n = uniform(g.ty);   // first level's descriptor and number, levels
    if (!uniform(a.active[uniform(a.levs[lev].slice)])) return;
    auto pass = [&](auto prolong, auto rmode, int l, int in_sel, int out_sel, int sweeps) __attribute__((always_inline)) {
        const LevelDesc L = uniform_level(a.levs[lev + l]);
        const Seg sx{0, 0, L.W, false}, sy{0, 0, L.H, false};
        constexpr bool P = decltype(prolong)::value;
        if (L.H <= kBlockRows)
            block_item<kR, T, S, S, false, false, P, !P, 0, decltype(rmode)::value, false, false>(
                a, L, sx, sy, 0, in_sel, out_sel, sweeps, sh);
        else
            block_item<2 * kR, T, S, S, false, false, P, !P, 0, decltype(rmode)::value, false, false>(
                a, L, sx, sy, 0, in_sel, out_sel, sweeps, sh);
        __syncthreads();
    };
    using std::integral_constant;
    for (int l = 0; l < n - 1; ++l)
        pass(integral_constant<bool, false>{}, integral_constant<int, RES_RESTRICT>{}, l, 0, 0, t.sweeps[l0 + l]);
    pass(integral_constant<bool, false>{}, integral_constant<int, RES_NONE>{}, n - 1, 0, 0, 2);
    for (int l = n - 2; l >= 0; --l)
        pass(integral_constant<bool, true>{}, integral_constant<int, RES_NONE>{}, l, 0, 1, t.sweeps[l0 + l]);
}

template <typename T, bool LEVEL0, bool PER, bool PROLONG, bool ZERO, int NHS, int RMODE>
hipError_t block_go(const BlockLaunch &a, hipStream_t s)
{
    typedef typename LevelStor<T>::Coarse SC;
    typedef typename std::conditional<LEVEL0, T, SC>::type SO;
    if (a.n_items <= 0) return hipSuccess;
    const dim3 g((unsigned)a.n_items), blk(kBlockWaves * kWave);
    hipLaunchKernelGGL((block_kernel<T, SO, SC, PER, false, PROLONG, ZERO, NHS, RMODE>), g, blk, 0, s, a);
    return hipGetLastError();
}

// half-sweeps by sweep count: 1, 2 (level 0), or 1 .. 3 (coarse levels)
template <typename T, bool LEVEL0, bool PER, bool PROLONG, bool ZERO, int RMODE>
hipError_t block_sw(int sweeps, const BlockLaunch &a, hipStream_t s)
{
    switch (sweeps) {
    case 1: return block_go<T, LEVEL0, PER, PROLONG, ZERO, 2, RMODE>(a, s);
    case 2: return block_go<T, LEVEL0, PER, PROLONG, ZERO, 4, RMODE>(a, s);
    case 3:
        if constexpr (!LEVEL0) return block_go<T, LEVEL0, PER, PROLONG, ZERO, 6, RMODE>(a, s);
    default: return hipErrorInvalidValue;
    }
}

// The fused finest pass of the Neumann hierarchy: prolongation, `sweeps` sweeps,
// residual with norms and restriction.
template <typename T, bool ZERO, int NHS, bool SOR>
hipError_t fine_go(const BlockLaunch &a, hipStream_t s)
{
    typedef typename LevelStor<T>::Coarse SC;
    if (a.n_items <= 0) return hipSuccess;
    hipLaunchKernelGGL((block_kernel<T, T, SC, false, true, true, ZERO, NHS, RES_BOTH, SOR>), dim3((unsigned)a.n_items),
                       dim3(kBlockWaves * kWave), 0, s, a);
    return hipGetLastError();
}
template <typename T, bool ZERO>
hipError_t fine_sw(int sweeps, bool sor, const BlockLaunch &a, hipStream_t s)
{
    if (sor) {
        if constexpr (sizeof(T) == 4) {
            if (sweeps == 4) return fine_go<T, ZERO, 8, true>(a, s);
            if (sweeps == 5) return fine_go<T, ZERO, 10, true>(a, s);
        }
        return hipErrorInvalidValue;
    }
    switch (sweeps) {
    case 2: return fine_go<T, ZERO, 4, false>(a, s);
    case 3: return fine_go<T, ZERO, 6, false>(a, s);
    case 4: return fine_go<T, ZERO, 8, false>(a, s);
    case 5: return fine_go<T, ZERO, 10, false>(a, s);
    case 6: return fine_go<T, ZERO, 12, false>(a, s);
    default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t block_t(BlockKind k, bool periodic, bool level0, int sweeps, const BlockLaunch &a, hipStream_t s)
{
    if (!periodic) {
        if (level0) return hipErrorInvalidValue;   // (level 0 of the Neumann hierarchy: strip kernel)
        switch (k) {
        case BK_DOWN_ZERO: return block_sw<T, false, false, false, true, RES_RESTRICT>(sweeps, a, s);
        case BK_UP: return block_sw<T, false, false, true, false, RES_NONE>(sweeps, a, s);
        case BK_LAST_ZERO: return block_go<T, false, false, false, true, 4, RES_NONE>(a, s);
        default: return hipErrorInvalidValue;
        }
    }
    if (level0) {
        switch (k) {
        case BK_DOWN_ZERO: return block_sw<T, true, true, false, true, RES_RESTRICT>(sweeps, a, s);
        case BK_DOWN: return block_sw<T, true, true, false, false, RES_RESTRICT>(sweeps, a, s);
        case BK_UP: return block_sw<T, true, true, true, false, RES_NORM>(sweeps, a, s);
        case BK_LAST_ZERO: return block_sw<T, true, true, false, true, RES_NONE>(sweeps, a, s);
        case BK_LAST_MID: return block_sw<T, true, true, false, false, RES_NONE>(sweeps, a, s);
        case BK_LAST: return block_sw<T, true, true, false, false, RES_NORM>(sweeps, a, s);
        default: return hipErrorInvalidValue;
        }
    }
    switch (k) {
    case BK_DOWN_ZERO: return block_sw<T, false, true, false, true, RES_RESTRICT>(sweeps, a, s);
    case BK_UP: return block_sw<T, false, true, true, false, RES_NONE>(sweeps, a, s);
    case BK_LAST_ZERO: return block_sw<T, false, true, false, true, RES_NONE>(sweeps, a, s);
    case BK_LAST: return block_sw<T, false, true, false, false, RES_NONE>(sweeps, a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_tail(bool fp64, const TailLaunch &t, hipStream_t s)
{
    if (t.a.n_items <= 0) return hipSuccess;
    const dim3 g((unsigned)t.a.n_items), blk(kBlockWaves * kWave);
    if (fp64) hipLaunchKernelGGL(tail_kernel<double>, g, blk, 0, s, t);
    else hipLaunchKernelGGL(tail_kernel<float>, g, blk, 0, s, t);
    return hipGetLastError();
}

hipError_t launch_block_fine(bool zero, int sweeps, bool sor, bool fp64, const BlockLaunch &a, hipStream_t s)
{
    if (fp64) return zero ? fine_sw<double, true>(sweeps, sor, a, s) : fine_sw<double, false>(sweeps, sor, a, s);
    return zero ? fine_sw<float, true>(sweeps, sor, a, s) : fine_sw<float, false>(sweeps, sor, a, s);
}

// Measured against what it replaced.  Neumann (the strip kernel's row march), per
// pass of 3 sweeps: level 1 of 24 x 901 x 1100, 35 -> 18 us up and 27 -> 18 us
// down; level 1 of 6 x 96 x 80 (one block a slice), 25 -> 6.7 and 21 -> 7.3 us.
// Large levels gain least: all coarse passes of 64 x 2048^2, 1.61 -> 1.25 ms a
// call; of 2 x 21504 x 26624, 6.80 -> 6.38 ms.  Periodic (one launch per
// half-sweep over memory), 12 x 1024 x 1200: 8.0 -> 0.55 ms a call.  Regions of
// 128 rows (16 per wave; less halo, 120 registers) were slower on every stack
// but the largest, and there not faster.
hipError_t launch_block(BlockKind k, bool periodic, bool level0, int sweeps, bool fp64, const BlockLaunch &a,
                        hipStream_t s)
{
    return fp64 ? block_t<double>(k, periodic, level0, sweeps, a, s)
                : block_t<float>(k, periodic, level0, sweeps, a, s);
}

}  // namespace gdf
