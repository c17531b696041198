// Arguments of the anisotropic smoothing (smooth_impl.h).
#pragma once
#include "device.h"

namespace gdf {

constexpr int kSmoothWaves = 8;   // waves per smoothing workgroup (one partial-sum slot each)
#ifndef GDF_SMOOTH_TILE_H
#define GDF_SMOOTH_TILE_H 24
#endif
// smoothing tile: one workgroup per kSmoothTileW x kSmoothTileH tile of every slice
constexpr int kSmoothTileW = 64, kSmoothTileH = GDF_SMOOTH_TILE_H;
static_assert(kSmoothTileH % kSmoothWaves == 0, "whole rows per thread");

struct SmoothArgs {
    const uint8_t *stack;
    long long pitch_row, pitch_slice;
    int S, H, W;
    int rxy, rz;
    double wxy[8];        // in-plane taps (0..rxy)
    double wz[16];        // cross-slice taps (0..rz)
    double alpha;
    float wxy_f[8];       // the same taps rounded to FP32 (FP32 kernel: kept in scalar registers)
    float wz_f[16];
    float alpha_f;
    int z_lo, z_hi;       // the output slices: [z_lo, z_hi) of the S (the others only feed
                          // their cross-slice windows); b_u, the level-1 right-hand side and
                          // the partial sums of slice z go to index z - z_lo
    void *gs_out;         // optional smoothed slices (contiguous [gs_zhi - gs_zlo][H][W])
    int gs_zlo, gs_zhi;   // output slices [gs_zlo, gs_zhi) are stored into gs_out (slice z at z - gs_zlo)
    void *b0;                 // level-0 right-hand side of slice 0 (b_u is written there);
                              // null: neither b_u nor the partial sums are stored
    long long b_slice_stride; // elements between consecutive slices' level-0 right-hand sides
    int b_pitch;              // its row pitch (elements)
    // 1 / (sum of the z taps inside the stack) for an output slice with lo
    // taps below it and hi above it inside the stack: inv_wz[lo][hi], lo, hi <= rz
    double inv_wz[13][13];
    float inv_wz_f[13][13];
    double *part_bb;      // [z_hi - z_lo][tiles] partial ||alpha g_s + L g_o||^2
    double *part_b0;      // [z_hi - z_lo][tiles] partial ||b_u||^2
    double *part_bs;      // [z_hi - z_lo][tiles] partial sum(b_u)
    int tiles_x, tiles_y;
    // optional (FP32): level-1 right-hand side (bfloat16) of slice 0, written as
    // the sum of each coarse cell's children's b_u (no mean removed); slices are
    // bc_slice_stride elements apart, rows bc_pitch
    void *bc0;
    long long bc_slice_stride;
    int bc_pitch;
    int robust;           // robust cross-slice averaging (FP32 only)
};

hipError_t launch_smooth(bool fp64, const SmoothArgs &a, hipStream_t s);

}  // namespace gdf
