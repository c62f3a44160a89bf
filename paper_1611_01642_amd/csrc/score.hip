// FP32 window scores of one image with many windows (pd_score_windows; fewer take
// a wave per sub-tile on the matrix cores, score32.hip), on the vector ALUs.
//
// The score of window (i, j) is a 2-D correlation of the feature planes with
// the model:  s(i,j) = sum_c sum_a sum_b F_c[i+a][j+b] * W[a][b][c] + bias.
// One wave64 owns a tile of 64 adjacent window columns (one per lane) x R
// window rows (registers).  For each feature plane c the wave stages the tile's
// (R + 14 or 15) x (64 + 6 or 7) patch in its own LDS region (coalesced loads of
// the next plane are in flight while the current one is used), then every patch
// value a lane reads from LDS serves up to R windows of its column.  Weights are
// wave-uniform (scalar loads).  FP32 products and FP32 sums in a fixed order.
//
// One wave's walk over the 95 planes takes 350 us, whatever the image; with
// enough tiles to fill the chip VALU issue bounds it, and a model costs half of
// what it does in a wave per sub-tile, whose 9 waves load each feature row once
// per two row pairs: 540x960 cells and 8 models 1506 us (there 1763), 1000x2000
// and one 779 (888), 2048x2048 and one 1503 (2017).
#include "pd_internal.h"

namespace pd {
namespace {

constexpr int SC_R = 8;      // window rows per lane
constexpr int SC_WAVES = 4;  // waves (independent tiles) per workgroup

constexpr int HOG_PR = SC_R + PD_WIN_BLOCKS_Y - 1;  // patch rows
constexpr int HOG_PC = SC_W + PD_WIN_BLOCKS_X - 1;  // patch columns
constexpr int LBP_PR = SC_R + PD_WIN_CELLS_Y - 1;
constexpr int LBP_PC = SC_W + PD_WIN_CELLS_X - 1;
constexpr int HOG_N = HOG_PR * HOG_PC, LBP_N = LBP_PR * LBP_PC;
constexpr int HOG_PQ = (HOG_N + 63) / 64;  // patch values per lane
constexpr int LBP_PQ = (LBP_N + 63) / 64;
constexpr int PATCH = HOG_N > LBP_N ? HOG_N : LBP_N;

__device__ __forceinline__ void score_tile(gptr<const float> __restrict__ hog, gptr<const uint8_t> __restrict__ lbp,
                                           int wc, int hc, const float* __restrict__ wt, float bias,
                                           gptr<float> __restrict__ out, int ty, int tx, int lane,
                                           float* __restrict__ patch) {
    const int hb = hc - 1, wb = wc - 1;
    const int ny = hc - PD_WIN_CELLS_Y + 1, nx = wc - PD_WIN_CELLS_X + 1;
    const int i0 = ty * SC_R, j0 = tx * SC_W;
    float acc[SC_R];
#pragma unroll
    for (int r = 0; r < SC_R; ++r) acc[r] = 0.0f;

    {
        const size_t plane = (size_t)hb * wb;
        // clamped byte offsets in a plane of this lane's patch values; the
        // loads are raw buffer loads with the plane's byte offset as a scalar,
        // so no address arithmetic is done per value
        const auto rsrc = planes_rsrc(hog, (uint64_t)PD_HOG_BLOCK * plane * 4);
        uint32_t off[HOG_PQ];
#pragma unroll
        for (int q = 0; q < HOG_PQ; ++q) {
            const int e = min(lane + 64 * q, HOG_N - 1);
            const int row = e / HOG_PC, col = e - row * HOG_PC;
            off[q] = 4u * (uint32_t)(min(i0 + row, hb - 1) * wb + min(j0 + col, wb - 1));
        }
        float pre[HOG_PQ];
#pragma unroll
        for (int q = 0; q < HOG_PQ; ++q)
            pre[q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, off[q], 0, 0));
        for (int c = 0; c < PD_HOG_BLOCK; ++c) {
#pragma unroll
            for (int q = 0; q < HOG_PQ; ++q)
                if (lane + 64 * q < HOG_N) patch[lane + 64 * q] = pre[q];
            if (c + 1 < PD_HOG_BLOCK) {
                const uint32_t pofs = (uint32_t)((c + 1) * plane * 4);
#pragma unroll
                for (int q = 0; q < HOG_PQ; ++q)
                    pre[q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, off[q], pofs, 0));
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll 1
            for (int b = 0; b < PD_WIN_BLOCKS_X; ++b) {
                float wa[PD_WIN_BLOCKS_Y];
#pragma unroll
                for (int a = 0; a < PD_WIN_BLOCKS_Y; ++a) wa[a] = wt[(a * PD_WIN_BLOCKS_X + b) * PD_HOG_BLOCK + c];
                const float* pr = patch + lane + b;
#pragma unroll
                for (int y = 0; y < HOG_PR; ++y) {
                    const float v = pr[y * HOG_PC];
#pragma unroll
                    for (int r = 0; r < SC_R; ++r) {
                        const int a = y - r;
                        if (a >= 0 && a < PD_WIN_BLOCKS_Y) acc[r] = fmaf(v, wa[a], acc[r]);
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    {
        const size_t plane = (size_t)hc * wc;
        const float* wl = wt + PD_HOG_DIM;
        const auto rsrc = planes_rsrc(lbp, (uint64_t)PD_LBP_BINS * plane);
        uint32_t off[LBP_PQ];  // clamped byte offsets in a plane (as for HOG)
#pragma unroll
        for (int q = 0; q < LBP_PQ; ++q) {
            const int e = min(lane + 64 * q, LBP_N - 1);
            const int row = e / LBP_PC, col = e - row * LBP_PC;
            off[q] = (uint32_t)(min(i0 + row, hc - 1) * wc + min(j0 + col, wc - 1));
        }
        uint32_t pre[LBP_PQ];
#pragma unroll
        for (int q = 0; q < LBP_PQ; ++q) pre[q] = __builtin_amdgcn_raw_buffer_load_b8(rsrc, off[q], 0, 0);
        for (int c = 0; c < PD_LBP_BINS; ++c) {
#pragma unroll
            for (int q = 0; q < LBP_PQ; ++q)
                if (lane + 64 * q < LBP_N) patch[lane + 64 * q] = (float)pre[q];
            if (c + 1 < PD_LBP_BINS) {
                const uint32_t pofs = (uint32_t)((c + 1) * plane);
#pragma unroll
                for (int q = 0; q < LBP_PQ; ++q) pre[q] = __builtin_amdgcn_raw_buffer_load_b8(rsrc, off[q], pofs, 0);
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll 1
            for (int b = 0; b < PD_WIN_CELLS_X; ++b) {
                float wa[PD_WIN_CELLS_Y];
#pragma unroll
                for (int a = 0; a < PD_WIN_CELLS_Y; ++a) wa[a] = wl[(a * PD_WIN_CELLS_X + b) * PD_LBP_BINS + c];
                const float* pr = patch + lane + b;
#pragma unroll
                for (int y = 0; y < LBP_PR; ++y) {
                    const float v = pr[y * LBP_PC];
#pragma unroll
                    for (int r = 0; r < SC_R; ++r) {
                        const int a = y - r;
                        if (a >= 0 && a < PD_WIN_CELLS_Y) acc[r] = fmaf(v, wa[a], acc[r]);
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    const int j = j0 + lane;
    if (j < nx) {
#pragma unroll
        for (int r = 0; r < SC_R; ++r) {
            const int i = i0 + r;
            if (i < ny) out[(size_t)i * nx + j] = acc[r] + bias;
        }
    }
}

__global__ void __launch_bounds__(256) score_single_kernel(LevelItem it, const float* __restrict__ wt,
                                                           const float* __restrict__ bias, int n_models) {
    __shared__ float patches[SC_WAVES][PATCH];
    const int local_wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave = blockIdx.x * SC_WAVES + local_wave;
    const int ntx = ceil_div(it.nx, SC_W), nty = ceil_div(it.ny, SC_R);
    const int per_model = ntx * nty;
    if (wave >= per_model * n_models) return;
    const int m = wave / per_model;
    const int local = wave - m * per_model;
    score_tile(gmem(it.hog), gmem(it.lbp), it.wc, it.hc, wt + (size_t)m * PD_FEATURE_DIM, bias[m],
               gmem(it.scores) + (size_t)m * it.ny * it.nx, local / ntx, local % ntx, threadIdx.x & 63,
               patches[local_wave]);
}

}  // namespace

hipError_t launch_score_single(const LevelItem& it, const float* weights, const float* bias, int n_models,
                               hipStream_t s) {
    if (it.nx <= 0 || it.ny <= 0 || n_models <= 0) return hipSuccess;
    const int64_t entries = score32_wave_entries(it.ny, it.wc) * n_models;
    if (score_single_by_waves(entries)) return launch_score32_waves_single(it, weights, bias, n_models, s);
    const int waves = ceil_div(it.nx, SC_W) * ceil_div(it.ny, SC_R) * n_models;
    score_single_kernel<<<ceil_div(waves, SC_WAVES), 64 * SC_WAVES, 0, s>>>(it, weights, bias, n_models);
    return hipGetLastError();
}

}  // namespace pd
