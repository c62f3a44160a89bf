// FP64 rescoring of near-threshold windows.
//
// After BF16 scoring, a window whose score lies within `margin` of its
// frame's threshold cannot be classified safely (Section 4.4: positive iff
// the distance to the hyper-plane exceeds the threshold).  This kernel
// recomputes such a window's features from the pixels of its pyramid level in
// FP64 -- gradients (Algorithm 4; orientation and magnitude from a table of
// every integer gradient, built in FP64 with the device's double atan2), trilinear
// HOG votes (Algorithm 5) as per-cell direction partials, L2-Hys -- and its LBP
// counts (exact integers), and scores every model in FP64 with the FP32 weights.  A window whose FP64 score (max over models)
// exceeds the threshold is appended to the frame's candidate list.
//
// A workgroup of two waves takes a near window, a lane one of its 128 cells and,
// after the votes, the block whose top left cell that is:
//  * pixels (130 x 66 with halo): gathered into LDS, every load of a thread in
//    flight before its first store; as words at any alignment where the window
//    allows it;
//  * LBP: a lane codes its cell's pixels, four per word, and counts them in LDS
//    (reading the counts from the feature planes, 944 runs of 8 bytes, each on a
//    cache line of its own, took 15 to 50 thousand cycles);
//  * votes: a row of 8 pixels is summed into 27 registers (3 target columns x 9
//    bins, the linear orientation vote as a hat over the 9 bins), which then
//    go to the two target rows with the row's weights; half a row's table
//    entries are in flight during the other half's votes.  No sum crosses
//    lanes;
//  * blocks: a lane adds its right neighbour's partials (data-parallel moves)
//    and those of the cell below (through LDS, first the votes upwards, then
//    the cell's own), and normalises its block in registers;
//  * dot products: all lanes stride over the features, four at a time, with
//    coalesced weights (a lane's own block against its 36 weights, a cache line
//    per lane and load, took 35000 cycles for 8 models), and a fixed-order
//    reduction.
//
// What bounds it is the FP64 arithmetic of the votes (about 50 instructions per
// pixel) and the two waves' latency; 38 KB of LDS and 256 registers leave room
// for four windows per CU.  A workgroup of four waves with the partials of nine
// cell rows in LDS (72 KB, two windows per CU; four lanes per cell, their sums
// meeting in 162 cross-lane exchanges per half window; one wave building the
// blocks) took 121 us for 1333 windows of one model and 94 for 663 of eight;
// this takes 70 and 50 (330 windows of one model: 37 and 29).
#include "lbp_codes.h"
#include "pd_internal.h"

namespace pd {
namespace {

__constant__ LbpTable kLbpRescore = make_lbp_table();

typedef uint32_t __attribute__((aligned(1))) u32_any;
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

constexpr int RS_THREADS = PD_WIN_CELLS_Y * PD_WIN_CELLS_X;  // 128: a thread per cell
constexpr int RS_PY = PD_WIN_H + 2;  // 130 pixel rows incl. halo
constexpr int RS_PX = PD_WIN_W + 2;  // 66 pixel columns incl. halo

// LDS pixel rows: byte RS_PX0 + c holds window column c - 1 (c = 0 .. 65),
// so that a row's source bytes from a word boundary of the window's columns
// land on aligned LDS words, and a cell's 8 pixels are two of them
constexpr int RS_PX0 = 3;
constexpr int RS_ROW = 72;                 // 18 words per row
constexpr int RS_ROW_WORDS = RS_ROW / 4;

struct RescoreShared {
    union {
        struct {
            double below[18][RS_THREADS];  // a cell's votes for the blocks that begin in the row above
            uint8_t px[RS_PY][RS_ROW];     // the window's pixels
        };
        double hog[PD_HOG_DIM];  // then its HOG values
    };
    uint32_t lbp[PD_LBP_DIM / 4];   // its LBP counts, bytes in feature order (cell, bin)
    uint8_t bin[256];               // of a bit-reversed code
    double part[RS_THREADS / 64][8];  // per wave and model
};

constexpr int RS_PX_PER_T = (RS_PY * RS_PX + RS_THREADS - 1) / RS_THREADS;   // pixel bytes per thread (border windows)
constexpr int RS_PXW_PER_T = (RS_PY * RS_ROW_WORDS + RS_THREADS - 1) / RS_THREADS;  // pixel words per thread (inner)
// Bilinear weight of pixel offset p in [0, 8) of a cell towards cell d in {-1, 0, 1}.
__device__ __forceinline__ double spatial_w(int p, int d) {
    const double w = 1.0 - fabs((double)p + 0.5 - (8.0 * d + 4.0)) / 8.0;
    return w > 0.0 ? w : 0.0;
}

// The value of the lane to the right (the cell to the right: rows of 8 cells lie
// within a row of 16 lanes).
__device__ __forceinline__ double right_lane(double v) {
    const uint64_t u = __double_as_longlong(v);
    constexpr int ROW_SHL1 = 0x101;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, ROW_SHL1, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), ROW_SHL1, 0xf, 0xf, true);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// Each model's dot product over the features [4 g_begin, 4 g_end), four at a time
// (one 16-byte weight load per model; HOG and LBP begin at multiples of 4), U
// groups per turn in flight together; M = 1 or 8 models unrolled (models past
// n_models repeat the last one; their sums are never read).
template <int M>
__device__ __forceinline__ void dot_models(RescoreShared& sm, const float* __restrict__ weights, int n_models,
                                           int g_begin, int g_end, int t) {
    static_assert(PD_HOG_DIM % 4 == 0 && PD_LBP_DIM % 4 == 0, "groups of one family");
    constexpr int U = M == 1 ? 4 : 2;
    double part[M];
#pragma unroll
    for (int m = 0; m < M; ++m) part[m] = 0.0;
#pragma unroll 1
    for (int g0 = g_begin + t; g0 < g_end; g0 += RS_THREADS * U) {
        f32x4_any w[U][M];
        double x[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int g = min(g0 + RS_THREADS * u, g_end - 1);
#pragma unroll
            for (int m = 0; m < M; ++m)
                w[u][m] = *reinterpret_cast<const f32x4_any*>(weights + (size_t)min(m, n_models - 1) * PD_FEATURE_DIM +
                                                              4 * g);
            if (g < PD_HOG_DIM / 4) {
#pragma unroll
                for (int j = 0; j < 4; ++j) x[u][j] = sm.hog[4 * g + j];
            } else {
                const uint32_t b = sm.lbp[g - PD_HOG_DIM / 4];
#pragma unroll
                for (int j = 0; j < 4; ++j) x[u][j] = (double)((b >> (8 * j)) & 255u);
            }
            if (g0 + RS_THREADS * u >= g_end) {
#pragma unroll
                for (int j = 0; j < 4; ++j) x[u][j] = 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int j = 0; j < 4; ++j) part[m] = fma(x[u][j], (double)w[u][m][j], part[m]);
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
        double s = part[m];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
        if ((t & 63) == 0) sm.part[t >> 6][m] = s;
    }
}

// A row of a cell's neighbourhood: its 8 pixels and those shifted by one.
struct LbpRow {
    uint32_t own[2], left[2], right[2];
    __device__ __forceinline__ void load(const uint8_t* p) {  // p: the first pixel, a word boundary
        own[0] = *reinterpret_cast<const uint32_t*>(p);
        own[1] = *reinterpret_cast<const uint32_t*>(p + 4);
        left[0] = own[0] << 8 | p[-1];
        left[1] = __builtin_amdgcn_alignbyte(own[1], own[0], 3);
        right[0] = __builtin_amdgcn_alignbyte(own[1], own[0], 1);
        right[1] = own[1] >> 8 | (uint32_t)p[8] << 24;
    }
};

// Adds the codes of cell t to its counts (cells share words at their ends).
__device__ __forceinline__ void count_lbp(RescoreShared& sm, int t) {
    const int cy = t / PD_WIN_CELLS_X, cx = t % PD_WIN_CELLS_X;
    const uint8_t* p = &sm.px[PD_CELL * cy][RS_PX0 + 1 + PD_CELL * cx];
    LbpRow U, C, D, N;
    U.load(p);
    C.load(p + RS_ROW);
    D.load(p + 2 * RS_ROW);
#pragma unroll 2
    for (int py = 0; py < PD_CELL; ++py) {
        N.load(p + min(py + 3, PD_CELL + 1) * RS_ROW);
#pragma unroll
        for (int hw = 0; hw < 2; ++hw) {
            // Algorithm 1's neighbours in its bit order
            const uint32_t nb[8] = {U.left[hw],  U.own[hw], U.right[hw], C.right[hw],
                                    D.right[hw], D.own[hw], D.left[hw],  C.left[hw]};
            uint32_t r[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) r[k] = ge_bytes(nb[k], C.own[hw], C.own[hw] & 0x7f7f7f7fu);
            const uint32_t code = lbp_codes4(r);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t e = PD_LBP_BINS * t + sm.bin[code >> (8 * u) & 255u];
                atomicAdd(&sm.lbp[e >> 2], 1u << (8 * (e & 3u)));
            }
        }
        U = C;
        C = D;
        D = N;
    }
}

// The votes of one cell (cy, cx), rows py0 .. py0 + 3 (a half): acc[0] towards
// the cells of the row above (py0 = 0) or its own (4), acc[1] its own or the row
// below; [dx + 1][bin].  Adds to acc.
__device__ __forceinline__ void half_votes(const RescoreShared& sm, const double2* __restrict__ orient, int cy, int cx,
                                           int py0, double (&acc)[2][3][PD_HOG_BINS]) {
    // pixels px0 .. px0 + 3 of row py: their table entries
    auto entries = [&](int py, int px0, double2 (&g)[4]) __attribute__((always_inline)) {
        const uint8_t* const row = &sm.px[PD_CELL * cy + py + 1][RS_PX0 + 1 + PD_CELL * cx + px0];
        const uint32_t up = *reinterpret_cast<const uint32_t*>(row - RS_ROW);
        const uint32_t down = *reinterpret_cast<const uint32_t*>(row + RS_ROW);
        const uint32_t own = *reinterpret_cast<const uint32_t*>(row);
        const int left = row[-1], right = row[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int a = u > 0 ? (int)(own >> (8 * (u - 1)) & 255u) : left;
            const int b = u < 3 ? (int)(own >> (8 * (u + 1)) & 255u) : right;
            const int dx = a - b;  // Algorithm 4
            const int dy = (int)(up >> (8 * u) & 255u) - (int)(down >> (8 * u) & 255u);
            g[u] = orient[abs(dy) * ORIENT_W + (dy < 0 ? -dx : dx) + 255];
        }
    };
    double R[3][PD_HOG_BINS];  // the row's sums
    auto votes = [&](int px0, const double2 (&g)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double tb = g[u].x, mag = g[u].y;
            const int q = px0 == 0 ? 0 : 1;  // target columns q - 1 and q (as dx)
            const double m0 = mag * spatial_w(px0 + u, q - 1), m1 = mag * spatial_w(px0 + u, q);
#pragma unroll
            for (int k = 0; k < PD_HOG_BINS; ++k) {
                // linear vote for the bin (wrap-around)
                const double d = k == 0 ? fmin(fabs(tb), fabs(tb - 9.0))
                                        : k == PD_HOG_BINS - 1 ? fmin(fabs(tb - 8.0), fabs(tb + 1.0))
                                                               : fabs(tb - (double)k);
                const double h = fmin(fmax(1.0 - d, 0.0), 1.0);  // one addition with its result clamped (d >= 0)
                R[q][k] = fma(m0, h, R[q][k]);
                R[q + 1][k] = fma(m1, h, R[q + 1][k]);
            }
        }
    };
    double2 g0[4], g1[4];
    entries(py0, 0, g0);
#pragma unroll 1
    for (int py = py0; py < py0 + 4; ++py) {
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
            for (int k = 0; k < PD_HOG_BINS; ++k) R[b][k] = 0.0;
        entries(py, 4, g1);
        votes(0, g0);
        entries(min(py + 1, py0 + 3), 0, g0);
        votes(4, g1);
        const double w0 = spatial_w(py, (py0 >> 2) - 1), w1 = spatial_w(py, py0 >> 2);
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
            for (int k = 0; k < PD_HOG_BINS; ++k) {
                acc[0][b][k] = fma(w0, R[b][k], acc[0][b][k]);
                acc[1][b][k] = fma(w1, R[b][k], acc[1][b][k]);
            }
    }
}

__global__ void __launch_bounds__(RS_THREADS) __attribute__((amdgpu_waves_per_eu(2))) rescore64_kernel(
    const LevelItem* __restrict__ items, const int32_t* __restrict__ first_item, int n_frames,
    const int32_t* __restrict__ near_count, const int4* __restrict__ near_key, const float* __restrict__ weights,
    const float* __restrict__ bias, int n_models, int features, double clip, double eps,
    const double* __restrict__ thresholds, int32_t* __restrict__ counters, float* __restrict__ cand_score,
    int4* __restrict__ cand_key, double* __restrict__ cand_s64, const double2* __restrict__ orient) {
    __shared__ RescoreShared sm;
    const int t = threadIdx.x;
    const bool use_hog = (features & PD_FEAT_HOG) != 0, use_lbp = (features & PD_FEAT_LBP) != 0;
    const int cy = t / PD_WIN_CELLS_X, cx = t % PD_WIN_CELLS_X;
    const int block = cy < PD_WIN_BLOCKS_Y && cx < PD_WIN_BLOCKS_X ? cy * PD_WIN_BLOCKS_X + cx : -1;
    if (use_lbp)
        for (int c = t; c < 256; c += RS_THREADS) sm.bin[c] = kLbpRescore.bin[__brev(c) >> 24];
    const int total = near_count[n_frames];  // dense list of every frame's near windows
    for (int q = blockIdx.x; q < total; q += gridDim.x) {
        const int4 key = near_key[q];
        const int f = key.x / PD_MAX_LEVELS, level = key.x - f * PD_MAX_LEVELS;
        const LevelItem& it = items[first_item[f] + level];
        const int wi = key.y, wj = key.z;

        // the thread index as a value opaque to the compiler, so the gathers'
        // index arithmetic stays in the loop instead of being held in
        // registers across windows
        int tt = t;
        asm volatile("" : "+v"(tt));
        if (use_lbp)
            for (int e = tt; e < PD_LBP_DIM / 4; e += RS_THREADS) sm.lbp[e] = 0u;
        // pixels of the window + one halo pixel: every load of a thread in
        // flight together, then the LDS stores.  A window whose halo, and the
        // three pixels after it, lie inside the level reads words (at any
        // alignment: level 0 is the caller's frame), so that no word leaves the
        // row; others read bytes, clamped to the level.
        const bool inner = wi > 0 && wj > 0 && PD_CELL * wi + PD_WIN_H < it.h && PD_CELL * wj + PD_WIN_W + 4 <= it.w;
        if (inner) {
            const auto base = it.pyr + (size_t)(PD_CELL * wi - 1) * it.pitch + (PD_CELL * wj - 4);
            uint32_t v[RS_PXW_PER_T];
#pragma unroll
            for (int k = 0; k < RS_PXW_PER_T; ++k) {
                const int e = min(tt + RS_THREADS * k, RS_PY * RS_ROW_WORDS - 1);
                const int r = e / RS_ROW_WORDS, d = e - r * RS_ROW_WORDS;
                v[k] = *reinterpret_cast<const u32_any*>(base + (size_t)r * it.pitch + 4 * d);
            }
#pragma unroll
            for (int k = 0; k < RS_PXW_PER_T; ++k) {
                const int e = tt + RS_THREADS * k;
                if (e < RS_PY * RS_ROW_WORDS) reinterpret_cast<uint32_t*>(&sm.px[0][0])[e] = v[k];
            }
        } else {
            uint32_t v[RS_PX_PER_T];
#pragma unroll
            for (int k = 0; k < RS_PX_PER_T; ++k) {
                const int e = min(tt + RS_THREADS * k, RS_PY * RS_PX - 1);
                const int r = e / RS_PX, c = e - (e / RS_PX) * RS_PX;
                const int y = min(max(PD_CELL * wi - 1 + r, 0), it.h - 1);
                const int x = min(max(PD_CELL * wj - 1 + c, 0), it.w - 1);
                v[k] = it.pyr[(size_t)y * it.pitch + x];
            }
#pragma unroll
            for (int k = 0; k < RS_PX_PER_T; ++k) {
                const int e = tt + RS_THREADS * k;
                if (e < RS_PY * RS_PX) {
                    const int r = e / RS_PX, c = e - (e / RS_PX) * RS_PX;
                    sm.px[r][RS_PX0 + c] = (uint8_t)v[k];
                }
            }
        }
        __syncthreads();
        if (use_lbp) count_lbp(sm, t);

        if (use_hog) {
            // slot (r, c) of the block that begins at this cell: the four cells'
            // partials aimed at it (exactly Algorithm 5's votes)
            double v[PD_HOG_BLOCK];
            // what the block's own row (this cell and the one to its right)
            // gives its left (c = 0) and right (c = 1) column
            auto pair = [](const double (&x)[3][PD_HOG_BINS], int c, int k) {
                return x[1 + c][k] + right_lane(x[c][k]);
            };
            double acc[2][3][PD_HOG_BINS];
            auto clear = [&](int a) {
#pragma unroll
                for (int b = 0; b < 3; ++b)
#pragma unroll
                    for (int k = 0; k < PD_HOG_BINS; ++k) acc[a][b][k] = 0.0;
            };
            clear(0);
            clear(1);
            half_votes(sm, orient, cy, cx, 0, acc);
            // acc[0]: votes upwards, for the blocks that begin in the row above
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int k = 0; k < PD_HOG_BINS; ++k) sm.below[c * PD_HOG_BINS + k][t] = pair(acc[0], c, k);
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
                for (int k = 0; k < PD_HOG_BINS; ++k) acc[0][b][k] = acc[1][b][k];
            clear(1);
            half_votes(sm, orient, cy, cx, 4, acc);
            // acc[0]: votes for the cell's own row, acc[1]: downwards
            const int under = min(t + PD_WIN_CELLS_X, RS_THREADS - 1);
            __syncthreads();
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int k = 0; k < PD_HOG_BINS; ++k)
                    v[c * PD_HOG_BINS + k] = pair(acc[0], c, k) + sm.below[c * PD_HOG_BINS + k][under];
            __syncthreads();
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int k = 0; k < PD_HOG_BINS; ++k) sm.below[c * PD_HOG_BINS + k][t] = pair(acc[0], c, k);
            __syncthreads();
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int k = 0; k < PD_HOG_BINS; ++k)
                    v[(2 + c) * PD_HOG_BINS + k] = pair(acc[1], c, k) + sm.below[c * PD_HOG_BINS + k][under];
            double ss = 0.0;
#pragma unroll
            for (int k = 0; k < PD_HOG_BLOCK; ++k) ss += v[k] * v[k];
            double inv = 1.0 / sqrt(ss + eps * eps);
            double ss2 = 0.0;
#pragma unroll
            for (int k = 0; k < PD_HOG_BLOCK; ++k) {
                v[k] = fmin(v[k] * inv, clip);
                ss2 += v[k] * v[k];
            }
            inv = 1.0 / sqrt(ss2 + eps * eps);
#pragma unroll
            for (int k = 0; k < PD_HOG_BLOCK; ++k) v[k] *= inv;
            __syncthreads();  // the votes (and pixels) are read
            if (block >= 0) {
#pragma unroll
                for (int k = 0; k < PD_HOG_BLOCK; ++k) sm.hog[block * PD_HOG_BLOCK + k] = v[k];
            }
        }
        __syncthreads();
        const int g_begin = use_hog ? 0 : PD_HOG_DIM / 4, g_end = use_lbp ? PD_FEATURE_DIM / 4 : PD_HOG_DIM / 4;
        if (n_models == 1) dot_models<1>(sm, weights, 1, g_begin, g_end, t);
        else dot_models<8>(sm, weights, n_models, g_begin, g_end, t);
        __syncthreads();
        if (t == 0) {
            double best = 0.0;
            int bm = 0;
            for (int m = 0; m < n_models; ++m) {
                const double s = (sm.part[0][m] + sm.part[1][m]) + (double)bias[m];
                if (m == 0 || s > best) {
                    best = s;
                    bm = m;
                }
            }
            if (best > thresholds[f]) {
                const int pos = atomicAdd(&counters[f], 1);
                if (pos < it.cand_cap) {  // always: a window is appended once at most
                    const size_t o = (size_t)it.cand_off + pos;
                    cand_score[o] = (float)best;
                    cand_key[o] = make_int4(level, wi, wj, bm);
                    cand_s64[o] = best;
                }
            }
        }
        __syncthreads();
    }
}

}  // namespace

hipError_t launch_rescore64(const LevelItem* items, const int32_t* frame_first_item, int n_frames,
                            const int32_t* near_count, const int4* near_key, const float* weights, const float* bias,
                            int n_models, int features, float clip, float eps, const double* thresholds,
                            int32_t* counters, float* cand_score, int4* cand_key, double* cand_s64,
                            const double2* orient, hipStream_t s) {
    if (n_frames <= 0) return hipSuccess;
    // persistent workgroups (four per CU) over the dense near list, whose length
    // is read on the device
    const int grid = 1024;
    rescore64_kernel<<<grid, RS_THREADS, 0, s>>>(items, frame_first_item, n_frames, near_count, near_key, weights, bias,
                                         n_models, features, (double)clip, (double)eps, thresholds, counters,
                                         cand_score, cand_key, cand_s64, orient);
    return hipGetLastError();
}

}  // namespace pd
