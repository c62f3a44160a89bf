// The learned window pruner: a 68-32-32-16 conv3x3 network with a 1x1
// sigmoid head over the per-cell feature map of every pyramid level, trained
// on the GPU with these kernels.  The network is not part of the paper; it
// predicts which windows the linear SVM of Section 4.4 will score above the
// threshold, so the others need not be scored.
//
// Layout: every map is planar FP32 [C][hc][wc]; one item per map (a pyramid
// level of a frame) carries pointers to its cell map, activations, gradient
// buffers, logits, labels and mask.  Work tiles are 64 consecutive cells of
// one row.
//
// The contractions run on v_mfma_f32_16x16x4_f32: FP32 products and sums, and
// the instruction adds its four products to the accumulator one by one, k
// ascending, each step rounded like fmaf (checked on 512,000 random outputs),
// so a chain of them is the chain of fmaf it replaces, bit for bit.
//
//  * conv3x3 (zero padding): a wave owns a tile (M = 16 cells, up to 4 times),
//    N = 16 output channels, K = (input channel, tap).  Four input channels'
//    3 x 66 neighbourhoods pass through the wave's LDS at a time (the next
//    four's loads in flight), the layer's weights lie in LDS in fragment order.
//    The same kernel computes the data gradient with the flipped, transposed
//    weights and the ReLU mask of the layer below.  The last layer fuses the
//    1x1 head.
//  * weight gradients: dW[o][c][u][v] = sum over cells of dZ[o] x X[c] at
//    offset (u - 1, v - 1): M = output channels, N = input channels of one tap,
//    K = cells.  A fixed set of workgroups strides over the tiles (both
//    operands staged in LDS); per-workgroup partials are then summed in FP64 in
//    a fixed order, so gradients are bitwise reproducible.
//  * loss: class-weighted binary cross-entropy over the masked cells; the
//    gradients are accumulated un-normalised and divided by the number of
//    masked cells in the final reduction.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "packed.h"
#include "pd_internal.h"

namespace pd {
namespace {

constexpr int NW = 64;  // cells per tile
constexpr int NWAVES = 4;
constexpr int HALO_W = NW + 2;
constexpr int PATCH = 3 * HALO_W;  // one channel's neighbourhood of a tile
// LDS stride of a channel's neighbourhood: 12 banks on, so that 16 channels x 4
// consecutive cells (and 16 cells of 4 channels) fall in distinct banks
constexpr int CH_S = 204;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// a byte offset past every buffer: the load returns zero
constexpr uint32_t NOWHERE = 0x80000000u;

// ---- FP32 convolution on the matrix cores -----------------------------------
// The vector-ALU form of this (a lane per cell, all output channels in
// registers) took 717 us for the five convolutions of a step of eight 1242x375
// frames, bound by VALU issue; this one takes 365 (floor 235: 28 GFLOP at the
// FP32 matrix rate; per tile, the first block's loads and the output are not
// overlapped with the products).
constexpr int CV_WAVES = 8;  // tiles in work per workgroup

template <int CIN, int COUT, bool HEAD>
__global__ void __launch_bounds__(64 * CV_WAVES) conv3x3_kernel(const NetItem* __restrict__ items,
                                                                const Tile* __restrict__ tiles, int n_tiles,
                                                                int in_slot, int out_slot, int mask_slot,
                                                                const float* __restrict__ frags,
                                                                const float* __restrict__ bias, int relu,
                                                                const float* __restrict__ head) {
    constexpr int NT = COUT / 16;        // N tiles
    constexpr int BLOCKS = CIN / 4;      // channel blocks: 36 K values, 9 MFMAs deep
    constexpr int STAGE = HEAD && 16 * (NW + 1) > 4 * CH_S ? 16 * (NW + 1) : 4 * CH_S;
    constexpr int PER = (4 * PATCH + 63) / 64;
    __shared__ __attribute__((aligned(16))) float ws[CIN * 9 * COUT];
    __shared__ float stage[CV_WAVES][STAGE];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, col = lane & 15, kk = lane >> 4;
    for (int e = threadIdx.x; e < CIN * 9 * COUT / 4; e += 64 * CV_WAVES)
        reinterpret_cast<f32x4*>(ws)[e] = reinterpret_cast<const f32x4*>(frags)[e];
    __syncthreads();
    float* const st = stage[wave];
    int aoff[9];  // this lane's A element of MFMA j of a block: K value 4 j + kk = (channel, tap)
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        const int k = 4 * j + kk, c = k / 9, t = k - 9 * c;
        aoff[j] = c * CH_S + (t / 3) * HALO_W + t % 3 + col;
    }
    for (int task = blockIdx.x * CV_WAVES + wave; task < n_tiles; task += gridDim.x * CV_WAVES) {
        const Tile tl = tiles[task];
        const NetItem& it = items[tl.item];
        const int wc = it.wc, hc = it.hc, p = tl.ty, q0 = tl.tx * NW;
        const uint32_t plane = (uint32_t)hc * (uint32_t)wc;
        const auto rs = planes_rsrc(it.buf[in_slot], (uint64_t)CIN * plane * 4);
        // staged element e = (channel of the block, row r, column) holds
        // in[c][p - 1 + r][q0 - 1 + column], zero outside the map
        uint32_t off[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int e = lane + 64 * i, c = e / PATCH, rem = e - c * PATCH, r = rem / HALO_W;
            const int y = p - 1 + r, x = q0 - 1 + rem - r * HALO_W;
            const bool in = c < 4 && y >= 0 && y < hc && x >= 0 && x < wc;
            off[i] = in ? 4u * ((uint32_t)c * plane + (uint32_t)(y * wc + x)) : NOWHERE;
        }
        float pre[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i)
            pre[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off[i], 0, 0));
        f32x4 acc[4][NT];
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            const float b0 = bias ? bias[16 * n + col] : 0.0f;
#pragma unroll
            for (int m = 0; m < 4; ++m) acc[m][n] = f32x4{b0, b0, b0, b0};
        }
        auto walk = [&](auto tiles_m) __attribute__((always_inline)) {
            constexpr int NM = decltype(tiles_m)::value;
            for (int cb = 0; cb < BLOCKS; ++cb) {
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    const int e = lane + 64 * i, c = e / PATCH;
                    if (e < 4 * PATCH) st[c * CH_S + e - c * PATCH] = pre[i];
                }
                if (cb + 1 < BLOCKS) {
#pragma unroll
                    for (int i = 0; i < PER; ++i)
                        pre[i] = __builtin_bit_cast(
                            float, __builtin_amdgcn_raw_buffer_load_b32(rs, off[i], 16u * (uint32_t)(cb + 1) * plane, 0));
                }
                __builtin_amdgcn_wave_barrier();
                const float* const wb = ws + cb * 9 * NT * 64 + lane;
#pragma unroll
                for (int j = 0; j < 9; ++j) {
                    float a[NM], b[NT];
#pragma unroll
                    for (int m = 0; m < NM; ++m) a[m] = st[aoff[j] + 16 * m];
#pragma unroll
                    for (int n = 0; n < NT; ++n) b[n] = wb[(j * NT + n) * 64];
#pragma unroll
                    for (int m = 0; m < NM; ++m)
#pragma unroll
                        for (int n = 0; n < NT; ++n)
                            acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m], b[n], acc[m][n], 0, 0, 0);
                }
                __builtin_amdgcn_wave_barrier();
            }
        };
        const int nm = min(4, (wc - q0 + 15) >> 4);  // M tiles with cells of the map (uniform)
        if (nm > 2) walk(std::integral_constant<int, 4>{});
        else walk(std::integral_constant<int, 2>{});
        // lane holds channel 16 n + col of cells 16 m + 4 kk + v
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int q = q0 + 16 * m + 4 * kk;
            const size_t at = (size_t)p * wc + q;
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                f32x4& d = acc[m][n];
                const size_t o = (size_t)(16 * n + col) * plane;
                if (relu) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) d[v] = fmaxf(d[v], 0.0f);
                }
                if (HEAD) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) st[col * (NW + 1) + 16 * m + 4 * kk + v] = d[v];
                }
                if (mask_slot >= 0) {  // data gradient through the ReLU of the layer below
                    const float* a = it.buf[mask_slot] + o + at;
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (q + v < wc) d[v] = a[v] > 0.0f ? d[v] : 0.0f;
                }
                if (out_slot >= 0) {
                    float* out = it.buf[out_slot] + o + at;
                    if (q + 3 < wc) {
                        *reinterpret_cast<f32x4_any*>(out) = d;
                    } else {
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (q + v < wc) out[v] = d[v];
                    }
                }
            }
        }
        if (HEAD) {
            __builtin_amdgcn_wave_barrier();
            float z = head[COUT];
#pragma unroll
            for (int o = 0; o < COUT; ++o) z = fmaf(head[o], st[o * (NW + 1) + lane], z);
            if (q0 + lane < wc) it.logit[(size_t)p * wc + q0 + lane] = z;
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// ---- weight gradients on the matrix cores ------------------------------------
// Partials of one layer.  A workgroup of 16 waves stages a tile's dZ and X (two
// LDS buffers, the next tile's loads in flight) and splits the products over
// WM groups of 16 output channels x WN sets of (16 input channels, tap) N tiles
// x WK sets of the tile's 16 K steps; the WK sums meet in LDS at the end.  The
// vector-ALU form (a thread per output channel and channel group, one LDS read
// per 9 or fewer products) took 1385 us for the three layers of a step of eight
// 1242x375 frames; this one takes 306 (floor 180).
constexpr int WG_THREADS = 1024;
constexpr int DZ_S = NW + 4;  // LDS stride of dZ: 16 channels x 4 cells in distinct banks

template <int CIN, int COUT>
struct WgradShape {
    static constexpr int WM = COUT / 16, WN = CIN > 32 ? 4 : 2, WK = 16 / (WM * WN);
    static constexpr int TILES = (CIN + 15) / 16 * 9;         // N tiles
    static constexpr int NPW = (TILES + WN - 1) / WN;         // of a wave
    static constexpr int NOUT = COUT * CIN * 9 + COUT;
    static constexpr int BUF = CIN * CH_S + COUT * DZ_S;      // floats of one staged tile
    static constexpr int RED = (WK - 1) * WM * WN * NPW * 256;
    static constexpr int LDS = 2 * BUF > RED ? 2 * BUF : RED;
};

template <int CIN, int COUT>
__global__ void __launch_bounds__(WG_THREADS) wgrad_kernel(const NetItem* __restrict__ items,
                                                           const Tile* __restrict__ tiles, int n_tiles, int x_slot,
                                                           int dz_slot, float* __restrict__ partial) {
    using S = WgradShape<CIN, COUT>;
    // X: threads 0 .. 989 take one place of the neighbourhood in XG channels at
    // a time, so that a tile costs one address and a scalar offset per load
    constexpr int XG = WG_THREADS / PATCH, XPER = (CIN + XG - 1) / XG, DPER = COUT * NW / WG_THREADS;
    __shared__ float sh[S::LDS];
    __shared__ float bsh[WG_THREADS];
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, kk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % S::WM, wn = wave / S::WM % S::WN, wk = wave / (S::WM * S::WN);
    int boff[S::NPW];  // this lane's B element of the wave's N tiles (channels past CIN read the last one)
#pragma unroll
    for (int i = 0; i < S::NPW; ++i) {
        const int n = min(wn + S::WN * i, S::TILES - 1), g = n / 9, t = n - 9 * g;
        boff[i] = min(16 * g + col, CIN - 1) * CH_S + (t / 3) * HALO_W + t % 3 + kk + 4 * wk;
    }
    const int aoff = CIN * CH_S + (16 * wm + col) * DZ_S + kk + 4 * wk;
    const int xg = tid / PATCH, xr = (tid - xg * PATCH) / HALO_W, xcol = tid - xg * PATCH - xr * HALO_W;
    f32x4 acc[S::NPW];
#pragma unroll
    for (int i = 0; i < S::NPW; ++i) acc[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float accb = 0.0f;  // bias gradient: channel tid % COUT, DPER cells per tile
    float xv[XPER], dv[DPER];
    // A tile's place: read (two dependent scalar loads) a tile before its pixels
    // are, so that no wave waits for it between the barrier and its products.
    struct Place {
        const float *x, *dz;
        int wc, hc, p, q0;
    };
    auto place = [&](int ti) __attribute__((always_inline)) {
        const Tile tl = tiles[min(ti, n_tiles - 1)];
        const NetItem& it = items[tl.item];
        return Place{it.buf[x_slot], it.buf[dz_slot], it.wc, it.hc, tl.ty, tl.tx * NW};
    };
    auto load = [&](const Place& t) __attribute__((always_inline)) {
        const uint32_t plane = (uint32_t)t.hc * (uint32_t)t.wc;
        const auto rx = planes_rsrc(t.x, (uint64_t)CIN * plane * 4);
        const auto rd = planes_rsrc(t.dz, (uint64_t)COUT * plane * 4);
        const int y = t.p - 1 + xr, x = t.q0 - 1 + xcol;
        const bool in = xg < XG && y >= 0 && y < t.hc && x >= 0 && x < t.wc;
        const uint32_t off = in ? 4u * ((uint32_t)xg * plane + (uint32_t)(y * t.wc + x)) : NOWHERE;
#pragma unroll
        for (int i = 0; i < XPER; ++i)  // channels past CIN lie past the buffer
            xv[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, off, 4u * XG * i * plane, 0));
#pragma unroll
        for (int i = 0; i < DPER; ++i) {
            const int e = tid + WG_THREADS * i, o = e / NW, q = t.q0 + e % NW;
            const uint32_t doff = q < t.wc ? 4u * ((uint32_t)o * plane + (uint32_t)(t.p * t.wc + q)) : NOWHERE;
            dv[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rd, doff, 0, 0));
        }
    };
    Place now = place(blockIdx.x), next = place(blockIdx.x + gridDim.x);
    load(now);
    int buf = 0;
    for (int ti = blockIdx.x; ti < n_tiles; ti += gridDim.x, buf ^= 1) {
        float* const xs = sh + buf * S::BUF;
#pragma unroll
        for (int i = 0; i < XPER; ++i)
            if (xg + XG * i < CIN && xg < XG) xs[(xg + XG * i) * CH_S + tid - xg * PATCH] = xv[i];
#pragma unroll
        for (int i = 0; i < DPER; ++i) {
            const int e = tid + WG_THREADS * i;
            xs[CIN * CH_S + e / NW * DZ_S + e % NW] = dv[i];
        }
        const int nk = min(16, (now.wc - now.q0 + 3) >> 2);  // K steps with cells (uniform)
        __syncthreads();  // this tile staged, and the tile before the last one's reads of this buffer done
        now = next;
        if (ti + (int)gridDim.x < n_tiles) load(now);
        next = place(ti + 2 * gridDim.x);
#pragma unroll
        for (int j = 0; j < 16 / S::WK; ++j) {
            if (wk + S::WK * j >= nk) break;  // uniform
            const float a = xs[aoff + 4 * S::WK * j];
#pragma unroll
            for (int i = 0; i < S::NPW; ++i)
                acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, xs[boff[i] + 4 * S::WK * j], acc[i], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < DPER; ++i) accb += xs[CIN * CH_S + tid % COUT * DZ_S + tid / COUT * DPER + i];
    }
    // the WK sums of each output, then the bias sums, in a fixed order
    __syncthreads();
    if (wk > 0) {
        float* const r = sh + ((wk - 1) * S::WM * S::WN + wn * S::WM + wm) * (S::NPW * 256) + lane;
#pragma unroll
        for (int i = 0; i < S::NPW; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) r[(4 * i + v) * 64] = acc[i][v];
    }
    bsh[tid] = accb;
    __syncthreads();
    float* const out = partial + (size_t)blockIdx.x * S::NOUT;
    if (wk == 0) {
#pragma unroll
        for (int i = 0; i < S::NPW; ++i) {
            const int n = wn + S::WN * i, g = n / 9, t = n - 9 * g, c = 16 * g + col;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float sum = acc[i][v];
#pragma unroll
                for (int k = 1; k < S::WK; ++k)
                    sum += sh[((k - 1) * S::WM * S::WN + wn * S::WM + wm) * (S::NPW * 256) + (4 * i + v) * 64 + lane];
                if (n < S::TILES && c < CIN) out[((16 * wm + 4 * kk + v) * CIN + c) * 9 + t] = sum;
            }
        }
    }
    if (tid < COUT) {
        float sum = 0.0f;
        for (int k = tid; k < WG_THREADS; k += COUT) sum += bsh[k];
        out[COUT * CIN * 9 + tid] = sum;
    }
}

// Loss and head: per cell dz = m((1 - y) s - pw y (1 - s)) (un-normalised),
// dZ3[c] = dz hw[c] [a3[c] > 0]; per-workgroup partials of dhw, dhb, the
// loss and the number of masked cells (NHEAD = 16 + 3 values).
constexpr int HEAD_C = 16;
constexpr int NHEAD = HEAD_C + 3;

__device__ __forceinline__ float softplus(float x) { return fmaxf(x, 0.0f) + log1pf(expf(-fabsf(x))); }

__global__ void __launch_bounds__(256) head_loss_kernel(const NetItem* __restrict__ items,
                                                        const Tile* __restrict__ tiles, int n_tiles, int a3_slot,
                                                        int dz_slot, const float* __restrict__ head, float pos_weight,
                                                        double* __restrict__ partial) {
    __shared__ double red[256][NHEAD];
    double mine[NHEAD];
#pragma unroll
    for (int k = 0; k < NHEAD; ++k) mine[k] = 0.0;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int task = blockIdx.x * NWAVES + wave;
    if (task < n_tiles) {
        const Tile tl = tiles[task];
        const NetItem& it = items[tl.item];
        const int q = tl.tx * NW + lane;
        if (q < it.wc) {
            const size_t plane = (size_t)it.hc * it.wc;
            const size_t at = (size_t)tl.ty * it.wc + q;
            const float z = it.logit[at], y = it.label[at], m = it.mask[at];
            const float s = 1.0f / (1.0f + expf(-z));
            const float dz = m * ((1.0f - y) * s - pos_weight * y * (1.0f - s));
            const float* a3 = it.buf[a3_slot];
            float* dz3 = it.buf[dz_slot];
#pragma unroll
            for (int c = 0; c < HEAD_C; ++c) {
                const float a = a3[c * plane + at];
                dz3[c * plane + at] = a > 0.0f ? dz * head[c] : 0.0f;
                mine[c] = (double)dz * (double)a;
            }
            mine[HEAD_C] = dz;
            mine[HEAD_C + 1] = m != 0.0f ? (double)m * ((double)pos_weight * y * softplus(-z) +
                                                         (1.0 - (double)y) * softplus(z))
                                         : 0.0;
            mine[HEAD_C + 2] = m;
        }
    }
#pragma unroll
    for (int k = 0; k < NHEAD; ++k) red[threadIdx.x][k] = mine[k];
    __syncthreads();
    for (int stride = 128; stride > 0; stride >>= 1) {
        if ((int)threadIdx.x < stride)
            for (int k = 0; k < NHEAD; ++k) red[threadIdx.x][k] += red[threadIdx.x + stride][k];
        __syncthreads();
    }
    if (threadIdx.x < NHEAD) partial[(size_t)blockIdx.x * NHEAD + threadIdx.x] = red[0][threadIdx.x];
}

// Head partials -> grad of hw and hb (divided by N), loss, N.  32 threads per
// value, each a run of the workgroups' partials, then the runs in order (one
// thread per value took 348 us for 1492 partials).
constexpr int HR_RUNS = 32;
__global__ void __launch_bounds__(32 * HR_RUNS) head_reduce_kernel(const double* __restrict__ partial, int n_blocks,
                                                                   float* __restrict__ grad_head,
                                                                   double* __restrict__ stats) {
    __shared__ double runs[HR_RUNS][NHEAD];
    __shared__ double sums[NHEAD];
    const int k = threadIdx.x & 31, run = threadIdx.x >> 5, len = (n_blocks + HR_RUNS - 1) / HR_RUNS;
    if (k < NHEAD) {
        double s = 0.0;
        for (int b = run * len; b < min(n_blocks, (run + 1) * len); ++b) s += partial[(size_t)b * NHEAD + k];
        runs[run][k] = s;
    }
    __syncthreads();
    if (threadIdx.x < NHEAD) {
        double s = 0.0;
        for (int r = 0; r < HR_RUNS; ++r) s += runs[r][threadIdx.x];
        sums[threadIdx.x] = s;
    }
    __syncthreads();
    if (threadIdx.x >= NHEAD) return;
    const double n = sums[HEAD_C + 2], s = sums[threadIdx.x];
    const double inv = n > 0.0 ? 1.0 / n : 0.0;
    if (threadIdx.x <= HEAD_C) grad_head[threadIdx.x] = (float)(s * inv);
    if (threadIdx.x == HEAD_C + 1) stats[0] = s * inv;  // mean loss
    if (threadIdx.x == HEAD_C + 2) stats[1] = n;        // masked cells
}

// The three layers' partials (one layer's after the other's) -> gradient,
// divided by N = stats[1].  64 outputs per workgroup, a wave per run of the
// partials, then the runs in order: FP64 throughout.
constexpr int N_W1 = 68 * 32 * 9 + 32, N_W2 = 32 * 32 * 9 + 32, N_W3 = 32 * 16 * 9 + 16;
constexpr int WR_RUNS = 8;
__global__ void __launch_bounds__(64 * WR_RUNS) wgrad_reduce_kernel(const float* __restrict__ partial, int n_blocks,
                                                                    const double* __restrict__ stats,
                                                                    float* __restrict__ grad) {
    __shared__ double runs[WR_RUNS][64];
    const int lane = threadIdx.x & 63, run = threadIdx.x >> 6, k = blockIdx.x * 64 + lane;
    const int layer = k < N_W1 ? 0 : k < N_W1 + N_W2 ? 1 : 2;
    const int first = layer == 0 ? 0 : layer == 1 ? N_W1 : N_W1 + N_W2;
    const int nout = layer == 0 ? N_W1 : layer == 1 ? N_W2 : N_W3;
    const int len = (n_blocks + WR_RUNS - 1) / WR_RUNS;
    double s = 0.0;
    if (k < N_W1 + N_W2 + N_W3) {
        const float* src = partial + (size_t)n_blocks * first + (k - first);
        for (int b = run * len; b < min(n_blocks, (run + 1) * len); ++b) s += (double)src[(size_t)b * nout];
    }
    runs[run][lane] = s;
    __syncthreads();
    if (run > 0 || k >= N_W1 + N_W2 + N_W3) return;
    for (int r = 1; r < WR_RUNS; ++r) s += runs[r][lane];
    const double n = stats[1];
    grad[k] = (float)(n > 0.0 ? s / n : 0.0);
}

// The conv weights in fragment order (element 64 ((k / 4) NT + o / 16) +
// 16 (k % 4) + o % 16 for K value k and output o): forward, k = 9 c + tap, o =
// the output channel; and for data gradients the flipped, transposed form,
// k = 9 (output channel) + 8 - tap, o = the input channel.
__global__ void __launch_bounds__(256) prep_weights_kernel(const float* __restrict__ params, float* __restrict__ prep) {
    int e = blockIdx.x * 256 + threadIdx.x;
    for (int l = 0; l < 3; ++l) {
        const int cin = l == 0 ? 68 : 32, cout = l == 2 ? 16 : 32, n = cin * cout * 9;
        if (e < n) {
            const int o = e / (cin * 9), rem = e - o * cin * 9, c = rem / 9, t = rem - c * 9;
            const float w = params[e];
            auto at = [](int k, int out, int nt) { return 64 * ((k >> 2) * nt + (out >> 4)) + 16 * (k & 3) + (out & 15); };
            prep[at(9 * c + t, o, cout / 16)] = w;
            if (l > 0) prep[n + at(9 * o + 8 - t, c, cin / 16)] = w;
            return;
        }
        e -= n;
        params += n + cout;
        prep += 2 * n;
    }
}

__global__ void __launch_bounds__(256) adam_kernel(float* __restrict__ p, const float* __restrict__ g,
                                                   float* __restrict__ m, float* __restrict__ v, int n, float lr,
                                                   float b1, float b2, float eps, float c1, float c2) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    const float gk = g[k];
    const float mk = b1 * m[k] + (1.0f - b1) * gk;
    const float vk = b2 * v[k] + (1.0f - b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    p[k] -= lr * (mk * c1) / (sqrtf(vk * c2) + eps);
}

__global__ void __launch_bounds__(256) window_labels_kernel(const float* __restrict__ scores, int nx, int ny,
                                                            int wc, int hc, const double* __restrict__ thr,
                                                            float* __restrict__ labels, float* __restrict__ mask) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= wc * hc) return;
    const int cy = e / wc, cx = e - cy * wc;
    const int i = cy - PRUNER_WIN_DI, j = cx - PRUNER_WIN_DJ;
    const bool win = i >= 0 && i < ny && j >= 0 && j < nx;
    mask[e] = win ? 1.0f : 0.0f;
    labels[e] = win && (double)scores[(size_t)i * nx + j] > thr[0] ? 1.0f : 0.0f;
}

// ---- BF16 MFMA inference ------------------------------------------------------
// Implicit GEMM per layer on v_mfma_f32_16x16x32_bf16: M = 16 cells of a row,
// N = 16 output channels, K = (tap, input channel) with the channel vector of
// each neighbour cell contiguous (channels-last maps).  Persistent workgroups:
// each wave loads the packed weight fragments of its output-channel tile into
// registers once, then the workgroup loops over tiles of 2 rows x 64 cells,
// staging the 4 x 66 input cells in LDS per tile (a contiguous run of the
// table per workgroup); the waves sharing an
// output-channel tile split its 8 M-tiles.  FP32 accumulation over K in
// ascending order; bias and ReLU in FP32, outputs rounded to BF16; the last
// layer applies the 1x1 head (cross-lane sum over its 16 channels) and writes
// FP32 logits.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int MR = 2;           // output rows per workgroup
constexpr int MC = 64;          // output cells per row
constexpr int XR = MR + 2, XC = MC + 2;

template <int L>
__global__ void __launch_bounds__(256) conv_mfma_kernel(const LevelItem* __restrict__ items,
                                                        const Tile* __restrict__ tiles, int n_tiles,
                                                        const uint16_t* __restrict__ packed,
                                                        const float* __restrict__ bias,
                                                        const float* __restrict__ head) {
    using D = LayerDims<L>;
    constexpr int CP = D::CP, XS = D::XS, KCH = D::KCH, NT = D::NT;
    constexpr int WPN = 4 / NT;                  // waves per output-channel tile
    constexpr int MT = (MR * MC / 16) / WPN;     // M-tiles per wave
    static_assert(MT * WPN * 16 == MR * MC && (MC / 16) % MT == 0, "a wave's M-tiles lie in one row");
    __shared__ __attribute__((aligned(16))) uint16_t xs[XR * XC * XS];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int nw = wave % NT;                    // this wave's output-channel tile
    const int m0 = (wave / NT) * MT;             // its first M-tile (row-major over MR x MC / 16)
    const int prow = m0 / (MC / 16), cbase = (m0 % (MC / 16)) * 16;

    // this wave's B fragments, fragment order (K chunk t, N tile nw, lane)
    u32x4 bw[KCH];
#pragma unroll
    for (int t = 0; t < KCH; ++t) bw[t] = reinterpret_cast<const u32x4*>(packed)[(t * NT + nw) * 64 + lane];

    // a contiguous run of the (row-major) tile table per workgroup, so the
    // input rows a tile shares with the previous row pair are still in this
    // XCD's L2
    const int run = (n_tiles + gridDim.x - 1) / gridDim.x;
    const int t_end = min(n_tiles, ((int)blockIdx.x + 1) * run);
    // the (MR + 2) x (MC + 2) input cells of a tile, zero outside the map, into
    // registers; the next tile's loads are issued before this tile's MFMAs
    // (software pipeline: the loads are in flight while the matrix cores run)
    constexpr int PARTS = CP / 8;
    constexpr int NXQ = (XR * XC * PARTS + 255) / 256;
    u32x4 xv[NXQ];
    auto load_tile = [&](int ti) __attribute__((always_inline)) {
        const Tile tl = tiles[ti];
        const LevelItem& it = items[tl.item];
        const int wc = it.wc, hc = it.hc;
        const int p0 = tl.ty * MR, q0 = tl.tx * MC;
        const uint16_t* in = L == 1 ? it.cmap16 : (L == 2 ? it.act1 : it.act2);
#pragma unroll
        for (int k = 0; k < NXQ; ++k) {
            const int e = tid + 256 * k;
            const int cell = e / PARTS, part = e - cell * PARTS;
            const int r = cell / XC, col = cell - r * XC;
            const int y = p0 - 1 + r, x = q0 - 1 + col;
            xv[k] = u32x4{0u, 0u, 0u, 0u};
            if (e < XR * XC * PARTS && y >= 0 && y < hc && x >= 0 && x < wc)
                xv[k] = *reinterpret_cast<const u32x4*>(in + ((size_t)y * wc + x) * CP + 8 * part);
        }
    };
    if ((int)blockIdx.x * run < t_end) load_tile(blockIdx.x * run);
    for (int ti = blockIdx.x * run; ti < t_end; ++ti) {
        const Tile tl = tiles[ti];
        const LevelItem& it = items[tl.item];
        const int wc = it.wc, hc = it.hc;
        const int p0 = tl.ty * MR, q0 = tl.tx * MC;
        __syncthreads();  // the previous tile's reads of xs are done
#pragma unroll
        for (int k = 0; k < NXQ; ++k) {
            const int e = tid + 256 * k;
            if (e < XR * XC * PARTS) {
                const int cell = e / PARTS, part = e - cell * PARTS;
                *reinterpret_cast<u32x4*>(xs + cell * XS + 8 * part) = xv[k];
            }
        }
        __syncthreads();
        if (ti + 1 < t_end) load_tile(ti + 1);

        f32x4 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int t = 0; t < KCH; ++t) {
            const int k0 = 32 * t + 8 * (lane >> 4);
            const int tap = k0 / CP, c0 = k0 - tap * CP;
            const int u = tap / 3, v = tap - 3 * (tap / 3);
            const bf16x8 b = __builtin_bit_cast(bf16x8, bw[t]);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int col = cbase + 16 * mt + (lane & 15);
                u32x4 av = {0u, 0u, 0u, 0u};
                if (tap < 9) av = *reinterpret_cast<const u32x4*>(xs + ((prow + u) * XC + col + v) * XS + c0);
                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av), b, acc[mt], 0, 0, 0);
            }
        }

        // lane holds D[cell 4 * (lane / 16) + r][channel lane % 16] of each tile
        const int p = p0 + prow;
        const int och = 16 * nw + (lane & 15);
        if (L < 3) {
            uint16_t* out = L == 1 ? it.act1 : it.act2;
            const float bo = bias[och];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int q = q0 + cbase + 16 * mt + 4 * (lane >> 4) + r;
                    if (p < hc && q < wc) out[((size_t)p * wc + q) * 32 + och] = f32_to_bf16(fmaxf(acc[mt][r] + bo, 0.0f));
                }
        } else {
            const float bo = bias[och], hw = head[och], hb = head[16];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float z = hw * fmaxf(acc[mt][r] + bo, 0.0f);
                    z += __shfl_xor(z, 8, 16);
                    z += __shfl_xor(z, 4, 16);
                    z += __shfl_xor(z, 2, 16);
                    z += __shfl_xor(z, 1, 16);
                    const int q = q0 + cbase + 16 * mt + 4 * (lane >> 4) + r;
                    if ((lane & 15) == 0 && p < hc && q < wc) it.logit[(size_t)p * wc + q] = z + hb;
                }
        }
    }
}

}  // namespace

int64_t pruner_prep_floats() {
    int64_t n = 0;
    for (int l = 0; l < 3; ++l) n += 2LL * PRUNER_CH[l] * PRUNER_CH[l + 1] * 9;
    return n;
}

hipError_t launch_pruner_prep(const float* params, float* prep, hipStream_t s) {
    const int n = 9 * (68 * 32 + 32 * 32 + 32 * 16);
    prep_weights_kernel<<<ceil_div(n, 256), 256, 0, s>>>(params, prep);
    return hipGetLastError();
}

namespace {

// A convolution over every tile: workgroups of 8 waves that keep the layer's
// weights in LDS, two per CU (one for the 78 KB of the first layer).
template <int CIN, int COUT, bool HEAD>
void launch_conv(const NetItem* items, const Tile* tiles, int n_tiles, int in_slot, int out_slot, int mask_slot,
                 const float* frags, const float* bias, int relu, const float* head, hipStream_t s) {
    const int grid = std::min(ceil_div(n_tiles, CV_WAVES), CIN > 32 ? 256 : 512);
    conv3x3_kernel<CIN, COUT, HEAD><<<grid, 64 * CV_WAVES, 0, s>>>(items, tiles, n_tiles, in_slot, out_slot, mask_slot,
                                                                   frags, bias, relu, head);
}

}  // namespace

hipError_t launch_pruner_forward(const NetItem* items, const Tile* tiles, int n_tiles, const float* params,
                                 const float* prep, bool keep_a3, hipStream_t s) {
    if (n_tiles <= 0) return hipSuccess;
    const float* b1 = params + 68 * 32 * 9;
    const float* b2 = b1 + 32 + 32 * 32 * 9;
    const float* b3 = b2 + 32 + 32 * 16 * 9;
    const float* head = b3 + 16;
    const float* w1 = prep;
    const float* w2 = w1 + 2 * 68 * 32 * 9;
    const float* w3 = w2 + 2 * 32 * 32 * 9;
    launch_conv<68, 32, false>(items, tiles, n_tiles, NET_X, NET_A1, -1, w1, b1, 1, nullptr, s);
    launch_conv<32, 32, false>(items, tiles, n_tiles, NET_A1, NET_A2, -1, w2, b2, 1, nullptr, s);
    launch_conv<32, 16, true>(items, tiles, n_tiles, NET_A2, keep_a3 ? NET_A3 : -1, -1, w3, b3, 1, head, s);
    return hipGetLastError();
}

// Workgroups of the weight gradients: one per CU, and about two tiles each when
// there are few (their partials then fill no more than one layer's did with a
// tile each).
int pruner_wgrad_blocks(int n_tiles) { return std::max(1, std::min(256, n_tiles * 7 / 12)); }

int64_t pruner_partial_floats(int n_tiles) {
    // the three layers' partials (+ head, as doubles)
    const int nb = pruner_wgrad_blocks(n_tiles);
    return (int64_t)nb * (N_W1 + N_W2 + N_W3) + 2LL * ceil_div(n_tiles, NWAVES) * NHEAD + 4;
}

hipError_t launch_pruner_backward(const NetItem* items, const Tile* tiles, int n_tiles, const float* params,
                                  const float* prep, float pos_weight, float* grad, double* stats, float* partial,
                                  hipStream_t s) {
    if (n_tiles <= 0) return hipSuccess;
    const int grid = ceil_div(n_tiles, NWAVES);
    const int nb = pruner_wgrad_blocks(n_tiles);
    const int n1 = 68 * 32 * 9, n2 = 32 * 32 * 9, n3 = 32 * 16 * 9;
    const float* head = params + n1 + 32 + n2 + 32 + n3 + 16;
    const float* w2b = prep + 2 * n1 + n2;
    const float* w3b = prep + 2 * n1 + 2 * n2 + n3;
    float* p1 = partial;
    float* p2 = p1 + (int64_t)nb * N_W1;
    float* p3 = p2 + (int64_t)nb * N_W2;
    double* hpart = reinterpret_cast<double*>(p3 + (int64_t)nb * N_W3);
    // head and loss, then the normaliser N
    head_loss_kernel<<<grid, 256, 0, s>>>(items, tiles, n_tiles, NET_A3, NET_GA, head, pos_weight, hpart);
    head_reduce_kernel<<<1, 32 * HR_RUNS, 0, s>>>(hpart, grid, grad + N_W1 + N_W2 + N_W3, stats);
    // layer 3: dW3 from dZ3 (GA) and a2; dZ2 = conv(dZ3, W3 flipped) [a2 > 0] -> GB
    wgrad_kernel<32, 16><<<nb, WG_THREADS, 0, s>>>(items, tiles, n_tiles, NET_A2, NET_GA, p3);
    launch_conv<16, 32, false>(items, tiles, n_tiles, NET_GA, NET_GB, NET_A2, w3b, nullptr, 0, nullptr, s);
    // layer 2: dW2 from dZ2 (GB) and a1; dZ1 = conv(dZ2, W2 flipped) [a1 > 0] -> GA
    wgrad_kernel<32, 32><<<nb, WG_THREADS, 0, s>>>(items, tiles, n_tiles, NET_A1, NET_GB, p2);
    launch_conv<32, 32, false>(items, tiles, n_tiles, NET_GB, NET_GA, NET_A1, w2b, nullptr, 0, nullptr, s);
    // layer 1: dW1 from dZ1 (GA) and the cell map
    wgrad_kernel<68, 32><<<nb, WG_THREADS, 0, s>>>(items, tiles, n_tiles, NET_X, NET_GA, p1);
    wgrad_reduce_kernel<<<ceil_div(N_W1 + N_W2 + N_W3, 64), 64 * WR_RUNS, 0, s>>>(partial, nb, stats, grad);
    return hipGetLastError();
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, int n, int step, float lr, float b1, float b2,
                       float eps, hipStream_t s) {
    const float c1 = (float)(1.0 / (1.0 - std::pow((double)b1, step)));
    const float c2 = (float)(1.0 / (1.0 - std::pow((double)b2, step)));
    adam_kernel<<<ceil_div(n, 256), 256, 0, s>>>(p, g, m, v, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_window_labels(const float* scores, int nx, int ny, int wc, int hc, const double* thr,
                                float* labels, float* mask, hipStream_t s) {
    window_labels_kernel<<<ceil_div(wc * hc, 256), 256, 0, s>>>(scores, nx, ny, wc, hc, thr, labels, mask);
    return hipGetLastError();
}

int pruner_mfma_tiles_y(int hc) { return ceil_div(hc, MR); }

hipError_t launch_pruner_mfma(const LevelItem* items, const Tile* tiles, int n_tiles, const float* params,
                              const uint16_t* packed, hipStream_t s) {
    if (n_tiles <= 0) return hipSuccess;
    const float* b1 = params + LayerDims<1>::PARAMS;
    const float* b2 = b1 + 32 + LayerDims<2>::PARAMS;
    const float* b3 = b2 + 32 + LayerDims<3>::PARAMS;
    const float* head = b3 + 16;
    // persistent workgroups: a few per CU, each looping over the tiles
    const int grid = std::min(n_tiles, 4 * 256);
    conv_mfma_kernel<1><<<grid, 256, 0, s>>>(items, tiles, n_tiles, packed, b1, nullptr);
    conv_mfma_kernel<2><<<grid, 256, 0, s>>>(items, tiles, n_tiles, packed + LayerDims<1>::PACKED, b2, nullptr);
    conv_mfma_kernel<3><<<grid, 256, 0, s>>>(items, tiles, n_tiles,
                                             packed + LayerDims<1>::PACKED + LayerDims<2>::PACKED, b3, head);
    return hipGetLastError();
}

namespace {

// Order-preserving map of a float to an unsigned key (larger float, larger key).
__device__ __forceinline__ uint32_t fkey(float z) {
    const uint32_t u = __float_as_uint(z + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// One workgroup of 16 waves per frame: radix selection (8 bits per pass, most
// significant first) of the K-th largest logit over the frame's windows, every
// level.  The logits are read from memory once, their keys kept in LDS (frames
// of more than TOPK_KEYS windows read them again in each pass); one wave finds
// a pass's bin.  (4 waves that read the logits in every pass, with one thread
// walking the bins, took 116 us for 16 frames of 1242x375; this takes 23.)
constexpr int TOPK_THREADS = 1024;
constexpr int TOPK_BATCH = 4;
constexpr int TOPK_KEYS = 36 * 1024;

__global__ void __launch_bounds__(TOPK_THREADS) topk_kernel(const LevelItem* __restrict__ items,
                                                            const int32_t* __restrict__ first_item,
                                                            const NmsGeom* __restrict__ geoms, int keep_k,
                                                            float* __restrict__ kth) {
    __shared__ uint32_t hist[256];
    __shared__ uint32_t found[2];
    __shared__ uint32_t keys[TOPK_KEYS];
    const int f = blockIdx.x, tid = threadIdx.x;
    const int i0 = first_item[f], nl = geoms[f].n_levels, total = geoms[f].cand_cap;
    if (keep_k >= total) {  // every window is kept
        if (tid == 0) kth[f] = -INFINITY;
        return;
    }
    const bool held = total <= TOPK_KEYS;
    // f(key, place) of every window, four loads of a thread in flight together
    auto each = [&](auto&& visit) __attribute__((always_inline)) {
        int base = 0;
        for (int l = 0; l < nl; ++l) {
            const LevelItem& it = items[i0 + l];
            const int n = it.nx * it.ny, nx = it.nx, wc = it.wc;
            const float* const z = it.logit + PRUNER_WIN_DI * wc + PRUNER_WIN_DJ;
            for (int q0 = tid; q0 < n; q0 += TOPK_THREADS * TOPK_BATCH) {
                uint32_t k[TOPK_BATCH];
#pragma unroll
                for (int u = 0; u < TOPK_BATCH; ++u) {
                    const int q = min(q0 + TOPK_THREADS * u, n - 1), wi = q / nx;
                    k[u] = fkey(z[(size_t)wi * wc + (q - wi * nx)]);
                }
#pragma unroll
                for (int u = 0; u < TOPK_BATCH; ++u)
                    if (q0 + TOPK_THREADS * u < n) visit(k[u], base + q0 + TOPK_THREADS * u);
            }
            base += n;
        }
    };
    uint32_t mask = 0u, prefix = 0u, rank = (uint32_t)keep_k;
    for (int shift = 24; shift >= 0; shift -= 8) {
        if (tid < 256) hist[tid] = 0u;
        __syncthreads();
        auto count = [&](uint32_t k) {
            if ((k & mask) == prefix) atomicAdd(&hist[(k >> shift) & 255u], 1u);
        };
        if (held && shift < 24) {
            for (int q = tid; q < total; q += TOPK_THREADS) count(keys[q]);
        } else {
            each([&](uint32_t k, int q) {
                if (held) keys[q] = k;
                count(k);
            });
        }
        __syncthreads();
        if (tid < 64) select_bin<false>(hist, rank, found);
        __syncthreads();
        prefix |= found[0] << shift;
        rank = found[1];
        mask |= 255u << shift;
        __syncthreads();  // found is rewritten by the next pass
    }
    if (tid == 0) kth[f] = __uint_as_float((prefix & 0x80000000u) ? (prefix & 0x7fffffffu) : ~prefix);
}

// One wave per score tile: does any of its windows have logit >= kth?
__global__ void __launch_bounds__(256) tile_filter_kernel(const LevelItem* __restrict__ items,
                                                          const Tile* __restrict__ tiles, int n_tiles, int rows,
                                                          int cols, const float* __restrict__ kth,
                                                          Tile* __restrict__ kept, int32_t* __restrict__ kept_count) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int t = blockIdx.x * 4 + wave;
    if (t >= n_tiles) return;
    const Tile tl = tiles[t];
    const LevelItem& it = items[tl.item];
    const float thr = kth[it.frame];
    // a tile of width w < cols (FP32 lane groups) covers cols / w row chunks
    const int w = cols == SC_W ? tile_width(tl) : cols;
    const int r0 = tl.ty * rows, nr = rows * (cols / w);
    bool any = false;
    for (int c = lane; c < w; c += 64) {
        const int j = tl.tx * cols + c;
        if (j >= it.nx) break;
        for (int r = 0; r < nr; ++r) {
            const int i = r0 + r;
            if (i >= it.ny) break;
            any = any || it.logit[(size_t)(i + PRUNER_WIN_DI) * it.wc + j + PRUNER_WIN_DJ] >= thr;
        }
    }
    if (__any(any) && lane == 0) kept[atomicAdd(kept_count, 1)] = tl;
}

}  // namespace

hipError_t launch_topk(const LevelItem* items, const int32_t* first_item, const NmsGeom* geoms, int n_frames,
                       int keep_k, float* kth, hipStream_t s) {
    if (n_frames <= 0) return hipSuccess;
    topk_kernel<<<n_frames, TOPK_THREADS, 0, s>>>(items, first_item, geoms, keep_k, kth);
    return hipGetLastError();
}

hipError_t launch_tile_filter(const LevelItem* items, const Tile* tiles, int n_tiles, int rows, int cols,
                              const float* kth, Tile* kept, int32_t* kept_count, hipStream_t s) {
    if (n_tiles <= 0) return hipSuccess;
    tile_filter_kernel<<<ceil_div(n_tiles, 4), 256, 0, s>>>(items, tiles, n_tiles, rows, cols, kth, kept, kept_count);
    return hipGetLastError();
}

}  // namespace pd
