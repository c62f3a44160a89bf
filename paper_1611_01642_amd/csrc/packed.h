// Layouts that a call's weights are packed into before they are used, and
// their elements: the scoring kernels' B operands (FP32, BF16 row GEMM, BF16
// window-row GEMM), the pruner's BF16 fragments and the FP64 rescore's gradient
// table.  prep.hip fills whichever a call needs in one launch.
#pragma once

#include "pd_internal.h"

namespace pd {

// ---- FP32 scoring --------------------------------------------------------------
constexpr int S32_HOG_T = PD_HOG_BLOCK / 4;             // 9 chunks of 4 channels
constexpr int S32_LBP_T = (PD_LBP_BINS + 3) / 4;         // 15: channel 59 has zero weight
constexpr int S32_HOG_K = PD_WIN_BLOCKS_Y + 1;           // 16 feature rows per pair
constexpr int S32_LBP_K = PD_WIN_CELLS_Y + 1;            // 17
// Weight row a of the model (HOG 0 .. 14, LBP 0 .. 15) holds [t][b 8][c 4]
// floats, plus 2: the s = 1 lanes then read 2 banks away from the s = 0 ones.
// One zero row follows: the B fragments of rows a' - s outside the model
// read it.
constexpr int S32_HOG_RS = S32_HOG_T * 32 + 2;
constexpr int S32_LBP_RS = S32_LBP_T * 32 + 2;
constexpr int S32_HOG_N = PD_WIN_BLOCKS_Y * S32_HOG_RS;
constexpr int S32_LBP_N = PD_WIN_CELLS_Y * S32_LBP_RS;
constexpr int S32_ZERO = S32_HOG_N + S32_LBP_N;  // the zero row (S32_LBP_RS floats)
constexpr int S32_MODEL = (S32_ZERO + S32_LBP_RS + 3) / 4 * 4;  // floats per packed model (50 KB)

// FP32 scoring (score32.hip): model m's floats at m * S32_MODEL, HOG rows
// a = 0 .. 14, then LBP rows a = 0 .. 15, then the zero row; element (a, t, b,
// k) = W[a][b][4 t + k] (zero for HOG b = 7 and LBP channel 59).
__device__ inline float packed_s32(const float* __restrict__ w, int e) {
    const int m = e / S32_MODEL, q = e - m * S32_MODEL;
    const float* wm = w + (size_t)m * PD_FEATURE_DIM;
    float v = 0.0f;
    if (q < S32_HOG_N) {
        const int a = q / S32_HOG_RS, x = q - a * S32_HOG_RS;
        const int t = x >> 5, b = (x >> 2) & 7, c = 4 * t + (x & 3);
        if (x < S32_HOG_T * 32 && b < PD_WIN_BLOCKS_X) v = wm[(a * PD_WIN_BLOCKS_X + b) * PD_HOG_BLOCK + c];
    } else if (q < S32_ZERO) {
        const int q2 = q - S32_HOG_N;
        const int a = q2 / S32_LBP_RS, x = q2 - a * S32_LBP_RS;
        const int t = x >> 5, b = (x >> 2) & 7, c = 4 * t + (x & 3);
        if (x < S32_LBP_T * 32 && c < PD_LBP_BINS) v = wm[PD_HOG_DIM + (a * PD_WIN_CELLS_X + b) * PD_LBP_BINS + c];
    }
    return v;
}

// ---- BF16 scoring, one model (row GEMM) -----------------------------------------
constexpr int RG_HOG_T = 8;    // K chunks of 32 per HOG row: 7 * 36 = 252 -> 256
constexpr int RG_LBP_T = 15;   // 8 * 60 = 480 (59 bins padded to 60)
constexpr int RG_HOG_C = PD_HOG_BLOCK;
constexpr int RG_LBP_C = 60;
// packed B fragments: [HOG hi: t 8][LBP hi: t 15][LBP lo: t 15], each
// [lane 64][8] bf16 (lane: column a = lane % 16, K group lane / 16)
constexpr int RG_FRAG = 64 * 8;
constexpr int RG_PACKED = (RG_HOG_T + 2 * RG_LBP_T) * RG_FRAG;
__device__ inline uint16_t packed_rowgemm(const float* __restrict__ w, int e) {
    const int f = e / RG_FRAG, r = e - f * RG_FRAG;
    const int lane = r >> 3, kk = r & 7;
    const int a = lane & 15;
    float v = 0.0f;
    bool lo = false;
    if (f < RG_HOG_T) {
        const int k = 32 * f + 8 * (lane >> 4) + kk;
        const int b = k / RG_HOG_C, c = k % RG_HOG_C;
        if (a < PD_WIN_BLOCKS_Y && b < PD_WIN_BLOCKS_X) v = w[(a * PD_WIN_BLOCKS_X + b) * PD_HOG_BLOCK + c];
    } else {
        const int t = (f - RG_HOG_T) % RG_LBP_T;
        lo = f >= RG_HOG_T + RG_LBP_T;
        const int k = 32 * t + 8 * (lane >> 4) + kk;
        const int b = k / RG_LBP_C, c = k % RG_LBP_C;
        if (b < PD_WIN_CELLS_X && c < PD_LBP_BINS) v = w[PD_HOG_DIM + (a * PD_WIN_CELLS_X + b) * PD_LBP_BINS + c];
    }
    const uint16_t hi = f32_to_bf16(v);
    return lo ? f32_to_bf16(v - __uint_as_float((uint32_t)hi << 16)) : hi;
}

// ---- BF16 scoring, 2 to 8 models -------------------------------------------------
constexpr int MF_HOG_C = PD_HOG_BLOCK;            // 36 channels per block
constexpr int MF_LBP_C = 60;                      // 59 bins + 1 zero
constexpr int MF_HOG_T = 8;                       // K chunks of 32 per offset: 7*36 = 252 -> 256
constexpr int MF_HOG_P = PD_WIN_BLOCKS_Y + 1;     // HOG weight slices: offset pairs (a, a + 1), a = -1 .. 14
constexpr int MF_LBP_T = 15;                      // 8*60 = 480
// HOG: [p 16][t 8][n 16][32]; LBP: [a 16][t 15][n 16][32] bf16; K index
// k = 32 t + kk maps to (b, c) = (k / C, k % C) of the offset row.  LBP:
// column n < 8 is the hi part of model n, n >= 8 the lo part of model n - 8.
// HOG features are BF16, and the HOG weights carry their BF16 part only, so
// a HOG slice holds two offsets: p = a + 1 for the pair (a, a + 1), column
// n < 8 model n at offset a, n >= 8 model n - 8 at offset a + 1 (zero outside
// 0 .. 14): one MFMA then serves two window rows.
constexpr int MF_HOG_ELEMS = MF_HOG_P * MF_HOG_T * 16 * 32;
constexpr int MF_PACKED = MF_HOG_ELEMS + PD_WIN_CELLS_Y * MF_LBP_T * 16 * 32;
__device__ inline uint16_t packed_mfma(const float* __restrict__ w, int n_models, int e) {
    const bool is_hog = e < MF_HOG_ELEMS;
    const int q = is_hog ? e : e - MF_HOG_ELEMS;
    const int T = is_hog ? MF_HOG_T : MF_LBP_T;
    const int kk = q & 31;
    const int n = (q >> 5) & 15;
    const int t = (q >> 9) % T;
    const int a = (q >> 9) / T;
    const int k = 32 * t + kk;
    const int m = n & 7;
    float v = 0.0f;
    if (m < n_models) {
        if (is_hog) {
            const int b = k / MF_HOG_C, c = k % MF_HOG_C;
            const int off = n < 8 ? a - 1 : a;  // a is the slice index p here
            if (b < PD_WIN_BLOCKS_X && off >= 0 && off < PD_WIN_BLOCKS_Y)
                v = w[(size_t)m * PD_FEATURE_DIM + (off * PD_WIN_BLOCKS_X + b) * PD_HOG_BLOCK + c];
        } else {
            const int b = k / MF_LBP_C, c = k % MF_LBP_C;
            if (b < PD_WIN_CELLS_X && c < PD_LBP_BINS)
                v = w[(size_t)m * PD_FEATURE_DIM + PD_HOG_DIM + (a * PD_WIN_CELLS_X + b) * PD_LBP_BINS + c];
        }
    }
    const uint16_t hi = f32_to_bf16(v);
    // LBP counts are exact, so LBP weights carry hi + lo
    return (is_hog || n < 8) ? hi : f32_to_bf16(v - __uint_as_float((uint32_t)hi << 16));
}

// ---- pruner inference ------------------------------------------------------------
template <int L>
struct Layer;
template <>
struct Layer<1> {
    static constexpr int CIN = 68, CP = PR_CP1, XS = PR_CP1, COUT = 32;
};
template <>
struct Layer<2> {
    static constexpr int CIN = 32, CP = 32, XS = 40, COUT = 32;
};
template <>
struct Layer<3> {
    static constexpr int CIN = 32, CP = 32, XS = 40, COUT = 16;
};
template <int L>
struct LayerDims : Layer<L> {
    static constexpr int KCH = (9 * Layer<L>::CP + 31) / 32;  // K chunks of 32
    static constexpr int NT = Layer<L>::COUT / 16;            // N tiles
    static constexpr int PACKED = KCH * NT * 64 * 8;          // bf16 values
    static constexpr int PARAMS = Layer<L>::COUT * Layer<L>::CIN * 9;
};
// Element e of layer L's B fragments; w: the layer's weights.
template <int L>
__device__ inline uint16_t packed_layer(const float* __restrict__ w, int e) {
    using D = LayerDims<L>;
    const int t = e / (D::NT * 512), n = (e / 512) % D::NT, l = (e / 8) % 64, j = e % 8;
    const int k = 32 * t + 8 * (l >> 4) + j, och = 16 * n + (l & 15);
    const int tap = k / D::CP, c = k - tap * D::CP;
    const float v = (tap < 9 && c < D::CIN) ? w[((size_t)och * D::CIN + c) * 9 + tap] : 0.0f;
    return f32_to_bf16(v);
}

// ---- FP64 rescore ------------------------------------------------------------------
// The gradient table: for dy in 0..255 and dx in -255..255, the
// orientation's bin coordinate t = angle / 20 - 0.5 in [-0.5, 8.5) (angle in
// degrees, folded into [0, 180): Algorithm 4 with the device's double atan2)
// and the magnitude sqrt(dx^2 + dy^2), both FP64.  A gradient with dy < 0
// looks up (-dx, -dy): the same magnitude and, mathematically, the same
// folded angle (its FP64 value may differ in the last bits).
__device__ inline double2 packed_orient(int e) {
    const int dy = e / ORIENT_W, dx = e - dy * ORIENT_W - 255;
    const double mag = sqrt((double)(dx * dx + dy * dy));
    double ang = atan2((double)dy, (double)dx) * 57.295779513082320876798154814105;
    if (ang < 0.0) ang += 180.0;
    if (ang >= 180.0) ang -= 180.0;
    return make_double2(ang / 20.0 - 0.5, mag);
}

}  // namespace pd
