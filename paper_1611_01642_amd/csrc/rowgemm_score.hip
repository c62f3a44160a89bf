// Window scoring of one linear SVM on BF16 MFMA (Section 4.4, Algorithm 6),
// with the model's row offsets as the GEMM columns.
//
// A window (i, j) scores s = sum_a P[i + a][j][a] with
//   P[y][j][a] = sum_{b, c} F[y][j + b][c] * W[a][b][c],
// HOG rows a = 0..14 (b < 7, c < 36) and LBP rows a = 0..15 (b < 8, c < 59).
// For one feature row y, P is a dense GEMM: rows = 16 windows j, K = the
// window's (b, c) run of that row (contiguous when the row is staged
// channel-innermost), columns = the 16 offsets a.  So every staged feature
// row is multiplied once with the whole model (the window-row formulation
// re-reads each feature row for every window row it covers), and all 16
// MFMA columns are useful.  The diagonal sums run in a 16-slot ring of
// window-row accumulators in LDS: at row y, column a belongs to window row
// y - a; window row y - 15 is complete after row y.
//
// Numerics: HOG features are BF16 and the HOG weights their BF16 part; LBP
// counts are exact and the LBP weights are hi + lo BF16 halves (two MFMAs per A
// fragment).  FP32 accumulation; fixed summation order.
//
// Tile: a workgroup of 4 waves owns 64 window columns of one level (16 per
// wave) and streams down all feature rows; a row's loads are issued two rows
// ahead, so they are in flight during two rows of MFMAs.
#include <type_traits>

#include "packed.h"
#include "pd_internal.h"

namespace pd {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int RG_COLS = 64;
constexpr int RG_HOG_SR = RG_COLS + PD_WIN_BLOCKS_X - 1;  // 70 staged blocks
constexpr int RG_LBP_SR = RG_COLS + PD_WIN_CELLS_X - 1;   // 71 staged cells
constexpr int RG_HOG_ROW = (RG_HOG_SR * RG_HOG_C + 8 + 7) / 8 * 8;
constexpr int RG_LBP_ROW = (RG_LBP_SR * RG_LBP_C + 8 + 7) / 8 * 8;

struct RowShared {
    __bf16 hog[2][RG_HOG_ROW];
    __bf16 lbp[2][RG_LBP_ROW];
    __bf16 blbp[RG_LBP_T * RG_FRAG];  // the LBP weights' lo fragments
    float ring[4][16][16];  // per wave: window-row slot x window column
};

// Staging takes channels in pairs: a thread loads both planes' values and writes
// them as one word, half as many LDS writes as channel by channel (those were a
// quarter of the kernel's LDS time: 224 -> 215 us for 64 frames of 1242x375).
template <bool HOG>
struct RowRegs {
    static constexpr int SR = HOG ? RG_HOG_SR : RG_LBP_SR;
    static constexpr int NC = HOG ? PD_HOG_BLOCK : PD_LBP_BINS;
    // per plane row, HOG: SR BF16 values; LBP: the SR count bytes as 4-byte
    // words (columns 4 d .. 4 d + 3)
    static constexpr int UNITS = HOG ? SR : (SR + 3) / 4;
    // elements: HOG, a pair's columns; LBP, blocks of 8 pairs x UNITS words (32
    // pair slots, those past the 30th empty), the pair fastest within a block
    static constexpr int N = HOG ? (UNITS * NC / 2 + 255) / 256 : (UNITS * 32 + 255) / 256;
    // HOG: BF16 bits; LBP: four raw counts (converted when stored)
    std::conditional_t<HOG, uint16_t, uint32_t> v[N][2];
};

// The per-thread offsets are taken once per tile: goff[q], the byte offset of
// the element's first plane without the row (raw buffer loads add the row's byte
// offset, and the second plane's, as a scalar), and soff[q], its byte offset in
// the staged row (LBP: that of the word's first column).  HOG elements past the
// last are clamped to it (same value, same place).  An LBP word is read from inside its
// plane row: where columns 4 d .. 4 d + 3 reach past the row's end, from the
// row's last four bytes, and shifted down by the difference (kept in the top
// byte of soff), so that its columns inside the row get their counts; the
// rest (past the level, feeding no stored window) get finite values.  The last
// LBP pair is channel 58 and an empty slot: channels 57 and 58 are loaded and
// change places (bit 26), the empty slot's weight being zero.
template <bool HOG>
struct RowOffsets {
    uint32_t goff[RowRegs<HOG>::N], soff[RowRegs<HOG>::N];
};

template <bool HOG>
__device__ __forceinline__ void row_offsets(RowOffsets<HOG>& o, int j0, int hcols, int hrows) {
    constexpr int U = RowRegs<HOG>::UNITS, NC = RowRegs<HOG>::NC;
    constexpr int C = HOG ? RG_HOG_C : RG_LBP_C;
    static_assert(RG_HOG_C % 2 == 0 && RG_LBP_C % 2 == 0 && PD_HOG_BLOCK % 2 == 0, "pairs on word boundaries");
    const uint32_t plane = (uint32_t)hrows * (uint32_t)hcols;
#pragma unroll
    for (int q = 0; q < RowRegs<HOG>::N; ++q) {
        if constexpr (HOG) {
            const int e = min((int)threadIdx.x + 256 * q, U * NC / 2 - 1);
            const int c = 2 * (e / U), col = e - (e / U) * U;
            o.goff[q] = ((uint32_t)c * plane + (uint32_t)min(j0 + col, hcols - 1)) * 2u;
            o.soff[q] = (uint32_t)(col * C + c) * 2u;
        } else {
            // lanes by 8 pairs x 8 words: a wave's staging writes fall in 64
            // banks (words 4 columns apart are 120 dwords apart, pairs one), its
            // loads in 8 plane rows of 32 contiguous bytes.  Slots past the last
            // pair or element load channel 57's word and store nothing (bit 31
            // of soff).
            const int g = (int)threadIdx.x + 256 * q;
            const int cl = g & 7, rest = g >> 3;
            const int uu = rest % U, cb = rest / U;
            const int c = 2 * (8 * cb + cl);
            const bool valid = c < NC && cb < 4;
            const int cs = min(c, NC - 2), col4 = 4 * uu;
            // hcols >= 8 (a level holds at least one window)
            const int start = min(j0 + col4, hcols - 4);
            o.goff[q] = (uint32_t)cs * plane + (uint32_t)start;
            o.soff[q] = (uint32_t)(col4 * C + min(c, NC - 1)) * 2u | (uint32_t)min(j0 + col4 - start, 3) << 24 |
                        (c == NC - 1 ? 1u << 26 : 0u) | (valid ? 0u : 0x80000000u);
        }
    }
}

template <bool HOG>
__device__ __forceinline__ void load_row_fast(RowRegs<HOG>& r, const RowOffsets<HOG>& o, __amdgpu_buffer_rsrc_t rsrc,
                                              int y, int hcols, int hrows) {
    const uint32_t roff = (uint32_t)min(y, hrows - 1) * (uint32_t)hcols * (HOG ? 2u : 1u);
    const uint32_t plane = (uint32_t)hrows * (uint32_t)hcols * (HOG ? 2u : 1u);
#pragma unroll
    for (int q = 0; q < RowRegs<HOG>::N; ++q)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // raw values: LBP counts are converted when stored, so that no
            // instruction waits on these loads before the MFMAs they overlap
            if (HOG) r.v[q][h] = __builtin_amdgcn_raw_buffer_load_b16(rsrc, o.goff[q], roff + h * plane, 0);
            else r.v[q][h] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, o.goff[q], roff + h * plane, 0);
        }
}

template <bool HOG>
__device__ __forceinline__ void store_row_fast(const RowRegs<HOG>& r, const RowOffsets<HOG>& o, __bf16* dst) {
    uint8_t* d = reinterpret_cast<uint8_t*>(dst);
#pragma unroll
    for (int q = 0; q < RowRegs<HOG>::N; ++q) {
        if constexpr (HOG) {
            *reinterpret_cast<uint32_t*>(d + o.soff[q]) = (uint32_t)r.v[q][0] | (uint32_t)r.v[q][1] << 16;
        } else {
            // LBP counts <= 64 are exact in BF16: the top half of their FP32
            // value; byte k of the word is column 4 d + k (its channels' slots
            // RG_LBP_C values further on), the last word's column 71 past the
            // staged row is skipped
            if (o.soff[q] & 0x80000000u) continue;
            const uint32_t so = o.soff[q] & 0xffffffu, shift = 8u * ((o.soff[q] >> 24) & 3u);
            const uint32_t w0 = r.v[q][0] >> shift, w1 = r.v[q][1] >> shift;
            const uint32_t halves = o.soff[q] & 1u << 26 ? 0x03020706u : 0x07060302u;
            const uint32_t col0 = so / (2u * RG_LBP_C);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t b0 = __float_as_uint((float)(w0 >> (8 * k) & 255u));
                const uint32_t b1 = __float_as_uint((float)(w1 >> (8 * k) & 255u));
                if (k < 3 || col0 + 3 < (uint32_t)RG_LBP_SR)
                    *reinterpret_cast<uint32_t*>(d + so + k * 2 * RG_LBP_C) = __builtin_amdgcn_perm(b1, b0, halves);
            }
        }
    }
}

__device__ __forceinline__ bf16x8 a_frag(const __bf16* p) {  // 8-byte aligned run of 8 bf16
    const uint2 lo = *reinterpret_cast<const uint2*>(p);
    const uint2 hi = *reinterpret_cast<const uint2*>(p + 4);
    const u32x4 v = {lo.x, lo.y, hi.x, hi.y};
    return __builtin_bit_cast(bf16x8, v);
}

__device__ __forceinline__ void rowgemm_tile(const LevelItem& it, const uint16_t* __restrict__ packed, float bias,
                                             int tx, RowShared& sm) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int hc = it.hc, wc = it.wc, hb = hc - 1, wb = wc - 1;
    const int ny = it.ny, nx = it.nx;
    const int j0 = tx * RG_COLS;
    const int mrow = lane & 15, kg = lane >> 4;
    // a wave whose 16 window columns lie past the level (a level's last tile)
    // stages rows with the others but does no MFMA work
    const bool col_live = j0 + 16 * wave < nx;

    // B fragments: HOG and LBP hi in registers, LBP lo in LDS (shared by the
    // 4 waves)
    bf16x8 bh[RG_HOG_T], blh[RG_LBP_T];
    const u32x4* pk = reinterpret_cast<const u32x4*>(packed);
#pragma unroll
    for (int t = 0; t < RG_HOG_T; ++t) bh[t] = __builtin_bit_cast(bf16x8, pk[t * 64 + lane]);
#pragma unroll
    for (int t = 0; t < RG_LBP_T; ++t) blh[t] = __builtin_bit_cast(bf16x8, pk[(RG_HOG_T + t) * 64 + lane]);
    for (int e = threadIdx.x; e < RG_LBP_T * 64; e += 256)
        reinterpret_cast<u32x4*>(sm.blbp)[e] = pk[(RG_HOG_T + RG_LBP_T) * 64 + e];
    for (int e = threadIdx.x; e < 4 * 16 * 16; e += 256) (&sm.ring[0][0][0])[e] = 0.0f;
    // zero the staged rows once so every value an MFMA reads is finite
    for (int e = threadIdx.x; e < (int)(sizeof(sm.hog) + sizeof(sm.lbp)) / 4; e += 256)
        reinterpret_cast<uint32_t*>(&sm.hog[0][0])[e] = 0u;
    __syncthreads();
    RowOffsets<true> oh;
    RowOffsets<false> ol;
    row_offsets<true>(oh, j0, wb, hb);
    row_offsets<false>(ol, j0, wc, hc);
    const auto rh_src = planes_rsrc(it.hog16, (uint64_t)PD_HOG_BLOCK * hb * wb * 2);
    const auto rl_src = planes_rsrc(it.lbp, (uint64_t)PD_LBP_BINS * hc * wc);
    // row 0 into LDS; row 1 (stored after step 0) into registers
    RowRegs<true> rh2[2];
    RowRegs<false> rl2[2];
    load_row_fast<true>(rh2[0], oh, rh_src, 0, wb, hb);
    load_row_fast<false>(rl2[0], ol, rl_src, 0, wc, hc);
    store_row_fast<true>(rh2[0], oh, sm.hog[0]);
    store_row_fast<false>(rl2[0], ol, sm.lbp[0]);
    if (1 < hc) {
        if (1 < hb) load_row_fast<true>(rh2[0], oh, rh_src, 1, wb, hb);
        load_row_fast<false>(rl2[0], ol, rl_src, 1, wc, hc);
    }
    __syncthreads();

    float (*ring)[16] = sm.ring[wave];
    // Step y: MFMAs on staged row y.  The row it stores at its end (y + 1)
    // was loaded one step earlier, and it issues the loads of row y + 2: a
    // row's loads have two steps of MFMAs to arrive.
    auto step = [&](int y, RowRegs<true>& ch, RowRegs<false>& cl, RowRegs<true>& nh, RowRegs<false>& nl)
                    __attribute__((always_inline)) {
        const int cur = y & 1;
        // issued on every step (the row index is clamped), so the number of
        // loads in flight is the same on every path and the store of row
        // y + 1 below waits only for its own loads
        load_row_fast<true>(nh, oh, rh_src, y + 2, wb, hb);
        load_row_fast<false>(nl, ol, rl_src, y + 2, wc, hc);
        // four accumulators (HOG even and odd chunks, LBP hi, LBP lo), so
        // consecutive MFMAs do not wait on one another; summed in a fixed order
        f32x4 acc_h = {0.0f, 0.0f, 0.0f, 0.0f}, acc_h1 = acc_h, acc_lh = acc_h, acc_ll = acc_h;
        if (col_live && y < hb) {
            const __bf16* row = sm.hog[cur] + (16 * wave + mrow) * RG_HOG_C + 8 * kg;
#pragma unroll
            for (int t = 0; t < RG_HOG_T; t += 2) {
                acc_h = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_frag(row + 32 * t), bh[t], acc_h, 0, 0, 0);
                acc_h1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_frag(row + 32 * t + 32), bh[t + 1], acc_h1, 0, 0, 0);
            }
        }
        if (col_live) {
            const __bf16* row = sm.lbp[cur] + (16 * wave + mrow) * RG_LBP_C + 8 * kg;
            const bf16x8* bl = reinterpret_cast<const bf16x8*>(sm.blbp);
#pragma unroll
            for (int t = 0; t < RG_LBP_T; ++t) {
                const bf16x8 av = a_frag(row + 32 * t);
                acc_lh = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, blh[t], acc_lh, 0, 0, 0);
                acc_ll = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bl[t * 64 + lane], acc_ll, 0, 0, 0);
            }
        }
        const f32x4 acc = ((acc_h + acc_h1) + acc_lh) + acc_ll;
        // acc[r] = P[y][window 4*kg + r][a = mrow] belongs to window row y - a
        {
            const int i = y - mrow;
            if (i >= 0 && i < ny) {
#pragma unroll
                for (int r = 0; r < 4; ++r) ring[i & 15][4 * kg + r] += acc[r];
            }
        }
        if (y >= PD_WIN_CELLS_Y - 1) {  // window row y - 15 is complete
            const int i = y - (PD_WIN_CELLS_Y - 1);
            if (lane < 16) {
                const float v = ring[i & 15][lane];
                ring[i & 15][lane] = 0.0f;
                const int j = j0 + 16 * wave + lane;
                if (i < ny && j < nx) gmem(it.scores)[(size_t)i * nx + j] = v + bias;
            }
        }
        if (y + 1 < hc) {
            if (y + 1 < hb) store_row_fast<true>(ch, oh, sm.hog[cur ^ 1]);
            store_row_fast<false>(cl, ol, sm.lbp[cur ^ 1]);
        }
        __syncthreads();
    };
    // two register sets for rows in flight, alternating (unrolled by two so
    // that each is a fixed set of registers)
    for (int y = 0; y < hc; y += 2) {
        step(y, rh2[0], rl2[0], rh2[1], rl2[1]);
        if (y + 1 < hc) step(y + 1, rh2[1], rl2[1], rh2[0], rl2[0]);
    }
}

__global__ void __launch_bounds__(256) rowgemm_single_kernel(LevelItem it, const uint16_t* __restrict__ packed,
                                                             const float* __restrict__ bias) {
    __shared__ RowShared sm;
    rowgemm_tile(it, packed, bias[0], blockIdx.x, sm);
}

// With LOOP a capped grid strides over the tile table (each tile ends on a
// barrier).
template <bool LOOP>
__global__ void __launch_bounds__(256) rowgemm_table_kernel(const LevelItem* __restrict__ items,
                                                            const Tile* __restrict__ tiles, int n_tiles,
                                                            const uint16_t* __restrict__ packed,
                                                            const float* __restrict__ bias) {
    __shared__ RowShared sm;
    if constexpr (LOOP) {
        for (int t = blockIdx.x; t < n_tiles; t += gridDim.x) {
            const Tile tl = tiles[t];
            rowgemm_tile(items[tl.item], packed, bias[0], tl.tx, sm);
        }
    } else {
        const Tile tl = tiles[blockIdx.x];
        rowgemm_tile(items[tl.item], packed, bias[0], tl.tx, sm);
    }
}

}  // namespace

hipError_t launch_rowgemm_single(const LevelItem& it, const uint16_t* packed, const float* bias, hipStream_t s) {
    if (it.nx <= 0 || it.ny <= 0) return hipSuccess;
    rowgemm_single_kernel<<<ceil_div(it.nx, RG_COLS), 256, 0, s>>>(it, packed, bias);
    return hipGetLastError();
}

hipError_t launch_rowgemm_table(const LevelItem* items, const Tile* tiles, int n_tiles, const uint16_t* packed,
                                const float* bias, int grid, hipStream_t s) {
    if (n_tiles <= 0) return hipSuccess;
    if (grid > 0 && grid < n_tiles)
        rowgemm_table_kernel<true><<<grid, 256, 0, s>>>(items, tiles, n_tiles, packed, bias);
    else
        rowgemm_table_kernel<false><<<n_tiles, 256, 0, s>>>(items, tiles, n_tiles, packed, bias);
    return hipGetLastError();
}

}  // namespace pd
