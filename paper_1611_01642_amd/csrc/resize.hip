// Pyramid resize (Section 4.1 step 2, Section 4.4): every level is resampled
// from the level-0 image with pixel-centre-aligned bilinear interpolation in
// Q8 fixed point, rounded half up.  All arithmetic is integer, so results are
// exact.
//
// A wave owns 256 columns (four per lane) x 4..16 rows of one level and walks
// down the rows.  The horizontal pass of a source row, (256 - fx) p0 + fx p1 per
// column, is one dot product of the bytes (p0, p0, p1) with (255 - fx, 1, fx),
// picked by one byte permutation out of 8 source bytes that the lane loads
// itself, + 128 (one load for all four columns up to a scale of 2, one for two
// columns up to 6, else one each: the three words that hold the 8 bytes, shifted;
// words past the row read as 0).  An output row is then (256 - fy) top + fy bot,
// the two 128 giving the rounding's 2^15 (the sum is below 2^25); the lower row's
// horizontal pass serves the next output row where that starts on it (9 of 10
// rows at a scale of 1.1, half of them at 1.5), and the next output row's loads
// are in flight during the current one's arithmetic.
//
// No LDS and no barrier.  Staging the tile's source rectangle in LDS took 389
// us for 256 frames of 1242x375 and 569 us for 64 of 1920x1080 (149 of the 389
// for a tile's set-up and barriers); loading the 8 bytes at any alignment 354 and
// 444 (an unaligned load takes a third more of the vector memory unit's time
// than the same load from a word boundary); this takes 311 and 400, bound by
// that unit and the loads' latency.
#include "pd_internal.h"

namespace pd {
namespace {

// Q8 source coordinate of output sample `x` along an axis of n0 -> nk
// samples: ((2x + 1) n0 - nk) * 128 / nk, the integer quotient truncated,
// split into index (s >> 8) and fraction (s & 255).  The numerator (>= 0,
// below 2^39) is exact in double; its product with the FP32 reciprocal of nk
// is off by less than 1 (a quotient is below 2^22, the reciprocal's error
// below 2^-23 of it), and the exact remainder says which way.  (A division in
// double takes four times the instructions.)
__device__ __forceinline__ uint32_t q8_coord(int x, int n0, int nk) {
    const double k = (double)nk;
    const double num = fma((double)(2 * x + 1), 128.0 * (double)n0, -128.0 * k);
    const double q = __builtin_trunc(num * (double)__builtin_amdgcn_rcpf((float)nk));
    const double r = fma(-q, k, num);
    return (uint32_t)q + (r >= k ? 1u : 0u) - (r < 0.0 ? 1u : 0u);
}

typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));

// The walk: columns x0 .. x0 + 3 of the lane, rows y0 .. y1 - 1 (at most 64),
// NL loads per source row.
template <int NL>
__device__ __forceinline__ void resize_walk(gptr<const uint8_t> __restrict__ src, int sw, int sh, int spitch,
                                            gptr<uint8_t> __restrict__ dst, int w, int h, int pitch, int x0, int y0,
                                            int y1) {
    constexpr int CPL = 4 / NL;  // columns per load
    const int lane = threadIdx.x & 63;
    // the lane's columns: the first source byte of each load, and each column's
    // byte selector and weights (a column past the edge repeats the last one;
    // its byte is masked off.  The right tap is the byte after the left one;
    // where the image clamps it, its weight is 0 instead.)
    uint32_t start[NL], sel[4], wt[4], keep = 0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t c = q8_coord(min(x0 + q, w - 1), sw, w);
        const int xa = (int)(c >> 8);
        if (q % CPL == 0) start[q / CPL] = (uint32_t)xa;
        const uint32_t f = xa + 1 < sw ? c & 255u : 0u, o = (uint32_t)xa - start[q / CPL];
        wt[q] = (255u - f) | 1u << 8 | f << 16;
        sel[q] = o | o << 8 | (o + 1u) << 16 | 0x0c000000u;
        if (x0 + q < w) keep |= 255u << (8 * q);
    }
    // row coordinates, lane r: row y0 + r
    const uint32_t rows = q8_coord(min(y0 + lane, h - 1), sh, h);
    struct Raw {
        u32x3 v[NL];
        uint32_t mis;  // the row's bytes past a word boundary
    };
    auto fetch = [&](int y, Raw& o) __attribute__((always_inline)) {
        const auto row = reinterpret_cast<uintptr_t>(src + (size_t)y * spitch);
        o.mis = (uint32_t)row & 3u;
        const auto rsrc = planes_rsrc(reinterpret_cast<const void*>(row - o.mis), (o.mis + (uint32_t)sw + 3u) & ~3u);
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const uint32_t off = (start[k] + o.mis) & ~3u;
            o.v[k] = __builtin_amdgcn_raw_buffer_load_b96(rsrc, off, 0, 0);
            asm volatile("" ::"v"(off));  // a register of its own (in the load's, it would wait for the last one)
        }
    };
    auto horizontal = [&](const Raw& r, uint32_t (&o)[4]) __attribute__((always_inline)) {
        uint32_t lo[NL], hi[NL];
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const uint32_t mis = (start[k] + r.mis) & 3u;
            lo[k] = __builtin_amdgcn_alignbyte(r.v[k].y, r.v[k].x, mis);
            hi[k] = __builtin_amdgcn_alignbyte(r.v[k].z, r.v[k].y, mis);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            o[q] = __builtin_amdgcn_udot4(__builtin_amdgcn_perm(hi[q / CPL], lo[q / CPL], sel[q]), wt[q], 128u, false);
    };
    // uniform: source row and weight of output row r; the lower source row
    auto coord = [&](int r) { return (uint32_t)__builtin_amdgcn_readlane(rows, r); };
    auto lower = [&](int ya) { return min(ya + 1, sh - 1); };
    uint32_t c = coord(0);
    Raw ra, rb, na, nb;
    fetch((int)(c >> 8), ra);
    fetch(lower((int)(c >> 8)), rb);
    uint32_t top[4], bot[4] = {0u, 0u, 0u, 0u};
    bool reuse = false;  // this row's upper source row is the last one's lower
    const int n = y1 - y0;
    auto o = dst + (size_t)y0 * pitch + x0;
    auto step = [&](int r, const Raw& ua, const Raw& ub, Raw& pa, Raw& pb) __attribute__((always_inline)) {
        // the next row's loads first (past the last row: its own again)
        const uint32_t c1 = coord(min(r + 1, n - 1));
        const int ya1 = (int)(c1 >> 8);
        const bool reuse1 = ya1 == lower((int)(c >> 8));
        if (!reuse1) fetch(ya1, pa);
        fetch(lower(ya1), pb);
        if (reuse) {
#pragma unroll
            for (int q = 0; q < 4; ++q) top[q] = bot[q];
        } else {
            horizontal(ua, top);
        }
        horizontal(ub, bot);
        const uint32_t fy = c & 255u;
        uint32_t d[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) d[q] = __umul24(top[q], 256u - fy) + __umul24(bot[q], fy);
        // the bytes at bits 16..23, one per column
        const uint32_t packed = __builtin_amdgcn_perm(d[1], d[0], 0x0c0c0602u) |
                                __builtin_amdgcn_perm(d[3], d[2], 0x06020c0cu);
        // pitch is a multiple of 16 >= w, so the 4-byte store stays in the row
        if (x0 < w) *reinterpret_cast<gptr<uint32_t>>(o) = packed & keep;
        o += pitch;
        c = c1;
        reuse = reuse1;
    };
    // two rows a turn, so that the loads land in registers of their own (a copy
    // at the end of a row would wait for them)
    for (int r = 0; r < n; r += 2) {
        step(r, ra, rb, na, nb);
        if (r + 1 < n) step(r + 1, na, nb, ra, rb);
    }
}

// Output rows y_base .. y_base + rows - 1, split over the workgroup's waves,
// columns tx * RS_TX .. + RS_TX - 1.
__device__ __forceinline__ void resize_tile(gptr<const uint8_t> __restrict__ src, int sw, int sh, int spitch,
                                            gptr<uint8_t> __restrict__ dst, int w, int h, int pitch, int y_base,
                                            int rows, int tx) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int x0 = tx * RS_TX + 4 * lane;
    const int per = (rows + 3) >> 2;
    const int y0 = y_base + wave * per, y1 = min(min(y0 + per, y_base + rows), h);
    if (y0 >= y1) return;
    if (sw <= 2 * w) resize_walk<1>(src, sw, sh, spitch, dst, w, h, pitch, x0, y0, y1);
    else if (sw <= 6 * w) resize_walk<2>(src, sw, sh, spitch, dst, w, h, pitch, x0, y0, y1);
    else resize_walk<4>(src, sw, sh, spitch, dst, w, h, pitch, x0, y0, y1);
}

struct ResizeArgs {
    const uint8_t* src;
    uint8_t* dst;
    int32_t sw, sh, spitch, n, rows;  // rows: per tile
    int32_t prefix[PD_MAX_LEVELS + 1];  // first tile of each level
    int32_t w[PD_MAX_LEVELS], h[PD_MAX_LEVELS], pitch[PD_MAX_LEVELS];
    int64_t off[PD_MAX_LEVELS];
};

__global__ void __launch_bounds__(256) resize_single_kernel(ResizeArgs a) {
    const int b = blockIdx.x;
    int k = 0;
    while (k + 1 < a.n && a.prefix[k + 1] <= b) ++k;
    const int local = b - a.prefix[k];
    const int ntx = (a.w[k] + RS_TX - 1) / RS_TX;
    resize_tile(gmem(a.src), a.sw, a.sh, a.spitch, gmem(a.dst) + a.off[k], a.w[k], a.h[k], a.pitch[k],
                (local / ntx) * a.rows, a.rows, local % ntx);
}

// Workgroups are dealt to the XCDs round-robin; each XCD takes a contiguous
// run of the table instead, so the levels of a frame, which all read the same
// source image, mostly share one XCD's L2.
__global__ void __launch_bounds__(256) resize_table_kernel(const LevelItem* __restrict__ items,
                                                           const Tile* __restrict__ tiles, int n_tiles,
                                                           int32_t* __restrict__ zero, int n_zero) {
    // the call's counters, cleared here (a launch of their own would cost 4 us)
    for (int e = (int)blockIdx.x * 256 + threadIdx.x; e < n_zero; e += (int)gridDim.x * 256) zero[e] = 0;
    const int run = (n_tiles + N_XCD - 1) / N_XCD;
    const int t = (int)(blockIdx.x % N_XCD) * run + (int)(blockIdx.x / N_XCD);
    if (t >= n_tiles) return;
    const Tile tl = tiles[t];
    const LevelItem& it = items[tl.item];
    // tile: first row in ty, row count in pad
    resize_tile(gmem(it.src), it.src_w, it.src_h, it.src_pitch, gmem(it.pyr), it.w, it.h, it.pitch, tl.ty, tl.pad,
                tl.tx);
}

}  // namespace

hipError_t launch_resize_single(const LevelItem* items, int n_items, hipStream_t s) {
    if (n_items <= 0) return hipSuccess;
    ResizeArgs a = {};
    a.src = items[0].src;
    a.dst = items[0].pyr;
    a.sw = items[0].src_w;
    a.sh = items[0].src_h;
    a.spitch = items[0].src_pitch;
    a.n = n_items;
    int total = 0;
    for (int k = 0; k < n_items; ++k) total += resize_tiles_x(items[k].w) * resize_tiles_y(items[k].h);
    a.rows = resize_rows(total);
    total = 0;
    for (int k = 0; k < n_items; ++k) {
        a.prefix[k] = total;
        a.w[k] = items[k].w;
        a.h[k] = items[k].h;
        a.pitch[k] = items[k].pitch;
        a.off[k] = items[k].pyr - items[0].pyr;
        total += resize_tiles_x(items[k].w) * ceil_div(items[k].h, a.rows);
    }
    a.prefix[n_items] = total;
    resize_single_kernel<<<total, 256, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_resize_table(const LevelItem* items, const Tile* tiles, int n_tiles, int32_t* zero, int n_zero,
                               hipStream_t s) {
    const int grid = N_XCD * ((n_tiles + N_XCD - 1) / N_XCD);
    resize_table_kernel<<<grid > 0 ? grid : 1, 256, 0, s>>>(items, tiles, n_tiles, zero, n_zero);
    return hipGetLastError();
}

}  // namespace pd
