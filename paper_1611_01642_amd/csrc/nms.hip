// Threshold classification (Section 4.4) and non-maximum-suppression
// refinement (Section 3; Section 4.1 step 5, done here on the GPU).
//
// compact: four windows per thread, their loads in flight together; a
//   window's score is the max over the models (lowest model index on ties);
//   windows with score > threshold are appended to their frame's candidate
//   list, a workgroup's together, with an atomic counter.  A frame's list has room for every one of
//   its windows, so none is dropped.
// select (in the NMS kernel): for a frame with more than PD_MAX_CANDIDATES candidates, the
//   PD_MAX_CANDIDATES highest-scoring ones (score descending, then level, i,
//   j ascending: a strict order, keys are distinct) by a radix select over
//   the 64-bit NMS sort key; the selected set does not depend on the order
//   in which compaction appended the list.
// nms: one workgroup (16 waves) per frame.  Candidates are sorted by (score descending,
//   level, i, j ascending) in LDS: dealt to 1024 buckets by score and ranked
//   within their bucket (by merging if one bucket holds many); the greedy pass takes the first 64 candidates not yet suppressed,
//   resolves them against each other (IoU > 0.5, decided exactly as 2*inter >
//   union on integer boxes; a 64x64 overlap mask, one row per lane), then tests
//   the boxes they keep against every later candidate and closes the list up.
//   This is exactly the serial greedy algorithm, and needs no n x n mask in
//   memory.  One CU's vector instructions bound it: candidates suppressed early
//   are never looked at again (in chunks of 64 tested against all boxes kept
//   before, 1414 candidates, 280 kept, took 126 us in FP64 and 105 in FP32; this
//   takes 42; 190 candidates 12, from 15.5).
#include "pd_internal.h"

namespace pd {
namespace {

__global__ void __launch_bounds__(CP_THREADS) compact_kernel(const LevelItem* __restrict__ items,
                                                             const Tile* __restrict__ tiles, int n_models,
                                                             const double* __restrict__ thresholds, float margin,
                                                             int32_t* __restrict__ counters,
                                                             float* __restrict__ cand_score,
                                                             int4* __restrict__ cand_key, double* __restrict__ cand_s64,
                                                             int32_t* __restrict__ near_count,
                                                             int4* __restrict__ near_key, int64_t near_cap, int n_frames,
                                                             const float* __restrict__ kth) {
    const Tile tl = tiles[blockIdx.x];
    const LevelItem& it = items[tl.item];
    const int n = it.nx * it.ny;
    const int q0 = tl.tx * CP_N + threadIdx.x;
    __shared__ int sums[2][CP_THREADS / 64], bases[2];
    // windows q0 + k * CP_THREADS: every load is issued before the first
    // decision (windows past the level read its last one and are skipped)
    int qk[CP_PER];
    float best[CP_PER];
    int bm[CP_PER];
    bool keep[CP_PER];
#pragma unroll
    for (int k = 0; k < CP_PER; ++k) {
        qk[k] = min(q0 + k * CP_THREADS, n - 1);
        best[k] = it.scores[qk[k]];
        bm[k] = 0;
        keep[k] = true;
        if (kth) {  // pruned: only windows the network keeps can be detections
            const int wi = qk[k] / it.nx, wj = qk[k] - wi * it.nx;
            keep[k] = it.logit[(size_t)(wi + PRUNER_WIN_DI) * it.wc + wj + PRUNER_WIN_DJ] >= kth[it.frame];
        }
    }
    for (int m = 1; m < n_models; ++m) {
#pragma unroll
        for (int k = 0; k < CP_PER; ++k) {
            const float v = it.scores[(size_t)m * n + qk[k]];
            if (v > best[k]) {
                best[k] = v;
                bm[k] = m;
            }
        }
    }
    const double thr = thresholds[it.frame];
    // near: too close to call in this precision, rescored in FP64.  A workgroup's
    // windows are of one frame, so it adds to each counter once: additions to the
    // same word follow one another (1.2 million windows, 1% of them listed: one
    // per window 37 us, per wave 27, per workgroup 15)
    uint64_t near[CP_PER], over[CP_PER];
    int n_near = 0, n_over = 0;
#pragma unroll
    for (int k = 0; k < CP_PER; ++k) {
        const bool in = q0 + k * CP_THREADS < n && keep[k];
        const bool close = margin > 0.0f && fabs((double)best[k] - thr) < (double)margin;
        near[k] = __ballot(in && close);
        over[k] = __ballot(in && !close && (double)best[k] > thr);
        n_near += __popcll(near[k]);
        n_over += __popcll(over[k]);
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (lane == 0) {
        sums[0][wave] = n_near;
        sums[1][wave] = n_over;
    }
    __syncthreads();
    int at_near = 0, at_over = 0, all_near = 0, all_over = 0;
#pragma unroll
    for (int v = 0; v < CP_THREADS / 64; ++v) {
        at_near += v < wave ? sums[0][v] : 0;
        at_over += v < wave ? sums[1][v] : 0;
        all_near += sums[0][v];
        all_over += sums[1][v];
    }
    if (all_near + all_over == 0) return;  // the whole workgroup
    if (threadIdx.x == 0) {
        // near_count holds one counter per frame and, after them, the length of
        // the dense list of all frames' near windows
        if (all_near) {
            bases[0] = atomicAdd(&near_count[n_frames], all_near);
            atomicAdd(&near_count[it.frame], all_near);
        }
        if (all_over) bases[1] = atomicAdd(&counters[it.frame], all_over);
    }
    __syncthreads();
    at_near += bases[0];
    at_over += bases[1];
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int k = 0; k < CP_PER; ++k) {
        const int q = q0 + k * CP_THREADS, i = q / it.nx;
        if ((near[k] >> lane) & 1ull) {
            // (room for every window of the batch: the bound is never reached)
            const int g = at_near + __popcll(near[k] & below);
            if (g < near_cap) near_key[g] = make_int4(it.frame * PD_MAX_LEVELS + it.level, i, q - i * it.nx, bm[k]);
        } else if ((over[k] >> lane) & 1ull) {
            const int pos = at_over + __popcll(over[k] & below);
            if (pos < it.cand_cap) {  // always: a window is appended once at most
                const size_t o = (size_t)it.cand_off + pos;
                cand_score[o] = best[k];
                cand_key[o] = make_int4(it.level, i, q - i * it.nx, bm[k]);
                if (cand_s64) cand_s64[o] = __longlong_as_double(0x7ff8000000000000LL);
            }
        }
        at_near += __popcll(near[k]);
        at_over += __popcll(over[k]);
    }
}

// One workgroup of 16 waves per frame: the frame's LDS scratch allows one
// workgroup per compute unit, and the overlap tests and the sort are
// latency-bound, so the workgroup brings its own waves to hide the latency.
constexpr int NMS_WAVES = 16;
constexpr int NMS_THREADS = NMS_WAVES * 64;
constexpr int NMS_BUCKET = 64;  // most candidates of a bucket that are ranked by counting

struct NmsSmem {
    union {
        unsigned long long key[PD_MAX_CANDIDATES];  // the sort's keys;
        uint16_t list[2][PD_MAX_CANDIDATES];        // then places in the sorted order, not yet kept or suppressed
    };
    uint16_t sidx[PD_MAX_CANDIDATES];  // the sorted order
    uint16_t kpos[PD_MAX_CANDIDATES];  // kept: places in it
    union {
        struct {
            int4 cbox[PD_MAX_CANDIDATES];  // boxes in the sorted order
            float carea[PD_MAX_CANDIDATES];
        };
        struct {  // the sort's second buffer
            unsigned long long key2[PD_MAX_CANDIDATES];
            uint16_t sidx2[PD_MAX_CANDIDATES];
        };
        struct {  // the buckets: their sizes, first places, candidates
            uint32_t hist[NMS_THREADS];
            uint16_t first[NMS_THREADS + 1];
            uint16_t dealt[PD_MAX_CANDIDATES];
        };
    };
    float4 nbox[64];  // boxes kept from the last 64 candidates, as `Overlap` takes them
    float narea[64];
    unsigned long long cmask[64];  // of the 64 in work: a candidate's earlier overlaps
    unsigned long long hits[64];  // of the later ones, by 64: suppressed now
    uint32_t lo, hi, most;  // the smallest and largest high key word, the fullest bucket
    uint32_t total[NMS_WAVES];
    int nnew;
};

__device__ inline unsigned long long sort_key(float s, int4 k) {
    s = s + 0.0f;  // -0 -> +0
    uint32_t f = __float_as_uint(s);
    f = (f & 0x80000000u) ? ~f : (f | 0x80000000u);  // ascending with the float
    const uint32_t lo = ((uint32_t)k.x << 22) | ((uint32_t)k.y << 11) | (uint32_t)k.z;
    // descending score first; real keys stay below the all-ones padding key
    return ((unsigned long long)min(~f, 0xFFFFFFFEu) << 32) | lo;
}

__device__ inline int4 window_box(const NmsGeom& g, int level, int i, int j) {
    level = min(max(level, 0), g.n_levels - 1);
    // floor(256 p n0 / nk) in double: both sides of the division are integers
    // below 2^37, so a quotient that is no integer lies at least 1 / nk > 2^-15
    // from one, far more than the division's rounding; the integer division it
    // stands for takes about five times the instructions
    auto q8 = [](int p, int n0, int nk) {
        return (int)((256.0 * (double)p) * (double)n0 / (double)nk);
    };
    const int w0 = g.wh[0][0], h0 = g.wh[0][1], wk = g.wh[level][0], hk = g.wh[level][1];
    int4 b;
    b.x = q8(PD_CELL * j, w0, wk);
    b.y = q8(PD_CELL * i, h0, hk);
    b.z = q8(PD_CELL * j + PD_WIN_W, w0, wk);
    b.w = q8(PD_CELL * i + PD_WIN_H, h0, hk);
    return b;
}

// 2 * inter > union on the integer Q8 boxes.  Sides are below 2^23, so
// every product and sum here is an integer below 2^53: exact in FP64.
__device__ inline bool overlaps(const int4& a, const int4& b) {
    const int iw = min(a.z, b.z) - max(a.x, b.x);
    const int ih = min(a.w, b.w) - max(a.y, b.y);
    if (iw <= 0 || ih <= 0) return false;
    const double inter = (double)iw * (double)ih;
    const double uni = (double)(a.z - a.x) * (double)(a.w - a.y) + (double)(b.z - b.x) * (double)(b.w - b.y) - inter;
    return 2.0 * inter > uni;
}

// A third of a box's area, less 2^-20 of it, for `Overlap`; NaN for a box (of
// keys that only callers of pd_nms could give) without positive sides or with
// coordinates below 0 or past what FP32 holds.
__device__ inline float box_third(const int4& a) {
    const int w = a.z - a.x, h = a.w - a.y, far = 1 << 24;
    const bool ok = w > 0 && h > 0 && a.x >= 0 && a.y >= 0 && a.z < far && a.w < far;
    return ok ? (float)((double)w * (double)h * ((1.0 - 0x1p-20) / 3.0)) : __uint_as_float(0x7fc00000u);
}

__device__ inline float4 box_float(const int4& a) {
    return make_float4((float)a.x, (float)a.y, (float)a.z, (float)a.w);
}

// `overlaps` of one box against others, decided in FP32 where that can decide:
// 2 inter > union is inter > S, S a third of the areas' sum.  Sides are exact
// (integers below 2^24); the product, the two areas and their sum are rounded
// once each, 2^-22 in all, so inter is at most S if it is not above the sum taken
// 2^-20 less, and more than S if it is above that sum made 2^-18 more.  Between
// (`unsure`, also for a NaN) `overlaps` decides.  12 vector instructions, FP64
// takes 35.
struct Overlap {
    float4 box;
    float third;
    bool hit = false, maybe = false;
    // minimum and maximum by the bits (floats >= 0; fminf of a value from memory
    // costs an instruction more, to quieten a NaN)
    static __device__ __forceinline__ float lesser(float a, float b) {
        return __int_as_float(min(__float_as_int(a), __float_as_int(b)));
    }
    static __device__ __forceinline__ float greater(float a, float b) {
        return __int_as_float(max(__float_as_int(a), __float_as_int(b)));
    }
    __device__ __forceinline__ void test(const float4& b, float b_third) {
        const float iw = lesser(box.z, b.z) - greater(box.x, b.x), ih = lesser(box.w, b.w) - greater(box.y, b.y);
        const float inter = fmaxf(iw, 0.0f) * ih;  // negative or 0 where they are apart
        const float s = third + b_third;
        hit = hit || inter > s * (1.0f + 0x1p-18f);
        maybe = maybe || !(inter <= s);
    }
    __device__ __forceinline__ bool unsure() const { return maybe && !hit; }
};

// Finds the PD_MAX_CANDIDATES-th smallest key of the frame's list, one byte per
// pass from the top (LDS histogram of the keys that share the bytes found so
// far), then copies every entry whose key is at most that one: exactly
// PD_MAX_CANDIDATES entries, the keys being distinct.  Their order in the
// output is immaterial (NMS sorts by key).  The whole workgroup.
__device__ void select_candidates(int n, const float* __restrict__ cs, const int4* __restrict__ ck,
                                  const double* __restrict__ c64, float* __restrict__ sel_score,
                                  int4* __restrict__ sel_key, double* __restrict__ sel_s64) {
    const int t = threadIdx.x;
    __shared__ uint32_t hist[256];
    __shared__ uint32_t found[2];
    __shared__ int s_out;
    unsigned long long prefix = 0ull, mask = 0ull;
    uint32_t rank = PD_MAX_CANDIDATES;  // 1-based rank sought among the keys matching prefix
    for (int shift = 56; shift >= 0; shift -= 8) {
        if (t < 256) hist[t] = 0u;
        __syncthreads();
        for (int q = t; q < n; q += NMS_THREADS) {
            const unsigned long long key = sort_key(cs[q], ck[q]);
            if ((key & mask) == prefix) atomicAdd(&hist[(uint32_t)(key >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (t < 64) select_bin<true>(hist, rank, found);
        __syncthreads();
        rank = found[1];
        prefix |= (unsigned long long)found[0] << shift;
        mask |= 255ull << shift;
        __syncthreads();  // found is rewritten by the next pass
    }
    if (t == 0) s_out = 0;
    __syncthreads();
    for (int q = t; q < n; q += NMS_THREADS) {
        if (sort_key(cs[q], ck[q]) <= prefix) {
            const int pos = atomicAdd(&s_out, 1);
            if (pos < PD_MAX_CANDIDATES) {
                sel_score[pos] = cs[q];
                sel_key[pos] = ck[q];
                if (sel_s64) sel_s64[pos] = c64[q];
            }
        }
    }
    __syncthreads();
}

// Lane 63: the wave's largest value; every lane: the sum up to it (data-parallel
// moves within a row of 16 lanes, then from row to row).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t moved(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
constexpr int ROW_SHR = 0x110, ROW_BCAST15 = 0x142, ROW_BCAST31 = 0x143;

__device__ __forceinline__ uint32_t wave_last_max(uint32_t v) {
    v = max(v, moved<ROW_SHR + 1, 0xf>(v));
    v = max(v, moved<ROW_SHR + 2, 0xf>(v));
    v = max(v, moved<ROW_SHR + 4, 0xf>(v));
    v = max(v, moved<ROW_SHR + 8, 0xf>(v));
    v = max(v, moved<ROW_BCAST15, 0xa>(v));
    return max(v, moved<ROW_BCAST31, 0xc>(v));
}

__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
    v += moved<ROW_SHR + 1, 0xf>(v);
    v += moved<ROW_SHR + 2, 0xf>(v);
    v += moved<ROW_SHR + 4, 0xf>(v);
    v += moved<ROW_SHR + 8, 0xf>(v);
    v += moved<ROW_BCAST15, 0xa>(v);
    return v + moved<ROW_BCAST31, 0xc>(v);
}

// Sorts keys and indices [0, n) in LDS, entries up to the next multiple of 64
// padded with the largest key: each wave sorts runs of 64 in registers (bitonic),
// then runs are merged pairwise, every element finding its place in the other
// run by bisection (equal keys stay in run order).
__device__ void merge_sort(NmsSmem& sm, int n) {
    const int t = threadIdx.x, lane = t & 63;
    const int np = (n + 63) & ~63;
    unsigned long long* ka = sm.key;
    uint16_t* ia = sm.sidx;
    unsigned long long* kb = sm.key2;
    uint16_t* ib = sm.sidx2;
    for (int q = t; q < np; q += NMS_THREADS) {  // whole waves
        unsigned long long key = ka[q];
        int idx = ia[q];
#pragma unroll
        for (int k = 2; k <= 64; k <<= 1) {
#pragma unroll
            for (int j = k >> 1; j > 0; j >>= 1) {
                const unsigned long long other = __shfl_xor(key, j, 64);
                const int oidx = __shfl_xor(idx, j, 64);
                const bool small = ((lane & k) == 0) == ((lane & j) == 0);  // this lane keeps the smaller
                // equal keys: neither lane takes the other's
                const bool take = small ? other < key : other > key;
                key = take ? other : key;
                idx = take ? oidx : idx;
            }
        }
        ka[q] = key;
        ia[q] = (uint16_t)idx;
    }
    __syncthreads();
    for (int len = 64; len < np; len *= 2) {
        for (int q = t; q < np; q += NMS_THREADS) {
            const unsigned long long key = ka[q];
            const bool right = (q & len) != 0;
            const int base = q & ~(2 * len - 1);                   // the pair of runs
            const int o0 = right ? base : base + len;              // the other run
            const int on = right ? len : max(min(len, np - o0), 0);
            int lo = 0, hi = on;  // elements of the other run before this one
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                const unsigned long long k = ka[o0 + mid];
                if (right ? k <= key : k < key) lo = mid + 1;
                else hi = mid;
            }
            const int at = base + (q & (len - 1)) + lo;
            kb[at] = key;
            ib[at] = ia[q];
        }
        __syncthreads();
        unsigned long long* const kt = ka;
        ka = kb;
        kb = kt;
        uint16_t* const it = ia;
        ia = ib;
        ib = it;
    }
    if (ia != sm.sidx) {  // (only the order is used from here on)
        for (int q = t; q < n; q += NMS_THREADS) sm.sidx[q] = ia[q];
        __syncthreads();
    }
}

// sm.sidx: the frame's n candidates in the order of their keys.  Buckets of
// equal width between the smallest and the largest score (their bits, which
// ascend with them), so that a bucket holds a few candidates of which each
// counts the smaller ones; merged where one holds more than NMS_BUCKET (many
// equal scores).  For 1414 candidates 11500 cycles, merging takes 35000; for 190
// 6500, each counting the smaller ones of all took 8500.
__device__ void sort_candidates(NmsSmem& sm, int n, const float* __restrict__ cs, const int4* __restrict__ ck) {
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int np = (n + 63) & ~63;
    if (t == 0) {
        sm.lo = ~0u;
        sm.hi = 0u;
        sm.most = 0u;
    }
    sm.hist[t] = 0u;
    __syncthreads();
    uint32_t lo = ~0u, hi = 0u;
    for (int q = t; q < np; q += NMS_THREADS) {
        const unsigned long long key = q < n ? sort_key(cs[q], ck[q]) : ~0ull;
        sm.key[q] = key;
        sm.sidx[q] = (uint16_t)q;
        if (q < n) {
            lo = min(lo, (uint32_t)(key >> 32));
            hi = max(hi, (uint32_t)(key >> 32));
        }
    }
    lo = ~wave_last_max(~lo);
    hi = wave_last_max(hi);
    if (lane == 63 && lo <= hi) {
        atomicMin(&sm.lo, lo);
        atomicMax(&sm.hi, hi);
    }
    __syncthreads();
    lo = sm.lo;
    // monotone in the key: each step rounds monotonically
    const float scale = (float)NMS_THREADS / ((float)(sm.hi - lo) + 1.0f);
    auto bucket = [&](int q) {
        return min((int)((float)((uint32_t)(sm.key[q] >> 32) - lo) * scale), NMS_THREADS - 1);
    };
    for (int q = t; q < n; q += NMS_THREADS) atomicAdd(&sm.hist[bucket(q)], 1u);
    __syncthreads();
    // the buckets' first places
    const uint32_t size = sm.hist[t];
    const uint32_t end = wave_scan(size), most = wave_last_max(size);
    if (lane == 63) sm.total[wave] = end;
    if (lane == 63 && most > NMS_BUCKET) sm.most = most;  // (any that is too full)
    __syncthreads();
    if (sm.most) {
        merge_sort(sm, n);
        return;
    }
    uint32_t before = 0;
#pragma unroll
    for (int v = 0; v < NMS_WAVES; ++v) before += v < wave ? sm.total[v] : 0u;
    sm.first[t + 1] = (uint16_t)(before + end);
    if (t == 0) sm.first[0] = 0;
    sm.hist[t] = before + end - size;  // the next free place
    __syncthreads();
    for (int q = t; q < n; q += NMS_THREADS) sm.dealt[atomicAdd(&sm.hist[bucket(q)], 1u)] = (uint16_t)q;
    __syncthreads();
    for (int e = t; e < n; e += NMS_THREADS) {
        const int q = sm.dealt[e], b = bucket(q);
        const unsigned long long mine = sm.key[q];
        const int f = sm.first[b], l = sm.first[b + 1];
        int rank = f;
        for (int x = f; x < l; ++x) {
            const int o = sm.dealt[x];
            const unsigned long long k = sm.key[o];
            rank += (k < mine || (k == mine && o < q)) ? 1 : 0;  // (equal keys: only callers of pd_nms)
        }
        sm.sidx[rank] = (uint16_t)q;
    }
    __syncthreads();
}

__device__ void nms_frame(const NmsGeom& g, int frame, int raw_count, const float* __restrict__ cs,
                          const int4* __restrict__ ck, const double* __restrict__ c64, int rescored,
                          pd_box* __restrict__ boxes, int cap, pd_counts* __restrict__ counts) {
    extern __shared__ __align__(16) uint8_t smem_raw[];
    NmsSmem& sm = *reinterpret_cast<NmsSmem*>(smem_raw);
    const int t = threadIdx.x;
    const int n = min(raw_count, PD_MAX_CANDIDATES);
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    sort_candidates(sm, n, cs, ck);
    for (int q = t; q < n; q += NMS_THREADS) {
        const int4 k = ck[sm.sidx[q]];
        const int4 box = window_box(g, k.x, k.y, k.z);
        sm.cbox[q] = box;
        sm.carea[q] = box_third(box);
        sm.list[0][q] = (uint16_t)q;
    }
    if (t < 64) sm.cmask[t] = 0ull;
    __syncthreads();
    int K = 0;  // kept so far
    uint16_t *list = sm.list[0], *next = sm.list[1];
    for (int left = n; left > 0;) {
        const int m = min(64, left);
        // overlaps among the first m: lane q with the candidate d after it
        // (around), 32 distances split over the waves
        if (lane < m) {
            const int p = list[lane];
            const int4 box = sm.cbox[p];
            const float4 fbox = box_float(box);
            const float third = sm.carea[p];
#pragma unroll
            for (int u = 0; u < 32 / NMS_WAVES; ++u) {
                const int r = (lane + 1 + wave * (32 / NMS_WAVES) + u) & 63;
                if (r < m) {
                    const int pr = list[r];
                    Overlap o{fbox, third};
                    o.test(box_float(sm.cbox[pr]), sm.carea[pr]);
                    if (o.unsure()) o.hit = overlaps(box, sm.cbox[pr]);
                    if (o.hit) atomicOr(&sm.cmask[max(lane, r)], 1ull << min(lane, r));
                }
            }
        }
        __syncthreads();
        if (wave == 0) {
            // a candidate all of whose earlier overlaps are suppressed is kept,
            // one with a kept earlier overlap suppressed: the first undecided
            // one is decided in each turn at least
            const unsigned long long earlier = sm.cmask[lane];
            sm.cmask[lane] = 0ull;
            sm.hits[lane] = 0ull;
            unsigned long long todo = m == 64 ? ~0ull : (1ull << m) - 1ull, kept = 0ull, gone = 0ull;
            while (todo) {
                const bool mine = (todo >> lane) & 1ull;
                kept |= __ballot(mine && (earlier & ~gone) == 0ull);
                gone |= __ballot(mine && (earlier & kept) != 0ull);
                todo &= ~(kept | gone);
            }
            if ((kept >> lane) & 1ull) {
                const int at = __popcll(kept & ((1ull << lane) - 1ull)), p = list[lane];
                sm.kpos[K + at] = (uint16_t)p;
                sm.nbox[at] = box_float(sm.cbox[p]);
                sm.narea[at] = sm.carea[p];
            }
            if (lane == 0) sm.nnew = __popcll(kept);
        }
        __syncthreads();
        const int fresh = sm.nnew;
        K += fresh;
        if (left == m) break;
        // the later ones, by 64, against the boxes just kept, four per step; with
        // few of them the boxes are split over the waves (above 16 groups in two,
        // so that the last turn is less empty)
        const int rest = left - m, groups = (rest + 63) >> 6;
        const int parts = groups <= NMS_WAVES / 2 ? NMS_WAVES / groups : groups <= NMS_WAVES ? 1 : 2;
        const int per = (fresh + parts - 1) / parts;
        for (int task = wave; task < groups * parts; task += NMS_WAVES) {
            const int part = task / groups, grp = task - part * groups;
            const int k_end = min(fresh, (part + 1) * per);
            const int e = m + 64 * grp + lane;
            bool in = e < left;
            const int p = list[min(e, left - 1)];
            const int4 box = sm.cbox[p];
            const float4 fbox = box_float(box);
            const float third = sm.carea[p];
            unsigned long long hit = 0ull;
            for (int k0 = part * per; k0 < k_end && __any(in); k0 += 4) {
                Overlap o{fbox, third};
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int k = min(k0 + u, k_end - 1);
                    o.test(sm.nbox[k], sm.narea[k]);
                }
                if (o.unsure())
                    for (int k = k0; k < min(k0 + 4, k_end); ++k)
                        o.hit = o.hit || overlaps(box, sm.cbox[sm.kpos[K - fresh + k]]);
                hit |= __ballot(in && o.hit);
                in = in && !o.hit;
            }
            if (lane == 0 && hit) atomicOr(&sm.hits[grp], hit);
        }
        __syncthreads();
        // closed up, in order; lane: a group's remaining ones
        const unsigned long long all = lane < groups - 1 || (lane == groups - 1 && (rest & 63) == 0)
                                           ? ~0ull
                                           : lane == groups - 1 ? (1ull << (rest & 63)) - 1ull : 0ull;
        const unsigned long long stay = lane < groups ? all & ~sm.hits[lane] : 0ull;
        const int c = __popcll(stay);  // 0..64
        auto count = [&](int end) {  // candidates left in the groups before `end`
            int sum = 0;
#pragma unroll
            for (int b = 0; b < 7; ++b) sum += __popcll(__ballot(lane < end && ((c >> b) & 1))) << b;
            return sum;
        };
        for (int grp = wave; grp < groups; grp += NMS_WAVES) {
            const unsigned long long mine =
                (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)stay, grp) |
                (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(stay >> 32), grp) << 32;
            const int at = count(grp);
            if ((mine >> lane) & 1ull)
                next[at + __popcll(mine & ((1ull << lane) - 1ull))] = list[m + 64 * grp + lane];
        }
        left = count(64);
        uint16_t* const swap = list;
        list = next;
        next = swap;
        __syncthreads();
    }

    const int nout = min(K, cap);
    for (int q = t; q < nout; q += NMS_THREADS) {
        const int src = sm.sidx[sm.kpos[q]];
        const int4 k = ck[src];
        pd_box b;
        b.frame = frame;
        b.level = k.x;
        b.i = k.y;
        b.j = k.z;
        b.model = k.w;
        const int4 bx = sm.cbox[sm.kpos[q]];
        b.x0 = bx.x;
        b.y0 = bx.y;
        b.x1 = bx.z;
        b.y1 = bx.w;
        b.score = cs[src];
        b.score64 = c64 ? c64[src] : __longlong_as_double(0x7ff8000000000000LL);
        boxes[(size_t)frame * cap + q] = b;
    }
    if (t == 0) {
        pd_counts c;
        c.candidates = raw_count;
        c.kept = nout;
        c.overflow = (raw_count > PD_MAX_CANDIDATES || K > cap) ? 1 : 0;
        c.rescored = rescored;
        counts[frame] = c;
    }
}

__global__ void __launch_bounds__(NMS_THREADS) nms_table_kernel(const NmsGeom* __restrict__ geoms,
                                                        const int32_t* __restrict__ counters,
                                                        const float* __restrict__ cand_score,
                                                        const int4* __restrict__ cand_key,
                                                        const double* __restrict__ cand_s64,
                                                        float* __restrict__ sel_score, int4* __restrict__ sel_key,
                                                        double* __restrict__ sel_s64,
                                                        const int32_t* __restrict__ near_count,
                                                        pd_box* __restrict__ boxes, int cap,
                                                        pd_counts* __restrict__ counts) {
    const int f = blockIdx.x;
    const int n = counters[f];
    const size_t o = (size_t)geoms[f].cand_off;
    const float* cs = cand_score + o;
    const int4* ck = cand_key + o;
    const double* c64 = cand_s64 ? cand_s64 + o : nullptr;
    if (n > PD_MAX_CANDIDATES) {  // the highest-scoring candidates, in the frame's slot of the sel_* arrays
        const size_t so = (size_t)f * PD_MAX_CANDIDATES;
        float* const ss = sel_score + so;
        int4* const sk = sel_key + so;
        double* const s64 = sel_s64 ? sel_s64 + so : nullptr;
        select_candidates(min(n, geoms[f].cand_cap), cs, ck, c64, ss, sk, s64);
        cs = ss;
        ck = sk;
        c64 = s64;
    }
    nms_frame(geoms[f], f, n, cs, ck, c64, near_count ? near_count[f] : 0, boxes, cap, counts);
}

__global__ void __launch_bounds__(NMS_THREADS) nms_single_kernel(NmsGeom g, int n, const float* __restrict__ cs,
                                                         const int4* __restrict__ ck, pd_box* __restrict__ boxes,
                                                         int cap, pd_counts* __restrict__ counts) {
    nms_frame(g, 0, n, cs, ck, nullptr, 0, boxes, cap, counts);
}

constexpr size_t kNmsSmem = sizeof(NmsSmem);
static_assert(kNmsSmem <= 160 * 1024, "NMS scratch exceeds LDS");

}  // namespace

hipError_t launch_compact(const LevelItem* items, const Tile* tiles, int n_tiles, int n_models,
                          const double* thresholds, float margin, int32_t* counters, float* cand_score,
                          int4* cand_key, double* cand_s64, int32_t* near_count, int4* near_key, int64_t near_cap,
                          int n_frames, const float* kth, hipStream_t s) {
    if (n_tiles <= 0) return hipSuccess;
    compact_kernel<<<n_tiles, CP_THREADS, 0, s>>>(items, tiles, n_models, thresholds, margin, counters, cand_score, cand_key,
                                           cand_s64, near_count, near_key, near_cap, n_frames, kth);
    return hipGetLastError();
}

hipError_t launch_nms_table(const NmsGeom* geoms, int n_frames, const int32_t* counters,
                            const float* cand_score, const int4* cand_key, const double* cand_s64,
                            float* sel_score, int4* sel_key, double* sel_s64,
                            const int32_t* near_count, pd_box* boxes, int cap, pd_counts* counts, hipStream_t s) {
    if (n_frames <= 0) return hipSuccess;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&nms_table_kernel),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kNmsSmem);
    if (attr != hipSuccess) return attr;
    nms_table_kernel<<<n_frames, NMS_THREADS, kNmsSmem, s>>>(geoms, counters, cand_score, cand_key, cand_s64,
                                                             sel_score, sel_key, sel_s64, near_count, boxes, cap,
                                                             counts);
    return hipGetLastError();
}

hipError_t launch_nms_single(const NmsGeom& g, int n, const float* cand_score, const int4* cand_key,
                             pd_box* boxes, int cap, pd_counts* counts, hipStream_t s) {
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&nms_single_kernel),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kNmsSmem);
    if (attr != hipSuccess) return attr;
    nms_single_kernel<<<1, NMS_THREADS, kNmsSmem, s>>>(g, n, cand_score, cand_key, boxes, cap, counts);
    return hipGetLastError();
}

}  // namespace pd
