// What a call computes once from its weights before the first use: the packed
// operands of packed.h, all in one launch (a launch each took 4 to 5 us, up to
// six of them for a pruned BF16 call).
#include "packed.h"

namespace pd {
namespace {

constexpr int L1 = LayerDims<1>::PACKED, L2 = LayerDims<2>::PACKED, L3 = LayerDims<3>::PACKED;

__global__ void __launch_bounds__(256) prep_kernel(Prep p) {
    int e = blockIdx.x * 256 + threadIdx.x;
    // the parts a call wants, one after another in the index
    if (p.s32) {
        if (e < p.n_models * S32_MODEL) {
            p.s32[e] = packed_s32(p.weights, e);
            return;
        }
        e -= p.n_models * S32_MODEL;
    }
    if (p.rowgemm) {
        if (e < RG_PACKED) {
            p.rowgemm[e] = packed_rowgemm(p.weights, e);
            return;
        }
        e -= RG_PACKED;
    }
    if (p.mfma) {
        if (e < MF_PACKED) {
            p.mfma[e] = packed_mfma(p.weights, p.n_models, e);
            return;
        }
        e -= MF_PACKED;
    }
    if (p.layers) {
        const float* w = p.pruner;
        if (e < L1 + L2 + L3) {
            uint16_t v;
            if (e < L1) v = packed_layer<1>(w, e);
            else if (e < L1 + L2) v = packed_layer<2>(w + LayerDims<1>::PARAMS + 32, e - L1);
            else v = packed_layer<3>(w + LayerDims<1>::PARAMS + 32 + LayerDims<2>::PARAMS + 32, e - L1 - L2);
            p.layers[e] = v;
            return;
        }
        e -= L1 + L2 + L3;
    }
    if (p.orient && e < ORIENT_W * ORIENT_H) p.orient[e] = packed_orient(e);
}

}  // namespace

int64_t score32_packed_floats(int n_models) { return (int64_t)n_models * S32_MODEL; }
int64_t packed_weight_elems() { return MF_PACKED; }
int64_t rowgemm_packed_elems() { return RG_PACKED; }
int64_t pruner_packed_bf16_elems() { return L1 + L2 + L3; }

hipError_t launch_prep(const Prep& p, hipStream_t s) {
    const int n = (p.s32 ? p.n_models * S32_MODEL : 0) + (p.rowgemm ? RG_PACKED : 0) + (p.mfma ? MF_PACKED : 0) +
                  (p.layers ? L1 + L2 + L3 : 0) + (p.orient ? ORIENT_W * ORIENT_H : 0);
    if (n <= 0) return hipSuccess;
    prep_kernel<<<ceil_div(n, 256), 256, 0, s>>>(p);
    return hipGetLastError();
}

}  // namespace pd
