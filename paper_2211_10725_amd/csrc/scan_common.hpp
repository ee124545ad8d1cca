// Shared by the forward scan (scan.hip) and the reverse scan (scan_bwd.hpp).
#pragma once

#include "neuron.hpp"

namespace snn {

constexpr int kThreads = 256;
// Lanes own 2 columns when there are enough columns to fill the chip (2^19:
// 4096 waves of 2-column lanes; on the 65536 x 64-column layer 2 columns and
// 16 steps ahead measured 4-7 % faster than 4 columns and 8 steps, and 1
// column slower still), otherwise 1; the forward loads 16 steps ahead.
constexpr int kWideColumns = 4 * 64 * 2048;
constexpr int kCkpt = kCheckpointInterval;  // steps per recomputed chunk
constexpr int kFoldMax = 16;   // most outputs of a dense layer whose input gradient is folded
constexpr int kFoldRows = 5;   // batch rows one workgroup's columns can span when folding

template <int VEC>
struct Vec;
template <>
struct Vec<2> {
    static __device__ inline void load(const float *p, float (&v)[2]) {
        const float2 x = *reinterpret_cast<const float2 *>(p);
        v[0] = x.x; v[1] = x.y;
    }
    static __device__ inline void store(float *p, const float (&v)[2]) {
        *reinterpret_cast<float2 *>(p) = make_float2(v[0], v[1]);
    }
};
template <>
struct Vec<1> {
    static __device__ inline void load(const float *p, float (&v)[1]) { v[0] = *p; }
    static __device__ inline void store(float *p, const float (&v)[1]) { *p = v[0]; }
};

__device__ inline float load_as_f32(const void *p, int64_t i, int dt) {
    if (dt == SNN_F32) return reinterpret_cast<const float *>(p)[i];
    const uint16_t h = reinterpret_cast<const uint16_t *>(p)[i];
    if (dt == SNN_BF16) return __uint_as_float((uint32_t)h << 16);
    return (float)__builtin_bit_cast(_Float16, h);
}

struct ScanArgs {
    int T;
    int64_t C, N;
    float alpha, beta, thr, slope;
    const float *vrec;
};

// The layer above, for an upstream gradient folded into the scan
struct FoldIn {
    const void *dup;  // [T, B, nup] of dt_up
    const void *wup;  // [nup, N] of dt_w
    int nup, dt_up, dt_w, B;
};

struct BwdBuffers {
    const float *cur, *ckpt, *g;
    FoldIn fold;
    void *dcur;
    uint16_t *dcur_t;
    bool planes;  // dcur_t holds the planes of an fp32 dL/dI in dcur's layout
    const float *dscale;
    float *colsum, *dvcol;
};

// Sources of the upstream gradient g_t = dL/dz_t of the reverse scan.
constexpr int GM_FULL = 0;   // g [T, C]
constexpr int GM_BCAST = 1;  // g [C], the same for every t
constexpr int GM_FOLD = 2;   // g_t[b, n] = sum_j dI_up[t, b, j] W_up[j, n]: the input
                             // gradient of a dense layer above with at most
                             // kFoldMax outputs, computed here instead of read
constexpr int GM_FOLD12 = 3; // the same for at most 12 outputs (10 classes)

// launch the reverse scan of one neuron model: vec columns per lane, rs the
// surrogate reset gradient, gm GM_*, gt the dtype of dL/dI
void scan_bwd_leaky(int vec, int rs, int gm, int gt, const ScanArgs &a, const BwdBuffers &b,
                    hipStream_t s);
void scan_bwd_synaptic(int vec, int rs, int gm, int gt, const ScanArgs &a, const BwdBuffers &b,
                       hipStream_t s);
void scan_bwd_rleaky(int vec, int rs, int gm, int gt, const ScanArgs &a, const BwdBuffers &b,
                     hipStream_t s);

}  // namespace snn
