// Neuron time scans for gfx950: forward (eqs. 3-7) and the BPTT reverse scan
// with the fast-sigmoid surrogate (eqs. 8-9).
//
// Layout: every tensor is time-major [T, C] with C = B * n columns, column
// fastest.  One lane owns VEC consecutive columns for all T steps and keeps
// the neuron state in registers; a wave therefore streams 64*VEC contiguous
// floats per step (512 bytes for VEC = 2), fully coalesced.  The inputs of the
// next D steps do not depend on the state, so each lane keeps a ring of D
// prefetched steps in registers to keep enough HBM requests in flight while
// the sequential recurrence runs.
//
// Saved state: the backward needs u_t at every step (the surrogate is a
// function of u_t alone).  Instead of writing u (4 B per step and column) the
// forward writes the state every kCkpt steps (checkpoints: u, and i for the
// current-based neuron), and the reverse scan recomputes each chunk of kCkpt
// steps forward from its checkpoint and the currents, in registers and with
// the forward's exact fp32 operations (so u is bit-identical), before
// running the chunk backwards.
#include <atomic>

#include "scan_common.hpp"

namespace snn {
namespace {

// spikes as bytes 0/1
template <int VEC>
__device__ inline void store_spikes_u8(uint8_t *p, const float (&z)[VEC]) {
    if constexpr (VEC == 2) {
        *reinterpret_cast<uint16_t *>(p) = (uint16_t)((uint32_t)z[0] | ((uint32_t)z[1] << 8));
    } else {
        p[0] = (uint8_t)z[0];
    }
}

// spikes as fp16 0.0 / 1.0 (0x3c00)
template <int VEC>
__device__ inline void store_spikes_f16(uint16_t *p, const float (&z)[VEC]) {
    if constexpr (VEC == 2) {
        *reinterpret_cast<uint32_t *>(p) =
            (z[0] != 0.f ? 0x3c00u : 0u) | (z[1] != 0.f ? 0x3c000000u : 0u);
    } else {
        p[0] = z[0] != 0.f ? 0x3c00u : 0u;
    }
}

// Spikes packed to bits, one wave's columns per step: a ballot per column
// slot of the lanes.  Lanes that pack bits own the columns w0 + lane + 64 v
// of their wave's 64 VEC columns (w0 the wave's first column, a multiple of
// 64 VEC: the launcher takes VEC = 2 only when C is a multiple of 128, and C
// is a multiple of 64), so ballot v is the 64-bit word of columns
// w0 + 64 v .. + 63.  Lane 0 stores the wave's VEC words.
template <int VEC>
__device__ inline void store_spikes_bits(uint64_t *words, int64_t wave_off, const float (&z)[VEC]) {
    const int lane = threadIdx.x & 63;
    const uint64_t w0 = __ballot(z[0] > 0.f);
    if constexpr (VEC == 2) {
        const uint64_t w1 = __ballot(z[1] > 0.f);
        if (lane == 0)
            *reinterpret_cast<ulonglong2 *>(words + wave_off / 64) = make_ulonglong2(w0, w1);
    } else {
        if (lane == 0) words[wave_off / 64] = w0;
    }
}

// Forward scan.  Writes the spikes, the spike counts (nullable), the full
// membrane (u_out with UOUT; it may alias cur exactly: each lane reads step t
// before it writes it) and the checkpoints: after step t with
// (t + 1) % kCkpt == 0 and t + 1 < T, u to ckpt[(t + 1) / kCkpt - 1][C]
// and, for the current-based neuron, i to the same slot of a second plane
// nck chunks further.  The recurrent neuron (eq. 7) adds its own previous
// spike through the recurrent weight: a spike at t-1 adds (v - thr) to u_t
// instead of the plain reset -thr; column c is neuron c % N.
//
// Blocks of kCkpt steps run from NB register sets in turn, the loads of the
// block NB - 1 further issued before a block's steps.  A whole block has no
// branches (loads past T repeat the last row): vector memory operations
// complete in order and the compiler counts them, so a branch around a store
// makes it wait for every load and store in flight, once per block.  That wait
// bounded layers of few waves, which leave nothing to run meanwhile (1000 steps
// of 65536 columns: 113 -> 76 us).
template <int NEURON, int VEC, int OUT, int NB, bool UOUT>
__global__ __launch_bounds__(kThreads) void neuron_fwd_kernel(int T, int64_t C, int64_t N,
                                                              float alpha, float beta, float thr,
                                                              const float *__restrict__ vrec,
                                                              const float *cur, void *spk,
                                                              float *u_out,
                                                              float *__restrict__ ckpt,
                                                              float *__restrict__ counts) {
    constexpr int D = kCkpt;
    // packed-bit output with two columns per lane: the lane's columns are col
    // and col + 64 (see store_spikes_bits), else col and col + 1
    constexpr bool SPLIT = OUT == SNN_SPK_BITS && VEC == 2;
    constexpr int CS = SPLIT ? 64 : 1;  // column stride within a lane
    const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t col = SPLIT ? (gid >> 6) * 128 + (gid & 63) : gid * VEC;
    if (col >= C) return;
    auto ld = [&](const float *p, float (&v)[VEC]) {
        if constexpr (SPLIT) {
            v[0] = p[0];
            v[1] = p[64];
        } else {
            Vec<VEC>::load(p, v);
        }
    };
    auto st = [&](float *p, const float (&v)[VEC]) {
        if constexpr (SPLIT) {
            p[0] = v[0];
            p[64] = v[1];
        } else {
            Vec<VEC>::store(p, v);
        }
    };
    const int nck = (T - 1) / kCkpt;
    float u[VEC], syn[VEC], zp[VEC], cnt[VEC], jump[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        u[v] = syn[v] = zp[v] = cnt[v] = 0.f;
        if constexpr (NEURON == SNN_RLEAKY) jump[v] = vrec[(col + CS * v) % N] - thr;
        else jump[v] = -thr;
    }

    float in[NB][D][VEC];
    auto load = [&](int t0, float (&x)[D][VEC]) {
#pragma unroll
        for (int j = 0; j < D; ++j) ld(cur + (int64_t)min(t0 + j, T - 1) * C + col, x[j]);
    };
    auto step = [&](int t, const float (&x)[VEC]) {
        float z[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            const float uu = neuron_step<NEURON>(u[v], syn[v], zp[v], x[v], alpha, beta, jump[v]);
            z[v] = (uu > thr) ? 1.f : 0.f;  // eq. (3), strict
            zp[v] = z[v];
            cnt[v] += z[v];
        }
        const int64_t off = (int64_t)t * C + col;
        if constexpr (UOUT) st(u_out + off, u);
        if constexpr (OUT == SNN_U8)
            store_spikes_u8<VEC>(reinterpret_cast<uint8_t *>(spk) + off, z);
        else if constexpr (OUT == SNN_SPK_BITS)
            store_spikes_bits<VEC>(reinterpret_cast<uint64_t *>(spk), off - (threadIdx.x & 63), z);
        else
            store_spikes_f16<VEC>(reinterpret_cast<uint16_t *>(spk) + off, z);
    };
#pragma unroll
    for (int b = 0; b < (NB > 1 ? NB - 1 : 1); ++b) load(b * D, in[b]);
    for (int t0 = 0; t0 < T; t0 += NB * D) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int tb = t0 + b * D;
            if (tb + D <= T) {
                if constexpr (NB > 1) load(tb + (NB - 1) * D, in[(b + NB - 1) % NB]);
#pragma unroll
                for (int j = 0; j < D; ++j) step(tb + j, in[b][j]);
                if (tb + D < T) {
                    const int64_t slot = (int64_t)(tb / kCkpt) * C + col;
                    st(ckpt + slot, u);
                    if constexpr (NEURON == SNN_SYNAPTIC) st(ckpt + (int64_t)nck * C + slot, syn);
                }
            } else {
#pragma unroll
                for (int j = 0; j < D; ++j)
                    if (tb + j < T) step(tb + j, in[b][j]);
                t0 = T;
                break;
            }
        }
    }
    if (counts) st(counts + col, cnt);
}

// Bias gradient: db[f] = sum over b of the per-column time sums.  A block
// owns 64 consecutive features (one per lane); its 16 waves take every 16th
// batch row, each lane summing in fp64 in a fixed order, and the 16 partial
// sums are added in wave order.
__global__ __launch_bounds__(1024) void bias_reduce_kernel(int B, int F,
                                                           const float *__restrict__ colsum,
                                                           float *__restrict__ db) {
    __shared__ double part[16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int f = blockIdx.x * 64 + lane;
    double acc = 0.0;
    if (f < F) {
#pragma unroll 4
        for (int b = wave; b < B; b += 16) acc += (double)colsum[(int64_t)b * F + f];
    }
    part[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && f < F) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) s += part[w][lane];
        db[f] = (float)s;
    }
}

// The same sum for layers with P > 1 positions per feature (conv channels):
// one 1024-thread block per feature, fp64 partial sums over a fixed
// assignment of (b, p) to threads, then a fixed-order tree.
constexpr int kReduceThreads = 1024;
__global__ __launch_bounds__(kReduceThreads) void bias_reduce_pos_kernel(
    int B, int F, int P, const float *__restrict__ colsum, float *__restrict__ db) {
    __shared__ double part[kReduceThreads];
    const int f = blockIdx.x;
    const int64_t n = (int64_t)B * P;
    double acc = 0.0;
    for (int64_t j = threadIdx.x; j < n; j += kReduceThreads)
        acc += (double)colsum[((j / P) * F + f) * P + j % P];
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int w = kReduceThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) db[f] = (float)part[0];
}

// ---- the power-of-two scale of an fp16 dL/dI ------------------------------
// |lam_t| <= G F with G a bound on |g| and F = sum_k c^k the growth of the
// reverse recursion (computed by the caller from beta, alpha, thr and T), so
// dL/dI S with S = 2^e, e = floor(log2(2^15 / (G F))), stays below 2^15
// (fp16 holds up to 65504: a factor 2 of headroom for the fp32 rounding of
// the bound and the recursion).  G is a max over the upstream gradient:
//   FULL / BCAST  G = max |g|
//   FOLD          G = max_{t,b} sum_j |dup[t,b,j]|  *  max_{j,n} |wup[j,n]|
//                 (>= |sum_j dup[t,b,j] wup[j,n]| for every n)
// First pass: per-workgroup maxima (partial[2 blk], partial[2 blk + 1]);
// second pass, one workgroup: the maxima, G and S (written to scale[0]).
// Max is order-independent: the result is deterministic.
constexpr int kScaleBlocks = 1024;

__device__ inline float block_max(float v, float *red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) red[wave] = v;
    __syncthreads();
    float m = 0.f;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) m = fmaxf(m, red[w]);
    __syncthreads();
    return m;
}

__global__ __launch_bounds__(kThreads) void grad_bound_kernel(int64_t rows, int width, int dt,
                                                              const void *__restrict__ src,
                                                              int64_t nw, int dt_w,
                                                              const void *__restrict__ w,
                                                              float *__restrict__ partial) {
    __shared__ float red[kThreads / 64];
    // rows of `width` values of type dt: the max over rows of sum |x| (fp32
    // rows of one value, the gradient of every step or of a column, are read
    // 64 bytes per lane at a time: 26 MB in 11.7 us one value at a time; a
    // folded layer of one output may bring 16-bit ones)
    float m1 = 0.f;
    if (width == 1 && dt == SNN_F32) {
        const float4 *x4 = reinterpret_cast<const float4 *>(src);
        const int64_t n4 = rows / 4, step = (int64_t)gridDim.x * kThreads;
        int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
        auto take = [&](const float4 &v) {
            m1 = fmaxf(fmaxf(m1, fmaxf(__builtin_fabsf(v.x), __builtin_fabsf(v.y))),
                       fmaxf(__builtin_fabsf(v.z), __builtin_fabsf(v.w)));
        };
        for (; i + 3 * step < n4; i += 4 * step) {
            float4 v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = x4[i + q * step];
#pragma unroll
            for (int q = 0; q < 4; ++q) take(v[q]);
        }
        for (; i < n4; i += step) take(x4[i]);
        if (blockIdx.x == 0 && threadIdx.x < rows - 4 * n4)
            m1 = fmaxf(m1, __builtin_fabsf(reinterpret_cast<const float *>(src)[4 * n4 + threadIdx.x]));
        rows = 0;
    }
    for (int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x; r < rows;
         r += (int64_t)gridDim.x * kThreads) {
        float a = 0.f;
        for (int j = 0; j < width; ++j) a += __builtin_fabsf(load_as_f32(src, r * width + j, dt));
        m1 = fmaxf(m1, a);
    }
    float m2 = 0.f;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < nw;
         i += (int64_t)gridDim.x * kThreads)
        m2 = fmaxf(m2, __builtin_fabsf(load_as_f32(w, i, dt_w)));
    m1 = block_max(m1, red);
    m2 = block_max(m2, red);
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = m1;
        partial[2 * blockIdx.x + 1] = m2;
    }
}

__global__ __launch_bounds__(kThreads) void grad_scale_kernel(int nblk, bool product, double growth,
                                                              const float *__restrict__ partial,
                                                              float *__restrict__ scale) {
    __shared__ float red[kThreads / 64];
    float m1 = 0.f, m2 = 0.f;
    for (int i = threadIdx.x; i < nblk; i += kThreads) {
        m1 = fmaxf(m1, partial[2 * i]);
        m2 = fmaxf(m2, partial[2 * i + 1]);
    }
    m1 = block_max(m1, red);
    m2 = block_max(m2, red);
    if (threadIdx.x == 0) {
        const double G = product ? (double)m1 * (double)m2 : (double)m1;
        const double bound = G * growth;
        int e = 0;
        if (bound > 0.0 && bound < 1e300) {
            int ex;
            (void)frexp(32768.0 / bound, &ex);  // 32768 / bound in [2^(ex-1), 2^ex)
            e = ex - 1;
            if (e > 120) e = 120;
            if (e < -120) e = -120;
        }
        scale[0] = ldexpf(1.f, e);
    }
}

__global__ __launch_bounds__(kThreads) void fill_zero_kernel(float *__restrict__ p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) p[i] = 0.f;
}

struct FwdBuffers {
    const float *cur;
    void *spk;
    float *u_out, *ckpt, *counts;
};

template <int NEURON, int VEC, int OUT, int NB, bool UOUT>
void fwd_launch_nb(const ScanArgs &a, const FwdBuffers &b, hipStream_t s) {
    const int64_t lanes = (a.C + VEC - 1) / VEC;
    const unsigned grid = (unsigned)((lanes + kThreads - 1) / kThreads);
    neuron_fwd_kernel<NEURON, VEC, OUT, NB, UOUT><<<grid, kThreads, 0, s>>>(
        a.T, a.C, a.N, a.alpha, a.beta, a.thr, a.vrec, b.cur, b.spk, b.u_out, b.ckpt, b.counts);
}

// Blocks in registers: one for sequences of one block, else two (four measured
// slower: 27.0 against 23.3 us on 100 steps of 262144 columns, 16.6 against 14.3
// on 50 current-based steps of 256000).
template <int NEURON, int VEC, int OUT>
void fwd_launch(const ScanArgs &a, const FwdBuffers &b, hipStream_t s) {
    if (b.u_out) fwd_launch_nb<NEURON, VEC, OUT, 2, true>(a, b, s);
    else if (a.T <= kCkpt) fwd_launch_nb<NEURON, VEC, OUT, 1, false>(a, b, s);
    else fwd_launch_nb<NEURON, VEC, OUT, 2, false>(a, b, s);
}

template <int NEURON, int VEC>
void fwd_dispatch(int out_dtype, const ScanArgs &a, const FwdBuffers &b, hipStream_t s) {
    if (out_dtype == SNN_U8) fwd_launch<NEURON, VEC, SNN_U8>(a, b, s);
    else if (out_dtype == SNN_SPK_BITS) fwd_launch<NEURON, VEC, SNN_SPK_BITS>(a, b, s);
    else fwd_launch<NEURON, VEC, SNN_F16>(a, b, s);
}

}  // namespace

int64_t neuron_ckpt_count(int T) { return T > 0 ? (T - 1) / kCkpt : 0; }

hipError_t launch_neuron_fwd(int neuron, int T, int64_t C, int64_t N, float alpha, float beta,
                             float thr, const float *vrec, const float *cur, void *spk,
                             int out_dtype, float *u_out, float *ckpt, float *counts,
                             hipStream_t s) {
    if (T <= 0 || C <= 0) return hipSuccess;
    if (neuron_ckpt_count(T) > 0 && ckpt == nullptr) return hipErrorInvalidValue;
    // packed spikes: whole 64-bit words per wave (C a multiple of 64 * VEC)
    if (out_dtype == SNN_SPK_BITS && C % 64 != 0) return hipErrorInvalidValue;
    const bool v2 = (C % 2) == 0 && C >= kWideColumns && (out_dtype != SNN_SPK_BITS || C % 128 == 0);
    const ScanArgs a{T, C, N, alpha, beta, thr, 0.f, vrec};
    const FwdBuffers b{cur, spk, u_out, ckpt, counts};
    switch (neuron) {
        case SNN_SYNAPTIC:
            if (v2) fwd_dispatch<SNN_SYNAPTIC, 2>(out_dtype, a, b, s);
            else fwd_dispatch<SNN_SYNAPTIC, 1>(out_dtype, a, b, s);
            break;
        case SNN_RLEAKY:
            if (v2) fwd_dispatch<SNN_RLEAKY, 2>(out_dtype, a, b, s);
            else fwd_dispatch<SNN_RLEAKY, 1>(out_dtype, a, b, s);
            break;
        default:
            if (v2) fwd_dispatch<SNN_LEAKY, 2>(out_dtype, a, b, s);
            else fwd_dispatch<SNN_LEAKY, 1>(out_dtype, a, b, s);
    }
    return hipGetLastError();
}

bool neuron_fold_supported(int64_t N) { return N >= 64; }

hipError_t launch_neuron_bwd(int neuron, int reset_surrogate, int T, int64_t C, int64_t N,
                             float alpha, float beta, float thr, float slope, const float *vrec,
                             const float *cur, const float *ckpt, const BwdGrad &grad, int B,
                             void *dcur, void *dcur_t, bool dcur_t_planes, int grad_dtype,
                             const float *dscale, float *colsum, float *dvcol, hipStream_t s) {
    if (dcur == nullptr && dcur_t == nullptr) return hipErrorInvalidValue;
    if (dcur_t && dcur_t_planes && grad_dtype != SNN_F32) return hipErrorInvalidValue;
    if (grad_dtype == SNN_F16 && dscale == nullptr) return hipErrorInvalidValue;
    if (T <= 0 || C <= 0) return hipSuccess;
    if (neuron_ckpt_count(T) > 0 && ckpt == nullptr) return hipErrorInvalidValue;
    int gm = grad.mode == SNN_GRAD_FOLD ? GM_FOLD
             : grad.mode == SNN_GRAD_BCAST ? GM_BCAST : GM_FULL;
    if (gm == GM_FOLD && (!neuron_fold_supported(N) || grad.nup < 1 || grad.nup > kFoldMax))
        return hipErrorInvalidValue;
    if (gm == GM_FOLD && grad.nup <= 12) gm = GM_FOLD12;
    const bool wide = C >= kWideColumns;
    int vec = 1;
    if (gm == GM_FULL) {
        if (wide && C % 2 == 0) vec = 2;
    } else if (gm == GM_BCAST) {
        if (wide && C % 2 == 0) vec = 2;
    } else if (wide && N % 2 == 0 && N >= 128) {
        // a lane's two columns in one batch row, and the workgroup's 512
        // columns within kFoldRows batch rows
        vec = 2;
    }
    const ScanArgs a{T, C, N, alpha, beta, thr, slope, vrec};
    const FoldIn fold{grad.dup, grad.wup, grad.nup, grad.dt_up, grad.dt_w, B};
    const BwdBuffers b{cur,  ckpt, grad.g, fold, dcur, reinterpret_cast<uint16_t *>(dcur_t),
                       dcur_t_planes, dscale, colsum, dvcol};
    const int rs = reset_surrogate, gt = grad_dtype;
    switch (neuron) {
        case SNN_SYNAPTIC: scan_bwd_synaptic(vec, rs, gm, gt, a, b, s); break;
        case SNN_RLEAKY: scan_bwd_rleaky(vec, rs, gm, gt, a, b, s); break;
        default: scan_bwd_leaky(vec, rs, gm, gt, a, b, s);
    }
    return hipGetLastError();
}

hipError_t launch_fill_zero(float *p, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    fill_zero_kernel<<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(p, n);
    return hipGetLastError();
}

size_t grad_scale_workspace_bytes() { return 2 * kScaleBlocks * sizeof(float); }

hipError_t launch_grad_scale(int T, int64_t C, const BwdGrad &grad, int B, double growth,
                             float *scale, float *scratch, hipStream_t s) {
    int64_t rows, nw = 0;
    int width = 1, dt = SNN_F32, dt_w = SNN_F32;
    const void *src, *w = nullptr;
    if (grad.mode == SNN_GRAD_FOLD) {
        rows = (int64_t)T * B;
        width = grad.nup;
        dt = grad.dt_up;
        src = grad.dup;
        nw = B > 0 ? (int64_t)grad.nup * (C / B) : 0;  // (an empty batch: no bound)
        w = grad.wup;
        dt_w = grad.dt_w;
    } else {
        rows = grad.mode == SNN_GRAD_BCAST ? C : (int64_t)T * C;
        src = grad.g;
    }
    const int64_t work = rows * width > nw ? rows * width : nw;
    int nblk = (int)((work + 16 * kThreads - 1) / (16 * kThreads));
    if (nblk < 1) nblk = 1;
    if (nblk > kScaleBlocks) nblk = kScaleBlocks;
    grad_bound_kernel<<<nblk, kThreads, 0, s>>>(rows, width, dt, src, nw, dt_w, w, scratch);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    grad_scale_kernel<<<1, kThreads, 0, s>>>(nblk, grad.mode == SNN_GRAD_FOLD, growth, scratch,
                                             scale);
    return hipGetLastError();
}

int device_cus() {
    static std::atomic<int> cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int v = cache[dev].load(std::memory_order_relaxed);
    if (v == 0) {
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            v <= 0)
            v = 256;
        cache[dev].store(v, std::memory_order_relaxed);
    }
    return v;
}

hipError_t launch_bias_reduce(int B, int F, int P, const float *colsum, float *db, hipStream_t s) {
    if (F <= 0) return hipSuccess;
    if (P > 1) bias_reduce_pos_kernel<<<F, kReduceThreads, 0, s>>>(B, F, P, colsum, db);
    else bias_reduce_kernel<<<(F + 63) / 64, 1024, 0, s>>>(B, F, colsum, db);
    return hipGetLastError();
}

}  // namespace snn
