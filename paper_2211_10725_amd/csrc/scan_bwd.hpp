// The reverse time scan (its kernel and dispatch), shared by one source file per
// neuron model (scan_bwd_leaky.hip, scan_bwd_synaptic.hip, scan_bwd_rleaky.hip),
// whose instantiations compile side by side.  See scan.hip for the layout of the
// tensors and the saved state.
#pragma once

#include <type_traits>

#include "scan_common.hpp"

namespace snn {
namespace {

__device__ inline uint16_t f32_to_bf16_rne(float x) {
    const uint32_t b = __float_as_uint(x);
    return (uint16_t)((b + 0x7fffu + ((b >> 16) & 1u)) >> 16);
}

// dL/dI in the operand type of the contractions.  fp16 is written scaled by
// the power of two `scale` (exact), chosen per call so that every value
// stays below 2^15 (grad_scale_*_kernel below).
template <int GT, int VEC>
__device__ inline void store_grad(void *base, int64_t off, const float (&v)[VEC], float scale) {
    if constexpr (GT == SNN_F32) {
        Vec<VEC>::store(reinterpret_cast<float *>(base) + off, v);
    } else {
        uint16_t h[VEC];
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            if constexpr (GT == SNN_F16) {
                const _Float16 f = (_Float16)(v[i] * scale);
                h[i] = __builtin_bit_cast(uint16_t, f);
            } else {
                h[i] = f32_to_bf16_rne(v[i]);
            }
        }
        uint16_t *p = reinterpret_cast<uint16_t *>(base) + off;
        if constexpr (VEC == 2)
            *reinterpret_cast<uint32_t *>(p) = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
        else
            p[0] = h[0];
    }
}

// The 16-bit parts of dL/dI for the weight-gradient contraction: fp32 as
// three exact bf16 parts (hi = bf16(x), mid = bf16(x - hi), lo = bf16(x - hi
// - mid), each subtraction exact), bf16 or fp16 (scaled) as one.
__device__ inline uint32_t bf16_rne_bits(float x) { return f32_to_bf16_rne(x); }
template <int GT>
__device__ inline uint32_t grad_part(float x, int p, float scale) {
    if constexpr (GT == SNN_F16) {
        const _Float16 f = (_Float16)(x * scale);
        return __builtin_bit_cast(uint16_t, f);
    } else if constexpr (GT == SNN_BF16) {
        return bf16_rne_bits(x);
    } else {
        const uint32_t hi = bf16_rne_bits(x);
        if (p == 0) return hi;
        const float r = x - __uint_as_float(hi << 16);
        const uint32_t mid = bf16_rne_bits(r);
        if (p == 1) return mid;
        return bf16_rne_bits(r - __uint_as_float(mid << 16));
    }
}

// The layer above, for GM_FOLD.  A workgroup's 256 VEC consecutive columns
// span at most kFoldRows batch rows (the launcher only folds layers with
// n >= 64, and n >= 128 for VEC = 2); the dI_up rows of those batch rows for
// one chunk of kCkpt steps are staged in LDS (double-buffered, one barrier
// per chunk), the next chunk's loaded into registers while this one runs.
// Values of a runtime type are loaded raw, all of them under one branch on the
// type, and converted when they are used: a branch per value would wait for
// each load before the next.
__device__ inline float raw_to_f32(uint32_t r, int dt) {
    if (dt == SNN_F32) return __uint_as_float(r);
    if (dt == SNN_BF16) return __uint_as_float(r << 16);
    return (float)__builtin_bit_cast(_Float16, (uint16_t)r);
}

template <int KF>
struct FoldStage {
    static constexpr int ROWS = kFoldRows;
    static constexpr int kElems = kCkpt * ROWS * KF;
    static constexpr int kPer = (kElems + kThreads - 1) / kThreads;  // per thread
    uint32_t v[kPer];
    uint32_t in;  // bit i: value i exists (else it is 0)

    // the dI_up values of the steps t0 .. t0 + kCkpt - 1 of a chunk and batch
    // rows b_lo .. b_lo + ROWS - 1
    __device__ inline void load(const FoldIn &f, int T, int t0, int64_t b_lo) {
        int64_t o[kPer];
        in = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = threadIdx.x + i * kThreads;
            const int jt = e / (ROWS * KF), bb = (e / KF) % ROWS, j = e % KF;
            const int t = t0 + jt;
            const int64_t b = b_lo + bb;
            const bool ok = e < kElems && t < T && b < f.B && j < f.nup;
            o[i] = ok ? ((int64_t)t * f.B + b) * f.nup + j : 0;
            in |= ok ? 1u << i : 0u;
        }
        if (f.dt_up == SNN_F32) {
#pragma unroll
            for (int i = 0; i < kPer; ++i) v[i] = reinterpret_cast<const uint32_t *>(f.dup)[o[i]];
        } else {
#pragma unroll
            for (int i = 0; i < kPer; ++i) v[i] = reinterpret_cast<const uint16_t *>(f.dup)[o[i]];
        }
    }
    __device__ inline void store(float *rows, int dt) const {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = threadIdx.x + i * kThreads;
            const float x = raw_to_f32(v[i], dt);
            if (e < kElems) rows[e] = (in >> i) & 1u ? x : 0.f;
        }
    }
};

// Reverse-time scan over chunks of kCkpt steps, last chunk first.  For each
// chunk the lane loads its currents and the checkpoint before it, recomputes
// u_t forward in registers, then runs the adjoint backwards.  lam carries
// dL/du_{t+1} (and lami dL/di_{t+1}).  For the recurrent neuron the spike z_t
// reaches u_{t+1} through (v - r thr), so the carry is beta + (v - r thr) s_t,
// and the recurrent weight's gradient collects lam_{t+1} z_t per column (dvcol,
// fp32).
//
// A chunk's loads are issued while the chunk after it runs, into the other of
// two register sets.  The loads and stores of a whole chunk are free of
// branches (addresses clamped to rows that exist, the lanes past the last
// column repeating it, in the wave that has it): vector memory operations
// complete in order and the compiler counts them, so a branch around one makes
// it wait for all of them, stores included, once per chunk.  That wait bounded
// layers of few waves, which leave nothing to run meanwhile (1000 steps of 65536
// columns: 186 -> 105 us; 101 recurrent steps of 25641: 19.9 -> 13.0 us).
//
// With TR = TR_TRANSPOSED, dL/dI is also written as the weight gradient's
// operand: dcur_t [P][N][B*T] (P = 3 bf16 parts of fp32, else 1 plane of the
// 16-bit type, planes t_plane elements apart), row n holding column n of
// every sample, K index b*T + t.  A lane's column is one row there and a
// chunk's steps are consecutive in it, so each chunk's values are packed in
// registers as the reverse loop produces them and stored together.  With
// TR = TR_PLANES (fp32 only), dcur_t holds the three bf16 parts in dcur's own
// layout, [3][T][C], written at every step like dcur.  The row-major dcur
// may be skipped (nullptr) in both cases.
//
// dcur may be cur or g itself: the value stored in a row follows from the values
// loaded from it, a lane that repeats a column does both in the same instructions
// as its owner, and a wave without columns does neither.  (The pointers stay
// declared as if apart: without that, 1000 steps of 524288 columns take 1456
// instead of 1428 us.)
constexpr int TR_NONE = 0, TR_TRANSPOSED = 1, TR_PLANES = 2;
template <int NEURON, int VEC, int GM, bool RESET_SURR, int GT, int TRM>
__global__ __launch_bounds__(kThreads) void neuron_bwd_kernel(
    int T, int64_t C, int64_t N, float alpha, float beta, float thr, float slope,
    const float *__restrict__ vrec, const float *__restrict__ cur, const float *__restrict__ ckpt,
    const float *__restrict__ g, FoldIn fold, void *__restrict__ dcur,
    uint16_t *__restrict__ dcur_t, int64_t t_plane,
    const float *__restrict__ dscale, float *__restrict__ colsum, float *__restrict__ dvcol) {
    constexpr bool BCAST = GM == GM_BCAST, FOLD = GM == GM_FOLD || GM == GM_FOLD12;
    constexpr bool FULL = GM == GM_FULL;
    constexpr int K = kCkpt;
    constexpr int P = GT == SNN_F32 ? 3 : 1;  // 16-bit parts per value in dcur_t
    constexpr bool TR = TRM == TR_TRANSPOSED;
    uint32_t pk[TR ? P : 1][TR ? VEC : 1][TR ? K / 2 : 1];  // packed parts of a chunk
    const float scale = GT == SNN_F16 ? *dscale : 1.f;
    constexpr int KF = GM == GM_FOLD12 ? 12 : kFoldMax;  // dI_up values per row (padded)
    using Stage = FoldStage<KF>;
    const int64_t lane_col = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * VEC;
    // (lanes past the last column repeat it, stores included)
    const int64_t col = lane_col < C ? lane_col : C - VEC;
    const int nch = (T + K - 1) / K, nck = nch - 1;
    __shared__ __attribute__((aligned(16))) float frows[FOLD ? 2 : 1][FOLD ? Stage::kElems : 1];
    const int wave0 = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63);
    // (a wave without a column only stages the fold's rows, barrier for barrier as below;
    // out of line: a training step of 125-workgroup scans 94.7 -> 94.0 us, 93.5 without it)
    if (__builtin_expect(((int64_t)blockIdx.x * kThreads + wave0) * VEC >= C, 0)) {
        if constexpr (FOLD) {
            const int64_t lo = ((int64_t)blockIdx.x * kThreads * VEC) / N;
            Stage st;
            for (int c = nck + 1; c >= 0; --c) {
                st.load(fold, T, max(c - 1, 0) * K, lo);
                st.store(frows[(c + 1) & 1], fold.dt_up);
                __syncthreads();
            }
        }
        return;
    }
    float lam[VEC], lami[VEC], acc[VEC], gb[VEC], vr[VEC], dv[VEC], jump[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        lam[v] = lami[v] = acc[v] = gb[v] = dv[v] = 0.f;
        const float vv = NEURON == SNN_RLEAKY ? vrec[(col + v) % N] : 0.f;
        jump[v] = NEURON == SNN_RLEAKY ? vv - thr : -thr;
        vr[v] = NEURON == SNN_RLEAKY ? (RESET_SURR ? vv - thr : vv) : 0.f;
    }
    if constexpr (BCAST) Vec<VEC>::load(g + col, gb);

    // fold: the lane's columns of W_up, its batch row within the staged rows
    float wcol[FOLD ? VEC : 1][FOLD ? KF : 1];
    int fbb = 0;
    int64_t b_lo = 0;
    Stage fst;
    // chunk registers: currents (then the recomputed membrane), the full
    // upstream gradient and the checkpointed state at the start
    struct Chunk {
        float x[K][VEC], g[FULL ? K : 1][VEC], su[VEC], si[VEC];
    };
    Chunk c0, c1;
    // chunk c; for c < 0 one row that exists, K times
    auto load_chunk = [&](int c, Chunk &k) {
        if (c > 0) {
            Vec<VEC>::load(ckpt + (int64_t)(c - 1) * C + col, k.su);
            if constexpr (NEURON == SNN_SYNAPTIC)
                Vec<VEC>::load(ckpt + (int64_t)(nck + c - 1) * C + col, k.si);
        }
        const int t_lo = max(c, 0) * K, step = c < 0 ? 0 : 1;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int64_t o = (int64_t)min(t_lo + j * step, T - 1) * C + col;
            Vec<VEC>::load(cur + o, k.x[j]);
            if constexpr (FULL) Vec<VEC>::load(g + o, k.g[j]);
        }
    };
    // the first chunk's loads and the fold's are in flight together
    if constexpr (FOLD) {
        b_lo = ((int64_t)blockIdx.x * kThreads * VEC) / N;
        fst.load(fold, T, nck * K, b_lo);
    }
    load_chunk(nck, c0);
    if constexpr (FOLD) {
        fbb = (int)(col / N - b_lo);
        uint32_t wr[VEC][KF];
        const int64_t n0 = col % N;  // (a lane's columns lie in one batch row)
        if (fold.dt_w == SNN_F32) {
#pragma unroll
            for (int v = 0; v < VEC; ++v)
#pragma unroll
                for (int j = 0; j < KF; ++j)
                    wr[v][j] = reinterpret_cast<const uint32_t *>(
                        fold.wup)[(int64_t)min(j, fold.nup - 1) * N + n0 + v];
        } else {
#pragma unroll
            for (int v = 0; v < VEC; ++v)
#pragma unroll
                for (int j = 0; j < KF; ++j)
                    wr[v][j] = reinterpret_cast<const uint16_t *>(
                        fold.wup)[(int64_t)min(j, fold.nup - 1) * N + n0 + v];
        }
#pragma unroll
        for (int v = 0; v < VEC; ++v)
#pragma unroll
            for (int j = 0; j < KF; ++j)
                wcol[v][j] = j < fold.nup ? raw_to_f32(wr[v][j], fold.dt_w) : 0.f;
        fst.store(frows[nck & 1], fold.dt_up);
        __syncthreads();
    }

    // chunk c from k (its last steps may not exist when !WHOLE)
    auto run = [&](int c, Chunk &k, auto whole) {
        constexpr bool WHOLE = whole();
        const int t_lo = c * K;
        // recompute u_t of the chunk from the state before it (u_{t_lo-1},
        // i_{t_lo-1}; z_{t_lo-1} = [u_{t_lo-1} > thr]), in place of I_t
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            float u = c > 0 ? k.su[v] : 0.f;
            float syn = NEURON == SNN_SYNAPTIC && c > 0 ? k.si[v] : 0.f;
            float zp = (c > 0 && u > thr) ? 1.f : 0.f;
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const float uu = neuron_step<NEURON>(u, syn, zp, k.x[j][v], alpha, beta, jump[v]);
                k.x[j][v] = uu;  // (past T: never used)
                zp = (uu > thr) ? 1.f : 0.f;
            }
        }
        const float *fr = FOLD ? frows[c & 1] : nullptr;
        if constexpr (TR) {
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int v = 0; v < VEC; ++v)
#pragma unroll
                    for (int q = 0; q < K / 2; ++q) pk[p][v][q] = 0u;
        }
#pragma unroll
        for (int j = K - 1; j >= 0; --j) {
            const int t = t_lo + j;
            if (WHOLE || t < T) {
                float d[VEC];
                float grow[FOLD ? KF : 1];
                if constexpr (FOLD) {
                    const float4 *r4 = reinterpret_cast<const float4 *>(
                        fr + (j * kFoldRows + fbb) * KF);
#pragma unroll
                    for (int q = 0; q < KF / 4; ++q) {
                        const float4 x = r4[q];
                        grow[4 * q] = x.x; grow[4 * q + 1] = x.y;
                        grow[4 * q + 2] = x.z; grow[4 * q + 3] = x.w;
                    }
                }
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    const float uu = k.x[j][v];
                    const float s = surrogate(uu, thr, slope);
                    float gt;
                    if constexpr (BCAST) {
                        gt = gb[v];
                    } else if constexpr (FOLD) {
                        gt = 0.f;  // j ascending: the order of the short contraction
#pragma unroll
                        for (int q = 0; q < KF; ++q) gt = __builtin_fmaf(grow[q], wcol[v][q], gt);
                    } else {
                        gt = k.g[j][v];
                    }
                    if constexpr (NEURON == SNN_RLEAKY) {
                        if (uu > thr) dv[v] += lam[v];  // lam_{t+1} z_t
                        const float carry = __builtin_fmaf(vr[v], s, beta);
                        lam[v] = __builtin_fmaf(carry, lam[v], gt * s);
                        d[v] = lam[v];
                    } else {
                        d[v] = adjoint_step<NEURON, RESET_SURR>(lam[v], lami[v], gt, s, alpha,
                                                                beta, thr);
                    }
                    acc[v] += d[v];
                }
                if (TRM == TR_NONE || dcur)
                    store_grad<GT, VEC>(dcur, (int64_t)t * C + col, d, scale);
                if constexpr (TRM == TR_PLANES) {
                    uint32_t part[3][VEC];
#pragma unroll
                    for (int v = 0; v < VEC; ++v)
                        split_bf16x3(d[v], part[0][v], part[1][v], part[2][v]);
#pragma unroll
                    for (int p = 0; p < 3; ++p) {
                        uint16_t *q = dcur_t + p * t_plane + (int64_t)t * C + col;
                        if constexpr (VEC == 2)
                            *reinterpret_cast<uint32_t *>(q) = part[p][0] | (part[p][1] << 16);
                        else
                            q[0] = (uint16_t)part[p][0];
                    }
                }
                if constexpr (TR) {
#pragma unroll
                    for (int p = 0; p < P; ++p)
#pragma unroll
                        for (int v = 0; v < VEC; ++v) {
                            const uint32_t h = grad_part<GT>(d[v], p, scale);
                            pk[p][v][j / 2] |= (j & 1) ? h << 16 : h;
                        }
                }
            }
        }
        if constexpr (TR) {
            // the chunk's steps of this lane's columns, row (col + v) % N,
            // K index b*T + t
            const int len = WHOLE ? K : min(K, T - t_lo);
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                const int64_t n = (col + v) % N, b = (col + v) / N;
                const int64_t base = n * ((int64_t)T * (C / N)) + b * T + t_lo;
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    uint16_t *row = dcur_t + p * t_plane + base;
                    if (len == K && (T & 3) == 0) {
#pragma unroll
                        for (int q = 0; q < K / 4; ++q)
                            *reinterpret_cast<uint2 *>(row + 4 * q) =
                                make_uint2(pk[p][v][2 * q], pk[p][v][2 * q + 1]);
                    } else {
#pragma unroll
                        for (int jj = 0; jj < K; ++jj)
                            if (jj < len)
                                row[jj] = (uint16_t)(pk[p][v][jj / 2] >> (16 * (jj & 1)));
                    }
                }
            }
        }
    };
    // Chunk c from k while chunk c - 1 loads into next (below 0: nothing of
    // use); the fold's rows of chunk c - 1 go to LDS after it (their buffer was
    // last read before the previous barrier)
    auto advance = [&](int c, Chunk &k, Chunk &next, auto whole) {
        if constexpr (FOLD) fst.load(fold, T, max(c - 1, 0) * K, b_lo);
        load_chunk(c - 1, next);
        run(c, k, whole);
        if constexpr (FOLD) {
            fst.store(frows[(c + 1) & 1], fold.dt_up);
            __syncthreads();
        }
    };
    advance(nck, c0, c1, std::false_type{});
    for (int c = nck - 1; c >= 0; c -= 2) {
        advance(c, c1, c0, std::true_type{});
        if (c == 0) break;
        advance(c - 1, c0, c1, std::true_type{});
    }
    if (colsum) Vec<VEC>::store(colsum + col, acc);
    if constexpr (NEURON == SNN_RLEAKY)
        if (dvcol) Vec<VEC>::store(dvcol + col, dv);
}


template <int NEURON, int VEC, int GM, bool RS, int GT>
void bwd_launch(const ScanArgs &a, const BwdBuffers &b, hipStream_t s) {
    const int64_t lanes = (a.C + VEC - 1) / VEC;
    const unsigned grid = (unsigned)((lanes + kThreads - 1) / kThreads);
    const int64_t t_plane = (int64_t)a.T * a.C;
    if (b.dcur_t && b.planes) {
        if constexpr (GT == SNN_F32)
            neuron_bwd_kernel<NEURON, VEC, GM, RS, GT, TR_PLANES><<<grid, kThreads, 0, s>>>(
                a.T, a.C, a.N, a.alpha, a.beta, a.thr, a.slope, a.vrec, b.cur, b.ckpt, b.g,
                b.fold, b.dcur, b.dcur_t, t_plane, b.dscale, b.colsum, b.dvcol);
    } else if (b.dcur_t) {
        neuron_bwd_kernel<NEURON, VEC, GM, RS, GT, TR_TRANSPOSED><<<grid, kThreads, 0, s>>>(
            a.T, a.C, a.N, a.alpha, a.beta, a.thr, a.slope, a.vrec, b.cur, b.ckpt, b.g, b.fold,
            b.dcur, b.dcur_t, t_plane, b.dscale, b.colsum, b.dvcol);
    } else {
        neuron_bwd_kernel<NEURON, VEC, GM, RS, GT, TR_NONE><<<grid, kThreads, 0, s>>>(
            a.T, a.C, a.N, a.alpha, a.beta, a.thr, a.slope, a.vrec, b.cur, b.ckpt, b.g, b.fold,
            b.dcur, nullptr, 0, b.dscale, b.colsum, b.dvcol);
    }
}

template <int NEURON, int VEC, int GM, bool RS>
void bwd_dispatch_gt(int gt, const ScanArgs &a, const BwdBuffers &b, hipStream_t s) {
    if (gt == SNN_F32) bwd_launch<NEURON, VEC, GM, RS, SNN_F32>(a, b, s);
    else if (gt == SNN_F16) bwd_launch<NEURON, VEC, GM, RS, SNN_F16>(a, b, s);
    else bwd_launch<NEURON, VEC, GM, RS, SNN_BF16>(a, b, s);
}

template <int NEURON, int VEC, int GM>
void bwd_dispatch_rs(int rs, int gt, const ScanArgs &a, const BwdBuffers &b, hipStream_t s) {
    if (rs) bwd_dispatch_gt<NEURON, VEC, GM, true>(gt, a, b, s);
    else bwd_dispatch_gt<NEURON, VEC, GM, false>(gt, a, b, s);
}

// Lane widths: two columns for layers of at least kWideColumns columns
// (measured on the 65536 x 64-column layer: 7.0 against 7.4 ms for four
// columns per lane, whose chunk registers left two waves per SIMD), else one.
template <int NEURON>
void bwd_dispatch(int vec, int rs, int gm, int gt, const ScanArgs &a, const BwdBuffers &b,
                  hipStream_t s) {
    if (gm == GM_BCAST) {
        if (vec == 2) bwd_dispatch_rs<NEURON, 2, GM_BCAST>(rs, gt, a, b, s);
        else bwd_dispatch_rs<NEURON, 1, GM_BCAST>(rs, gt, a, b, s);
    } else if (gm == GM_FOLD12) {
        if (vec == 2) bwd_dispatch_rs<NEURON, 2, GM_FOLD12>(rs, gt, a, b, s);
        else bwd_dispatch_rs<NEURON, 1, GM_FOLD12>(rs, gt, a, b, s);
    } else if (gm == GM_FOLD) {
        if (vec == 2) bwd_dispatch_rs<NEURON, 2, GM_FOLD>(rs, gt, a, b, s);
        else bwd_dispatch_rs<NEURON, 1, GM_FOLD>(rs, gt, a, b, s);
    } else {
        if (vec == 2) bwd_dispatch_rs<NEURON, 2, GM_FULL>(rs, gt, a, b, s);
        else bwd_dispatch_rs<NEURON, 1, GM_FULL>(rs, gt, a, b, s);
    }
}

}  // namespace
}  // namespace snn
