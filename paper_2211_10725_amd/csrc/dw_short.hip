// Weight gradients of small fp32 layers,
//
//   C[M,N] = sum_k A[k][m] B[k][n],   A fp32 (dL/dI), B spike bytes,
//
// both in their own row-major layouts, on the 16-bit matrix cores: a value of
// A as its three exact bf16 parts, the smallest first, fp32 accumulation.
//
// What bounds these products (well below a G multiply-adds) is latency: staged
// through LDS, k-tile after k-tile behind barriers, 64 .. 280 workgroups of the
// 16-bit kernel took 16 .. 27 us for work of 2.  Here no operand passes through
// LDS: lane (r, h) of a fragment loads its 8 values k = 8 h .. 8 h + 7 of row r
// straight from the k-rows (32 lanes read 128 consecutive bytes of A), so the
// loads of two k16 steps are in flight per wave without a barrier.  Small
// tiles (32 x 64) give enough workgroups, and the four waves of one take a
// quarter of K each and add their sums in LDS, in order, instead of in a
// second launch.  The price, every A value split by N / 64 workgroups, is
// below 5 us of vector work at the largest size taken.
// The call, 128 x 500 x 1000 (rows, outputs, inputs) 17.5 -> 9.4 us (on inputs
// out of the caches 21.1 -> 8.2), 800 x 1000 x 784 32.9 -> 22.8 (31.7 -> 26.1),
// 512 x 1000 x 1000 30.2 -> 15.1.  Layers: 300 rows of 3000 to 1000 130 -> 116,
// 800 of 1000 to 1000 125 -> 104.
#include "snn_internal.hpp"

namespace snn {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kTM = 32, kTN = 64;

__device__ inline floatx16 mfma32(const u32x4 &a, const u32x4 &b, const floatx16 &c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// the values of one k16 step as loaded
struct Raw {
    float a[8];
    uint8_t b[2][8];
};

__global__ __launch_bounds__(kThreads) void dw_short_kernel(int M, int N, int K, int tiles_n,
                                                            const float *__restrict__ A, int lda,
                                                            const uint8_t *__restrict__ B, int ldb,
                                                            float *__restrict__ C, int64_t ldc) {
    __shared__ float red[4][2][16][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
    const int m0 = blockIdx.x / tiles_n * kTM, n0 = blockIdx.x % tiles_n * kTN;
    const int am = min(m0 + r, M - 1), b0 = min(n0 + r, N - 1), b1 = min(n0 + 32 + r, N - 1);
    const int nk = (K + 15) / 16, per = (nk + 3) / 4;
    const int s0 = wave * per, s1 = min(nk, s0 + per), kend = min(K, s1 * 16);

    // clamped addresses: a step past the wave's share is multiplied as zeros
    auto load = [&](Raw &w, int s) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = min(16 * s + 8 * h + e, K - 1);
            w.a[e] = A[k * lda + am];
            w.b[0][e] = B[k * ldb + b0];
            w.b[1][e] = B[k * ldb + b1];
        }
    };
    floatx16 acc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[j][i] = 0.f;
    auto multiply = [&](const Raw &w, int s) {
        uint32_t p[3][8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            split_bf16x3(16 * s + 8 * h + e < kend ? w.a[e] : 0.f, p[0][e], p[1][e], p[2][e]);
        u32x4 bf[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int d = 0; d < 4; ++d)
                bf[j][d] = __float_as_uint((float)w.b[j][2 * d]) >> 16 |
                           (__float_as_uint((float)w.b[j][2 * d + 1]) & 0xffff0000u);
#pragma unroll
        for (int q = 2; q >= 0; --q) {
            u32x4 a;
#pragma unroll
            for (int d = 0; d < 4; ++d) a[d] = p[q][2 * d] | (p[q][2 * d + 1] << 16);
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[j] = mfma32(a, bf[j], acc[j]);
        }
    };
    Raw x, y;
    load(x, s0);
    load(y, s0 + 1);
    for (int s = s0; s < s1; s += 2) {
        multiply(x, s);
        load(x, s + 2);
        multiply(y, s + 1);
        load(y, s + 3);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) red[wave][j][i][lane] = acc[j][i];
    __syncthreads();
    // wave w adds registers 8 (w & 1) .. + 7 of half w / 2
    const int j = wave >> 1, n = n0 + 32 * j + r;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int i = 8 * (wave & 1) + q;
        const float v = ((red[0][j][i][lane] + red[1][j][i][lane]) + red[2][j][i][lane]) +
                        red[3][j][i][lane];
        const int m = m0 + 8 * (i >> 2) + 4 * h + (i & 3);
        if (m < M && n < N) C[(int64_t)m * ldc + n] = v;
    }
}

}  // namespace

bool dw_short_applies(const GemmArgs &g) {
    if (!g.allow_split || g.a_kc || g.b_kc || g.bias || g.c_div || g.pool_hw > 0) return false;
    if (g.a_dtype != SNN_F32 || g.b_dtype != SNN_U8 || g.M < 64 || g.N < 64) return false;
    if ((int64_t)g.K * g.lda >= (int64_t)1 << 31 || (int64_t)g.K * g.ldb >= (int64_t)1 << 31)
        return false;
    // A wave goes through a quarter of K: at 2500 rows of 784 x 100 the 16-bit
    // kernel's split of K wins (95 against 108 us for the step), at 25600 of
    // 64 x 64 by far; at 8 rows of 3000 x 3000 (77 against 86 us) the tiles'
    // sums and stores outweigh the product.
    if (g.K < 64 || g.K > 1024) return false;
    // The 16-bit kernel is at its best with rows of B of whole 16 bytes.  There it
    // splits outputs of at most 65536 elements over K further (1024 rows of 256 x
    // 256 16.5 against 17.8 us, 800 rows 17.1 against 16.0).
    const bool whole = g.ldb % 16 == 0;
    if (whole && g.K > 896 && (int64_t)g.M * g.N <= 65536) return false;
    // From 1024 tiles on (four workgroups per compute unit), splitting A once per
    // 64 columns costs more than the barriers over few rows (64 of 2000 x 2000,
    // 2016 tiles, 13.7 against 21.1 us; of 1500 x 1500 14.2 against 15.2), over
    // more rows where the 16-bit kernel is at its best and from 1280 tiles (200
    // rows of 2000 x 1000, 1024 tiles, 20.3 against 17.1; of 3072 x 1000, 1536,
    // 23.0 against 23.5; of 2000 x 2000 24.0 against 29.6), else nowhere (100 rows
    // of 3000 x 3000, 4418 tiles, 44.9 against 39.9).
    const int64_t tiles = (int64_t)((g.M + kTM - 1) / kTM) * ((g.N + kTN - 1) / kTN);
    if (tiles >= 1024 && (g.K < 96 || (whole && tiles >= 1280))) return false;
    // (above, the joint kernel takes the rest)
    return (double)g.M * g.N * g.K < 1073741824.0;
}

hipError_t launch_dw_short(const GemmArgs &g, hipStream_t s) {
    const int tiles_m = (g.M + kTM - 1) / kTM, tiles_n = (g.N + kTN - 1) / kTN;
    dw_short_kernel<<<(unsigned)(tiles_m * tiles_n), kThreads, 0, s>>>(
        g.M, g.N, g.K, tiles_n, reinterpret_cast<const float *>(g.A), (int)g.lda,
        reinterpret_cast<const uint8_t *>(g.B), (int)g.ldb, g.C, g.ldc);
    return hipGetLastError();
}

}  // namespace snn
