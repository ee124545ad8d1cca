// Contractions on the 16-bit matrix cores whose operand parts are staged
// together:
//
//   C[M,N] = sum_k A(m,k) B(n,k) (/ c_div) (+ bias[n]),  fp32 accumulate,
//
// each operand one 16-bit part (spikes, fp16 or bf16 values) or an fp32 array
// as its three exact bf16 parts (hi, mid, lo).  Three shapes of product:
//
//  * one part by one part (the fp16 network's mid-size products);
//  * spikes by three parts (currents and weight gradients of fp32 layers):
//    three passes, every product exact;
//  * three parts by three parts (the input gradient dL/dI W of an fp32
//    layer): six of the nine part products, smallest first: lo hi, mid mid,
//    hi lo, mid hi, hi mid, hi hi.  |mid| <= 2^-9 |x| and |lo| <= 2^-18 |x|,
//    so the three left out are below 2^-26 of |a b|, a quarter of an fp32
//    rounding.  Six bf16 passes cost 6/16 of the fp32 MFMA's time.
//
// What bounds them: the matrix cores under the card's power limit (with no
// copies at all the 51200 x 4096 x 4096 product runs at 1.23 PF), then the
// copies from L2 into LDS (a fifth of the time); the LDS reads cost nothing
// measurable.  So all parts of a k-tile are staged at once: a spike tile is
// copied once for three MFMAs per fragment, and every copy instruction should
// touch whole 128-byte lines: operands that are rewritten anyway go in
// fragment order, 1 KiB of consecutive memory per copy.  Measured, stage calls
// with their rewriting and reductions (before: the 16-bit kernel, the 256 x 256
// kernel with its planes in turn, or fp32 MFMA), rows x inputs x outputs:
//    6400 x 1000 x 1000  fp32 forward 84 -> 63, dW 85 -> 70, dx 181 -> 106 us
//    2013 x 1003 x 1101  fp32 forward 95 -> 37, dW 65 -> 39, dx  88 ->  52 us
//    5000 x  700 x 1500  fp32 forward 150 -> 42, dW 107 -> 61, dx 147 -> 86 us
//    6400 x 1000 x 1000  fp16 forward 39 -> 27, dW 46 -> 32, dx  45 ->  27 us
//    2013 x 1003 x 1101  fp16 forward 91 -> 30, dW 102 -> 48, dx 133 -> 31 us
//
// A workgroup copies k-tiles of KT straight from global memory into a ring of
// LDS slots (global_load_lds_dwordx4: lane i of a wave writes the 16 bytes at
// M0 + 16 i), the next tiles in flight while the current one is multiplied.
// Operands are K-contiguous ([row][k], row stride ld) or M/N-contiguous
// ([k][row], read with transposing LDS loads).  The workgroups are persistent.
//
// Operands that the copies cannot take (spike bytes, fp32 arrays, rows that
// do not start on 16 bytes or are not whole 16-byte chunks) are rewritten
// into the workspace by one launch for both (pack_kernel), rows padded with
// zeros to a multiple of 8 values.
#include <type_traits>

#include "snn_internal.hpp"

namespace snn {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void lds_void;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int MT_BF16 = 0, MT_F16 = 1;
constexpr int kGroupM = 4;  // tile rows per group of the tile order

template <int MT>
__device__ inline floatx16 mfma32(const u32x4 &a, const u32x4 &b, const floatx16 &c) {
    if constexpr (MT == MT_F16)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, a),
                                                      __builtin_bit_cast(half8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ inline uint32_t lds_addr(const void *p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}

// Fragment reads are asm so that the compiler's wait insertion does not hold
// them back for the copies in flight into the other stage; wait_frags names
// every fragment before its first use.
template <int OFF>
__device__ inline void lds_read(u32x4 &v, uint32_t addr) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
}
template <int OFF>
__device__ inline void lds_read_tr(u32x2 &v, uint32_t addr) {
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
}

// Chunk swizzles: 16-byte chunk c of row r (K-contiguous) or of k-row k
// (M/N-contiguous) lies at slot c ^ swz.  K-contiguous rows of 64 bytes (KT =
// 32): 8 consecutive rows of one chunk fall on 8 distinct 16-byte groups of a
// 128-byte line and 16 on the 16 of a 256-byte line; rows of 128 bytes
// likewise.  M/N-contiguous: the 4 k-rows a transposing read's 16 lanes
// address fall on distinct banks.
template <int KT>
__device__ inline int kc_swz(int r) {
    if constexpr (KT == 32) return (((r >> 1) ^ (r >> 3)) & 1) | (((r >> 2) & 1) << 1);
    else return ((r >> 1) & 7) ^ ((r & 1) << 2);
}
__device__ inline int mn_swz(int k) { return 2 * ((k & 3) | ((k & 1) << 2)); }

// The part products of a k16 step, smallest first.  Three parts by spikes (a
// weight gradient) keep two sums, lo and mid in one, hi in the other, added at
// the end: the hi products are 8-bit numbers whose sums are mostly exact in
// fp32, while adding all three parts into one sum rounds three times per step
// at full magnitude (2.4e-7 against 4.6e-8 of the result's rms over K = 784).
// The currents (spikes by three parts) keep one sum: see sum_order().
template <int PA, int PB>
struct Products {
    static constexpr int kCount = PA * PB == 9 ? 6 : PA * PB;
    static constexpr int kSums = PA == 3 && PB == 1 ? 2 : 1;
    static constexpr int a(int q) {
        if (PA * PB == 9) {
            constexpr int t[6] = {2, 1, 0, 1, 0, 0};
            return t[q];
        }
        return PA == 3 ? 2 - q : 0;
    }
    static constexpr int b(int q) {
        if (PA * PB == 9) {
            constexpr int t[6] = {0, 1, 2, 0, 1, 0};
            return t[q];
        }
        return PB == 3 ? 2 - q : 0;
    }
    static constexpr int sum(int q) { return kSums == 2 && q < 2 ? 1 : 0; }
};

// Operand layouts in global memory
enum : int {
    L_KC = 0,  // [row][k], K-contiguous
    L_MN = 1,  // [k][row], M/N-contiguous
    L_PK = 2,  // fragment order: [row / 32][k / 16] blocks of 64 lanes x 8 values, lane l
               // holding row l % 32, k 8 (l / 32) .. + 7 of the block
};

// One operand's tile of ROWS rows x KT k as the waves copy it.  `rows` rows
// exist; a K-contiguous row has `cols` readable values (a multiple of 8), an
// M/N-contiguous k-row `cols` readable rows (likewise).  A fragment-ordered
// operand has whole blocks, ld elements per 32 rows.
template <int L, int ROWS, int KT, int NW>
struct Tile {
    static constexpr int kPlane = ROWS * KT * 2;        // bytes per part and stage
    static constexpr int kBlocks = kPlane / 1024;       // 1 KiB copies per part
    static constexpr int kPer = kBlocks / NW;           // per wave
    static_assert(kBlocks % NW == 0, "whole copies per wave");
    static constexpr int kRowsPerBlock = L == L_MN ? 1024 / (ROWS * 2) : 1024 / (KT * 2);
    static constexpr int kChunksPerRow = L == L_MN ? ROWS / 8 : KT / 8;
    uint32_t off[L == L_MN ? 1 : kPer];  // element offsets of this lane's rows or blocks
    int sub;  // chunk offset within the row (K-contiguous) or row offset (M/N-contiguous)
    int kr;   // first k-row of this lane's copies (M/N-contiguous)

    __device__ inline void init(uint32_t ld, int rows, int cols, int r0) {
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        const int in = lane / kChunksPerRow, slot = lane % kChunksPerRow;
        if constexpr (L == L_MN) {
            kr = w * kRowsPerBlock + in;  // k mod 4 is the same for all of a lane's copies
            sub = min(r0 + 8 * (slot ^ mn_swz(kr)), cols - 8);
        } else if constexpr (L == L_KC) {
            const int r = w * kRowsPerBlock + in;
            sub = 8 * (slot ^ kc_swz<KT>(r));
#pragma unroll
            for (int i = 0; i < kPer; ++i)
                off[i] = (uint32_t)min(r0 + r + i * NW * kRowsPerBlock, rows - 1) * ld;
        } else {
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int b = w + i * NW, rb = min(r0 / 32 + b / (KT / 16), (rows + 31) / 32 - 1);
                off[i] = (uint32_t)rb * ld + (b % (KT / 16)) * 512 + lane * 8;
            }
        }
    }
    // the k-tile at k0 of one part into its place in a stage
    __device__ inline void copy(const uint16_t *X, uint32_t ld, int cols, int K, int k0,
                                char *stage) const {
        const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int k = k0 + sub;
        const uint32_t koff = L == L_PK ? (uint32_t)k0 * 32 : k < cols ? (uint32_t)k : 0u;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            uint32_t o;
            if constexpr (L == L_MN)
                o = (uint32_t)min(k0 + kr + i * NW * kRowsPerBlock, K - 1) * ld + (uint32_t)sub;
            else
                o = off[i] + koff;
            __builtin_amdgcn_global_load_lds(X + o, (lds_void *)(stage + (w + i * NW) * 1024), 16,
                                             0, 0);
        }
    }
};

// The wave's fragments of one operand: F blocks of 32 rows from row w0 of P
// parts, two register sets (k16 step s uses set s & 1).
template <int L, int P, int F, int ROWS, int KT>
struct Frags {
    static constexpr bool MN = L == L_MN;
    static constexpr int kPlane = ROWS * KT * 2;
    static constexpr int kReads = P * F;
    static constexpr int kBases = MN ? F : L == L_KC ? KT / 16 : 1;
    uint32_t base[kBases];  // LDS byte addresses within slot 0
    u32x2 h[MN ? 2 : 1][P][F][2];
    u32x4 q[2][P][F];

    __device__ inline void init(const char *op, int w0) {
        const int lane = threadIdx.x & 63;
        const uint32_t a = lds_addr(op);
        if constexpr (MN) {
            // lane L of 16-lane group g points at k-row 8 (g / 2) + L / 4 and
            // rows 16 (g & 1) + 4 (L % 4) of the block: lane i of the group
            // receives 4 consecutive k of row 16 (g & 1) + i
            const int g = lane >> 4, ll = lane & 15, k = 8 * (g >> 1) + (ll >> 2);
#pragma unroll
            for (int i = 0; i < F; ++i) {
                const int r = w0 + 32 * i + 16 * (g & 1) + 4 * (ll & 3);
                base[i] = a + (k * ROWS + (((r >> 3) ^ mn_swz(k)) * 8 + (r & 7))) * 2;
            }
        } else if constexpr (L == L_KC) {
            const int r = w0 + (lane & 31);
#pragma unroll
            for (int s = 0; s < KT / 16; ++s)
                base[s] = a + r * KT * 2 + ((2 * s + (lane >> 5)) ^ kc_swz<KT>(r)) * 16;
        } else {
            base[0] = a + (w0 / 32) * KT * 64 + lane * 16;
        }
    }
    // issue read number N of k16 step S from the slot at byte offset d
    template <int S, int N>
    __device__ inline void read(uint32_t d) {
        constexpr int p = N / F, i = N % F;
        if constexpr (MN) {
            lds_read_tr<p * kPlane + S * 16 * ROWS * 2>(h[S & 1][p][i][0], base[i] + d);
            lds_read_tr<p * kPlane + (S * 16 + 4) * ROWS * 2>(h[S & 1][p][i][1], base[i] + d);
        } else if constexpr (L == L_KC) {
            lds_read<p * kPlane + i * 32 * KT * 2>(q[S & 1][p][i], base[S] + d);
        } else {
            lds_read<p * kPlane + (i * (KT / 16) + S) * 1024>(q[S & 1][p][i], base[0] + d);
        }
    }
    // after the wait: name the fragments of step S; zero the values at or
    // past kvalid (of the k-tile's KT) of a last, partial tile (a
    // fragment-ordered operand holds zeros there)
    template <int S>
    __device__ inline void ready(int kvalid) {
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int i = 0; i < F; ++i) {
                if constexpr (MN) {
                    asm volatile("" : "+v"(h[S & 1][p][i][0]), "+v"(h[S & 1][p][i][1]));
                    q[S & 1][p][i] = __builtin_shufflevector(h[S & 1][p][i][0],
                                                             h[S & 1][p][i][1], 0, 1, 2, 3);
                } else {
                    asm volatile("" : "+v"(q[S & 1][p][i]));
                }
            }
        if (L != L_PK && kvalid < KT) {
            const int kb = 16 * S + 8 * ((threadIdx.x & 63) >> 5);
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const uint32_t m = (kb + 2 * d < kvalid ? 0xffffu : 0u) |
                                   (kb + 2 * d + 1 < kvalid ? 0xffff0000u : 0u);
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int i = 0; i < F; ++i) q[S & 1][p][i][d] &= m;
            }
        }
    }
};

template <int I, int N, typename Fn>
__device__ inline void static_for(const Fn &f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

struct JointArgs {
    int M, N, K, k_chunk, tiles_n, tiles, total;
    int sum_chunk;  // FOLD: K is summed in chunks of this length, added in order
    const uint16_t *A, *B;
    int64_t lda, ldb, a_ps, b_ps;
    int a_cols, b_cols;
    float *C;
    int64_t ldc, split_stride;
    const float *bias, *c_div;
};

// Work item j of persistent workgroup w of G: the items are cut into kXcds
// contiguous ranges, one per XCD (workgroup w runs on XCD w % kXcds), taken
// in turn by that XCD's workgroups.
__device__ inline int persistent_item(int w, int G, int total, int j) {
    const int xcd = w % kXcds, lw = w / kXcds;
    const int gx = G / kXcds + (xcd < G % kXcds ? 1 : 0);
    const int per = total / kXcds, rem = total % kXcds;
    const int beg = xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per;
    const int cnt = per + (xcd < rem ? 1 : 0);
    const int k = lw + j * gx;
    return k < cnt ? beg + k : -1;
}

struct Item {
    int m0, n0, zk, kbeg, kend;
};
// Tiles in groups of kGroupM tile rows, column by column within a group: the
// tiles an XCD holds at once share operand panels in its L2.
template <int BM, int BN>
__device__ inline Item locate(const JointArgs &g, int it) {
    Item r;
    r.zk = it / g.tiles;
    const int tile = it % g.tiles;
    const int grp = tile / (kGroupM * g.tiles_n), first = grp * kGroupM;
    const int gm = min(kGroupM, g.tiles / g.tiles_n - first), local = tile % (kGroupM * g.tiles_n);
    r.m0 = (first + local % gm) * BM;
    r.n0 = (local / gm) * BN;
    r.kbeg = r.zk * g.k_chunk;
    r.kend = min(g.K, r.kbeg + g.k_chunk);
    return r;
}

// A 32 x 32 block of the product from the whole fp32 values of its operands'
// parts (exact: hi + mid is, and adding lo gives the value back), A [row][k] and B
// [k][row], on the fp32 matrix cores.  m, n: the lane's row and column
// (clamped to ones that exist); lane half h takes k 8 h .. + 7 of each 16.
__device__ inline float part_f32(uint32_t h) { return __uint_as_float(h << 16); }
__device__ inline floatx16 whole_block(const uint16_t *A, int64_t lda,
                                                          int64_t a_ps, const uint16_t *B,
                                                          int64_t ldb, int64_t b_ps, int m, int n,
                                                          int kbeg, int kend) {
    const int h8 = 8 * ((threadIdx.x & 63) >> 5);
    floatx16 t;
#pragma unroll
    for (int r = 0; r < 16; ++r) t[r] = 0.f;
#pragma unroll 1
    for (int k0 = kbeg; k0 < kend; k0 += 16) {
        // (rows of A hold whole 16-byte chunks, k0 is a multiple of 16)
        const int k = k0 + h8;
        const uint16_t *a = A + (int64_t)m * lda + (k < kend ? k : 0);
        u32x4 w[3];
        uint32_t b[3][8];
#pragma unroll
        for (int p = 0; p < 3; ++p) w[p] = *reinterpret_cast<const u32x4 *>(a + p * a_ps);
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int p = 0; p < 3; ++p) b[p][e] = B[p * b_ps + (int64_t)min(k + e, kend - 1) * ldb + n];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float x = 0.f, y = 0.f;
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                x += part_f32((w[p][e / 2] >> (16 * (e & 1))) & 0xffffu);
                y += part_f32(b[p][e]);
            }
            const bool in = k + e < kend;
            t = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? x : 0.f, in ? y : 0.f, t, 0, 0, 0);
        }
    }
    return t;
}

// two waves per SIMD: one workgroup of 8 waves, or two of 4 where their rings
// fit a compute unit's LDS
template <int PA, int PB, int BM, int BN, int KT, int R, int NW>
constexpr int waves_per_simd() {
    return NW == 8 || R * (PA * BM + PB * BN) * KT * 2 <= 76 * 1024 ? 2 : 1;
}

// NP = 3: B's parts are taken in turn, all k-tiles of a chunk with lo, then
// with mid, then with hi.  FOLD: the sum over each chunk of K starts from
// zero and is added to the total (the order of a split K whose partials are
// added in turn, without writing the partials).
//
// The k-tiles of a workgroup's items, item after item, run through a ring of
// R LDS slots; step t multiplies the tile in slot t % R.  With R = 3, at the
// barrier that opens a step every wave has finished reading slot (t - 1) % R
// and tile t + 1 has landed in every wave's view: the step issues the copies
// of tile t + 2 into the slot just freed, and its last k16 step already
// reads tile t + 1's first fragments, so the matrix cores do not wait for
// LDS reads across the barrier.  With R = 2 the barrier only gives tile t,
// and the step copies tile t + 1.  The next item's first tiles are copied by
// the current item's last steps and are in flight during its stores.
template <int MT, int PA, int PB, int LA, int LB, int BM, int BN, int KT, int R, int WM, int WN,
          int NP, bool FOLD>
__global__ __launch_bounds__(64 * WM * WN, (waves_per_simd<PA, PB, BM, BN, KT, R, WM * WN>()))
void gemm_joint_kernel(JointArgs g) {
    constexpr int NW = WM * WN;
    static_assert(R == 2 || R == 3, "the waits below");
    constexpr bool kCross = R == 3;
    using PR = Products<PA, PB>;
    using TA = Tile<LA, BM, KT, NW>;
    using TB = Tile<LB, BN, KT, NW>;
    constexpr int FM = BM / WM / 32, FN = BN / WN / 32;
    using FA = Frags<LA, PA, FM, BM, KT>;
    using FB = Frags<LB, PB, FN, BN, KT>;
    constexpr int kOffB = PA * TA::kPlane, kSlot = kOffB + PB * TB::kPlane;
    constexpr int NS = KT / 16;
    static_assert(NS % 2 == 0, "register sets alternate with the k16 steps of a tile");
    constexpr int NR = FA::kReads + FB::kReads, NM = FM * FN * PR::kCount;
    constexpr int kStores = FM * FN * 16;                   // of a whole tile, per wave
    __shared__ __attribute__((aligned(1024))) char smem[R * kSlot];
    __shared__ __attribute__((aligned(16))) float sbias[2][BN];

    const int wave = threadIdx.x >> 6, wm = wave % WM, wn = wave / WM;
    const int lane = threadIdx.x & 63;
    const float inv = g.c_div ? 1.f / g.c_div[0] : 1.f;
    int item = persistent_item(blockIdx.x, gridDim.x, g.total, 0);
    if (item < 0) return;

    FA fa;
    FB fb;
    fa.init(smem, wm * FM * 32);
    fb.init(smem + kOffB, wn * FN * 32);
    auto read_all = [&](uint32_t d) {
        static_for<0, FA::kReads>([&](auto n) { fa.template read<0, n()>(d); });
        static_for<0, FB::kReads>([&](auto n) { fb.template read<0, n()>(d); });
    };

    // the copying side: the item and k-tile to copy next
    TA ta;
    TB tb;
    int cj = 0, citem = item, cslot = 0;
    Item ci = locate<BM, BN>(g, citem);
    int ck = ci.kbeg, cbeg = ci.kbeg, cplane = NP - 1;  // k-tile, its chunk's start, B's part
    auto copy_setup = [&] {
        ta.init((uint32_t)g.lda, g.M, g.a_cols, ci.m0);
        tb.init((uint32_t)g.ldb, g.N, g.b_cols, ci.n0);
        if (g.bias && wave < BN / 64) {
            const int w = __builtin_amdgcn_readfirstlane(wave);
            __builtin_amdgcn_global_load_lds(g.bias + min(ci.n0 + w * 64 + lane, g.N - 1),
                                             (lds_void *)(&sbias[cj & 1][w * 64]), 4, 0, 0);
        }
    };
    // the copies of one tile in three pieces, spread over a step's MFMAs
    auto copy_piece = [&](auto piece) {
        if (citem < 0) return;
        char *to = smem + cslot * kSlot;
        if constexpr (piece() == 0) {
#pragma unroll
            for (int p = 0; p < PA; ++p)
                ta.copy(g.A + p * g.a_ps, (uint32_t)g.lda, g.a_cols, g.K, ck, to + p * TA::kPlane);
        } else if constexpr (piece() == 1) {
#pragma unroll
            for (int p = 0; p < PB; ++p)
                tb.copy(g.B + (p + (NP > 1 ? cplane : 0)) * g.b_ps, (uint32_t)g.ldb, g.b_cols, g.K, ck,
                        to + kOffB + p * TB::kPlane);
        } else {
            cslot = cslot + 1 == R ? 0 : cslot + 1;
            ck += KT;
            if constexpr (NP > 1) {
                if (ck >= min(cbeg + g.sum_chunk, ci.kend)) {
                    if (cplane > 0) {
                        --cplane;
                        ck = cbeg;
                    } else {
                        cplane = NP - 1;
                        cbeg = ck;
                    }
                }
            }
            if (ck >= ci.kend) {
                citem = persistent_item(blockIdx.x, gridDim.x, g.total, ++cj);
                if (citem >= 0) {
                    ci = locate<BM, BN>(g, citem);
                    ck = cbeg = ci.kbeg;
                    copy_setup();
                }
            }
        }
    };
    copy_setup();
#pragma unroll
    for (int i = 0; i < R - 1; ++i)
        static_for<0, 3>([&](auto piece) { copy_piece(piece); });
    if constexpr (kCross) asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    int slot = 0;
    bool stored = false;  // a whole tile, just before this step

    for (int j = 0; item >= 0; ++j) {
        const Item it = locate<BM, BN>(g, item);
        static_assert(!FOLD || PR::kSums == 1, "the second sum is the total");
        constexpr int kAcc = FOLD ? 2 : PR::kSums;
        floatx16 acc[kAcc][FM][FN];
#pragma unroll
        for (int z = 0; z < kAcc; ++z)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int q = 0; q < FN; ++q)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[z][i][q][r] = 0.f;
        if constexpr (kCross) read_all(slot * kSlot);
        int plane = NP - 1, beg = it.kbeg;
        for (int k0 = it.kbeg, nk; k0 < it.kend; k0 = nk) {
            nk = k0 + KT;
            bool chunk_done = false;
            if constexpr (NP > 1 || FOLD) {
                if (nk >= min(beg + g.sum_chunk, it.kend)) {
                    if (plane > 0) {
                        --plane;
                        nk = beg;
                    } else {
                        plane = NP - 1;
                        beg = nk;
                        chunk_done = true;
                    }
                }
            }
            // The tile this barrier gives (t + 1, or t for R = 2) has landed.
            // A whole tile's stores may be in flight: they were issued after
            // every copy that this step waits for, and vector memory
            // operations complete in order.
            if (stored && kStores >= 64)
                asm volatile("s_waitcnt vmcnt(63)\n\ts_barrier" ::: "memory");
            else
                asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
            stored = false;
            const int kvalid = it.kend - k0;
            const bool more = nk < it.kend;
            const uint32_t d = slot * kSlot;
            const int ns = slot + 1 == R ? 0 : slot + 1;
            const uint32_t dn = more ? ns * kSlot : d;
            if constexpr (!kCross) {
                read_all(d);
                __builtin_amdgcn_sched_barrier(0);
                static_for<0, 3>([&](auto piece) { copy_piece(piece); });
                __builtin_amdgcn_sched_barrier(0);
            }
            static_for<0, NS>([&](auto sc) {
                constexpr int S = sc();
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                fa.template ready<S>(kvalid);
                fb.template ready<S>(kvalid);
                __builtin_amdgcn_sched_barrier(0);
                static_for<0, NM>([&](auto nc) {
                    constexpr int n = nc(), q = n / (FM * FN), i = n % (FM * FN) / FN, c = n % FN;
                    acc[PR::sum(q)][i][c] = mfma32<MT>(fa.q[S & 1][PR::a(q)][i],
                                                       fb.q[S & 1][PR::b(q)][c],
                                                       acc[PR::sum(q)][i][c]);
                    __builtin_amdgcn_sched_barrier(0);
                    // the copies, after MFMAs that keep the cores busy
                    if constexpr (kCross && S == 0) {
                        constexpr int piece = n == 0 ? 0 : n == NM / 4 ? 1 : n == NM / 2 ? 2 : 3;
                        if constexpr (piece < 3) copy_piece(std::integral_constant<int, piece>{});
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    // the next step's reads, spread over this step's MFMAs
                    // (past the item's last tile: that tile again, dropped)
                    if constexpr (kCross || S + 1 < NS) {
                        constexpr int lo = n * NR / NM, hi = (n + 1) * NR / NM;
                        static_for<lo, hi>([&](auto rc) {
                            constexpr int r = rc(), S1 = (S + 1) % NS;
                            const uint32_t dd = S + 1 < NS ? d : dn;
                            if constexpr (r < FA::kReads) fa.template read<S1, r>(dd);
                            else fb.template read<S1, r - FA::kReads>(dd);
                        });
                        __builtin_amdgcn_sched_barrier(0);
                    }
                });
            });
            slot = ns;
            if (FOLD && chunk_done) {
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int q = 0; q < FN; ++q)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            acc[kAcc - 1][i][q][r] += acc[0][i][q][r];
                            acc[0][i][q][r] = 0.f;
                        }
            }
        }
        if constexpr (kCross) {
            // the reads past the last tile land before their registers are
            // used for anything else
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            fa.template ready<0>(KT);
            fb.template ready<0>(KT);
        }
        item = persistent_item(blockIdx.x, gridDim.x, g.total, j + 1);
        float bn[FN];
#pragma unroll
        for (int q = 0; q < FN; ++q) bn[q] = 0.f;
        if (g.bias) {
            // landed: copied before this item's tiles
#pragma unroll
            for (int q = 0; q < FN; ++q)
                asm volatile("ds_read_b32 %0, %1"
                             : "=v"(bn[q])
                             : "v"(lds_addr(&sbias[j & 1][(wn * FN + q) * 32 + (lane & 31)])));
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int q = 0; q < FN; ++q) asm volatile("" : "+v"(bn[q]));
        }
        float *Cz = g.C + (int64_t)it.zk * g.split_stride;
        const bool full = it.m0 + BM <= g.M && it.n0 + BN <= g.N;
        stored = full;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int q = 0; q < FN; ++q) {
                const int n = it.n0 + (wn * FN + q) * 32 + (lane & 31);
                const int mb = it.m0 + (wm * FM + i) * 32 + 4 * (lane >> 5);
                floatx16 v = acc[FOLD ? 1 : 0][i][q];
                if constexpr (PR::kSums == 2) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) v[r] += acc[PR::kSums - 1][i][q][r];
                }
                if constexpr (PA * PB == 9) {
                    // An infinity or NaN among the inputs leaves NaN against
                    // zero parts: such a block is taken again from the whole
                    // values.
                    static_assert(PA * PB != 9 || (LA == L_KC && LB == L_MN), "whole_block's layouts");
                    bool bad = false;
#pragma unroll
                    for (int r = 0; r < 16; ++r) bad |= !(__builtin_fabsf(v[r]) < INFINITY);
                    if (__builtin_expect(__any(bad), 0)) {
                        const int mf = it.m0 + (wm * FM + i) * 32 + (lane & 31);
                        const floatx16 t =
                            whole_block(g.A, g.lda, g.a_ps, g.B, g.ldb, g.b_ps, min(mf, g.M - 1),
                                        min(n, g.N - 1), it.kbeg, it.kend);
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            if (!(__builtin_fabsf(v[r]) < INFINITY)) v[r] = t[r];
                    }
                }
                float *row = Cz + (int64_t)mb * g.ldc + n;
                if (full) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        row[(int64_t)(8 * (r >> 2) + (r & 3)) * g.ldc] = v[r] * inv + bn[q];
                } else if (n < g.N) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (mb + 8 * (r >> 2) + (r & 3) < g.M)
                            row[(int64_t)(8 * (r >> 2) + (r & 3)) * g.ldc] = v[r] * inv + bn[q];
                }
            }
    }
    // the workgroup's LDS must not be released with copies into it in flight
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// ---- operands rewritten for the copies --------------------------------------
// Spike bytes widened to the MFMA type, 16-bit values as they are, or fp32
// values as three bf16 parts.  In rows: dst[p][r][ld] from src[r * lds + c], c <
// cols; columns cols .. ld - 1 are zero.  In fragment order (frag): rows and
// columns past the end are zero.  A thread writes one 16-byte chunk of each
// part.  Both operands of a contraction go in one launch: workgroups below
// `split` take the first.
constexpr int kPackThreads = 256;
enum : int { PACK_U8 = 0, PACK_H16 = 1, PACK_F32 = 2 };
struct PackOp {
    const void *src;
    uint16_t *dst;
    int64_t lds, ld, rows, ps;
    int cols, kind, frag;
    __host__ __device__ int64_t chunks() const {
        return frag ? (rows + 31) / 32 * (ld / 8) : rows * (ld / 8);
    }
};

__device__ inline void pack_chunk(const PackOp &o, int64_t i, int mt) {
    if (i >= o.chunks()) return;
    int64_t r, d;
    int c0;
    if (o.frag) {
        // 32 consecutive threads take 32 rows of one chunk: a wave writes 1 KiB
        const int c8 = (int)(o.ld / 256);  // chunks per row
        const int64_t rb = i / (32 * c8);
        const int in = (int)(i - rb * (32 * c8)), c = in >> 5;
        r = rb * 32 + (in & 31);
        c0 = c * 8;
        d = rb * o.ld + (c >> 1) * 512 + (c & 1) * 256 + (in & 31) * 8;
    } else {
        const int cpr = (int)(o.ld / 8);
        r = i / cpr;
        c0 = (int)(i - r * cpr) * 8;
        d = r * o.ld + c0;
    }
    // (a chunk may hold padding only)
    const int valid = r < o.rows ? min(8, o.cols - c0) : 0;
    const int64_t so = r * o.lds + c0;
    uint32_t h[8];
    if (o.kind == PACK_U8) {
        const uint8_t *s = reinterpret_cast<const uint8_t *>(o.src) + so;
        uint32_t b[8];
        if (valid == 8 && ((uintptr_t)s & 7) == 0) {
            const uint2 w = *reinterpret_cast<const uint2 *>(s);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                b[e] = (w.x >> (8 * e)) & 0xffu;
                b[4 + e] = (w.y >> (8 * e)) & 0xffu;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) b[e] = e < valid ? s[e] : 0u;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v = (float)b[e];
            h[e] = mt == MT_F16 ? (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)v)
                                : __float_as_uint(v) >> 16;
        }
    } else if (o.kind == PACK_H16) {
        const uint16_t *s = reinterpret_cast<const uint16_t *>(o.src) + so;
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = e < valid ? s[e] : 0u;
    } else {
        const float *s = reinterpret_cast<const float *>(o.src) + so;
        float v[8];
        if (valid == 8 && ((uintptr_t)s & 15) == 0) {
            const float4 a = *reinterpret_cast<const float4 *>(s);
            const float4 b = *reinterpret_cast<const float4 *>(s + 4);
            v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
            v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = e < valid ? s[e] : 0.f;
        }
        uint32_t mid[8], lo[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) split_bf16x3(v[e], h[e], mid[e], lo[e]);
        *reinterpret_cast<uint4 *>(o.dst + o.ps + d) =
            make_uint4(mid[0] | (mid[1] << 16), mid[2] | (mid[3] << 16), mid[4] | (mid[5] << 16),
                       mid[6] | (mid[7] << 16));
        *reinterpret_cast<uint4 *>(o.dst + 2 * o.ps + d) =
            make_uint4(lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16), lo[4] | (lo[5] << 16),
                       lo[6] | (lo[7] << 16));
    }
    *reinterpret_cast<uint4 *>(o.dst + d) =
        make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
}

__global__ __launch_bounds__(kPackThreads) void pack_kernel(PackOp a, PackOp b, unsigned split,
                                                            int mt) {
    if (blockIdx.x < split)
        pack_chunk(a, (int64_t)blockIdx.x * kPackThreads + threadIdx.x, mt);
    else
        pack_chunk(b, (int64_t)(blockIdx.x - split) * kPackThreads + threadIdx.x, mt);
}

// ---- planning ------------------------------------------------------------------
bool fp32ish(int t) { return t == SNN_F32 || t == kPlanes3; }

// MFMA type of an operand pair (-1: not a pair of this file)
int pair_type(int a, int b) {
    if (fp32ish(a) || fp32ish(b)) {
        const int o = fp32ish(a) ? b : a;
        return fp32ish(o) || o == SNN_U8 || o == SNN_BF16 ? MT_BF16 : -1;
    }
    auto f16ish = [](int t) { return t == SNN_U8 || t == SNN_F16; };
    auto bf16ish = [](int t) { return t == SNN_U8 || t == SNN_BF16; };
    if (f16ish(a) && f16ish(b)) return MT_F16;
    if (bf16ish(a) && bf16ish(b)) return MT_BF16;
    return -1;
}

struct Operand {
    int layout;        // L_*
    bool pack;         // rewritten into the workspace
    int64_t ld, rows;  // stride and number of memory rows as the copies see them
    int cols;          // readable values per memory row
    int64_t ps;        // elements per part when packed
    size_t bytes;      // workspace
};

// frag: the operand may be packed in fragment order (K-contiguous operands
// that are rewritten anyway, or `always`: 1 KiB of consecutive memory per copy)
Operand plan_operand(int dtype, bool kc, int64_t ld, int64_t ps, int rows, int K, bool frag,
                     bool always) {
    Operand o{};
    const int mr = kc ? rows : K, mc = kc ? K : rows;  // memory rows, columns
    o.rows = mr;
    o.layout = kc ? L_KC : L_MN;
    o.pack = always || dtype == SNN_U8 || dtype == SNN_F32 || mc % 8 != 0 || ld % 8 != 0 ||
             (dtype == kPlanes3 && ps % 8 != 0);
    o.cols = (mc + 7) / 8 * 8;
    o.ld = o.pack ? o.cols : ld;
    o.ps = o.rows * o.ld;
    if (frag && o.pack) {
        o.layout = L_PK;
        o.ld = (int64_t)((K + 63) / 64 * 64) * 32;
        o.ps = (rows + 31) / 32 * o.ld;
    }
    o.bytes = o.pack ? align_up((size_t)(fp32ish(dtype) ? 3 : 1) * o.ps * 2) : 0;
    return o;
}

// Tile configurations: tile, k-tile, ring slots, items per CU at once
enum : int { kNone = 0, kOne, kThree, kThreeT, kNineBig, kNineSmall, kTurnBig, kTurn, kThreeSmall };
struct Shape { int BM, BN, KT, R, per_cu; float step_us; };
// Time of one k-tile step of one item with the CU's other items beside it, from
// contractions of 2013 .. 16000 rows with 700 .. 2048 inputs and outputs.  Two
// 128 x 128 workgroups per CU beat one of 256 x 128 with three slots for one
// by one part (26 against 29 us on 6400 x 1000 x 1000); for spikes by three
// parts the latter moves 5/8 of the bytes into LDS (53 against 55 us); for
// three by three, 256 x 128 takes 122 against 126 us there, but 128 x 128
// leaves a smaller last wave on narrow outputs (181 against 203 us on 12800 x
// 784 x 1000).  Currents: parts in turn, 256 x 256 tiles one chunk each (73 us
// on 12800 x 1000 x 784, 200 tiles) or 256 x 128 ones that fold the chunks (56
// us on 6400 x 1000 x 1000); parts within a step, 128 x 128 tiles where 256 x
// 128 ones leave most compute units idle (25 against 37 us on 2013 x 1101 x
// 1003, 144 and 72 tiles).
constexpr Shape kShapes[] = {{0, 0, 0, 0, 0, 0.f},
                             {128, 128, 64, 2, 2, 1.4f},
                             {256, 128, 32, 3, 1, 1.3f},
                             {128, 256, 32, 3, 1, 1.3f},
                             {256, 128, 32, 2, 1, 2.8f},
                             {128, 128, 32, 3, 1, 1.6f},
                             {256, 256, 64, 2, 1, 1.8f},
                             {256, 128, 64, 3, 1, 1.1f},
                             {128, 128, 32, 3, 1, 0.75f}};

struct JointPlan {
    int cfg, mt, tiles_m, tiles_n, splits, k_chunk, sum_chunk;
    Operand a, b;
    size_t part_bytes;
    double us;  // estimated kernel time (with the reduction of split partials)
};

void plan_cfg(const GemmArgs &g, int cfg, JointPlan &best) {
    const Shape &sh = kShapes[cfg];
    const int tm = (g.M + sh.BM - 1) / sh.BM, tn = (g.N + sh.BN - 1) / sh.BN;
    const double tiles = (double)tm * tn;
    const int nk = (g.K + sh.KT - 1) / sh.KT;
    // (host time: no 64-bit division in this loop, which several plans of a
    // layer call run)
    const double per_round = 1.0 / (kPlanCus * sh.per_cu);
    for (int S = 1; S <= 32 && (S == 1 || 4 * S <= nk); ++S) {
        const int per = (nk + S - 1) / S;
        if ((S - 1) * per >= nk) continue;  // fewer splits than S
        const double rounds = __builtin_ceil(tiles * S * per_round);
        // an item: its steps and about 3 us of first copies and stores; split
        // partials are written and read once more at the copy rate
        double us = rounds * (per * (double)sh.step_us + 3.0);
        if (S > 1) us += 4.0 + (double)g.M * g.N * 4.0 * (2 * S + 1) / 4.5e6;
        if (us < best.us) {
            best.us = us;
            best.cfg = cfg;
            best.tiles_m = tm;
            best.tiles_n = tn;
            best.splits = S;
            best.k_chunk = per * sh.KT;
        }
    }
}

// The order in which a product of two K-contiguous operands, the currents, is
// summed.  A membrane within rounding of the threshold turns a spike with the
// last bit of its current, so kernels that take over a size keep the order
// that it is summed in by the others, bit for bit: where 256 x 256 tiles fill
// the device (gemm_async_sum_chunk), its chunks of K, an fp32 operand's parts in
// turn over each; else the 16-bit kernel's chunks, the parts in turn at each
// k16 step.
struct SumOrder {
    int chunk;
    bool turn;
};
SumOrder sum_order(const GemmArgs &g) {
    GemmArgs o = g;
    if (fp32ish(g.b_dtype)) o.a_dtype = SNN_U8;  // bf16 spikes as the bytes they stand for
    SumOrder r{};
    r.chunk = gemm_async_sum_chunk(o);
    r.turn = r.chunk > 0 && fp32ish(g.b_dtype);
    if (r.chunk == 0) r.chunk = gemm16_sum_chunk(o);
    if (r.chunk == 0) r.chunk = g.K;
    return r;
}

// Currents: the chunks of the order summed by one workgroup in turn, or one
// item each with their partials added by the reduction (the wide reduction of
// 16 or more adds quarters: only the split takes its order).
void plan_order(const GemmArgs &g, int cfg, bool fold, const SumOrder &o, JointPlan &best) {
    const Shape &sh = kShapes[cfg];
    const int tm = (g.M + sh.BM - 1) / sh.BM, tn = (g.N + sh.BN - 1) / sh.BN;
    const int chunks = (g.K + o.chunk - 1) / o.chunk, slots = kPlanCus * sh.per_cu;
    const int passes = o.turn ? 3 : 1;
    for (const int S : {1, chunks}) {
        if (S == 1 && chunks > 1 && (!fold || chunks >= 16)) continue;
        const int span = S == 1 ? g.K : o.chunk;
        const int64_t rounds = ((int64_t)tm * tn * S + slots - 1) / slots;
        double us = rounds * (passes * ((span + sh.KT - 1) / sh.KT) * (double)sh.step_us + 3.0);
        if (S > 1) us += 4.0 + (double)g.M * g.N * 4.0 * (2 * S + 1) / 4.5e6;
        if (us < best.us) {
            best.us = us;
            best.cfg = cfg;
            best.tiles_m = tm;
            best.tiles_n = tn;
            best.splits = S;
            best.k_chunk = S == 1 ? (g.K + 63) / 64 * 64 : o.chunk;
            best.sum_chunk = o.chunk;
        }
    }
}

JointPlan make_plan(const GemmArgs &g) {
    JointPlan p{};
    p.us = 1e300;
    p.mt = pair_type(g.a_dtype, g.b_dtype);
    const int pa = fp32ish(g.a_dtype) ? 3 : 1, pb = fp32ish(g.b_dtype) ? 3 : 1;
    const bool currents = g.a_kc && g.b_kc;
    const SumOrder o = currents ? sum_order(g) : SumOrder{};
    const bool frag = pa * pb == 3 && currents;
    // (taking the parts in turn, both come in fragment order)
    p.a = plan_operand(g.a_dtype, g.a_kc, g.lda, g.a_ps, g.M, g.K,
                       frag && (g.a_dtype == SNN_U8 || o.turn), frag && o.turn);
    p.b = plan_operand(g.b_dtype, g.b_kc, g.ldb, g.b_ps, g.N, g.K, frag, false);
    if (pa * pb == 9) {
        plan_cfg(g, kNineBig, p);
        plan_cfg(g, kNineSmall, p);
    } else if (o.turn) {
        plan_order(g, kTurnBig, false, o, p);
        plan_order(g, kTurn, true, o, p);
    } else if (currents) {
        plan_order(g, pb == 3 ? kThree : kOne, true, o, p);
        if (pb == 3) plan_order(g, kThreeSmall, true, o, p);
    } else {
        plan_cfg(g, pa == 3 ? kThreeT : kOne, p);
    }
    p.part_bytes = p.splits > 1 ? align_up((size_t)p.splits * g.M * g.N * sizeof(float)) : 0;
    return p;
}

template <int MT, int PA, int PB, int LA, int LB, int CFG, int WM, int WN, int NP = 1,
          bool FOLD = false>
void launch_cfg(const JointArgs &a, hipStream_t s) {
    constexpr Shape sh = kShapes[CFG];
    const unsigned grid = (unsigned)min(a.total, device_cus() * sh.per_cu);
    gemm_joint_kernel<MT, PA, PB, LA, LB, sh.BM, sh.BN, sh.KT, sh.R, WM, WN, NP, FOLD>
        <<<grid, 64 * WM * WN, 0, s>>>(a);
}

template <int MT>
void launch_one(const GemmArgs &g, const JointArgs &a, hipStream_t s) {
    if (g.a_kc && g.b_kc) launch_cfg<MT, 1, 1, L_KC, L_KC, kOne, 2, 2, 1, true>(a, s);
    else if (g.a_kc) launch_cfg<MT, 1, 1, L_KC, L_MN, kOne, 2, 2>(a, s);
    else launch_cfg<MT, 1, 1, L_MN, L_MN, kOne, 2, 2>(a, s);
}

}  // namespace

bool gemm_joint_fits(const GemmArgs &g) {
    if (!g.allow_split || g.pool_hw > 0 || g.M < 64 || g.N < 64 || g.K < 192) return false;
    if (pair_type(g.a_dtype, g.b_dtype) < 0) return false;
    if (!g.a_kc && g.b_kc) return false;
    if (g.a_dtype == kPlanes3 &&
        plan_operand(kPlanes3, g.a_kc, g.lda, g.a_ps, g.M, g.K, false, false).pack)
        return false;
    if (g.b_dtype == kPlanes3) return false;
    const bool nine = fp32ish(g.a_dtype) && fp32ish(g.b_dtype);
    const bool three = !nine && (fp32ish(g.a_dtype) || fp32ish(g.b_dtype));
    if (nine != (g.a_kc && !g.b_kc) && (nine || three)) return false;
    if (nine && g.c_div) return false;
    if (three && (g.c_div || fp32ish(g.a_dtype) != !g.a_kc)) return false;
    // 32-bit element offsets within a part
    const int64_t lim = (int64_t)1 << 31;
    if ((int64_t)(g.M + 32) * (g.K + 64) >= lim || (int64_t)(g.N + 32) * (g.K + 64) >= lim ||
        (g.a_kc ? g.M : g.K) * g.lda >= lim || (g.b_kc ? g.N : g.K) * g.ldb >= lim)
        return false;
    // Below, the rewriting and the split reduction cost what the kernel saves
    // (800 x 784 x 1000, 0.6 G products: 32 us for dx on either path).
    return (double)g.M * g.N * g.K >= 1073741824.0;
}

namespace {
// The kernel with its rewriting against the kernels that run a product without
// it, both from fits to measured times (1090 products of 64 .. 400000 rows and
// 64 .. 16384 inputs and outputs, three classes: currents, dW, dx; this one
// nine in ten within 12 %).  Tiles half empty, few rows or narrow layers and
// deep splits go to the others: us, other kernel / this one,
//   fp32 currents   64 rows 8192 -> 2048  30 / 59,  10715 rows 5776 -> 96  78 / 111
//                   (6400 rows 1000 -> 1000  84 / 63,  2013 rows 1003 -> 1101  95 / 37)
//   fp32 dW         262144 rows 64 -> 64  78 / 293,  4096 rows 64 -> 4096  29 / 59
//                   (2013 rows 1003 -> 1101  65 / 39,  3000 rows 600 -> 600  42 / 31)
//   fp32 dx         64 rows 8192 <- 2048  38 / 59,  16384 rows 64 <- 1024  50 / 62
//                   (6400 rows 1000 <- 1000  181 / 106)
// Choosing so loses 0.5 % against the better one on average.
bool faster(const GemmArgs &g) {
    GemmArgs o = g;
    // (planes as the fp32 values they stand for: one choice for both)
    if (o.a_dtype == kPlanes3) o.a_dtype = SNN_F32;
    const bool dw = !o.a_kc && !o.b_kc;
    const bool one = !fp32ish(o.a_dtype) && !fp32ish(o.b_dtype);
    const bool nine = o.a_dtype == SNN_F32 && o.b_dtype == SNN_F32;
    if (one && !dw) return true;
    // bf16 spikes against fp32 go to the fp32 matrix cores otherwise
    if (!one && !nine && o.a_dtype != SNN_U8 && o.b_dtype != SNN_U8) return true;
    const JointPlan p = make_plan(o);
    if (p.cfg == kTurnBig || p.cfg == kTurn) return true;
    const Shape &sh = kShapes[p.cfg];
    if (dw && (one || g.K > 8192)) {
        // whole tiles' worth of work in flight
        const double items = (double)p.splits * g.M * g.N / (sh.BM * sh.BN);
        // 16-bit pairs: only the smallest outputs over the longest K are slower
        // (64 x 64 over 262144 rows 53 / 115 us, 100 x 100 over 200000 71 / 69)
        if (one) return items >= 18.0;
        // More than 8192 rows are transposed for the other kernels: always
        // slower where the rows are no whole 8 (96 x 5776 over 10715 464 / 86
        // us), from 20 items where no whole 16 (120 x 264 over 61976 118 / 92; 96 x
        // 200 over 365000 470 / 523), else from 50 (88 x 792 over 15504 55 / 45;
        // 256 x 64 over 65536 64 / 101) of tiles more than half full (64 x 1024
        // over 16384 42 / 45)
        if (g.K % 16 != 0) return g.K % 8 != 0 || items >= 20.0;
        return items >= 50.0 && 2 * g.M > p.tiles_m * sh.BM;
    }
    if (o.a_kc && o.b_kc) {
        // currents: rewriting the weights for fewer than 100 rows costs more
        // than it saves (80 rows 9420 <- 4722 133 / 201 us); with both sides long
        // the 16-bit kernel's many tiles leave its estimate (4129 rows 192 ->
        // 2584 49 / 33 us, 3968 of 592 -> 2544 70 / 55)
        if (g.M < 100) return false;
        if (g.M >= 2048 && g.N >= 2048) return true;
    }
    const double step = p.cfg == kThree ? 0.97 : p.cfg == kThreeSmall ? 0.56 : p.cfg == kThreeT ? 1.07
                        : p.cfg == kNineBig ? 2.5 : 1.34;
    const int64_t rounds = ((int64_t)p.tiles_m * p.tiles_n * p.splits + kPlanCus - 1) / kPlanCus;
    const int steps = ((p.splits > 1 ? p.k_chunk : g.K) + sh.KT - 1) / sh.KT;
    const double mb = (double)g.M * g.N * 4.0 * (p.splits > 1 ? 2 * p.splits + 2 : 1) / 1e6;
    auto packed = [](int t, double n) { return n * (t == SNN_F32 ? 10.0 : 3.0) / 1e6; };
    const double us = 13.0 + rounds * steps * step + 0.17 * mb +
                      0.165 * (packed(o.a_dtype, (double)g.M * g.K) + packed(o.b_dtype, (double)g.N * g.K));
    return us < (nine ? gemm_f32_us(g.M, g.N, g.K) : gemm16_us(o));
}
}  // namespace

bool gemm_joint_applies(const GemmArgs &g) { return gemm_joint_fits(g) && faster(g); }

double gemm_joint_us(const GemmArgs &g) {
    return gemm_joint_applies(g) ? make_plan(g).us : 1e300;
}

namespace {
size_t gemm_order_part_bytes(const GemmArgs &g) {
    GemmArgs o = g;
    if (fp32ish(g.b_dtype)) o.a_dtype = SNN_U8;
    const int chunk = gemm_async_sum_chunk(o);
    const size_t turn = chunk > 0 && chunk < g.K
                            ? align_up((size_t)((g.K + chunk - 1) / chunk) * g.M * g.N * sizeof(float))
                            : 0;
    return larger(turn, gemm16_workspace_bytes(o));
}
}  // namespace

size_t gemm_joint_workspace_bytes(const GemmArgs &g) {
    if (!gemm_joint_fits(g)) return 0;
    const JointPlan p = make_plan(g);
    size_t part = p.part_bytes;
    // the chunks may depend on the device and on a bias: any plan's partials
    if (g.a_kc && g.b_kc) part = larger(part, gemm_order_part_bytes(g));
    return p.a.bytes + p.b.bytes + part;
}

hipError_t launch_gemm_joint(const GemmArgs &g, void *ws, size_t ws_bytes, hipStream_t s) {
    const JointPlan p = make_plan(g);
    const size_t need = p.a.bytes + p.b.bytes + p.part_bytes;
    if (need > 0 && (ws == nullptr || ws_bytes < need)) return hipErrorInvalidValue;
    char *w = reinterpret_cast<char *>(ws);
    JointArgs a{};
    a.M = g.M; a.N = g.N; a.K = g.K;
    a.k_chunk = p.k_chunk;
    a.sum_chunk = p.sum_chunk;
    a.tiles_n = p.tiles_n;
    a.tiles = p.tiles_m * p.tiles_n;
    a.total = a.tiles * p.splits;
    a.A = reinterpret_cast<const uint16_t *>(g.A);
    a.B = reinterpret_cast<const uint16_t *>(g.B);
    a.lda = p.a.ld; a.ldb = p.b.ld;
    a.a_ps = g.a_ps; a.b_ps = g.b_ps;
    a.a_cols = p.a.cols; a.b_cols = p.b.cols;
    PackOp ops[2] = {};
    int n_ops = 0;
    auto pack = [&](const Operand &o, int dtype, const void *src, int64_t ld, int cols,
                    uint16_t *dst) {
        PackOp &q = ops[n_ops++];
        q.src = src; q.dst = dst; q.lds = ld; q.ld = o.ld; q.rows = o.rows; q.cols = cols;
        q.ps = o.ps;
        q.frag = o.layout == L_PK;
        q.kind = dtype == SNN_U8 ? PACK_U8 : dtype == SNN_F32 ? PACK_F32 : PACK_H16;
    };
    if (p.a.pack) {
        uint16_t *d = reinterpret_cast<uint16_t *>(w);
        pack(p.a, g.a_dtype, g.A, g.lda, g.a_kc ? g.K : g.M, d);
        a.A = d;
        a.a_ps = p.a.ps;
    }
    if (p.b.pack) {
        uint16_t *d = reinterpret_cast<uint16_t *>(w + p.a.bytes);
        pack(p.b, g.b_dtype, g.B, g.ldb, g.b_kc ? g.K : g.N, d);
        a.B = d;
        a.b_ps = p.b.ps;
    }
    if (n_ops > 0) {
        unsigned nb[2] = {0, 0};
        for (int i = 0; i < n_ops; ++i)
            nb[i] = (unsigned)((ops[i].chunks() + kPackThreads - 1) / kPackThreads);
        pack_kernel<<<nb[0] + nb[1], kPackThreads, 0, s>>>(ops[0], ops[1], nb[0], p.mt);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    a.C = g.C; a.ldc = g.ldc; a.bias = g.bias; a.c_div = g.c_div;
    if (p.splits > 1) {
        a.C = reinterpret_cast<float *>(w + p.a.bytes + p.b.bytes);
        a.ldc = g.N;
        a.split_stride = (int64_t)g.M * g.N;
        a.bias = nullptr;
        a.c_div = nullptr;  // divided in the reduction
    }
    switch (p.cfg) {
        case kNineBig: launch_cfg<MT_BF16, 3, 3, L_KC, L_MN, kNineBig, 4, 2>(a, s); break;
        case kNineSmall: launch_cfg<MT_BF16, 3, 3, L_KC, L_MN, kNineSmall, 2, 4>(a, s); break;
        case kThree:
            if (p.a.layout == L_PK)
                launch_cfg<MT_BF16, 1, 3, L_PK, L_PK, kThree, 4, 2, 1, true>(a, s);
            else
                launch_cfg<MT_BF16, 1, 3, L_KC, L_PK, kThree, 4, 2, 1, true>(a, s);
            break;
        case kThreeSmall:
            if (p.a.layout == L_PK)
                launch_cfg<MT_BF16, 1, 3, L_PK, L_PK, kThreeSmall, 4, 2, 1, true>(a, s);
            else
                launch_cfg<MT_BF16, 1, 3, L_KC, L_PK, kThreeSmall, 4, 2, 1, true>(a, s);
            break;
        case kTurnBig: launch_cfg<MT_BF16, 1, 1, L_PK, L_PK, kTurnBig, 2, 4, 3>(a, s); break;
        case kTurn: launch_cfg<MT_BF16, 1, 1, L_PK, L_PK, kTurn, 4, 2, 3, true>(a, s); break;
        case kThreeT: launch_cfg<MT_BF16, 3, 1, L_MN, L_MN, kThreeT, 2, 4>(a, s); break;
        default:
            if (p.mt == MT_F16) launch_one<MT_F16>(g, a, s);
            else launch_one<MT_BF16>(g, a, s);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (p.splits > 1)
        e = launch_splitk_reduce(g.M, g.N, p.splits, a.C, g.C, g.ldc, g.bias, s, g.c_div);
    return e;
}

}  // namespace snn
