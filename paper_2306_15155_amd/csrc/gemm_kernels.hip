// Dense kernels for gfx950: the fp32 update GEMM on the matrix cores with the activation fused into the
// epilogue (small products: v_mfma_f32_32x32x2_f32; large ones: v_mfma_f32_32x32x16_bf16 on three exact
// bf16 pieces per fp32 operand), the dense tiles of the hub region of a skewed graph (the same bf16
// instruction), the weight-gradient GEMM with fp64 slabs, and a two-vector GEMV for the attention projections.
#include "sensei_internal.h"

#include <type_traits>

namespace sensei {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kThreads = kSideThreads;
constexpr int KT = 16;  // k extent of one LDS tile

struct GemmArgs {
    const float *A, *W, *row_scale;  // row_scale: optional per-row factor applied before the activation
    float *Y;
    long long lda, ldw, ldy, n;
    int k, m, m_store, act, n_bn;
    int n_parts, by_xcd, a_lds;   // k_gemm_bf: shares of the rows; whether the blocks of columns of a share run on one XCD; where in LDS the rows of A are
    int y_sliced;  // Y stored slice-major in tiles of 32 columns: (row, col) at Y[(col / 32) * n * 32 + row * 32 + col % 32]
    long long a_slice;   // floats from columns 32 s .. 32 s + 31 of A to the next 32: 32 for a row-major A, n * 32 (with lda = 32) for a slice-major one
    const float *add;    // optional n x pad32(m) slice-major matrix added to the product before scaling and activation
    SideWork side;       // small work of the call this product belongs to, done by the first workgroups
};

// Block tile BM x BN, 4 wavefronts laid out WGM x WGN, each computing TM x TN tiles of 32 x 32
// with the 32x32x2 fp32 MFMA.  LDS holds A as [k][row] and W as [k][col] so that the MFMA operand
// reads (lane l takes k = l / 32, row or col = l % 32) are consecutive words.  The next k-tile is
// fetched from HBM into registers while the current one is multiplied.
template <int BM, int BN, int WGM, int WGN, int AVEC, int BVEC>
__global__ __launch_bounds__(kThreads) void k_gemm(GemmArgs g) {
    if ((int)blockIdx.x < g.side.blocks) return side_block(g.side, (int)blockIdx.x);
    const unsigned block = blockIdx.x - g.side.blocks;
    constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;
    constexpr int APAD = 36, BPAD = 36;  // row stride = 36 mod 64 words: the two k-rows an MFMA operand read touches fall on (nearly) disjoint LDS banks, and the four k-rows a stash writes are 16 banks apart
    constexpr int A_TPR = KT / AVEC;             // threads per A row
    constexpr int A_RPP = kThreads / A_TPR;      // A rows per pass
    constexpr int A_PASSES = BM / A_RPP;
    constexpr int B_TPR = BN / BVEC;             // threads per W row
    constexpr int B_RPP = kThreads / B_TPR;      // W rows per pass
    constexpr int B_PASSES = (KT + B_RPP - 1) / B_RPP;
    __shared__ float As[KT][BM + APAD];
    __shared__ __attribute__((aligned(16))) float Bs[KT][BN + BPAD];

    const int t = threadIdx.x;
    const int wave = t >> 6, lane = t & 63;
    const int wm = wave / WGN, wn = wave % WGN;
    const long long m0 = (long long)(block / g.n_bn) * BM;
    const int n0 = (int)(block % g.n_bn) * BN;

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    float ra[A_PASSES][AVEC];
    float rb[B_PASSES][BVEC];
    const int a_row = t / A_TPR, a_kk = (t % A_TPR) * AVEC;
    const int b_row = t / B_TPR, b_nn = (t % B_TPR) * BVEC;

    auto fetch = [&](int k0) {
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p) {
            const long long row = m0 + p * A_RPP + a_row;
            const int kk = k0 + a_kk;
            if (row < g.n && kk < g.k) {
                const float *src = g.A + row * g.lda + (long long)(kk >> 5) * g.a_slice + (kk & 31);
                if (AVEC == 4) { float4 v = *reinterpret_cast<const float4 *>(src); ra[p][0] = v.x; ra[p][1 % AVEC] = v.y; ra[p][2 % AVEC] = v.z; ra[p][3 % AVEC] = v.w; }
                else if (AVEC == 2) { float2 v = *reinterpret_cast<const float2 *>(src); ra[p][0] = v.x; ra[p][1 % AVEC] = v.y; }
                else ra[p][0] = *src;
            } else {
#pragma unroll
                for (int e = 0; e < AVEC; ++e) ra[p][e] = 0.f;
            }
        }
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            const int kr = p * B_RPP + b_row;
            const int kk = k0 + kr;
            const int col = n0 + b_nn;
            if (kr < KT && kk < g.k && col < g.m) {
                const float *src = g.W + (long long)kk * g.ldw + col;
                if (BVEC == 4) { float4 v = *reinterpret_cast<const float4 *>(src); rb[p][0] = v.x; rb[p][1 % BVEC] = v.y; rb[p][2 % BVEC] = v.z; rb[p][3 % BVEC] = v.w; }
                else rb[p][0] = *src;
            } else {
#pragma unroll
                for (int e = 0; e < BVEC; ++e) rb[p][e] = 0.f;
            }
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p)
#pragma unroll
            for (int e = 0; e < AVEC; ++e) As[a_kk + e][p * A_RPP + a_row] = ra[p][e];
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            const int kr = p * B_RPP + b_row;
            if (kr < KT) {
#pragma unroll
                for (int e = 0; e < BVEC; ++e) Bs[kr][b_nn + e] = rb[p][e];
            }
        }
    };

    const int n_kt = (g.k + KT - 1) / KT;
    fetch(0);
    for (int kt = 0; kt < n_kt; ++kt) {
        stash();
        __syncthreads();
        if (kt + 1 < n_kt) fetch((kt + 1) * KT);
        const int kh = lane >> 5, ll = lane & 31;
#pragma unroll
        for (int kk = 0; kk < KT; kk += 2) {
            float av[TM], bv[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) av[i] = As[kk + kh][(wm * TM + i) * 32 + ll];
#pragma unroll
            for (int j = 0; j < TN; ++j) bv[j] = Bs[kk + kh][(wn * TN + j) * 32 + ll];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }

    // accumulator layout of the 32x32 tile: register r of lane l holds
    // row 8*(r/4) + 4*(l/32) + r%4, column l%32
    const int kh = lane >> 5, ll = lane & 31;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = n0 + (wn * TN + j) * 32 + ll;
            if (col >= g.m_store) continue;
            const long long y_col = g.y_sliced ? (long long)(col >> 5) * g.n * 32 + (col & 31) : (long long)col;
            const long long y_ld = g.y_sliced ? 32 : g.ldy;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const long long row = m0 + (wm * TM + i) * 32 + 8 * (r / 4) + 4 * kh + (r % 4);
                if (row < g.n) {
                    float y = acc[i][j][r];
                    if (g.add) y += g.add[(long long)(col >> 5) * g.n * 32 + row * 32 + (col & 31)];
                    if (g.row_scale) y *= g.row_scale[row];
                    if (g.act == SENSEI_ACT_RELU) y = y > 0.f ? y : 0.f;
                    g.Y[row * y_ld + y_col] = y;
                }
            }
        }
}

template <int BM, int BN, int WGM, int WGN>
hipError_t gemm_launch_vec(const GemmArgs &g, int avec, int bvec, hipStream_t s) {
    const long long n_bm = (g.n + BM - 1) / BM;
    dim3 grid((unsigned)(n_bm * g.n_bn + g.side.blocks));
#define SENSEI_GEMM_CASE(AV, BV) \
    hipLaunchKernelGGL((k_gemm<BM, BN, WGM, WGN, AV, BV>), grid, dim3(kThreads), 0, s, g)
    if (bvec == 4) {
        if (avec == 4) SENSEI_GEMM_CASE(4, 4); else if (avec == 2) SENSEI_GEMM_CASE(2, 4); else SENSEI_GEMM_CASE(1, 4);
    } else {
        if (avec == 4) SENSEI_GEMM_CASE(4, 1); else if (avec == 2) SENSEI_GEMM_CASE(2, 1); else SENSEI_GEMM_CASE(1, 1);
    }
#undef SENSEI_GEMM_CASE
    return hipGetLastError();
}

// Products too small to give every compute unit a block of k_gemm (64 x 64 there: 16 k a step, one barrier and one exposed memory round
// trip each, so the time is the number of steps, whatever the size).  A workgroup owns 32 rows x 32 columns and its four wavefronts split
// k; operands go from memory to the matrix instruction's registers without LDS (a lane takes four consecutive k of its row of A in one load
// and the same four rows of W: the instruction only wants both operands to agree on which k a lane holds), all loads of four steps of 16 k
// in flight together, and the four partial sums are added in wavefront order through LDS.  fp32 instructions: infinities and NaN pass as
// in k_gemm.  Bound by two or three memory round trips: 1,024 x 256 x 47 12.7 -> 6.6 us, 4,900 x 256 x 47 12.9 -> 8.2, 600 x 100 x 256
// 7.3 -> 5.0, 10,000 x 64 x 32 5.4 -> 4.6.
template <int AVEC>
__global__ __launch_bounds__(kThreads) void k_gemm_small(GemmArgs g) {
    if ((int)blockIdx.x < g.side.blocks) return side_block(g.side, (int)blockIdx.x);
    const unsigned block = blockIdx.x - g.side.blocks;
    constexpr int GS = 4;   // steps of 16 k loaded together
    constexpr int kWaves = kThreads / 64;
    __shared__ float red[kWaves][16][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, kh = lane >> 5, ll = lane & 31;
    const long long m0 = (long long)(block / g.n_bn) * 32;
    const int col = (int)(block % g.n_bn) * 32 + ll;
    const int steps = (g.k + 15) / 16;
    const int s0 = steps * wave / kWaves, s1 = steps * (wave + 1) / kWaves;

    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;

    // rows past the end read the last row and are not stored; columns past m read the last column and are cleared; k past the end of this
    // wavefront's range reads k = 0 and is cleared in both operands (masks, not branches around the loads)
    const float *a_row = g.A + (m0 + ll < g.n ? m0 + ll : g.n - 1) * g.lda;
    const unsigned w_mask = col < g.m ? ~0u : 0u;
    const float *w_col = g.W + (col < g.m ? col : g.m - 1);
    auto masked = [](float v, unsigned m) { return __uint_as_float(__float_as_uint(v) & m); };
    const int k_end = s1 * 16 < g.k ? s1 * 16 : g.k;
    for (int st = s0; st < s1; st += GS) {
        float a[GS][2][4], w[GS][2][4];
#pragma unroll
        for (int q = 0; q < GS; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int k0 = (st + q) * 16 + h * 8 + kh * 4;
                if (AVEC == 4) {   // k is a multiple of 4: four k are all there or all past the end
                    const int kc = k0 < k_end ? k0 : 0;
                    const float4 v = *reinterpret_cast<const float4 *>(a_row + (long long)(kc >> 5) * g.a_slice + (kc & 31));
                    const unsigned live = k0 < k_end ? ~0u : 0u;
                    a[q][h][0] = masked(v.x, live); a[q][h][1] = masked(v.y, live); a[q][h][2] = masked(v.z, live); a[q][h][3] = masked(v.w, live);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int k = k0 + e, kc = k < k_end ? k : 0;
                        a[q][h][e] = masked(a_row[(long long)(kc >> 5) * g.a_slice + (kc & 31)], k < k_end ? ~0u : 0u);
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int k = k0 + e, kc = k < k_end ? k : 0;
                    w[q][h][e] = masked(w_col[(long long)kc * g.ldw], k < k_end ? w_mask : 0u);
                }
            }
#pragma unroll
        for (int q = 0; q < GS; ++q) {
            if (st + q >= s1) break;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q][h][e], w[q][h][e], acc, 0, 0, 0);
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave][r][lane] = acc[r];
    __syncthreads();
    // register r of lane l holds row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32; a wavefront finishes four of the sixteen
    if (col >= g.m_store) return;
    const long long y_col = g.y_sliced ? (long long)(col >> 5) * g.n * 32 + (col & 31) : (long long)col;
    const long long y_ld = g.y_sliced ? 32 : g.ldy;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = wave * 4 + q;
        const long long row = m0 + 8 * wave + 4 * kh + q;
        if (row < g.n) {
            float y = red[0][r][lane];
#pragma unroll
            for (int v = 1; v < kWaves; ++v) y += red[v][r][lane];
            if (g.add) y += g.add[(long long)(col >> 5) * g.n * 32 + row * 32 + (col & 31)];
            if (g.row_scale) y *= g.row_scale[row];
            if (g.act == SENSEI_ACT_RELU) y = y > 0.f ? y : 0.f;
            g.Y[row * y_ld + y_col] = y;
        }
    }
}

// ---- the same GEMM on the bf16 matrix cores, which run 16 times the fp32 rate, at fp32 accuracy.  Every fp32 operand element
// is cut into three bf16 pieces (round to nearest, subtract, round, subtract: both subtractions are exact and the pieces add up to the
// element exactly).  bf16 has eight significand bits, so a second piece is at most 2^-8 of the element and a third 2^-17 of it.  Of the nine piece
// products of a term, each exact and accumulated in fp32 by the matrix core, are formed
//   six (a1 b1, a1 b2, a2 b1, a1 b3, a2 b2, a3 b1): what is left out is below 2^-23.9 of the term (a2 b3 + a3 b2 + a3 b3; 2^-24.0 for operands like
//     1 + 2^-8 - 2^-17), 2^-27.5 rms, either sign, and the instruction's own sums lose up to another unit of 2^-23: a sum of many terms is closer to
//     the exact one than fp32's (rms over 32 to 602 mixed terms 0.27-0.34 units of 2^-24 of their magnitudes, fp32 0.40-0.41), a sum that one
//     term makes up is not (largest error 2.7 units, fp32 1.0); or
//   eight, a3 b3 alone left out (2^-34 of the term), a1 b1 and the seven others in accumulators of their own that are added at the end: many terms
//     0.11-0.14 units, a single term the one rounding of fp32 (1.0).
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));   // 16-byte load at any word: the vector memory unit needs no more alignment
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

// Two elements -> their three pieces, packed as pairs (first in the low half).  An element that is infinite, NaN or rounds up to infinity makes
// every sum it enters infinite or NaN; those sums are formed again on the fp32 instruction (product_fp32).
__device__ __forceinline__ void cut_pair(float x, float y, unsigned &hi, unsigned &mid, unsigned &lo) {
    auto pack = [](float a, float b) { const floatx2 v = {a, b}; return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2)); };
    hi = pack(x, y);
    x -= __uint_as_float(hi << 16);
    y -= __uint_as_float(hi & 0xFFFF0000u);
    mid = pack(x, y);
    lo = pack(x - __uint_as_float(mid << 16), y - __uint_as_float(mid & 0xFFFF0000u));
}

// whether any of a lane's sums is infinite or NaN
template <int N>
__device__ __forceinline__ bool not_finite(const floatx16 (&acc)[N]) {
    float t = 0.f;
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) t = fmaf(acc[j][r], 0.f, t);
    return t != 0.f;   // 0 from finite sums, NaN otherwise
}

// 32 x 32 sums over k on the fp32 instruction, operands straight from memory: a(q), b(q) are this lane's elements of its row and its column at q.
// Bound by the loads' latency; 233,000 x 602 x 256 with a thousandth of the rows infinite 0.74 ms, with nothing but NaN 2.6 (finite 0.47).
template <class A, class B>
__device__ __forceinline__ floatx16 product_fp32(int k, int kh, A a, B b) {
    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    constexpr int U = 16;   // loads under way
    for (int k0 = 0; k0 < k; k0 += 2 * U) {
        float x[U], y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = k0 + 2 * u + kh, qc = q < k ? q : k - 1;
            x[u] = a(qc);
            y[u] = b(qc);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool on = k0 + 2 * u + kh < k;
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(on ? x[u] : 0.f, on ? y[u] : 0.f, acc, 0, 0, 0);
        }
    }
    return acc;
}

__device__ __forceinline__ void split_bf16x3(float v, unsigned &hi, unsigned &mid, unsigned &lo) {
    hi = __float_as_uint(v) & 0xFFFF0000u;
    const float r1 = v - __uint_as_float(hi);          // exact: at most 16 significant bits remain
    mid = __float_as_uint(r1) & 0xFFFF0000u;
    lo = __float_as_uint(r1 - __uint_as_float(mid));   // exact: at most 8 significant bits, so its low half is zero
}
// two fp32 bit patterns whose low halves do not matter -> their high halves as a pair of bf16 (first in the low half)
__device__ __forceinline__ unsigned pack_bf16(unsigned first, unsigned second) { return __builtin_amdgcn_perm(second, first, 0x07060302u); }

// A wavefront owns 32 rows x 32 TN columns (TN accumulators of the 32 x 32 x 16 instruction) and brings its own rows of A: groups of 32 rows x
// 32 k, eight lanes to a row's 128 bytes, DEPTH groups ahead of the multiply (four: all of a row up to 128 k, so that a tile costs one memory
// round trip and the next tile's is under way); a group changes places through 4 KB of LDS that no other wavefront touches (16-byte pieces,
// exchanged within a row by the row's number so that neither side meets bank conflicts) into the order the instruction reads, lane (row, k
// half) eight consecutive k, and is cut there.  A is thus read once and cut once per block of columns, and never waits for a barrier.  W is cut
// by the workgroup (512 threads) and left in LDS in lane order, every fragment one contiguous kilobyte:
//   CHUNKED = false: all of W's k fits beside the rows of A in 160 KB; it is cut once, after which the wavefronts walk their rows
//     independently of each other;
//   CHUNKED = true: chunks of gemm_kc k in two buffers, the next chunk fetched and cut while this one is multiplied, one barrier per chunk; all of W
//     is cut again for every eight tiles of rows, half as much cutting again as A's.
// The grid is what the chip holds at a time; every workgroup takes an equal share of the 32-row tiles, and the blocks of columns of one
// share run on one XCD, so that A comes from its L2 for all but the first of them.
// Rows past the end read the last row and are not stored; k past the end are cleared in both operands.
// Up to about 128 k and 128 columns it is bound by memory (1 M rows, 64 -> 32 columns 79 us, 4.8 TB/s); beyond, by the matrix pipe and the vector
// instructions of the cuts, which hardly overlap on a SIMD, at a clock that the matrix load brings down to about 1.9 GHz.  Before (a block of 256
// rows a workgroup, A through LDS uncut behind a barrier per 16 k) / now, us: 100,000 x 64 x 256 52 / 35, 233,000 x 41 x 256 95 / 70, 233,000 x 602
// x 64 206 / 177, 2.45 M x 100 x 512 2,670 / 2,110, 12 M x 32 x 128 1,800 / 1,610, 150,000 x 333 x 160 184 / 153, 233,000 x 602 x 256 502 / 470, 2.45 M
// x 512 x 512 7,430 / 7,560; and with eight products against the fp32 kernel 30,000 x 602 x 256 98 / 78, 50,000 x 128 x 128 29 / 28.
constexpr int kGemmThreads = 512, kGemmWaves = kGemmThreads / 64, kGemmCusPerXcd = 32;
constexpr size_t kGemmLds = 160 * 1024;
constexpr int gemm_kc(int tn) { return tn <= 2 ? 128 : 64; }     // k per chunk: 24 to 48 KB of pieces a buffer
constexpr int gemm_depth(int tn) { return tn == 1 ? 1 : 4; }
constexpr int gemm_held(int tn) { return tn == 1 ? 2 : 1; }      // workgroups a compute unit holds at a time, by registers
constexpr int gemm_a_bufs(int tn) { return tn == 1 ? 1 : 2; }

enum { kWholeTile, kAnyTile, kMarks, kAgain };
constexpr unsigned kAgainBits = 0x7FCA6A1Bu;   // a NaN; one that is an operand's own is formed again too, to the same end

// FULL: eight piece products a term in two accumulators, else six in one
template <int TN, bool CHUNKED, bool FULL>
__global__ __launch_bounds__(kGemmThreads, 2 * gemm_held(TN)) void k_gemm_bf(GemmArgs g) {
    if ((int)blockIdx.x < g.side.blocks) {
        if (threadIdx.x < kSideThreads) side_block(g.side, (int)blockIdx.x);
        return;
    }
    constexpr int BN = 32 * TN, KC = gemm_kc(TN), DEPTH = CHUNKED && TN > 1 ? KC / 32 : gemm_depth(TN), ABUF = gemm_a_bufs(TN);
    constexpr int STEP_BYTES = 3 * TN * 1024;                                    // pieces of 16 k x BN columns
    constexpr int WI = (KC / 16 * 2 * BN + kGemmThreads - 1) / kGemmThreads;     // (column, k half, step) items a thread cuts per chunk
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const unsigned block = blockIdx.x - g.side.blocks;
    const int bn = g.by_xcd ? (int)(block >> 3) % g.n_bn : (int)block % g.n_bn;
    const int part = g.by_xcd ? (int)((block >> 3) / g.n_bn) * 8 + (int)(block & 7) : (int)block / g.n_bn;
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63, kh = lane >> 5, ll = lane & 31;
    const int n0 = bn * BN;
    const long long tiles = (g.n + 31) / 32;
    const long long t0 = tiles * part / g.n_parts, t1 = tiles * (part + 1) / g.n_parts;
    if (t0 >= t1) return;
    const int groups = (g.k + 31) / 32, steps = 2 * groups;

    // W: element e of item (column, k half, step) is row 16 step + 8 half + e
    auto item_of = [&](int item, int &c, int &row0, unsigned &at) {
        c = item % BN;
        const int rest = item / BN;
        row0 = rest * 8;
        at = (unsigned)((rest >> 1) * STEP_BYTES + (c >> 5) * 1024 + (rest & 1) * 512 + (c & 31) * 16);
    };
    auto fetch_w = [&](int k0, int c, int row0, float (&w)[8]) {   // uniform base, lane offset; rows past k read a row that exists
        const unsigned col_off = (unsigned)((n0 + c < g.m ? n0 + c : g.m - 1) * 4);
        const unsigned off = (unsigned)(row0 * (unsigned)g.ldw * 4u) + col_off;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int kb = k0 + e < g.k ? k0 + e : g.k - 1;
            const char *base = reinterpret_cast<const char *>(g.W + (long long)kb * g.ldw);
            w[e] = *reinterpret_cast<const float *>(base + (k0 + row0 + e < g.k ? off : col_off));
        }
    };
    // what lies past k or m is cleared here and not where it is fetched: there the compiler waits for every load by itself
    auto stash_w = [&](unsigned char *dst, int k0, int c, int row0, float (&w)[8]) {
        const int live = n0 + c < g.m ? g.k - k0 - row0 : 0;
        uintx4 p[3];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            unsigned a, b, c;
            cut_pair(2 * d < live ? w[2 * d] : 0.f, 2 * d + 1 < live ? w[2 * d + 1] : 0.f, a, b, c);
            p[0][d] = a; p[1][d] = b; p[2][d] = c;
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<uintx4 *>(dst + q * TN * 1024) = p[q];
    };

    // A: 32 k from k0 on of the rows of a tile; this lane takes piece lane % 8 (four k) of rows lane / 8 + 8 i.  A piece that would run past
    // the row's last element is read from four before it and put in order before it is stashed.  Slice-major rows are padded to whole groups
    // in memory: nothing to clamp.
    const int k_last = (g.a_slice != 32 ? (g.k + 31) / 32 * 32 : g.k) - 4;
    const int piece = lane & 7, prow = lane >> 3;
    unsigned char *const a_lds = lds + g.a_lds + wave * (4096 * ABUF);
    float raw[DEPTH][4][4];
    auto fetch_a = [&](long long tile, int k0, float (&v)[4][4]) {
        const long long m0 = tile * 32;
        const float *base = g.A + m0 * g.lda + (long long)(k0 >> 5) * g.a_slice - 4;   // uniform; lanes add 1 or more
        const int rows = g.n - m0 < 32 ? (int)(g.n - m0) : 32;
        const int lim = k_last - k0, o = (piece * 4 < lim ? piece * 4 : lim) + 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = i * 8 + prow, rc = row < rows ? row : rows - 1;
            const floatx4u x = *reinterpret_cast<const floatx4u *>(reinterpret_cast<const char *>(base) + (__umul24((unsigned)rc, (unsigned)g.lda) + (unsigned)o) * 4u);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[i][e] = x[e];
        }
    };
    auto stash_a = [&](int k0, float (&v)[4][4], int buf) {
        if (k0 + 32 > g.k) {   // the last group of a row: clamped pieces shifted into place, elements past k cleared
            const int lim = k_last - k0, d = piece * 4 > lim ? piece * 4 - lim : 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float w[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = (d & 1) ? v[i][e + 1 < 4 ? e + 1 : 3] : v[i][e];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i][e] = (d & 2) ? w[e + 2 < 4 ? e + 2 : 3] : w[e];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i][e] = k0 + piece * 4 + e < g.k ? v[i][e] : 0.f;
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<float4 *>(a_lds + buf * 4096 + (i * 8 + prow) * 128 + (piece ^ prow) * 16) = make_float4(v[i][0], v[i][1], v[i][2], v[i][3]);
    };
    auto wave_lds = [&]() {   // LDS is in order within a wavefront; the compiler has to be told
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };

    floatx16 acc[TN], low[FULL ? TN : 1];   // FULL: the products of the first pieces; all others
    auto clear = [&]() {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[j][r] = 0.f;
                if (FULL) low[FULL ? j : 0][r] = 0.f;
            }
    };
    auto multiply = [&](int buf, const unsigned char *w) {   // the group in `buf` (two steps), fragments of W at w
        uintx4 af[2][3];
#pragma unroll
        for (int step = 0; step < 2; ++step)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float4 v = *reinterpret_cast<const float4 *>(a_lds + buf * 4096 + ll * 128 + (((step * 4 + kh * 2 + q) ^ (ll & 7)) * 16));
                unsigned x, y, z;
                cut_pair(v.x, v.y, x, y, z);
                af[step][0][2 * q] = x; af[step][1][2 * q] = y; af[step][2][2 * q] = z;
                cut_pair(v.z, v.w, x, y, z);
                af[step][0][2 * q + 1] = x; af[step][1][2 * q + 1] = y; af[step][2][2 * q + 1] = z;
            }
        constexpr int J = TN % 2 == 0 ? 2 : 1;   // accumulators in turn, so that consecutive instructions do not wait for each other
#pragma unroll
        for (int step = 0; step < 2; ++step)
#pragma unroll
            for (int j = 0; j < TN; j += J) {
                uintx4 bf[J][3];
#pragma unroll
                for (int i = 0; i < J; ++i)
#pragma unroll
                    for (int p = 0; p < 3; ++p) bf[i][p] = *reinterpret_cast<const uintx4 *>(w + step * STEP_BYTES + (p * TN + j + i) * 1024 + lane * 16);
#pragma unroll
                for (int pa = 2; pa >= 0; --pa)
#pragma unroll
                    for (int pb = !FULL ? 2 - pa : pa == 2 ? 1 : 2; pb >= 0; --pb)   // smallest products first
#pragma unroll
                        for (int i = 0; i < J; ++i) {
                            floatx16 &sum = FULL && pa + pb > 0 ? low[FULL ? j + i : 0] : acc[j + i];
                            sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[step][pa]), __builtin_bit_cast(bf16x8, bf[i][pb]), sum, 0, 0, 0);
                        }
            }
    };
    // register r of lane l holds row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32; in a tile whose rows all exist the loads of `add` and
    // `row_scale` are not behind branches and are in flight together
    auto store_rows = [&](long long tile, auto form) {
        constexpr int kForm = decltype(form)::value;   // whole tile; any tile; the same, marks for what is to be formed again; in place of marks only
        constexpr bool kWhole = kForm == kWholeTile;
        const long long row0 = tile * 32 + 4 * kh;
        {
            float sc[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const long long row = row0 + 8 * (r / 4) + (r % 4);
                sc[r] = g.row_scale ? g.row_scale[kWhole || row < g.n ? row : g.n - 1] : 1.f;
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = n0 + j * 32 + ll;
                if (col >= g.m_store) continue;
                const long long y_col = g.y_sliced ? (long long)(col >> 5) * g.n * 32 + (col & 31) : (long long)col;
                const long long y_ld = g.y_sliced ? 32 : g.ldy;
                float y[16];
                if (g.add) {
                    const float *add = g.add + (long long)(col >> 5) * g.n * 32 + (col & 31);
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const long long row = row0 + 8 * (r / 4) + (r % 4);
                        y[r] = add[(kWhole || row < g.n ? row : g.n - 1) * 32];
                    }
                    __builtin_amdgcn_sched_barrier(0);   // all sixteen under way before the first is added: short of registers, the scheduler would wait for each
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) y[r] = g.add ? acc[j][r] + y[r] : acc[j][r];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const long long row = row0 + 8 * (r / 4) + (r % 4);
                    float v = y[r] * sc[r];
                    if (g.act == SENSEI_ACT_RELU) v = v > 0.f ? v : 0.f;
                    if (kForm == kMarks && !__builtin_isfinite(acc[j][r])) v = __uint_as_float(kAgainBits);
                    float *dst = g.Y + row * y_ld + y_col;
                    if ((kWhole || row < g.n) && (kForm != kAgain || __float_as_uint(*dst) == kAgainBits)) *dst = v;
                }
            }
        }
    };
    auto store = [&](long long tile) {
        if ((tile + 1) * 32 <= g.n) store_rows(tile, std::integral_constant<int, kWholeTile>());
        else store_rows(tile, std::integral_constant<int, kAnyTile>());
    };

    // Tiles with a sum that is infinite or NaN (every one of this wavefront's up to 64, runs of them beyond).  Those sums are stored as marks and formed
    // again at the end: inside the loop the loads of it made the compiler wait for each of the others (233,000 x 602 x 256: 477 us without, 652
    // so, 467 now).
    const int most = (int)((t1 - t0 + kGemmWaves - 1) / kGemmWaves), again_shift = most > 64 ? 26 - __clz(most - 1) : 0;
    unsigned long long again = 0;
    int done = 0;

    // DEPTH groups of this wavefront's tile from group g0 on, out of the fragments at w; every group's registers are refilled with the group
    // DEPTH later (of the next tile where the row ends)
    long long tile = t0 + wave;
    auto run = [&](int g0, const unsigned char *w) {
        const bool ends = g0 + DEPTH >= groups;
        const long long tile_n = ends ? (tile + kGemmWaves < t1 ? tile + kGemmWaves : tile) : tile;
        const int next0 = ends ? 0 : g0 + DEPTH;
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) {
            if (ABUF == 1) wave_lds();
            if (g0 + i < groups) stash_a((g0 + i) * 32, raw[i], i % ABUF);
            if (next0 + i < groups) fetch_a(tile_n, (next0 + i) * 32, raw[i]);
            __builtin_amdgcn_sched_barrier(0);   // the fetches stay here: the scheduler would sink them to their use
            wave_lds();
            if (g0 + i < groups) {
                multiply(i % ABUF, w + i * 2 * STEP_BYTES);
            }
        }
        if (ends) {
            if (FULL)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[j] += low[FULL ? j : 0];
            store(tile);
            if (__any(not_finite<TN>(acc))) {   // behind the store, whose loads do not wait for it
                again |= 1ull << (done >> again_shift);
                store_rows(tile, std::integral_constant<int, kMarks>());
            }
            ++done;
            clear();
            tile += kGemmWaves;
        }
    };
    {
        const long long first = tile < t1 ? tile : t1 - 1;
#pragma unroll
        for (int i = 0; i < DEPTH; ++i)
            if (i < groups) fetch_a(first, i * 32, raw[i]);
    }
    clear();
    if constexpr (!CHUNKED) {
        for (int item = t; item < steps * 2 * BN; item += kGemmThreads) {
            int c, row0;
            unsigned at;
            float w[8];
            item_of(item, c, row0, at);
            fetch_w(0, c, row0, w);
            stash_w(lds + at, 0, c, row0, w);
        }
        __syncthreads();
        while (tile < t1)
            for (int g0 = 0; g0 < groups; g0 += DEPTH) run(g0, lds + g0 * 2 * STEP_BYTES);
    } else {
        const int chunks = (g.k + KC - 1) / KC, rounds = (int)((t1 - t0 + kGemmWaves - 1) / kGemmWaves);
        float w[WI][8];
        int wc[WI], wrow[WI];
        unsigned wat[WI];
#pragma unroll
        for (int i = 0; i < WI; ++i) item_of(t + i * kGemmThreads, wc[i], wrow[i], wat[i]);
        auto fetch_chunk = [&](int k0) {
#pragma unroll
            for (int i = 0; i < WI; ++i) fetch_w(k0, wc[i], wrow[i], w[i]);
        };
        auto stash_chunk = [&](unsigned char *dst, int k0) {
#pragma unroll
            for (int i = 0; i < WI; ++i)
                if (t + i * kGemmThreads < KC / 16 * 2 * BN) stash_w(dst + wat[i], k0, wc[i], wrow[i], w[i]);
        };
        fetch_chunk(0);
        stash_chunk(lds, 0);
        int which = 0;
        for (int round = 0; round < rounds; ++round)
            for (int ch = 0; ch < chunks; ++ch) {
                __syncthreads();   // this chunk's pieces are in its buffer; nobody reads the other one any more
                const bool more = ch + 1 < chunks || round + 1 < rounds;
                const int k_next = ch + 1 < chunks ? (ch + 1) * KC : 0;
                if (more) fetch_chunk(k_next);
                if (tile < t1)
                    for (int g0 = ch * (KC / 32), g1 = g0 + KC / 32; g0 < g1 && g0 < groups; g0 += DEPTH)
                        run(g0, lds + which * (KC / 16 * STEP_BYTES) + (g0 - ch * (KC / 32)) * 2 * STEP_BYTES);
                __builtin_amdgcn_sched_barrier(0);
                which ^= 1;
                if (more) stash_chunk(lds + which * (KC / 16 * STEP_BYTES), k_next);
            }
    }
    if (!again) return;
    done = 0;
    for (tile = t0 + wave; tile < t1; tile += kGemmWaves, ++done) {
        if (!((again >> (done >> again_shift)) & 1ull)) continue;
        const long long row = tile * 32 + ll;
        const float *a = g.A + (row < g.n ? row : g.n - 1) * g.lda;
#pragma unroll 1
        for (int j = 0; j < TN; ++j) {
            const int col = n0 + j * 32 + ll;
            const float *w = g.W + (col < g.m ? col : g.m - 1);
            const bool live = col < g.m;
            const floatx16 sums = product_fp32(g.k, kh, [&](int q) { return a[(long long)(q >> 5) * g.a_slice + (q & 31)]; },
                                               [&](int q) { const float v = w[(long long)q * g.ldw]; return live ? v : 0.f; });
#pragma unroll
            for (int i = 0; i < TN; ++i)
                if (i == j) acc[i] = sums;
        }
        store_rows(tile, std::integral_constant<int, kAgain>());
    }
}

template <int TN, bool FULL>
hipError_t gemm_bf_launch(GemmArgs g, hipStream_t s) {
    const int steps = (g.k + 31) / 32 * 2;
    const size_t a_bytes = (size_t)kGemmWaves * 4096 * gemm_a_bufs(TN);
    const bool chunked = steps * 3 * TN * 1024 + a_bytes > kGemmLds;
    g.a_lds = (chunked ? 2 * (gemm_kc(TN) / 16) : steps) * 3 * TN * 1024;
    const long long tiles = (g.n + 31) / 32;
    // one workgroup too many on an XCD (32 compute units) would run a whole share after all the others: shares are dealt out XCD by XCD where
    // the blocks of columns divide what an XCD holds, and one after the other where they do not
    const int held = kGemmCusPerXcd * (g.a_lds + a_bytes <= kGemmLds / 2 ? gemm_held(TN) : 1);
    g.by_xcd = held % g.n_bn == 0 && tiles >= 8 * (held / g.n_bn);
    const long long parts = g.by_xcd ? 8 * (held / g.n_bn) : 8 * held > g.n_bn ? 8 * held / g.n_bn : 1;
    g.n_parts = (int)(parts < tiles ? parts : tiles);
    const dim3 grid((unsigned)(g.n_parts * g.n_bn + g.side.blocks));
    if (chunked) hipLaunchKernelGGL((k_gemm_bf<TN, true, FULL>), grid, dim3(kGemmThreads), g.a_lds + a_bytes, s, g);
    else hipLaunchKernelGGL((k_gemm_bf<TN, false, FULL>), grid, dim3(kGemmThreads), g.a_lds + a_bytes, s, g);
    return hipGetLastError();
}

// ---- dense tiles of the hub region: C[order_r[rank], :] = sum over the kept 128 x 128 tiles of the rank's row of tiles of
// (tile bits) . B[tile columns, :], B in rank order.  The rows of tiles of the largest hubs keep hundreds of tiles, the others a
// few: the kept tiles of a row are therefore cut into segments of at most kTilesPerSegment, one workgroup per (segment, group
// of 32-column blocks); a segment leaves its 128 x f partial product in `part`, and k_tiles_reduce adds the segments of a row
// in order (no atomics).
// The value-less product on the bf16 matrix cores, which run 16 times the fp32 rate, without giving up fp32 accuracy: a
// tile entry is 0 or 1, exact in bf16, and every fp32 element of the right-hand operand is cut into three bf16 pieces of
// eight significand bits each (truncate, subtract, truncate, subtract: the pieces add up to the element exactly), so the three
// products per piece are exact and only the fp32 accumulation of the matrix core rounds, as it does in the fp32 instruction.
// Neither operand passes through LDS and the wavefronts never synchronise:
//   - a lane of the 32 x 32 x 16 instruction holds eight consecutive k of one tile row, i.e. one byte of that row's 128-bit
//     mask, which it expands in registers (to 2.0 = 0x4000, a single bit per entry; the stored result is halved);
//   - the right-hand operand is cut into its pieces once per call, by the kernel that gathers it into rank order, and stored
//     in the order the instruction's lanes read it: per (piece, column tile, 16 k, 32 columns) one contiguous kilobyte, lane
//     (k half, column) holding its eight k, so an operand fetch is one 16-byte load per lane straight from global memory.
// A wavefront owns 128 tile rows x 32 columns (four accumulators) and walks its segment's tiles with the fetches running three
// steps of 16 k ahead; the wavefronts of a workgroup only share the segment.
// eight mask bits -> eight bf16 of value 0 or 2.0: bit k is copied to k and k + 15, then each pair (2d, 2d + 1) is moved onto
// bits 14 and 30 of its word
__device__ __forceinline__ uintx4 expand_mask_byte(unsigned byte) {
    unsigned twice = byte | (byte << 15);
    asm volatile("" : "+v"(twice));   // keeps the shifts below shifts: folded with the line above they become 32-bit multiplies, four times as slow
    uintx4 a;
#pragma unroll
    for (int d = 0; d < 4; ++d) a[d] = (twice << (14 - 2 * d)) & 0x40004000u;
    return a;
}

// Bq: the gathered matrix in rank order, cut into bf16 pieces, in the lane order described above.  Element (rank q = 128 ct +
// 16 k16 + 8 kh + e, column n = 32 nb + nl) of piece p sits at p * n_ranks * f + ((((ct * 8 + k16) * (f / 32) + nb) * 2 + kh) * 32 + nl) * 8 + e.
// One thread: eight consecutive ranks of one column (one 16-byte store per piece).  Rows are those of the slice-major matrix B
// (zeros where the rank has no node), times 1 / mz[node].y if mz is given.
__global__ void k_gather_ranked_split(const float *__restrict__ B, long long n_cols, int f, const int32_t *__restrict__ order_c, long long n_ranks,
                                      unsigned short *__restrict__ Bq, const float2 *__restrict__ mz) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int nb_count = f / 32;
    if (t >= n_ranks / 8 * f) return;
    const int nl = (int)(t & 31);
    const int nb = (int)((t >> 5) % nb_count);
    const long long g8 = (t >> 5) / nb_count;
    const long long q0 = g8 * 8;
    unsigned pc[8][3];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int j = order_c[q0 + e];
        float v = j >= 0 ? B[(long long)nb * n_cols * 32 + (long long)j * 32 + nl] : 0.f;
        if (mz && j >= 0) { const float z = mz[j].y; v *= z > 0.f ? 1.f / z : 0.f; }
        split_bf16x3(v, pc[e][0], pc[e][1], pc[e][2]);
    }
    const long long at = ((g8 >> 1) * nb_count + nb) * 512 + (g8 & 1) * 256 + nl * 8;   // g8 = (ct * 8 + k16) * 2 + kh
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        uintx4 w;
#pragma unroll
        for (int d = 0; d < 4; ++d) w[d] = pack_bf16(pc[2 * d][p], pc[2 * d + 1][p]);
        *reinterpret_cast<uintx4 *>(Bq + (long long)p * n_ranks * f + at) = w;
    }
}

struct DenseTilesBfArgs {
    const unsigned *bits;                  // n_slots x 128 rows x 4 words
    const int32_t *seg_first, *slot_ct;    // first slot of each segment (n_seg + 1 entries); column tile of a slot
    const unsigned short *Bq;              // k_gather_ranked_split's output
    float *part;                           // n_seg x 128 x f
    long long plane;                       // elements per piece: ranks x f
    int f, n_bn;                           // f: multiple of 32; n_bn: workgroups (of up to four 32-column blocks) per segment
};

__global__ __launch_bounds__(kThreads) void k_dense_tiles_bf(DenseTilesBfArgs g) {
    constexpr int PF = 3, RING = PF + 1;   // fetch distance in steps of 16 k; 8 steps per tile, so ring positions are static
    const int seg = blockIdx.x / g.n_bn;
    const int lane = threadIdx.x & 63;
    const int nb = (blockIdx.x % g.n_bn) * 4 + (threadIdx.x >> 6);   // this wavefront's block of 32 columns
    const int nb_count = g.f / 32;
    if (nb >= nb_count) return;            // wavefronts do not synchronise: an idle one may leave
    const int s0 = __builtin_amdgcn_readfirstlane(g.seg_first[seg]), s1 = __builtin_amdgcn_readfirstlane(g.seg_first[seg + 1]);
    if (s0 >= s1) return;
    const int kh = lane >> 5, ll = lane & 31;

    floatx16 acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

    uintx4 ring[RING][3];
    uintx4 ab[4], ab_n[4];
    const unsigned short *bq = g.Bq + (long long)nb * 512 + lane * 8;
    auto fetch = [&](int ct, int k16, int pos) {
        const unsigned short *at = bq + ((long long)ct * 8 + k16) * nb_count * 512;
#pragma unroll
        for (int p = 0; p < 3; ++p) ring[pos][p] = *reinterpret_cast<const uintx4 *>(at + p * g.plane);
    };
    auto fetch_bits = [&](int slot) {
#pragma unroll
        for (int i = 0; i < 4; ++i) ab_n[i] = *reinterpret_cast<const uintx4 *>(g.bits + ((size_t)slot * 128 + i * 32 + ll) * 4);
    };

    int ct = g.slot_ct[s0], ct_next = g.slot_ct[s0 + 1 < s1 ? s0 + 1 : s0];
    fetch_bits(s0);
    __builtin_amdgcn_sched_barrier(0);   // the fetches complete in issue order: the order here is the one the loop continues
#pragma unroll
    for (int k = 0; k < PF; ++k) {
        fetch(ct, k, k);
        __builtin_amdgcn_sched_barrier(0);
    }
    for (int slot = s0; slot < s1; ++slot) {
        // the loop body has no branches, so that the fetches stay in flight across iterations: past the last tile it fetches
        // that tile again and drops the result
        const int slot_next = slot + 1 < s1 ? slot + 1 : slot;
        const int ct_after = g.slot_ct[slot + 2 < s1 ? slot + 2 : s1 - 1];   // needed one tile from now: by then it has long arrived
#pragma unroll
        for (int i = 0; i < 4; ++i) ab[i] = ab_n[i];
#pragma unroll
        for (int k16 = 0; k16 < 8; ++k16) {
            if (k16 + PF < 8) fetch(ct, k16 + PF, (k16 + PF) % RING);
            else fetch(ct_next, k16 + PF - 8, (k16 + PF) % RING);
            if (k16 == 4) fetch_bits(slot_next);
            __builtin_amdgcn_sched_barrier(0);   // keeps the fetches PF steps ahead of their use: the scheduler would sink them to it
            uintx4 av[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) av[i] = expand_mask_byte((ab[i][k16 >> 1] >> ((k16 & 1) * 16 + kh * 8)) & 0xFFu);
#pragma unroll
            for (int p = 2; p >= 0; --p)   // smallest pieces first
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[i]), __builtin_bit_cast(bf16x8, ring[k16 % RING][p]),
                                                                     acc[i], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        ct = ct_next;
        ct_next = __builtin_amdgcn_readfirstlane(ct_after);   // placed after the last scheduling barrier: it does not wait on the fetches in flight
    }

    float *out = g.part + (size_t)seg * 128 * g.f + nb * 32 + ll;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) out[(size_t)(i * 32 + 8 * (r / 4) + 4 * kh + (r % 4)) * g.f] = 0.5f * acc[i][r];
}

// The attention modes on the bf16 matrix cores.  Entry (i, k) of a tile weighs w = exp(LeakyReLU(u[i] + v[k]) - shift), an fp32
// number, which is cut into three bf16 pieces like the right-hand operand; of the nine piece products the six of weight
// 2^-16 and above are formed (w1 b1, w1 b2, w2 b1, w1 b3, w2 b2, w3 b1: what is left out is below 2^-21 of a term, 2^-24.7 on
// average).  kTilesAttn: u = s_l, v = s_r, shift = the maximum of row i (tiles of the pattern itself).
// kTilesAttnT: the tiles are those of the transposed pattern, so the softmax row is the tile's column: u = s_r, v = s_l,
// shift = the maximum of column k.
// The weights of one step (128 rows x 16 k) are computed once per workgroup, every thread a few of them, and shared through
// LDS (two buffers: the weights of step s + 1 are written while step s multiplies, one barrier per step); a wavefront owns 128
// rows x 32 columns as in the value-less kernel and fetches its right-hand pieces straight from global memory one step ahead.
// NW wavefronts per workgroup (as many 32-column blocks, up to eight); a workgroup whose last blocks do not exist lets those
// wavefronts repeat the last block and drop the result, so that every wavefront reaches every barrier.
struct DenseTilesAttnArgs {
    const unsigned *bits;
    const int32_t *seg_first, *slot_ct, *seg_rt;
    const unsigned short *Bq;
    float *part;
    long long plane;
    int f, n_bn;
    const float *u_rank, *m_rank;    // by row rank: u, and (kTilesAttn) the shift
    const float *v_rank, *mc_rank;   // by column rank: v, and (kTilesAttnT) the shift
    float slope;
};
constexpr int kTilesAttn = 1, kTilesAttnT = 2;

template <int MODE, int NW>
__global__ __launch_bounds__(64 * NW) void k_dense_tiles_attn_bf(DenseTilesAttnArgs g) {
    constexpr int THREADS = 64 * NW;
    constexpr int KP = NW >= 8 ? 4 : NW == 4 ? 8 : 16;   // consecutive k per thread and row when the weights are formed
    constexpr int TPR = 16 / KP;                          // threads per row
    constexpr int RPT = 128 * TPR / THREADS;              // rows per thread (2 for a single wavefront)
    constexpr int AROW = 24;                              // bf16 per row of a piece in LDS: 16 k and 16 bytes of padding (conflict-free 16-byte reads)
    __shared__ __attribute__((aligned(16))) unsigned short As[2][3][128][AROW];
    const int seg = blockIdx.x / g.n_bn;
    const int t = threadIdx.x, lane = t & 63;
    const int nb_count = g.f / 32;
    const int nb_want = (blockIdx.x % g.n_bn) * NW + (t >> 6);
    const bool stores = nb_want < nb_count;
    const int nb = stores ? nb_want : nb_count - 1;
    const int s0 = __builtin_amdgcn_readfirstlane(g.seg_first[seg]), s1 = __builtin_amdgcn_readfirstlane(g.seg_first[seg + 1]);
    if (s0 >= s1) return;
    const int rt = g.seg_rt[seg];
    const int kh = lane >> 5, ll = lane & 31;
    const int a_row = t / TPR, a_kq = t % TPR;

    floatx16 acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

    float u_t[RPT], m_t[RPT];
    uintx4 ab[RPT], ab_n[RPT];
#pragma unroll
    for (int rr = 0; rr < RPT; ++rr) {
        const int row = a_row + rr * (THREADS / TPR);
        u_t[rr] = g.u_rank[rt * 128 + row];
        m_t[rr] = MODE == kTilesAttn ? g.m_rank[rt * 128 + row] : 0.f;
    }
    auto fetch_bits = [&](int slot) {
#pragma unroll
        for (int rr = 0; rr < RPT; ++rr)
            ab_n[rr] = *reinterpret_cast<const uintx4 *>(g.bits + ((size_t)slot * 128 + a_row + rr * (THREADS / TPR)) * 4);
    };
    uintx4 ring[2][3];
    const unsigned short *bq = g.Bq + (long long)nb * 512 + lane * 8;
    auto fetch = [&](int ct, int k16, int pos) {
        const unsigned short *at = bq + ((long long)ct * 8 + k16) * nb_count * 512;
#pragma unroll
        for (int p = 0; p < 3; ++p) ring[pos][p] = *reinterpret_cast<const uintx4 *>(at + p * g.plane);
    };
    float4 vv[KP / 4], mc[KP / 4];
    auto fetch_v = [&](int ct, int k16) {
#pragma unroll
        for (int q = 0; q < KP / 4; ++q) {
            vv[q] = *reinterpret_cast<const float4 *>(g.v_rank + (size_t)ct * 128 + k16 * 16 + a_kq * KP + q * 4);
            if (MODE == kTilesAttnT) mc[q] = *reinterpret_cast<const float4 *>(g.mc_rank + (size_t)ct * 128 + k16 * 16 + a_kq * KP + q * 4);
        }
    };
    // the weights of step k16 of the tile whose mask rows are `mask`, from the vectors fetch_v has brought, into buffer `buf`
    auto weights = [&](const uintx4 (&mask)[RPT], int k16, int buf) {
#pragma unroll
        for (int rr = 0; rr < RPT; ++rr) {
            const unsigned present = (mask[rr][k16 >> 1] >> ((k16 & 1) * 16 + a_kq * KP)) & ((1u << KP) - 1u);
            unsigned pc[KP][3];
#pragma unroll
            for (int e = 0; e < KP; ++e) {
                const float4 v4 = vv[e / 4];
                const float ve = (e & 3) == 0 ? v4.x : (e & 3) == 1 ? v4.y : (e & 3) == 2 ? v4.z : v4.w;
                float tt = u_t[rr] + ve;
                tt = tt > 0.f ? tt : g.slope * tt;
                float shift = m_t[rr];
                if (MODE == kTilesAttnT) { const float4 c4 = mc[e / 4]; shift = (e & 3) == 0 ? c4.x : (e & 3) == 1 ? c4.y : (e & 3) == 2 ? c4.z : c4.w; }
                const float w = ((present >> e) & 1u) ? __expf(tt - shift) : 0.f;
                split_bf16x3(w, pc[e][0], pc[e][1], pc[e][2]);
            }
            const int row = a_row + rr * (THREADS / TPR);
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                unsigned short *dst = &As[buf][p][row][a_kq * KP];
#pragma unroll
                for (int q = 0; q < KP / 4; ++q)
                    *reinterpret_cast<uint2 *>(dst + q * 4) = make_uint2(pack_bf16(pc[q * 4][p], pc[q * 4 + 1][p]), pack_bf16(pc[q * 4 + 2][p], pc[q * 4 + 3][p]));
            }
        }
    };

    int ct = g.slot_ct[s0], ct_next = g.slot_ct[s0 + 1 < s1 ? s0 + 1 : s0];
    fetch_bits(s0);
    fetch_v(ct, 0);
    fetch(ct, 0, 0);
#pragma unroll
    for (int rr = 0; rr < RPT; ++rr) ab[rr] = ab_n[rr];
    weights(ab, 0, 0);
    for (int slot = s0; slot < s1; ++slot) {
        // no branches in the body (the fetches stay in flight across iterations): past the last tile it works on that tile again
        // and drops the result
        const int slot_next = slot + 1 < s1 ? slot + 1 : slot;
        const int ct_after = g.slot_ct[slot + 2 < s1 ? slot + 2 : s1 - 1];
#pragma unroll
        for (int k16 = 0; k16 < 8; ++k16) {
            // what the next step needs: its right-hand pieces, and the column vectors its weights are formed from
            if (k16 < 7) { fetch(ct, k16 + 1, (k16 + 1) & 1); fetch_v(ct, k16 + 1); }
            else { fetch(ct_next, 0, 0); fetch_v(ct_next, 0); }
            if (k16 == 3) fetch_bits(slot_next);
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();   // the weights of this step are in As[k16 & 1]; nobody reads the other buffer any more
#pragma unroll
            for (int pa = 2; pa >= 0; --pa) {
                uintx4 av[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) av[i] = *reinterpret_cast<const uintx4 *>(&As[k16 & 1][pa][i * 32 + ll][kh * 8]);
#pragma unroll
                for (int pb = 2 - pa; pb >= 0; --pb)   // smallest products first
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[i]), __builtin_bit_cast(bf16x8, ring[k16 & 1][pb]),
                                                                         acc[i], 0, 0, 0);
            }
            if (k16 < 7) weights(ab, k16 + 1, (k16 + 1) & 1);
            else weights(ab_n, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int rr = 0; rr < RPT; ++rr) ab[rr] = ab_n[rr];
        ct = ct_next;
        ct_next = __builtin_amdgcn_readfirstlane(ct_after);
    }

    if (!stores) return;
    float *out = g.part + (size_t)seg * 128 * g.f + nb * 32 + ll;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) out[(size_t)(i * 32 + 8 * (r / 4) + 4 * kh + (r % 4)) * g.f] = acc[i][r];
}

// Dh[rank, :] = sum of the partial products of the segments of the rank's row of tiles, in segment order (zeros for a row of
// tiles that kept none)
__global__ void k_tiles_reduce(const float *__restrict__ part, const int32_t *__restrict__ rt_seg, int nt_r, int f, float *__restrict__ Dh) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int f4 = f / 4;
    if (t >= (long long)nt_r * 128 * f4) return;
    const int col = (int)(t % f4) * 4;
    const int rank = (int)(t / f4);
    const int rt = rank >> 7, row = rank & 127;
    const int g0 = rt_seg[rt], g1 = rt_seg[rt + 1];
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int sg = g0; sg < g1; ++sg) {
        const float4 v = *reinterpret_cast<const float4 *>(part + ((size_t)sg * 128 + row) * f + col);
        sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
    }
    *reinterpret_cast<float4 *>(Dh + (size_t)rank * f + col) = sum;
}

// C[i, :] = act(scale_i * (C[i, :] + Dh[rank of i, :])): joins the raw sums of the sparse remainder with those of the tiles
// and applies what the SpMM epilogue would have applied (scale_i = r[i], or 1 / z_i in attention mode)
__global__ void k_tiles_combine(float *__restrict__ C, long long n_rows, int f_store, long long ldc, long long c_tile, const float *__restrict__ Dh,
                                int f, const int32_t *__restrict__ rank_r, int n_ranks, const float *__restrict__ r, const float2 *__restrict__ mz,
                                int act, int vec4, const int32_t *__restrict__ row_ptr, int chunk_nnz, const float *__restrict__ carry, int f_carry,
                                const float *__restrict__ tile_shift) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int f4 = (f_store + 3) / 4;
    if (t >= n_rows * f4) return;
    const long long i = t / f4;
    const int col = (int)(t % f4) * 4;
    const int rank = rank_r[i];
    float sc = 1.f;
    if (mz) { const float z = mz[i].y; sc = z > 0.f ? 1.f / z : 0.f; }
    else if (r) sc = r[i];
    float *dst = C + (long long)(col >> 5) * c_tile + i * ldc + (col & 31);
    const float *add = (rank < n_ranks) ? Dh + (size_t)rank * f + col : nullptr;
    // attention tiles that were multiplied before the row maxima were known used the maximum over the row's tile entries as the shift:
    // exp(that - the row maximum) brings their sum to the row's scale
    float tf = 1.f;
    if (tile_shift && add) { const float ts = tile_shift[rank]; tf = ts > -INFINITY ? __expf(ts - mz[i].x) : 0.f; }
    // the SpMM's own fix-up, when the caller left it to this pass: a row that spans chunk boundaries has its later pieces in the
    // carry slots of the chunks it continues into, c * chunk_nnz strictly inside the row; they are added in chunk order
    long long c_first = 1, c_last = 0;
    if (row_ptr) {
        const long long rs = row_ptr[i], re = row_ptr[i + 1];
        if (re > rs) {
            c_first = rs / chunk_nnz + 1;
            c_last = (re - 1) / chunk_nnz;
        }
    }
    if (vec4 && col + 3 < f_store) {  // 16-byte accesses when the caller found every row start aligned
        float4 y = *reinterpret_cast<const float4 *>(dst);
#pragma unroll 4
        for (long long c = c_first; c <= c_last; ++c) {
            const float4 p = *reinterpret_cast<const float4 *>(carry + (size_t)c * f_carry + col);
            y.x += p.x; y.y += p.y; y.z += p.z; y.w += p.w;
        }
        if (add) {
            const float4 a4 = *reinterpret_cast<const float4 *>(add);
            y.x += tf * a4.x; y.y += tf * a4.y; y.z += tf * a4.z; y.w += tf * a4.w;
        }
        y.x *= sc; y.y *= sc; y.z *= sc; y.w *= sc;
        if (act == SENSEI_ACT_RELU) {
            y.x = y.x > 0.f ? y.x : 0.f; y.y = y.y > 0.f ? y.y : 0.f; y.z = y.z > 0.f ? y.z : 0.f; y.w = y.w > 0.f ? y.w : 0.f;
        }
        *reinterpret_cast<float4 *>(dst) = y;
        return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (col + e < f_store) {
            float y = dst[e];
            for (long long c = c_first; c <= c_last; ++c) y += carry[(size_t)c * f_carry + col + e];
            y = (y + (add ? tf * add[e] : 0.f)) * sc;
            if (act == SENSEI_ACT_RELU) y = y > 0.f ? y : 0.f;
            dst[e] = y;
        }
    }
}

// The join for a remainder that ran panel-major: the row's raw sum is spread over its n_panels segments (panel q, row i), each with
// the carry slots of the chunks the segment continues into; they are added panel by panel, chunk by chunk (a fixed order).
__global__ void k_tiles_combine_pm(float *__restrict__ C, long long n_rows, int f_store, long long ldc, long long c_tile, const float *__restrict__ Dh,
                                   int f, const int32_t *__restrict__ rank_r, int n_ranks, const float *__restrict__ r, const float2 *__restrict__ mz,
                                   int act, int vec4, const float *__restrict__ part, int n_panels, const int32_t *__restrict__ seg_ptr, int chunk_nnz,
                                   const float *__restrict__ carry, int f_carry, const float *__restrict__ tile_shift) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int f4 = (f_store + 3) / 4;
    if (t >= n_rows * f4) return;
    const long long i = t / f4;
    const int col = (int)(t % f4) * 4;
    const int rank = rank_r[i];
    float sc = 1.f;
    if (mz) { const float z = mz[i].y; sc = z > 0.f ? 1.f / z : 0.f; }
    else if (r) sc = r[i];
    const long long part_tile = (long long)n_panels * n_rows * 32;
    float4 y = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int q = 0; q < n_panels; ++q) {
        const long long seg = (long long)q * n_rows + i;
        const float4 p = *reinterpret_cast<const float4 *>(part + (long long)(col >> 5) * part_tile + seg * 32 + (col & 31));
        y.x += p.x; y.y += p.y; y.z += p.z; y.w += p.w;
        const long long rs = seg_ptr[seg], re = seg_ptr[seg + 1];
        if (re > rs) {
            for (long long c = rs / chunk_nnz + 1; c <= (re - 1) / chunk_nnz; ++c) {
                const float4 v = *reinterpret_cast<const float4 *>(carry + (size_t)c * f_carry + col);
                y.x += v.x; y.y += v.y; y.z += v.z; y.w += v.w;
            }
        }
    }
    if (rank < n_ranks) {
        float tf = 1.f;   // see k_tiles_combine
        if (tile_shift) { const float ts = tile_shift[rank]; tf = ts > -INFINITY ? __expf(ts - mz[i].x) : 0.f; }
        const float4 a4 = *reinterpret_cast<const float4 *>(Dh + (size_t)rank * f + col);
        y.x += tf * a4.x; y.y += tf * a4.y; y.z += tf * a4.z; y.w += tf * a4.w;
    }
    y.x *= sc; y.y *= sc; y.z *= sc; y.w *= sc;
    if (act == SENSEI_ACT_RELU) {
        y.x = y.x > 0.f ? y.x : 0.f; y.y = y.y > 0.f ? y.y : 0.f; y.z = y.z > 0.f ? y.z : 0.f; y.w = y.w > 0.f ? y.w : 0.f;
    }
    float *dst = C + (long long)(col >> 5) * c_tile + i * ldc + (col & 31);
    if (vec4 && col + 3 < f_store) {
        *reinterpret_cast<float4 *>(dst) = y;
    } else {
        if (col < f_store) dst[0] = y.x;
        if (col + 1 < f_store) dst[1] = y.y;
        if (col + 2 < f_store) dst[2] = y.z;
        if (col + 3 < f_store) dst[3] = y.w;
    }
}

// Dt[slot] = Lh[rows of the slot's row tile] . Rh[rows of its column tile]^T, 128 x 128 per kept tile: the per-entry dot product
// <dP_i, Theta_j> of the attention backward for all entries of a tile at once, on the matrix cores (the cells outside the tile's
// bit mask are computed too and never read).  bf16 instruction on three exact pieces per operand, eight products a term in two accumulators: these
// are single dot products, used one by one.  With the fp32 instruction the kernel was bound by it (16 k of a tile: 2,048 matrix cycles per
// wavefront, here 1,024).  Both operands are rows with k contiguous: two neighbouring threads take the 16 k of a row and step, cut eight each and leave
// them in LDS in lane order, so that an element is cut once per workgroup; two buffers, one barrier per step (8 rows of padding between the
// halves of k: the two threads' 16-byte writes fall on different banks).  22,334 tiles at 256 columns, beside the remainder's dot products: GAT
// training on 115 M entries 17.9 ms with the fp32 instruction, 17.3 so (six products: 17.2).  Against fp64, in 2^-24 of the terms' magnitudes, fp32
// instruction / so: rms of sums over 128 to 256 columns 0.39-0.40 / 0.11-0.12, with terms of one sign 2.6-3.6 / 1.0-1.4; single products 0.43 / 0.43,
// the largest 1.00 / 1.00 (six products: 1.4 measured, 2.0 where a second piece is as large as it gets).
__global__ __launch_bounds__(kThreads, 2) void k_tiles_sddmm(const float *__restrict__ Lh, const float *__restrict__ Rh, int f,
                                                              const int32_t *__restrict__ slot_rt, const int32_t *__restrict__ slot_ct,
                                                              float *__restrict__ Dt) {
    constexpr int WGN = 2, TM = 2, TN = 2, ROWS = 128 + 8;
    __shared__ __attribute__((aligned(16))) unsigned short Ps[2][2][3][2][ROWS][8];   // buffer, operand, piece, half of k, row
    const int slot = blockIdx.x;
    const int t = threadIdx.x;
    const int wave = t >> 6, lane = t & 63, kh = lane >> 5, ll = lane & 31;
    const int wm = wave / WGN, wn = wave % WGN;
    const int row = t >> 1, half = t & 1;
    const float *src[2] = {Lh + ((size_t)slot_rt[slot] * 128 + row) * f + half * 8, Rh + ((size_t)slot_ct[slot] * 128 + row) * f + half * 8};

    floatx16 acc[TM][TN], low[TM][TN];   // the products of the first pieces; all others
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = low[i][j][r] = 0.f;

    float4 raw[2][2];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            raw[o][0] = *reinterpret_cast<const float4 *>(src[o] + k0);
            raw[o][1] = *reinterpret_cast<const float4 *>(src[o] + k0 + 4);
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            const float v[8] = {raw[o][0].x, raw[o][0].y, raw[o][0].z, raw[o][0].w, raw[o][1].x, raw[o][1].y, raw[o][1].z, raw[o][1].w};
            uintx4 w[3];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                unsigned a, b, c;
                cut_pair(v[2 * d], v[2 * d + 1], a, b, c);
                w[0][d] = a; w[1][d] = b; w[2][d] = c;
            }
#pragma unroll
            for (int p = 0; p < 3; ++p) *reinterpret_cast<uintx4 *>(&Ps[buf][o][p][half][row][0]) = w[p];
        }
    };
    const int n_steps = f / 16;  // f is a multiple of 32
    fetch(0);
    stash(0);
    for (int st = 0; st < n_steps; ++st) {
        fetch((st + 1 < n_steps ? st + 1 : st) * 16);   // the last step's fetch is not used
        __builtin_amdgcn_sched_barrier(0);              // the fetches stay here, their use below the multiply
        __syncthreads();   // this step's pieces are in Ps[st & 1]; nobody reads the other buffer any more
        uintx4 af[TM][3];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int p = 0; p < 3; ++p) af[i][p] = *reinterpret_cast<const uintx4 *>(&Ps[st & 1][0][p][kh][(wm * TM + i) * 32 + ll][0]);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            uintx4 bf[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) bf[p] = *reinterpret_cast<const uintx4 *>(&Ps[st & 1][1][p][kh][(wn * TN + j) * 32 + ll][0]);
#pragma unroll
            for (int pa = 2; pa >= 0; --pa)
#pragma unroll
                for (int pb = pa == 2 ? 1 : 2; pb >= 0; --pb)   // smallest products first
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        floatx16 &sum = pa + pb > 0 ? low[i][j] : acc[i][j];
                        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[i][pa]), __builtin_bit_cast(bf16x8, bf[pb]), sum, 0, 0, 0);
                    }
        }
        __builtin_amdgcn_sched_barrier(0);
        stash((st + 1) & 1);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] += low[i][j];
    if (__any(not_finite<TN>(acc[0]) || not_finite<TN>(acc[1]))) {
#pragma unroll 1
        for (int u = 0; u < TM * TN; ++u) {
            const float *l = Lh + ((size_t)slot_rt[slot] * 128 + (wm * TM + u / TN) * 32 + ll) * f;
            const float *r = Rh + ((size_t)slot_ct[slot] * 128 + (wn * TN + u % TN) * 32 + ll) * f;
            const floatx16 sums = product_fp32(f, kh, [&](int q) { return l[q]; }, [&](int q) { return r[q]; });
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    if (i * TN + j == u)
#pragma unroll
                        for (int q = 0; q < 16; ++q)
                            if (!__builtin_isfinite(acc[i][j][q])) acc[i][j][q] = sums[q];
        }
    }
    float *out = Dt + (size_t)slot * 128 * 128;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int orow = (wm * TM + i) * 32 + 8 * (r / 4) + 4 * kh + (r % 4);
#pragma unroll
            for (int j = 0; j < TN; ++j) out[(size_t)orow * 128 + (wn * TN + j) * 32 + ll] = acc[i][j][r];
        }
}

// the projections of every head (blockIdx.y) of one slice: eight lanes a row, four rows of a lane in flight
constexpr int kScoreRows = 4;
__global__ __launch_bounds__(kThreads) void k_head_scores(const float *__restrict__ theta, long long n, int d, const float *__restrict__ a_l,
                                                          const float *__restrict__ a_r, float *__restrict__ s_l, float *__restrict__ s_r) {
    const int head = blockIdx.y, li = threadIdx.x & 7;
    const long long row0 = (long long)blockIdx.x * (kThreads / 8 * kScoreRows) + threadIdx.x / 8;
    float4 x[kScoreRows];
#pragma unroll
    for (int u = 0; u < kScoreRows; ++u) {
        const long long row = row0 + u * (kThreads / 8), rc = row < n ? row : n - 1;
        x[u] = *reinterpret_cast<const float4 *>(theta + ((size_t)head * n + rc) * 32 + li * 4);
    }
    float al[4], ar[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int q = li * 4 + e;
        al[e] = q < d ? a_l[head * d + q] : 0.f;
        ar[e] = q < d ? a_r[head * d + q] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kScoreRows; ++u) {
        float l = fmaf(x[u].x, al[0], fmaf(x[u].y, al[1], fmaf(x[u].z, al[2], x[u].w * al[3])));
        float r = fmaf(x[u].x, ar[0], fmaf(x[u].y, ar[1], fmaf(x[u].z, ar[2], x[u].w * ar[3])));
#pragma unroll
        for (int off = 4; off > 0; off >>= 1) {
            l += __shfl_xor(l, off, 64);
            r += __shfl_xor(r, off, 64);
        }
        const long long row = row0 + u * (kThreads / 8);
        if (li == 0 && row < n) { s_l[head * n + row] = l; s_r[head * n + row] = r; }
    }
}

__global__ void k_pad_heads(const float *__restrict__ W, long long ldw, int f_in, int heads, int d, int dp, float *__restrict__ out, long long ldo) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int cols = heads * dp;
    if (t >= (long long)f_in * cols) return;
    const int q = (int)(t % cols), c = q % dp;
    const long long k = t / cols;
    out[k * ldo + q] = c < d ? W[k * ldw + (q / dp) * d + c] : 0.f;
}

// the attention vectors in rank order (zeros where a rank has no node)
__global__ void k_gather_ranked_vecs(const float *__restrict__ s_l, const float *__restrict__ s_r, const float2 *__restrict__ mz,
                                     const int32_t *__restrict__ order_r, int n_r, const int32_t *__restrict__ order_c, int n_c,
                                     float *__restrict__ sl_rank, float *__restrict__ m_rank, float *__restrict__ sr_rank) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n_r) {
        const int i = order_r[q];
        sl_rank[q] = i >= 0 ? s_l[i] : 0.f;
        if (mz) m_rank[q] = i >= 0 ? mz[i].x : 0.f;
    }
    if (q < n_c) {
        const int j = order_c[q];
        sr_rank[q] = j >= 0 ? s_r[j] : 0.f;
    }
}

// (max, sum of exp) of the attention logits over the entries of one segment of tiles, per row of its row of tiles: two threads per
// row, each walks the set bits of its half of the row's mask in every tile of the segment; the column vector of the tile sits in LDS.
// A tile is first searched for its maximum, then summed against the running maximum, so a row costs one rescale per tile.
__global__ __launch_bounds__(256) void k_tile_stats(const unsigned *__restrict__ bits, const int32_t *__restrict__ seg_first,
                                                    const int32_t *__restrict__ slot_ct, const int32_t *__restrict__ seg_rt,
                                                    const float *__restrict__ sl_rank, const float *__restrict__ sr_rank, float slope,
                                                    float2 *__restrict__ seg_stats) {
    __shared__ float sr_s[128];
    const int seg = blockIdx.x;
    const int s0 = seg_first[seg], s1 = seg_first[seg + 1];
    const int t = threadIdx.x, row = t >> 1, half = t & 1;
    const float sl = sl_rank[(size_t)seg_rt[seg] * 128 + row];
    float m = -INFINITY, z = 0.f;
    for (int slot = s0; slot < s1; ++slot) {
        __syncthreads();  // the previous tile's column vector is no longer read
        if (t < 128) sr_s[t] = sr_rank[(size_t)slot_ct[slot] * 128 + t];
        __syncthreads();
        const uint2 w = *reinterpret_cast<const uint2 *>(bits + ((size_t)slot * 128 + row) * 4 + half * 2);
        const float *sr = sr_s + half * 64;
        float tm = -INFINITY;
        for (unsigned b = w.x; b; b &= b - 1) {
            float e = sl + sr[__ffs(b) - 1];
            e = e > 0.f ? e : slope * e;
            tm = e > tm ? e : tm;
        }
        for (unsigned b = w.y; b; b &= b - 1) {
            float e = sl + sr[32 + __ffs(b) - 1];
            e = e > 0.f ? e : slope * e;
            tm = e > tm ? e : tm;
        }
        if (tm == -INFINITY) continue;  // no entry of this row in this half of the tile
        const float mm = m > tm ? m : tm;
        z *= __expf(m - mm);            // m = -inf at the start: exp(-inf) = 0 and z = 0
        m = mm;
        for (unsigned b = w.x; b; b &= b - 1) {
            float e = sl + sr[__ffs(b) - 1];
            e = e > 0.f ? e : slope * e;
            z += __expf(e - m);
        }
        for (unsigned b = w.y; b; b &= b - 1) {
            float e = sl + sr[32 + __ffs(b) - 1];
            e = e > 0.f ? e : slope * e;
            z += __expf(e - m);
        }
    }
    // the two halves of the row sit in neighbouring lanes
    const float m2 = __shfl_xor(m, 1, 64), z2 = __shfl_xor(z, 1, 64);
    const float mm = m > m2 ? m : m2;
    if (half == 0) {
        float2 out = make_float2(-INFINITY, 0.f);
        if (mm != -INFINITY) out = make_float2(mm, z * __expf(m - mm) + z2 * __expf(m2 - mm));
        seg_stats[(size_t)seg * 128 + row] = out;
    }
}

// stats[i] (the pair over the remainder's entries of row i) merged with the pairs of the segments of the row's row of tiles, in
// segment order
__global__ void k_tile_stats_merge(float2 *__restrict__ stats, long long n_rows, const int32_t *__restrict__ rank_r, int n_ranks,
                                   const int32_t *__restrict__ rt_seg, const float2 *__restrict__ seg_stats) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_rows) return;
    const int rank = rank_r[i];
    if (rank >= n_ranks) return;
    float2 a = stats[i];
    const int rt = rank >> 7, lr = rank & 127;
    for (int seg = rt_seg[rt]; seg < rt_seg[rt + 1]; ++seg) {
        const float2 b = seg_stats[(size_t)seg * 128 + lr];
        const float mm = a.x > b.x ? a.x : b.x;
        if (mm == -INFINITY) continue;
        a.y = a.y * expf(a.x - mm) + b.y * expf(b.x - mm);
        a.x = mm;
    }
    stats[i] = a;
}

// m_rank[q] = the largest logit among the tile entries of the row of rank q (-inf: none): the shift the attention tiles can use before
// the row maxima over all entries are known
__global__ void k_tile_row_max(const int32_t *__restrict__ rt_seg, const float2 *__restrict__ seg_stats, int n_ranks, float *__restrict__ m_rank) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n_ranks) return;
    float m = -INFINITY;
    for (int seg = rt_seg[q >> 7]; seg < rt_seg[(q >> 7) + 1]; ++seg) { const float v = seg_stats[(size_t)seg * 128 + (q & 127)].x; m = v > m ? v : m; }
    m_rank[q] = m;
}

// the same for the tiles of the transposed pattern: its rows are the sources (s_r), its columns the destinations (s_l and their maxima)
__global__ void k_gather_ranked_vecs_t(const float *__restrict__ s_l, const float *__restrict__ s_r, const float2 *__restrict__ mz,
                                       const int32_t *__restrict__ order_r, int n_r, const int32_t *__restrict__ order_c, int n_c,
                                       float *__restrict__ sr_rank, float *__restrict__ sl_rank, float *__restrict__ m_rank) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n_r) {
        const int j = order_r[q];
        sr_rank[q] = j >= 0 ? s_r[j] : 0.f;
    }
    if (q < n_c) {
        const int i = order_c[q];
        sl_rank[q] = i >= 0 ? s_l[i] : 0.f;
        m_rank[q] = i >= 0 ? mz[i].x : 0.f;
    }
}

// Bh[q, 0:f) = row order_c[q] of the slice-major matrix B (zeros where the rank has no node), times 1 / mz[node].y if mz is given
__global__ void k_gather_ranked_rows(const float *__restrict__ B, long long n_cols, int f, const int32_t *__restrict__ order_c, long long n_ranks,
                                     float *__restrict__ Bh, const float2 *__restrict__ mz) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int f4 = f / 4;
    if (t >= n_ranks * f4) return;
    const long long q = t / f4;
    const int col = (int)(t % f4) * 4;
    const int j = order_c[q];
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (j >= 0) v = *reinterpret_cast<const float4 *>(B + (long long)(col >> 5) * n_cols * 32 + (long long)j * 32 + (col & 31));
    if (mz && j >= 0) {
        const float z = mz[j].y, iz = z > 0.f ? 1.f / z : 0.f;
        v.x *= iz; v.y *= iz; v.z *= iz; v.w *= iz;
    }
    *reinterpret_cast<float4 *>(Bh + q * f + col) = v;
}

// ---- C[M x N] = A^T . B with A stored [K x M] and B stored [K x N] (both row-major), K very long: the weight
// gradient dW = X^T . G of a layer, reduced over all nodes.  The K range is cut into `splits` slabs, one
// workgroup per (output tile, slab); slab s writes its partial tile to part[s] and k_sum_splits adds the slabs
// in order, so the result does not depend on scheduling.  Both operands arrive k-major, which is the layout the
// MFMA operand reads want, so both use the loader the forward kernel uses for W.  A sum over 10^5..10^7 nodes
// in one fp32 accumulator would lose the small entries of dW (rounding grows with the running sum, about
// 6e-4 of a term's spread at K = 233,000): the fp32 MFMA accumulators are therefore emptied into fp64 registers
// after every kFlushTiles k-tiles, the slabs are stored and added in fp64, and only the final sum is rounded to fp32.
struct GemmTnArgs {
    const float *A, *B;
    double *part;     // splits x M x N
    long long lda, ldb, k;
    int m, n, n_bn, n_tiles, k_per_split;
    int segs;           // several products with the same A in one launch: B's columns h * b_seg .. + n belong to product h, n_bn blocks of columns each
    long long b_seg;
};

constexpr int kFlushTiles = 1;  // k-tiles (of KT = 16) summed in fp32 before the accumulators move to fp64

template <int VA, int VB>
__global__ __launch_bounds__(kThreads) void k_gemm_tn(GemmTnArgs g) {
    constexpr int BM = 128, BN = 128, TM = 2, TN = 2, PAD = 4;
    __shared__ __attribute__((aligned(16))) float As[KT][BM + PAD];
    __shared__ __attribute__((aligned(16))) float Bs[KT][BN + PAD];
    const int t = threadIdx.x;
    const int wave = t >> 6, lane = t & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const int tile = (int)(blockIdx.x % g.n_tiles), split = (int)(blockIdx.x / g.n_tiles);
    const int jn = tile % (g.n_bn * g.segs), seg = jn / g.n_bn;
    const int m0 = tile / (g.n_bn * g.segs) * BM, n0 = jn % g.n_bn * BN;
    const float *const B = g.B + seg * g.b_seg;
    const long long k_lo = (long long)split * g.k_per_split;
    const long long k_hi = (k_lo + g.k_per_split < g.k) ? k_lo + g.k_per_split : g.k;

    floatx16 acc[TM][TN];
    double dacc[TM][TN][16];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) { acc[i][j][r] = 0.f; dacc[i][j][r] = 0.0; }
    auto flush = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) { dacc[i][j][r] += (double)acc[i][j][r]; acc[i][j][r] = 0.f; }
    };

    // loader: KT rows of 128 floats per operand; VEC floats per thread and pass
    constexpr int A_TPR = BM / VA, A_RPP = kThreads / A_TPR, A_PASSES = (KT + A_RPP - 1) / A_RPP;
    constexpr int B_TPR = BN / VB, B_RPP = kThreads / B_TPR, B_PASSES = (KT + B_RPP - 1) / B_RPP;
    float ra[A_PASSES][VA], rb[B_PASSES][VB];
    const int a_row = t / A_TPR, a_cc = (t % A_TPR) * VA;
    const int b_row = t / B_TPR, b_cc = (t % B_TPR) * VB;

    auto fetch = [&](long long k0) {
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p) {
            const int kr = p * A_RPP + a_row;
            const long long kk = k0 + kr;
            const int col = m0 + a_cc;
            if (kr < KT && kk < k_hi && col < g.m) {  // VA == 4 implies m % 4 == 0: a piece never straddles the edge
                const float *src = g.A + kk * g.lda + col;
                if (VA == 4) { float4 v = *reinterpret_cast<const float4 *>(src); ra[p][0] = v.x; ra[p][1 % VA] = v.y; ra[p][2 % VA] = v.z; ra[p][3 % VA] = v.w; }
                else ra[p][0] = *src;
            } else {
#pragma unroll
                for (int e = 0; e < VA; ++e) ra[p][e] = 0.f;
            }
        }
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            const int kr = p * B_RPP + b_row;
            const long long kk = k0 + kr;
            const int col = n0 + b_cc;
            if (kr < KT && kk < k_hi && col < g.n) {
                const float *src = B + kk * g.ldb + col;
                if (VB == 4) { float4 v = *reinterpret_cast<const float4 *>(src); rb[p][0] = v.x; rb[p][1 % VB] = v.y; rb[p][2 % VB] = v.z; rb[p][3 % VB] = v.w; }
                else rb[p][0] = *src;
            } else {
#pragma unroll
                for (int e = 0; e < VB; ++e) rb[p][e] = 0.f;
            }
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p) {
            const int kr = p * A_RPP + a_row;
            if (kr < KT) {
#pragma unroll
                for (int e = 0; e < VA; ++e) As[kr][a_cc + e] = ra[p][e];
            }
        }
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            const int kr = p * B_RPP + b_row;
            if (kr < KT) {
#pragma unroll
                for (int e = 0; e < VB; ++e) Bs[kr][b_cc + e] = rb[p][e];
            }
        }
    };

    const int kh = lane >> 5, ll = lane & 31;
    if (k_lo < k_hi) fetch(k_lo);
    int since_flush = 0;
    for (long long k0 = k_lo; k0 < k_hi; k0 += KT) {
        stash();
        __syncthreads();
        if (k0 + KT < k_hi) fetch(k0 + KT);
#pragma unroll
        for (int kk = 0; kk < KT; kk += 2) {
            float av[TM], bv[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) av[i] = As[kk + kh][(wm * TM + i) * 32 + ll];
#pragma unroll
            for (int j = 0; j < TN; ++j) bv[j] = Bs[kk + kh][(wn * TN + j) * 32 + ll];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
        if (++since_flush == kFlushTiles) { flush(); since_flush = 0; }
        __syncthreads();
    }
    flush();

    const size_t width = (size_t)g.n * g.segs;
    double *out = g.part + (size_t)split * (size_t)g.m * width + (size_t)seg * g.n;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = n0 + (wn * TN + j) * 32 + ll;
            if (col >= g.n) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = m0 + (wm * TM + i) * 32 + 8 * (r / 4) + 4 * kh + (r % 4);
                if (row < g.m) out[(size_t)row * width + col] = dacc[i][j][r];
            }
        }
}

// The same reduction on the bf16 matrix instruction at fp32 accuracy (three exact bf16 pieces per operand element, six piece
// products per term, as in k_gemm_bf).  Both operands arrive k-major, while a lane of the 32 x 32 x 16 instruction wants eight
// consecutive k of one column: a thread fetches exactly that (eight rows of its column, neighbouring lanes on neighbouring columns),
// cuts the eight values into pieces and leaves them in LDS in lane order, for both operands alike; two buffers, one barrier per step
// of 16 k, fetches one step ahead.  The fp32 accumulators are emptied into fp64 registers after every second step.
constexpr int kFlushStepsBf = 2;

// A wavefront takes 64 x 32 outputs; a block of 128 columns has eight.  As four wavefronts of 64 x 64 they held 312 registers (fp32 and fp64 accumulators), one wavefront a SIMD
// and nothing beside its cuts, flushes and waits: 602 x 233,000 x 256 833 us, now 560; 128 x 100,000 x 128 with its slab sums 80 -> 43.
// TN = 1 (blocks of 128 x 64) where the product has at most 64 columns: half of the matrix work, of the pieces of B and of the fp64
// accumulators of a 128-column block would be for columns that are not there (100,000 rows, 100 x 47: 45 -> 26.5 us; 233,000 rows,
// 256 x 41: 150 -> 97; 50,000 rows, 100 x 64: 33 -> 19.6).
template <int TN>
__global__ __launch_bounds__(kThreads * TN, 2) void k_gemm_tn_bf(GemmTnArgs g) {
    constexpr int BM = 128, BN = 64 * TN, TM = 2;
    // [buffer][piece][32-column block: four of A, then 2 TN of B][k half][column][8 k]
    __shared__ __attribute__((aligned(16))) unsigned short Ps[2][3][4 + 2 * TN][2][32][8];
    const int t = threadIdx.x;
    const int wave = t >> 6, lane = t & 63;
    const int wm = wave / (2 * TN), wn = wave % (2 * TN);   // a wavefront takes 64 x 32
    const int kh = lane >> 5, ll = lane & 31;
    const int tile = (int)(blockIdx.x % g.n_tiles), split = (int)(blockIdx.x / g.n_tiles);
    const int jn = tile % (g.n_bn * g.segs), seg = jn / g.n_bn;
    const int m0 = tile / (g.n_bn * g.segs) * BM, n0 = jn % g.n_bn * BN;
    const float *const B = g.B + seg * g.b_seg;
    const long long k_lo = (long long)split * g.k_per_split;
    const long long k_hi = (k_lo + g.k_per_split < g.k) ? k_lo + g.k_per_split : g.k;

    floatx16 acc[TM];
    double dacc[TM][16];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) { acc[i][r] = 0.f; dacc[i][r] = 0.0; }
    // Every other group of steps multiplies -A and is subtracted: the instruction's sum of 16 products and the accumulator loses
    // low bits of the smaller addends downwards whatever their sign (measured: about -2^-29 of the sum of the terms' magnitudes),
    // which over 10^5 rows would add up to several units of fp32 rounding of the root-sum-square; in alternating groups it cancels.
    int neg = split & 1;   // slabs with an odd number of groups leave one over: neighbouring slabs start with opposite signs
    auto flush = [&]() {
        const double sg = neg ? -1.0 : 1.0;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) { dacc[i][r] = fma(sg, (double)acc[i][r], dacc[i][r]); acc[i][r] = 0.f; }
    };

    // staging: thread -> (operand, column, k half): with 512 threads one column of one operand each, with 256 a column of A and, half of them, one of
    // B; columns past the edge read the last column and are cleared, rows past the slab read its last row and are cleared (masks, not branches
    // around the fetches).  Addresses: a uniform row pointer per k plus one 32-bit byte offset per lane (its k half and column), fixed before the loop
    struct Column { const float *base; long long ld; unsigned mask, off; int block, half, at; bool on; float v[8]; };
    auto column = [&](bool of_a, int task) {
        Column c;
        const int cols = of_a ? BM : BN, col = task % cols, first = of_a ? m0 : n0, n_cols = of_a ? g.m : g.n;
        c.on = task < 2 * cols;
        c.half = (task / cols) & 1;
        c.base = of_a ? g.A : B;
        c.ld = of_a ? g.lda : g.ldb;
        const bool ok = first + col < n_cols;
        c.mask = ok ? ~0u : 0u;
        c.off = (unsigned)(((long long)c.half * 8 * c.ld + (ok ? first + col : n_cols - 1)) * 4);
        c.block = (of_a ? 0 : 4) + (col >> 5);
        c.at = col & 31;
        return c;
    };
    const bool mine_a = TN == 1 || __builtin_amdgcn_readfirstlane(wave) < 4;
    Column own = column(mine_a, t & 255), second = TN == 1 ? column(false, t) : own;
    auto fetch_one = [&](Column &c, bool of_a, long long k0, auto whole) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if constexpr (decltype(whole)::value) {   // all 16 rows of the step lie inside the slab
                const char *r = reinterpret_cast<const char *>(c.base + (k0 + e) * c.ld);
                c.v[e] = __uint_as_float(__float_as_uint(*reinterpret_cast<const float *>(r + c.off)) & c.mask);
            } else {
                const long long k = k0 + c.half * 8 + e, kc = (k < k_hi ? k : k_hi - 1) - c.half * 8;
                const unsigned live = k < k_hi || !of_a ? ~0u : 0u;   // a row past the slab is cleared in A
                const char *r = reinterpret_cast<const char *>(c.base + kc * c.ld);
                c.v[e] = __uint_as_float(__float_as_uint(*reinterpret_cast<const float *>(r + c.off)) & c.mask & live);
            }
        }
    };
    auto fetch = [&](long long k0, auto whole) {
        fetch_one(own, mine_a, k0, whole);
        if constexpr (TN == 1) fetch_one(second, false, k0, whole);
    };
    auto stash_one = [&](const Column &c, bool of_a, int buf) {
        unsigned pc[8][3];
#pragma unroll
        for (int e = 0; e < 8; ++e) split_bf16x3(c.v[e], pc[e][0], pc[e][1], pc[e][2]);
        const unsigned flip = (of_a && neg) ? 0x80008000u : 0u;   // the sign bits of a pair of bf16
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            uintx4 w;
#pragma unroll
            for (int d = 0; d < 4; ++d) w[d] = pack_bf16(pc[2 * d][p], pc[2 * d + 1][p]) ^ flip;
            if (c.on) *reinterpret_cast<uintx4 *>(&Ps[buf][p][c.block][c.half][c.at][0]) = w;
        }
    };
    auto stash = [&](int buf) {
        stash_one(own, mine_a, buf);
        if constexpr (TN == 1) {
            __builtin_amdgcn_sched_barrier(0);   // one operand's pieces at a time in registers
            stash_one(second, false, buf);
        }
    };

    if (k_lo < k_hi) {
        int buf = 0, since_flush = 0;
        auto step = [&](long long k0, auto next_whole) {
            fetch(k0 + 16 < k_hi ? k0 + 16 : k0, next_whole);   // past the last step: this step again, not used
            __builtin_amdgcn_sched_barrier(0);      // the fetches stay here and their use stays below the multiply
            __syncthreads();                        // this step's pieces are in Ps[buf]; nobody reads the other buffer any more
            // few fragments live at a time (the fp64 accumulators take half the registers): the pieces of B are read again for each
            // piece of A they meet
#pragma unroll
            for (int pa = 2; pa >= 0; --pa) {
                uintx4 af[TM];
#pragma unroll
                for (int i = 0; i < TM; ++i) af[i] = *reinterpret_cast<const uintx4 *>(&Ps[buf][pa][wm * TM + i][kh][ll][0]);
#pragma unroll
                for (int pb = 2 - pa; pb >= 0; --pb) {   // smallest products first
                    const uintx4 bf = *reinterpret_cast<const uintx4 *>(&Ps[buf][pb][4 + wn][kh][ll][0]);
#pragma unroll
                    for (int i = 0; i < TM; ++i)
                        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[i]), __builtin_bit_cast(bf16x8, bf), acc[i], 0, 0, 0);
                }
            }
            if (++since_flush == kFlushStepsBf) { flush(); since_flush = 0; neg ^= 1; }   // the pieces stashed below belong to the next group
            __builtin_amdgcn_sched_barrier(0);
            stash(buf ^ 1);
            buf ^= 1;
        };
        if (k_lo + 16 <= k_hi) fetch(k_lo, std::true_type()); else fetch(k_lo, std::false_type());
        stash(0);
        long long k0 = k_lo;
        for (; k0 + 32 <= k_hi; k0 += 16) step(k0, std::true_type());   // the next step is whole
        for (; k0 < k_hi; k0 += 16) step(k0, std::false_type());
    }
    flush();

    const size_t width = (size_t)g.n * g.segs;
    double *out = g.part + (size_t)split * (size_t)g.m * width + (size_t)seg * g.n;
    const int c = n0 + wn * 32 + ll;
    if (c >= g.n) return;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = m0 + (wm * TM + i) * 32 + 8 * (r / 4) + 4 * kh + (r % 4);
            if (row < g.m) out[(size_t)row * width + c] = dacc[i][r];
        }
}

// C[i] = sum over the slabs.  What bounds it is latency: with one thread per element walking all slabs (768 of them for a small product)
// a 100 x 47 result kept 19 workgroups busy for 188 us.  A workgroup takes 16 elements (one 128-byte line of a slab) and deals the slabs
// to 16 lanes each, which keep eight loads in flight; the 16 partial sums are added in lane order through LDS, so the order of the
// additions is fixed.  100 x 47, 768 slabs: 188 -> 10 us; 602 x 256, 77 slabs: 66 -> under 22 us.
constexpr int kSumElems = 16, kSumLanes = 16;
__global__ __launch_bounds__(kSumElems * kSumLanes) void k_sum_splits(const double *__restrict__ part, int splits, long long mn, int n, int segs,
                                                                       float *__restrict__ C, long long ldc, long long c_seg) {
    __shared__ double red[kSumLanes][kSumElems];
    const int q = threadIdx.x % kSumElems, y = threadIdx.x / kSumElems;
    const long long e = (long long)blockIdx.x * kSumElems + q;
    double s = 0.0;
    if (e < mn) {
        const double *src = part + e;
#pragma unroll 8
        for (int p = y; p < splits; p += kSumLanes) s += src[(size_t)p * (size_t)mn];
    }
    red[y][q] = s;
    __syncthreads();
    if (y != 0 || e >= mn) return;
#pragma unroll
    for (int u = 1; u < kSumLanes; ++u) s += red[u][q];
    const int q_all = (int)(e % ((long long)n * segs));
    C[q_all / n * c_seg + (e / ((long long)n * segs)) * ldc + q_all % n] = (float)s;
}

// Wt[c][r] = W[r][c] for small matrices (the layer weights; blockIdx.z: several, w_step and wt_step floats apart)
__global__ void k_transpose(const float *__restrict__ W, long long ldw, int rows, int cols, float *__restrict__ Wt, long long ldt, long long w_step,
                            long long wt_step) {
    W += blockIdx.z * w_step;
    Wt += blockIdx.z * wt_step;
    __shared__ float tile[32][33];
    const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
    for (int y = ty; y < 32; y += 8)
        if (r0 + y < rows && c0 + tx < cols) tile[y][tx] = W[(long long)(r0 + y) * ldw + c0 + tx];
    __syncthreads();
    for (int y = ty; y < 32; y += 8)
        if (c0 + y < cols && r0 + tx < rows) Wt[(long long)(c0 + y) * ldt + r0 + tx] = tile[tx][y];
}

// y1 = A.v1, y2 = A.v2; LPR lanes per row stride over k, 64 / LPR rows per wavefront.  LPR is the smallest power of two (8 or more) whose
// lanes take the row in one step: with a whole wavefront per row 7 of 8 lanes idled on the 32 columns of an attention head (100,000 rows:
// 18 -> 4.8 us, 2.7 TB/s).
template <int VEC, int LPR>
__global__ __launch_bounds__(kThreads) void k_gemv2(const float *__restrict__ A, long long lda, long long n, int k,
                                                     const float *__restrict__ v1, const float *__restrict__ v2,
                                                     float *__restrict__ y1, float *__restrict__ y2, int a_sliced) {
    const int lane = threadIdx.x % LPR;
    const long long row = (long long)blockIdx.x * (kThreads / LPR) + threadIdx.x / LPR;
    const long long row_c = row < n ? row : n - 1;   // the reduction below needs every lane
    const float *a0 = a_sliced ? A + row_c * 32 : A + row_c * lda;
    float d1 = 0.f, d2 = 0.f;
    for (int kk = lane * VEC; kk < k; kk += LPR * VEC) {
        // slice-major: columns kk.. of this row sit in tile kk / 32 (a 4-float piece never straddles tiles)
        const float *a = a_sliced ? a0 + (long long)(kk >> 5) * n * 32 + (kk & 31) - kk : a0;
        float x[VEC];
        if (VEC == 4) { float4 v = *reinterpret_cast<const float4 *>(a + kk); x[0] = v.x; x[1 % VEC] = v.y; x[2 % VEC] = v.z; x[3 % VEC] = v.w; }
        else if (VEC == 2) { float2 v = *reinterpret_cast<const float2 *>(a + kk); x[0] = v.x; x[1 % VEC] = v.y; }
        else x[0] = a[kk];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            d1 = fmaf(x[e], v1[kk + e], d1);
            d2 = fmaf(x[e], v2[kk + e], d2);
        }
    }
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) {
        d1 += __shfl_xor(d1, off, 64);
        d2 += __shfl_xor(d2, off, 64);
    }
    if (lane == 0 && row < n) { y1[row] = d1; y2[row] = d2; }
}

template <int VEC>
void gemv2_launch(const float *A, long long lda, long long n, int k, const float *v1, const float *v2, float *y1, float *y2, int sl, hipStream_t s) {
    const int pieces = (k + VEC - 1) / VEC;
    const int lpr = pieces <= 8 ? 8 : pieces <= 16 ? 16 : pieces <= 32 ? 32 : 64;
    const dim3 grid((unsigned)((n + kThreads / lpr - 1) / (kThreads / lpr)));
    if (lpr == 8) hipLaunchKernelGGL((k_gemv2<VEC, 8>), grid, dim3(kThreads), 0, s, A, lda, n, k, v1, v2, y1, y2, sl);
    else if (lpr == 16) hipLaunchKernelGGL((k_gemv2<VEC, 16>), grid, dim3(kThreads), 0, s, A, lda, n, k, v1, v2, y1, y2, sl);
    else if (lpr == 32) hipLaunchKernelGGL((k_gemv2<VEC, 32>), grid, dim3(kThreads), 0, s, A, lda, n, k, v1, v2, y1, y2, sl);
    else hipLaunchKernelGGL((k_gemv2<VEC, 64>), grid, dim3(kThreads), 0, s, A, lda, n, k, v1, v2, y1, y2, sl);
}

}  // namespace

// blocks of 32 columns a wavefront of k_gemm_bf takes: as many as split the columns evenly in up to four, fewer where that leaves less
// than half of the chip's 2,048 wavefronts a tile of rows
static int gemm_bf_blocks(int64_t n, int m_store) {
    const int blocks = (m_store + 31) / 32;
    const long long tiles = (n + 31) / 32;
    int tn = (blocks + (blocks + 3) / 4 - 1) / ((blocks + 3) / 4);
    while (tn > 1 && tiles * ((blocks + tn - 1) / tn) < 1024) tn = tn > 2 ? 2 : 1;
    return tn;
}

// Products of 256 blocks of 256 rows by up to 128 columns and more (a block per compute unit) take six piece products, smaller ones eight: there the
// matrix pipe is seldom the bound and the two cost little (30,000 x 602 x 256 61 -> 72 us, 16,000 x 100 x 64 9.9 -> 10.1), and what a single term makes
// up stays as exact as on the fp32 instruction, which these sizes would take otherwise (96 us, 8.1).  Above, eight cost 13 % on average (64,000 x
// 602 x 256 119 -> 139).
static bool gemm_is_large(int64_t n, int m_store) {
    const int64_t blocks = (m_store + 31) / 32;
    return (n + 255) / 256 * (blocks <= 2 ? 1 : (blocks + 3) / 4) >= 256;
}

// Where the fixed costs of k_gemm_bf (about 6 us: W is fetched and cut before the first multiply, and a wavefront walks all of k) are earned
// back, in us on the fp32 kernels / here.  Large products by k and rows, outputs wider than 192 columns counting more: k = 16, 32 columns,
// 50,000 rows 6.2 / 7.2, 100,000 8.7 / 8.3.  Below that size, with eight piece products:
//   at most 32 columns: k = 48, 40,000 rows 7.6 / 7.9; k = 64, 20,000 rows 7.1 / 7.1; k = 128, 16,000 rows 7.6 / 8.6, 20,000 9.7 / 9.4; k = 512, 6,000
//     rows 10.6 / 15.8, 12,000 18.8 / 15.7;
//   at most 48: k = 100, 16,000 rows 8.7 / 10.0, 20,000 10.7 / 10.1;
//   64, for which the fp32 kernel has whole blocks: k = 100, 30,000 rows 9.7 / 11.0; k = 256, 16,000 rows 12.4 / 14.1, 20,000 15.7 / 14.5; k = 1024, 16,000
//     rows 36.5 / 42.7, 20,000 48.6 / 43.2;
//   more: k = 32, 192 columns, 30,000 rows 15.9 / 12.6; k = 64, 192 columns, 16,000 rows 10.2 / 10.7, 20,000 19.5 / 12.8; k = 128, 256 columns, 12,000 rows
//     14.7 / 14.5; k = 300, 96 columns, 6,000 rows 13.2 / 12.7; k = 1024, 96 columns, 6,000 rows 35.6 / 41.6, 9,000 48.6 / 43.0, 192 columns,
//     6,000 rows 48.3 / 44.1.
bool gemm_uses_pieces(int64_t n, int k, int m_store) {
    if (k < 16 || m_store <= 0) return false;
    const int64_t blocks = (m_store + 31) / 32, rows = n * (blocks > 6 ? blocks : 6) / 6;
    if (gemm_is_large(n, m_store)) return rows >= (k >= 64 ? 16000 : k >= 32 ? 28000 : 65536);
    if (k < 32) return false;
    if (blocks > 2) return rows >= (k >= 700 && blocks < 6 ? 8000 : k >= 300 ? 6000 : k >= 64 ? 16000 : 28000);
    if (k >= 300) return n >= (k >= 700 ? 20000 : 12000);
    if (k >= 128) return n >= (m_store > 48 ? 20000 : 16000);
    if (m_store > 32) return k >= 64 && n >= (m_store > 48 ? 65536 : 16000);
    return n >= (k >= 64 ? 20000 : 40000);
}

hipError_t launch_gemm(const float *A, int64_t lda, const float *W, int64_t ldw, float *Y, int64_t ldy, int64_t n,
                       int k, int m, int m_store, int act, hipStream_t s, const float *row_scale, KernelTimer *timer, bool y_sliced,
                       bool a_sliced, const float *add_sliced, SideWork *side) {
    if (n <= 0 || m_store <= 0) return launch_side(side, s);
    if (a_sliced) lda = 32;
    hipEvent_t t0 = timer ? timer->next() : nullptr, t1 = t0 ? timer->next() : nullptr;
    if (t1 && hipEventRecord(t0, s) != hipSuccess) return hipErrorUnknown;
    auto done = [&](hipError_t e) {
        if (e == hipSuccess && t1 && hipEventRecord(t1, s) != hipSuccess) return hipErrorUnknown;
        return e;
    };
    GemmArgs g;
    g.side = take_side(side);
    g.row_scale = row_scale;
    g.A = A; g.W = W; g.Y = Y; g.lda = lda; g.ldw = ldw; g.ldy = ldy; g.n = n;
    g.k = k; g.m = m; g.m_store = m_store; g.act = act; g.y_sliced = y_sliced ? 1 : 0;
    g.a_slice = a_sliced ? n * 32 : 32; g.add = add_sliced;
    int avec = 1, bvec = 1;
    const uintptr_t aa = reinterpret_cast<uintptr_t>(A), wa = reinterpret_cast<uintptr_t>(W);
    if (k % 4 == 0 && lda % 4 == 0 && aa % 16 == 0) avec = 4;
    else if (k % 2 == 0 && lda % 2 == 0 && aa % 8 == 0) avec = 2;
    if (m % 4 == 0 && ldw % 4 == 0 && wa % 16 == 0) bvec = 4;
    // Large products go to the bf16-piece kernel
    {
        const int tn = gemm_bf_blocks(n, m_store), blocks = (m_store + 31) / 32;
        g.n_bn = (blocks + tn - 1) / tn;
        // (a matrix to add costs the fp32 kernels more: TAGCN, update first, 100 -> 64 columns twice on 20,000 rows 80.6 / 72.3 us)
        const bool pieces = gemm_uses_pieces(n, k, m_store) || (add_sliced && k >= 64 && n >= 16000);
        if (pieces && lda < (1 << 20) && ldw < (1 << 20)) {   // leading dimensions: 32-bit byte offsets within a block
            auto launch = [&](auto full) {
                constexpr bool kFull = decltype(full)::value;
                switch (tn) {
                    case 1: return gemm_bf_launch<1, kFull>(g, s);
                    case 2: return gemm_bf_launch<2, kFull>(g, s);
                    case 3: return gemm_bf_launch<3, kFull>(g, s);
                    default: return gemm_bf_launch<4, kFull>(g, s);
                }
            };
            return done(gemm_is_large(n, m_store) ? launch(std::false_type()) : launch(std::true_type()));
        }
    }
    // Few enough 64 x 64 blocks to leave compute units idle: 32 x 32 blocks with k split over the wavefronts.  A small block reads its operands
    // for a quarter of the output and without LDS, so the line lies lower the more blocks there are and the longer k is.  Small / 64 x 64, us
    // with one call's launch in them (9.8), A in 16-byte loads: 308 small blocks (4,900 x 47) k = 256 10.0 / 13.5, 2,048 60 / 78; 504 (2,000 x
    // 256) k = 512 16.3 / 19.0, 8,192 226 / 248; 626 (10,000 x 64) k = 256 10.4 / 11.9, 384 16.6 / 15.7, 2,048 71 / 66.  A in 4-byte loads:
    // 40 blocks of 64 (600 x 256) k = 1,024 23 / 36, 4,096 131 / 137; 77 (4,900 x 47) k = 512 17.5 / 24.2, 1,024 42 / 44, 1,536 68 / 64; 128
    // (2,000 x 256) k = 384 16.1 / 16.6, 512 22.9 / 20.7; 157 (10,000 x 16) k = 384 15.2 / 16.0, 1,024 44 / 37; 157, but 626 small (10,000 x
    // 64) k = 128 10.2 / 9.9, 256 14.6 / 12.6, 1,024 58 / 37.
    const long long small_blocks = ((n + 31) / 32) * ((m_store + 31) / 32), blocks_64 = ((n + 63) / 64) * ((m_store + 63) / 64);
    const int small_k = avec == 4 ? (small_blocks <= 512 ? INT32_MAX : 256)
                                  : blocks_64 <= 64 ? INT32_MAX : blocks_64 <= 96 ? 1024 : small_blocks <= 512 ? 384 : 128;
    if (blocks_64 <= 160 && k <= small_k) {
        g.n_bn = (m_store + 31) / 32;
        const dim3 grid((unsigned)(((n + 31) / 32) * g.n_bn + g.side.blocks));
        if (avec == 4) hipLaunchKernelGGL(k_gemm_small<4>, grid, dim3(kThreads), 0, s, g);
        else hipLaunchKernelGGL(k_gemm_small<1>, grid, dim3(kThreads), 0, s, g);
        return done(hipGetLastError());
    }
    // tile choice: widest column tile that the output needs; small tiles when the big ones
    // would leave most of the 256 compute units without a workgroup
    const long long big_blocks = ((n + 127) / 128) * ((m_store + 127) / 128);
    if (m_store <= 32) {
        g.n_bn = 1;
        if ((n + 255) / 256 >= 256) return done(gemm_launch_vec<256, 32, 4, 1>(g, avec, bvec, s));
        g.n_bn = (m_store + 63) / 64;
        return done(gemm_launch_vec<64, 64, 2, 2>(g, avec, bvec, s));
    }
    if (m_store <= 64) {
        g.n_bn = 1;
        if ((n + 255) / 256 >= 256) return done(gemm_launch_vec<256, 64, 4, 1>(g, avec, bvec, s));
        return done(gemm_launch_vec<64, 64, 2, 2>(g, avec, bvec, s));
    }
    if (big_blocks >= 256) {
        g.n_bn = (m_store + 127) / 128;
        return done(gemm_launch_vec<128, 128, 2, 2>(g, avec, bvec, s));
    }
    g.n_bn = (m_store + 63) / 64;
    return done(gemm_launch_vec<64, 64, 2, 2>(g, avec, bvec, s));
}

hipError_t launch_tiles_gather(const TileSplit &T, const float *B_sliced, int64_t n_cols, int f, float *Bh, hipStream_t s) {
    if (T.n_slots <= 0 || f <= 0) return hipSuccess;
    const long long n_ranks = (long long)T.nt_c * 128;
    hipLaunchKernelGGL(k_gather_ranked_split, dim3((unsigned)((n_ranks / 8 * f + 255) / 256)), dim3(256), 0, s, B_sliced, (long long)n_cols, f,
                       T.order_c, n_ranks, reinterpret_cast<unsigned short *>(Bh), (const float2 *)nullptr);
    return hipGetLastError();
}

template <int MODE>
static void launch_attn_tiles(const DenseTilesAttnArgs &a, int n_seg, int nb_count, hipStream_t s) {
    DenseTilesAttnArgs g = a;
    const int nw = nb_count >= 5 ? 8 : nb_count >= 3 ? 4 : nb_count;   // wavefronts (32-column blocks) per workgroup
    g.n_bn = (nb_count + nw - 1) / nw;
    const dim3 grid((unsigned)(n_seg * g.n_bn));
    if (nw == 8) hipLaunchKernelGGL((k_dense_tiles_attn_bf<MODE, 8>), grid, dim3(512), 0, s, g);
    else if (nw == 4) hipLaunchKernelGGL((k_dense_tiles_attn_bf<MODE, 4>), grid, dim3(256), 0, s, g);
    else if (nw == 2) hipLaunchKernelGGL((k_dense_tiles_attn_bf<MODE, 2>), grid, dim3(128), 0, s, g);
    else hipLaunchKernelGGL((k_dense_tiles_attn_bf<MODE, 1>), grid, dim3(64), 0, s, g);
}

// f: a multiple of 32.  Bh: room for 6 bytes per (rank, column).
// local_shift (attention on the pattern itself): launch_tile_stats has run on this stream - the vectors are in rank order and the shift of a
// row is the maximum over its tile entries, so the call needs no row statistics; the join rescales (tile_shift of the combine launchers)
hipError_t launch_dense_tiles(const TileSplit &T, const float *B_sliced, int64_t n_cols, int f, float *Bh, hipStream_t s, const float *s_l,
                              const float *s_r, const float2 *mz, float slope, bool transposed, bool gathered, bool local_shift) {
    if (T.n_slots <= 0 || f <= 0) return hipSuccess;
    const long long n_ranks = (long long)T.nt_c * 128;
    unsigned short *Bq = reinterpret_cast<unsigned short *>(Bh);
    const int nb_count = f / 32;
    if (!gathered)   // pieces of the operand in lane order (the transposed attention mode folds 1 / z of the softmax row into them)
        hipLaunchKernelGGL(k_gather_ranked_split, dim3((unsigned)((n_ranks / 8 * f + 255) / 256)), dim3(256), 0, s, B_sliced, (long long)n_cols, f,
                           T.order_c, n_ranks, Bq, (s_l && transposed) ? mz : (const float2 *)nullptr);
    if (!s_l) {
        DenseTilesBfArgs b;
        b.bits = T.bits; b.seg_first = T.seg_first; b.slot_ct = T.slot_ct; b.Bq = Bq; b.part = T.part;
        b.plane = n_ranks * f; b.f = f;
        const int waves = nb_count < 4 ? nb_count : 4;
        b.n_bn = (nb_count + 3) / 4;
        hipLaunchKernelGGL(k_dense_tiles_bf, dim3((unsigned)(T.n_seg * b.n_bn)), dim3(64 * waves), 0, s, b);
    } else {
        DenseTilesAttnArgs g;
        g.bits = T.bits; g.seg_first = T.seg_first; g.slot_ct = T.slot_ct; g.seg_rt = T.seg_rt; g.Bq = Bq; g.part = T.part;
        g.plane = n_ranks * f; g.f = f; g.n_bn = 1; g.slope = slope;
        const int n_r = T.nt_r * 128, n_c = T.nt_c * 128;
        const dim3 vgrid((unsigned)(((n_r > n_c ? n_r : n_c) + 255) / 256));
        if (transposed) {
            g.u_rank = T.rank_vec; g.m_rank = nullptr; g.v_rank = T.rank_vec + n_r; g.mc_rank = T.rank_vec + n_r + n_c;
            hipLaunchKernelGGL(k_gather_ranked_vecs_t, vgrid, dim3(256), 0, s, s_l, s_r, mz, T.order_r, n_r, T.order_c, n_c, T.rank_vec,
                               T.rank_vec + n_r, T.rank_vec + n_r + n_c);
            launch_attn_tiles<kTilesAttnT>(g, T.n_seg, nb_count, s);
        } else {
            g.u_rank = T.rank_vec; g.m_rank = T.rank_vec + n_r; g.v_rank = T.rank_vec + 2 * n_r; g.mc_rank = nullptr;
            if (!local_shift)
                hipLaunchKernelGGL(k_gather_ranked_vecs, vgrid, dim3(256), 0, s, s_l, s_r, mz, T.order_r, n_r, T.order_c, n_c, T.rank_vec,
                                   T.rank_vec + n_r, T.rank_vec + 2 * n_r);
            launch_attn_tiles<kTilesAttn>(g, T.n_seg, nb_count, s);
        }
    }
    const long long threads = (long long)T.nt_r * 128 * (f / 4);
    hipLaunchKernelGGL(k_tiles_reduce, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, (const float *)T.part, T.rt_seg, T.nt_r, f, T.dh);
    return hipGetLastError();
}

hipError_t launch_tile_stats(const TileSplit &T, const float *s_l, const float *s_r, float slope, hipStream_t s) {
    if (T.n_slots <= 0 || T.n_seg <= 0) return hipSuccess;
    const int n_r = T.nt_r * 128, n_c = T.nt_c * 128;
    hipLaunchKernelGGL(k_gather_ranked_vecs, dim3((unsigned)(((n_r > n_c ? n_r : n_c) + 255) / 256)), dim3(256), 0, s, s_l, s_r, (const float2 *)nullptr,
                       T.order_r, n_r, T.order_c, n_c, T.rank_vec, T.rank_vec + n_r, T.rank_vec + 2 * n_r);
    hipLaunchKernelGGL(k_tile_stats, dim3((unsigned)T.n_seg), dim3(256), 0, s, T.bits, T.seg_first, T.slot_ct, T.seg_rt, (const float *)T.rank_vec,
                       (const float *)(T.rank_vec + 2 * n_r), slope, T.seg_stats);
    hipLaunchKernelGGL(k_tile_row_max, dim3((unsigned)((n_r + 255) / 256)), dim3(256), 0, s, T.rt_seg, (const float2 *)T.seg_stats, n_r, T.rank_vec + n_r);
    return hipGetLastError();
}

hipError_t launch_tile_stats_merge(const TileSplit &T, float2 *stats, int64_t n_rows, hipStream_t s) {
    if (T.n_slots <= 0 || T.n_seg <= 0 || n_rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tile_stats_merge, dim3((unsigned)((n_rows + 255) / 256)), dim3(256), 0, s, stats, (long long)n_rows, T.rank_r, T.nt_r * 128,
                       T.rt_seg, (const float2 *)T.seg_stats);
    return hipGetLastError();
}

hipError_t launch_tiles_sddmm(const TileSplit &T, const float *L_sliced, int64_t n_rows, const float *R_sliced, int64_t n_cols, int f, float *Lh,
                              float *Rh, float *Dt, hipStream_t s) {
    if (T.n_slots <= 0 || f <= 0) return hipSuccess;
    const long long nr = (long long)T.nt_r * 128, nc = (long long)T.nt_c * 128;
    hipLaunchKernelGGL(k_gather_ranked_rows, dim3((unsigned)((nr * (f / 4) + 255) / 256)), dim3(256), 0, s, L_sliced, (long long)n_rows, f, T.order_r, nr, Lh, (const float2 *)nullptr);
    hipLaunchKernelGGL(k_gather_ranked_rows, dim3((unsigned)((nc * (f / 4) + 255) / 256)), dim3(256), 0, s, R_sliced, (long long)n_cols, f, T.order_c, nc, Rh, (const float2 *)nullptr);
    hipLaunchKernelGGL(k_tiles_sddmm, dim3((unsigned)T.n_slots), dim3(kThreads), 0, s, (const float *)Lh, (const float *)Rh, f, T.slot_rt, T.slot_ct, Dt);
    return hipGetLastError();
}

hipError_t launch_tiles_combine(const TileSplit &T, float *C, int64_t n_rows, int f_store, int64_t ldc, bool c_sliced, int f, const float *r,
                                const float2 *mz, int act, hipStream_t s, const int32_t *row_ptr_rem, int chunk_nnz, const float *carry, int f_carry,
                                const float *tile_shift) {
    if (n_rows <= 0 || f_store <= 0) return hipSuccess;
    const long long threads = (long long)n_rows * ((f_store + 3) / 4);
    // T.dh rows are f floats, f a multiple of 32; carry slots are f_carry floats apart
    const int vec4 = (reinterpret_cast<uintptr_t>(C) % 16 == 0 && (c_sliced || ldc % 4 == 0) &&
                      (!carry || (f_carry % 4 == 0 && reinterpret_cast<uintptr_t>(carry) % 16 == 0))) ? 1 : 0;
    if (!carry || chunk_nnz <= 0) row_ptr_rem = nullptr;
    hipLaunchKernelGGL(k_tiles_combine, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, C, (long long)n_rows, f_store,
                       c_sliced ? 32LL : (long long)ldc, c_sliced ? (long long)n_rows * 32 : 32LL, (const float *)T.dh, f, T.rank_r, T.nt_r * 128, r, mz,
                       act, vec4, row_ptr_rem, chunk_nnz, carry, f_carry, mz ? tile_shift : nullptr);
    return hipGetLastError();
}

hipError_t launch_tiles_combine_pm(const TileSplit &T, float *C, int64_t n_rows, int f_store, int64_t ldc, bool c_sliced, int f, const float *r,
                                   const float2 *mz, int act, hipStream_t s, const float *part, int n_panels, const int32_t *seg_ptr, int chunk_nnz,
                                   const float *carry, int f_carry, const float *tile_shift) {
    if (n_rows <= 0 || f_store <= 0) return hipSuccess;
    if (f % 32 != 0 || f_carry % 4 != 0 || reinterpret_cast<uintptr_t>(part) % 16 != 0 || reinterpret_cast<uintptr_t>(carry) % 16 != 0 || chunk_nnz <= 0)
        return hipErrorInvalidValue;
    const long long threads = (long long)n_rows * ((f_store + 3) / 4);
    const int vec4 = (reinterpret_cast<uintptr_t>(C) % 16 == 0 && (c_sliced || ldc % 4 == 0)) ? 1 : 0;
    hipLaunchKernelGGL(k_tiles_combine_pm, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, C, (long long)n_rows, f_store,
                       c_sliced ? 32LL : (long long)ldc, c_sliced ? (long long)n_rows * 32 : 32LL, (const float *)T.dh, f, T.rank_r, T.nt_r * 128, r, mz,
                       act, vec4, part, n_panels, seg_ptr, chunk_nnz, carry, f_carry, mz ? tile_shift : nullptr);
    return hipGetLastError();
}

hipError_t launch_head_scores(const float *theta, int64_t n, int heads, int d, const float *a_l, const float *a_r, float *s_l, float *s_r, hipStream_t s) {
    if (n <= 0 || heads <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_head_scores, dim3((unsigned)((n + kThreads / 8 * kScoreRows - 1) / (kThreads / 8 * kScoreRows)), (unsigned)heads), dim3(kThreads), 0,
                       s, theta, (long long)n, d, a_l, a_r, s_l, s_r);
    return hipGetLastError();
}

hipError_t launch_pad_heads(const float *W, int64_t ldw, int f_in, int heads, int d, float *out, int64_t ldo, hipStream_t s) {
    const int dp = pad32(d);
    const long long total = (long long)f_in * heads * dp;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pad_heads, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, W, (long long)ldw, f_in, heads, d, dp, out, (long long)ldo);
    return hipGetLastError();
}

hipError_t launch_gemv2(const float *A, int64_t lda, int64_t n, int k, const float *v1, const float *v2, float *y1,
                        float *y2, hipStream_t s, bool a_sliced) {
    if (n <= 0) return hipSuccess;
    const uintptr_t aa = reinterpret_cast<uintptr_t>(A);
    if (a_sliced) lda = 32;
    const int sl = a_sliced ? 1 : 0;
    if (k % 4 == 0 && lda % 4 == 0 && aa % 16 == 0) gemv2_launch<4>(A, (long long)lda, (long long)n, k, v1, v2, y1, y2, sl, s);
    else if (k % 2 == 0 && lda % 2 == 0 && aa % 8 == 0) gemv2_launch<2>(A, (long long)lda, (long long)n, k, v1, v2, y1, y2, sl, s);
    else gemv2_launch<1>(A, (long long)lda, (long long)n, k, v1, v2, y1, y2, sl, s);
    return hipGetLastError();
}

// Slabs: as many workgroups as the chip holds at once, one a compute unit (two of the 64-column kernel's): the slab sums are 128 KB a block in fp64,
// written and read again, and the workgroups that did not fit ran in a round of their own.  With 256 / 512 / 768 workgroups (twice as many
// of the 64-column kernel), training passes, us: four heads on 100,000 nodes 570 / 575 / 592, GATv2 on 50,000 601 / 619 / 631, K-hop on 100,000 390 / 402 / 421, two layers on
// 233,000 8,580 / 8,549 / 8,584.
// Where that leaves an eighth of the chip idle (from 86 blocks on a whole number of slabs seldom fills it) as many slabs, up to three rounds of them, as make the rounds
// shortest: a round is a slab's rows at 59 ns (a block of 128 x 128), a slab more its sums at 5 TB/s.  dW of 1,433 x 1,433 over 50,000 rows (144 blocks) with 1 / 2 / 3 / 5 / 6
// slabs 2,957 / 3,188 / 2,277 / 2,146 / 2,305 us, of 1,433 x 1,000 (96) with 2 / 3 / 5 / 8 1,547 / 1,984 / 1,358 / 1,325, of 1,280 x 1,100 over 20,000 (90) with 2 / 5 / 8 / 9 634 / 557 /
// 553 / 623; 3,703 x 500 (116 blocks, nine tenths of the chip) with 2 / 4 / 6 661 / 660 / 674.
int gemm_tn_splits(int64_t k, int m, int n, int segs) {
    const long long tiles = (long long)((m + 127) / 128) * ((n + 127) / 128) * segs;
    const long long most = (768 + tiles - 1) / tiles;   // below 4,096 rows the fp32 kernel runs, three workgroups a compute unit
    long long s = most;
    if (k >= 4096) {
        const long long slots = n <= 64 ? 512 : 256;
        auto rounds = [&](long long c) { return (c * tiles + slots - 1) / slots; };
        s = slots / tiles > 1 ? slots / tiles : 1;
        if (8 * s * tiles < 7 * rounds(s) * slots) {
            const double sums = 16.0 * m * n * segs / 5e12, rows = 59e-9 * (double)k;
            auto time = [&](long long c) { return rows * (double)rounds(c) / (double)c + sums * (double)c; };
            for (long long c = s + 1; c <= most; ++c)
                if (time(c) < time(s)) s = c;
        }
    }
    const long long max_s = (k + 4 * KT - 1) / (4 * KT);  // at least four k-tiles per slab
    if (s > max_s) s = max_s;
    return (int)(s < 1 ? 1 : s);
}

size_t gemm_tn_bytes(int64_t k, int m, int n, int segs) {
    return align_up((size_t)gemm_tn_splits(k, m, n, segs) * (size_t)m * (size_t)n * segs * sizeof(double), 256);
}

hipError_t launch_gemm_tn(const float *A, int64_t lda, const float *B, int64_t ldb, int64_t k, int m, int n, float *C, int64_t ldc,
                          const Slabs &part, hipStream_t s, int segs, int64_t b_seg, int64_t c_seg) {
    if (m <= 0 || n <= 0) return hipSuccess;
    if (gemm_tn_bytes(k, m, n, segs) > part.bytes) return hipErrorInvalidValue;
    GemmTnArgs g;
    g.A = A; g.B = B; g.part = part.p; g.lda = lda; g.ldb = ldb; g.k = k > 0 ? k : 0; g.m = m; g.n = n;
    g.segs = segs; g.b_seg = b_seg;
    g.n_bn = (n + 127) / 128;
    g.n_tiles = ((m + 127) / 128) * g.n_bn * segs;
    const int splits = gemm_tn_splits(k, m, n, segs);
    g.k_per_split = (int)(((g.k + splits - 1) / splits + KT - 1) / KT * KT);
    if (g.k_per_split < KT) g.k_per_split = KT;
    const bool va = (m % 4 == 0 && lda % 4 == 0 && reinterpret_cast<uintptr_t>(A) % 16 == 0);
    const bool vb = (n % 4 == 0 && ldb % 4 == 0 && (segs == 1 || b_seg % 4 == 0) && reinterpret_cast<uintptr_t>(B) % 16 == 0);
    dim3 grid((unsigned)(g.n_tiles * splits));
    // long reductions (the weight gradients of a layer) take the bf16-piece kernel
    if (g.k >= 4096 && g.k_per_split >= 64) {
        if (n <= 64) hipLaunchKernelGGL(k_gemm_tn_bf<1>, grid, dim3(kThreads), 0, s, g);   // one block of columns either way
        else hipLaunchKernelGGL(k_gemm_tn_bf<2>, grid, dim3(2 * kThreads), 0, s, g);
    }
    else if (va && vb) hipLaunchKernelGGL((k_gemm_tn<4, 4>), grid, dim3(kThreads), 0, s, g);
    else if (va) hipLaunchKernelGGL((k_gemm_tn<4, 1>), grid, dim3(kThreads), 0, s, g);
    else if (vb) hipLaunchKernelGGL((k_gemm_tn<1, 4>), grid, dim3(kThreads), 0, s, g);
    else hipLaunchKernelGGL((k_gemm_tn<1, 1>), grid, dim3(kThreads), 0, s, g);
    const long long mn = (long long)m * n * segs;
    hipLaunchKernelGGL(k_sum_splits, dim3((unsigned)((mn + kSumElems - 1) / kSumElems)), dim3(kSumElems * kSumLanes), 0, s, part.p, splits, mn, n,
                       segs, C, (long long)ldc, (long long)c_seg);
    return hipGetLastError();
}

hipError_t launch_transpose(const float *W, int64_t ldw, int rows, int cols, float *Wt, int64_t ldt, hipStream_t s, int count, int64_t w_step,
                            int64_t wt_step) {
    if (rows <= 0 || cols <= 0 || count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_transpose, dim3((unsigned)((cols + 31) / 32), (unsigned)((rows + 31) / 32), (unsigned)count), dim3(256), 0, s, W, (long long)ldw,
                       rows, cols, Wt, (long long)ldt, (long long)w_step, (long long)wt_step);
    return hipGetLastError();
}

}  // namespace sensei
