// Learned surrogate: a Fourier neural operator that maps eight pulse and
// optics parameters to the six-component focal-window field, trained on the
// solver's own output.  The paper motivates fast generation of many focusing
// runs as training data for learned models (Sec. I and Sec. III.B.3); the
// operator itself is this library's.
//
// Architecture (fixed): 64^3 window, width 32, 12 kept modes per axis
// (kx in [0, 12), ky and kz in [0, 12) U [52, 64)), 3 Fourier layers,
// projection 32 -> 128 -> 6, GELU(x) = x (1 + erf(x / sqrt 2)) / 2.
//   v0      = [p, x, y, z] W0 + b0                      (lift, fp32)
//   z_l     = irfft3(R_l . rfft3(v_l)|kept) + v_l W_l + b_l
//   v_l+1   = GELU(z_l) (l < 2),  v_3 = z_2
//   out     = GELU(v_3 P1 + c1) P2 + c2
// Loss: mean over samples of ||out - y|| / ||y||.
//
// Arithmetic: every contraction runs on bf16 MFMA with fp32 accumulation.
// Learned weights enter as bf16 working copies of fp32 master weights; the
// truncated DFT matrices (float64-built) and the activations they multiply
// are split into bf16 hi + lo parts and multiplied with three MFMAs, which
// keeps the spectral transforms at about fp32 accuracy.
//
// Data layout (fp32, one sample; B samples are stacked outermost):
//   node tensor  [z][y][x][c]                 64^3 x 32, channel fastest
//   X1 (x pass)  [z][y][s][kx][c]             s: 0 real, 1 imaginary
//   X2 (y pass)  [ky][z][s][kx][c]
//   modes        [kz][s][ky][kx][c]           mode q = (kz * 24 + ky) * 12 + kx
//   out, target  [6][z][y][x]
// Every stage is "a small constant matrix applied along one axis" and runs as
// one strided GEMM whose row/column index maps are two-level affine.
#include "engine.h"

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <memory>

namespace tf {
namespace fno {

constexpr int N = 64, N3 = N * N * N, C = 32, M = 12, NPAR = 8, HID = 128, NOUT = 6, LAYERS = 3;
constexpr int KS = 2 * M;                 // kept ky / kz values
constexpr int NMODES = KS * KS * M;       // 6912
constexpr int LINE = M * C;               // 384 floats: one (kx, c) block
constexpr int64_t NODE_SZ = int64_t(N3) * C;                // node tensor per sample
constexpr int64_t X1_SZ = int64_t(N) * N * 2 * LINE;        // 3,145,728
constexpr int64_t X2_SZ = int64_t(KS) * N * 2 * LINE;       // 1,179,648
constexpr int64_t X3_SZ = int64_t(KS) * 2 * KS * LINE;      // 442,368
constexpr int64_t OUT_SZ = int64_t(NOUT) * N3;
constexpr int CHUNK = 4096;               // nodes per split-K block of the weight gradients
constexpr int KSLOTS = 4 * 2 * 2 * 32 * 8; // one 128-row operand in kappa fragment order
constexpr int NCHUNK = N3 / CHUNK;

// Flat parameter vector (fp32): W0 (11x32), b0, then per layer W (32x32),
// b (32), R (NMODES x 32 x 32 complex as [q][c][o][re, im]), then P1 (32x128),
// c1, P2 (128 x 6K), c2 (6K) for a head of K basis fields.  Row-major, input
// index first.
constexpr int64_t OFF_W0 = 0, OFF_B0 = 11 * C;
constexpr int64_t LAYER_SZ = C * C + C + int64_t(NMODES) * C * C * 2;
constexpr int64_t OFF_L0 = OFF_B0 + C;
constexpr int64_t off_w(int l) { return OFF_L0 + l * LAYER_SZ; }
constexpr int64_t off_b(int l) { return off_w(l) + C * C; }
constexpr int64_t off_r(int l) { return off_b(l) + C; }
constexpr int64_t OFF_P1 = OFF_L0 + LAYERS * LAYER_SZ;
constexpr int64_t OFF_C1 = OFF_P1 + C * HID;
constexpr int64_t OFF_P2 = OFF_C1 + HID;
constexpr int64_t off_c2(int nb) { return OFF_P2 + int64_t(HID) * NOUT * nb; }
constexpr int64_t nparams(int nb) { return off_c2(nb) + NOUT * nb; }

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// erf by Abramowitz & Stegun 7.1.28 (|error| <= 3e-7; about 2e-6 after
// float32 rounding, far below the bf16 rounding of every value a GELU
// feeds): for u >= 0, erf(u) = 1 - 1 / (1 + a1 u + ... + a6 u^6)^16.  One
// reciprocal and no exponential; large u gives an infinite power and 1.
__device__ __forceinline__ float erf_as(float u) {
    const float a = fabsf(u);
    const float q = 1.0f + a * (0.0705230784f + a * (0.0422820123f + a * (0.0092705272f +
                                a * (0.0001520143f + a * (0.0002765672f + a * 0.0000430638f)))));
    const float q2 = q * q, q4 = q2 * q2, q8 = q4 * q4;
    const float r = 1.0f - __builtin_amdgcn_rcpf(q8 * q8);
    return __builtin_copysignf(r, u);      // r >= 0
}
__device__ __forceinline__ float gelu(float x) {
    return 0.5f * x * (1.0f + erf_as(x * 0.70710678118654752f));
}
// GELU'(x) = Phi(x) + x phi(x), with the standard normal density phi
__device__ __forceinline__ float gelu_d(float x) {
    const float ex = __expf(-0.5f * x * x);
    return 0.5f * (1.0f + erf_as(x * 0.70710678118654752f)) + x * ex * 0.39894228040143268f;
}

// ---------------------------------------------------------------------------
// Generic strided GEMM  C[b] = A[b] (M x K) . B[b] (K x N)
// ---------------------------------------------------------------------------

// Two-level affine index map: i -> (i >> sh) * hi + (i & (2^sh - 1)) * lo.
// Within one batch entry every operand spans fewer than 2^31 elements (the
// largest, the modes of 128 samples, 57 M).
struct Ix {
    int sh, hi, lo;
};
__device__ __forceinline__ uint32_t ixoff(Ix a, int i) {
    return uint32_t(i >> a.sh) * uint32_t(a.hi) + uint32_t(i & ((1 << a.sh) - 1)) * uint32_t(a.lo);
}

struct Operand {
    const void* p;
    int64_t b1, b2;       // element strides of blockIdx.y and blockIdx.z
    Ix r, c;              // row and column maps
    int ones_from;        // rows >= ones_from read 1 (A only; large value: none)
    int fast_k;           // consecutive threads walk k (k is the contiguous index)
    int vec;              // groups of 4 along the contiguous index are contiguous and aligned
};
struct Result {
    float* p;
    int64_t b1, b2;
    Ix r, c;
};
struct GemmArgs {
    Operand a, b;
    Result c;
    int M, N, K;
};

template <typename T> struct Vec4;
template <> struct Vec4<float> { typedef __attribute__((ext_vector_type(4))) float type; };
template <> struct Vec4<bf16> { typedef __attribute__((ext_vector_type(4))) __bf16 type; };

// One thread's share of a ROWS x 32 slice of an operand, on its way from memory
// to LDS ("rows" are the M index of A or the N index of B).  Each item is one
// row and 8 consecutive k, stored as bf16 (hi and, for SPLIT, lo parts), k
// contiguous, with one 16-byte LDS write per part.  Neighbouring threads take
// neighbouring k groups when k is the contiguous index in memory (two 4-element
// loads when aligned), else neighbouring rows (coalesced single loads); either
// way the 16-byte writes of a quarter-wave start 20 banks apart (row pitch 80 B)
// or are contiguous, so they do not collide.  load() keeps the elements as they
// are in memory, so that nothing waits for them before store(); positions past
// the end are read from the last valid one and replaced in store().
template <int ROWS, int NT, typename TT, bool SPLIT, bool IS_B> struct Slice {
    static constexpr int BK = 32, PITCH = BK + 8, KG = BK / 8, ITEMS = ROWS * KG, IT = (ITEMS + NT - 1) / NT;
    typedef typename Vec4<TT>::type V4;
    V4 v[IT][2];

    static __device__ __forceinline__ void item(const Operand& o, int it, int& rr, int& kg) {
        const int t = (int(threadIdx.x) + it * NT) % ITEMS;
        if (o.fast_k) { rr = t / KG; kg = t % KG; }
        else          { rr = t % ROWS; kg = t / ROWS; }
    }
    __device__ __forceinline__ void load(const TT* P, const Operand& o, const uint32_t* rowoff, int k0, int K) {
        const Ix km = IS_B ? o.r : o.c;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            int rr, kg;
            item(o, it, rr, kg);
            const int k = k0 + 8 * kg;
            if (o.vec) {
                v[it][0] = *(const V4*)(P + (rowoff[it] + ixoff(km, min(k, K - 4))));
                v[it][1] = *(const V4*)(P + (rowoff[it] + ixoff(km, min(k + 4, K - 4))));
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[it][e >> 2][e & 3] = P[rowoff[it] + ixoff(km, min(k + e, K - 1))];
            }
        }
    }
    static __device__ __forceinline__ void rows(uint32_t* rowoff, const Operand& o, int r0, int nrows) {
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            int rr, kg;
            item(o, it, rr, kg);
            const int last = (IS_B ? nrows : min(nrows, o.ones_from)) - 1;
            rowoff[it] = ixoff(IS_B ? o.c : o.r, min(r0 + rr, last));
        }
    }
    __device__ __forceinline__ void store(bf16* s0, bf16* s1, const Operand& o, int r0, int k0, int nrows,
                                          int K) const {
        const bool whole = r0 + ROWS <= (IS_B ? nrows : min(nrows, o.ones_from)) && k0 + BK <= K;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            int rr, kg;
            item(o, it, rr, kg);
            if (ITEMS % NT != 0 && int(threadIdx.x) + it * NT >= ITEMS) break;
            float f[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = (float)v[it][e >> 2][e & 3];
            if (!whole) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int gr = r0 + rr;
                    if (!IS_B && gr >= o.ones_from) f[e] = 1.0f;
                    if (gr >= nrows || k0 + 8 * kg + e >= K) f[e] = 0.0f;
                }
            }
            bf16x8 hi, lo;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bf16 h = (bf16)f[e];
                hi[e] = h;
                lo[e] = (bf16)(f[e] - (float)h);
            }
            *(bf16x8*)&s0[rr * PITCH + 8 * kg] = hi;
            if constexpr (SPLIT) *(bf16x8*)&s1[rr * PITCH + 8 * kg] = lo;
        }
    }
};

// Each wave owns 32x32 output sub-tiles; the K loop stages 32-wide slices of
// A and B in LDS as bf16 (hi and, for SPLIT, lo parts), k contiguous so each
// lane reads its eight k values with one 16-byte LDS load.  DEPTH slices are in
// flight in registers ahead of the one being multiplied: the two of a mode's
// mixing (batch 1: 20 -> 15 us, the matrices' 57 MB bound it), one where the
// slices of five blocks per CU cover the latency (the x contraction, 137 us at
// 16 samples, 5.1 TB/s; with four in flight 160).
template <int BM, int BN, int NW, typename TA, typename TB, bool SPLIT, int DEPTH>
__global__ __launch_bounds__(64 * NW) void k_gemm(GemmArgs g) {
    constexpr int BK = 32, PITCH = BK + 8, NT = 64 * NW;
    constexpr int SUBN = BN / 32, SUB = (BM / 32) * SUBN, PER = SUB / NW;
    static_assert(SUB % NW == 0, "sub-tiles must divide among the waves");
    constexpr int NP = SPLIT ? 2 : 1;
    __shared__ __attribute__((aligned(16))) bf16 sa[NP][BM * PITCH];
    __shared__ __attribute__((aligned(16))) bf16 sb[NP][BN * PITCH];

    const int tilesN = (g.N + BN - 1) / BN;
    const int m0 = (blockIdx.x / tilesN) * BM, n0 = (blockIdx.x % tilesN) * BN;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t = lane & 31, grp = lane >> 5;
    const TA* A = (const TA*)g.a.p + blockIdx.y * g.a.b1 + blockIdx.z * g.a.b2;
    const TB* B = (const TB*)g.b.p + blockIdx.y * g.b.b1 + blockIdx.z * g.b.b2;

    typedef Slice<BM, NT, TA, SPLIT, false> SA;
    typedef Slice<BN, NT, TB, SPLIT, true> SB;
    SA ra[DEPTH];
    SB rb[DEPTH];
    uint32_t rowa[SA::IT], rowb[SB::IT];
    SA::rows(rowa, g.a, m0, g.M);
    SB::rows(rowb, g.b, n0, g.N);
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        if (d * BK < g.K) {
            ra[d].load(A, g.a, rowa, d * BK, g.K);
            rb[d].load(B, g.b, rowb, d * BK, g.K);
        }

    f32x16 acc[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[p][r] = 0.0f;

    for (int kb = 0; kb < g.K; kb += DEPTH * BK) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const int k0 = kb + d * BK;
            if (k0 >= g.K) break;
            ra[d].store(sa[0], sa[NP - 1], g.a, m0, k0, g.M, g.K);
            rb[d].store(sb[0], sb[NP - 1], g.b, n0, k0, g.N, g.K);
            if (k0 + DEPTH * BK < g.K) {
                ra[d].load(A, g.a, rowa, k0 + DEPTH * BK, g.K);
                rb[d].load(B, g.b, rowb, k0 + DEPTH * BK, g.K);
            }
            __syncthreads();
#pragma unroll
            for (int p = 0; p < PER; ++p) {
                const int st = wave * PER + p, mt = st / SUBN, nt = st % SUBN;
#pragma unroll
                for (int ks = 0; ks < BK / 16; ++ks) {
                    const int ao = (mt * 32 + t) * PITCH + ks * 16 + 8 * grp;
                    const int bo = (nt * 32 + t) * PITCH + ks * 16 + 8 * grp;
                    const bf16x8 ah = *(const bf16x8*)&sa[0][ao];
                    const bf16x8 bh = *(const bf16x8*)&sb[0][bo];
                    acc[p] = mfma(ah, bh, acc[p]);
                    if constexpr (SPLIT) {
                        const bf16x8 al = *(const bf16x8*)&sa[NP - 1][ao];
                        const bf16x8 bl = *(const bf16x8*)&sb[NP - 1][bo];
                        acc[p] = mfma(ah, bl, acc[p]);
                        acc[p] = mfma(al, bh, acc[p]);
                    }
                }
            }
            __syncthreads();
        }
    }

    float* Cp = g.c.p + blockIdx.y * g.c.b1 + blockIdx.z * g.c.b2;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int st = wave * PER + p, mt = st / SUBN, nt = st % SUBN;
        const int col = n0 + nt * 32 + t;
        if (col >= g.N) continue;
        float* Cc = Cp + ixoff(g.c.c, col);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = m0 + mt * 32 + 8 * (r >> 2) + 4 * grp + (r & 3);
            if (row < g.M) Cc[ixoff(g.c.r, row)] = acc[p][r];
        }
    }
}

// ---------------------------------------------------------------------------
// y and z transforms: out = A (M x K) . in, A one of the block DFT matrices
// ---------------------------------------------------------------------------

// in and out are the X1, X2 and mode layouts: rows (index, s) at (i >> 1) * hi +
// (i & 1) * lo, LINE contiguous columns, one such matrix per (y, b).
struct AxisArgs {
    const float* A;       // [M][K]
    const float* in;
    float* out;
    int in_hi, in_lo, out_hi, out_lo;
    int64_t in_y, in_b, out_y, out_b;
    int ny, nitems;       // an item: 32 columns of one matrix and MT row tiles
};

// element e of (hi, lo) <- bf16 split of v, as v is rounded to float32: lo must
// not contract with the product that v comes from
__device__ __forceinline__ void split(float v, bf16x8& hi, bf16x8& lo, int e) {
#pragma clang fp contract(off)
    const bf16 h = (bf16)v;
    hi[e] = h;
    lo[e] = (bf16)(v - (float)h);
}

// A wave takes 32 columns and MT tiles of 32 rows of A at a time.  Its columns
// are the B operand as they lie (lane (column, k group), 128 bytes per row and
// group), so they go from memory to the MFMAs without LDS, and the registers of
// a k step are refilled for the wave's next item as soon as they are split.  A
// is split once per block into LDS in fragment order.  The order of the
// products is that of k_gemm.  Memory bounds it; see launch_axis for MT.
template <int M, int K, int MT>
__global__ __launch_bounds__(256) void k_axis(AxisArgs a) {
    constexpr int KN = K / 16, MTOT = (M + 31) / 32, MG = MTOT / MT, CG = LINE / 32;
    __shared__ bf16x8 frag[KN * MTOT][2][64];
    const int lane = threadIdx.x & 63, t = lane & 31, grp = lane >> 5;
    const int stride = gridDim.x * 4;
    int item = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    float v[KN][8];
    auto column = [&](int i, int64_t y, int64_t b) {
        const int q = i / MG / CG;
        return int64_t(q / a.ny) * b + int64_t(q % a.ny) * y + (i / MG % CG) * 32;
    };
    auto load = [&](const float* src, int ks) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[ks][e] = (src + (8 * ks + (e >> 1)) * a.in_hi + (e & 1) * a.in_lo)[uint32_t(4 * grp * a.in_hi + t)];
    };
    {
        const float* src = a.in + column(min(item, a.nitems - 1), a.in_y, a.in_b);
#pragma unroll
        for (int ks = 0; ks < KN; ++ks) load(src, ks);
    }
    for (int f = threadIdx.x; f < KN * MTOT * 64; f += 256) {
        const int ft = f & 31, fg = (f >> 5) & 1, q = f >> 6, row = 32 * (q % MTOT) + ft;
        const float* src = a.A + min(row, M - 1) * K + 16 * (q / MTOT) + 8 * fg;
        const float4 u0 = *(const float4*)src, u1 = *(const float4*)(src + 4);
        const float w[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
        bf16x8 h, l;
#pragma unroll
        for (int e = 0; e < 8; ++e) split(row < M ? w[e] : 0.0f, h, l, e);
        frag[q][0][f & 63] = h;
        frag[q][1][f & 63] = l;
    }
    __syncthreads();
    while (item < a.nitems) {
        const int next = item + stride, m0 = (item % MG) * MT;
        int fl = lane;
        asm volatile("" : "+v"(fl));     // A stays in LDS: hoisted out of the loop it takes half the registers
        const float* src = a.in + column(min(next, a.nitems - 1), a.in_y, a.in_b);
        f32x16 acc[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[m][r] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KN; ++ks) {
            bf16x8 bh, bl;
#pragma unroll
            for (int e = 0; e < 8; ++e) split(v[ks][e], bh, bl, e);
            if (next < a.nitems) load(src, ks);
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const bf16x8 ah = frag[ks * MTOT + m0 + m][0][fl], al = frag[ks * MTOT + m0 + m][1][fl];
                acc[m] = mfma(ah, bh, acc[m]);
                acc[m] = mfma(ah, bl, acc[m]);
                acc[m] = mfma(al, bh, acc[m]);
            }
        }
        float* dst = a.out + column(item, a.out_y, a.out_b);
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int r0 = 32 * (m0 + m) + 8 * (r >> 2) + (r & 3);   // + 4 grp: whole groups of 16 rows are valid
                if (M % 32 == 0 || r0 < M)
                    (dst + (r0 >> 1) * a.out_hi + (r0 & 1) * a.out_lo)[uint32_t(2 * grp * a.out_hi + t)] = acc[m][r];
            }
        item = next;
    }
}

// ---------------------------------------------------------------------------
// Weight gradients: part[b][chunk] = [A | 1]^T-style sums over CHUNK nodes
// ---------------------------------------------------------------------------

// Operand fragments of a 16-node step (lane: row or column t, nodes 8 grp + e),
// read from memory as they lie.
struct NodeFrag {                     // float [node][32]: one tile, bf16 hi + lo
    static constexpr int TILES = 1;
    static constexpr bool LO = true;
    float v[8];
    __device__ __forceinline__ void load(const void* p, int, int k, int t, int grp) {
        const float* q = (const float*)p + int64_t(k) * C;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (q + e * C)[uint32_t(8 * grp * C + t)];
    }
    __device__ __forceinline__ void get(int, bf16x8& hi, bf16x8& lo) const {
#pragma unroll
        for (int e = 0; e < 8; ++e) split(v[e], hi, lo, e);
    }
};
struct HiddenFrag {                   // bf16 [N3 / 16][128][16]: two tiles, exact
    static constexpr int TILES = 2;
    static constexpr bool LO = false;
    bf16x8 v[2];
    __device__ __forceinline__ void load(const void* p, int row0, int k, int t, int grp) {
        const bf16* q = (const bf16*)p + int64_t(k) * HID + row0 * 16;
#pragma unroll
        for (int i = 0; i < 2; ++i) v[i] = *(const bf16x8*)&(q + 32 * i * 16)[uint32_t(t * 16 + 8 * grp)];
    }
    __device__ __forceinline__ void get(int i, bf16x8& hi, bf16x8& lo) const { hi = v[i]; lo = v[i]; }
};
struct OutFrag {                      // float [6][N3]: one tile of 6 columns, bf16 hi + lo
    static constexpr int TILES = 1;
    static constexpr bool LO = true;
    float4 v[2];
    __device__ __forceinline__ void load(const void* p, int, int k, int t, int grp) {
        const float* q = (const float*)p + k;
        const uint32_t off = uint32_t(min(t, NOUT - 1) * N3 + 8 * grp);
        v[0] = *(const float4*)&q[off];
        v[1] = *(const float4*)&(q + 4)[off];
    }
    __device__ __forceinline__ void get(int, bf16x8& hi, bf16x8& lo) const {
        const float w[8] = {v[0].x, v[0].y, v[0].z, v[0].w, v[1].x, v[1].y, v[1].z, v[1].w};
#pragma unroll
        for (int e = 0; e < 8; ++e) split(w[e], hi, lo, e);
    }
};

struct GradArgs {
    const void *a, *b;
    int64_t a_b, b_b;     // bytes per sample
    float* part;          // [B][NCHUNK][rows + 1][cols], the last row the sums of b
    int rows, cols;
};

// One wave per sample, chunk and pair of hidden-unit tiles walks its 4096 nodes
// in steps of 16, the order of the products that of k_gemm; the row of ones
// that gives the bias gradient is a constant A operand.  A wave's loads bound
// it, there being one or two waves per SIMD at 16 samples: DEPTH steps are in
// flight in registers.  16 samples: [W; b] 442 us with the operands staged in
// LDS (k_gemm), 200 so (5.4 TB/s); [P2; c2] 652 -> 195, [P1; c1] 514 -> 364.
template <typename FA, typename FB>
__global__ __launch_bounds__(64) void k_wgrad(GradArgs a) {
    constexpr int DEPTH = 8, TA = FA::TILES, TB = FB::TILES;
    static_assert(N3 % CHUNK == 0 && CHUNK % (16 * DEPTH) == 0, "whole chunks of whole steps");
    static_assert((HID + 1) * NOUT <= (C + 1) * HID, "the sums of every weight fit the buffer of [P1; c1]");
    const int t = threadIdx.x & 31, grp = threadIdx.x >> 5;
    const int tile0 = 2 * blockIdx.x, k0 = blockIdx.y * CHUNK;
    const char* A = (const char*)a.a + blockIdx.z * a.a_b;
    const char* B = (const char*)a.b + blockIdx.z * a.b_b;
    FA fa[DEPTH];
    FB fb[DEPTH];
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
        fa[d].load(A, 32 * tile0, k0 + 16 * d, t, grp);
        fb[d].load(B, 32 * tile0, k0 + 16 * d, t, grp);
    }
    f32x16 acc[TA][TB], ones[TB];
    bf16x8 one;
#pragma unroll
    for (int e = 0; e < 8; ++e) one[e] = (bf16)1.0f;
#pragma unroll
    for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            ones[j][r] = 0.0f;
#pragma unroll
            for (int i = 0; i < TA; ++i) acc[i][j][r] = 0.0f;
        }
    for (int k = 0; k < CHUNK; k += 16 * DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            bf16x8 ah[TA], al[TA], bh[TB], bl[TB];
#pragma unroll
            for (int i = 0; i < TA; ++i) fa[d].get(i, ah[i], al[i]);
#pragma unroll
            for (int j = 0; j < TB; ++j) fb[d].get(j, bh[j], bl[j]);
            const int kn = k + 16 * (d + DEPTH);
            if (kn < CHUNK) {
                fa[d].load(A, 32 * tile0, k0 + kn, t, grp);
                fb[d].load(B, 32 * tile0, k0 + kn, t, grp);
            }
#pragma unroll
            for (int j = 0; j < TB; ++j) {
#pragma unroll
                for (int i = 0; i < TA; ++i) {
                    acc[i][j] = mfma(ah[i], bh[j], acc[i][j]);
                    if constexpr (FB::LO) acc[i][j] = mfma(ah[i], bl[j], acc[i][j]);
                    if constexpr (FA::LO) acc[i][j] = mfma(al[i], bh[j], acc[i][j]);
                }
                ones[j] = mfma(one, bh[j], ones[j]);
                if constexpr (FB::LO) ones[j] = mfma(one, bl[j], ones[j]);
            }
        }
    }
    float* o = a.part + (int64_t(blockIdx.z) * NCHUNK + blockIdx.y) * (a.rows + 1) * a.cols;
    const int row0 = TA == 2 ? 32 * tile0 : 0, col0 = TB == 2 ? 32 * tile0 : 0;
#pragma unroll
    for (int j = 0; j < TB; ++j) {
        const int col = col0 + 32 * j + t;
        if (col >= a.cols) continue;
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                o[(row0 + 32 * i + 8 * (r >> 2) + 4 * grp + (r & 3)) * a.cols + col] = acc[i][j][r];
        if (grp == 0 && row0 == 0) o[a.rows * a.cols + col] = ones[j][0];
    }
}

// ---------------------------------------------------------------------------
// Fused per-line kernels
// ---------------------------------------------------------------------------

// The constant matrices of the line kernels are held in LDS in fragment order
// ([half][step][hi, lo][lane]), split once per block; a wave takes lpw
// consecutive lines (of one sample: lpw divides 4096) and requests the next
// line's inputs as soon as it has split the present ones.
//
// [64][24] inverse x matrix: rows x = 32 h + t, k = (s, kx) < 24, zeros beyond
__device__ __forceinline__ void stage_gx(const float* gx, bf16x8 (*fr)[2][2][64]) {
    const int t = threadIdx.x & 31, grp = (threadIdx.x >> 5) & 1, s = (threadIdx.x >> 6) & 1, h = threadIdx.x >> 7;
    const int k0 = 16 * s + 8 * grp;
    const float* src = gx + (32 * h + t) * 24 + min(k0, 16);
    const float4 u0 = *(const float4*)src, u1 = *(const float4*)(src + 4);
    const float w[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
    bf16x8 hi, lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) split(k0 < 24 ? w[e] : 0.0f, hi, lo, e);
    fr[h][s][0][threadIdx.x & 63] = hi;
    fr[h][s][1][threadIdx.x & 63] = lo;
}
// a line's (s, kx) x c block as an operand: k < 24, column t (the lanes of k >=
// 24 read the row of their k - 8, which the zeros of the matrix do not cover: it
// may be infinite)
__device__ __forceinline__ void load_line(const float* ln, int t, int grp, float v[2][8]) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) v[s][e] = (ln + (16 * s + e) * C)[uint32_t((s == 0 ? 8 * grp : 0) * C + t)];
}
__device__ __forceinline__ void split_line(const float v[2][8], int grp, bf16x8 hi[2], bf16x8 lo[2]) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) split(s == 1 && grp == 1 ? 0.0f : v[s][e], hi[s], lo[s], e);
}
// node x = 32 h + t, channels 16 s + 8 grp + e
__device__ __forceinline__ void load_act(const float* act, int t, int grp, float4 v[2][2][2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int q = 0; q < 2; ++q)
                v[h][s][q] = *(const float4*)&(act + 32 * h * C + 16 * s + 4 * q)[uint32_t(t * C + 8 * grp)];
}
__device__ __forceinline__ bf16x8 to_bf16(float4 u0, float4 u1) {
    bf16x8 f;
    f[0] = (bf16)u0.x; f[1] = (bf16)u0.y; f[2] = (bf16)u0.z; f[3] = (bf16)u0.w;
    f[4] = (bf16)u1.x; f[5] = (bf16)u1.y; f[6] = (bf16)u1.z; f[7] = (bf16)u1.w;
    return f;
}

// x-lines (64 nodes, two 32-node halves), one wave per line:
//   acc[x][j] = sum_k CM[x][k] LN[k][j]   (k < 24, split bf16)
//             + sum_c ACT[x][c] Wt[c][j]  (bf16)
// Forward (inverse x transform + pointwise branch of a layer):
//   CM = inverse x matrix, LN = the line's (s, kx) x c block, Wt = W,
//   z = acc + b; zout <- z; out <- GELU(z) or z.
// Backward (adjoint): CM = transpose of the forward x matrix, LN = gradient
//   block, ACT = dL/dz_l, Wt = W^T; out <- acc * GELU'(z_{l-1}) or acc.
struct LineArgs {
    const float* cm;      // [64][24]
    const float* ln;      // [lines][24][32]
    const float* act;     // [lines][64][32], or nullptr: no pointwise term
    const bf16* w;        // [32][32] row-major W[c][o]
    const float* bias;    // [32] (forward) or nullptr
    const float* zprev;   // backward: z_{l-1} for GELU', or nullptr
    float* zout;          // forward: pre-activation, or nullptr
    float* out;
    int lpw;              // lines per wave
    int act_gelu;         // forward: out = GELU(z)
};

// Memory bounds it (16 samples, z kept or read: 1.8 GB, 370 us at a copy's
// rate): 429 us (mean of a step's six) with one line per wave and the matrices split
// by each, 345 so.
template <bool BWD>
__global__ __launch_bounds__(256, 3) void k_lineout(LineArgs a) {
    __shared__ bf16x8 cm[2][2][2][64];
    const int lane = threadIdx.x & 63, t = lane & 31, grp = lane >> 5;
    const int64_t line0 = (int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6)) * a.lpw;
    const float* ln = a.ln + line0 * 24 * C;
    const float* act = a.act ? a.act + line0 * N * C : nullptr;
    const float* zprev = BWD && a.zprev ? a.zprev + line0 * N * C : nullptr;
    float* zout = a.zout ? a.zout + line0 * N * C : nullptr;
    float* out = a.out + line0 * N * C;
    float v[2][8];
    float4 u[2][2][2] = {};
    load_line(ln, t, grp, v);
    if (act) load_act(act, t, grp, u);
    bf16x8 wf[2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = 16 * s + 8 * grp + e;
            wf[s][e] = BWD ? a.w[t * C + k] : a.w[k * C + t];
        }
    const float bt = a.bias ? a.bias[t] : 0.0f;
    stage_gx(a.cm, cm);
    __syncthreads();
    for (int i = 0; i < a.lpw; ++i) {
        int fl = lane;
        asm volatile("" : "+v"(fl));     // the matrix stays in LDS
        bf16x8 lh[2], ll[2], af[2][2];
        split_line(v, grp, lh, ll);
        if (act)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int s = 0; s < 2; ++s) af[h][s] = to_bf16(u[h][s][0], u[h][s][1]);
        float zp[2][16];
        if (BWD && zprev)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    zp[h][r] = (zprev + (32 * h + 8 * (r >> 2) + (r & 3)) * C)[uint32_t(4 * grp * C + t)];
        if (i + 1 < a.lpw) {
            load_line(ln + 24 * C, t, grp, v);
            if (act) load_act(act + N * C, t, grp, u);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const bf16x8 ch = cm[h][s][0][fl], cl = cm[h][s][1][fl];
                acc = mfma(ch, lh[s], acc);
                acc = mfma(ch, ll[s], acc);
                acc = mfma(cl, lh[s], acc);
            }
            if (act)
#pragma unroll
                for (int s = 0; s < 2; ++s) acc = mfma(af[h][s], wf[s], acc);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = (32 * h + 8 * (r >> 2) + (r & 3)) * C;
                const uint32_t at = uint32_t(4 * grp * C + t);
                float x = acc[r];
                if (!BWD) {
                    if (a.bias) x += bt;
                    if (zout) (zout + row)[at] = x;
                    (out + row)[at] = a.act_gelu ? gelu(x) : x;
                } else {
                    if (zprev) x *= gelu_d(zp[h][r]);
                    (out + row)[at] = x;
                }
            }
        }
        ln += 24 * C;
        out += N * C;
        if (act) act += N * C;
        if (zout) zout += N * C;
        if (BWD && zprev) zprev += N * C;
    }
}

// Lines per wave: four waves per SIMD where the batch has them, then more lines
// for each, to 16 (beyond that nothing is gained).
inline int lines_per_wave(int lines) {
    int lpw = 1;
    while (lpw < 16 && lines / (2 * lpw) >= 4096) lpw *= 2;
    return lpw;
}

// Projection 32 -> 128 -> 6.  The hidden layer is computed transposed
// (h^T = P1^T v^T): its MFMA accumulator holds, in lane (node t, group g),
// register r, the hidden unit
//   kappa(r) = 8 (r >> 2) + 4 g + (r & 3)  within a 32-unit block,
// which is exactly the k slot an MFMA operand in that lane needs when the
// K index is relabelled by kappa.  So the hidden layer feeds the next
// contraction straight from registers, with the constant operand (P2 or P1)
// gathered in the same kappa order.
//
// A wave takes 64 nodes as two tiles, tile i of nodes 2 t + i: the constant
// operands are loaded for both at once, and the hidden values of two
// neighbouring nodes leave as one 4-byte store.  The backward pass keeps them
// for the weight gradients in blocks of 16 nodes, [B][N3 / 16][128][16], the
// order in which those read them (rows of all nodes put every row of a fragment
// on a page of its own).
constexpr int HB = 16;                    // nodes per block of the stored hidden layer
static_assert(CHUNK % HB == 0, "a chunk of nodes is whole blocks");
struct ProjArgs {
    const float* v;       // [B][N3][32]
    const bf16* p1;       // [32][128]
    const bf16* p1f;      // P1^T in fragment order [4][2][2][32][8]: P1[16 s + 8 g + e][32 mt + t]
    const float* c1;      // [128]
    const bf16* p2;       // [B][128][6]: the head's effective projection per sample
    const bf16* p2k;      // the same in kappa fragment order
    const float* c2;      // [B][6]
    float* out;           // forward: [B][6][N3]
    const float* gout;    // backward: dL/dout [B][6][N3]
    float* gv;            // backward: [B][N3][32]
    bf16* hT;             // backward: GELU(hidden)
    bf16* ghT;            // backward: dL/d(pre-activation)
};

__device__ __forceinline__ int kappa(int s, int grp, int e) { return 16 * s + 8 * (e >> 2) + 4 * grp + (e & 3); }

// 8 floats at kappa(s, grp, 0 .. 7): two runs of 4
__device__ __forceinline__ void ld_kappa(const float* p, int s, int grp, float v[8]) {
    const float4 a = *(const float4*)(p + kappa(s, grp, 0)), b = *(const float4*)(p + kappa(s, grp, 4));
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// 16 samples: forward 558 -> 360 us, backward 1835 -> 890 us with one tile of
// neighbouring nodes per wave and 2-byte stores before; the GELUs bound the
// forward pass, the stores of the hidden layer (2.1 GB) the backward one.
template <bool BWD>
__global__ __launch_bounds__(256, BWD ? 3 : 4) void k_proj(ProjArgs a) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
    const int lane = threadIdx.x & 63, t = lane & 31, grp = lane >> 5;
    const int item = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int b = item / (N3 / 64), node0 = (item % (N3 / 64)) * 64;

    // B operand v^T: lane (node 2 t + i), k = c
    bf16x8 vf[2][2];
    const float* vp = a.v + (int64_t(b) * N3 + node0 + 2 * t) * C + 8 * grp;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int s = 0; s < 2; ++s)
            vf[i][s] = to_bf16(*(const float4*)(vp + i * C + 16 * s), *(const float4*)(vp + i * C + 16 * s + 4));

    const bf16x8* p1f = (const bf16x8*)a.p1f + grp * 32 + t;          // + (mt * 2 + s) * 64
    if constexpr (!BWD) {
        const bf16x8* p2k = (const bf16x8*)(a.p2k + int64_t(b) * KSLOTS) + grp * 32 + t;
        f32x16 oacc[2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[i][r] = 0.0f;
#pragma unroll 1
        for (int mt = 0; mt < 4; ++mt) {
            f32x16 acc[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][r] = 0.0f;
                acc[i] = mfma(p1f[(mt * 2) * 64], vf[i][0], acc[i]);
                acc[i] = mfma(p1f[(mt * 2 + 1) * 64], vf[i][1], acc[i]);
            }
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                float c1[8];
                ld_kappa(a.c1 + 32 * mt, s, grp, c1);
                const bf16x8 pf = p2k[(mt * 2 + s) * 64];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    bf16x8 hf;
#pragma unroll
                    for (int e = 0; e < 8; ++e) hf[e] = (bf16)gelu(acc[i][8 * s + e] + c1[e]);
                    oacc[i] = mfma(pf, hf, oacc[i]);
                }
            }
        }
        // rows are output components: group 0 holds 0..3 (r = 0..3), group 1 holds 4, 5 (r = 0, 1)
        float* op = a.out + int64_t(b) * OUT_SZ + node0 + 2 * t;
        const float* c2 = a.c2 + b * NOUT;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = 4 * grp + r;
            if (o < NOUT) {
                op[int64_t(o) * N3] = oacc[0][r] + c2[o];
                op[int64_t(o) * N3 + 1] = oacc[1][r] + c2[o];
            }
        }
    } else {
        const bf16* p2 = a.p2 + int64_t(b) * HID * NOUT;
        // dL/dout^T as the B operand of dL/dh^T = P2 . dL/dout^T (K = 6 padded to 16)
        bf16x8 gf[2];
        const float* gp = a.gout + int64_t(b) * OUT_SZ + node0 + 2 * t;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float2 g = *(const float2*)(gp + int64_t(min(e, NOUT - 1)) * N3);
            const bool in = e < NOUT && grp == 0;
            gf[0][e] = in ? (bf16)g.x : (bf16)0.0f;
            gf[1][e] = in ? (bf16)g.y : (bf16)0.0f;
        }
        f32x16 gvacc[2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) gvacc[i][r] = 0.0f;
        const int64_t ho = ((int64_t(b) * (N3 / HB) + node0 / HB + t / 8) * HID) * HB + 2 * (t & 7);
        bf16 *hp = a.hT + ho, *ghp = a.ghT + ho;
#pragma unroll 1
        for (int mt = 0; mt < 4; ++mt) {
            bf16x8 p2f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bf16 q = p2[(32 * mt + t) * NOUT + min(e, NOUT - 1)];
                p2f[e] = e < NOUT && grp == 0 ? q : (bf16)0.0f;
            }
            f32x16 acc[2], gacc[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int r = 0; r < 16; ++r) { acc[i][r] = 0.0f; gacc[i][r] = 0.0f; }
                acc[i] = mfma(p1f[(mt * 2) * 64], vf[i][0], acc[i]);
                acc[i] = mfma(p1f[(mt * 2 + 1) * 64], vf[i][1], acc[i]);
                gacc[i] = mfma(p2f, gf[i], gacc[i]);
            }
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                float c1[8];
                ld_kappa(a.c1 + 32 * mt, s, grp, c1);
                bf16x8 af[2], bfr;
                const bf16x4 b0 = *(const bf16x4*)&a.p1[t * HID + 32 * mt + kappa(s, grp, 0)];
                const bf16x4 b1 = *(const bf16x4*)&a.p1[t * HID + 32 * mt + kappa(s, grp, 4)];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int r = 8 * s + e, hd = 32 * mt + kappa(s, grp, e);
                    bf16x2 h2, g2;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const float pre = acc[i][r] + c1[e];
                        h2[i] = (bf16)gelu(pre);
                        g2[i] = (bf16)(gacc[i][r] * gelu_d(pre));
                        af[i][e] = g2[i];
                    }
                    *(bf16x2*)&hp[hd * HB] = h2;
                    *(bf16x2*)&ghp[hd * HB] = g2;
                    bfr[e] = e < 4 ? b0[e & 3] : b1[e & 3];
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) gvacc[i] = mfma(af[i], bfr, gvacc[i]);
            }
        }
        float* gvp = a.gv + (int64_t(b) * N3 + node0) * C + t;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) gvp[(2 * (8 * (r >> 2) + 4 * grp + (r & 3)) + i) * C] = gvacc[i][r];
    }
}

// ---------------------------------------------------------------------------
// Elementwise and reduction kernels
// ---------------------------------------------------------------------------

__device__ __forceinline__ float coord(int i) { return float(i - N / 2) / float(N / 2); }

// v0[b][node][c] = b0[c] + sum_i p[b][i] W0[i][c] + x W0[8][c] + y W0[9][c] + z W0[10][c],
// summed in this order, each coordinate's product fused into the sum (k_lift_x
// rounds some of them first, see there)
__device__ __forceinline__ float lift_base(const float* pb, const float* w0, const float* b0, int c) {
    float s = b0[c];
    for (int i = 0; i < NPAR; ++i) s += pb[i] * w0[i * C + c];
    return s;
}
__device__ __forceinline__ float lift_term(float s, float w, int i) { return fmaf(coord(i), w, s); }
// the same with the product rounded on its own
__device__ __forceinline__ float lift_term_r(float s, float w, int i) {
#pragma clang fp contract(off)
    const float q = coord(i) * w;
    return s + q;
}
__device__ __forceinline__ float lift_at(float base, const float* w0, int c, int x, int y, int z) {
    return lift_term(lift_term(lift_term(base, w0[8 * C + c], x), w0[9 * C + c], y), w0[10 * C + c], z);
}

// One block per LIFT_LINES lines of one z: a thread keeps four channels and walks
// the lines two nodes each in 16-byte stores.  16 samples: 330 us with one element per
// thread, each summing its base anew, 88 so (537 MB).
constexpr int LIFT_LINES = 8;             // lines per block (64 divides into them)
__global__ __launch_bounds__(256) void k_lift(const float* p, const float* w0, const float* b0, float* v) {
    const int line0 = blockIdx.x * LIFT_LINES, b = line0 / (N * N), z = line0 / N % N;
    const int c = 4 * (threadIdx.x & 7), x0 = threadIdx.x >> 3;
    float base[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) base[q] = lift_base(p + b * NPAR, w0, b0, c + q);
    for (int i = 0; i < LIFT_LINES; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int x = x0 + 32 * h, y = (line0 + i) % N;
            float4 o;
            o.x = lift_at(base[0], w0, c, x, y, z);
            o.y = lift_at(base[1], w0, c + 1, x, y, z);
            o.z = lift_at(base[2], w0, c + 2, x, y, z);
            o.w = lift_at(base[3], w0, c + 3, x, y, z);
            *(float4*)&v[(int64_t(line0 + i) * N + x) * C + c] = o;
        }
}

// ---------------------------------------------------------------------------
// Fused inference kernels: no activation of the forward pass is kept, and
// the first x contraction of every layer is taken from the registers of the
// kernel that produced the layer's input.
// ---------------------------------------------------------------------------

// Forward x matrix [24][64] as an A operand in LDS, rows i = t < 24, steps of 16
// x: in order (x = 16 ks + 8 g + e), or in kappa order (x = 32 (ks >> 1) +
// kappa(ks & 1, g, e)) to meet an accumulator's rows.
template <bool KAPPA> __device__ __forceinline__ void stage_fx(const float* fx, bf16x8 (*fr)[2][64]) {
    const int t = threadIdx.x & 31, grp = (threadIdx.x >> 5) & 1, ks = threadIdx.x >> 6;
    const float* src = fx + min(t, 23) * N + (KAPPA ? 32 * (ks >> 1) + kappa(ks & 1, grp, 0) : 16 * ks + 8 * grp);
    const float4 u0 = *(const float4*)src, u1 = *(const float4*)(src + (KAPPA ? 8 : 4));
    const float w[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
    bf16x8 hi, lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) split(t < 24 ? w[e] : 0.0f, hi, lo, e);
    fr[ks][0][threadIdx.x & 63] = hi;
    fr[ks][1][threadIdx.x & 63] = lo;
}

struct InfArgs {
    const float* gx;      // inverse x matrix [64][24]
    const float* fx;      // forward x matrix [24][64]
    const float* ln;      // spectral lines [lines][24][32] (U1); overwritten by the next layer's X1
    const float* act;     // v_l [lines][64][32], or nullptr: v_0 recomputed from the lift
    const float* p;       // [B][8] parameters (lift)
    const float* w0;
    const float* b0;
    const bf16* w;        // W_l [32][32]
    const float* bias;    // b_l
    float* vout;          // v_{l+1} (not the last layer)
    float* x1out;         // X1 of layer l+1, written over the line's U1
    // projection (last layer), operands in kappa fragment order
    const bf16* p1k;      // [4][2][2][32][8]
    const float* c1;
    const bf16* p2k;      // [B][4][2][2][32][8]
    const float* c2e;     // [B][6]
    float* out;           // [B][6][N3]
    int lpw;              // lines per wave
};

// Lift and the first x contraction, one wave per x-line:
//   X1[(s,kx)][c] = sum_x Fx[(s,kx)][x] v0[x][c]    (split bf16)
// Batch 64: 305 us with the matrix split by every wave, 149 so (805 MB written,
// 165 us at a copy's rate).  The y and z terms of the lift are fused into the
// sum for x < 16 and rounded first beyond.  Either is as accurate, and no rule of
// the method chooses between them; this is the mixture that the windows of
// surrogates trained so far were computed and their errors quoted with, and
// another one moves outputs by up to 1e-4 (a float32 rounding here can flip a
// bf16 one in the mixing).
__global__ __launch_bounds__(256) void k_lift_x(InfArgs a) {
    __shared__ bf16x8 fx[4][2][64];
    const int lane = threadIdx.x & 63, t = lane & 31, grp = lane >> 5;
    const int line0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * a.lpw;
    const float base = lift_base(a.p + line0 / (N * N) * NPAR, a.w0, a.b0, t);
    // the lift's sum up to its x term, as lift_at forms it
    float bx[4][8];
    const float wx = a.w0[8 * C + t], wy = a.w0[9 * C + t], wz = a.w0[10 * C + t];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) bx[ks][e] = lift_term(base, wx, 16 * ks + 8 * grp + e);
    stage_fx<false>(a.fx, fx);
    __syncthreads();
    for (int line = line0; line < line0 + a.lpw; ++line) {
        const int zy = line % (N * N);
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            bf16x8 bh, bl;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                split(ks == 0 ? lift_term(lift_term(bx[ks][e], wy, zy % N), wz, zy / N)
                              : lift_term_r(lift_term_r(bx[ks][e], wy, zy % N), wz, zy / N), bh, bl, e);
            acc = mfma(fx[ks][0][lane], bh, acc);
            acc = mfma(fx[ks][0][lane], bl, acc);
            acc = mfma(fx[ks][1][lane], bh, acc);
        }
        float* o = a.x1out + int64_t(line) * 24 * C;
#pragma unroll
        for (int r = 0; r < 12; ++r) (o + (8 * (r >> 2) + (r & 3)) * C)[uint32_t(4 * grp * C + t)] = acc[r];
    }
}

// Inverse x transform + pointwise branch + GELU of a layer that is not the
// last, then the next layer's x contraction from the registers:
//   v[x][o]  = GELU(sum_k Gx[x][k] U1[k][o] + sum_c v_l[x][c] W[c][o] + b[o])
//   X1[i][o] = sum_x Fx[i][x] v[x][o]
// The accumulator of v holds row x = 32 h + kappa(s, g, e) in register 8 s + e
// of lane (o, g), so it is the B operand of the contraction over x with the
// constant Fx gathered in that order.  LIFT: v_l is v_0, recomputed from the
// parameters, never stored.  Memory bounds it (batch 64: 3.8 GB and, with v_l
// read, 5.9): 1.32 ms and 1.50 with one line per wave and the matrices
// split by each, 0.77 and 1.21 so.
template <bool LIFT>
__global__ __launch_bounds__(256, 3) void k_line_fwd(InfArgs a) {
    __shared__ bf16x8 gx[2][2][2][64], fx[4][2][64];
    __shared__ __attribute__((aligned(16))) float lift[4][C];     // LIFT: base and the x, y, z weights
    const int lane = threadIdx.x & 63, t = lane & 31, grp = lane >> 5;
    const int line0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * a.lpw;
    const float* ln = a.ln + int64_t(line0) * 24 * C;
    const float* act = LIFT ? nullptr : a.act + int64_t(line0) * N * C;
    float v[2][8];
    float4 u[2][2][2];
    load_line(ln, t, grp, v);
    if constexpr (!LIFT) load_act(act, t, grp, u);
    if constexpr (LIFT)                   // a block's lines are of one sample
        if (threadIdx.x < C) {
            const int c = threadIdx.x;
            lift[0][c] = lift_base(a.p + line0 / (N * N) * NPAR, a.w0, a.b0, c);
#pragma unroll
            for (int d = 0; d < 3; ++d) lift[1 + d][c] = a.w0[(8 + d) * C + c];
        }
    bf16x8 wf[2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) wf[s][e] = a.w[(16 * s + 8 * grp + e) * C + t];
    const float bt = a.bias[t];
    stage_gx(a.gx, gx);
    stage_fx<true>(a.fx, fx);
    __syncthreads();
    for (int i = 0; i < a.lpw; ++i) {
        const int line = line0 + i, zy = line % (N * N);
        int fl = lane;
        asm volatile("" : "+v"(fl));     // the matrices stay in LDS
        bf16x8 lh[2], ll[2], af[2][2];
        split_line(v, grp, lh, ll);
        if constexpr (LIFT) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int c = 16 * s + 8 * (fl >> 5);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float q = lift_term(lift[0][c + e], lift[1][c + e], 32 * h + t);
                        af[h][s][e] = (bf16)lift_term(lift_term(q, lift[2][c + e], zy % N), lift[3][c + e], zy / N);
                    }
            }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int s = 0; s < 2; ++s) af[h][s] = to_bf16(u[h][s][0], u[h][s][1]);
        }
        if (i + 1 < a.lpw) {
            load_line(a.ln + int64_t(line + 1) * 24 * C, t, grp, v);
            if constexpr (!LIFT) load_act(a.act + int64_t(line + 1) * N * C, t, grp, u);
        }
        float* vout = a.vout + int64_t(line) * N * C;
        f32x16 xacc;
#pragma unroll
        for (int r = 0; r < 16; ++r) xacc[r] = 0.0f;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const bf16x8 gh = gx[h][s][0][fl], gl = gx[h][s][1][fl];
                acc = mfma(gh, lh[s], acc);
                acc = mfma(gh, ll[s], acc);
                acc = mfma(gl, lh[s], acc);
            }
#pragma unroll
            for (int s = 0; s < 2; ++s) acc = mfma(af[h][s], wf[s], acc);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                bf16x8 bh, bl;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int r = 8 * s + e;
                    const float x = gelu(acc[r] + bt);
                    (vout + (32 * h + 8 * (r >> 2) + (r & 3)) * C)[uint32_t(4 * grp * C + t)] = x;
                    split(x, bh, bl, e);
                }
                const bf16x8 ah = fx[2 * h + s][0][fl], al = fx[2 * h + s][1][fl];
                xacc = mfma(ah, bh, xacc);
                xacc = mfma(ah, bl, xacc);
                xacc = mfma(al, bh, xacc);
            }
        }
        float* o = a.x1out + int64_t(line) * 24 * C;
#pragma unroll
        for (int r = 0; r < 12; ++r) (o + (8 * (r >> 2) + (r & 3)) * C)[uint32_t(4 * grp * C + t)] = xacc[r];
    }
}

// Last layer fused with the projection.  The layer is computed transposed,
// v^T[o][x] = sum_k U1^T[o][k] Gx^T[k][x] + sum_c W^T[o][c] v_l^T[c][x] + b[o],
// so lane (x, g) holds channel o = kappa(s, g, e) in register 8 s + e: the B
// operand of h^T = P1^T v^T over c, with P1 gathered in that order.  The
// projection then runs as in k_proj.  A wave takes one half (32 nodes) of its
// lines: twice the independent waves.  The constant operands are in LDS; the
// 64 GELUs per lane and half line bound it (batch 64: 2.1e9 of about 22
// instructions, 1.2 ms): 1.82 ms with the operands loaded by every wave, 1.65 so.
__global__ __launch_bounds__(256, 4) void k_line_proj(InfArgs a) {
    __shared__ bf16x8 gx[2][2][2][64], p1s[8][64], p2s[8][64];
    __shared__ __attribute__((aligned(16))) float c1s[HID], bs[C];
    const int lane = threadIdx.x & 63, t = lane & 31, grp = lane >> 5, h = (threadIdx.x >> 6) & 1;
    const int line0 = (blockIdx.x * 2 + (threadIdx.x >> 7)) * a.lpw, b = line0 / (N * N);
    float v[2][8];
    float4 u[2][2];
    auto fetch = [&](int line) {
        load_line(a.ln + int64_t(line) * 24 * C, t, grp, v);
        const float* act = a.act + (int64_t(line) * N + 32 * h) * C;
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int q = 0; q < 2; ++q)
                u[s][q] = *(const float4*)&(act + 16 * s + 4 * q)[uint32_t(t * C + 8 * grp)];
    };
    fetch(line0);
    bf16x8 wf[2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) wf[s][e] = a.w[(16 * s + 8 * grp + e) * C + t];
    stage_gx(a.gx, gx);
    const bf16x8* p2k = (const bf16x8*)(a.p2k + int64_t(b) * KSLOTS);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        (&p1s[0][0])[threadIdx.x + 256 * q] = ((const bf16x8*)a.p1k)[threadIdx.x + 256 * q];
        (&p2s[0][0])[threadIdx.x + 256 * q] = p2k[threadIdx.x + 256 * q];
    }
    if (threadIdx.x < HID) c1s[threadIdx.x] = a.c1[threadIdx.x];
    if (threadIdx.x < C) bs[threadIdx.x] = a.bias[threadIdx.x];
    __syncthreads();
    const float* c2 = a.c2e + b * NOUT;
    for (int i = 0; i < a.lpw; ++i) {
        const int line = line0 + i;
        int fl = lane;
        asm volatile("" : "+v"(fl));     // the operands stay in LDS
        bf16x8 lh[2], ll[2], af[2];
        split_line(v, grp, lh, ll);
#pragma unroll
        for (int s = 0; s < 2; ++s) af[s] = to_bf16(u[s][0], u[s][1]);
        if (i + 1 < a.lpw) fetch(line + 1);
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const bf16x8 gh = gx[h][s][0][fl], gl = gx[h][s][1][fl];
            acc = mfma(lh[s], gh, acc);
            acc = mfma(ll[s], gh, acc);
            acc = mfma(lh[s], gl, acc);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) acc = mfma(wf[s], af[s], acc);
        bf16x8 vf[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float bias[8];
            ld_kappa(bs, s, fl >> 5, bias);
#pragma unroll
            for (int e = 0; e < 8; ++e) vf[s][e] = (bf16)(acc[8 * s + e] + bias[e]);
        }
        f32x16 oacc;
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[r] = 0.0f;
#pragma unroll 1
        for (int mt = 0; mt < 4; ++mt) {
            f32x16 hacc;
#pragma unroll
            for (int r = 0; r < 16; ++r) hacc[r] = 0.0f;
#pragma unroll
            for (int s = 0; s < 2; ++s) hacc = mfma(p1s[mt * 2 + s][fl], vf[s], hacc);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                float c1[8];
                ld_kappa(c1s + 32 * mt, s, grp, c1);
                bf16x8 hf;
#pragma unroll
                for (int e = 0; e < 8; ++e) hf[e] = (bf16)gelu(hacc[8 * s + e] + c1[e]);
                oacc = mfma(p2s[mt * 2 + s][fl], hf, oacc);
            }
        }
        float* op = a.out + int64_t(b) * OUT_SZ + int64_t(line % (N * N)) * N + 32 * h + t;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = 4 * grp + r;
            if (o < NOUT) op[int64_t(o) * N3] = oacc[r] + c2[o];
        }
    }
}

// per (sample, z plane): sum_node g, and sum_node coord_d g, for every channel;
// thread (ng, c) takes the nodes ng (mod 8) in increasing order, sixteen loads
// in flight (16 samples: 253 us with one, 118 so; 537 MB)
__global__ __launch_bounds__(256) void k_lift_grad_part(const float* gv, float* part) {
    const int z = blockIdx.x, b = blockIdx.y;
    const int c = threadIdx.x & 31, ng = threadIdx.x >> 5;
    const float* g = gv + (int64_t(b) * N3 + int64_t(z) * N * N) * C;
    float s = 0, sx = 0, sy = 0;
    for (int n0 = ng; n0 < N * N; n0 += 8 * 16) {
        float v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = g[(n0 + 8 * k) * C + c];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int nd = n0 + 8 * k;
            s += v[k];
            sx += coord(nd % N) * v[k];
            sy += coord(nd / N) * v[k];
        }
    }
    __shared__ float red[3][8][32];
    red[0][ng][c] = s; red[1][ng][c] = sx; red[2][ng][c] = sy;
    __syncthreads();
    if (ng == 0) {
        float a0 = 0, a1 = 0, a2 = 0;
        for (int k = 0; k < 8; ++k) { a0 += red[0][k][c]; a1 += red[1][k][c]; a2 += red[2][k][c]; }
        float* o = part + (int64_t(b) * N + z) * 4 * C;
        o[c] = a0; o[C + c] = a1; o[2 * C + c] = a2; o[3 * C + c] = coord(z) * a0;
    }
}

// dL/dW0, dL/db0 from the per-plane sums (one thread per channel)
// One block of LIFT_THREADS: thread (bq, c) takes the samples b = bq (mod
// 32) in increasing b; the 32 lane sums of each of the 12 outputs are then
// added in order bq = 0..31.
constexpr int LIFT_THREADS = 1024;
__global__ __launch_bounds__(LIFT_THREADS) void k_lift_grad_final(const float* part, const float* p, int B,
                                                                  float* grad) {
    constexpr int NQ = LIFT_THREADS / C, NV = 12;
    const int c = threadIdx.x % C, bq = threadIdx.x / C;
    float gw[NV] = {0};                       // 8 parameter weights, 3 coordinate weights, bias
    for (int b = bq; b < B; b += NQ) {
        float s = 0, sx = 0, sy = 0, sz = 0;
#pragma unroll 8
        for (int z = 0; z < N; ++z) {
            const float* o = part + (int64_t(b) * N + z) * 4 * C;
            s += o[c]; sx += o[C + c]; sy += o[2 * C + c]; sz += o[3 * C + c];
        }
        for (int i = 0; i < NPAR; ++i) gw[i] += p[b * NPAR + i] * s;
        gw[8] += sx; gw[9] += sy; gw[10] += sz;
        gw[11] += s;
    }
    __shared__ float red[NQ][NV][C];
    for (int i = 0; i < NV; ++i) red[bq][i][c] = gw[i];
    __syncthreads();
    for (int idx = threadIdx.x; idx < NV * C; idx += LIFT_THREADS) {
        const int i = idx / C, cc = idx % C;
        float t = 0;
        for (int q = 0; q < NQ; ++q) t += red[q][i][cc];
        if (i < 11) grad[OFF_W0 + i * C + cc] = t;
        else grad[OFF_B0 + cc] = t;
    }
}

// per (chunk, sample): sum (out - y)^2 and sum y^2 in float64
__global__ __launch_bounds__(256) void k_loss_part(const float* out, const float* y, double* part) {
    const int ch = blockIdx.x, b = blockIdx.y;
    const int64_t len = OUT_SZ / gridDim.x;
    const float* o = out + int64_t(b) * OUT_SZ + ch * len;
    const float* t = y + int64_t(b) * OUT_SZ + ch * len;
    double sd = 0, sy = 0;
    for (int64_t i = threadIdx.x; i < len; i += 256) {
        const double d = double(o[i]) - double(t[i]);
        sd += d * d;
        sy += double(t[i]) * double(t[i]);
    }
    __shared__ double rd[256], ry[256];
    rd[threadIdx.x] = sd; ry[threadIdx.x] = sy;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) { rd[threadIdx.x] += rd[threadIdx.x + w]; ry[threadIdx.x] += ry[threadIdx.x + w]; }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[(int64_t(b) * gridDim.x + ch) * 2] = rd[0];
        part[(int64_t(b) * gridDim.x + ch) * 2 + 1] = ry[0];
    }
}

// res[0] = loss; res[1 + b] = dL/dout scale 1 / (B ||d_b|| ||y_b||).  One
// thread per sample (strided over the block); the loss sums the samples in
// order b = 0..B-1.  Launched with one block of LOSS_THREADS threads.
constexpr int LOSS_THREADS = 256;
__global__ __launch_bounds__(LOSS_THREADS) void k_loss_final(const double* part, int nch, int B, double* res,
                                                             double* ratio) {
    for (int b = threadIdx.x; b < B; b += LOSS_THREADS) {
        double sd = 0, sy = 0;
        for (int k = 0; k < nch; ++k) { sd += part[(b * nch + k) * 2]; sy += part[(b * nch + k) * 2 + 1]; }
        const double nd = sqrt(sd), ny = sqrt(sy);
        ratio[b] = nd / ny;
        res[1 + b] = nd > 0 ? 1.0 / (double(B) * nd * ny) : 0.0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double L = 0;
        for (int b = 0; b < B; ++b) L += ratio[b];
        res[0] = L / B;
    }
}

__global__ void k_gout(const float* out, const float* y, const double* res, float* g, int64_t total) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const int b = int(i / OUT_SZ);
    g[i] = float(double(out[i] - y[i]) * res[1 + b]);
}

// dst[y][e] = sum_p part[y][p][e] (y = blockIdx.y), in a fixed order: a
// block takes 64 consecutive e; lane q = threadIdx.x / 64 of column e sums
// the partials p = q (mod 4) in increasing p, eight loads in flight, and
// the four lane sums are added in order q = 0..3.
__global__ __launch_bounds__(256) void k_reduce(const float* part, int nparts, int len, float* dst) {
    const int el = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + el;
    const float* src = part + int64_t(blockIdx.y) * nparts * len;
    float s = 0;
    if (e < len) {
        int p = q;
        for (; p + 28 < nparts; p += 32) {
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = src[int64_t(p + 4 * k) * len + e];
#pragma unroll
            for (int k = 0; k < 8; ++k) s += v[k];
        }
        for (; p < nparts; p += 4) s += src[int64_t(p) * len + e];
    }
    __shared__ float red[4][64];
    red[q][el] = s;
    __syncthreads();
    if (q == 0 && e < len)
        dst[int64_t(blockIdx.y) * len + e] = ((red[0][el] + red[1][el]) + red[2][el]) + red[3][el];
}

// dL/dR from the real 64x64 block gradient G* of Y* = X* R*:
//   re = G*[c][o] + G*[32+c][32+o],  im = G*[c][32+o] - G*[32+c][o]
__global__ void k_fold_r(const float* gs, float* gr) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= int64_t(NMODES) * C * C) return;
    const int o = i & 31, c = (i >> 5) & 31;
    const float* G = gs + (i >> 10) * 4096;
    gr[2 * i] = G[c * 64 + o] + G[(32 + c) * 64 + 32 + o];
    gr[2 * i + 1] = G[c * 64 + 32 + o] - G[(32 + c) * 64 + o];
}

// bf16 working copy of R as the real block matrix R*[(s,c)][(s',o)]:
//   s = s': re,  s = 0, s' = 1: im,  s = 1, s' = 0: -im
// as it is for a surrogate that trains, whose adjoint mixing contracts over
// (s',o), and transposed, R*^T[(s',o)][(s,c)], for one that only infers (the
// forward mixing contracts over (s,c), and reads it 16 bytes at a time).
// One block per mode: R is read once into LDS, and every thread writes 16
// bytes of two rows of the block (one element per thread took 67 us, 1.3 TB/s).
__global__ __launch_bounds__(256) void k_expand_r(const float* r, bf16* rb, int transposed) {
    const int64_t q = blockIdx.x;
    __shared__ float2 e[C * (C + 1)];
    const float4* src = (const float4*)(r + q * C * C * 2);
    for (int i = threadIdx.x; i < C * C / 2; i += 256) {
        const float4 v = src[i];
        const int c = (2 * i) / C, o = (2 * i) % C;
        e[c * (C + 1) + o] = make_float2(v.x, v.y);
        e[c * (C + 1) + o + 1] = make_float2(v.z, v.w);
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int i = threadIdx.x + 256 * h, row = i >> 3, col0 = 8 * (i & 7);
        bf16x8 v;
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            const int k = transposed ? col0 + x : row, j = transposed ? row : col0 + x;
            const float2 f = e[(k & 31) * (C + 1) + (j & 31)];
            v[x] = (bf16)((k >> 5) == (j >> 5) ? f.x : (k >> 5) == 0 ? f.y : -f.y);
        }
        *(bf16x8*)&rb[q * 4096 + 8 * i] = v;
    }
}

// Effective projection of sample b for a head of nb basis fields:
//   P2eff[b][hd][c] = sum_k w[b][k] P2[hd][6k + c],  c2eff[b][c] = sum_k w[b][k] c2[6k + c]
// (w = 1 when nb = 1 and no weights are given).
// and in the projection's kappa order, padded to 32 outputs:
//   p2k[b][mt][s][g][t][e] = P2eff[b][32 mt + kappa(s, g, e)][t]  (0 for t >= 6)
__global__ void k_head_eff(const float* p2, const float* c2, const float* w, int nb, int B, bf16* p2e, float* c2e,
                           bf16* p2k) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int per = (HID + 1) * NOUT;
    if (i >= B * per) return;
    const int b = i / per, r = (i % per) / NOUT, c = i % NOUT;
    const float* src = r < HID ? p2 + int64_t(r) * NOUT * nb : c2;
    float s = 0.0f;
    for (int k = 0; k < nb; ++k) s += (w ? w[b * nb + k] : 1.0f) * src[NOUT * k + c];
    if (r < HID) {
        p2e[(int64_t(b) * HID + r) * NOUT + c] = (bf16)s;
        // r = 32 mt + kappa(s', g, e): invert kappa (16 s' + 8 (e >> 2) + 4 g + (e & 3))
        const int mt = r >> 5, q = r & 31, sp = q >> 4, eh = (q >> 3) & 1, g = (q >> 2) & 1, el = q & 3;
        const int e = 4 * eh + el;
        bf16* d = p2k + int64_t(b) * KSLOTS;
        d[((((mt * 2 + sp) * 2 + g) * 32 + c) * 8) + e] = (bf16)s;
    } else {
        c2e[b * NOUT + c] = s;
    }
}

// dL/dP2 and dL/dc2 from the per-sample gradients of the effective head
// (geff [B][129][6], row 128 the bias):  G[r][6k + c] = sum_b w[b][k] geff[b][r][c]
__global__ void k_head_grad(const float* geff, const float* w, int nb, int B, float* g) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int cols = NOUT * nb;
    if (i >= (HID + 1) * cols) return;
    const int r = i / cols, col = i % cols, k = col / NOUT, c = col % NOUT;
    float s = 0.0f;
    for (int b = 0; b < B; ++b) s += (w ? w[b * nb + k] : 1.0f) * geff[(int64_t(b) * (HID + 1) + r) * NOUT + c];
    g[int64_t(r) * cols + col] = s;
}

// P1^T in fragment order: [mt][s][g][t][e] = P1[k][32 mt + t] with k = kappa(s, g,
// e) for the fused last layer, 16 s + 8 g + e for k_proj
__global__ void k_p1_frag(const float* p1, bf16* kap, bf16* plain) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= C * HID) return;
    const int e = i & 7, t = (i >> 3) & 31, g = (i >> 8) & 1, s = (i >> 9) & 1, mt = i >> 10;
    kap[i] = (bf16)p1[kappa(s, g, e) * HID + 32 * mt + t];
    plain[i] = (bf16)p1[(16 * s + 8 * g + e) * HID + 32 * mt + t];
}

__global__ void k_to_bf16(const float* src, bf16* dst, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = (bf16)src[i];
}

// Adam with bias correction (Kingma and Ba, Algorithm 1).  The factors
// 1 - b1 and 1 - b2 come in rounded from float64: formed in float32 from the
// rounded b2 = 0.999 they would be off by 1.3e-5 relative.
__global__ void k_adam(float* p, float* m, float* v, const float* g, int64_t n, float lr, float b1, float omb1,
                       float b2, float omb2, float eps, float bc1, float bc2) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + omb1 * gi;
    const float vi = b2 * v[i] + omb2 * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

// ---- device-side training loop (tf_fno_train, tf_fno_eval) ----

// Per-block float64 sums of squares over n floats (fixed grid, so the
// partials and their host sum in block order are deterministic).
constexpr int SQ_BLOCKS = 2048;
__global__ __launch_bounds__(256) void k_sumsq32(const float* x, int64_t n, double* part) {
    double s = 0;
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(SQ_BLOCKS) * 256) {
        const double v = x[i];
        s += v * v;
    }
    __shared__ double r[256];
    r[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) r[threadIdx.x] += r[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = r[0];
}

// Minibatch gather: sample b of the batch is row idx[b] of the data set;
// targets are multiplied by tscale on the way (grid: (blocks, B)).
__global__ __launch_bounds__(256) void k_gather_targets(const float* y, const int* idx, float tscale, float* yb) {
    const int b = blockIdx.y;
    const float4* src = reinterpret_cast<const float4*>(y + int64_t(idx[b]) * OUT_SZ);
    float4* dst = reinterpret_cast<float4*>(yb + int64_t(b) * OUT_SZ);
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < OUT_SZ / 4; i += int64_t(gridDim.x) * 256) {
        float4 v = src[i];
        v.x *= tscale; v.y *= tscale; v.z *= tscale; v.w *= tscale;
        dst[i] = v;
    }
}
__global__ void k_gather_rows(const float* p, const float* w, const int* idx, int B, int nb, float* pb, float* wb) {
    for (int i = threadIdx.x; i < B * NPAR; i += blockDim.x) pb[i] = p[int64_t(idx[i / NPAR]) * NPAR + i % NPAR];
    if (w)
        for (int i = threadIdx.x; i < B * nb; i += blockDim.x) wb[i] = w[int64_t(idx[i / nb]) * nb + i % nb];
}
__global__ void k_log_loss(const double* res, double* log, int step) { log[step] = res[0]; }
__global__ void k_scale(float* x, int64_t n, float s) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) x[i] *= s;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

using host::fail;

constexpr Ix plain(int s) { return Ix{30, 0, s}; }
constexpr Ix two(int sh, int hi, int lo) { return Ix{sh, hi, lo}; }

// largest element offset an operand touches (all strides non-negative)
constexpr int64_t max_ix(Ix a, int n) {
    if (n <= 0) return 0;
    const int64_t mask = (int64_t(1) << a.sh) - 1;
    return int64_t((n - 1) >> a.sh) * a.hi + std::min<int64_t>(n - 1, mask) * a.lo;
}

typedef void (*GemmLaunch)(const GemmArgs&, int, int, hipStream_t);

template <int BM, int BN, int NW, typename TA, typename TB, bool SPLIT, int DEPTH>
void launch(const GemmArgs& g, int by, int bz, hipStream_t st) {
    const int tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
    hipLaunchKernelGGL((k_gemm<BM, BN, NW, TA, TB, SPLIT, DEPTH>), dim3(tiles, by, bz), dim3(64 * NW), 0, st, g);
}

struct Gemm {
    GemmArgs g;
    int by, bz;
    GemmLaunch fn;
};

// Checks an operand against the size of the buffer it addresses.
inline bool fits(const Operand& o, int rows, int cols, int by, int bz, int64_t size) {
    const int r = std::min(rows, o.ones_from);
    const int64_t mx = int64_t(by - 1) * o.b1 + int64_t(bz - 1) * o.b2 + max_ix(o.r, r) + max_ix(o.c, cols);
    return mx < size;
}
inline bool fits(const Result& o, int rows, int cols, int by, int bz, int64_t size) {
    const int64_t mx = int64_t(by - 1) * o.b1 + int64_t(bz - 1) * o.b2 + max_ix(o.r, rows) + max_ix(o.c, cols);
    return mx < size;
}

inline Operand opnd(const void* p, Ix r, Ix c, int64_t b1, int64_t b2, int fast_k, int ones_from = 1 << 30) {
    return Operand{p, b1, b2, r, c, ones_from, fast_k, 0};
}

// Whether groups of 4 along the operand's contiguous index are contiguous and
// aligned for 4-element loads (rows x cols is the operand's shape).  Rows
// from ones_from on are never loaded (stage takes them first), so they do
// not bar the vector loads of the others.
inline bool vec_ok(const Operand& o, int rows, int cols, bool is_b, size_t elem) {
    if (!o.fast_k) return false;
    const bool k_is_row = is_b;                 // A: (M, K); B: (K, N)
    const Ix fast = o.fast_k ? (k_is_row ? o.r : o.c) : (k_is_row ? o.c : o.r);
    const Ix slow = o.fast_k ? (k_is_row ? o.c : o.r) : (k_is_row ? o.r : o.c);
    const int fext = o.fast_k ? (k_is_row ? rows : cols) : (k_is_row ? cols : rows);
    auto mult4 = [](int64_t v) { return v % 4 == 0; };
    if (fast.lo != 1 || fast.sh < 2 || fext % 4) return false;
    if (fast.sh < 30 && !mult4(fast.hi)) return false;
    if (!mult4(slow.lo) || (slow.sh < 30 && !mult4(slow.hi))) return false;
    if (!mult4(o.b1) || !mult4(o.b2)) return false;
    return (uintptr_t)o.p % (4 * elem) == 0;
}
inline Result res(float* p, Ix r, Ix c, int64_t b1, int64_t b2) {
    return Result{p, b1, b2, r, c};
}

// DFT tables, float64-built from the exact integer phase (j k mod P), for
// the spectral transform of period P >= N: the window extended by zeros to
// P nodes per axis, the kept modes [0, M) (x) and [0, M) U [P - M, P) (y, z)
// of the period-P DFT, and the inverse's 1/P per axis, cut back to the N
// window nodes.  P = N is the plain transform; the backward passes use the
// transposed tables, so they are the exact adjoints for any P.
struct Tables {
    std::vector<float> fx, fxT, gx, gxT, fs, fsT, gs, gsT;
};

inline Tables build_tables(int P) {
    Tables t;
    auto ang = [P](int a, int b) { return 2.0 * M_PI * double((int64_t(a) * b) % P) / P; };
    auto side = [P](int i) { return i < M ? i : P - 2 * M + i; };
    t.fx.assign(24 * N, 0.f);
    t.gx.assign(N * 24, 0.f);
    for (int kx = 0; kx < M; ++kx)
        for (int x = 0; x < N; ++x) {
            const double th = ang(kx, x), mult = kx == 0 ? 1.0 : 2.0;
            t.fx[(0 * M + kx) * N + x] = float(std::cos(th));
            t.fx[(1 * M + kx) * N + x] = float(-std::sin(th));
            t.gx[x * 24 + 0 * M + kx] = float(mult / P * std::cos(th));
            t.gx[x * 24 + 1 * M + kx] = float(-mult / P * std::sin(th));
        }
    t.fs.assign(48 * 128, 0.f);
    t.gs.assign(128 * 48, 0.f);
    for (int ki = 0; ki < KS; ++ki)
        for (int n = 0; n < N; ++n) {
            const double th = ang(side(ki), n);
            const double fr = std::cos(th), fi = -std::sin(th);       // e^{-i th}
            const double gr = std::cos(th) / P, gi = std::sin(th) / P; // e^{+i th} / P
            // forward block [[fr, -fi], [fi, fr]] at (row (ki, s'), col (n, s))
            t.fs[(2 * ki + 0) * 128 + 2 * n + 0] = float(fr);
            t.fs[(2 * ki + 0) * 128 + 2 * n + 1] = float(-fi);
            t.fs[(2 * ki + 1) * 128 + 2 * n + 0] = float(fi);
            t.fs[(2 * ki + 1) * 128 + 2 * n + 1] = float(fr);
            // inverse block at (row (n, s), col (ki, s'))
            t.gs[(2 * n + 0) * 48 + 2 * ki + 0] = float(gr);
            t.gs[(2 * n + 0) * 48 + 2 * ki + 1] = float(-gi);
            t.gs[(2 * n + 1) * 48 + 2 * ki + 0] = float(gi);
            t.gs[(2 * n + 1) * 48 + 2 * ki + 1] = float(gr);
        }
    auto tr = [](const std::vector<float>& a, int r, int c) {
        std::vector<float> o(a.size());
        for (int i = 0; i < r; ++i)
            for (int j = 0; j < c; ++j) o[j * r + i] = a[i * c + j];
        return o;
    };
    t.fxT = tr(t.fx, 24, N);
    t.gxT = tr(t.gx, N, 24);
    t.fsT = tr(t.fs, 48, 128);
    t.gsT = tr(t.gs, 128, 48);
    return t;
}

}  // namespace fno
}  // namespace tf

using namespace tf::fno;
using tf::host::fail;

struct tf_fno {
    int dev = 0;
    hipStream_t st = nullptr;   // the caller's stream
    hipStream_t cur = nullptr;  // stream launches go to (st, or cap while capturing)
    hipStream_t cap = nullptr;  // private stream inference graphs are captured on
    hipGraphExec_t exec = nullptr;
    const float* g_params = nullptr;
    float* g_out = nullptr;
    int g_batch = 0;
    int maxB = 0;
    int nb = 1;                 // basis fields of the output head
    int64_t np = 0;             // parameter count
    const float* g_w = nullptr;
    bool training = false;
    int64_t adam_t = 0;
    bool working_stale = true;

    std::vector<void*> allocs;
    float *prm = nullptr, *grad = nullptr, *am = nullptr, *av = nullptr;
    bf16 *wb[LAYERS] = {}, *rb[LAYERS] = {}, *p1b = nullptr, *p2e = nullptr, *p1k = nullptr, *p1f = nullptr, *p2k = nullptr;
    float *c2e = nullptr, *geff = nullptr;
    float *fx, *fxT, *gx, *gxT, *fs, *fsT, *gs, *gsT;
    float* tab = nullptr;       // the eight tables, one allocation
    int period = N;             // period of the spectral transform (tables built for it)
    float* V[4] = {};
    float* Z[2] = {};
    float* X3[LAYERS] = {};
    float *T1 = nullptr, *T2 = nullptr, *Y = nullptr, *Y2 = nullptr;
    float *G[2] = {};
    float *out = nullptr, *gout = nullptr, *part = nullptr, *gstar = nullptr;
    bf16 *hT = nullptr, *ghT = nullptr;
    float *pbuf = nullptr, *wbuf = nullptr, *ybuf = nullptr;   // tf_fno_train minibatches (on first use)
    double* dres = nullptr;
    double* lpart = nullptr;

    ~tf_fno() {
        if (st) hipStreamSynchronize(st);
        else hipDeviceSynchronize();
        if (exec) (void)hipGraphExecDestroy(exec);
        if (cap) (void)hipStreamDestroy(cap);
        for (void* p : allocs) hipFree(p);
    }

    template <typename T>
    tf_status alloc(T** p, int64_t n) {
        void* q = nullptr;
        const hipError_t e = tf::host::BlockCache::get().alloc(&q, size_t(n) * sizeof(T));
        if (e != hipSuccess) return fail(TF_ENOMEM, std::string("hipMalloc: ") + hipGetErrorString(e));
        allocs.push_back(q);
        *p = (T*)q;
        return TF_OK;
    }
};

namespace {

constexpr int LOSS_CH = 64;

#define TRY(x)                           \
    do {                                 \
        tf_status s_ = (x);              \
        if (s_ != TF_OK) return s_;      \
    } while (0)

tf_status launched() {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(TF_EDEVICE, std::string("kernel launch: ") + hipGetErrorString(e));
    return TF_OK;
}

tf_status run(tf_fno* f, Gemm g, int64_t sa, int64_t sb, int64_t sc, size_t ea = 4, size_t eb = 4) {
    if (!fits(g.g.a, g.g.M, g.g.K, g.by, g.bz, sa) || !fits(g.g.b, g.g.K, g.g.N, g.by, g.bz, sb) ||
        !fits(g.g.c, g.g.M, g.g.N, g.by, g.bz, sc))
        return fail(TF_EINVAL, "internal: GEMM operand exceeds its buffer");
    g.g.a.vec = vec_ok(g.g.a, g.g.M, g.g.K, false, ea);
    g.g.b.vec = vec_ok(g.g.b, g.g.K, g.g.N, true, eb);
    g.fn(g.g, g.by, g.bz, f->cur);
    return launched();
}

// ---- the spectral stages (per sample b = blockIdx.z) ----

// x contraction: out[(s,kx)][(zy,c)] = sum_x A[(s,kx)][x] in[(zy,x,c)]
Gemm g_xcontract(const float* A, const float* in, float* out, int B) {
    GemmArgs g{opnd(A, plain(N), plain(1), 0, 0, 1),
               opnd(in, plain(C), two(5, N * C, 1), 0, NODE_SZ, 0),
               res(out, plain(C), two(5, 2 * LINE, 1), 0, X1_SZ), 24, N * N * C, N};
    return Gemm{g, 1, B, launch<32, 128, 4, float, float, true, 1>};
}
// Whether rows k < n of ny matrices y apart, LINE columns each, lie in a sample
// of `size` elements (the buffers hold whole samples, and check_batch bounds
// their number).
constexpr bool axis_fits(Ix k, int n, int64_t y, int ny, int64_t size) {
    return (ny - 1) * y + max_ix(k, n) + LINE <= size;
}

// One y or z transform: the layouts of its operands, checked as it is compiled.
template <int M_, int K_, int NY> struct AxisLayout {
    Ix in_k, out_r;
    int64_t in_y, in_b, out_y, out_b;
    constexpr bool fits() const {
        return axis_fits(in_k, K_, in_y, NY, in_b) && axis_fits(out_r, M_, out_y, NY, out_b);
    }
};

// The y and z transforms of B samples.  MT = all row tiles of A per wave reads
// the input once (batch 64, the twelve of a pass: 2.14 ms through k_gemm, 1.79
// so, 5.1 TB/s); below FEW waves (one per SIMD) the tiles go to waves of their
// own, which share the columns through the L1 (batch 1: 11 -> 6.7 us each).
template <int M, int K, int NY>
tf_status axis(tf_fno* f, const float* A, const float* in, float* out, const AxisLayout<M, K, NY>& l, int B) {
    constexpr int MTOT = (M + 31) / 32, FEW = 1024;
    const auto hi = [](Ix x) { return x.sh == 1 ? x.hi : 2 * x.lo; };
    AxisArgs a{A, in, out, hi(l.in_k), l.in_k.lo, hi(l.out_r), l.out_r.lo, l.in_y, l.in_b, l.out_y, l.out_b, NY, 0};
    const int cols = B * NY * (LINE / 32);
    const auto go = [&](auto kernel, int items) {
        a.nitems = items;
        // at most four blocks per CU: a wave takes several items, and A is split less often
        hipLaunchKernelGGL(kernel, dim3(std::min((items + 3) / 4, 1024)), dim3(256), 0, f->cur, a);
    };
    if (cols < FEW) go(k_axis<M, K, 1>, cols * MTOT);
    else go(k_axis<M, K, MTOT>, cols);
    return launched();
}
// y contraction (per z): X1 layout in, X2 layout out; A is 48 x 128
tf_status ycontract(tf_fno* f, const float* A, const float* in, float* out, int B) {
    constexpr AxisLayout<48, 128, N> l{plain(LINE), two(1, N * 2 * LINE, LINE), int64_t(N) * 2 * LINE, X1_SZ, 2 * LINE,
                                       X2_SZ};
    static_assert(l.fits());
    return axis(f, A, in, out, l, B);
}
// z contraction (per ky): X2 layout in, mode layout out
tf_status zcontract(tf_fno* f, const float* A, const float* in, float* out, int B) {
    constexpr AxisLayout<48, 128, KS> l{plain(LINE), plain(KS * LINE), int64_t(N) * 2 * LINE, X2_SZ, LINE, X3_SZ};
    static_assert(l.fits());
    return axis(f, A, in, out, l, B);
}
// z expansion (per ky): mode layout in, X2 layout out; A is 128 x 48
tf_status zexpand(tf_fno* f, const float* A, const float* in, float* out, int B) {
    constexpr AxisLayout<128, 48, KS> l{plain(KS * LINE), plain(LINE), LINE, X3_SZ, int64_t(N) * 2 * LINE, X2_SZ};
    static_assert(l.fits());
    return axis(f, A, in, out, l, B);
}
// y expansion (per z): X2 layout in, X1 layout out
tf_status yexpand(tf_fno* f, const float* A, const float* in, float* out, int B) {
    constexpr AxisLayout<128, 48, N> l{two(1, N * 2 * LINE, LINE), plain(LINE), 2 * LINE, X2_SZ, int64_t(N) * 2 * LINE,
                                       X1_SZ};
    static_assert(l.fits());
    return axis(f, A, in, out, l, B);
}

// x-lines of B samples
template <bool BWD> tf_status lineout(tf_fno* f, LineArgs a, int B) {
    a.lpw = lines_per_wave(B * N * N);
    hipLaunchKernelGGL(k_lineout<BWD>, dim3(B * N * N / (4 * a.lpw)), dim3(256), 0, f->cur, a);
    return launched();
}

// ---- per-mode complex channel mixing as real 64 x 64 blocks ----
// mode q = kz * 288 + (ky * 12 + kx): blockIdx.y = ky * 12 + kx, blockIdx.z = kz
constexpr int64_t MODE_Y = C, MODE_Z = 2 * KS * LINE;

// Y*[b][(s',o)] = sum X*[b][(s,c)] Wq[(s,c)][(s',o)]  (trans: Wq^T); kfast:
// R holds the matrices with the contracted index contiguous
Gemm g_mix(const float* X, const bf16* R, float* Yo, int B, bool trans, bool kfast) {
    const Ix rr = kfast ? plain(1) : plain(64), rc = kfast ? plain(64) : plain(1);
    GemmArgs g{opnd(X, plain(X3_SZ), two(5, KS * LINE, 1), MODE_Y, MODE_Z, 1),
               opnd(R, rr, rc, 4096, int64_t(KS * M) * 4096, kfast ? 1 : 0),
               res(Yo, plain(X3_SZ), two(5, KS * LINE, 1), MODE_Y, MODE_Z), B, 64, 64};
    // the adjoint (trans) splits the gradient operand into bf16 hi + lo; the
    // forward keeps one bf16 copy of the modes
    return Gemm{g, KS * M, KS, trans ? launch<32, 64, 2, float, bf16, true, 2>
                                        : launch<32, 64, 2, float, bf16, false, 2>};
}
// G*[q][(s,c)][(s',o)] = sum_b X*[b][(s,c)] gY*[b][(s',o)]
Gemm g_mix_grad(const float* X, const float* gY, float* gs, int B) {
    GemmArgs g{opnd(X, two(5, KS * LINE, 1), plain(X3_SZ), MODE_Y, MODE_Z, 0),
               opnd(gY, plain(X3_SZ), two(5, KS * LINE, 1), MODE_Y, MODE_Z, 0),
               res(gs, plain(64), plain(1), 4096, int64_t(KS * M) * 4096), 64, 64, B};
    return Gemm{g, KS * M, KS, launch<64, 64, 4, float, float, true, 1>};
}

}  // namespace

extern "C" {

int64_t tf_fno_param_count(int32_t nbasis) {
    return (nbasis == 1 || nbasis == 2 || nbasis == 4) ? nparams(nbasis) : -1;
}

tf_status tf_fno_phasor_weights(const tf_pulse* pulse, int32_t nbasis, double* w) {
    if (!w) return fail(TF_EINVAL, "w is NULL");
    if (nbasis != 1 && nbasis != 2 && nbasis != 4) return fail(TF_EINVAL, "nbasis must be 1, 2 or 4");
    TRY(tf::host::validate_pulse(pulse));
    if (nbasis == 1) {
        w[0] = 1.0;
        return TF_OK;
    }
    // envelope Re[exp(i sig phase) G]: sig = +1 spectral, -1 for the sin(k z - phase) envelopes
    const double sig = pulse->envelope == TF_ENV_SPECTRAL ? 1.0 : -1.0;
    double gnorm = 1.0;
    if (pulse->envelope == TF_ENV_SPECTRAL) {
        std::vector<double> tab;
        tf::host::spectral_table(pulse, tab, gnorm);
        if (!(gnorm > 0.0)) return fail(TF_EINVAL, "spectral pulse vanishes in its window");
    }
    const double zr = std::cos(sig * pulse->cep), zi = std::sin(sig * pulse->cep);
    if (nbasis == 2) {
        w[0] = zr / gnorm;
        w[1] = -zi / gnorm;
        return TF_OK;
    }
    double ar = 1.0, ai = 0.0, br = 0.0, bi = 0.0;
    if (pulse->polarization == TF_POL_LINEAR) {
        const double e = pulse->ellipticity, n = std::sqrt(1.0 + e * e);
        const double c = std::cos(pulse->pol_angle), s = std::sin(pulse->pol_angle);
        ar = c / n; ai = -sig * e * s / n;
        br = s / n; bi = sig * e * c / n;
    }
    w[0] = (zr * ar - zi * ai) / gnorm;     // Re(z a)
    w[1] = -(zr * ai + zi * ar) / gnorm;    // -Im(z a)
    w[2] = (zr * br - zi * bi) / gnorm;
    w[3] = -(zr * bi + zi * br) / gnorm;
    return TF_OK;
}

// Builds the DFT tables of period P and copies them into f->tab (synchronous).
static tf_status upload_tables(tf_fno* f, int P) {
    Tables t = build_tables(P);
    std::vector<float> all;
    auto put = [&](const std::vector<float>& v, float** p) {
        *p = f->tab + all.size();
        all.insert(all.end(), v.begin(), v.end());
    };
    put(t.fx, &f->fx); put(t.fxT, &f->fxT); put(t.gx, &f->gx); put(t.gxT, &f->gxT);
    put(t.fs, &f->fs); put(t.fsT, &f->fsT); put(t.gs, &f->gs); put(t.gsT, &f->gsT);
    TF_HIP(hipMemcpyAsync(f->tab, all.data(), all.size() * sizeof(float), hipMemcpyHostToDevice, f->st));
    TF_HIP(hipStreamSynchronize(f->st));
    f->period = P;
    return TF_OK;
}

tf_status tf_fno_set_period(tf_fno* f, int32_t period) {
    if (!f) return fail(TF_EINVAL, "NULL argument");
    if (period < N || period > 4 * N) return fail(TF_EINVAL, "period must be in [64, 256]");
    if (period == f->period) return TF_OK;
    TF_HIP(hipSetDevice(f->dev));
    TF_HIP(hipStreamSynchronize(f->st));
    return upload_tables(f, period);
}

tf_status tf_fno_get_period(const tf_fno* f, int32_t* period) {
    if (!f || !period) return fail(TF_EINVAL, "NULL argument");
    *period = f->period;
    return TF_OK;
}

tf_status tf_fno_create(int32_t max_batch, int32_t training, int32_t nbasis, void* hip_stream, tf_fno** out) {
    if (!out) return fail(TF_EINVAL, "out is NULL");
    *out = nullptr;
    if (max_batch < 1 || max_batch > 128) return fail(TF_EINVAL, "max_batch must be in [1, 128]");
    if (nbasis != 1 && nbasis != 2 && nbasis != 4) return fail(TF_EINVAL, "nbasis must be 1, 2 or 4");
    tf::host::BlockCache::get().clear();      // blocks kept from finished solvers and batches
    std::unique_ptr<tf_fno> f(new tf_fno());
    f->nb = nbasis;
    f->np = nparams(nbasis);
    f->maxB = max_batch;
    f->training = training != 0;
    f->st = (hipStream_t)hip_stream;
    f->cur = f->st;
    TF_HIP(hipGetDevice(&f->dev));
    TF_HIP(hipStreamCreateWithFlags(&f->cap, hipStreamNonBlocking));
    const int64_t B = max_batch;

    const int64_t NPARAMS = f->np;
    TRY(f->alloc(&f->prm, NPARAMS));
    TF_HIP(hipMemset(f->prm, 0, NPARAMS * sizeof(float)));
    for (int l = 0; l < LAYERS; ++l) {
        TRY(f->alloc(&f->wb[l], C * C));
        TRY(f->alloc(&f->rb[l], int64_t(NMODES) * 4096));
    }
    TRY(f->alloc(&f->p1b, C * HID));
    TRY(f->alloc(&f->p2e, B * HID * NOUT));
    TRY(f->alloc(&f->c2e, B * NOUT));
    TRY(f->alloc(&f->p1k, C * HID));
    TRY(f->alloc(&f->p1f, C * HID));
    TRY(f->alloc(&f->p2k, B * KSLOTS));
    TF_HIP(hipMemset(f->p2k, 0, B * KSLOTS * sizeof(bf16)));     // rows t >= 6 stay 0

    const int64_t ntab = 4 * 24 * N + 4 * 48 * 128;
    TRY(f->alloc(&f->tab, ntab));
    TRY(upload_tables(f.get(), N));

    TRY(f->alloc(&f->V[0], B * NODE_SZ));
    TRY(f->alloc(&f->V[1], B * NODE_SZ));
    TRY(f->alloc(&f->T1, B * X1_SZ));
    TRY(f->alloc(&f->T2, B * X2_SZ));
    TRY(f->alloc(&f->X3[0], B * X3_SZ));
    TRY(f->alloc(&f->Y, B * X3_SZ));
    TRY(f->alloc(&f->out, B * OUT_SZ));
    TRY(f->alloc(&f->dres, 1 + 2 * B));      // loss, per-sample scales, per-sample ratios
    TRY(f->alloc(&f->lpart, B * LOSS_CH * 2));
    if (f->training) {
        TRY(f->alloc(&f->grad, NPARAMS));
        TRY(f->alloc(&f->am, NPARAMS));
        TRY(f->alloc(&f->av, NPARAMS));
        TF_HIP(hipMemset(f->am, 0, NPARAMS * sizeof(float)));
        TF_HIP(hipMemset(f->av, 0, NPARAMS * sizeof(float)));
        TRY(f->alloc(&f->V[2], B * NODE_SZ));
        TRY(f->alloc(&f->V[3], B * NODE_SZ));
        TRY(f->alloc(&f->Z[0], B * NODE_SZ));
        TRY(f->alloc(&f->Z[1], B * NODE_SZ));
        TRY(f->alloc(&f->G[0], B * NODE_SZ));
        TRY(f->alloc(&f->G[1], B * NODE_SZ));
        TRY(f->alloc(&f->X3[1], B * X3_SZ));
        TRY(f->alloc(&f->X3[2], B * X3_SZ));
        TRY(f->alloc(&f->Y2, B * X3_SZ));
        TRY(f->alloc(&f->gout, B * OUT_SZ));
        TRY(f->alloc(&f->hT, B * HID * N3));
        TRY(f->alloc(&f->ghT, B * HID * N3));
        TRY(f->alloc(&f->part, B * NCHUNK * 33 * HID));
        TRY(f->alloc(&f->gstar, int64_t(NMODES) * 4096));
        TRY(f->alloc(&f->geff, B * (HID + 1) * NOUT));
    }
    TF_HIP(hipDeviceSynchronize());
    *out = f.release();
    return TF_OK;
}

tf_status tf_fno_destroy(tf_fno* f) {
    delete f;
    return TF_OK;
}

}  // extern "C"

namespace {

tf_status refresh_working(tf_fno* f) {
    if (!f->working_stale) return TF_OK;
    for (int l = 0; l < LAYERS; ++l) {
        hipLaunchKernelGGL(k_to_bf16, dim3((C * C + 255) / 256), dim3(256), 0, f->cur, f->prm + off_w(l), f->wb[l],
                           C * C);
        hipLaunchKernelGGL(k_expand_r, dim3(NMODES), dim3(256), 0, f->cur, f->prm + off_r(l), f->rb[l],
                           f->training ? 0 : 1);
    }
    hipLaunchKernelGGL(k_to_bf16, dim3((C * HID + 255) / 256), dim3(256), 0, f->cur, f->prm + OFF_P1, f->p1b, C * HID);
    hipLaunchKernelGGL(k_p1_frag, dim3((C * HID + 255) / 256), dim3(256), 0, f->cur, f->prm + OFF_P1, f->p1k, f->p1f);
    TRY(launched());
    f->working_stale = false;
    return TF_OK;
}

// Forward pass.  Training keeps v_l, z_l and the modes of every layer for the
// backward pass; inference ping-pongs two node tensors.
tf_status forward_infer(tf_fno* f, const float* params, int B, float* out);

tf_status forward_body(tf_fno* f, const float* params, const float* hw, int B, float* out) {
    const int64_t nb = B;
    {
        const int n = B * (HID + 1) * NOUT;
        hipLaunchKernelGGL(k_head_eff, dim3((n + 255) / 256), dim3(256), 0, f->cur, f->prm + OFF_P2,
                           f->prm + off_c2(f->nb), hw, f->nb, B, f->p2e, f->c2e, f->p2k);
    }
    if (!f->training) return forward_infer(f, params, B, out);
    hipLaunchKernelGGL(k_lift, dim3(B * N * N / LIFT_LINES), dim3(256), 0, f->cur, params, f->prm + OFF_W0,
                       f->prm + OFF_B0, f->V[0]);
    TRY(launched());
    const int64_t szN = nb * NODE_SZ, sz1 = nb * X1_SZ, sz3 = nb * X3_SZ;
    float* v = f->V[0];
    for (int l = 0; l < LAYERS; ++l) {
        float* modes = f->training ? f->X3[l] : f->X3[0];
        TRY(run(f, g_xcontract(f->fx, v, f->T1, B), 24 * N, szN, sz1));
        TRY(ycontract(f, f->fs, f->T1, f->T2, B));
        TRY(zcontract(f, f->fs, f->T2, modes, B));
        TRY(run(f, g_mix(modes, f->rb[l], f->Y, B, false, false), sz3, int64_t(NMODES) * 4096, sz3, 4, 2));
        TRY(zexpand(f, f->gs, f->Y, f->T2, B));
        TRY(yexpand(f, f->gs, f->T2, f->T1, B));
        float* nv = f->training ? f->V[l + 1] : (v == f->V[0] ? f->V[1] : f->V[0]);
        LineArgs a{f->gx, f->T1, v, f->wb[l], f->prm + off_b(l), nullptr,
                   (f->training && l < LAYERS - 1) ? f->Z[l] : nullptr, nv, 0, l < LAYERS - 1};
        TRY(lineout<false>(f, a, B));
        v = nv;
    }
    const ProjArgs p{v, f->p1b, f->p1f, f->prm + OFF_C1, f->p2e, f->p2k, f->c2e, out, nullptr, nullptr, nullptr, nullptr};
    hipLaunchKernelGGL(k_proj<false>, dim3(B * (N3 / 256)), dim3(256), 0, f->cur, p);
    return launched();
}

// Inference: lift + first x contraction, then per layer the y and z
// contractions, mixing and expansions, and one fused x-line kernel.
tf_status forward_infer(tf_fno* f, const float* params, int B, float* out) {
    const int64_t nb = B;
    const int64_t sz3 = nb * X3_SZ;
    const int lines = B * N * N, lpw = lines_per_wave(lines);
    InfArgs a{f->gx, f->fx, f->T1, nullptr, params, f->prm + OFF_W0, f->prm + OFF_B0, nullptr, nullptr,
              nullptr, f->T1, f->p1k, f->prm + OFF_C1, f->p2k, f->c2e, out, lpw};
    hipLaunchKernelGGL(k_lift_x, dim3(lines / (4 * lpw)), dim3(256), 0, f->cur, a);
    TRY(launched());
    const float* v = nullptr;                 // v_0 is recomputed, never stored
    for (int l = 0; l < LAYERS; ++l) {
        TRY(ycontract(f, f->fs, f->T1, f->T2, B));
        TRY(zcontract(f, f->fs, f->T2, f->X3[0], B));
        TRY(run(f, g_mix(f->X3[0], f->rb[l], f->Y, B, false, true), sz3, int64_t(NMODES) * 4096, sz3, 4, 2));
        TRY(zexpand(f, f->gs, f->Y, f->T2, B));
        TRY(yexpand(f, f->gs, f->T2, f->T1, B));
        a.act = v;
        a.w = f->wb[l];
        a.bias = f->prm + off_b(l);
        if (l < LAYERS - 1) {
            float* nv = (v == f->V[0]) ? f->V[1] : f->V[0];
            a.vout = nv;
            if (v) hipLaunchKernelGGL(k_line_fwd<false>, dim3(lines / (4 * lpw)), dim3(256), 0, f->cur, a);
            else hipLaunchKernelGGL(k_line_fwd<true>, dim3(lines / (4 * lpw)), dim3(256), 0, f->cur, a);
            v = nv;
        } else {
            hipLaunchKernelGGL(k_line_proj, dim3(lines / (2 * lpw)), dim3(256), 0, f->cur, a);
        }
        TRY(launched());
    }
    return TF_OK;
}

tf_status forward(tf_fno* f, const float* params, const float* hw, int B, float* out) {
    TRY(refresh_working(f));
    return forward_body(f, params, hw, B, out);
}

// split-K weight gradient [A | 1]^T-style reductions into the flat gradient
tf_status reduce_into(tf_fno* f, int nparts, int len, float* dst, int groups = 1) {
    hipLaunchKernelGGL(k_reduce, dim3((len + 63) / 64, groups), dim3(256), 0, f->cur, f->part, nparts, len, dst);
    return launched();
}

// Backward pass.  The weight-gradient GEMMs and the adjoint of the mixing
// take their float32 operands as bf16 hi + lo parts (three MFMAs, about
// float32 products): a one-part bf16 copy of each activation would put a
// relative error of up to 2^-9 on every term of sums that cancel heavily.
// The bf16 weights themselves are exact in either form.
tf_status backward(tf_fno* f, const float* params, const float* hw, const float* target, int B) {
    const int64_t nb = B;
    const int64_t szN = nb * NODE_SZ, sz1 = nb * X1_SZ, sz3 = nb * X3_SZ;
    const int64_t szO = nb * OUT_SZ;
    // loss and dL/dout
    hipLaunchKernelGGL(k_loss_part, dim3(LOSS_CH, B), dim3(256), 0, f->cur, f->out, target, f->lpart);
    hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(LOSS_THREADS), 0, f->cur, f->lpart, LOSS_CH, B, f->dres,
                       f->dres + 1 + B);
    hipLaunchKernelGGL(k_gout, dim3((szO + 255) / 256), dim3(256), 0, f->cur, f->out, target, f->dres, f->gout, szO);
    TRY(launched());
    // projection
    float* g = f->G[0];
    const ProjArgs p{f->V[3], f->p1b, f->p1f, f->prm + OFF_C1, f->p2e, f->p2k, f->c2e, nullptr, f->gout, g, f->hT,
                     f->ghT};
    hipLaunchKernelGGL(k_proj<true>, dim3(B * (N3 / 256)), dim3(256), 0, f->cur, p);
    TRY(launched());
    {   // [P1; c1] = [v3 | 1]^T dL/dpre
        GradArgs a{f->V[3], f->ghT, NODE_SZ * 4, int64_t(HID) * N3 * 2, f->part, C, HID};
        hipLaunchKernelGGL((k_wgrad<NodeFrag, HiddenFrag>), dim3(HID / 64, NCHUNK, B), dim3(64), 0, f->cur, a);
        TRY(launched());
        TRY(reduce_into(f, B * NCHUNK, 33 * HID, f->grad + OFF_P1));
    }
    {   // [P2; c2] = [h | 1]^T dL/dout
        GradArgs a{f->hT, f->gout, int64_t(HID) * N3 * 2, OUT_SZ * 4, f->part, HID, NOUT};
        hipLaunchKernelGGL((k_wgrad<HiddenFrag, OutFrag>), dim3(HID / 64, NCHUNK, B), dim3(64), 0, f->cur, a);
        TRY(launched());
        // per-sample gradient of the effective head, then through the head weights
        TRY(reduce_into(f, NCHUNK, 129 * NOUT, f->geff, B));
        const int n = (HID + 1) * NOUT * f->nb;
        hipLaunchKernelGGL(k_head_grad, dim3((n + 255) / 256), dim3(256), 0, f->cur, f->geff, hw, f->nb, B,
                           f->grad + OFF_P2);
        TRY(launched());
    }
    for (int l = LAYERS - 1; l >= 0; --l) {
        float* gn = g == f->G[0] ? f->G[1] : f->G[0];
        {   // [W_l; b_l] = [v_l | 1]^T dL/dz_l
            GradArgs a{f->V[l], g, NODE_SZ * 4, NODE_SZ * 4, f->part, C, C};
            hipLaunchKernelGGL((k_wgrad<NodeFrag, NodeFrag>), dim3(1, NCHUNK, B), dim3(64), 0, f->cur, a);
            TRY(launched());
            TRY(reduce_into(f, B * NCHUNK, 33 * C, f->grad + off_w(l)));
        }
        // adjoint of the inverse transform: modes gradient
        TRY(run(f, g_xcontract(f->gxT, g, f->T1, B), 24 * N, szN, sz1));
        TRY(ycontract(f, f->gsT, f->T1, f->T2, B));
        TRY(zcontract(f, f->gsT, f->T2, f->Y, B));
        // mixing: dR and dX
        TRY(run(f, g_mix_grad(f->X3[l], f->Y, f->gstar, B), sz3, sz3, int64_t(NMODES) * 4096));
        {
            const int64_t n = int64_t(NMODES) * C * C;
            hipLaunchKernelGGL(k_fold_r, dim3((n + 255) / 256), dim3(256), 0, f->cur, f->gstar, f->grad + off_r(l));
            TRY(launched());
        }
        TRY(run(f, g_mix(f->Y, f->rb[l], f->Y2, B, true, true), sz3, int64_t(NMODES) * 4096, sz3, 4, 2));
        // adjoint of the forward transform, then the x line with the pointwise branch
        TRY(zexpand(f, f->fsT, f->Y2, f->T2, B));
        TRY(yexpand(f, f->fsT, f->T2, f->T1, B));
        LineArgs a{f->fxT, f->T1, g, f->wb[l], nullptr, l > 0 ? f->Z[l - 1] : nullptr, nullptr, gn, 0, 0};
        TRY(lineout<true>(f, a, B));
        g = gn;
    }
    hipLaunchKernelGGL(k_lift_grad_part, dim3(N, B), dim3(256), 0, f->cur, g, f->part);
    hipLaunchKernelGGL(k_lift_grad_final, dim3(1), dim3(LIFT_THREADS), 0, f->cur, f->part, params, B, f->grad);
    return launched();
}

// splitmix64 (Steele, Lea and Flood, OOPSLA 2014): the shuffles' generator.
uint64_t splitmix64(uint64_t& st) {
    uint64_t z = (st += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Device buffers of one call, freed on every return path after the stream
// has drained.
struct CallBuffers {
    hipStream_t st;
    std::vector<void*> ptrs;
    explicit CallBuffers(hipStream_t s) : st(s) {}
    ~CallBuffers() {
        if (!ptrs.empty()) (void)hipStreamSynchronize(st);
        for (void* p : ptrs) (void)hipFree(p);
    }
    template <typename T>
    tf_status alloc(T** p, int64_t n) {
        void* q = nullptr;
        const hipError_t e = tf::host::BlockCache::get().alloc(&q, size_t(n) * sizeof(T));
        if (e != hipSuccess) return fail(TF_ENOMEM, std::string("hipMalloc: ") + hipGetErrorString(e));
        ptrs.push_back(q);
        *p = static_cast<T*>(q);
        return TF_OK;
    }
};

tf_status check_batch(tf_fno* f, int B, const float* hw, bool need_w = true) {
    if (!f) return fail(TF_EINVAL, "surrogate is NULL");
    if (B < 1 || B > f->maxB) return fail(TF_EINVAL, "batch must be in [1, max_batch]");
    if (need_w && !hw && f->nb != 1) return fail(TF_EINVAL, "a head of several basis fields needs its weights");
    TF_HIP(hipSetDevice(f->dev));
    return TF_OK;
}

}  // namespace

extern "C" {

tf_status tf_fno_set_params(tf_fno* f, const float* src, int32_t src_on_device) {
    if (!f || !src) return fail(TF_EINVAL, "NULL argument");
    const int64_t NPARAMS = f->np;
    TF_HIP(hipSetDevice(f->dev));
    TF_HIP(hipMemcpyAsync(f->prm, src, NPARAMS * sizeof(float),
                          src_on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, f->st));
    if (f->training) {
        TF_HIP(hipMemsetAsync(f->am, 0, NPARAMS * sizeof(float), f->st));
        TF_HIP(hipMemsetAsync(f->av, 0, NPARAMS * sizeof(float), f->st));
    }
    f->adam_t = 0;
    f->working_stale = true;
    if (!src_on_device) TF_HIP(hipStreamSynchronize(f->st));
    return TF_OK;
}

tf_status tf_fno_get_params(tf_fno* f, float* dst, int32_t dst_on_device) {
    if (!f || !dst) return fail(TF_EINVAL, "NULL argument");
    const int64_t NPARAMS = f->np;
    TF_HIP(hipSetDevice(f->dev));
    TF_HIP(hipMemcpyAsync(dst, f->prm, NPARAMS * sizeof(float),
                          dst_on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, f->st));
    if (!dst_on_device) TF_HIP(hipStreamSynchronize(f->st));
    return TF_OK;
}

tf_status tf_fno_forward(tf_fno* f, const float* params, const float* head_w, int32_t batch, float* out) {
    TRY(check_batch(f, batch, head_w));
    if (!params || !out) return fail(TF_EINVAL, "NULL argument");
    return forward(f, params, head_w, batch, out);
}

tf_status tf_fno_infer(tf_fno* f, const float* params, const float* head_w, int32_t batch, float* out) {
    TRY(check_batch(f, batch, head_w));
    if (!params || !out) return fail(TF_EINVAL, "NULL argument");
    TRY(refresh_working(f));
    if (!f->exec || f->g_params != params || f->g_w != head_w || f->g_out != out || f->g_batch != batch) {
        if (f->exec) {
            TF_HIP(hipStreamSynchronize(f->st));
            TF_HIP(hipGraphExecDestroy(f->exec));
            f->exec = nullptr;
        }
        hipGraph_t graph = nullptr;
        TF_HIP(hipStreamBeginCapture(f->cap, hipStreamCaptureModeThreadLocal));
        f->cur = f->cap;
        const tf_status st = forward_body(f, params, head_w, batch, out);
        f->cur = f->st;
        const hipError_t e = hipStreamEndCapture(f->cap, &graph);
        if (st != TF_OK || e != hipSuccess) {
            if (graph) (void)hipGraphDestroy(graph);
            return st != TF_OK ? st : fail(TF_EDEVICE, std::string("graph capture: ") + hipGetErrorString(e));
        }
        const hipError_t e2 = hipGraphInstantiate(&f->exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e2 != hipSuccess) {
            f->exec = nullptr;
            return fail(TF_EDEVICE, std::string("graph instantiate: ") + hipGetErrorString(e2));
        }
        f->g_params = params;
        f->g_w = head_w;
        f->g_out = out;
        f->g_batch = batch;
    }
    TF_HIP(hipGraphLaunch(f->exec, f->st));
    return TF_OK;
}

tf_status tf_fno_loss_grad(tf_fno* f, const float* params, const float* head_w, const float* target, int32_t batch,
                           double* loss, float* grad) {
    TRY(check_batch(f, batch, head_w));
    if (!f->training) return fail(TF_ESTATE, "surrogate was created for inference only");
    if (!params || !target) return fail(TF_EINVAL, "NULL argument");
    const int64_t NPARAMS = f->np;
    TRY(forward(f, params, head_w, batch, f->out));
    TRY(backward(f, params, head_w, target, batch));
    if (grad) TF_HIP(hipMemcpyAsync(grad, f->grad, NPARAMS * sizeof(float), hipMemcpyDeviceToHost, f->st));
    if (loss) TF_HIP(hipMemcpyAsync(loss, f->dres, sizeof(double), hipMemcpyDeviceToHost, f->st));
    if (grad || loss) TF_HIP(hipStreamSynchronize(f->st));
    return TF_OK;
}

tf_status tf_fno_train_step(tf_fno* f, const float* params, const float* head_w, const float* target,
                            int32_t batch, double lr, double* loss) {
    if (!(lr >= 0.0) || !std::isfinite(lr)) return fail(TF_EINVAL, "lr must be finite and >= 0");
    TRY(tf_fno_loss_grad(f, params, head_w, target, batch, nullptr, nullptr));
    const int64_t NPARAMS = f->np;
    f->adam_t += 1;
    const double b1 = 0.9, b2 = 0.999;
    const float bc1 = float(1.0 - std::pow(b1, double(f->adam_t))), bc2 = float(1.0 - std::pow(b2, double(f->adam_t)));
    hipLaunchKernelGGL(k_adam, dim3((NPARAMS + 255) / 256), dim3(256), 0, f->cur, f->prm, f->am, f->av, f->grad,
                       NPARAMS, float(lr), float(b1), float(1.0 - b1), float(b2), float(1.0 - b2), 1e-8f, bc1, bc2);
    TRY(launched());
    f->working_stale = true;
    if (loss) {
        TF_HIP(hipMemcpyAsync(loss, f->dres, sizeof(double), hipMemcpyDeviceToHost, f->st));
        TF_HIP(hipStreamSynchronize(f->st));
    }
    return TF_OK;
}

tf_status tf_fno_train(tf_fno* f, const float* params, const float* head_w, const float* targets, int64_t n,
                       const tf_train_cfg* cfg, double* final_loss) {
    if (!f || !cfg) return fail(TF_EINVAL, "surrogate and cfg must not be NULL");
    if (!f->training) return fail(TF_ESTATE, "surrogate was created for inference only");
    if (!params || !targets) return fail(TF_EINVAL, "params and targets must not be NULL");
    if (f->nb != 1 && !head_w) return fail(TF_EINVAL, "a head of several basis fields needs its weights");
    const int B = cfg->batch;
    if (B < 1 || B > f->maxB) return fail(TF_EINVAL, "batch must be in [1, max_batch]");
    if (n < B || n > (int64_t(1) << 30)) return fail(TF_EINVAL, "need batch <= n < 2^30");
    if (cfg->epochs < 1) return fail(TF_EINVAL, "epochs must be >= 1");
    if (!std::isfinite(cfg->lr) || cfg->lr < 0.0) return fail(TF_EINVAL, "lr must be finite and >= 0");
    if (!(cfg->lr_min_frac >= 0.0 && cfg->lr_min_frac <= 1.0)) return fail(TF_EINVAL, "lr_min_frac must be in [0, 1]");
    TF_HIP(hipSetDevice(f->dev));
    const int64_t NPARAMS = f->np;
    if (!f->ybuf) {
        TRY(f->alloc(&f->pbuf, int64_t(f->maxB) * NPAR));
        TRY(f->alloc(&f->wbuf, int64_t(f->maxB) * f->nb));
        TRY(f->alloc(&f->ybuf, int64_t(f->maxB) * OUT_SZ));
    }
    const int64_t spe = n / B, total = spe * cfg->epochs;
    CallBuffers cb(f->st);
    int* idx = nullptr;
    double *log = nullptr, *part = nullptr;
    TRY(cb.alloc(&idx, n));
    TRY(cb.alloc(&log, spe));
    TRY(cb.alloc(&part, SQ_BLOCKS));
    // target scale: the root mean square of every target value
    double scale = 1.0;
    if (cfg->scale_targets) {
        hipLaunchKernelGGL(k_sumsq32, dim3(SQ_BLOCKS), dim3(256), 0, f->st, targets, n * OUT_SZ, part);
        TRY(launched());
        std::vector<double> h(SQ_BLOCKS);
        TF_HIP(hipMemcpyAsync(h.data(), part, SQ_BLOCKS * sizeof(double), hipMemcpyDeviceToHost, f->st));
        TF_HIP(hipStreamSynchronize(f->st));
        double ss = 0;
        for (double v : h) ss += v;
        scale = std::sqrt(ss / (double(n) * double(OUT_SZ)));
        if (!(scale > 0.0) || !std::isfinite(scale)) return fail(TF_ENONFINITE, "targets have no finite nonzero RMS");
    }
    const float tscale = float(1.0 / scale);
    std::vector<int> perm(n);
    std::vector<double> hlog(spe);
    uint64_t rng = cfg->seed;
    double last = 0.0;
    f->cur = f->st;
    const double b1 = 0.9, b2 = 0.999;
    for (int ep = 0; ep < cfg->epochs; ++ep) {
        // Fisher-Yates shuffle of the sample order
        for (int64_t i = 0; i < n; ++i) perm[i] = int(i);
        for (int64_t i = n - 1; i > 0; --i) std::swap(perm[i], perm[splitmix64(rng) % uint64_t(i + 1)]);
        TF_HIP(hipMemcpyAsync(idx, perm.data(), n * sizeof(int), hipMemcpyHostToDevice, f->st));
        for (int64_t k = 0; k < spe; ++k) {
            const int* bi = idx + k * B;
            hipLaunchKernelGGL(k_gather_rows, dim3(1), dim3(256), 0, f->st, params, f->nb != 1 ? head_w : nullptr, bi,
                               B, f->nb, f->pbuf, f->wbuf);
            hipLaunchKernelGGL(k_gather_targets, dim3(512, B), dim3(256), 0, f->st, targets, bi, tscale, f->ybuf);
            TRY(launched());
            const float* hw = f->nb != 1 ? f->wbuf : nullptr;
            TRY(forward(f, f->pbuf, hw, B, f->out));
            TRY(backward(f, f->pbuf, hw, f->ybuf, B));
            // cosine decay from lr to lr * lr_min_frac over all steps
            const double step = double(ep) * double(spe) + double(k);
            const double a = cfg->lr * (cfg->lr_min_frac +
                                        (1.0 - cfg->lr_min_frac) * 0.5 * (1.0 + std::cos(M_PI * step / double(total))));
            f->adam_t += 1;
            const float bc1 = float(1.0 - std::pow(b1, double(f->adam_t)));
            const float bc2 = float(1.0 - std::pow(b2, double(f->adam_t)));
            hipLaunchKernelGGL(k_adam, dim3((NPARAMS + 255) / 256), dim3(256), 0, f->st, f->prm, f->am, f->av, f->grad,
                               NPARAMS, float(a), float(b1), float(1.0 - b1), float(b2), float(1.0 - b2), 1e-8f, bc1,
                               bc2);
            hipLaunchKernelGGL(k_log_loss, dim3(1), dim3(1), 0, f->st, f->dres, log, int(k));
            TRY(launched());
            f->working_stale = true;
        }
        TF_HIP(hipMemcpyAsync(hlog.data(), log, spe * sizeof(double), hipMemcpyDeviceToHost, f->st));
        TF_HIP(hipStreamSynchronize(f->st));
        double m = 0;
        for (double v : hlog) m += v;
        last = m / double(spe);
        if (cfg->epoch_loss) cfg->epoch_loss[ep] = last;
        if (cfg->progress) cfg->progress(int32_t(ep), last, cfg->progress_user);
        if (!std::isfinite(last)) return fail(TF_ENONFINITE, "training loss is not finite");
    }
    if (cfg->scale_targets) {
        // fold the scale into the projection so the operator predicts the
        // targets themselves; the Adam moments no longer match: reset them
        const int64_t m = NPARAMS - OFF_P2;
        hipLaunchKernelGGL(k_scale, dim3((m + 255) / 256), dim3(256), 0, f->st, f->prm + OFF_P2, m, float(scale));
        TRY(launched());
        TF_HIP(hipMemsetAsync(f->am, 0, NPARAMS * sizeof(float), f->st));
        TF_HIP(hipMemsetAsync(f->av, 0, NPARAMS * sizeof(float), f->st));
        f->adam_t = 0;
        f->working_stale = true;
    }
    TF_HIP(hipStreamSynchronize(f->st));
    if (final_loss) *final_loss = last;
    return TF_OK;
}

tf_status tf_fno_eval(tf_fno* f, const float* params, const float* head_w, const float* targets, int64_t n,
                      double* rel_l2) {
    if (!f || !params || !targets || !rel_l2) return fail(TF_EINVAL, "NULL argument");
    if (f->nb != 1 && !head_w) return fail(TF_EINVAL, "a head of several basis fields needs its weights");
    if (n < 1 || n > (int64_t(1) << 30)) return fail(TF_EINVAL, "need 1 <= n < 2^30");
    TF_HIP(hipSetDevice(f->dev));
    CallBuffers cb(f->st);
    double* res = nullptr;
    TRY(cb.alloc(&res, n));
    f->cur = f->st;
    for (int64_t i0 = 0; i0 < n; i0 += f->maxB) {
        const int nb = int(std::min<int64_t>(f->maxB, n - i0));
        TRY(forward(f, params + i0 * NPAR, f->nb != 1 ? head_w + i0 * f->nb : nullptr, nb, f->out));
        hipLaunchKernelGGL(k_loss_part, dim3(LOSS_CH, nb), dim3(256), 0, f->st, f->out, targets + i0 * OUT_SZ,
                           f->lpart);
        hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(LOSS_THREADS), 0, f->st, f->lpart, LOSS_CH, nb, f->dres,
                           f->dres + 1 + nb);
        TRY(launched());
        TF_HIP(hipMemcpyAsync(res + i0, f->dres + 1 + nb, nb * sizeof(double), hipMemcpyDeviceToDevice, f->st));
    }
    TF_HIP(hipMemcpyAsync(rel_l2, res, n * sizeof(double), hipMemcpyDeviceToHost, f->st));
    TF_HIP(hipStreamSynchronize(f->st));
    return TF_OK;
}

tf_status tf_fno_spectral_forward(tf_fno* f, const float* v, int32_t batch, float* modes) {
    TRY(check_batch(f, batch, nullptr, false));
    if (!v || !modes) return fail(TF_EINVAL, "NULL argument");
    TRY(run(f, g_xcontract(f->fx, v, f->T1, batch), 24 * N, batch * NODE_SZ, batch * X1_SZ));
    TRY(ycontract(f, f->fs, f->T1, f->T2, batch));
    return zcontract(f, f->fs, f->T2, modes, batch);
}

tf_status tf_fno_spectral_inverse(tf_fno* f, const float* modes, int32_t batch, float* u) {
    TRY(check_batch(f, batch, nullptr, false));
    if (!modes || !u) return fail(TF_EINVAL, "NULL argument");
    TRY(zexpand(f, f->gs, modes, f->T2, batch));
    TRY(yexpand(f, f->gs, f->T2, f->T1, batch));
    LineArgs a{f->gx, f->T1, nullptr, f->wb[0], nullptr, nullptr, nullptr, u, 0, 0};
    return lineout<false>(f, a, batch);
}

// Checkpoint: magic, version, parameter count, Adam step, then the fp32
// parameters and (when training) the two Adam moments.
tf_status tf_fno_save(tf_fno* f, const char* path) {
    if (!f || !path) return fail(TF_EINVAL, "NULL argument");
    const int64_t NPARAMS = f->np;
    TF_HIP(hipSetDevice(f->dev));
    std::vector<float> h(NPARAMS);
    FILE* fp = std::fopen(path, "wb");
    if (!fp) return fail(TF_EINVAL, std::string("cannot open ") + path);
    // version 1: the plain transform; version 2 adds the period of the
    // spectral transform as a fifth header word
    const int64_t hdr[5] = {0x4f4e4646554354LL, f->period == N ? 1 : 2, NPARAMS, f->training ? f->adam_t : -1,
                            f->period};
    bool ok = std::fwrite(hdr, sizeof(int64_t), f->period == N ? 4 : 5, fp) == size_t(f->period == N ? 4 : 5);
    const float* srcs[3] = {f->prm, f->am, f->av};
    for (int k = 0; ok && k < (f->training ? 3 : 1); ++k) {
        if (hipMemcpyAsync(h.data(), srcs[k], NPARAMS * sizeof(float), hipMemcpyDeviceToHost, f->st) != hipSuccess ||
            hipStreamSynchronize(f->st) != hipSuccess) {
            std::fclose(fp);
            return fail(TF_EDEVICE, "copy of the parameters failed");
        }
        ok = std::fwrite(h.data(), sizeof(float), NPARAMS, fp) == size_t(NPARAMS);
    }
    ok = (std::fclose(fp) == 0) && ok;
    return ok ? TF_OK : fail(TF_EINVAL, std::string("write failed: ") + path);
}

tf_status tf_fno_load(tf_fno* f, const char* path) {
    if (!f || !path) return fail(TF_EINVAL, "NULL argument");
    const int64_t NPARAMS = f->np;
    TF_HIP(hipSetDevice(f->dev));
    FILE* fp = std::fopen(path, "rb");
    if (!fp) return fail(TF_EINVAL, std::string("cannot open ") + path);
    int64_t hdr[4];
    if (std::fread(hdr, sizeof(hdr), 1, fp) != 1 || hdr[0] != 0x4f4e4646554354LL || (hdr[1] != 1 && hdr[1] != 2) ||
        hdr[2] != NPARAMS) {
        std::fclose(fp);
        return fail(TF_EINVAL, "not a surrogate checkpoint of this architecture");
    }
    int64_t period = N;
    if (hdr[1] == 2 && (std::fread(&period, sizeof(period), 1, fp) != 1 || period < N || period > 4 * N)) {
        std::fclose(fp);
        return fail(TF_EINVAL, "bad period in the surrogate checkpoint");
    }
    std::vector<float> h(NPARAMS);
    float* dsts[3] = {f->prm, f->am, f->av};
    const int nk = (hdr[3] >= 0 && f->training) ? 3 : 1;
    for (int k = 0; k < nk; ++k) {
        if (std::fread(h.data(), sizeof(float), NPARAMS, fp) != size_t(NPARAMS)) {
            std::fclose(fp);
            return fail(TF_EINVAL, "truncated checkpoint");
        }
        hipError_t e = hipMemcpyAsync(dsts[k], h.data(), NPARAMS * sizeof(float), hipMemcpyHostToDevice, f->st);
        if (e == hipSuccess) e = hipStreamSynchronize(f->st);
        if (e != hipSuccess) {
            std::fclose(fp);
            return fail(TF_EDEVICE, std::string("checkpoint upload: ") + hipGetErrorString(e));
        }
    }
    std::fclose(fp);
    if (period != f->period) {
        tf_status st = upload_tables(f, int(period));
        if (st != TF_OK) return st;
    }
    if (f->training) {
        if (nk == 1) {
            TF_HIP(hipMemsetAsync(f->am, 0, NPARAMS * sizeof(float), f->st));
            TF_HIP(hipMemsetAsync(f->av, 0, NPARAMS * sizeof(float), f->st));
        }
        f->adam_t = nk == 3 ? hdr[3] : 0;
    }
    f->working_stale = true;
    TF_HIP(hipStreamSynchronize(f->st));
    return TF_OK;
}

}  // extern "C"
