// cae_mlp.hip -- bfloat16 matrix-core training and inference kernels of the calibration surrogate.
//
// The surrogate is a multilayer perceptron d_in -> H -> H -> d_out with SiLU hidden activations
// that maps agent-population parameters to ensemble statistics.  It is not part of the paper's
// method; it accelerates the parameter sweeps the paper motivates (section IV-J) and the exact
// engine stays its fallback and the reference that measures its error.
//
// Precision: weights, inputs, hidden activations and back-propagated gradients are stored in
// bfloat16 (round to nearest even); every product is accumulated in fp32 on the matrix cores
// (gfx950's v_mfma_f32_32x32x16_bf16 and v_mfma_f32_16x16x32_bf16); biases, pre-activations, outputs, weight
// gradients and the Adam state are fp32.  Parameter layout (row-major, input index first):
//   W1[d_in][H], b1[H], W2[H][H], b2[H], W3[H][d_out], b3[d_out]
// and the bfloat16 weight copies are W1, W2, W3 in the same layouts, back to back, followed by
// W2 transposed (W2T[n][k] = W2[k][n]) for the fused inference kernel, whose matrix-core
// operands want four consecutive input indices per lane.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <mutex>
#include <type_traits>

#include "cae.h"

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f)  // round to nearest even
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u) return (uint16_t)(u >> 16);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// The same rounding in one instruction, for values computed here (a NaN stays a NaN).
__device__ __forceinline__ uint16_t f2bf_hw(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }

__device__ __forceinline__ float dsilu(float z)
{
    const float s = 1.0f / (1.0f + expf(-z));
    return s * (1.0f + z * (1.0f - s));
}

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// Eight bfloat16 (or four floats) at any address of their element's alignment: the caller's
// buffers carry no stronger promise, and gfx950 loads them in one instruction either way.
typedef uint32_t v4u_any __attribute__((ext_vector_type(4), aligned(2), may_alias));
typedef uint32_t v2u_any __attribute__((ext_vector_type(2), aligned(2), may_alias));
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4), may_alias));

__device__ __forceinline__ uint4 ld8u(const uint16_t *p)
{
    const v4u_any v = *reinterpret_cast<const v4u_any *>(p);
    return make_uint4(v[0], v[1], v[2], v[3]);
}

// The same at a uniform base and a 32-bit byte offset per lane (no address arithmetic per load).
__device__ __forceinline__ uint4 ld8u(const uint16_t *base, uint32_t bytes)
{
    return ld8u(reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(base) + bytes));
}

__device__ __forceinline__ uint16_t ld1u(const uint16_t *base, uint32_t bytes)
{
    return *reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(base) + bytes);
}

__device__ __forceinline__ v8bf ld8(const uint16_t *p)  // eight bfloat16, 16-byte aligned
{
    return __builtin_bit_cast(v8bf, *reinterpret_cast<const uint4 *>(p));
}

__device__ __forceinline__ v8bf pack8(const uint16_t (&e)[8])
{
    uint4 u;
    u.x = (uint32_t)e[0] | ((uint32_t)e[1] << 16);
    u.y = (uint32_t)e[2] | ((uint32_t)e[3] << 16);
    u.z = (uint32_t)e[4] | ((uint32_t)e[5] << 16);
    u.w = (uint32_t)e[6] | ((uint32_t)e[7] << 16);
    return __builtin_bit_cast(v8bf, u);
}

// Four bfloat16 of a k-major LDS tile, transposed: within each 16 lanes, lane i addresses row
// i / 4, columns 4 (i % 4) .. + 3 of a 4 x 16 block and receives column i of its four rows.
typedef short v4h __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4h lds_v4h;

__device__ __forceinline__ v8bf ld8_tr(const uint16_t *p, uint32_t ld)  // rows r .. r+3 and r+4 .. r+7
{
    const v4h lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4h *)p);
    const v4h hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4h *)(p + 4u * ld));
    return __builtin_bit_cast(v8bf, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// One matrix-core instruction on an MF x MF tile: 32x32x16 or 16x16x32.  Both add their products
// in increasing k, four at a time, so a chain over k gives the same bits with either (and with
// the half-depth forms); every product that a bfloat16 rounding follows is one such chain.
template <int MF>
struct Mfma;
template <>
struct Mfma<32> {
    typedef v16f acc_t;
    static constexpr uint32_t kDepth = 16, kRegs = 16;
    static __device__ __forceinline__ acc_t mac(v8bf a, v8bf b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ uint32_t row(uint32_t i, uint32_t lane)
    {
        return 8u * (i >> 2) + 4u * (lane >> 5) + (i & 3u);
    }
};
template <>
struct Mfma<16> {
    typedef v4f acc_t;
    static constexpr uint32_t kDepth = 32, kRegs = 4;
    static __device__ __forceinline__ acc_t mac(v8bf a, v8bf b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ uint32_t row(uint32_t i, uint32_t lane) { return 4u * (lane >> 4) + i; }
};

// LDS tiles.  A row-major operand keeps kBK consecutive k per row, padded by 8 elements (rows of
// 144 bytes: the 16-byte fragment reads of a wave spread over the banks).  A k-major operand keeps
// its rows of consecutive columns, padded by 32 elements, so the four rows of a transposing read
// start a quarter of the banks apart.
constexpr uint32_t kBK = 64;
constexpr uint32_t kLdR = kBK + 8u;
constexpr uint32_t kPadK = 32;
// Operand blocks in registers or on their way there (a third measured 5 % slower).
constexpr uint32_t kAhead = 2;

// Fragment of MF rows (or columns) starting at `at`, reduction elements from kk.
template <int MF, bool KMAJOR>
__device__ __forceinline__ v8bf frag(const uint16_t *tile, uint32_t ld, uint32_t at, uint32_t kk, uint32_t lane)
{
    if constexpr (!KMAJOR) {
        return ld8(tile + (at + (lane & (MF - 1u))) * ld + kk + 8u * (lane / MF));
    } else {
        const uint32_t i = lane & 15u, q = lane >> 4;
        const uint32_t kg = MF == 32 ? q >> 1 : q, cg = MF == 32 ? q & 1u : 0u;
        return ld8_tr(tile + (kk + 8u * kg + (i >> 2)) * ld + at + 16u * cg + 4u * (i & 3u), ld);
    }
}

__device__ __forceinline__ uint4 keep(bool in, const uint4 &v)  // v, or zero
{
    return make_uint4(in ? v.x : 0u, in ? v.y : 0u, in ? v.z : 0u, in ? v.w : 0u);
}

// Contiguous ranges of tiles per XCD (workgroups are dealt round-robin over the 8 XCDs, each with
// its own L2): tile index of workgroup `b` of `n`.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t b, uint32_t n)
{
    const uint32_t x = b & 7u, per = n >> 3, rem = n & 7u;
    return x * per + min(x, rem) + (b >> 3);
}

enum Epi : int {
    EPI_HIDDEN = 0,  // z = acc + bias -> Z (f32), O = bf16(silu(z))
    EPI_DSILU = 1,   // O = bf16(acc * silu'(Z))
};

struct LayerArgs {
    const uint16_t *A;   // bfloat16 rows (M x K, contiguous) ...
    const float *Af;     // ... or fp32 rows converted on the way in (K <= 64), and ...
    uint16_t *Acopy;     // ... the bfloat16 copy of them kept for the backward pass, in rows of
    uint32_t ldc;        //     ldc elements (K rounded up to 16), zero past K
    const uint16_t *B;   // row n of K consecutive elements, or (k-major) row k of N
    uint32_t M, N, K;
    const float *bias;   // EPI_HIDDEN
    float *Z;            // EPI_HIDDEN: written; EPI_DSILU: read (M x N)
    uint16_t *O;         // M x N
};

// One layer product of the hidden width, C = A B with a fused epilogue: four waves per workgroup,
// WC of them side by side, with WM x WN output tiles each, operands staged through LDS in blocks of
// 64 of the reduction, the next block's global loads in flight during the current block's products.
//   AF32: A is fp32 and short (the input, or the output gradient): one block.
//   KMAJOR: B is read k-major through transposing LDS reads (W1, W2 forward); otherwise its rows
//   are the reduction (W2 backward), or short rows of any length (W3 backward, AF32).
// Every output is one chain over the reduction in increasing k, whatever the tile.  At 4096 x 1024
// x 1024 the forward product takes 21.5 us and the backward one 20.3 (one wave per 16 x 16 tile
// with two-byte operand loads: 475 and 882 us), of which the products are about half (matrix cores
// busy 8.4e6 of 1.9e7 SIMD cycles); the other half is the exponentials and the stores of the
// epilogue, which the short products (12 and 9 us, from 35 and 20) consist of.
template <int WM, int WN, uint32_t WC, bool AF32, bool KMAJOR, int EPI>
__global__ void __launch_bounds__(256) mlp_layer(const LayerArgs g)
{
    constexpr int MF = WM >= 32 ? 32 : 16;
    constexpr uint32_t MI = WM / MF, NI = WN / MF, BM = 4u / WC * WM, TN = WC * WN;
    constexpr uint32_t BN = TN < 32u ? 32u : TN;  // columns brought to LDS for the tile's TN
    using MM = Mfma<MF>;
    constexpr uint32_t kBufs = AF32 ? 1u : 2u;
    constexpr uint32_t kLdB = KMAJOR ? BN + kPadK : kLdR;
    constexpr uint32_t kTileB = KMAJOR ? kBK * kLdB : BN * kLdR;
    __shared__ __align__(16) uint16_t sA[kBufs * BM * kLdR];
    __shared__ __align__(16) uint16_t sB[kBufs * kTileB];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t wm = wave / WC, wn = wave % WC;
    const uint32_t tn = (g.N + TN - 1u) / TN;
    const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const uint32_t row0 = tile / tn * BM, col0 = tile % tn * TN;

    // 16-byte chunks of each operand block per thread, at 32-bit offsets from the block's uniform
    // base.  Every load is issued without a condition: rows and columns past the end are clamped
    // and reach only outputs that are not stored, a reduction block past the end is the last one
    // again, and what its chunks read past the reduction (the next row; the hidden arrays have
    // kPadRows of slack, W2 is followed by W3 and W2T) is zeroed on its way into LDS.  A masked
    // load would make the compiler drain the loads still in flight.
    constexpr uint32_t CA = BM / 32u, CB = BN / 32u, NB = BN / 8u;
    constexpr uint32_t PD = AF32 ? 1u : kAhead;
    const uint32_t nk = AF32 ? 1u : (g.K + kBK - 1u) / kBK, klast = (nk - 1u) * kBK;
    uint4 sa[PD][CA], sb[PD][CB];
    uint32_t oa[CA], ob[CB], obt[CB];
    const uint32_t ka = 8u * (tid & 7u);  // a row-major chunk's first reduction element in its block
    const uint16_t *Ab = nullptr, *Bb = KMAJOR ? g.B + col0 : g.B + (size_t)col0 * g.K;
    if constexpr (!AF32) {
        Ab = g.A + (size_t)row0 * g.K;
#pragma unroll
        for (uint32_t c = 0; c < CA; ++c) oa[c] = 2u * (min((tid + 256u * c) >> 3, g.M - 1u - row0) * g.K + ka);
    }
#pragma unroll
    for (uint32_t c = 0; c < CB; ++c) {
        const uint32_t e = tid + 256u * c;
        if constexpr (KMAJOR) {  // ob: a whole block, obt: the last one, its rows clamped
            const uint32_t n = min(8u * (e % NB), g.N - 8u - col0), kr = e / NB;
            ob[c] = 2u * (kr * g.N + n);
            obt[c] = 2u * (min(kr, g.K - 1u - klast) * g.N + n);
        } else {
            ob[c] = obt[c] = 2u * (min(e >> 3, g.N - 1u - col0) * g.K + ka);
        }
    }
    auto fetch = [&](uint32_t k0, uint4 (&ra)[CA], uint4 (&rb)[CB]) {
        const uint32_t k = min(k0, klast);
        if constexpr (!AF32) {
#pragma unroll
            for (uint32_t c = 0; c < CA; ++c) ra[c] = ld8u(Ab + k, oa[c]);
        }
        if constexpr (KMAJOR) {
            const bool tail = k + kBK > g.K;
#pragma unroll
            for (uint32_t c = 0; c < CB; ++c) rb[c] = ld8u(Bb + (size_t)k * g.N, tail ? obt[c] : ob[c]);
        } else if constexpr (!AF32) {
#pragma unroll
            for (uint32_t c = 0; c < CB; ++c) rb[c] = ld8u(Bb + k, ob[c]);
        }
    };
    auto store = [&](uint32_t buf, uint32_t k0, const uint4 (&ra)[CA], const uint4 (&rb)[CB], auto whole) {
        constexpr bool kWhole = decltype(whole)::value;
        uint16_t *la = sA + buf * BM * kLdR, *lb = sB + buf * kTileB;
        const bool in = kWhole || k0 + ka < g.K;
        if constexpr (!AF32) {
#pragma unroll
            for (uint32_t c = 0; c < CA; ++c)
                *reinterpret_cast<uint4 *>(la + ((tid + 256u * c) >> 3) * kLdR + ka) = keep(in, ra[c]);
        }
        if constexpr (KMAJOR) {
#pragma unroll
            for (uint32_t c = 0; c < CB; ++c) {
                const uint32_t e = tid + 256u * c, kr = e / NB;
                *reinterpret_cast<uint4 *>(lb + kr * kLdB + 8u * (e % NB)) = keep(kWhole || k0 + kr < g.K, rb[c]);
            }
        } else if constexpr (!AF32) {
#pragma unroll
            for (uint32_t c = 0; c < CB; ++c)
                *reinterpret_cast<uint4 *>(lb + ((tid + 256u * c) >> 3) * kLdR + ka) = keep(in, rb[c]);
        }
    };
    auto stage = [&](uint32_t buf, uint32_t k0, const uint4 (&ra)[CA], const uint4 (&rb)[CB]) {
        if (k0 + kBK <= g.K) store(buf, k0, ra, rb, std::true_type{});
        else store(buf, k0, ra, rb, std::false_type{});
    };

    const uint32_t kpad = (min(g.K, kBK) + MM::kDepth - 1u) / MM::kDepth * MM::kDepth;
#pragma unroll
    for (uint32_t u = 0; u < PD; ++u) fetch(u * kBK, sa[u], sb[u]);
    if constexpr (AF32) {
        // short rows: convert, keep the copy (one column of workgroups), zero the padding; eight
        // loads in flight per thread
        const uint32_t ks = kpad <= 16u ? 4u : (kpad <= 32u ? 5u : 6u), kp = 1u << ks;
        for (uint32_t e0 = tid; e0 < BM << ks; e0 += 2048u) {
            float v[8];
#pragma unroll
            for (uint32_t c = 0; c < 8u; ++c) {
                const uint32_t e = e0 + 256u * c, r = e >> ks, k = e & (kp - 1u);
                v[c] = (e < BM << ks && row0 + r < g.M && k < g.K) ? g.Af[(size_t)(row0 + r) * g.K + k] : 0.f;
            }
#pragma unroll
            for (uint32_t c = 0; c < 8u; ++c) {
                const uint32_t e = e0 + 256u * c, r = e >> ks, k = e & (kp - 1u);
                if (e >= BM << ks) continue;
                const uint16_t b = f2bf(v[c]);
                sA[r * kLdR + k] = b;
                if (col0 == 0u && row0 + r < g.M && k < g.ldc) g.Acopy[(size_t)(row0 + r) * g.ldc + k] = b;
            }
        }
        if constexpr (!KMAJOR) {
            for (uint32_t e = tid; e < BN << ks; e += 256u) {
                const uint32_t r = e >> ks, k = e & (kp - 1u);
                sB[r * kLdR + k] = (col0 + r < g.N && k < g.K) ? g.B[(size_t)(col0 + r) * g.K + k] : (uint16_t)0;
            }
        }
    }
    stage(0, 0u, sa[0], sb[0]);
    __syncthreads();

    typename MM::acc_t acc[MI][NI];
#pragma unroll
    for (uint32_t i = 0; i < MI; ++i)
#pragma unroll
        for (uint32_t j = 0; j < NI; ++j)
#pragma unroll
            for (uint32_t t = 0; t < MM::kRegs; ++t) acc[i][j][t] = 0.f;
    auto step = [&](const uint16_t *pa, const uint16_t *pb, uint32_t kk) {
        v8bf fa[MI], fb[NI];
#pragma unroll
        for (uint32_t i = 0; i < MI; ++i) fa[i] = frag<MF, false>(pa, kLdR, wm * WM + i * MF, kk, lane);
#pragma unroll
        for (uint32_t j = 0; j < NI; ++j) fb[j] = frag<MF, KMAJOR>(pb, kLdB, wn * WN + j * MF, kk, lane);
#pragma unroll
        for (uint32_t i = 0; i < MI; ++i)
#pragma unroll
            for (uint32_t j = 0; j < NI; ++j) acc[i][j] = MM::mac(fa[i], fb[j], acc[i][j]);
    };
    if constexpr (AF32) {
        for (uint32_t kk = 0; kk < kpad; kk += MM::kDepth) step(sA, sB, kk);
    } else {
        // block t is computed from LDS while block t + 1 waits in registers and the loads of the
        // PD - 1 blocks after it are in flight (blocks past the reduction are zero)
        for (uint32_t t0 = 0; t0 < nk; t0 += PD) {
#pragma unroll
            for (uint32_t u = 0; u < PD; ++u) {
                const uint32_t t = t0 + u, buf = PD % 2u ? t & 1u : u & 1u;
                fetch((t + PD) * kBK, sa[u], sb[u]);
                __builtin_amdgcn_sched_barrier(0);  // the loads leave before the products
#pragma unroll
                for (uint32_t kk = 0; kk < kBK; kk += MM::kDepth)
                    step(sA + buf * BM * kLdR, sB + buf * kTileB, kk);
                stage(buf ^ 1u, (t + 1u) * kBK, sa[(u + 1u) % PD], sb[(u + 1u) % PD]);
                __syncthreads();
            }
        }
    }

    // epilogue: rows and columns checked only in the tiles at the edges (a branch per element makes
    // the compiler wait for every store before the next element)
    float bn[NI];
#pragma unroll
    for (uint32_t j = 0; j < NI; ++j) {
        bn[j] = 0.f;
        if constexpr (EPI == EPI_HIDDEN) bn[j] = g.bias[min(col0 + wn * WN + j * MF + (lane & (MF - 1u)), g.N - 1u)];
    }
    float *Zt = g.Z + (size_t)row0 * g.N + col0;
    uint16_t *Ot = g.O + (size_t)row0 * g.N + col0;
    auto finish = [&](auto whole) {
        constexpr bool kWhole = decltype(whole)::value;
        const uint32_t mr = g.M - row0, nr = g.N - col0;  // rows and columns from the tile's origin
#pragma unroll
        for (uint32_t j = 0; j < NI; ++j) {
            const uint32_t n = wn * WN + j * MF + (lane & (MF - 1u));
            if (!kWhole && n >= nr) continue;
#pragma unroll
            for (uint32_t i = 0; i < MI; ++i) {
                const uint32_t m0 = wm * WM + i * MF;
                float z[MM::kRegs];
                if constexpr (EPI == EPI_DSILU) {  // every load before the first use
#pragma unroll
                    for (uint32_t t = 0; t < MM::kRegs; ++t) {
                        const uint32_t m = m0 + MM::row(t, lane);
                        z[t] = Zt[(kWhole ? m : min(m, mr - 1u)) * g.N + n];
                    }
                }
#pragma unroll
                for (uint32_t t = 0; t < MM::kRegs; ++t) {
                    const uint32_t m = m0 + MM::row(t, lane);
                    if (!kWhole && m >= mr) continue;
                    const uint32_t o = m * g.N + n;
                    if constexpr (EPI == EPI_HIDDEN) {
                        const float zv = acc[i][j][t] + bn[j];
                        Zt[o] = zv;
                        Ot[o] = f2bf_hw(silu(zv));
                    } else {
                        Ot[o] = f2bf_hw(acc[i][j][t] * dsilu(z[t]));
                    }
                }
            }
        }
    };
    if (row0 + BM <= g.M && col0 + TN <= g.N) finish(std::true_type{});
    else finish(std::false_type{});
}

// Output layer y = h W3 + b3: NB blocks of 16 rows per workgroup.  All four waves bring the rows and
// W3 (rows of 16 columns, read transposed) into LDS, one wave per block runs the chain over H.  At
// H = 16 the chain is one step and the workgroups' fixed costs are the time: 65536 rows take 6.4 us
// with one block, 4.6 with four (wider layers gain less or lose).
template <uint32_t NB>
__global__ void __launch_bounds__(256) mlp_out(const uint16_t *h, const uint16_t *W3, const float *b3, float *y,
                                               uint32_t M, uint32_t H, uint32_t dout)
{
    extern __shared__ __align__(16) uint16_t olds[];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, r = lane & 15u, gq = lane >> 4;
    const uint32_t Hp = (H + 31u) & ~31u, ldh = Hp + 8u;
    uint16_t *hs = olds, *w3s = olds + 16u * NB * ldh;  // [16 NB][ldh], [Hp][16]
    const uint32_t row0 = blockIdx.x * 16u * NB, hc = Hp / 8u;
    for (uint32_t e0 = tid; e0 < 16u * NB * hc; e0 += 2048u) {
        uint4 v[8];
#pragma unroll
        for (uint32_t c = 0; c < 8u; ++c) {
            const uint32_t e = e0 + 256u * c, rr = e / hc, k = 8u * (e % hc);
            v[c] = ld8u(h + (size_t)min(row0 + min(rr, 16u * NB - 1u), M - 1u) * H + min(k, H - 8u));
        }
#pragma unroll
        for (uint32_t c = 0; c < 8u; ++c) {
            const uint32_t e = e0 + 256u * c;
            if (e >= 16u * NB * hc) continue;
            *reinterpret_cast<uint4 *>(hs + e / hc * ldh + 8u * (e % hc)) = keep(8u * (e % hc) < H, v[c]);
        }
    }
    if (dout == 16u) {
        for (uint32_t e = tid; e < Hp * 2u; e += 256u)
            *reinterpret_cast<uint4 *>(w3s + 8u * e) = e < H * 2u ? ld8u(W3 + 8u * e) : make_uint4(0, 0, 0, 0);
    } else {
        for (uint32_t e = tid; e < Hp * 16u; e += 256u) {
            const uint32_t k = e >> 4, c = e & 15u;
            w3s[e] = (k < H && c < dout) ? W3[(size_t)k * dout + c] : (uint16_t)0;
        }
    }
    __syncthreads();
    if (tid >= 64u * NB) return;
    const uint32_t at = 16u * (tid >> 6), wrow = row0 + at;  // the wave's rows
    v4f acc = {0.f, 0.f, 0.f, 0.f};
    for (uint32_t k0 = 0; k0 < Hp; k0 += 32u)
        acc = Mfma<16>::mac(frag<16, false>(hs, ldh, at, k0, lane), frag<16, true>(w3s, 16u, 0u, k0, lane), acc);
    if (r < dout) {
#pragma unroll
        for (uint32_t t = 0; t < 4u; ++t)
            if (wrow + 4u * gq + t < M) y[(size_t)(wrow + 4u * gq + t) * dout + r] = acc[t] + b3[r];
    }
}

// Weight gradients [A; 1]^T B over the batch (A: a layer's input, B: its output gradient, both
// batch-major, so both operands are k-major LDS tiles read transposed; the row of ones gives the
// bias gradient).  The batch is cut into chunks of at most 256 rows (more beyond 16384 rows): each
// chunk is one matrix-core chain and the chunks' results are added in chunk order, so a gradient
// does not depend on how the chunks are spread over workgroups.  One launch holds the tiles of
// all three gradients.  A workgroup either takes one chunk and leaves its result for grad_reduce,
// or (parts = 1) takes every chunk of its tile and adds them in registers.
// At a batch of 4096 and H = 1024 the launch takes 45 us (two-byte strided loads, three products
// and three sums in six launches: 155 us): one workgroup of four waves per CU, so the time is
// that of 64 blocks' chains of LDS write, barrier, transposing reads and matrix-core steps.
struct GradArgs {
    const uint16_t *x, *h1, *h2, *dy, *dz2, *dz1;
    uint32_t batch, din, H, dout;
    uint32_t parts, chunk;
    uint32_t tiles1, tiles2, tiles3;  // tiles of W1, W2, W3
    float *o1, *o2, *o3;              // part 0 of each gradient, its bias row after its last row
    size_t stride;                    // floats between parts
};

// One BM x BN tile by four waves (WR along M), wave tiles of 32 x 32 products.  lda, ldb: the
// operands' row lengths, multiples of 16 (the rows are zero past M and N).
template <uint32_t BM, uint32_t BN, uint32_t WR>
__device__ __forceinline__ void grad_tile(uint16_t *lds, const uint16_t *A, const uint16_t *B, uint32_t lda,
                                          uint32_t ldb, uint32_t M, uint32_t N, uint32_t m0, uint32_t n0,
                                          uint32_t kbeg, uint32_t kend, uint32_t chunk, float *out)
{
    constexpr uint32_t WC = 4u / WR, MI = BM / WR / 32u, NI = BN / WC / 32u;
    constexpr uint32_t kLdA = BM + kPadK, kLdB = BN + kPadK, kTA = kBK * kLdA, kTB = kBK * kLdB;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6)), wm = wave / WC, wn = wave % WC;
    uint16_t *sA = lds, *sB = lds + 2u * kTA;
    constexpr uint32_t CA = kBK * BM / 8u / 256u, CB = kBK * BN / 8u / 256u;
    const bool bias = m0 == 0u && wm == 0u;  // this wave also forms the row of ones of its columns
    // blocks of 64 batch rows, nb to a chunk; as in mlp_layer, loads are not masked (the arrays have
    // kPadRows rows of slack), and rows past the chunk's end (ce) are zeroed on their way into LDS
    const uint32_t nb = (chunk + kBK - 1u) / kBK;
    struct Block {
        uint32_t c0, j;  // the chunk's first row, the block in it
    };
    auto next = [&](Block b) { return b.j + 1u < nb ? Block{b.c0, b.j + 1u} : Block{b.c0 + chunk, 0u}; };
    auto first = [&](Block b) { return b.c0 + b.j * kBK; };
    auto end = [&](Block b) { return (uint32_t)min(kend, b.c0 + chunk); };
    uint4 sa[kAhead][CA], sb[kAhead][CB];
    const uint32_t ra0 = tid / (BM / 8u), rb0 = tid / (BN / 8u);  // rows of the thread's first chunks
    constexpr uint32_t kStepA = 256u / (BM / 8u), kStepB = 256u / (BN / 8u);
    const uint32_t ca = 8u * (tid % (BM / 8u)), cb = 8u * (tid % (BN / 8u));
    const uint32_t oa = 2u * (ra0 * lda + min(ca, lda - 8u - m0)), ob = 2u * (rb0 * ldb + min(cb, ldb - 8u - n0));
    const uint32_t klast = kbeg + (kend - 1u - kbeg) / chunk * chunk;  // the last chunk's first row ...
    const uint32_t kclamp = klast + (kend - 1u - klast) / kBK * kBK;   // ... and its last block's
    auto fetch = [&](Block b, uint4 (&ra)[CA], uint4 (&rb)[CB]) {
        const uint32_t k0 = min(first(b), kclamp);
        const uint16_t *pa = A + (size_t)k0 * lda + m0, *pb = B + (size_t)k0 * ldb + n0;
#pragma unroll
        for (uint32_t c = 0; c < CA; ++c) ra[c] = ld8u(pa + (size_t)(kStepA * c) * lda, oa);
#pragma unroll
        for (uint32_t c = 0; c < CB; ++c) rb[c] = ld8u(pb + (size_t)(kStepB * c) * ldb, ob);
    };
    auto store = [&](uint32_t buf, uint32_t k0, uint32_t ce, const uint4 (&ra)[CA], const uint4 (&rb)[CB], auto whole) {
        constexpr bool kWhole = decltype(whole)::value;
        uint16_t *la = sA + buf * kTA + ra0 * kLdA + ca, *lb = sB + buf * kTB + rb0 * kLdB + cb;
#pragma unroll
        for (uint32_t c = 0; c < CA; ++c)
            *reinterpret_cast<uint4 *>(la + kStepA * c * kLdA) = keep(kWhole || k0 + ra0 + kStepA * c < ce, ra[c]);
#pragma unroll
        for (uint32_t c = 0; c < CB; ++c)
            *reinterpret_cast<uint4 *>(lb + kStepB * c * kLdB) = keep(kWhole || k0 + rb0 + kStepB * c < ce, rb[c]);
    };
    auto stage = [&](uint32_t buf, Block b, const uint4 (&ra)[CA], const uint4 (&rb)[CB]) {
        const uint32_t k0 = first(b), ce = end(b);
        if (k0 + kBK <= ce) store(buf, k0, ce, ra, rb, std::true_type{});
        else store(buf, k0, ce, ra, rb, std::false_type{});
    };
    const v16f zero = {};
    v16f acc[MI][NI], tot[MI][NI], accb[NI], totb[NI];
#pragma unroll
    for (uint32_t j = 0; j < NI; ++j) {
        accb[j] = totb[j] = zero;
#pragma unroll
        for (uint32_t i = 0; i < MI; ++i) acc[i][j] = tot[i][j] = zero;
    }
    v8bf ones;
#pragma unroll
    for (uint32_t t = 0; t < 8u; ++t) ones[t] = (__bf16)1.0f;
    Block cur{kbeg, 0u}, ahead = cur;  // the block computed, the next to fetch
#pragma unroll
    for (uint32_t u = 0; u < kAhead; ++u) {
        fetch(ahead, sa[u], sb[u]);
        ahead = next(ahead);
    }
    stage(0, cur, sa[0], sb[0]);
    __syncthreads();
    uint32_t buf = 0;
    while (first(cur) < kend) {  // (kAhead blocks a turn; those past the end are zero)
#pragma unroll
        for (uint32_t u = 0; u < kAhead; ++u) {
            fetch(ahead, sa[u], sb[u]);
            ahead = next(ahead);
            __builtin_amdgcn_sched_barrier(0);
            const uint16_t *ta = sA + buf * kTA, *tb = sB + buf * kTB;
            constexpr uint32_t NK = kBK / 16u;
            v8bf fa[NK][MI], fb[NK][NI];
#pragma unroll
            for (uint32_t q = 0; q < NK; ++q) {
#pragma unroll
                for (uint32_t i = 0; i < MI; ++i) fa[q][i] = frag<32, true>(ta, kLdA, (wm * MI + i) * 32u, 16u * q, lane);
#pragma unroll
                for (uint32_t j = 0; j < NI; ++j) fb[q][j] = frag<32, true>(tb, kLdB, (wn * NI + j) * 32u, 16u * q, lane);
            }
#pragma unroll
            for (uint32_t q = 0; q < NK; ++q)
#pragma unroll
                for (uint32_t i = 0; i < MI; ++i)
#pragma unroll
                    for (uint32_t j = 0; j < NI; ++j) acc[i][j] = Mfma<32>::mac(fa[q][i], fb[q][j], acc[i][j]);
            if (bias) {
#pragma unroll
                for (uint32_t q = 0; q < NK; ++q)
#pragma unroll
                    for (uint32_t j = 0; j < NI; ++j) accb[j] = Mfma<32>::mac(ones, fb[q][j], accb[j]);
            }
            const Block after = next(cur);
            if (after.j == 0u) {  // the chunk's last block
#pragma unroll
                for (uint32_t j = 0; j < NI; ++j) {
                    totb[j] += accb[j];
                    accb[j] = zero;
#pragma unroll
                    for (uint32_t i = 0; i < MI; ++i) {
                        tot[i][j] += acc[i][j];
                        acc[i][j] = zero;
                    }
                }
            }
            stage(buf ^ 1u, after, sa[(u + 1u) % kAhead], sb[(u + 1u) % kAhead]);
            __syncthreads();
            buf ^= 1u;
            cur = after;
        }
    }
#pragma unroll
    for (uint32_t j = 0; j < NI; ++j) {
        const uint32_t n = n0 + (wn * NI + j) * 32u + (lane & 31u);
        if (n >= N) continue;
#pragma unroll
        for (uint32_t i = 0; i < MI; ++i)
#pragma unroll
            for (uint32_t t = 0; t < 16u; ++t) {
                const uint32_t m = m0 + (wm * MI + i) * 32u + Mfma<32>::row(t, lane);
                if (m < M) out[(size_t)m * N + n] = tot[i][j][t] + acc[i][j][t];
            }
        if (bias && lane < 32u) out[(size_t)M * N + n] = totb[j][0] + accb[j][0];
    }
}

__global__ void __launch_bounds__(256) mlp_grad(const GradArgs g)
{
    constexpr uint32_t kLds2 = 4u * kBK * (64u + kPadK), kLds3 = 2u * kBK * (128u + kPadK + 32u + kPadK);
    __shared__ __align__(16) uint16_t lds[kLds2 > kLds3 ? kLds2 : kLds3];
    const uint32_t ntiles = g.tiles1 + g.tiles2 + g.tiles3;
    const uint32_t job = xcd_tile(blockIdx.x, gridDim.x);
    const uint32_t part = job / ntiles;
    uint32_t tile = job % ntiles;
    const uint32_t kbeg = part * g.chunk, kend = g.parts > 1u ? min(g.batch, kbeg + g.chunk) : g.batch;
    const size_t off = part * g.stride;
    if (tile < g.tiles2) {
        const uint32_t tn = (g.H + 63u) / 64u;
        grad_tile<64, 64, 2>(lds, g.h1, g.dz2, g.H, g.H, g.H, g.H, tile / tn * 64u, tile % tn * 64u, kbeg, kend,
                                         g.chunk, g.o2 + off);
    } else if ((tile -= g.tiles2) < g.tiles1) {
        grad_tile<64, 64, 2>(lds, g.x, g.dz1, (g.din + 15u) & ~15u, g.H, g.din, g.H, 0u, tile * 64u, kbeg, kend, g.chunk,
                                          g.o1 + off);
    } else {
        tile -= g.tiles1;
        grad_tile<128, 32, 4>(lds, g.h2, g.dy, g.H, 16u, g.H, g.dout, tile * 128u, 0u, kbeg, kend, g.chunk,
                                           g.o3 + off);
    }
}

// The chunks' results added in chunk order (n parameters, the parameter layout).
__global__ void __launch_bounds__(256) grad_reduce(const float *part, uint32_t parts, size_t stride, uint64_t n,
                                                   float *grads)
{
    const uint64_t e = ((uint64_t)blockIdx.x * 256u + threadIdx.x) * 4u;
    if (e >= n) return;
    if (e + 4u <= n) {
        v4f s = *reinterpret_cast<const v4f_any *>(part + e);
#pragma unroll 4
        for (uint32_t p = 1; p < parts; ++p) s += *reinterpret_cast<const v4f_any *>(part + p * stride + e);
        *reinterpret_cast<v4f_any *>(grads + e) = s;
    } else {
        for (uint64_t i = e; i < n; ++i) {
            float s = part[i];
            for (uint32_t p = 1; p < parts; ++p) s += part[p * stride + i];
            grads[i] = s;
        }
    }
}

// Mean loss over n values and its gradient, r = y - t:
//   kind 0 (squared error): loss = mean r^2,                         dy = 2 r / n
//   kind 1 (Huber, delta):  loss = mean(r^2/2 if |r| <= delta else delta (|r| - delta/2)),
//                           dy = clamp(r, -delta, delta) / n
// Workgroup 0 sums the loss, one strided chain per thread and then a tree over the threads (a
// fixed order whatever the grid), kLossAhead of a chain's values in flight; the other workgroups write
// the gradient, or workgroup 0 does when it is alone.
constexpr uint32_t kLossThreads = 1024, kLossAhead = 32;

__global__ void __launch_bounds__(kLossThreads) loss_grad(const float *y, const float *t, float *dy, float *loss,
                                                          uint32_t n, int kind, float delta)
{
    __shared__ float part[kLossThreads];
    const float inv = 1.0f / (float)n;
    auto grad = [&](float d) { return kind == 0 ? 2.0f * d * inv : fminf(fmaxf(d, -delta), delta) * inv; };
    if (blockIdx.x > 0u) {
        const uint64_t step = (uint64_t)(gridDim.x - 1u) * kLossThreads;
        for (uint64_t i = (uint64_t)(blockIdx.x - 1u) * kLossThreads + threadIdx.x; i < n; i += step)
            dy[i] = grad(y[i] - t[i]);
        return;
    }
    const bool alone = gridDim.x == 1u;
    float s = 0.f;
    for (uint64_t i0 = threadIdx.x; i0 < n; i0 += (uint64_t)kLossAhead * kLossThreads) {
        float d[kLossAhead];
#pragma unroll
        for (uint32_t u = 0; u < kLossAhead; ++u) {
            const uint64_t i = i0 + u * kLossThreads;
            const uint64_t c = i < n ? i : n - 1u;
            d[u] = y[c] - t[c];
        }
#pragma unroll
        for (uint32_t u = 0; u < kLossAhead; ++u) {
            const uint64_t i = i0 + u * kLossThreads;
            if (i >= n) continue;
            if (alone) dy[i] = grad(d[u]);
            const float a = fabsf(d[u]);
            s += kind == 0 ? d[u] * d[u] : (a <= delta ? 0.5f * d[u] * d[u] : delta * (a - 0.5f * delta));
        }
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (uint32_t w = kLossThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = part[0] / (float)n;
}

struct Layout {
    uint64_t w1, b1, w2, b2, w3, b3, P;  // param offsets
    uint64_t w2t;                        // bf16 offset of the transposed W2 copy
    uint64_t W;                          // bf16 weight count
};

__host__ __device__ inline Layout layout(uint32_t din, uint32_t H, uint32_t dout)
{
    Layout l;
    l.w1 = 0;
    l.b1 = l.w1 + (uint64_t)din * H;
    l.w2 = l.b1 + H;
    l.b2 = l.w2 + (uint64_t)H * H;
    l.w3 = l.b2 + H;
    l.b3 = l.w3 + (uint64_t)H * dout;
    l.P = l.b3 + dout;
    l.w2t = (uint64_t)din * H + (uint64_t)H * H + (uint64_t)H * dout;
    l.W = l.w2t + (uint64_t)H * H;
    return l;
}

// Adam (Kingma and Ba 2015, algorithm 1) on the fp32 parameters; weights also refresh their
// bfloat16 copies.  c1 = 1 - beta1^t, c2 = 1 - beta2^t; update 0 only rewrites the copies.
struct AdamArgs {
    float *p;
    const float *g;
    float *m, *v;
    uint16_t *wb;
    Layout l;
    uint32_t H, tiles;  // tiles of 64 along a side of W2
    float lr, beta1, beta2, eps, c1, c2;
    int update;
};

__device__ __forceinline__ float adam_value(const AdamArgs &a, float p, float g, float &m, float &v)
{
    m = a.beta1 * m + (1.0f - a.beta1) * g;
    v = a.beta2 * v + (1.0f - a.beta2) * g * g;
    return p - a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
}

// The first tiles^2 workgroups each take 64 x 64 of W2 (four parameters per access; the transposed
// copy goes through LDS so that both copies are written in rows), the others the remaining
// parameters one by one.  Bound by the 28 bytes per parameter it reads and writes.
__global__ void __launch_bounds__(256) adam_step(const AdamArgs a)
{
    constexpr uint32_t kLd = 72;
    __shared__ __align__(16) uint16_t t[64 * kLd];
    const uint32_t tid = threadIdx.x, H = a.H;
    if (blockIdx.x < a.tiles * a.tiles) {
        const uint32_t k0 = blockIdx.x / a.tiles * 64u, n0 = blockIdx.x % a.tiles * 64u;
        const uint32_t n = n0 + 4u * (tid & 15u), r = tid >> 4;
        v4f p[4], g[4], m[4], v[4];
#pragma unroll
        for (uint32_t j = 0; j < 4u; ++j) {
            const uint32_t k = k0 + r + 16u * j;
            if (k < H && n < H) {  // H is a multiple of 16
                const size_t i = a.l.w2 + (size_t)k * H + n;
                p[j] = *reinterpret_cast<const v4f_any *>(a.p + i);
                if (a.update) {
                    g[j] = *reinterpret_cast<const v4f_any *>(a.g + i);
                    m[j] = *reinterpret_cast<const v4f_any *>(a.m + i);
                    v[j] = *reinterpret_cast<const v4f_any *>(a.v + i);
                }
            }
        }
#pragma unroll
        for (uint32_t j = 0; j < 4u; ++j) {
            const uint32_t k = k0 + r + 16u * j;
            if (k < H && n < H) {
                const size_t i = a.l.w2 + (size_t)k * H + n;
                if (a.update) {
#pragma unroll
                    for (uint32_t c = 0; c < 4u; ++c) {
                        float mc = m[j][c], vc = v[j][c];
                        p[j][c] = adam_value(a, p[j][c], g[j][c], mc, vc);
                        m[j][c] = mc;
                        v[j][c] = vc;
                    }
                    *reinterpret_cast<v4f_any *>(a.m + i) = m[j];
                    *reinterpret_cast<v4f_any *>(a.v + i) = v[j];
                    *reinterpret_cast<v4f_any *>(a.p + i) = p[j];
                }
                uint16_t b[4];
#pragma unroll
                for (uint32_t c = 0; c < 4u; ++c) {
                    b[c] = f2bf(p[j][c]);
                    t[(4u * (tid & 15u) + c) * kLd + r + 16u * j] = b[c];
                }
                *reinterpret_cast<v2u_any *>(a.wb + a.l.b1 + (size_t)k * H + n) =
                    v2u_any{(uint32_t)b[0] | ((uint32_t)b[1] << 16), (uint32_t)b[2] | ((uint32_t)b[3] << 16)};
            }
        }
        __syncthreads();
#pragma unroll
        for (uint32_t j = 0; j < 2u; ++j) {  // W2T[n][k]: rows of 64, eight per access
            const uint32_t e = tid + 256u * j, nl = e >> 3, kl = 8u * (e & 7u);
            if (n0 + nl < H && k0 + kl < H) {
                const uint4 w = *reinterpret_cast<const uint4 *>(t + nl * kLd + kl);
                *reinterpret_cast<v4u_any *>(a.wb + a.l.w2t + (size_t)(n0 + nl) * H + k0 + kl) = v4u_any{w.x, w.y, w.z, w.w};
            }
        }
        return;
    }
    const uint64_t e = (uint64_t)(blockIdx.x - a.tiles * a.tiles) * 256u + tid;
    const uint64_t i = e < a.l.w2 ? e : e + (a.l.b2 - a.l.w2);  // W1 b1, then b2 W3 b3
    if (i >= a.l.P) return;
    float pi = a.p[i];
    if (a.update) {
        float mi = a.m[i], vi = a.v[i];
        pi = adam_value(a, pi, a.g[i], mi, vi);
        a.m[i] = mi;
        a.v[i] = vi;
        a.p[i] = pi;
    }
    if (i < a.l.b1) a.wb[i] = f2bf(pi);
    else if (i >= a.l.w3 && i < a.l.b3) a.wb[a.l.b1 + (a.l.b2 - a.l.w2) + (i - a.l.w3)] = f2bf(pi);
}

// Inference of the whole network in one launch: a workgroup of 16 waves keeps its weights over
// all of its tiles of rows.  A wave owns NT 16-column tiles of each hidden layer, over RT blocks
// of 16 rows; narrow layers (H <= 128) split the waves over 2 to 16 groups of rows.  With RES
// (H <= 256) the wave's W2 fragments stay in registers, otherwise they come from L2 for every
// tile, whose RT = 4 blocks of rows share them; both steps of W1 stay in registers (fetched again
// for every tile, the second one of wide inputs made d_in = 40, H = 304, 65536 rows 103 us, 65
// now).  SKIP: a wave does nothing for tiles of columns that a layer does not have; without it the
// last tile's work is repeated (H = 272, 65536 rows: 106 us, 54 with it; H = 16, 300000 rows, all
// waves on rows: 38 and 17).  The input of the next tile is fetched under the current one, both
// hidden activations go through LDS, W3 sits in LDS as rows of 16 columns read transposed; the
// output layer of 16 rows is one wave's chain, under the others' next tile.
// Same rounding points and the same chains over k as mlp_layer and mlp_out, so the outputs equal
// cae_mlp_forward's bit for bit.
// H = 256: 6553 rows take 12.1 us, 65536 rows 39.6, one row 9.3 (32-row tiles on four waves that
// streamed W2 from L2 for each: 21.5, 82.3 and 20.1); H = 272, 65536 rows: 54 (70); H = 496: 110
// (205); H = 16: 8.2 (8.1), 300000 rows 17 (25).  A tile of 32 rows costs 2 us, of which the
// exponentials' instructions are 1.6; the set-up is instructions and two memory latencies, about
// 7 us.
constexpr uint32_t kPredMaxH = 496;
constexpr uint32_t kPredWaves = 16, kPredThreads = 64 * kPredWaves;

struct PredArgs {
    const float *x;
    float *y;
    uint32_t N, din, H, dout;
    uint32_t cols_log2;  // log2 of the waves along the columns
    const uint16_t *W1, *W2T, *W3;
    const float *b1, *b2, *b3;
};

template <uint32_t NT, bool RES, uint32_t RT, bool SKIP, uint32_t XN>
__global__ void __launch_bounds__(kPredThreads) mlp_predict(const PredArgs a)
{
    extern __shared__ __align__(16) uint16_t plds[];
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint32_t r = lane & 15u, g = lane >> 4;
    const uint32_t H = a.H, Hp = (H + 31u) & ~31u, ldh = Hp + 8u, ct = H / 16u;
    const uint32_t Kx = (a.din + 31u) & ~31u, ldx = Kx + 8u;
    const uint32_t wcols = 1u << a.cols_log2, groups = kPredWaves >> a.cols_log2;
    // (with tiles missing, the waves of one column tile are consecutive: they lie on different SIMDs)
    const uint32_t wc = SKIP ? wave / groups : wave & (wcols - 1u), rg = SKIP ? wave & (groups - 1u) : wave >> a.cols_log2;
    const uint32_t rows = 16u * RT * groups;  // rows of a tile
    const uint32_t mine = wc >= ct ? 0u : min((ct - wc + wcols - 1u) >> a.cols_log2, NT);  // the wave's tiles per layer
    // [rows][ldh] twice, the input [rows][ldx] twice, [Hp][16]
    uint16_t *h1 = plds, *h2 = h1 + rows * ldh, *xs = h2 + rows * ldh, *w3s = xs + 2u * rows * ldx;
    constexpr uint32_t K2 = 8;  // steps of 32 over H <= 256
    const uint32_t tiles = (a.N + rows - 1u) / rows;

    // Every wave of the CU issues the set-up once (about 7 ns per instruction), so it is kept short:
    // 32-bit offsets from uniform bases, no division per element.
    // The input tile is contiguous: at most XN values per thread, thread tid + 1024 i.
    const uint32_t xcount = rows * a.din;
    float xv[XN];
    uint32_t xo[XN];  // where they go in the LDS tile
    auto load_x = [&](uint32_t tile) {
        const uint64_t first = (uint64_t)tile * xcount;
        const float *base = a.x + first;
        const uint64_t left = (uint64_t)a.N * a.din - first;  // >= 1
        const uint32_t last = left > xcount ? xcount - 1u : (uint32_t)left - 1u;
#pragma unroll
        for (uint32_t i = 0; i < XN; ++i)
            if (kPredThreads * i < xcount) xv[i] = base[min(tid + kPredThreads * i, last)];
    };
    auto store_x = [&](uint16_t *to) {
#pragma unroll
        for (uint32_t i = 0; i < XN; ++i)
            if (kPredThreads * i < xcount && tid + kPredThreads * i < xcount) to[xo[i]] = f2bf(xv[i]);
    };
    load_x(blockIdx.x);
    // the wave's weights (W1's rows past the input and W2T's past a ragged H are masked; W1 is
    // followed by W2 and W2T, so up to 64 of its rows may be read)
    v8bf w2[NT][RES ? K2 : 1];
    float b1[NT], b2[NT];
    const uint32_t klim = H == Hp ? 0xFFFFFFFFu : H - 8u;
#pragma unroll
    for (uint32_t j = 0; j < NT; ++j) {
        const uint32_t n = min(16u * (wc + wcols * j), H - 16u) + r;  // a missing tile repeats the last
        b1[j] = a.b1[n];
        b2[j] = a.b2[n];
        if constexpr (RES) {
#pragma unroll
            for (uint32_t u = 0; u < K2; ++u)
                if (32u * u < H) w2[j][u] = __builtin_bit_cast(v8bf, ld8u(a.W2T, 2u * (n * H + min(32u * u + 8u * g, klim))));
        }
    }
    auto load_w1 = [&](uint32_t j, uint32_t k0) {
        const uint32_t n = min(16u * (wc + wcols * j), H - 16u) + r, k = k0 + 8u * g;
        const uint32_t off = 2u * (k * H + n);
        uint16_t e[8];
#pragma unroll
        for (uint32_t t = 0; t < 8u; ++t) e[t] = ld1u(a.W1 + (size_t)t * H, off);
#pragma unroll
        for (uint32_t t = 0; t < 8u; ++t) e[t] = k + t < a.din ? e[t] : (uint16_t)0;
        return pack8(e);
    };
    v8bf w1[NT], w1b[NT];  // both steps of W1 (the second one of inputs wider than 32)
#pragma unroll
    for (uint32_t j = 0; j < NT; ++j) w1[j] = load_w1(j, 0u);
    if (Kx > 32u) {
#pragma unroll
        for (uint32_t j = 0; j < NT; ++j) w1b[j] = load_w1(j, 32u);
    }
    const float b3 = a.b3[min(r, a.dout - 1u)];
    {
        const uint32_t k = tid >> 4, c = tid & 15u, off = 2u * (k * a.dout + min(c, a.dout - 1u));
        for (uint32_t k0 = 0; k0 < Hp; k0 += 64u) {  // 64 rows of W3 per turn
            const uint16_t w = ld1u(a.W3 + (size_t)min(k0, H - 16u) * a.dout, k0 + k < H ? off : 0u);
            if (k0 + k < Hp) w3s[(k0 + k) * 16u + c] = (k0 + k < H && c < a.dout) ? w : (uint16_t)0;
        }
    }
#pragma unroll
    for (uint32_t i = 0; i < XN; ++i)
        if (kPredThreads * i < xcount) {
            const uint32_t e = tid + kPredThreads * i, row = e / a.din;
            xo[i] = row * ldx + (e - row * a.din);
        }
    if (RES && H != Hp) {  // the last step's second half lies past H
#pragma unroll
        for (uint32_t j = 0; j < NT; ++j)
#pragma unroll
            for (uint32_t u = 0; u < (RES ? K2 : 1u); ++u)
                w2[j][u] = __builtin_bit_cast(v8bf, keep(32u * u + 8u * g < H, __builtin_bit_cast(uint4, w2[j][u])));
    }
    // zero columns past the widths (rows of the input tiles are a multiple of 16 bytes)
    for (uint32_t e = tid; e < rows * ldx / 4u; e += kPredThreads) reinterpret_cast<uint4 *>(xs)[e] = make_uint4(0, 0, 0, 0);
    if (H != Hp) {
        for (uint32_t e = tid; e < 2u * rows * 16u; e += kPredThreads) h1[(e >> 4) * ldh + H + (e & 15u)] = 0;
    }
    __syncthreads();
    store_x(xs);
    load_x(min(blockIdx.x + gridDim.x, tiles - 1u));
    __syncthreads();
    uint32_t turn = 0, buf = 0;
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const uint32_t row0 = rg * 16u * RT;  // the wave's rows of the tile
        uint16_t *xb = xs + buf * rows * ldx, *xn = xs + (buf ^ 1u) * rows * ldx;
        v4f acc[RT][NT];
        // a hidden layer of the wave's first T tiles of columns
        auto activate = [&](uint16_t *h, const float (&b)[NT], auto count) {
            constexpr uint32_t T = decltype(count)::value;
#pragma unroll
            for (uint32_t j = 0; j < T; ++j) {
                const uint32_t c = wc + wcols * j;
                if (!SKIP && c >= ct) continue;
#pragma unroll
                for (uint32_t q = 0; q < RT; ++q)
#pragma unroll
                    for (uint32_t t = 0; t < 4u; ++t)
                        h[(row0 + 16u * q + 4u * g + t) * ldh + 16u * c + r] = f2bf_hw(silu(acc[q][j][t] + b[j]));
            }
        };
        auto layer1 = [&](auto count) {
            constexpr uint32_t T = decltype(count)::value;
#pragma unroll
            for (uint32_t q = 0; q < RT; ++q) {
                const v8bf f = frag<16, false>(xb, ldx, row0 + 16u * q, 0u, lane);
#pragma unroll
                for (uint32_t j = 0; j < T; ++j) acc[q][j] = Mfma<16>::mac(f, w1[j], v4f{0.f, 0.f, 0.f, 0.f});
            }
            if (Kx > 32u) {
#pragma unroll
                for (uint32_t j = 0; j < T; ++j) {
#pragma unroll
                    for (uint32_t q = 0; q < RT; ++q)
                        acc[q][j] = Mfma<16>::mac(frag<16, false>(xb, ldx, row0 + 16u * q, 32u, lane), w1b[j], acc[q][j]);
                }
            }
            activate(h1, b1, count);
        };
        auto layer2 = [&](auto count) {
            constexpr uint32_t T = decltype(count)::value;
#pragma unroll
            for (uint32_t q = 0; q < RT; ++q)
#pragma unroll
                for (uint32_t j = 0; j < T; ++j) acc[q][j] = v4f{0.f, 0.f, 0.f, 0.f};
            if constexpr (RES) {
#pragma unroll
                for (uint32_t u = 0; u < K2; ++u)
                    if (32u * u < H) {
#pragma unroll
                        for (uint32_t q = 0; q < RT; ++q) {
                            const v8bf f = frag<16, false>(h1, ldh, row0 + 16u * q, 32u * u, lane);
#pragma unroll
                            for (uint32_t j = 0; j < T; ++j) acc[q][j] = Mfma<16>::mac(f, w2[j][u], acc[q][j]);
                        }
                    }
            } else {
                constexpr uint32_t KB = 2;  // steps whose weights are in flight together
#pragma unroll 1
                for (uint32_t k0 = 0; k0 < H; k0 += 32u * KB) {
                    uint4 w[KB][T];
#pragma unroll
                    for (uint32_t u = 0; u < KB; ++u)
#pragma unroll
                        for (uint32_t j = 0; j < T; ++j) {
                            const uint32_t n = min(16u * (wc + wcols * j), H - 16u) + r, k = k0 + 32u * u + 8u * g;
                            w[u][j] = ld8u(a.W2T + (size_t)n * H + min(k, H - 8u));
                        }
#pragma unroll
                    for (uint32_t u = 0; u < KB; ++u)
                        if (k0 + 32u * u < H) {
#pragma unroll
                            for (uint32_t j = 0; j < T; ++j) w[u][j] = keep(k0 + 32u * u + 8u * g < H, w[u][j]);
#pragma unroll
                            for (uint32_t q = 0; q < RT; ++q) {
                                const v8bf f = frag<16, false>(h1, ldh, row0 + 16u * q, k0 + 32u * u, lane);
#pragma unroll
                                for (uint32_t j = 0; j < T; ++j)
                                    acc[q][j] = Mfma<16>::mac(f, __builtin_bit_cast(v8bf, w[u][j]), acc[q][j]);
                            }
                        }
                }
            }
            activate(h2, b2, count);
        };
        auto of_mine = [&](auto layer) {  // no work for tiles that the layer does not have
            if (!SKIP || (NT == 2u && mine == 2u)) layer(std::integral_constant<uint32_t, NT>{});
            else if (mine != 0u) layer(std::integral_constant<uint32_t, 1>{});
        };
        of_mine(layer1);
        store_x(xn);
        load_x(min(tile + 2u * gridDim.x, tiles - 1u));
        __syncthreads();
        of_mine(layer2);
        __syncthreads();
        // layer 3, 16 rows to a wave; it passes the next tile's first barrier before h2 is
        // written again
        const uint32_t blocks = RT * groups, q = (wave + kPredWaves - turn) % kPredWaves;
        if (q < blocks) {
            v4f y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (uint32_t k0 = 0; k0 < Hp; k0 += 32u)
                y = Mfma<16>::mac(frag<16, false>(h2, ldh, 16u * q, k0, lane), frag<16, true>(w3s, 16u, 0u, k0, lane), y);
            if (r < a.dout) {
#pragma unroll
                for (uint32_t t = 0; t < 4u; ++t) {
                    const uint64_t row = (uint64_t)tile * rows + 16u * q + 4u * g + t;
                    if (row < a.N) a.y[row * a.dout + r] = y[t] + b3;
                }
            }
        }
        turn = (turn + blocks) % kPredWaves;
        buf ^= 1u;
    }
}

// ------------------------------------------------------------------------------------------
// Fused training step: forward, loss gradient, back-propagation and Adam in two launches, on
// gfx950's v_mfma_f32_16x16x32_bf16 (eight bfloat16 of the reduction per lane and operand).
//
// mlp_train_rows: one workgroup per 16 batch rows.  The rows' input, both hidden activations, the
//   loss gradient and the first back-propagated gradient stay in LDS, the pre-activations in
//   registers; every operand fragment is one 16-byte read (LDS rows, the bfloat16 W2 and its
//   transposed copy).  The activations and gradients the weight gradients need are written to the
//   workspace transposed ([feature][batch], 8-byte stores), so that the next kernel reads its
//   fragments (eight consecutive batch rows) with 16-byte loads as well.
// mlp_train_params: four waves per 16x16 tile of a weight gradient (with the bias as the extra row
//   of ones, as in the unfused path), each reducing an interleaved quarter of the batch; their sums
//   are added in a fixed order -- deterministic -- and each wave then applies Adam to a quarter of
//   the tile and stores the bfloat16 copies of the updated weights.
// Rounding points and fp32 accumulation are those of the unfused kernels; only the order of the
// fp32 sums differs.
// ------------------------------------------------------------------------------------------
constexpr uint32_t kTrainRows = 16;
constexpr uint32_t kParamSplit = 4;  // waves that reduce one weight-gradient tile, each a quarter of the batch
// reduction steps whose global operand loads are issued together before their matrix-core chain
// (the chain's order, and so every rounding, is the step-by-step one)
constexpr uint32_t kLoadAhead = 8;
constexpr uint32_t kTrainMaxH = 256;
constexpr uint32_t kTrainMaxIn = 32;
constexpr uint32_t kTrainPad = 8;  // bf16 elements of padding per LDS row

__device__ __forceinline__ v4f mfma32(v8bf a, v8bf b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// four bfloat16 of consecutive batch rows into a transposed [feature][batch] array
__device__ __forceinline__ void st4(uint16_t *p, uint16_t a, uint16_t b, uint16_t c, uint16_t d)
{
    *reinterpret_cast<uint2 *>(p) = make_uint2((uint32_t)a | ((uint32_t)b << 16), (uint32_t)c | ((uint32_t)d << 16));
}

struct TrainArgs {
    const float *x, *t;      // all samples: x[n][din], t[n][dout]
    const uint32_t *idx;     // the batch's sample indices (NULL: 0..B-1)
    uint32_t B, Bp;          // batch, and batch rounded up to 32 (leading dim of the T arrays)
    uint32_t din, H, dout;
    const uint16_t *W1, *W2, *W2T, *W3;
    float *p, *m, *v, *grads;  // fp32 parameters, Adam moments, optional gradient output
    uint16_t *wb;              // bfloat16 weight copies
    uint16_t *xT, *h1T, *h2T, *dyT, *dz2T, *dz1T;
    float *loss_part, *loss;
    Layout l;
    int kind;
    float delta, inv_n;        // Huber delta; 1 / (B dout)
    float lr, beta1, beta2, eps, c1, c2;
    uint32_t tiles1, tiles2, tiles3;  // gradient tiles of W1|b1, W2|b2, W3|b3
};

// Eight bfloat16 of B operands that lie `stride` apart from `first` on (a column of row-major
// weights, or a row too short for a wide load); zero past `left`, the lane's own number of them
// (lanes past their end read the first element of all), and a uniform `count` >= left spares the
// second four loads.
__device__ __forceinline__ v8bf gather8(const uint16_t *base, uint32_t first, uint32_t stride, uint32_t count,
                                        uint32_t left)
{
    uint32_t e[8] = {};
#pragma unroll
    for (uint32_t t = 0; t < 4u; ++t) e[t] = ld1u(base, t < left ? 2u * (first + t * stride) : 0u);
    if (count > 4u) {
#pragma unroll
        for (uint32_t t = 4u; t < 8u; ++t) e[t] = ld1u(base, t < left ? 2u * (first + t * stride) : 0u);
    }
    uint4 u;
    u.x = (left > 0u ? e[0] : 0u) | (left > 1u ? e[1] << 16 : 0u);
    u.y = (left > 2u ? e[2] : 0u) | (left > 3u ? e[3] << 16 : 0u);
    u.z = (left > 4u ? e[4] : 0u) | (left > 5u ? e[5] << 16 : 0u);
    u.w = (left > 6u ? e[6] : 0u) | (left > 7u ? e[7] << 16 : 0u);
    return __builtin_bit_cast(v8bf, u);
}

// One wave per 16 columns of the hidden layers, H / 16 of them: every wave has one tile per layer
// and at most kLoadAhead matrix-core steps over H.  A batch of 1024 is 64 workgroups, so only a
// quarter of the chip works and each of its SIMDs issues for four waves: the instructions of one
// wave, and the latencies between the barriers, are the kernel's time.  Therefore H is a template
// argument (addresses are immediate offsets; every multiple of 32 up to 256 has its own code);
// every operand that does not depend on the rows is requested at the start, before the first
// wait (W2's fragments for the last phase after layer 2); pre-activations stay in the registers
// of the wave that needs them again; and silu' is computed by the waves that have nothing to do
// while wave 0 computes layer 3 and the loss.  H = 256, 1024 rows: 18.0 us with H an argument,
// pre-activations in LDS and silu' at its use, 14.3 us here.
template <uint32_t H>
__global__ void __launch_bounds__(H * 4) mlp_train_rows(const TrainArgs a)
{
    constexpr uint32_t kSteps = H / 32u, ldh = H + kTrainPad;
    static_assert(H <= kTrainMaxH && kSteps <= kLoadAhead, "one load chunk");
    __shared__ __align__(16) uint16_t xs[kTrainRows * 32u], dys[kTrainRows * 16u];
    __shared__ __align__(16) uint16_t h1s[kTrainRows * ldh], h2s[kTrainRows * ldh], dzs[kTrainRows * ldh];
    __shared__ __align__(16) uint16_t w3s[16u * ldh];  // W3 transposed: [d_out][H]
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t r = lane & 15u, g = lane >> 4;
    const uint32_t row0 = blockIdx.x * kTrainRows, last = a.B - 1u;
    const uint32_t n = 16u * wave + r;  // the wave's output columns
    const uint32_t din = a.din, dout = a.dout;
    // the samples of the rows this thread stages, and in wave 0 those of its four loss rows
    constexpr uint32_t kStage = (kTrainRows * 32u + H * 4u - 1u) / (H * 4u);
    uint32_t xsrc[kStage], tsrc[4];
#pragma unroll
    for (uint32_t j = 0; j < kStage; ++j) {
        xsrc[j] = min(row0 + (threadIdx.x + H * 4u * j) / 32u % kTrainRows, last);
        if (a.idx) xsrc[j] = a.idx[xsrc[j]];
    }
    if (wave == 0)
#pragma unroll
        for (uint32_t t = 0; t < 4u; ++t) {
            tsrc[t] = min(row0 + 4u * g + t, last);
            if (a.idx) tsrc[t] = a.idx[tsrc[t]];
        }
    // layer 1 (W1 column n), layer 2 (W2T row n), layer 3 and its gradient (W3 row n), the biases
    const v8bf w1 = gather8(a.W1, 8u * g * H + n, H, min(din, 8u), din > 8u * g ? din - 8u * g : 0u);
    v8bf w2t[kSteps];
#pragma unroll
    for (uint32_t u = 0; u < kSteps; ++u)
        w2t[u] = __builtin_bit_cast(v8bf, ld8u(a.W2T + 32u * u, 2u * (n * H + 8u * g)));
    const v8bf w3 = gather8(a.W3, n * dout + 8u * g, 1u, min(dout, 8u), dout > 8u * g ? dout - 8u * g : 0u);
    const float b1n = a.p[a.l.b1 + n], b2n = a.p[a.l.b2 + n];
    const uint32_t c = threadIdx.x % 32u;
    float xv[kStage];
#pragma unroll
    for (uint32_t j = 0; j < kStage; ++j) xv[j] = a.x[(size_t)xsrc[j] * din + min(c, din - 1u)];
    // wave 0's layer-3 operands: b3 and the rows' targets
    float b3r = 0.f, tv[4] = {0.f, 0.f, 0.f, 0.f};
    const uint32_t rc = min(r, dout - 1u);  // columns past d_out repeat the last; theirs are not used
    if (wave == 0) {
        b3r = a.p[a.l.b3 + rc];
#pragma unroll
        for (uint32_t t = 0; t < 4u; ++t) tv[t] = a.t[(size_t)tsrc[t] * dout + rc];
    }
    // inputs of the rows (zero past the batch) and their transposed copy
#pragma unroll
    for (uint32_t j = 0; j < kStage; ++j) {
        const uint32_t i = threadIdx.x + H * 4u * j, row = row0 + i / 32u;
        if (kTrainRows * 32u % (H * 4u) != 0u && i >= kTrainRows * 32u) break;  // whole waves
        const uint16_t v = (uint16_t)(f2bf(xv[j]) & (row < a.B && c < din ? 0xFFFFu : 0u));
        xs[i] = v;
        if (c < din) a.xT[(size_t)c * a.Bp + row] = v;
    }
    if (g < 2u) {  // zeros past d_out
        const uint4 u = __builtin_bit_cast(uint4, w3);
        const uint32_t e[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (uint32_t t = 0; t < 8u; ++t)
            w3s[(8u * g + t) * ldh + n] = (uint16_t)(e[t / 2u] >> (16u * (t & 1u)));
    }
    __syncthreads();
    // layer 1: z1 = x W1 + b1, h1 = silu(z1)  (one reduction step: d_in <= 32)
    float z1[4], z2[4];
    uint16_t hb[4];
    v4f acc = {0.f, 0.f, 0.f, 0.f};
    acc = mfma32(ld8(xs + r * 32u + 8u * g), w1, acc);
    const uint32_t at = 4u * g * ldh + n;  // the lane's first element of a [16][ldh] array
#pragma unroll
    for (uint32_t t = 0; t < 4u; ++t) {
        z1[t] = acc[t] + b1n;
        hb[t] = f2bf_hw(silu(z1[t]));
        h1s[at + t * ldh] = hb[t];
    }
    const size_t tat = (size_t)n * a.Bp + row0 + 4u * g;  // and of a transposed array
    st4(a.h1T + tat, hb[0], hb[1], hb[2], hb[3]);
    __syncthreads();
    // layer 2: z2 = h1 W2 + b2, B fragments from the transposed copy W2T[n][k]; then the W2
    // fragments of the dz1 step, in flight through layer 3 and the dz2 step
    acc = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (uint32_t u = 0; u < kSteps; ++u) acc = mfma32(ld8(h1s + r * ldh + 32u * u + 8u * g), w2t[u], acc);
    v8bf w2[kSteps];
#pragma unroll
    for (uint32_t u = 0; u < kSteps; ++u)
        w2[u] = __builtin_bit_cast(v8bf, ld8u(a.W2 + 32u * u, 2u * (n * H + 8u * g)));
#pragma unroll
    for (uint32_t t = 0; t < 4u; ++t) {
        z2[t] = acc[t] + b2n;
        hb[t] = f2bf_hw(silu(z2[t]));
        h2s[at + t * ldh] = hb[t];
    }
    st4(a.h2T + tat, hb[0], hb[1], hb[2], hb[3]);
    __syncthreads();
    // layer 3, loss and its gradient (one wave): y = h2 W3 + b3; dy = dloss/dy, zero past the batch
    if (wave == 0) {
        __builtin_amdgcn_s_setprio(2);
        acc = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (uint32_t u = 0; u < kSteps; ++u)
            acc = mfma32(ld8(h2s + r * ldh + 32u * u + 8u * g), ld8(w3s + r * ldh + 32u * u + 8u * g), acc);
        float ls = 0.f;
        uint16_t db[4];
#pragma unroll
        for (uint32_t t = 0; t < 4u; ++t) {
            const bool in = row0 + 4u * g + t < a.B && r < dout;
            const float d = acc[t] + b3r - tv[t];
            float dy, l;
            if (a.kind == CAE_LOSS_MSE) {
                dy = 2.0f * d * a.inv_n;
                l = d * d;
            } else {
                const float ad = fabsf(d);
                dy = fminf(fmaxf(d, -a.delta), a.delta) * a.inv_n;
                l = ad <= a.delta ? 0.5f * d * d : a.delta * (ad - 0.5f * a.delta);
            }
            ls += in ? l : 0.f;
            db[t] = in ? f2bf_hw(dy) : (uint16_t)0;
            dys[(4u * g + t) * 16u + r] = db[t];
        }
        st4(a.dyT + (size_t)r * a.Bp + row0 + 4u * g, db[0], db[1], db[2], db[3]);
        // the rows' loss, summed over the wave in a fixed order
#pragma unroll
        for (uint32_t off = 32u; off > 0u; off >>= 1) ls += __shfl_xor(ls, (int)off);
        if (lane == 0) a.loss_part[blockIdx.x] = ls;
        __builtin_amdgcn_s_setprio(0);
    }
#pragma unroll
    for (uint32_t t = 0; t < 4u; ++t) {
        z1[t] = dsilu(z1[t]);
        z2[t] = dsilu(z2[t]);
        asm volatile("" : "+v"(z1[t]), "+v"(z2[t]));  // here, not after the barrier
    }
    __syncthreads();
    // dz2 = (dy W3^T) silu'(z2)  (one reduction step: d_out <= 16)
    v8bf dyf = ld8(dys + r * 16u + 8u * (g & 1u));
    if (g >= 2u) dyf = __builtin_bit_cast(v8bf, make_uint4(0u, 0u, 0u, 0u));
    acc = v4f{0.f, 0.f, 0.f, 0.f};
    acc = mfma32(dyf, w3, acc);
    uint16_t zb[4];
#pragma unroll
    for (uint32_t t = 0; t < 4u; ++t) {
        zb[t] = f2bf_hw(acc[t] * z2[t]);
        dzs[at + t * ldh] = zb[t];
    }
    st4(a.dz2T + tat, zb[0], zb[1], zb[2], zb[3]);
    __syncthreads();
    // dz1 = (dz2 W2^T) silu'(z1): B fragments W2[n][k], eight consecutive k
    acc = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (uint32_t u = 0; u < kSteps; ++u) acc = mfma32(ld8(dzs + r * ldh + 32u * u + 8u * g), w2[u], acc);
#pragma unroll
    for (uint32_t t = 0; t < 4u; ++t) zb[t] = f2bf_hw(acc[t] * z1[t]);
    st4(a.dz1T + tat, zb[0], zb[1], zb[2], zb[3]);
}

// Each of the tile's kParamSplit waves reduces its share of the batch, then updates one of the
// four rows that a lane holds: its parameter and moments are requested before the reduction.  The
// loss is the last workgroup's: 64 partial sums per load, added in row order.  H = 256, 1024 rows:
// 8.4 us with the update and the moments' loads in one wave after the reduction and the loss
// partials loaded one by one, 6.2 us here.
static_assert(kParamSplit == 4u, "one wave per row of a lane's accumulator");

__global__ void __launch_bounds__(kParamSplit * 64) mlp_train_params(const TrainArgs a)
{
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t r = lane & 15u, g = lane >> 4;
    uint32_t tile = blockIdx.x;
    const uint32_t H = a.H, din = a.din, dout = a.dout, ct = H / 16u;
    // which gradient: [A^T ; 1] B over the batch, A the layer's input, B its output gradient
    const uint16_t *AT, *BT;
    uint32_t M, N, ti, tj;
    uint64_t woff, boff, wcopy;
    if (tile < a.tiles1) {
        AT = a.xT, BT = a.dz1T, M = din, N = H, ti = tile / ct, tj = tile % ct;
        woff = a.l.w1, boff = a.l.b1, wcopy = 0;
    } else if ((tile -= a.tiles1) < a.tiles2) {
        AT = a.h1T, BT = a.dz2T, M = H, N = H, ti = tile / ct, tj = tile % ct;
        woff = a.l.w2, boff = a.l.b2, wcopy = (uint64_t)din * H;
    } else if ((tile -= a.tiles2) < a.tiles3) {
        AT = a.h2T, BT = a.dyT, M = H, N = dout, ti = tile, tj = 0;
        woff = a.l.w3, boff = a.l.b3, wcopy = (uint64_t)din * H + (uint64_t)H * H;
    } else {
        if (wave != 0u) return;
        const uint32_t parts = a.Bp / kTrainRows;
        float s = 0.f, next = lane < parts ? a.loss_part[lane] : 0.f;
        for (uint32_t i = 0; i < parts; i += 64u) {  // zeros past the end change nothing
            const float v = next;
            next = i + 64u + lane < parts ? a.loss_part[i + 64u + lane] : 0.f;
#pragma unroll
            for (uint32_t j = 0; j < 64u; ++j)
                s += __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), (int)j));
        }
        if (lane == 0u) a.loss[0] = s * a.inv_n;
        return;
    }
    // the parameter this lane updates: row ic of the gradient (M: the bias), column jc
    const uint32_t ic = ti * 16u + 4u * g + wave, jc = tj * 16u + r;
    const bool mine = ic <= M && jc < N;
    const uint64_t at = !mine ? boff : ic < M ? woff + (uint64_t)ic * N + jc : boff + jc;
    const float m0 = a.m[at], v0 = a.v[at], p0 = a.p[at];
    // A row and B column this lane feeds; those past the end repeat the last, and their products
    // are not used, except the row of ones
    const uint32_t arow = min(ti * 16u + r, M - 1u), bcol = min(jc, N - 1u);
    const uint16_t *const ap = AT + (size_t)arow * a.Bp + 8u * g, *const bp = BT + (size_t)bcol * a.Bp + 8u * g;
    const bool has_ones = ti * 16u + 16u > M, ones = ti * 16u + r == M;
    // wave w reduces the batch chunks w, w + kParamSplit, ... of 32 rows; the partial sums are
    // then added in wave order (a fixed order: deterministic)
    __shared__ float part[kParamSplit][4][64];
    v4f acc = {0.f, 0.f, 0.f, 0.f};
    for (uint32_t c0 = 32u * wave; c0 < a.Bp; c0 += 32u * kParamSplit * kLoadAhead) {
        uint4 av[kLoadAhead], bv[kLoadAhead];  // the chunk's fragments, in flight together
#pragma unroll
        for (uint32_t u = 0; u < kLoadAhead; ++u) {
            const uint32_t b0 = min(c0 + 32u * kParamSplit * u, a.Bp - 32u);  // past the end: not used
            av[u] = ld8u(ap + b0);
            bv[u] = ld8u(bp + b0);
        }
        if (has_ones) {
#pragma unroll
            for (uint32_t u = 0; u < kLoadAhead; ++u)
                if (ones) av[u] = make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u);
        }
#pragma unroll
        for (uint32_t u = 0; u < kLoadAhead; ++u)
            if (c0 + 32u * kParamSplit * u < a.Bp)
                acc = mfma32(__builtin_bit_cast(v8bf, av[u]), __builtin_bit_cast(v8bf, bv[u]), acc);
    }
#pragma unroll
    for (uint32_t t = 0; t < 4u; ++t) part[wave][t][lane] = acc[t];
    __syncthreads();
    if (!mine) return;
    float gi = part[0][wave][lane];
#pragma unroll
    for (uint32_t w = 1; w < kParamSplit; ++w) gi += part[w][wave][lane];
    // Adam (Kingma and Ba 2015, algorithm 1) and the bfloat16 copies
    const float mi = a.beta1 * m0 + (1.0f - a.beta1) * gi;
    const float vi = a.beta2 * v0 + (1.0f - a.beta2) * gi * gi;
    const float pi = p0 - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
    a.m[at] = mi;
    a.v[at] = vi;
    a.p[at] = pi;
    if (a.grads) a.grads[at] = gi;
    if (ic < M) {
        const uint16_t w = f2bf(pi);
        a.wb[wcopy + (uint64_t)ic * N + jc] = w;
        if (woff == a.l.w2) a.wb[a.l.w2t + (uint64_t)jc * H + ic] = w;
    }
}

using TrainRowsFn = void (*)(TrainArgs);

// The instantiation for d_hidden = H (a multiple of 32 up to kTrainMaxH, as the callers check).
TrainRowsFn train_rows_fn(uint32_t H)
{
    static const TrainRowsFn fn[kTrainMaxH / 32u] = {
        mlp_train_rows<32>,  mlp_train_rows<64>,  mlp_train_rows<96>,  mlp_train_rows<128>,
        mlp_train_rows<160>, mlp_train_rows<192>, mlp_train_rows<224>, mlp_train_rows<256>};
    return fn[H / 32u - 1u];
}

}  // namespace

namespace {
int forward_impl(const cae_mlp *net, const float *x, float *y, uint32_t N, void *ws, hipStream_t s);
int backward_impl(const cae_mlp *net, const float *dy, float *grads, uint32_t N, void *ws, hipStream_t s);
}  // namespace

namespace cae_detail {
int set_error(int code, const char *msg);  // cae_engine.hip: message for cae_last_error()
}

namespace {

int mfail(int code, const char *msg) { return cae_detail::set_error(code, msg); }

// Workspace of the layer-by-layer path: activations and pre-activations of the forward pass,
// back-propagated gradients and the weight gradients' split-batch parts.
struct WsLayout {
    size_t xb, z1, h1, z2, h2, dyb, dz2, dz1, part, total;
};

// The bfloat16 arrays end in a block of rows that may be read (its values are never used).
constexpr uint64_t kPadRows = kBK;

size_t al(size_t x) { return (x + 255) / 256 * 256; }

// Chunks of the batch in the weight gradients (kSplitChunk rows, more beyond kMaxParts of them),
// and whether each is a workgroup of its own.  The chunks' results then cross memory twice, so
// tiles that already fill the chip take every chunk themselves.
constexpr uint32_t kSplitChunk = 256;
constexpr uint32_t kMaxParts = 64;
constexpr uint32_t kGradTiles = 128;  // tiles of W2 from which a workgroup takes all chunks

struct GradSplit {
    uint32_t tiles1, tiles2, tiles3, parts, chunk;
};

GradSplit grad_split(uint32_t H, uint32_t N)
{
    GradSplit s;
    const uint32_t t = (H + 63u) / 64u;
    s.tiles1 = t;
    s.tiles2 = t * t;
    s.tiles3 = (H + 127u) / 128u;
    const uint32_t chunks = (uint32_t)std::min<uint64_t>(kMaxParts, ((uint64_t)N + kSplitChunk - 1u) / kSplitChunk);
    s.chunk = (uint32_t)(((uint64_t)N + chunks - 1u) / chunks + 15u) / 16u * 16u;
    s.parts = s.tiles2 >= kGradTiles ? 1u : (uint32_t)(((uint64_t)N + s.chunk - 1u) / s.chunk);
    return s;
}

size_t part_stride(uint64_t P) { return (size_t)(P + 3u) / 4u * 4u; }  // floats per part, 16-byte steps

WsLayout ws_layout(uint32_t din, uint32_t H, uint32_t dout, uint32_t N)
{
    WsLayout w;
    size_t o = 0;
    w.xb = o; o = al(o + 2ull * (N + kPadRows) * ((din + 15u) & ~15u));
    w.z1 = o; o = al(o + 4ull * N * H);
    w.h1 = o; o = al(o + 2ull * (N + kPadRows) * H);
    w.z2 = o; o = al(o + 4ull * N * H);
    w.h2 = o; o = al(o + 2ull * (N + kPadRows) * H);
    w.dyb = o; o = al(o + 2ull * (N + kPadRows) * 16u);
    w.dz2 = o; o = al(o + 2ull * (N + kPadRows) * H);
    w.dz1 = o; o = al(o + 2ull * (N + kPadRows) * H);
    // parts grow with the batch, so a workspace for N holds every smaller batch's
    const size_t parts = grad_split(H, std::max(N, 1u)).tiles2 >= kGradTiles
                             ? 0u
                             : std::min<size_t>(kMaxParts, ((size_t)N + kSplitChunk - 1u) / kSplitChunk);
    w.part = o; o = al(o + 4ull * parts * part_stride(layout(din, H, dout).P));
    w.total = o;
    return w;
}

// Workspace of the fused training step: the transposed activations and gradients ([rows][Bp]
// bfloat16, Bp = the batch rounded up to 32) and one loss partial per 16 rows.
struct TrainWs {
    size_t xT, h1T, h2T, dyT, dz2T, dz1T, loss_part, total;
};

TrainWs train_ws(uint32_t din, uint32_t H, uint32_t N)
{
    const size_t Bp = (N + 31u) / 32u * 32u;
    TrainWs w;
    size_t o = 0;
    w.xT = o; o = al(o + 2 * din * Bp);
    w.h1T = o; o = al(o + 2 * (size_t)H * Bp);
    w.h2T = o; o = al(o + 2 * (size_t)H * Bp);
    w.dyT = o; o = al(o + 2 * 16 * Bp);
    w.dz2T = o; o = al(o + 2 * (size_t)H * Bp);
    w.dz1T = o; o = al(o + 2 * (size_t)H * Bp);
    w.loss_part = o; o = al(o + 4 * (Bp / kTrainRows));
    w.total = o;
    return w;
}

int check_net(const cae_mlp *net)
{
    if (!net || !net->params || !net->weights) return mfail(CAE_EINVAL, "NULL network or buffer");
    if (net->d_in < 1 || net->d_in > 64) return mfail(CAE_EINVAL, "d_in must be in 1..64");
    if (net->d_hidden < 16 || net->d_hidden > 1024 || net->d_hidden % 16)
        return mfail(CAE_EINVAL, "d_hidden must be a multiple of 16 in 16..1024");
    if (net->d_out < 1 || net->d_out > 16) return mfail(CAE_EINVAL, "d_out must be in 1..16");
    return CAE_OK;
}

int launch_status()
{
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return mfail(CAE_EHIP, hipGetErrorString(e));
    return CAE_OK;
}

void launch_adam(const cae_mlp *net, const float *g, float *m, float *v, float lr, float beta1, float beta2,
                 float eps, float c1, float c2, int update, hipStream_t s)
{
    AdamArgs a;
    a.p = net->params;
    a.g = g;
    a.m = m;
    a.v = v;
    a.wb = net->weights;
    a.l = layout(net->d_in, net->d_hidden, net->d_out);
    a.H = net->d_hidden;
    a.tiles = (a.H + 63u) / 64u;
    a.lr = lr;
    a.beta1 = beta1;
    a.beta2 = beta2;
    a.eps = eps;
    a.c1 = c1;
    a.c2 = c2;
    a.update = update;
    const uint32_t rest = (uint32_t)((a.l.P - (a.l.b2 - a.l.w2) + 255u) / 256u);
    hipLaunchKernelGGL(adam_step, dim3(a.tiles * a.tiles + rest), dim3(256), 0, s, a);
}

// Scratch of cae_mlp_train_step_noalloc: the fused training step's workspace (transposed
// activations and gradients, loss partials) for callers that cannot allocate device memory.
// Every device the library runs on holds its own copy until the process ends; host code must not
// pass the array's name to a kernel (it is a host-side stand-in), only the per-device address
// that hipGetSymbolAddress returns.  Nothing in it needs clearing between calls: each call's
// first kernel writes every word its second kernel reads.
constexpr size_t kScratchBytes = size_t(8) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// The address of the current device's copy of `scratch`, looked up once per device.
int scratch_of_current_device(void **out)
{
    int dev = -1;
    hipError_t he = hipGetDevice(&dev);
    if (he != hipSuccess) return mfail(CAE_EHIP, hipGetErrorString(he));
    if (dev < 0 || dev >= kMaxDevices) return mfail(CAE_EINVAL, "device index beyond the scratch table");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        he = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (he != hipSuccess || !p)
            return mfail(CAE_EHIP, he != hipSuccess ? hipGetErrorString(he) : "no address for the scratch array");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return CAE_OK;
}

// Compute units of the current device, looked up once per device (a look-up is 0.25 us of a call).
int cus_of_current_device(uint32_t *out)
{
    static std::atomic<uint32_t> known[kMaxDevices];
    int dev = -1, n = 0;
    hipError_t he = hipGetDevice(&dev);
    const bool slot = he == hipSuccess && dev >= 0 && dev < kMaxDevices;
    *out = slot ? known[dev].load(std::memory_order_relaxed) : 0u;
    if (*out) return CAE_OK;
    if (he == hipSuccess) he = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
    if (he != hipSuccess || n < 1) return mfail(CAE_EHIP, hipGetErrorString(he));
    *out = (uint32_t)n;
    if (slot) known[dev].store(*out, std::memory_order_relaxed);
    return CAE_OK;
}

// Argument checks shared by both training-step entry points (no device call).
int check_train_args(const cae_mlp *net, const float *x, const float *target, const float *m, const float *v,
                     uint32_t N, uint32_t step, int loss_kind, float delta, const float *loss)
{
    int rc = check_net(net);
    if (rc) return rc;
    const uint32_t din = net->d_in, H = net->d_hidden;
    if (H % 32u || H > kTrainMaxH || din > kTrainMaxIn)
        return mfail(CAE_EINVAL, "cae_mlp_train_step needs d_hidden a multiple of 32 up to 256 and d_in <= 32");
    if (!x || !target || !m || !v || !loss) return mfail(CAE_EINVAL, "NULL pointer");
    if (N == 0) return mfail(CAE_EINVAL, "N must be >= 1");
    if (step < 1) return mfail(CAE_EINVAL, "step counts from 1");
    if (loss_kind != CAE_LOSS_MSE && loss_kind != CAE_LOSS_HUBER) return mfail(CAE_EINVAL, "unknown loss kind");
    if (loss_kind == CAE_LOSS_HUBER && !(delta > 0.0f)) return mfail(CAE_EINVAL, "Huber delta must be > 0");
    return CAE_OK;
}

// The fused training step (two launches) on a workspace of train_ws(d_in, H, N).total bytes.
int train_step_impl(const cae_mlp *net, const float *x, const float *target, const uint32_t *idx, uint32_t N,
                    float *m, float *v, uint32_t step, float lr, float beta1, float beta2, float eps, int loss_kind,
                    float delta, float *loss, float *grads, void *ws, hipStream_t s)
{
    const uint32_t din = net->d_in, H = net->d_hidden, dout = net->d_out;
    const Layout l = layout(din, H, dout);
    const TrainWs w = train_ws(din, H, N);
    unsigned char *b = static_cast<unsigned char *>(ws);
    TrainArgs a;
    a.x = x;
    a.t = target;
    a.idx = idx;
    a.B = N;
    a.Bp = (N + 31u) / 32u * 32u;
    a.din = din;
    a.H = H;
    a.dout = dout;
    a.W1 = net->weights;
    a.W2 = a.W1 + (size_t)din * H;
    a.W3 = a.W2 + (size_t)H * H;
    a.W2T = net->weights + l.w2t;
    a.p = net->params;
    a.m = m;
    a.v = v;
    a.grads = grads;
    a.wb = net->weights;
    a.xT = reinterpret_cast<uint16_t *>(b + w.xT);
    a.h1T = reinterpret_cast<uint16_t *>(b + w.h1T);
    a.h2T = reinterpret_cast<uint16_t *>(b + w.h2T);
    a.dyT = reinterpret_cast<uint16_t *>(b + w.dyT);
    a.dz2T = reinterpret_cast<uint16_t *>(b + w.dz2T);
    a.dz1T = reinterpret_cast<uint16_t *>(b + w.dz1T);
    a.loss_part = reinterpret_cast<float *>(b + w.loss_part);
    a.loss = loss;
    a.l = l;
    a.kind = loss_kind;
    a.delta = delta;
    a.inv_n = 1.0f / (float)((double)N * dout);
    a.lr = lr;
    a.beta1 = beta1;
    a.beta2 = beta2;
    a.eps = eps;
    a.c1 = (float)(1.0 - std::pow((double)beta1, (double)step));
    a.c2 = (float)(1.0 - std::pow((double)beta2, (double)step));
    const uint32_t ct = H / 16u;
    a.tiles1 = (din + 1u + 15u) / 16u * ct;
    a.tiles2 = (H / 16u + 1u) * ct;
    a.tiles3 = H / 16u + 1u;
    hipLaunchKernelGGL(train_rows_fn(H), dim3(a.Bp / kTrainRows), dim3(H * 4u), 0, s, a);
    const uint32_t tiles = a.tiles1 + a.tiles2 + a.tiles3;  // and the loss
    hipLaunchKernelGGL(mlp_train_params, dim3(tiles + 1u), dim3(kParamSplit * 64u), 0, s, a);
    return launch_status();
}

}  // namespace

extern "C" {

int cae_mlp_sizes(uint32_t d_in, uint32_t d_hidden, uint32_t d_out, uint32_t max_batch, cae_mlp_sizes_t *out)
{
    if (!out) return mfail(CAE_EINVAL, "out is NULL");
    cae_mlp probe{d_in, d_hidden, d_out, 0, reinterpret_cast<float *>(1), reinterpret_cast<uint16_t *>(1)};
    int rc = check_net(&probe);
    if (rc) return rc;
    const Layout l = layout(d_in, d_hidden, d_out);
    out->n_params = l.P;
    out->n_weights = l.W;
    out->workspace_bytes = std::max(ws_layout(d_in, d_hidden, d_out, max_batch).total,
                                    train_ws(d_in, d_hidden, max_batch).total);
    return CAE_OK;
}

int cae_mlp_refresh_weights(const cae_mlp *net, void *stream)
{
    int rc = check_net(net);
    if (rc) return rc;
    launch_adam(net, nullptr, nullptr, nullptr, 0.f, 0.f, 0.f, 0.f, 1.f, 1.f, 0, (hipStream_t)stream);
    return launch_status();
}

int cae_mlp_forward(const cae_mlp *net, const float *x, float *y, uint32_t N, void *ws, void *stream)
{
    int rc = check_net(net);
    if (rc) return rc;
    if (!x || !y || !ws) return mfail(CAE_EINVAL, "NULL x, y or workspace");
    if (N == 0) return CAE_OK;
    return forward_impl(net, x, y, N, ws, (hipStream_t)stream);
}

int cae_mlp_predict(const cae_mlp *net, const float *x, float *y, uint32_t N, void *stream)
{
    int rc = check_net(net);
    if (rc) return rc;
    if (!x || !y) return mfail(CAE_EINVAL, "NULL x or y");
    if (net->d_hidden > kPredMaxH) return mfail(CAE_EINVAL, "cae_mlp_predict needs d_hidden <= 496");
    if (N == 0) return CAE_OK;
    const uint32_t din = net->d_in, H = net->d_hidden, dout = net->d_out;
    const Layout l = layout(din, H, dout);
    PredArgs a;
    a.x = x;
    a.y = y;
    a.N = N;
    a.din = din;
    a.H = H;
    a.dout = dout;
    a.W1 = net->weights;
    a.W2T = net->weights + l.w2t;
    a.W3 = net->weights + (size_t)din * H + (size_t)H * H;
    a.b1 = net->params + l.b1;
    a.b2 = net->params + l.b2;
    a.b3 = net->params + l.b3;
    uint32_t cus = 0;
    rc = cus_of_current_device(&cus);
    if (rc) return rc;
    a.cols_log2 = H > 128u ? 4u : (H > 64u ? 3u : 2u);
    const uint64_t Hp = (H + 31u) & ~31u, Kx = (din + 31u) & ~31u;
    const auto lds_bytes = [&](uint64_t rows) { return 2u * (2u * rows * (Hp + 8u) + 2u * rows * (Kx + 8u) + Hp * 16u); };
    // waves without a tile of columns skip its work where that leaves every SIMD less of it (beyond
    // 448 columns some SIMD's four waves all have two tiles: H = 464, 65536 rows 105 us either way)
    const auto skips = [&](uint32_t cols_log2) { return H <= 256u ? H < 16u << cols_log2 : H <= 448u; };
    // more rows share each pass over the weights, once every CU has a tile of them and as long as
    // the tile's input fits its threads' registers: first the waves that a narrow layer has no
    // columns for take rows, then blocks of 16 rows per wave.  Eight input values per thread instead
    // of four pay where the waves are few (d_in = 40, 300000 rows: H = 16 36 us to 27, H = 48 46 to
    // 41) and cost registers elsewhere (H = 208 148 to 154)
    const auto may_double = [&](uint32_t rows, uint32_t cols_log2) {
        const uint32_t inputs = H <= 48u && skips(cols_log2) ? 8u : 4u;
        return (uint64_t)rows * cus < N && 2u * rows * din <= inputs * kPredThreads && lds_bytes(2u * rows) <= 160u * 1024u;
    };
    while (a.cols_log2 > 0u && H <= 8u << a.cols_log2 && may_double(16u * (kPredWaves >> a.cols_log2), a.cols_log2 - 1u))
        --a.cols_log2;
    const uint32_t groups = kPredWaves >> a.cols_log2, most = H > 256u ? 4u : std::min(2u, kPredWaves / groups);
    uint32_t rt = 1;
    while (2u * rt <= most && may_double(16u * rt * groups, a.cols_log2)) rt *= 2u;
    const uint32_t rows = 16u * rt * groups;
    const size_t lds = lds_bytes(rows);
    const uint32_t tiles = (uint32_t)(((uint64_t)N + rows - 1u) / rows);
    const bool skip = skips(a.cols_log2);
    const dim3 grid(std::min(tiles, cus)), block(kPredThreads);
    const hipStream_t s = (hipStream_t)stream;
    const auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, lds, s, a); };
    const auto either = [&](auto whole, auto some) { launch(skip ? some : whole); };
    if (rows * din > 4u * kPredThreads) launch(rt == 1u ? mlp_predict<1, true, 1, true, 8> : mlp_predict<1, true, 2, true, 8>);
    else if (H <= 256u && rt == 1u) either(mlp_predict<1, true, 1, false, 4>, mlp_predict<1, true, 1, true, 4>);
    else if (H <= 256u) either(mlp_predict<1, true, 2, false, 4>, mlp_predict<1, true, 2, true, 4>);
    else if (rt == 1u) either(mlp_predict<2, false, 1, false, 4>, mlp_predict<2, false, 1, true, 4>);
    else if (rt == 2u) either(mlp_predict<2, false, 2, false, 4>, mlp_predict<2, false, 2, true, 4>);
    else either(mlp_predict<2, false, 4, false, 4>, mlp_predict<2, false, 4, true, 4>);
    return launch_status();
}

int cae_mlp_backward(const cae_mlp *net, const float *x, const float *dy, float *grads, uint32_t N, void *ws,
                     void *stream)
{
    (void)x;  // the bfloat16 input is taken from the forward pass's workspace
    int rc = check_net(net);
    if (rc) return rc;
    if (!dy || !grads || !ws) return mfail(CAE_EINVAL, "NULL dy, grads or workspace");
    if (N == 0) return mfail(CAE_EINVAL, "backward needs N >= 1");
    return backward_impl(net, dy, grads, N, ws, (hipStream_t)stream);
}

int cae_mlp_adam(const cae_mlp *net, const float *grads, float *m, float *v, uint32_t step, float lr, float beta1,
                 float beta2, float eps, void *stream)
{
    int rc = check_net(net);
    if (rc) return rc;
    if (!grads || !m || !v) return mfail(CAE_EINVAL, "NULL grads or moments");
    if (step < 1) return mfail(CAE_EINVAL, "step counts from 1");
    const float c1 = (float)(1.0 - std::pow((double)beta1, (double)step));
    const float c2 = (float)(1.0 - std::pow((double)beta2, (double)step));
    launch_adam(net, grads, m, v, lr, beta1, beta2, eps, c1, c2, 1, (hipStream_t)stream);
    return launch_status();
}

int cae_mlp_train_step(const cae_mlp *net, const float *x, const float *target, const uint32_t *idx, uint32_t N,
                       float *m, float *v, uint32_t step, float lr, float beta1, float beta2, float eps, int loss_kind,
                       float delta, float *loss, float *grads, void *ws, void *stream)
{
    int rc = check_train_args(net, x, target, m, v, N, step, loss_kind, delta, loss);
    if (rc) return rc;
    if (!ws) return mfail(CAE_EINVAL, "NULL workspace");
    return train_step_impl(net, x, target, idx, N, m, v, step, lr, beta1, beta2, eps, loss_kind, delta, loss, grads,
                           ws, (hipStream_t)stream);
}

int cae_mlp_train_step_noalloc(const cae_mlp *net, const float *x, const float *target, const uint32_t *idx,
                               uint32_t N, float *m, float *v, uint32_t step, float lr, float beta1, float beta2,
                               float eps, int loss_kind, float delta, float *loss, float *grads, void *stream)
{
    int rc = check_train_args(net, x, target, m, v, N, step, loss_kind, delta, loss);
    if (rc) return rc;
    const size_t need = train_ws(net->d_in, net->d_hidden, N).total;
    if (need > kScratchBytes) {
        char msg[160];
        std::snprintf(msg, sizeof msg,
                      "cae_mlp_train_step_noalloc: batch %u needs %zu bytes of scratch, the library holds %zu", N,
                      need, kScratchBytes);
        return mfail(CAE_EINVAL, msg);
    }
    void *ws = nullptr;
    rc = scratch_of_current_device(&ws);
    if (rc) return rc;
    return train_step_impl(net, x, target, idx, N, m, v, step, lr, beta1, beta2, eps, loss_kind, delta, loss, grads,
                           ws, (hipStream_t)stream);
}

int cae_mlp_loss_grad(const float *y, const float *target, float *dy, float *loss, uint32_t n, int kind, float delta,
                      void *stream)
{
    if (!y || !target || !dy || !loss) return mfail(CAE_EINVAL, "NULL pointer");
    if (n == 0) return mfail(CAE_EINVAL, "n must be >= 1");
    if (kind != CAE_LOSS_MSE && kind != CAE_LOSS_HUBER) return mfail(CAE_EINVAL, "unknown loss kind");
    if (kind == CAE_LOSS_HUBER && !(delta > 0.0f)) return mfail(CAE_EINVAL, "Huber delta must be > 0");
    // the gradient in workgroups of its own, unless it is short, or it or the loss overwrites words
    // that another workgroup reads or writes
    const size_t nb = 4u * (size_t)n;
    const auto apart = [](const void *a, size_t na, const void *b, size_t nb) {
        const uintptr_t x = reinterpret_cast<uintptr_t>(a), z = reinterpret_cast<uintptr_t>(b);
        return x + na <= z || z + nb <= x;
    };
    const bool split = n > 2u * kLossThreads && apart(dy, nb, y, nb) && apart(dy, nb, target, nb) &&
                       apart(loss, 4u, y, nb) && apart(loss, 4u, target, nb) && apart(loss, 4u, dy, nb);
    const uint32_t blocks = split ? 1u + std::min<uint32_t>((n + kLossThreads - 1u) / kLossThreads, 512u) : 1u;
    hipLaunchKernelGGL(loss_grad, dim3(blocks), dim3(kLossThreads), 0, (hipStream_t)stream, y, target, dy, loss, n,
                       kind, delta);
    return launch_status();
}

}  // extern "C"

namespace {

constexpr uint32_t kLayerBlocks = 256;  // workgroups that fill the chip

// Launches one layer product in the widest workgroup tile that gives every CU a workgroup: at
// 4096 x 1024 x 1024 tiles of 128 x 64 take 21.5 us, 64 x 64 22.4, 128 x 128 (one workgroup of four
// waves per CU) 22.9.  Short products spend their time in the epilogue and take 64 x 64 at most.
// Layers of 16 and 32 columns leave wider tiles mostly empty: 65536 rows of H = 16 take 13.4 us
// (second layer) in 128 x 64, 7.9 in 32 x 32 and 5.8 with the four waves below each other, 64 x 16;
// the forward pass of H = 32 28.9 us with tiles of 64 columns, 22.8 of 32.
template <bool AF32, bool KMAJOR, int EPI>
void layer(const LayerArgs &g, hipStream_t s)
{
    auto blocks = [&](uint32_t bm, uint32_t bn) { return ((g.M + bm - 1u) / bm) * ((g.N + bn - 1u) / bn); };
    const dim3 block(256);
    if (g.N == 16u && blocks(64u, 16u) >= kLayerBlocks) {
        hipLaunchKernelGGL((mlp_layer<16, 16, 1, AF32, KMAJOR, EPI>), dim3(blocks(64u, 16u)), block, 0, s, g);
        return;
    }
    if constexpr (!AF32) {
        if (g.N > 32u && blocks(128u, 64u) >= kLayerBlocks) {
            hipLaunchKernelGGL((mlp_layer<64, 32, 2, AF32, KMAJOR, EPI>), dim3(blocks(128u, 64u)), block, 0, s, g);
            return;
        }
    }
    if (g.N > 32u && blocks(64u, 64u) >= kLayerBlocks)
        hipLaunchKernelGGL((mlp_layer<32, 32, 2, AF32, KMAJOR, EPI>), dim3(blocks(64u, 64u)), block, 0, s, g);
    else
        hipLaunchKernelGGL((mlp_layer<16, 16, 2, AF32, KMAJOR, EPI>), dim3(blocks(32u, 32u)), block, 0, s, g);
}

// The layer-by-layer forward pass: activations and pre-activations are kept in ws for
// backward_impl.
int forward_impl(const cae_mlp *net, const float *x, float *y, uint32_t N, void *ws, hipStream_t s)
{
    const uint32_t din = net->d_in, H = net->d_hidden, dout = net->d_out;
    const Layout l = layout(din, H, dout);
    const WsLayout w = ws_layout(din, H, dout, N);
    unsigned char *b = static_cast<unsigned char *>(ws);
    const uint16_t *W1 = net->weights, *W2 = W1 + (size_t)din * H, *W3 = W2 + (size_t)H * H;
    LayerArgs g{};
    g.Af = x;
    g.Acopy = reinterpret_cast<uint16_t *>(b + w.xb);
    g.ldc = (din + 15u) & ~15u;
    g.B = W1;
    g.M = N;
    g.N = H;
    g.K = din;
    g.bias = net->params + l.b1;
    g.Z = reinterpret_cast<float *>(b + w.z1);
    g.O = reinterpret_cast<uint16_t *>(b + w.h1);
    layer<true, true, EPI_HIDDEN>(g, s);
    g.A = g.O;
    g.B = W2;
    g.K = H;
    g.bias = net->params + l.b2;
    g.Z = reinterpret_cast<float *>(b + w.z2);
    g.O = reinterpret_cast<uint16_t *>(b + w.h2);
    layer<false, true, EPI_HIDDEN>(g, s);
    const size_t Hp = (H + 31u) & ~31u;
    const auto out = [&](auto kernel, uint32_t rows) {
        hipLaunchKernelGGL(kernel, dim3((N + rows - 1u) / rows), dim3(256), 2u * (rows * (Hp + 8u) + 16u * Hp), s, g.O, W3,
                           net->params + l.b3, y, N, H, dout);
    };
    if (H == 16u && N >= 64u * kLayerBlocks) out(mlp_out<4>, 64u);
    else out(mlp_out<1>, 16u);
    return launch_status();
}

// Back-propagation through both hidden layers, then the three weight gradients in one launch (and
// their parts added up in another).
int backward_impl(const cae_mlp *net, const float *dy, float *grads, uint32_t N, void *ws, hipStream_t s)
{
    const uint32_t din = net->d_in, H = net->d_hidden, dout = net->d_out;
    const Layout l = layout(din, H, dout);
    const WsLayout w = ws_layout(din, H, dout, N);
    unsigned char *b = static_cast<unsigned char *>(ws);
    const uint16_t *W2 = net->weights + (size_t)din * H, *W3 = W2 + (size_t)H * H;
    // dz2 = (dy W3^T) * silu'(z2)
    LayerArgs g{};
    g.Af = dy;
    g.Acopy = reinterpret_cast<uint16_t *>(b + w.dyb);
    g.ldc = 16u;
    g.B = W3;
    g.M = N;
    g.N = H;
    g.K = dout;
    g.Z = reinterpret_cast<float *>(b + w.z2);
    g.O = reinterpret_cast<uint16_t *>(b + w.dz2);
    layer<true, false, EPI_DSILU>(g, s);
    // dz1 = (dz2 W2^T) * silu'(z1)
    g.A = g.O;
    g.B = W2;
    g.K = H;
    g.Z = reinterpret_cast<float *>(b + w.z1);
    g.O = reinterpret_cast<uint16_t *>(b + w.dz1);
    layer<false, false, EPI_DSILU>(g, s);

    const GradSplit sp = grad_split(H, N);
    GradArgs a;
    a.x = reinterpret_cast<const uint16_t *>(b + w.xb);
    a.h1 = reinterpret_cast<const uint16_t *>(b + w.h1);
    a.h2 = reinterpret_cast<const uint16_t *>(b + w.h2);
    a.dy = reinterpret_cast<const uint16_t *>(b + w.dyb);
    a.dz2 = reinterpret_cast<const uint16_t *>(b + w.dz2);
    a.dz1 = reinterpret_cast<const uint16_t *>(b + w.dz1);
    a.batch = N;
    a.din = din;
    a.H = H;
    a.dout = dout;
    a.parts = sp.parts;
    a.chunk = sp.chunk;
    a.tiles1 = sp.tiles1;
    a.tiles2 = sp.tiles2;
    a.tiles3 = sp.tiles3;
    a.stride = part_stride(l.P);
    float *out = sp.parts > 1u ? reinterpret_cast<float *>(b + w.part) : grads;  // in the parameter layout
    a.o1 = out + l.w1;
    a.o2 = out + l.w2;
    a.o3 = out + l.w3;
    const uint32_t tiles = sp.tiles1 + sp.tiles2 + sp.tiles3;
    hipLaunchKernelGGL(mlp_grad, dim3(tiles * sp.parts), dim3(256), 0, s, a);
    if (sp.parts > 1u)
        hipLaunchKernelGGL(grad_reduce, dim3((uint32_t)((l.P + 1023u) / 1024u)), dim3(256), 0, s, out, sp.parts,
                           a.stride, l.P, grads);
    return launch_status();
}

}  // namespace
