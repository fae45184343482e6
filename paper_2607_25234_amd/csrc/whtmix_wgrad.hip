// Weight gradients of the block (section III-B, eqs. (1), (4)) formed inside
// the last pass of the mixer's transform, for gfx950.
//
//     dW_out = sum over b, n of Z'[b,n,:]^T dY[b,n,:],
//     dW_in  = sum over b, n of X[b,n,:]^T dZ[b,n,:],
//
// where Z' and dZ are the middle pass's workspaces inverse-transformed over
// the A low bits of the flat index (channel bits 0 .. CB-1, token bits CB ..
// A-1).  Two facts keep Z' and dZ out of memory and most of that inverse out
// of the kernel:
//   * the sum runs over tokens only, so the inverse over the channel bits
//     commutes with it: it is applied once, to the C x C result
//     (wgrad_final_kernel), instead of to every element;
//   * a 2^A workspace tile holds whole tokens, so a workgroup that has done
//     the token bits of its tile can multiply it at once with the tile of
//     dY (or X) of the same tokens.
// So a tile costs one read of the workspace, one of dY (X), at most one LDS
// exchange, the splits and the products.
// Measured on 4 slices of 2^23 (C = 128, bf16), both gradients: 91 us, and
// 7.7 us for the final sums, where storing Z' and dZ took 63 and 30 us, the
// products from memory 2 x 65 us and their sums 4 x 5.6 us.  The 403 MB it
// reads take 87 us at the rate of a large copy (4.6 TB/s), so it is near its floor;
// the VALU (530 instructions per wave and tile) is busy 33 us and the matrix unit
// 20 us.
//
// Products (float32 accumulation), Z' / dZ rows against dY / X columns:
//   v_mfma_f32_16x16x32_bf16 on three-term bf16 splits of the float operand,
//   against bf16 dY / X (both exact) or against the same split of float32 dY /
//   X: the six products down to 2^-25 of the largest, below float32's own
//   rounding, at 2.7 times the rate of the fp32 instruction.
// The terms of Inf, of |v| past the largest bf16 (rounded) and, below 2^-110, of
// the smallest floats are not v, and an infinite sum over channel frequencies says
// nothing of the channels.  A column that comes out NaN or Inf, and the matrix of a
// float32 operand that is tiny throughout (Seen), are formed again in float32 by the
// final sum (exact_column).  For that the float32 kernels look at every operand:
// 28.6 -> 30.6 us on 2 slices of 36864 x 64, and 4.8 -> 5.5 us for the sum.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "whtmix_launch.h"
#include "whtmix_module.h"
#include "whtmix_plan.h"
#include "whtmix_tile.h"

namespace whtmix {
namespace {

using namespace tile;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A staged plane of dY / X: [channel][2^NB chunks of 8 tokens], in 16-byte
// units.  Column j of the product's column block n is channel NNB j + n, so
// that the chunks of a channel can be permuted by j alone: the 16 lanes of an
// operand read (one chunk, one n) fall on different 16-byte bank groups and
// n is a constant offset; the transposing writes, whose lanes hold different
// j, spread the same way.  Rows of fewer than 16 chunks are shifted besides.
template <int NB, int CB>
struct Plane {
    static constexpr int NNB = 1 << (CB - 4);
    __host__ __device__ static constexpr uint32_t at(uint32_t j, uint32_t n, uint32_t chunk)
    {
        constexpr uint32_t mask = NB < 4 ? (1u << NB) - 1u : 15u;
        const uint32_t row = ((j << (CB - 4)) | n) << NB;
        return row + (NB < 4 ? ((j >> NB) << NB) : 0u) + (chunk ^ (j & mask));
    }
    static constexpr uint32_t UNITS =
        (16u << (CB - 4 + NB)) + (NB < 4 ? ((15u >> NB) << NB) : 0u);
};

// LDS of a workgroup whose tiles lie as W (Wg, Wd below).  The tile of dY / X is
// transposed: [channel][8-token chunk] of bf16 with the chunks of a channel permuted
// (Plane).  float32 takes three such planes (the three-term split), half of the tokens
// at a time where there are two k steps or more.  One region per tile serves the
// exchange and the planes, one after the other, and the teams' sums at the end.
template <class W, typename T>
struct Staged {
    static constexpr int ROUNDS = sizeof(T) == 2 || W::RT == 3 ? 1 : 2;
    static constexpr int CHUNK_BITS = W::NCHB - (ROUNDS - 1);
    static constexpr uint32_t WORDS =
        (sizeof(T) == 2 ? 1u : 3u) * 4u * Plane<CHUNK_BITS, W::CBITS>::UNITS;
    static constexpr uint32_t REGION = ((W::XCH > WORDS ? W::XCH : WORDS) + 3u) & ~3u;
    static constexpr uint32_t SUMS = W::TEAMS > 1 ? (uint32_t)(W::C * W::C) : 0u;
    static constexpr uint32_t LDS = REGION << W::E > SUMS ? REGION << W::E : SUMS;
};

// Waves per SIMD of the product kernels, for their launch bounds.
template <int A, int CB, typename T>
constexpr int waves_per_simd()
{
    return wgrad_waves(A, CB, sizeof(T) == 2 ? DTYPE_BF16 : DTYPE_F32);
}

// How a 2^A tile of C = 2^CB channels lies in the waves for the products: lane
// 16 q + i of the MFMA operand holds channel 16 strip + i and, per k step,
// eight consecutive tokens of group q.
//   lanes 0-3   channel bits 0-3
//   lanes 4-5   token bits RT, RT+1 (q)
//   registers   SR channel bits (the strips a wave holds), then token bits
//               0 .. RT-1
//   waves       SW channel bits from 4, then the remaining token bits
// Workgroups have at least 8 waves: 2^E tiles of fewer waves go side by side.
template <int A, int CB>
struct Wg {
    static constexpr int CBITS = CB, C = 1 << CB;
    static constexpr int TW = A - 11;                  // wave bits of one tile
    static constexpr int SB = CB - 4;                  // strip bits
    static constexpr int SW = SB < TW ? SB : TW;
    static constexpr int SR = SB - SW;
    static constexpr int RT = VB - SR;
    static constexpr int REM = A - VB - CB;            // token bits below layout A-5
    static constexpr int WB = wgrad_wave_bits(A, CB);  // wave bits of the workgroup
    static constexpr int E = wgrad_group_bits(A, CB);
    static constexpr uint32_t THREADS = 64u << WB;
    static constexpr uint32_t TEAMS = 1u << (WB - SW); // wave sets covering all strips
    static constexpr int NNB = C / 16;
    static constexpr int NS = 1 << SR;                 // strips per wave
    static constexpr int NCHB = A - CB - 3;            // log2 of 8-token chunks per tile
    static constexpr int QB = CB + RT;                 // tile bit of q

    // LDS words of the exchange: one pad word per 32, and the four token
    // groups q 16 banks apart so that the product layout's reads (16
    // consecutive words per group) cover 64 banks.  (The shift grows with
    // every bit from q up, so at() is injective.)
    static constexpr uint32_t SHIFT = (16u - (1u << (QB - 5))) & 63u;
    __host__ __device__ static constexpr uint32_t at(uint32_t t)
    {
        return t + (t >> 5) + SHIFT * (t >> QB);
    }
    static constexpr uint32_t XCH = (1u << A) + (1u << (A - 5)) + SHIFT * ((1u << (A - QB)) - 1u);
    __device__ static uint32_t base(uint32_t t)   // thread t of the tile
    {
        const uint32_t lane = t & 63u, w = t >> 6;
        return (lane & 15u) | ((w & ((1u << SW) - 1u)) << 4) | ((lane >> 4) << QB) |
               ((w >> SW) << (QB + 2));
    }
    __host__ __device__ static constexpr uint32_t reg(uint32_t k)
    {
        return ((k & ((1u << SR) - 1u)) << (4 + SW)) | ((k >> SR) << CB);
    }
};

template <bool EXACT>
__device__ __forceinline__ void split3(const float (&z)[8], bf16x8 &hi, bf16x8 &mid, bf16x8 &lo)
{
    u32x4 h, m, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t a, b, c;
        split3_pair<EXACT>(z[2 * e], z[2 * e + 1], a, b, c);
        h[e] = a;
        m[e] = b;
        l[e] = c;
    }
    hi = __builtin_bit_cast(bf16x8, h);
    mid = __builtin_bit_cast(bf16x8, m);
    lo = __builtin_bit_cast(bf16x8, l);
}

// The magnitudes of a float32 operand, or-ed: no bit from 2^28 up is set where all
// are below 2^-95, whose splits may lose bits that matter.  (Against larger ones a
// tiny value's loss, 2^-134 at most, is below the sum's own rounding.)
struct Seen {
    uint32_t x = 0u, z = 0u;
    static constexpr uint32_t LARGE = 0x70000000u, ANY = 0x7fffffffu;
    template <int N>
    __device__ __forceinline__ void add_z(const float (&v)[N])
    {
#pragma unroll
        for (int k = 0; k < N; ++k)
            z |= as_u32(v[k]);
        asm volatile("" : "+v"(z));   // here, before the values are split
    }
    template <int N>
    __device__ __forceinline__ void add_x(const u32x4 (&v)[N])
    {
#pragma unroll
        for (int k = 0; k < N; ++k)
            x |= (v[k][0] | v[k][1]) | (v[k][2] | v[k][3]);
        asm volatile("" : "+v"(x));
    }
    // bit 0, 1: a large x, any x; bit 2, 3: z.  One word per wave.
    __device__ __forceinline__ void store(uint32_t *word) const
    {
        const auto some = [](uint32_t v) { return __builtin_amdgcn_ballot_w64(v != 0u) != 0u; };
        *word = (some(x & LARGE) ? 1u : 0u) | (some(x & ANY) ? 2u : 0u) |
                (some(z & LARGE) ? 4u : 0u) | (some(z & ANY) ? 8u : 0u);
    }
    // of all words or-ed
    __device__ static bool tiny(uint32_t words)
    {
        return (words & 3u) == 2u || (words & 12u) == 8u;
    }
};

// acc += a b over k steps [s0, s1) of a round (a: the lane's float operand, b:
// the staged planes; rs0 the round's first step).  Steps go in groups whose
// split operand takes 48 registers, the registers of 32 values and a half.
// Each group's sum is formed from zero, the leading product apart from the
// others, and added to the running sum in float32: a chain of accumulations
// in the matrix unit rounds at every step at the size of the running sum,
// which measured up to twice the error of the sums it replaces.
template <typename T, int CB, int NB, int RT, int SR, int S0, int S1, int NS, int NNB, int VV>
__device__ __forceinline__ void multiply(f32x4 (&acc)[NS][NNB], const float (&v)[VV],
                                         const float *region, uint32_t j, uint32_t chunk0)
{
    constexpr bool F32 = sizeof(T) == 4;
    constexpr uint32_t PLANE = Plane<NB, CB>::UNITS;
    constexpr int GS = S1 - S0 < 4 / NS ? S1 - S0 : 4 / NS;
    static_assert(GS >= 1 && (S1 - S0) % GS == 0, "whole groups of k steps");
    const bf16x8 *xb = reinterpret_cast<const bf16x8 *>(region);
#pragma unroll
    for (int s0 = S0; s0 < S1; s0 += GS) {
        bf16x8 a0[GS][NS], a1[GS][NS], a2[GS][NS];
        const bf16x8 *col[GS];
#pragma unroll
        for (int g = 0; g < GS; ++g) {
            col[g] = xb + Plane<NB, CB>::at(j, 0, chunk0 | (uint32_t)(s0 - S0 + g));
#pragma unroll
            for (int sr = 0; sr < NS; ++sr) {
                float z[8];
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    z[e] = v[sr | ((8 * (s0 + g) + e) << SR)];
                split3<!F32>(z, a0[g][sr], a1[g][sr], a2[g][sr]);
            }
        }
#pragma unroll
        for (int n = 0; n < NNB; ++n) {
            f32x4 lead[NS], rest[NS];
#pragma unroll
            for (int sr = 0; sr < NS; ++sr)
                lead[sr] = rest[sr] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int g = 0; g < GS; ++g) {
                const bf16x8 b0 = col[g][n << NB];
                bf16x8 b1, b2;
                if constexpr (F32) {
                    b1 = col[g][(n << NB) + PLANE];
                    b2 = col[g][(n << NB) + 2u * PLANE];
                }
#pragma unroll
                for (int sr = 0; sr < NS; ++sr) {
                    f32x4 d = rest[sr];
                    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2[g][sr], b0, d, 0, 0, 0);
                    if constexpr (F32) {
                        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[g][sr], b2, d, 0, 0, 0);
                        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1[g][sr], b1, d, 0, 0, 0);
                    }
                    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1[g][sr], b0, d, 0, 0, 0);
                    if constexpr (F32)
                        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[g][sr], b1, d, 0, 0, 0);
                    rest[sr] = d;
                    lead[sr] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[g][sr], b0, lead[sr], 0, 0, 0);
                }
            }
#pragma unroll
            for (int sr = 0; sr < NS; ++sr)
                acc[sr][n] += lead[sr] + rest[sr];
            __builtin_amdgcn_sched_barrier(0);   // few operand reads in registers at a time
        }
    }
}

// The workgroup's sums: lane 16 q + j holds rows a = 16 strip + 4 q + [0, 4) of
// column b = NNB j + n, strip = strip0 | sr << SW.  The teams' sums are added
// in team order through LDS and stored to part[blockIdx.x][b][a].
template <int C, int NS, int NNB, int SW, int CB>
__device__ __forceinline__ void store_sums(f32x4 (&acc)[NS][NNB], float *lds,
                                           float *__restrict__ part, uint32_t team,
                                           uint32_t teams, uint32_t strip0, uint32_t lane)
{
    const uint32_t j = lane & 15u, q = lane >> 4;
    const auto at = [&](int sr, int n) {
        return (((uint32_t)NNB * j + n) << CB) + 16u * (strip0 | ((uint32_t)sr << SW)) + 4u * q;
    };
    for (uint32_t k = 1; k < teams; ++k) {
        __syncthreads();
        if (team == k) {
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int n = 0; n < NNB; ++n)
                    *reinterpret_cast<f32x4 *>(lds + at(s, n)) = acc[s][n];
        }
        __syncthreads();
        if (team == 0) {
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int n = 0; n < NNB; ++n)
                    acc[s][n] += *reinterpret_cast<const f32x4 *>(lds + at(s, n));
        }
    }
    if (team == 0) {
        float *out = part + ((size_t)blockIdx.x << (2 * CB));
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int n = 0; n < NNB; ++n)
                *reinterpret_cast<f32x4 *>(out + at(s, n)) = acc[s][n];
    }
}

// The thread's share of a tile of dY / X (valid elements, a multiple of C;
// rows past it read as zero): 32 elements in 16-byte pieces.  bf16: channels
// 8 cg + [0, 8) of tokens 4 u + i.  float32: channels 4 cg + [0, 4) of tokens
// 4 u + i of either half of the tokens (token bit RT-1, which u leaves out).
template <int A, int CB, typename T>
__device__ __forceinline__ void load_x(u32x4 (&xr)[V * sizeof(T) / 16], const T *tile,
                                       uint32_t valid, uint32_t t)
{
    using W = Wg<A, CB>;
    const __amdgpu_buffer_rsrc_t r = buffer(tile, valid * (uint32_t)sizeof(T));
    constexpr int LV = sizeof(T) == 2 ? 3 : 2;   // log2 of elements per piece
    const uint32_t cg = t & ((1u << (CB - LV)) - 1u);
    uint32_t u = t >> (CB - LV);
    if constexpr (sizeof(T) == 4)
        u = (u & ((1u << (W::RT - 3)) - 1u)) | ((u >> (W::RT - 3)) << (W::RT - 2));
    const uint32_t e0 = (u << (CB + 2)) + (cg << LV);
#pragma unroll
    for (uint32_t h = 0; h < sizeof(T) / 2; ++h) {
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            const uint32_t off = (i << CB) + (h << (CB + W::RT - 1));
            u32x4 d = {0u, 0u, 0u, 0u};
            if (e0 + off < valid)
                d = __builtin_bit_cast(
                    u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                               r, e0 * (uint32_t)sizeof(T), off * (uint32_t)sizeof(T), kStreaming));
            xr[4 * h + i] = d;
        }
    }
}

// Transposing writes of a piece group (channels 2^LV cg + [0, 2^LV) of the
// four tokens 4 quad + i, LV = 3 for bf16, 2 for float32): 8 bytes of four
// tokens per channel, into the three planes of the split for float32.
template <int NB, int CB, typename T>
__device__ __forceinline__ void stage_quad(float *lds, const u32x4 *x, uint32_t cg, uint32_t quad)
{
    constexpr int LV = sizeof(T) == 2 ? 3 : 2, NNB = 1 << (CB - 4);
    constexpr uint32_t PLANE = 16u * Plane<NB, CB>::UNITS;
    char *const base = reinterpret_cast<char *>(lds) + 8u * (quad & 1u);
#pragma unroll
    for (uint32_t i = 0; i < (1u << LV); ++i) {
        // channel 2^LV cg + i = NNB j + n
        uint32_t j, n;
        if constexpr (NNB >= (1 << LV)) {
            j = cg / (NNB >> LV);
            n = ((cg & ((NNB >> LV) - 1u)) << LV) + i;
        } else {
            j = cg * ((1u << LV) / NNB) + i / NNB;
            n = i % NNB;
        }
        char *d = base + 16u * (Plane<NB, CB>::at(j, 0, quad >> 1) + (n << NB));
        if constexpr (sizeof(T) == 2) {
            const uint32_t w = i >> 1;
            u32x2 o;
            if (i & 1u) {
                o[0] = high_halves(x[0][w], x[1][w]);
                o[1] = high_halves(x[2][w], x[3][w]);
            } else {
                o[0] = __builtin_amdgcn_perm(x[1][w], x[0][w], 0x05040100u);
                o[1] = __builtin_amdgcn_perm(x[3][w], x[2][w], 0x05040100u);
            }
            *reinterpret_cast<u32x2 *>(d) = o;
        } else {
            u32x2 p0, p1, p2;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                uint32_t a, b, c;
                split3_pair<false>(as_f32(x[2 * k][i]), as_f32(x[2 * k + 1][i]), a, b, c);
                p0[k] = a;
                p1[k] = b;
                p2[k] = c;
            }
            *reinterpret_cast<u32x2 *>(d) = p0;
            *reinterpret_cast<u32x2 *>(d + PLANE) = p1;
            *reinterpret_cast<u32x2 *>(d + 2u * PLANE) = p2;
        }
    }
}

// Round h of the staged tile (float32 in one round: both halves).
template <int A, int CB, typename T>
__device__ __forceinline__ void stage_x(float *lds, const u32x4 (&xr)[V * sizeof(T) / 16],
                                        uint32_t t, [[maybe_unused]] int h)
{
    using W = Wg<A, CB>;
    constexpr int NB = Staged<W, T>::CHUNK_BITS;
    constexpr int LV = sizeof(T) == 2 ? 3 : 2;
    const uint32_t cg = t & ((1u << (CB - LV)) - 1u), u = t >> (CB - LV);
    if constexpr (sizeof(T) == 2) {
        stage_quad<NB, CB, T>(lds, xr, cg, u);
    } else if constexpr (Staged<W, T>::ROUNDS == 1) {
        // u gets its missing bit back (RT = 3: bit 0)
#pragma unroll
        for (uint32_t hh = 0; hh < 2; ++hh)
            stage_quad<NB, CB, T>(lds, xr + 4 * hh, cg, (u << 1) | hh);
    } else {
        stage_quad<NB, CB, T>(lds, xr + 4 * h, cg, u);
    }
}

// Workgroups [0, nwg) form dW_out from (wsx, dy), the next nwg dW_in from
// (wsd, x).  Workgroup p takes tile groups p, p + nwg, ... and stores its sum
// as part[p][b][a], a the workspace's channel (still a channel frequency), b
// the channel of dY / X.
template <int A, int HB, int R, typename T, int CB>
__global__ void __launch_bounds__((Wg<A, CB>::THREADS), (waves_per_simd<A, CB, T>()))
wgrad_tiles_kernel(const float *__restrict__ wsx, const T *__restrict__ dy,
                   const float *__restrict__ wsd, const T *__restrict__ x,
                   float *__restrict__ part, uint32_t *__restrict__ seen_words, uint32_t nvalid,
                   uint32_t live, uint32_t ntiles, uint32_t nwg)
{
    using W = Wg<A, CB>;
    using Run = RunMap<HB, R>;
    constexpr int C = W::C, NNB = W::NNB, NS = W::NS;
    __shared__ __attribute__((aligned(16))) float lds[Staged<W, T>::LDS];
    const uint32_t tau = threadIdx.x;
    const uint32_t t = tau & ((1u << (A - VB)) - 1u);   // thread of the tile
    const uint32_t lane = tau & 63u;
    // wave-uniform: which tile of the group, which strips and tokens of it
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tau >> 6);
    const uint32_t sub = wave >> W::TW;
    const uint32_t tw = (wave & ((1u << W::TW) - 1u)) >> W::SW;
    float *const region = lds + sub * Staged<W, T>::REGION;
    const bool second = blockIdx.x >= nwg;
    const uint32_t p = blockIdx.x - (second ? nwg : 0u);
    const float *ws = second ? wsd : wsx;
    const T *xs = second ? x : dy;
    // tiles that hold real rows: `live` per slice, numbered through the batch
    const uint32_t ngroups = (ntiles + (1u << W::E) - 1u) >> W::E;
    const auto locate = [&](uint32_t g, size_t &b, uint32_t &hi) -> uint32_t {
        const uint32_t i = (g << W::E) | sub;
        // past the last tile: tile 0 again, none of its rows real
        const bool past = W::E > 0 && i >= ntiles;
        const uint32_t sl = past ? 0u : i / live;
        b = sl;
        hi = past ? 0u : i - sl * live;
        return past ? 0u : tile_valid<A>(nvalid, hi);
    };

    f32x4 acc[NS][NNB];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int n = 0; n < NNB; ++n)
            acc[s][n] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};

    // The next group's dY / X (bf16) is loaded once this group's is staged and
    // its workspace registers after the products, ahead of the next exchange.
    constexpr int ROUNDS = Staged<W, T>::ROUNDS, STEPS = 1 << (W::RT - 3);
    constexpr int NB = Staged<W, T>::CHUNK_BITS;
    [[maybe_unused]] Seen seen;   // float32
    float v[V];
    u32x4 xr[V * sizeof(T) / 16];
    size_t b;
    uint32_t hi;
    uint32_t valid = locate(p, b, hi);
    const uint32_t voff = Run::at(layout_base<A - VB>(t)) * 4u;
    const auto load_ws = [&]() {
        const __amdgpu_buffer_rsrc_t r =
            buffer(ws + (b << (A + HB)) + ((size_t)hi << R), extent_bytes<Run, A, float>());
#pragma unroll
        for (int k = 0; k < V; ++k)
            v[k] = Elt<float>::load(r, voff, Run::at((uint32_t)k << (A - VB)) * 4u);
    };
    constexpr bool PREFETCH_X = sizeof(T) == 2;   // float32: 32 registers more
    if constexpr (PREFETCH_X)
        load_x<A, CB, T>(xr, xs + b * nvalid + ((size_t)hi << A), valid, t);
    load_ws();
#pragma unroll 1
    for (uint32_t g = p; g < ngroups; g += nwg) {   // uniform over the workgroup
        const bool more = g + nwg < ngroups;
        const bool real = W::E == 0 || valid > 0;
#pragma unroll
        for (int k = 0; k < V; ++k)
            v[k] = real ? v[k] : 0.0f;
        // token bits [A-5, A), then [CB, A-5) in the product layout
        butterflies<0, VB>(v);
        __syncthreads();   // the previous group's product reads are done
        {
            const uint32_t pa = W::at(layout_base<A - VB>(t));
#pragma unroll
            for (int k = 0; k < V; ++k)
                region[pa + W::at((uint32_t)k << (A - VB))] = v[k];
            if constexpr (!PREFETCH_X)   // the registers are free until the read
                load_x<A, CB, T>(xr, xs + b * nvalid + ((size_t)hi << A), valid, t);
            __syncthreads();
            const uint32_t pb = W::at(W::base(t));
#pragma unroll
            for (int k = 0; k < V; ++k)
                v[k] = region[pb + W::at(W::reg((uint32_t)k))];
        }
        butterflies<W::SR, W::SR + W::REM>(v);
        if constexpr (sizeof(T) == 4) {
            seen.add_z(v);
            seen.add_x(xr);
        }
        // opaque per group: the operand and staging addresses are cheap to form
        // and, hoisted out of the loop, would take some forty registers
        uint32_t ln = lane, tt = t;
        asm volatile("" : "+v"(ln), "+v"(tt));
        const uint32_t j = ln & 15u, q = ln >> 4;
        const auto round = [&](auto H) {
            constexpr int h = decltype(H)::value;
            __syncthreads();   // exchange reads, or the previous round's, are done
            stage_x<A, CB, T>(region, xr, tt, h);
            if (h == ROUNDS - 1 && more) {
                valid = locate(g + nwg, b, hi);
                if constexpr (PREFETCH_X)
                    load_x<A, CB, T>(xr, xs + b * nvalid + ((size_t)hi << A), valid, t);
            }
            __syncthreads();
            // k step s: tokens 8 s + [0, 8) of each group q
            constexpr int SB2 = W::RT - 3 - (ROUNDS - 1);   // step bits of a round
            multiply<T, CB, NB, W::RT, W::SR, h * STEPS / ROUNDS, (h + 1) * STEPS / ROUNDS>(
                acc, v, region, j, (q << SB2) | (tw << (SB2 + 2)));
        };
        round(std::integral_constant<int, 0>{});
        if constexpr (ROUNDS == 2)
            round(std::integral_constant<int, 1>{});
        if (more)
            load_ws();
    }

    store_sums<C, NS, NNB, W::SW, CB>(acc, lds, part, wave >> W::SW, W::TEAMS,
                                      wave & ((1u << W::SW) - 1u), lane);
    if constexpr (sizeof(T) == 4)
        seen.store(seen_words + (blockIdx.x << W::WB) + wave);
}

// ---------------------------------------------------------------- direct form
// Where the waves of a tile hold nothing but channel strips (2^6 values per
// lane at most), no token bit lies across waves and the tile needs no exchange
// at all: every lane loads its values straight in a product layout,
//   lanes 0-3   channel bits 0-3        (64-byte pieces of the runs)
//   lanes 4-5   token bits 0, 1
//   waves       SW channel bits from 4
//   registers   SR channel bits, then token bits RT, RT+1, 2 .. RT-1,
// transforms the RT token bits in its registers, and trades token bits 0 and
// 1 for RT and RT+1 between lanes 4-5 and registers (v_permlane16/32_swap) to
// transform those too.  That ends in the product layout above with q = token
// bits RT, RT+1.  LDS holds the staged dY / X only.  On 2 slices of 36864 x 64
// float32 (2^14 tiles, 64 values per lane) it took 26.7 us against 29.1 us for
// the form with the exchange, on 2^14 tiles of C = 128 97.5 against 97.7 us (both
// before the operand addresses and splits were cut down).
template <int A, int CB>
struct Wd {
    static constexpr int CBITS = CB, C = 1 << CB;
    static constexpr int TW = A - 11;
    static constexpr int SB = CB - 4;
    static constexpr int SW = SB < TW ? SB : TW;       // wave bits of a tile
    static constexpr int SR = SB - SW;
    static constexpr int LB = A - 6 - SW;              // log2 of values per lane
    static constexpr int VV = 1 << LB;
    static constexpr int RT = LB - SR;
    static constexpr int WB = wgrad_wave_bits(A, CB);  // wave bits of the workgroup
    static constexpr int E = wgrad_group_bits(A, CB);
    static constexpr uint32_t THREADS = 64u << WB;
    static constexpr uint32_t TEAMS = 1u << E;
    static constexpr int NNB = C / 16;
    static constexpr int NS = 1 << SR;
    static constexpr int NCHB = A - CB - 3;
    static_assert(A - CB == RT + 2, "every token bit in a lane or its registers");
    static constexpr uint32_t XCH = 0;   // no exchange
    // 16-byte pieces of dY / X a thread stages per round
    template <typename T>
    static constexpr int pieces()
    {
        return VV * (int)sizeof(T) / 16 / Staged<Wd, T>::ROUNDS;
    }

    __device__ static uint32_t base(uint32_t lane, uint32_t strips)
    {
        return (lane & 15u) | (strips << 4) | ((lane >> 4) << CB);
    }
    __host__ __device__ static constexpr uint32_t reg(uint32_t k)
    {
        const uint32_t tok = k >> SR;
        return ((k & ((1u << SR) - 1u)) << (4 + SW)) | ((tok & 3u) << (CB + RT)) |
               ((tok >> 2) << (CB + 2));
    }
};

// Butterflies over register bits [J0, J1) of VV values.
template <int J0, int J1, int VV>
__device__ __forceinline__ void bfly(float (&v)[VV])
{
#pragma unroll
    for (int j = J0; j < J1; ++j) {
#pragma unroll
        for (int k = 0; k < VV; ++k) {
            if (!(k & (1 << j))) {
                const float a = v[k], b = v[k | (1 << j)];
                v[k] = a + b;
                v[k | (1 << j)] = a - b;
            }
        }
    }
}

// Trades lane bit 4 (W = 16) or 5 (W = 32) for register bit J.
template <int W, int J, int VV>
__device__ __forceinline__ void swap_lane_bit(float (&v)[VV])
{
#pragma unroll
    for (int k = 0; k < VV; ++k) {
        if (!(k & (1 << J))) {
            const uint32_t a = __builtin_bit_cast(uint32_t, v[k]);
            const uint32_t b = __builtin_bit_cast(uint32_t, v[k | (1 << J)]);
            if constexpr (W == 16) {
                const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
                v[k] = __builtin_bit_cast(float, (uint32_t)r[0]);
                v[k | (1 << J)] = __builtin_bit_cast(float, (uint32_t)r[1]);
            } else {
                const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
                v[k] = __builtin_bit_cast(float, (uint32_t)r[0]);
                v[k | (1 << J)] = __builtin_bit_cast(float, (uint32_t)r[1]);
            }
        }
    }
}

// Round h of the thread's dY / X pieces.  Piece group m (four pieces): channels
// 2^LV cg + [0, 2^LV) of tokens 4 quad + i, quad = (t >> (CB - LV)) + m * QS
// of the round's half of the tokens (two rounds: token bit RT-1 is the round).
template <int A, int CB, typename T>
struct StageX {
    using W = Wd<A, CB>;
    static constexpr int LV = sizeof(T) == 2 ? 3 : 2;
    static constexpr int ROUNDS = Staged<W, T>::ROUNDS;
    static constexpr int NP = W::template pieces<T>();
    static constexpr int NM = NP / 4;
    static constexpr uint32_t QS = (64u << W::SW) >> (CB - LV);   // quads per pass of the threads
    static_assert(6 + W::SW >= CB - LV, "a tile's threads cover a row of pieces");
    static_assert(NP % 4 == 0, "whole groups of four tokens");

    // the quad of the tile (all tokens) from the round's quad
    __device__ static uint32_t full(uint32_t quad, int h)
    {
        if constexpr (ROUNDS == 1)
            return quad;
        constexpr int B = W::RT - 3;   // quad bit of token bit RT-1
        return (quad & ((1u << B) - 1u)) | ((uint32_t)h << B) | ((quad >> B) << (B + 1));
    }
    template <bool WHOLE>
    __device__ static void load_rows(u32x4 (&xr)[NP], const T *tile, uint32_t valid, uint32_t t,
                                     int h)
    {
        const __amdgpu_buffer_rsrc_t r = buffer(tile, valid * (uint32_t)sizeof(T));
        const uint32_t cg = t & ((1u << (CB - LV)) - 1u), q0 = t >> (CB - LV);
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const uint32_t e0 = (full(q0 + m * QS, h) << (CB + 2)) + (cg << LV);
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i)
                if (WHOLE || e0 + (i << CB) < valid)
                    xr[4 * m + i] = __builtin_bit_cast(
                        u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                   r, e0 * (uint32_t)sizeof(T), (i << CB) * (uint32_t)sizeof(T),
                                   kStreaming));
                else
                    xr[4 * m + i] = (u32x4){0u, 0u, 0u, 0u};
        }
    }
    // valid real elements of the tile, a multiple of C; rows past it read as zero
    __device__ static void load(u32x4 (&xr)[NP], const T *tile, uint32_t valid, uint32_t t, int h)
    {
        if (valid >= (1u << A))   // uniform over the wave
            load_rows<true>(xr, tile, valid, t, h);
        else
            load_rows<false>(xr, tile, valid, t, h);
    }
    __device__ static void stage(float *lds, const u32x4 (&xr)[NP], uint32_t t)
    {
        const uint32_t cg = t & ((1u << (CB - LV)) - 1u), q0 = t >> (CB - LV);
#pragma unroll
        for (int m = 0; m < NM; ++m)
            stage_quad<Staged<W, T>::CHUNK_BITS, CB, T>(lds, xr + 4 * m, cg, q0 + m * QS);
    }
};

template <int A, int HB, int R, typename T, int CB>
__global__ void __launch_bounds__((Wd<A, CB>::THREADS), (waves_per_simd<A, CB, T>()))
wgrad_direct_kernel(const float *__restrict__ wsx, const T *__restrict__ dy,
                    const float *__restrict__ wsd, const T *__restrict__ x,
                    float *__restrict__ part, uint32_t *__restrict__ seen_words, uint32_t nvalid,
                    uint32_t live, uint32_t ntiles, uint32_t nwg)
{
    using W = Wd<A, CB>;
    using X = StageX<A, CB, T>;
    using Run = RunMap<HB, R>;
    constexpr int C = W::C, NNB = W::NNB, NS = W::NS, VV = W::VV;
    __shared__ __attribute__((aligned(16))) float lds[Staged<W, T>::LDS];
    const uint32_t tau = threadIdx.x;
    const uint32_t t = tau & ((64u << W::SW) - 1u);   // thread of the tile
    const uint32_t lane = tau & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tau >> 6);
    const uint32_t team = wave >> W::SW;              // tile of the group
    const uint32_t strip0 = wave & ((1u << W::SW) - 1u);
    float *const region = lds + team * Staged<W, T>::REGION;
    const bool second = blockIdx.x >= nwg;
    const uint32_t p = blockIdx.x - (second ? nwg : 0u);
    const float *ws = second ? wsd : wsx;
    const T *xs = second ? x : dy;
    const uint32_t ngroups = (ntiles + (1u << W::E) - 1u) >> W::E;
    const auto locate = [&](uint32_t g, size_t &b, uint32_t &hi) -> uint32_t {
        const uint32_t i = (g << W::E) | team;
        // past the last tile: tile 0 again, none of its rows real
        const bool past = W::E > 0 && i >= ntiles;
        const uint32_t sl = past ? 0u : i / live;
        b = sl;
        hi = past ? 0u : i - sl * live;
        return past ? 0u : tile_valid<A>(nvalid, hi);
    };

    f32x4 acc[NS][NNB];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int n = 0; n < NNB; ++n)
            acc[s][n] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};

    constexpr int ROUNDS = X::ROUNDS, STEPS = 1 << (W::RT - 3);
    constexpr int NB = Staged<W, T>::CHUNK_BITS;
    [[maybe_unused]] Seen seen;   // float32
    float v[VV];
    u32x4 xr[X::NP];
    size_t b;
    uint32_t hi;
    uint32_t valid = locate(p, b, hi);
    const uint32_t voff = Run::at(W::base(lane, strip0)) * 4u;
    const auto load_ws = [&]() {
        const __amdgpu_buffer_rsrc_t r =
            buffer(ws + (b << (A + HB)) + ((size_t)hi << R), extent_bytes<Run, A, float>());
#pragma unroll
        for (int k = 0; k < VV; ++k)
            v[k] = Elt<float>::load(r, voff, Run::at(W::reg((uint32_t)k)) * 4u);
    };
    X::load(xr, xs + b * nvalid + ((size_t)hi << A), valid, t, 0);
    load_ws();
#pragma unroll 1
    for (uint32_t g = p; g < ngroups; g += nwg) {   // uniform over the workgroup
        const bool more = g + nwg < ngroups;
        const bool real = W::E == 0 || valid > 0;
        // opaque per group: the operand and staging addresses are cheap to form
        // and, hoisted out of the loop, would take some forty registers
        uint32_t ln = lane, tt = t;
        asm volatile("" : "+v"(ln), "+v"(tt));
        const uint32_t j = ln & 15u, q = ln >> 4;
        const auto round = [&](auto H) {
            constexpr int h = decltype(H)::value;
            __syncthreads();   // the previous round's product reads are done
            if constexpr (sizeof(T) == 4)
                seen.add_x(xr);
            X::stage(region, xr, tt);
            // the next round's pieces, or the next group's
            if (h + 1 < ROUNDS) {
                X::load(xr, xs + b * nvalid + ((size_t)hi << A), valid, tt, h + 1);
            } else if (more) {
                valid = locate(g + nwg, b, hi);
                X::load(xr, xs + b * nvalid + ((size_t)hi << A), valid, tt, 0);
            }
            if constexpr (h == 0) {
#pragma unroll
                for (int k = 0; k < VV; ++k)
                    v[k] = real ? v[k] : 0.0f;
                bfly<W::SR, W::LB>(v);
                swap_lane_bit<16, W::SR>(v);
                swap_lane_bit<32, W::SR + 1>(v);
                bfly<W::SR, W::SR + 2>(v);
                if constexpr (sizeof(T) == 4)
                    seen.add_z(v);
            }
            __syncthreads();
            // k step s: tokens 8 s + [0, 8) of each group q
            constexpr int SB2 = W::RT - 3 - (ROUNDS - 1);   // step bits of a round
            multiply<T, CB, NB, W::RT, W::SR, h * STEPS / ROUNDS, (h + 1) * STEPS / ROUNDS>(
                acc, v, region, j, q << SB2);
        };
        round(std::integral_constant<int, 0>{});
        if constexpr (ROUNDS == 2)
            round(std::integral_constant<int, 1>{});
        if (more)
            load_ws();
    }
    store_sums<C, NS, NNB, W::SW, CB>(acc, lds, part, team, W::TEAMS, strip0, lane);
    if constexpr (sizeof(T) == 4)
        seen.store(seen_words + (blockIdx.x << W::WB) + wave);
}

// Bits [J, S + 5) of the transform of the 2^A tile in LDS (pad(t)), J >= S.
template <int A, int S, int J>
__device__ __forceinline__ void transform_window(float *lds, uint32_t tau)
{
    for (uint32_t i = tau; i < (1u << (A - VB)); i += 256u) {
        const uint32_t at = pad(layout_base<S>(i));
        float v[V];
#pragma unroll
        for (int k = 0; k < V; ++k)
            v[k] = lds[at + pad((uint32_t)k << S)];
        butterflies<J - S, VB>(v);
#pragma unroll
        for (int k = 0; k < V; ++k)
            lds[at + pad((uint32_t)k << S)] = v[k];
    }
    __syncthreads();
}

__device__ __forceinline__ bool not_finite(float v)
{
    return (as_u32(v) & 0x7f800000u) == 0x7f800000u;
}

// Column `col` of dW in float32 as the formulas have it: tiles inverse-transformed
// whole, their rows times their elements of dY / X.  Returns element tau of the
// column (tau < C).  z_finite: Z' (dZ) is finite throughout, so that a column that
// is not has its infinities and NaN from dY / X, and only the tiles that hold them
// are looked at; otherwise, or if there are none, every tile.  A column that is NaN
// throughout ends the loop.  Rare, so simple rather than fast: the backward of 4 x
// 65536 x 128 bf16 takes 2.5 ms with one Inf in dY (0.4 without), of 2 x 36864 x 64
// float32 0.4 ms; with operands that are tiny throughout, 6.8 ms.
template <int CB, int A, typename T>
__device__ float exact_column(float *lds, float *xcol, const float *ws, const T *xs, uint32_t col,
                              bool z_finite, uint32_t nvalid, uint32_t live, uint32_t nslices,
                              int HB, int R, uint32_t tau)
{
    constexpr uint32_t C = 1u << CB, G = 256u / C, TOKENS = 1u << (A - CB);
    const uint32_t a = tau & (C - 1u), g = tau >> CB;
    float total = 0.0f;
    bool found = false, ended = false;
    for (uint32_t pass = z_finite ? 0u : 1u; pass < 2u && !found && !ended; ++pass) {
        for (uint32_t i = 0; i < nslices * live && !ended; ++i) {   // uniform
            const uint32_t b = i / live, hi = i - b * live;
            const T *x = xs + (size_t)b * nvalid + ((size_t)hi << A) + col;
            const uint32_t tokens = tile_valid<A>(nvalid, hi) >> CB;
            bool bad = false;
            __syncthreads();   // the previous tile's readers
            for (uint32_t n = tau; n < TOKENS; n += 256u) {
                const float v = n < tokens ? (float)x[(size_t)n << CB] : 0.0f;
                xcol[n] = v;
                bad |= not_finite(v);
            }
            const bool some = __syncthreads_or(bad);
            if (pass == 0u && !some)
                continue;
            found |= some;
            const float *src = ws + ((size_t)b << (A + HB)) + ((size_t)hi << R);
#pragma unroll 8
            for (uint32_t t = tau; t < (1u << A); t += 256u)
                lds[pad(t)] = src[((size_t)(t >> R) << (HB + R)) | (t & ((1u << R) - 1u))];
            __syncthreads();
            transform_window<A, 0, 0>(lds, tau);
            transform_window<A, 5, 5>(lds, tau);
            transform_window<A, A - VB, 10>(lds, tau);
            float s = 0.0f;
            for (uint32_t n = g; n < tokens; n += G)
                s = fmaf(lds[pad((n << CB) | a)], xcol[n], s);
            total += s;
            ended = __syncthreads_and(total != total);
        }
    }
    __syncthreads();
    lds[tau] = total;
    __syncthreads();
    float v = 0.0f;
    for (uint32_t k = 0; k < G; ++k)
        v += lds[k * C + a];
    return v;
}

// Block b < C: column b of dW_out, block C + b: row b of dW_in.  Adds the
// nwg partial vectors part[p][b][0 .. C) in a fixed order (each of the 1024/C
// thread groups takes every (1024/C)-th, then the groups in order) and applies
// the channel inverse the tiles left out, over a.
template <int CB, int A, typename T>
__global__ void __launch_bounds__(256)
wgrad_final_kernel(const float *__restrict__ part, const uint32_t *__restrict__ seen_words,
                   float *__restrict__ dw_out, float *__restrict__ dw_in, uint32_t nwg,
                   uint32_t nwords, const float *__restrict__ wsx, const T *__restrict__ dy,
                   const float *__restrict__ wsd, const T *__restrict__ x, uint32_t nvalid,
                   uint32_t live, uint32_t nslices, int HB, int R)
{
    constexpr uint32_t C = 1u << CB, G = 1024u / C;
    static_assert(pad(1u << A) >= 1024u, "LDS holds either use");
    __shared__ __attribute__((aligned(16))) float red[pad(1u << A)];
    __shared__ uint32_t found[4];
    __shared__ float xcol[1u << (A - CB)];
    const uint32_t tau = threadIdx.x;
    const bool second = blockIdx.x >= C;
    const uint32_t b = blockIdx.x & (C - 1u);
    const uint32_t a4 = tau & (C / 4u - 1u), pg = tau / (C / 4u);
    uint32_t words = 0u;
    if constexpr (sizeof(T) == 4) {
        for (uint32_t i = tau; i < nwords; i += 256u)
            words |= seen_words[(second ? nwords : 0u) + i];
    }
    const auto column_sums = [&](uint32_t col) {
        const f32x4 *src = reinterpret_cast<const f32x4 *>(
                               part + (((size_t)(second ? nwg : 0u)) << (2 * CB)) +
                               ((size_t)col << CB)) +
                           a4;
        constexpr uint32_t STRIDE = C * C / 4u;   // f32x4 per partial matrix
        f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
        uint32_t p = pg;
        for (; p + 7u * G < nwg; p += 8u * G) {
            f32x4 u[8];
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i)
                u[i] = src[(size_t)(p + i * G) * STRIDE];
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i)
                s += u[i];
        }
        for (; p < nwg; p += G)
            s += src[(size_t)p * STRIDE];
        return s;
    };
    const f32x4 s = column_sums(b);
    *reinterpret_cast<f32x4 *>(red + pg * C + 4u * a4) = s;
    __syncthreads();
    float v = 0.0f;
    if (tau < C) {
        for (uint32_t k = 0; k < G; ++k)
            v += red[k * C + tau];
    }
    for (uint32_t h = 1; h < C; h <<= 1) {
        __syncthreads();
        if (tau < C)
            red[tau] = v;
        __syncthreads();
        if (tau < C) {
            const float o = red[tau ^ h];
            v = (tau & h) ? o - v : v + o;
        }
    }
    // bits 0-3: Seen's; bit 4: NaN or Inf in the column
    if (tau < C && not_finite(v))
        words |= 16u;
    uint32_t all = 0u;
#pragma unroll
    for (uint32_t i = 0; i < 5u; ++i)
        all |= __builtin_amdgcn_ballot_w64((words >> i) & 1u) != 0u ? 1u << i : 0u;
    if ((tau & 63u) == 0u)
        found[tau >> 6] = all;
    __syncthreads();
    all = (found[0] | found[1]) | (found[2] | found[3]);
    const bool tiny = sizeof(T) == 4 && Seen::tiny(all);
    if (__builtin_expect((all & 16u) || tiny, 0)) {
        // A row of Z' (dZ) that is not finite leaves no column finite: one finite
        // neighbour shows that there is none.
        bool z_finite = false;
        for (uint32_t k = 1; k <= 8u && !z_finite && !tiny; ++k) {
            const f32x4 u = column_sums((b + k) & (C - 1u));
            z_finite = !__syncthreads_or(not_finite(u[0]) || not_finite(u[1]) ||
                                         not_finite(u[2]) || not_finite(u[3]));
        }
        v = exact_column<CB, A, T>(red, xcol, second ? wsd : wsx, second ? x : dy, b, z_finite,
                                   nvalid, live, nslices, HB, R, tau);
    }
    if (tau < C) {
        if (second)
            dw_in[(b << CB) | tau] = v;
        else
            dw_out[(tau << CB) | b] = v;
    }
}

template <typename T, int K, int CB>
hipError_t launch_k(const WgradTilesArgs &a)
{
    constexpr Split sp = module_split(K);
    if constexpr (wgrad_tiles_shape(sp.A, CB)) {
        const uint32_t live = wgrad_live_tiles(K, a.nvalid);
        const uint32_t ntiles = (uint32_t)a.B * live;
        const uint32_t nwg = wgrad_tiles_parts(K, CB, a.dtype, a.B, a.nvalid);
        const T *x = static_cast<const T *>(a.x), *dy = static_cast<const T *>(a.dy);
        uint32_t *words = reinterpret_cast<uint32_t *>(a.part + 2 * ((size_t)nwg << (2 * CB)));
        uint32_t wave_bits;
        if constexpr (wgrad_direct_shape(sp.A, CB)) {
            wave_bits = Wd<sp.A, CB>::WB;
            hipLaunchKernelGGL((wgrad_direct_kernel<sp.A, sp.HB, sp.R, T, CB>), dim3(2u * nwg),
                               dim3(Wd<sp.A, CB>::THREADS), 0, a.stream, a.wsx, dy, a.wsd, x,
                               a.part, words, a.nvalid, live, ntiles, nwg);
        } else {
            wave_bits = Wg<sp.A, CB>::WB;
            hipLaunchKernelGGL((wgrad_tiles_kernel<sp.A, sp.HB, sp.R, T, CB>), dim3(2u * nwg),
                               dim3(Wg<sp.A, CB>::THREADS), 0, a.stream, a.wsx, dy, a.wsd, x,
                               a.part, words, a.nvalid, live, ntiles, nwg);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((wgrad_final_kernel<CB, sp.A, T>), dim3(2u << CB), dim3(256), 0,
                           a.stream, a.part, words, a.dw_out, a.dw_in, nwg, nwg << wave_bits,
                           a.wsx, dy, a.wsd, x, a.nvalid, live, (uint32_t)a.B, sp.HB, sp.R);
        return hipGetLastError();
    } else {
        return hipErrorInvalidValue;
    }
}

template <typename T, int CB>
hipError_t launch_cb(const WgradTilesArgs &a)
{
    switch (a.K) {
#define WHTMIX_WT_CASE(k) \
    case k: return launch_k<T, k, CB>(a);
        WHTMIX_WT_CASE(12) WHTMIX_WT_CASE(13) WHTMIX_WT_CASE(14) WHTMIX_WT_CASE(15)
        WHTMIX_WT_CASE(16) WHTMIX_WT_CASE(17) WHTMIX_WT_CASE(18) WHTMIX_WT_CASE(19)
        WHTMIX_WT_CASE(20) WHTMIX_WT_CASE(21) WHTMIX_WT_CASE(22) WHTMIX_WT_CASE(23)
        WHTMIX_WT_CASE(24) WHTMIX_WT_CASE(25)
#undef WHTMIX_WT_CASE
    default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t launch_t(const WgradTilesArgs &a)
{
    switch (a.cbits) {
    case 4: return launch_cb<T, 4>(a);
    case 5: return launch_cb<T, 5>(a);
    case 6: return launch_cb<T, 6>(a);
    case 7: return launch_cb<T, 7>(a);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_wgrad_tiles(const WgradTilesArgs &a)
{
    return a.dtype == DTYPE_BF16 ? launch_t<__bf16>(a) : launch_t<float>(a);
}

}  // namespace whtmix
