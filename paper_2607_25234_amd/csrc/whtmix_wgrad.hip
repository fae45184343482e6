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
// So a tile costs one read of the workspace, one of dY (X), one LDS exchange,
// the splits and the products.
//
// Products (float32 accumulation), Z' / dZ rows against dY / X columns:
//   v_mfma_f32_16x16x32_bf16 on three-term bf16 splits of the float operand
//   (residual below 2^-27 of each value) against bf16 dY / X, exact, or
//   against the same split of float32 dY / X: the six products down to 2^-25
//   of the largest, below float32's own rounding, at 2.7 times the rate of the
//   fp32 instruction.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "whtmix_launch.h"
#include "whtmix_module.h"
#include "whtmix_plan.h"
#include "whtmix_tile.h"

namespace whtmix {
namespace {

using namespace tile;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

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
    static constexpr int C = 1 << CB;
    static constexpr int TW = A - 11;                  // wave bits of one tile
    static constexpr int SB = CB - 4;                  // strip bits
    static constexpr int SW = SB < TW ? SB : TW;
    static constexpr int SR = SB - SW;
    static constexpr int RT = VB - SR;
    static constexpr int REM = A - VB - CB;            // token bits below layout A-5
    static constexpr int WB = TW > 3 ? TW : 3;         // wave bits of the workgroup
    static constexpr int E = WB - TW;
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
    // The tile of dY / X, transposed: [channel][8-token chunk] of bf16 with the
    // chunks of a channel permuted (swz).  float32 takes three such planes (the
    // three-term split), half of the tokens at a time where there are two k
    // steps or more.
    template <typename T>
    static constexpr int rounds() { return sizeof(T) == 2 || RT == 3 ? 1 : 2; }
    template <typename T>
    static constexpr int chunk_bits() { return rounds<T>() == 1 ? NCHB : NCHB - 1; }
    template <typename T>
    static constexpr uint32_t plane_bytes() { return (2u << A) / rounds<T>(); }
    template <typename T>
    static constexpr uint32_t xwords()
    {
        return (sizeof(T) == 2 ? 1u : 3u) * plane_bytes<T>() / 4u;
    }
    // One region serves both, one after the other.
    template <typename T>
    static constexpr uint32_t region()
    {
        const uint32_t w = XCH > xwords<T>() ? XCH : xwords<T>();
        return (w + 3u) & ~3u;
    }
    template <typename T>
    static constexpr uint32_t lds_words()
    {
        const uint32_t w = region<T>() << E;
        const uint32_t cc = TEAMS > 1 ? (uint32_t)C * C : 0u;   // team sums at the end
        return w > cc ? w : cc;
    }
    // Chunk permutation of a plane with 2^NB chunks per channel: the 16 lanes
    // of an operand read (consecutive channels, one chunk) and, from 16 chunks,
    // of a transposing write (every eighth channel) fall on different 16-byte
    // bank groups.
    // Bitwise linear: swz(a | b) = swz(a) ^ swz(b) for disjoint a, b.
    template <int NB>
    __host__ __device__ static constexpr uint32_t swz(uint32_t c)
    {
        constexpr int sh = NB < 4 ? 4 - NB : 0;
        constexpr uint32_t mask = NB < 4 ? (1u << NB) - 1u : 15u;
        return ((c >> sh) ^ (c >> 3)) & mask;
    }
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

// Three-term bf16 split of eight floats: v = hi + mid + lo + d, each term the
// nearest bf16 of what the previous ones leave, |d| <= 2^-27 |v|.
__device__ __forceinline__ void split3(const float (&z)[8], bf16x8 &hi, bf16x8 &mid, bf16x8 &lo)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const __bf16 h = (__bf16)z[e];
        const float r1 = z[e] - (float)h;
        const __bf16 m = (__bf16)r1;
        hi[e] = h;
        mid[e] = m;
        lo[e] = (__bf16)(r1 - (float)m);
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

// Round h of the staged tile: 8-byte writes of four tokens of a channel
// (float32 in one round: both halves).
template <int A, int CB, typename T>
__device__ __forceinline__ void stage_x(float *lds, const u32x4 (&xr)[V * sizeof(T) / 16],
                                        uint32_t t, [[maybe_unused]] int h)
{
    using W = Wg<A, CB>;
    constexpr int NB = W::template chunk_bits<T>();
    constexpr int LV = sizeof(T) == 2 ? 3 : 2;
    const uint32_t cg = t & ((1u << (CB - LV)) - 1u), u = t >> (CB - LV);
    char *const base = reinterpret_cast<char *>(lds);
    if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) {
            const uint32_t w = i >> 1;
            u32x2 d;
            if (i & 1u) {
                d[0] = (xr[0][w] >> 16) | (xr[1][w] & 0xffff0000u);
                d[1] = (xr[2][w] >> 16) | (xr[3][w] & 0xffff0000u);
            } else {
                d[0] = (xr[0][w] & 0xffffu) | (xr[1][w] << 16);
                d[1] = (xr[2][w] & 0xffffu) | (xr[3][w] << 16);
            }
            *reinterpret_cast<u32x2 *>(
                base + 16u * ((cg << (NB + 3)) + (i << NB) +
                              (((u >> 1) ^ W::template swz<NB>(8u * cg)) ^ W::template swz<NB>(i))) +
                8u * (u & 1u)) = d;
        }
    } else {
        constexpr uint32_t PLANE = W::template plane_bytes<T>();
        constexpr int ROUNDS = W::template rounds<T>();
#pragma unroll
        for (int hh = ROUNDS == 1 ? 0 : h; hh < (ROUNDS == 1 ? 2 : h + 1); ++hh) {
            // in one round u gets its missing bit back (RT = 3: bit 0)
            const uint32_t quad = ROUNDS == 1 ? (u << 1) | (uint32_t)hh : u;
            f32x4 row[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                row[i] = __builtin_bit_cast(f32x4, xr[4 * hh + i]);
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) {
                bf16x4 p0, p1, p2;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float z = row[k][i];
                    const __bf16 hi = (__bf16)z;
                    const float r1 = z - (float)hi;
                    const __bf16 mid = (__bf16)r1;
                    p0[k] = hi;
                    p1[k] = mid;
                    p2[k] = (__bf16)(r1 - (float)mid);
                }
                char *d = base +
                          16u * ((cg << (NB + 2)) + (i << NB) +
                                 (((quad >> 1) ^ W::template swz<NB>(4u * cg)) ^
                                  W::template swz<NB>(i))) +
                          8u * (quad & 1u);
                *reinterpret_cast<bf16x4 *>(d) = p0;
                *reinterpret_cast<bf16x4 *>(d + PLANE) = p1;
                *reinterpret_cast<bf16x4 *>(d + 2u * PLANE) = p2;
            }
        }
    }
}

// Workgroups [0, nwg) form dW_out from (wsx, dy), the next nwg dW_in from
// (wsd, x).  Workgroup p takes tile groups p, p + nwg, ... and stores its sum
// as part[p][b][a], a the workspace's channel (still a channel frequency), b
// the channel of dY / X.
template <int A, int HB, int R, typename T, int CB>
__global__ void __launch_bounds__((Wg<A, CB>::THREADS), (Wg<A, CB>::NS == 1 ? 4 : 2))
wgrad_tiles_kernel(const float *__restrict__ wsx, const T *__restrict__ dy,
                   const float *__restrict__ wsd, const T *__restrict__ x,
                   float *__restrict__ part, uint32_t nvalid, uint32_t live, uint32_t ntiles,
                   uint32_t nwg)
{
    using W = Wg<A, CB>;
    using Run = RunMap<HB, R>;
    constexpr int C = W::C, NNB = W::NNB, NS = W::NS;
    __shared__ __attribute__((aligned(16))) float lds[W::template lds_words<T>()];
    const uint32_t tau = threadIdx.x;
    const uint32_t t = tau & ((1u << (A - VB)) - 1u);   // thread of the tile
    const uint32_t lane = tau & 63u;
    // wave-uniform: which tile of the group, which strips and tokens of it
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tau >> 6);
    const uint32_t sub = wave >> W::TW;
    const uint32_t tw = (wave & ((1u << W::TW) - 1u)) >> W::SW;
    float *const region = lds + sub * W::template region<T>();
    const bool second = blockIdx.x >= nwg;
    const uint32_t p = blockIdx.x - (second ? nwg : 0u);
    const float *ws = second ? wsd : wsx;
    const T *xs = second ? x : dy;
    // tiles that hold real rows: `live` per slice, numbered through the batch
    const uint32_t ngroups = (ntiles + (1u << W::E) - 1u) >> W::E;
    const auto locate = [&](uint32_t g, size_t &b, uint32_t &hi) -> uint32_t {
        const uint32_t i = (g << W::E) | sub;
        const uint32_t sl = i / live;
        b = sl;
        hi = i - sl * live;
        return i < ntiles ? tile_valid<A>(nvalid, hi) : 0u;
    };

    f32x4 acc[NS][NNB];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int n = 0; n < NNB; ++n)
            acc[s][n] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};

    // The next group's dY / X (bf16) is loaded once this group's is staged and
    // its workspace registers after the products, ahead of the next exchange.
    constexpr int ROUNDS = W::template rounds<T>(), STEPS = 1 << (W::RT - 3);
    constexpr int NB = W::template chunk_bits<T>();
    float v[V];
    u32x4 xr[V * sizeof(T) / 16];
    size_t b;
    uint32_t hi;
    uint32_t valid = locate(p, b, hi);
    const uint32_t voff = Run::at(layout_base<A - VB>(t)) * 4u;
    const auto load_ws = [&](size_t bb, uint32_t hh, bool any) {
        const __amdgpu_buffer_rsrc_t r =
            buffer(ws + (bb << (A + HB)) + ((size_t)hh << R), extent_bytes<Run, A, float>());
#pragma unroll
        for (int k = 0; k < V; ++k)
            v[k] = W::E == 0 || any ? Elt<float>::load(r, voff, Run::at((uint32_t)k << (A - VB)) * 4u) : 0.0f;
    };
    constexpr bool PREFETCH_X = sizeof(T) == 2;   // float32: 32 registers more
    if constexpr (PREFETCH_X)
        load_x<A, CB, T>(xr, xs + b * nvalid + ((size_t)hi << A), valid, t);
    load_ws(b, hi, valid > 0);
    for (uint32_t g = p; g < ngroups; g += nwg) {   // uniform over the workgroup
        const bool more = g + nwg < ngroups;
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
        // opaque per group: the operand and staging addresses are cheap to form
        // and, hoisted out of the loop, would take some forty registers
        uint32_t ln = lane, tt = t;
        asm volatile("" : "+v"(ln), "+v"(tt));
        const uint32_t j = ln & 15u, q = ln >> 4;
        const bf16x8 *xb = reinterpret_cast<const bf16x8 *>(region);
#pragma unroll
        for (int h = 0; h < ROUNDS; ++h) {
            __syncthreads();   // exchange reads, or the previous round's, are done
            stage_x<A, CB, T>(region, xr, tt, h);
            if (h == ROUNDS - 1 && more) {
                valid = locate(g + nwg, b, hi);
                if constexpr (PREFETCH_X)
                    load_x<A, CB, T>(xr, xs + b * nvalid + ((size_t)hi << A), valid, t);
            }
            __syncthreads();
#pragma unroll
            for (int s = h * STEPS / ROUNDS; s < (h + 1) * STEPS / ROUNDS; ++s) {
                // k step: tokens 8 s + [0, 8) of each group q
                const uint32_t sh = (uint32_t)(s - h * STEPS / ROUNDS);
                const uint32_t chunk = ROUNDS == 1
                                           ? (uint32_t)s | (q << (W::RT - 3)) | (tw << (W::RT - 1))
                                           : sh | (q << (W::RT - 4)) | (tw << (W::RT - 2));
                const uint32_t xo = chunk ^ W::template swz<NB>(j);
                bf16x8 a0[NS], a1[NS], a2[NS];
#pragma unroll
                for (int sr = 0; sr < NS; ++sr) {
                    float z[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        z[e] = v[sr | ((8 * s + e) << W::SR)];
                    split3(z, a0[sr], a1[sr], a2[sr]);
                }
#pragma unroll
                for (int n = 0; n < NNB; ++n) {
                    const bf16x8 *src =
                        xb + (j << NB) + (xo ^ W::template swz<NB>(16u * n)) + (16u * n << NB);
                    const bf16x8 b0 = src[0];
                    bf16x8 b1, b2;
                    if constexpr (sizeof(T) == 4) {
                        b1 = src[W::template plane_bytes<T>() / 16u];
                        b2 = src[W::template plane_bytes<T>() / 8u];
                    }
#pragma unroll
                    for (int sr = 0; sr < NS; ++sr) {
                        f32x4 d = acc[sr][n];
                        if constexpr (sizeof(T) == 4) {   // products down to 2^-25 of the largest
                            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2[sr], b0, d, 0, 0, 0);
                            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[sr], b2, d, 0, 0, 0);
                            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1[sr], b1, d, 0, 0, 0);
                            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1[sr], b0, d, 0, 0, 0);
                            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[sr], b1, d, 0, 0, 0);
                            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[sr], b0, d, 0, 0, 0);
                        } else {
                            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2[sr], b0, d, 0, 0, 0);
                            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1[sr], b0, d, 0, 0, 0);
                            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[sr], b0, d, 0, 0, 0);
                        }
                        acc[sr][n] = d;
                    }
                    if (n % 2 == 1)   // few operand reads in registers at a time
                        __builtin_amdgcn_sched_barrier(0);
                }
                __builtin_amdgcn_sched_barrier(0);   // later steps' splits stay below
            }
        }
        if (more)
            load_ws(b, hi, valid > 0);
    }

    // lane 16 q + j holds rows a = 16 strip + 4 q + [0, 4) of column b = 16 n + j;
    // the teams' sums are added in team order through LDS
    const uint32_t j = lane & 15u, q = lane >> 4;
    const uint32_t team = wave >> W::SW;
    const uint32_t strip0 = wave & ((1u << W::SW) - 1u);
    const auto at = [&](int sr, int n) {
        return ((16u * n + j) << CB) + 16u * (strip0 | ((uint32_t)sr << W::SW)) + 4u * q;
    };
    for (uint32_t k = 1; k < W::TEAMS; ++k) {
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

// Block b < C: column b of dW_out, block C + b: row b of dW_in.  Adds the
// nwg partial vectors part[p][b][0 .. C) in a fixed order (each of the 1024/C
// thread groups takes every (1024/C)-th, then the groups in order) and applies
// the channel inverse the tiles left out, over a.
template <int CB>
__global__ void __launch_bounds__(256)
wgrad_final_kernel(const float *__restrict__ part, float *__restrict__ dw_out,
                   float *__restrict__ dw_in, uint32_t nwg)
{
    constexpr uint32_t C = 1u << CB, G = 1024u / C;
    __shared__ __attribute__((aligned(16))) float red[1024];
    const uint32_t tau = threadIdx.x;
    const bool second = blockIdx.x >= C;
    const uint32_t b = blockIdx.x & (C - 1u);
    const uint32_t a4 = tau & (C / 4u - 1u), pg = tau / (C / 4u);
    const f32x4 *src = reinterpret_cast<const f32x4 *>(
                           part + (((size_t)(second ? nwg : 0u)) << (2 * CB)) + ((size_t)b << CB)) +
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
        using W = Wg<sp.A, CB>;
        const uint32_t live = wgrad_live_tiles(K, a.nvalid);
        const uint32_t ntiles = (uint32_t)a.B * live;
        const uint32_t nwg = wgrad_tiles_parts(K, CB, a.B, a.nvalid);
        hipLaunchKernelGGL((wgrad_tiles_kernel<sp.A, sp.HB, sp.R, T, CB>), dim3(2u * nwg),
                           dim3(W::THREADS), 0, a.stream, a.wsx, static_cast<const T *>(a.dy),
                           a.wsd, static_cast<const T *>(a.x), a.part, a.nvalid, live, ntiles, nwg);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((wgrad_final_kernel<CB>), dim3(2u << CB), dim3(256), 0, a.stream,
                           a.part, a.dw_out, a.dw_in, nwg);
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
