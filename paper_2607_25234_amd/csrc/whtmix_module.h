// Internal interface between the C entry points and the kernels of the whole
// block with its projections (whtmix_module.hip).
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "whtmix_launch.h"
#include "whtmix_plan.h"

namespace whtmix {

// ---------------------------------------------------------------- the block
// How the block with its projections runs (whtmix_module.hip):
//   SMALL       the mixer's SMALL plan, projections on the VALU in LDS;
//   FUSED_MFMA  16 <= C <= 128 with the FUSED or THREE_PASS plan, and bf16
//               C = 256 with the THREE_PASS plan from 2^17 elements per slice
//               (2^16 outer tiles): MFMA prologue and epilogue inside the
//               mixer's kernels;
//   UNFUSED     any other C: projection kernels around the fp32 mixer.
enum ModulePath { MODULE_SMALL = 0, MODULE_FUSED_MFMA = 1, MODULE_UNFUSED = 2 };
constexpr int kModuleMfmaMinCbits = 4;
constexpr int kModuleMfmaMaxCbits = 7;
constexpr int kModuleMaxCbits = 12;   // weights of C*C elements, C <= 4096

inline int module_path(int plan, int cbits, int dtype, int K)
{
    if (plan == PLAN_SMALL) return MODULE_SMALL;
    if (cbits >= kModuleMfmaMinCbits && cbits <= kModuleMfmaMaxCbits) return MODULE_FUSED_MFMA;
    if (cbits == kPairModuleCbits && dtype == DTYPE_BF16 && plan == PLAN_THREE_PASS &&
        K >= kPairModuleMinK)
        return MODULE_FUSED_MFMA;
    return MODULE_UNFUSED;
}

// Flat-index bits of the outer passes of the block's THREE_PASS plan.
inline int module_outer_bits(int path, int cbits, int K)
{
    if (path == MODULE_FUSED_MFMA)
        return cbits == kPairModuleCbits ? pair_split(K).A : module_split(K).A;
    return three_pass_split(K).A;   // UNFUSED: the mixer's own plan
}

// Bytes of one repacked weight matrix.  The projections inside the mixer's
// kernels up to C = 128 read the weights as they lie in memory.
inline int64_t module_packed_bytes(int cbits, int dtype)
{
    return int64_t(dtype == DTYPE_BF16 ? 2 : 4) << (2 * cbits);
}
inline bool module_packs_weights(int path, int cbits)
{
    return path == MODULE_UNFUSED || (path == MODULE_FUSED_MFMA && cbits > kModuleMfmaMaxCbits);
}

// Except that a thousand one-wave workgroups and more, each with a matrix eight
// times its tile, read a matrix repacked once per call: bf16, C = 128, 2^11 outer
// tiles.  The packing launch takes 3 to 5 us; at 512 x 128 and 1024 x 128 tokens the
// forward takes 17.9 us packed and 18.1 with the weights as they lie at 512 tiles,
// 28.1 and 28.7 at 1024, 36.6 and 38.8 at 2048, 189 and 218 at 16384, the backward
// 62.3 and 61.8, 78.8 and 80.5, 111 and 117, 532 and 553.
constexpr int64_t kModulePackTiles = 1024;
constexpr bool module_packs_shape(int A, int cbits) { return A == 11 && cbits == 7; }
inline bool module_packs_for_tiles(int dtype, int cbits, int K, int64_t B)
{
    const Split sp = module_split(K);
    return dtype == DTYPE_BF16 && module_packs_shape(sp.A, cbits) &&
           (B << sp.HB) >= kModulePackTiles;
}

// A validated call of the block.  Workspace: the THREE_PASS workspace `ws`
// (B * 2^K floats, else none), then for UNFUSED `z` (B * N * C floats), then
// `wpack` (the two repacked weight matrices, where module_packs_weights).
struct ModuleArgs {
    const void *x;
    const void *w_in;       // [C][C], dtype of x
    const void *w_out;      // [C][C]
    void *y;
    int gain_kind;          // GainKind
    const float *gain;
    const float *gain_t;
    const float *gain_c;
    int cbits;
    float *ws;
    void *wpack;
    float *z;
    int64_t B;
    int K;
    uint32_t nvalid;
    int dtype;
    int plan;
    hipStream_t stream;
    hipEvent_t events[4];   // FUSED_MFMA three-pass: around each of the three
                            // passes; otherwise [0] before, [1] after
};

hipError_t launch_module(const ModuleArgs &m);

// ---------------------------------------------------------------- backward
// Split of a weight gradient dW = A^T B over rows (A, B [rows][C]): `chunks`
// partial C x C sums of `rows_per_chunk` rows each, added in a fixed order:
// first in groups of kWgradGroup consecutive chunks, then the group sums.
constexpr uint32_t kWgradGroup = 16;
struct WgradPlan {
    uint32_t chunks;
    uint32_t rows_per_chunk;
    uint32_t groups() const { return (chunks + kWgradGroup - 1) / kWgradGroup; }
    // floats of partial sums: the chunks' and the groups'
    uint64_t partial_floats(int cbits) const
    {
        return (uint64_t)(chunks + groups()) << (2 * cbits);
    }
};

// About 512 workgroups (two per CU) over the chunks and the (C/T)^2 output
// blocks of the matrix-core kernel (T = min(C, 128)), at least 64 rows per
// chunk; C < 16 (the VALU kernel, one block per chunk) the same.
inline WgradPlan wgrad_plan(uint64_t rows, int cbits)
{
    if (rows == 0) return WgradPlan{0, 4};   // no partials: the sums are zero
    const uint64_t C = uint64_t(1) << cbits;
    const uint64_t T = C < 128 ? C : 128;
    const uint64_t blocks = C >= 16 ? (C / T) * (C / T) : 1;
    uint64_t chunks = 512 / blocks;
    if (chunks < 1) chunks = 1;
    const uint64_t most = (rows + 63) / 64;   // at least 64 rows per chunk
    if (chunks > most) chunks = most;
    uint64_t rpc = (rows + chunks - 1) / chunks;
    rpc = (rpc + 3) / 4 * 4;
    if (rpc == 0) rpc = 4;
    return WgradPlan{(uint32_t)((rows + rpc - 1) / rpc), (uint32_t)rpc};
}

// The block's backward runs its projections inside the mixer backward's
// passes (THREE_PASS, when a gain gradient is requested: 16 <= C <= 128 on
// slices up to 2^25 elements, and bf16 C = 256 on 2^26..2^28, where the
// block's and the mixer's splits agree); otherwise as projection kernels
// around the mixer's forward and backward on float32 Z, Z' and dZ'.
inline bool module_backward_fused(int plan, int cbits, int dtype, int K)
{
    if (plan != PLAN_THREE_PASS) return false;
    if (cbits >= kModuleMfmaMinCbits && cbits <= kModuleMfmaMaxCbits) return K >= 12 && K <= 25;
    return dtype == DTYPE_BF16 && cbits == kPairModuleCbits && K >= 26 && K <= 28;
}

// Weight gradients inside the last pass (whtmix_wgrad.hip), for the fused
// backward's tiles of 2^A elements and C = 2^cbits channels: the product
// layout needs three token bits in a lane's registers beside the channel
// strips its wave holds, and every token bit below layout A-5 in registers.
// That is every fused shape but C = 128 on 2^11 tiles (K = 16, 17) and
// C = 16 on 2^15 tiles (K = 24, 25).
constexpr bool wgrad_tiles_shape(int A, int cbits)
{
    const int tw = A - 11, sb = cbits - 4;
    const int rt = 5 - (sb > tw ? sb - tw : 0);
    return rt >= 3 && A - 5 - cbits >= 0 && A - 5 - cbits <= rt;
}

// Outer tiles of one slice that hold real rows (nvalid = N * C).
inline uint32_t wgrad_live_tiles(int K, uint32_t nvalid)
{
    const Split sp = module_split(K);
    return (uint32_t)(((uint64_t)nvalid + (uint64_t(1) << sp.A) - 1) >> sp.A);
}

// The form without an exchange: waves that hold channel strips only, with
// 2^6 values per lane at most.
constexpr bool wgrad_direct_shape(int A, int cbits)
{
    const int tw = A - 11, sb = cbits - 4;
    return wgrad_tiles_shape(A, cbits) && A - 6 - (sb < tw ? sb : tw) <= 6;
}

// log2 of the waves of a workgroup: eight, or as many as a tile has; the direct form
// with 64 values per lane and less than eight strips of waves: four.
constexpr int wgrad_wave_bits(int A, int cbits)
{
    const int tw = A - 11, sb = cbits - 4, sw = sb < tw ? sb : tw;
    if (wgrad_direct_shape(A, cbits))
        return A - 6 - sw > 5 && sw < 3 ? 2 : 3;
    return tw > 3 ? tw : 3;
}

// Waves per SIMD that the registers are held to: four with one strip of channels per
// wave (two with float32 at C = 128, whose operands take more), two with several;
// with 64 values per lane three, or two with eight strips of waves.  (float32, C = 64
// on 2^14 tiles spills 15 registers at three: 28.4 us on 2 slices of 36864 x 64, against
// 32.2 at two without spills and 32.2 and 45 with a half and a quarter of the k steps
// per group.)
constexpr int wgrad_waves(int A, int cbits, int dtype)
{
    const int tw = A - 11, sb = cbits - 4, sw = sb < tw ? sb : tw;
    if (!wgrad_direct_shape(A, cbits))
        return sb > tw ? 2 : 4;
    if (A - 6 - sw > 5)
        return wgrad_wave_bits(A, cbits) == 2 ? 3 : 2;
    return sb > tw || (dtype == DTYPE_F32 && cbits == 7) ? 2 : 4;
}

// log2 of the outer tiles a workgroup takes at a time.
constexpr int wgrad_group_bits(int A, int cbits)
{
    const int tw = A - 11, sb = cbits - 4, sw = sb < tw ? sb : tw;
    return wgrad_wave_bits(A, cbits) - (wgrad_direct_shape(A, cbits) ? sw : tw);
}

// Workgroups (and partial sums) per weight gradient: as many as fit the CUs
// over both, and no more than there are tile groups.  Each adds up its tile
// groups in registers, so its partial C x C matrix is written once.
inline uint32_t wgrad_tiles_parts(int K, int cbits, int dtype, int64_t B, uint32_t nvalid)
{
    const Split sp = module_split(K);
    const int e = wgrad_group_bits(sp.A, cbits);
    const uint64_t groups =
        ((uint64_t)B * wgrad_live_tiles(K, nvalid) + (uint64_t(1) << e) - 1) >> e;
    const uint64_t most =
        128u * (4u * (uint32_t)wgrad_waves(sp.A, cbits, dtype) >> wgrad_wave_bits(sp.A, cbits));
    return (uint32_t)(groups < most ? groups : most);
}

// Floats of `part`: the partial matrices, then (float32) a word per wave about its
// operands.
inline int64_t wgrad_tiles_floats(int K, int cbits, int dtype, int64_t B, uint32_t nvalid)
{
    const int64_t words = dtype == DTYPE_F32 ? 16 : 0;   // waves of a workgroup at most
    return 2 * (int64_t)wgrad_tiles_parts(K, cbits, dtype, B, nvalid) *
           ((int64_t(1) << (2 * cbits)) + words);
}

struct WgradTilesArgs {
    const float *wsx;       // middle pass's output of Z and of dZ'
    const float *wsd;
    const void *x;
    const void *dy;
    float *part;            // wgrad_tiles_floats
    float *dw_in;
    float *dw_out;
    int cbits;
    int64_t B;              // > 0
    int K;                  // 12 .. 25, wgrad_tiles_shape(module_split(K).A, cbits)
    uint32_t nvalid;        // N * C
    int dtype;
    hipStream_t stream;
};

hipError_t launch_wgrad_tiles(const WgradTilesArgs &a);

// A validated backward call of the block.  Workspace pieces (floats unless
// noted): z, zp, dzp [B*N*C] (Z = X W_in, Z' = mixer(Z), dZ' then dZ; unused
// and absent with `tiles`);
// wpack: W_in, W_out^T and W_in^T packed (3*C*C elements of the dtype; absent
// where the fused backward runs with C <= 128);
// wpart: the weight gradients' partial sums (wgrad_plan, or
// wgrad_tiles_floats with `tiles`); mix_ws: the
// THREE_PASS workspace (B * 2^K, else none); bwd_ws: the mixer backward's
// workspace (backward_layout).
struct ModuleBackwardArgs {
    const void *x;
    const void *w_in;
    const void *w_out;
    const void *dy;
    void *dx;               // [B][N][C] dtype
    float *dw_in;           // [C][C]
    float *dw_out;          // [C][C]
    int gain_kind;
    const float *gain;
    const float *gain_t;
    const float *gain_c;
    float *dgain;
    float *dgt;
    float *dgc;
    int cbits;
    int64_t B;
    int K;
    uint32_t nvalid;        // N * C
    int dtype;
    int plan;               // the mixer's plan for [B, N, C]
    hipStream_t stream;
    hipEvent_t events[4];   // [0] before; then after each phase: unfused, [1] Z, Z',
                            // dZ', dW_out, [2] the mixer's gradient, [3] dX and dW_in;
                            // fused, [1] the transforms of Z and dZ' and dG, [2] Z'
                            // and dW_out, [3] dX and dW_in
    bool tiles;             // fused, with the weight gradients inside the last pass
    float *z;
    float *zp;
    float *dzp;
    void *wpack;
    float *wpart;
    float *mix_ws;
    float *bwd_ws;
};

// Whether this call runs the fused backward: the shape (above), a requested
// gain gradient, and a first launch of 2*B*2^K/32 work-items (a 32-bit grid).
inline bool module_backward_fused_call(const ModuleBackwardArgs &m)
{
    const bool want_dg = m.gain_kind == GAIN_LOG_SEPARABLE ? (m.dgt != nullptr)
                                                           : (m.dgain != nullptr);
    return want_dg && m.B > 0 && ((uint64_t)m.B << m.K) / 16u <= 0xffffffffull &&
           module_backward_fused(m.plan, m.cbits, m.dtype, m.K);
}

hipError_t launch_module_backward(const ModuleBackwardArgs &m);

}  // namespace whtmix
