// Weight gradients of narrow layers (at most 32 outputs: the last layer of a few classes).
//
// [dW ; db] = [A 1]^T dZ has one column of tiles and a sum as short as the minibatch: what a launch takes is a chain of trips to
// memory on a chip that is nearly idle.  A wavefront owns sixteen rows and all columns; its lanes load the operands of
// v_mfma_f32_16x16x4_f32 straight from memory (A and dZ are both contiguous along what the lanes run over), sixteen values
// of each in flight, together with the replica, center and momentum values of its epilogue: one trip for a minibatch of 64, no
// LDS, no barrier.  An element is the chain of fused multiply-adds in ascending k that the other fp32 tiles compute: same bits.
// Bound: latency.  784->10, 4 workers, 64 rows with the momentum rule 7.0 us (128x32 tile through LDS) -> 4.2; 2048->10, 32, 100
// 16.4 -> 10.2.
#pragma once
#include "gemm_mfma.h"

namespace easgd {

// TN: tiles of sixteen columns.  A block of four wavefronts owns 64 rows.
template <int TN, int EPI>
__device__ __forceinline__ void narrow_dw_block(const GemmArgs &p, const unsigned bid)
{
    constexpr bool ELASTIC = (EPI == EPI_ELASTIC || EPI == EPI_ELASTIC_MOM || EPI == EPI_ELASTIC_MOM_BF16);
    constexpr bool MOM = (EPI == EPI_ELASTIC_MOM), MOM16 = (EPI == EPI_ELASTIC_MOM_BF16), OUT16 = (EPI == EPI_STORE_BF16);
    constexpr int CH = 16;                               // matrix instructions, of four k each, per trip to memory
    BlockTile bt;
    if (!block_tile(p, bid, bt)) return;
    const int w = __builtin_amdgcn_readfirstlane(bt.w);
    const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
    const int mw = __builtin_amdgcn_readfirstlane(bt.tile_m) * 64 + 16 * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (mw >= p.M) return;                               // uniform; no barrier follows
    // lane l supplies A[m = l%16][k + l/16] and dZ[k + l/16][n = l%16] of each matrix instruction; rows and columns outside the
    // operands are read from the nearest one inside, and only reach elements that are not stored
    const bool one = mw + l16 == p.a_ones;               // the row that sums dZ up
    const float *__restrict__ A = p.A + (size_t)w * p.a_ws + min(mw + l16, p.a_lim - 1);
    const float *__restrict__ B[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) B[j] = p.B + (size_t)w * p.b_ws + min(16 * j + l16, p.N - 1);

    float a[CH], b[TN][CH];
    auto load = [&](int k0) {
        if (k0 + 4 * CH <= p.K) {                        // uniform
#pragma unroll
            for (int e = 0; e < CH; ++e) {
                const size_t k = (size_t)(k0 + 4 * e + q);
                a[e] = A[k * p.lda];
#pragma unroll
                for (int j = 0; j < TN; ++j) b[j][e] = B[j][k * p.ldb];
            }
        } else {
#pragma unroll
            for (int e = 0; e < CH; ++e) {
                const size_t k = (size_t)min(k0 + 4 * e + q, p.K - 1);
                a[e] = A[k * p.lda];
#pragma unroll
                for (int j = 0; j < TN; ++j) b[j][e] = B[j][k * p.ldb];
            }
        }
    };
    load(0);
    // the epilogue's tiles: register r of lane l is C[4*(l/16) + r][l%16]
    float *__restrict__ Wr = ELASTIC ? p.Wt + (size_t)w * p.c_ws : nullptr;
    float *__restrict__ Vr = MOM ? p.Vt + (size_t)w * p.c_ws : nullptr;
    unsigned short *__restrict__ Vr16 = MOM16 ? p.Vt16 + (size_t)w * p.c_ws : nullptr;
    float wv[TN][4], cv[TN][4], vv[TN][4];
    unsigned v16[TN][4];                                 // one register per code
    (void)wv; (void)cv; (void)vv; (void)v16;
    if constexpr (ELASTIC) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const size_t at = (size_t)min(mw + 4 * q + r, p.M - 1) * p.ldc + min(16 * j + l16, p.N - 1);
                wv[j][r] = Wr[at];
                cv[j][r] = p.center[at];
                if constexpr (MOM) vv[j][r] = Vr[at];
                if constexpr (MOM16) v16[j][r] = Vr16[at];
            }
    }
    f32x4 acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < p.K; k0 += 4 * CH) {
        float ca[CH], cb[TN][CH];
#pragma unroll
        for (int e = 0; e < CH; ++e) {
            const bool in = k0 + 4 * e + q < p.K;        // always, but for the end of the sum
            ca[e] = !in ? 0.f : one ? 1.f : a[e];
#pragma unroll
            for (int j = 0; j < TN; ++j) cb[j][e] = in ? b[j][e] : 0.f;
        }
        if (k0 + 4 * CH < p.K) load(k0 + 4 * CH);
#pragma unroll
        for (int e = 0; e < CH; ++e)
            if (k0 + 4 * e < p.K) {                      // uniform
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ca[e], cb[j][e], acc[j], 0, 0, 0);
            }
    }
    const bool keep = !OUT16 && (!ELASTIC || p.C != nullptr);                         // uniform
    float *__restrict__ C = keep ? p.C + (size_t)w * p.c_ws : nullptr;
    unsigned short *__restrict__ C16 = OUT16 ? p.C16 + (size_t)w * p.c_ws : nullptr;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = 16 * j + l16;
        if (n >= p.N) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = mw + 4 * q + r;
            if (m >= p.M) continue;
            const size_t at = (size_t)m * p.ldc + n;
            const float g = acc[j][r];
            if constexpr (ELASTIC) {
                float x = wv[j][r];
                if constexpr (MOM16) {
                    unsigned short v = (unsigned short)v16[j][r];
                    worker_rule_bf16<true>(x, v, g, cv[j][r], p.eta, p.rho, p.alpha, p.delta);
                    Vr16[at] = v;
                } else {
                    float v = MOM ? vv[j][r] : 0.f;
                    worker_rule<MOM>(x, v, g, cv[j][r], p.eta, p.rho, p.alpha, p.delta);
                    if constexpr (MOM) Vr[at] = v;
                }
                Wr[at] = x;
            }
            if constexpr (OUT16) C16[at] = bf16_narrow(g);
            else if (keep) C[at] = g;
        }
    }
}

template <int TN, int EPI>
__global__ __launch_bounds__(256) void narrow_dw_kernel(GemmArgs p)
{
    if (p.mean.blocks > 0 && blockIdx.x >= p.mean.first_block) mean_loss_block(p.mean, blockIdx.x - p.mean.first_block);
    else narrow_dw_block<TN, EPI>(p, blockIdx.x);
}

}  // namespace easgd
