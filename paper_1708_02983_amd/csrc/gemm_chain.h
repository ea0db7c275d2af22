// Products of small grids on the fp32 matrix instruction: the rows are the minibatch (forward, input gradient).
//
// v_mfma_f32_16x16x4_f32, 32x32x2 and 4x4x1 all compute what a chain of fused multiply-adds in ascending k does, bit for bit
// (denormal numbers included; compared on the device), so an element's value depends on the order of k alone and not on the
// tile that it is computed in.  The 64x64 tiles of gemm_mfma.h, with 32x32x2, need 64 cycles for two values of k: a
// product whose grid does not fill the chip takes that long for its whole sum however few tiles there are.  The 16x16x4
// instruction needs 32 cycles for four, and its tile has a quarter of the elements, so that the same product gives work to four
// times as many SIMDs.
//
// Bound: the serial chain of K/4 matrix instructions per wavefront (38 cycles each, since every one waits for the one before),
// then the first trip to memory.  784->500, 8 workers, 50 rows: 18.2 us -> 8.7; 1023->777, 6, 37: 23.2 -> 10.4; 3072->432, 8, 48:
// 59.2 -> 20.8, of which the matrix instructions and their operands from LDS alone take 17.6.  With the LDS accesses of a slab
// in bursts between the matrix instructions instead of one behind each of them that last product takes 26.1.
#pragma once
#include "gemm_mfma.h"

namespace easgd {

typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

// WM x WN = 4 wavefronts, each with TM tiles of 16x16 of C one below the other: a block owns (16*TM*WM) x (16*WN).  A slab is
// 64 values of k.  In LDS an operand that arrives k-contiguous lies in groups of 16 k, [k % 4][row][k / 4 % 4] each: the k of a
// lane's next four matrix instructions (q, q+4, q+8, q+12 of a group) lie next to each other, so that it fetches them with one
// 128-bit read; an operand that arrives n-contiguous stays [k][n].
template <int WM, int WN, int TM, int B_LAYOUT>
struct ChainTile {
    static_assert(WM * WN == 4, "four wavefronts");
    static constexpr int BM = 16 * TM * WM, BN = 16 * WN, BK = 64;
    // floats of a group, padded by 16 so that the scattered stores of a wavefront (four rows, sixteen pieces of four k each)
    // go to 64 different banks
    static constexpr int GA = 16 * BM + 16, GB = 16 * BN + 16;
    static constexpr int PB = BN == 16 ? 16 : BN + 16;               // [k][n]: four rows of k start 16 banks apart
    static constexpr int A_FLOATS = 4 * GA, B_FLOATS = B_LAYOUT == K_CONTIG ? 4 * GB : BK * PB;
    static constexpr int LDS_FLOATS = 2 * (A_FLOATS + B_FLOATS);
    static constexpr int ITA = BM * 16 / 256, ITB = BN * 16 / 256;   // 128-bit loads per thread and slab
    static constexpr int STAGES = ITA + ITB <= 5 ? 4 : 2;            // slabs between memory and LDS, in registers
};

template <int WM, int WN, int TM, int B_LAYOUT, int EPI>
__device__ __forceinline__ void chain_block(const GemmArgs &p, const unsigned bid, float *__restrict__ lds)
{
    typedef ChainTile<WM, WN, TM, B_LAYOUT> T;
    constexpr int BM = T::BM, BN = T::BN, BK = T::BK, ITA = T::ITA, ITB = T::ITB, NS = T::STAGES;
    BlockTile bt;
    if (!block_tile(p, bid, bt)) return;
    const int w = __builtin_amdgcn_readfirstlane(bt.w), split = __builtin_amdgcn_readfirstlane(bt.split);
    const int m0 = __builtin_amdgcn_readfirstlane(bt.tile_m) * BM, n0 = __builtin_amdgcn_readfirstlane(bt.tile_n) * BN;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WN, wn = wave % WN;
    const int k_begin = split * p.k_per_split, k_end = min(p.K, k_begin + p.k_per_split);
    const float *__restrict__ A = p.A + (size_t)w * p.a_ws;
    const float *__restrict__ B = p.B + (size_t)w * p.b_ws;

    // Buffer loads: a 32-bit byte offset per lane, a uniform one per slab, and zeros for what lies behind the operand's end.
    // What runs over a row's end inside the operand brings the next row's values: the last slab replaces them (cut).
    const unsigned a_bytes = 4u * (unsigned)p.M * (unsigned)p.lda, b_bytes = 4u * (unsigned)(B_LAYOUT == K_CONTIG ? p.N : p.K) * (unsigned)p.ldb;
    const int n_slabs = (k_end - k_begin + BK - 1) / BK;
    unsigned a_off[ITA], b_off[ITB];
    int a_dst[ITA], b_dst[ITB];
#pragma unroll
    for (int it = 0; it < ITA; ++it) {
        const int u = tid + it * 256, kq = u & 15, m = u >> 4;
        a_off[it] = 4u * ((unsigned)min(m0 + m, p.M - 1) * (unsigned)p.lda + 4u * (unsigned)kq);
        a_dst[it] = (kq >> 2) * T::GA + 4 * m + (kq & 3);
    }
#pragma unroll
    for (int it = 0; it < ITB; ++it) {
        const int u = tid + it * 256;
        if (B_LAYOUT == K_CONTIG) {
            const int kq = u & 15, n = u >> 4;
            b_off[it] = 4u * ((unsigned)min(n0 + n, p.N - 1) * (unsigned)p.ldb + 4u * (unsigned)kq);
            b_dst[it] = (kq >> 2) * T::GB + 4 * n + (kq & 3);
        } else {
            const int nq = u % (BN / 4), k = u / (BN / 4);
            b_off[it] = 4u * ((unsigned)k * (unsigned)p.ldb + (unsigned)min(n0 + 4 * nq, p.N - 1));
            b_dst[it] = k * T::PB + 4 * nq;
        }
    }
    struct Raw { f32x4 a[ITA], b[ITB]; };
    // A slab behind the last one is "loaded" from operands of no length (zeros, no memory access): the loads of the loop are
    // unconditional, so that the compiler knows how many are younger than the ones it waits for.
    auto load = [&](int s, Raw &r) {
        const unsigned k0 = (unsigned)(s < n_slabs ? k_begin + s * BK : 0);
        const auto ab = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(A), 0, (int)(s < n_slabs ? a_bytes : 0u), 0x00020000);
        const auto bb = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(B), 0, (int)(s < n_slabs ? b_bytes : 0u), 0x00020000);
        auto get = [](auto rs, unsigned off, unsigned uni) {
            const u32x4_t u = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, (int)uni, 0);
            return __builtin_bit_cast(f32x4, u);
        };
#pragma unroll
        for (int it = 0; it < ITA; ++it) r.a[it] = get(ab, a_off[it], 4u * k0);
#pragma unroll
        for (int it = 0; it < ITB; ++it) r.b[it] = get(bb, b_off[it], B_LAYOUT == K_CONTIG ? 4u * k0 : 4u * k0 * (unsigned)p.ldb);
    };
    const int a_klim = min(p.a_lim, k_end), k_ones = p.a_ones < k_end ? p.a_ones : -1;
    const int n_whole = max(a_klim - k_begin, 0) / BK;               // slabs that need no replacement
    auto cut = [&](int s, Raw &r) {
        const int k0 = k_begin + s * BK;
#pragma unroll
        for (int it = 0; it < ITA; ++it) {
            const int k = k0 + 4 * ((tid + it * 256) & 15);
#pragma unroll
            for (int e = 0; e < 4; ++e) r.a[it][e] = k + e < a_klim ? r.a[it][e] : (k + e == k_ones ? 1.f : 0.f);
        }
#pragma unroll
        for (int it = 0; it < ITB; ++it) {
            const int u = tid + it * 256;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = k0 + (B_LAYOUT == K_CONTIG ? 4 * (u & 15) + e : u / (BN / 4));
                r.b[it][e] = k < k_end ? r.b[it][e] : 0.f;
            }
        }
    };
    // load `it` of a slab (A's first, then B's) from the registers to LDS
    auto store_piece = [&](int buf, int it, const Raw &r) {
        float *as = lds + buf * (T::A_FLOATS + T::B_FLOATS), *bs = as + T::A_FLOATS;
        if (it < ITA)
#pragma unroll
            for (int e = 0; e < 4; ++e) as[a_dst[it] + e * 4 * BM] = r.a[it][e];
        else if (B_LAYOUT == K_CONTIG)
#pragma unroll
            for (int e = 0; e < 4; ++e) bs[b_dst[it - ITA] + e * 4 * BN] = r.b[it - ITA][e];
        else *reinterpret_cast<f32x4 *>(bs + b_dst[it - ITA]) = r.b[it - ITA];
    };
    auto store = [&](int s, int buf, Raw &r) {
        if (s >= n_whole) cut(s, r);
#pragma unroll
        for (int it = 0; it < ITA + ITB; ++it) store_piece(buf, it, r);
    };
    // all operands of a slab's matrix instructions: lane l supplies A[m = l%16][k + l/16] and B[k + l/16][n = l%16]
    struct Frag { f32x4 a[4][TM], b[4]; };
    const int fa = q * 4 * BM + 4 * (wm * 16 * TM + l16);
    const int fb = B_LAYOUT == K_CONTIG ? q * 4 * BN + 4 * (wn * 16 + l16) : q * T::PB + wn * 16 + l16;
    // the operands of four (e < 0) or of one of the sixteen matrix instructions; A's come four at a time
    auto fetch_piece = [&](int buf, int t, int e, Frag &f) {
        const float *as = lds + buf * (T::A_FLOATS + T::B_FLOATS), *bs = as + T::A_FLOATS;
        if (e <= 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i) f.a[t][i] = *reinterpret_cast<const f32x4 *>(as + t * T::GA + fa + 64 * i);
            if (B_LAYOUT == K_CONTIG) f.b[t] = *reinterpret_cast<const f32x4 *>(bs + t * T::GB + fb);
        }
        if (B_LAYOUT == MN_CONTIG)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (e < 0 || u == e) f.b[t][u] = bs[(16 * t + 4 * u) * T::PB + fb];
    };
    f32x4 acc[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const Frag &f, int t, int e) {
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[t][i][e], f.b[t][e], acc[i], 0, 0, 0);
    };

    // gates of the input gradient: requested first, used last
    const int n = n0 + wn * 16 + l16, mr = m0 + wm * 16 * TM + 4 * q;
    float gate[TM][4];
    if constexpr (EPI == EPI_MASK) {
        const float *__restrict__ mask = p.mask + (size_t)w * p.mask_ws;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) gate[i][r] = mask[(size_t)min(mr + 16 * i + r, p.M - 1) * p.ldmask + min(n, p.N - 1)];
    }

    // Slab s is multiplied from registers while the operands of slab s+1 come out of LDS, slab s+2 goes into the buffer that
    // slab s has left, and the slabs behind it are on their way from memory: one barrier per slab, no wait behind it.  Every
    // LDS access has its place behind a matrix instruction: in a burst they hold back the matrix instructions behind them.
    Raw raw[NS];
    Frag frag[2];
#pragma unroll
    for (int d = 0; d < NS; ++d) load(d, raw[d]);
    store(0, 0, raw[0]);
    load(NS, raw[0]);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 4; ++t) fetch_piece(0, t, -1, frag[0]);
    store(1, 1, raw[1]);
    load(NS + 1, raw[1]);
    __syncthreads();
    auto step = [&](int s, auto phase) {
        constexpr int PH = decltype(phase)::value, CUR = PH & 1, ST = (PH + 2) % NS;
        if (s + 2 >= n_whole) cut(s + 2, raw[ST]);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            __builtin_amdgcn_sched_barrier(0);
            multiply(frag[CUR], j / 4, j % 4);
            __builtin_amdgcn_sched_barrier(0);
            fetch_piece(CUR ^ 1, j / 4, j % 4, frag[CUR ^ 1]);
#pragma unroll
            for (int it = 0; it < ITA + ITB; ++it)
                if (j == 1 + it * 13 / (ITA + ITB)) store_piece(CUR, it, raw[ST]);
            if (j == 14) load(s + 2 + NS, raw[ST]);
        }
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
    };
    constexpr std::integral_constant<int, 0> p0{};
    constexpr std::integral_constant<int, 1> p1{};
    constexpr std::integral_constant<int, 2> p2{};
    constexpr std::integral_constant<int, 3> p3{};
    int s = 0;
    for (; s + 4 <= n_slabs; s += 4) {          // no way out in the middle: the waits of all four steps stay exact
        step(s, p0);
        step(s + 1, p1);
        step(s + 2, p2);
        step(s + 3, p3);
    }
    if (s < n_slabs) {
        step(s, p0);
        if (s + 1 < n_slabs) {
            step(s + 1, p1);
            if (s + 2 < n_slabs) step(s + 2, p2);
        }
    }

    // register r of lane l is C[4*(l/16) + r][l%16] of its tile
    float *__restrict__ C = p.C + (size_t)w * p.c_ws + (size_t)split * p.c_ss;
    if (n < p.N) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = mr + 16 * i + r;
                float v = acc[i][r];
                if (EPI == EPI_RELU) v = fmaxf(v, 0.f);
                if constexpr (EPI == EPI_MASK) v = gate[i][r] > 0.f ? v : 0.f;
                if (m < p.M) C[(size_t)m * p.ldc + n] = v;
            }
    }
}

template <int WM, int WN, int TM, int B_LAYOUT, int EPI>
__global__ __launch_bounds__(256, 2) void gemm_chain_kernel(GemmArgs p)
{
    __shared__ __attribute__((aligned(16))) float lds[ChainTile<WM, WN, TM, B_LAYOUT>::LDS_FLOATS];
    if (B_LAYOUT == MN_CONTIG && p.ctr.blocks > 0 && blockIdx.x >= p.ctr.first_block) {         // uniform for the block
        center_rule_block(p.ctr.W, p.ctr.Wc, p.ctr.old, p.ctr.P, p.ctr.N, p.ctr.ld, p.ctr.alpha, blockIdx.x - p.ctr.first_block, p.ctr.blocks, threadIdx.x);
        return;
    }
    chain_block<WM, WN, TM, B_LAYOUT, EPI>(p, blockIdx.x, lds);
}

}  // namespace easgd
