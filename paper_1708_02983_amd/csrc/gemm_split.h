// Batched fp32 matrix products on the bfloat16 matrix cores, without giving up fp32 accuracy.
//
// Every fp32 operand is the exact sum of three bfloat16 numbers, x = h + m + l (h = x rounded to nearest, m = x - h
// rounded, l = the rest: 8 + 8 + 8 significant bits), a published method: G. Henry, P. T. P. Tang, A. Heinecke,
// "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", ARITH 2019.  Of the nine
// products of two such sums the six that matter are taken,
//     x*y = hh + (hm + mh) + (mm + hl + lh)      what is left out is below 2^-24 of |x*y|
// each exact in fp32, accumulated in fp32 by v_mfma_f32_32x32x16_bf16.  The large products hh and the small rest go
// to two accumulators that meet once at the end, so that a rounding of the large sum happens once per 16 values of k
// (the fp32 instruction rounds at every one): against 64-bit sums the result is two and a half to three times closer than
// that of v_mfma_f32_32x32x2_f32 (relative error of a sum of 1 024: 1.9e-7 against 5.7e-7, of 64: 4.9e-8 against 1.4e-7).
// The bfloat16 instruction has sixteen times the fp32 one's rate, so six of them still leave 2.7 times; the 6.5 vector
// instructions per operand element that scale and split it run beside the matrix instructions of the same SIMD (24 matrix
// instructions with four or six vector instructions behind each take as long as, or 3 to 15 % longer than without).
// Range: every operand is multiplied by 2^32 on its way into the split, every result by 2^-64.  A bfloat16 has fp32's
// exponents but its last part lies 16 bits below the number, so without that an operand below 2^-110 would lose bits;
// with it every fp32 number, denormal ones included, is split exactly into normal bfloat16 numbers.  Finite operands from
// 2^96 on, sums from 2^64 on, infinities and NaN make a sum that is not finite; a wavefront that finds one computes its
// tiles again with the fp32 instruction, whose result (finite, infinite or NaN) stands.  (The multiplication costs 2 to 3 %:
// 3072->2048 forward, 8 workers, 256 rows 148 us -> 152, 2048->2048 input gradient, 32 workers, 100 rows 197 -> 201.  The
// second computation costs as much as the fp32 kernels' or more, but only where values are that far out.)
//
#pragma once
#include "gemm_mfma.h"
#include "narrow_dw.h"
#include <utility>

namespace easgd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr float SPLIT_SCALE = 0x1p32f, SPLIT_UNSCALE = 0x1p-64f;     // of an operand, of a product (head of the file)

struct SplitFrag { u32x4 h, m, l; };       // eight values of k: three bfloat16 planes of 16 bytes

// two floats rounded to nearest even, a in the low half
__device__ __forceinline__ unsigned bf16_pack(float a, float b)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a, b}, bf16x2));      // v_cvt_pk_bf16_f32
}

// The split of eight values in twelve parts of four or so independent instructions each (x is used up), to be placed behind matrix
// instructions; no instruction waits for the one before it.  ONES: x * mul + add is split, which puts ones in the place
// of x (mul = 0) at no cost; otherwise x alone.
constexpr int SPLIT_PARTS = 12;
template <bool ONES = false>
__device__ __forceinline__ void split_part(int part, f32x8 &x, SplitFrag &f, u32x4 &t, float mul = SPLIT_SCALE, float add = 0.f)
{
    auto low = [](unsigned d) { return d << 16; };                       // the two numbers of a pair as fp32 bits
    auto high = [](unsigned d) { return d & 0xffff0000u; };
    auto scale1 = [&](float v) { return ONES ? fmaf(v, mul, add) : v * SPLIT_SCALE; };
    auto scale = [&](int e) { x[2 * e] = scale1(x[2 * e]); x[2 * e + 1] = scale1(x[2 * e + 1]); };
    auto take = [&](u32x4 &plane, int e) { plane[e] = bf16_pack(x[2 * e], x[2 * e + 1]); };
    auto widen = [&](const u32x4 &plane, int e) { f.l[e] = low(plane[e]); t[e] = high(plane[e]); };
    auto rest = [&](int e) { x[2 * e] -= __uint_as_float(f.l[e]); x[2 * e + 1] -= __uint_as_float(t[e]); };
    if (part == 0) { scale(0); scale(1); }
    if (part == 1) { scale(2); scale(3); }
    if (part == 2) { take(f.h, 0); take(f.h, 1); take(f.h, 2); take(f.h, 3); }
    if (part == 3) { widen(f.h, 0); widen(f.h, 1); }
    if (part == 4) { widen(f.h, 2); widen(f.h, 3); }
    if (part == 5) { rest(0); rest(1); }
    if (part == 6) { rest(2); rest(3); }
    if (part == 7) { take(f.m, 0); take(f.m, 1); take(f.m, 2); take(f.m, 3); }
    if (part == 8) { widen(f.m, 0); widen(f.m, 1); }
    if (part == 9) { widen(f.m, 2); widen(f.m, 3); rest(0); }
    if (part == 10) { rest(1); rest(2); take(f.l, 0); }
    if (part == 11) { rest(3); take(f.l, 1); take(f.l, 2); take(f.l, 3); }
}

template <bool ONES = false>
__device__ __forceinline__ void split8(f32x8 &x, SplitFrag &f, float mul = SPLIT_SCALE, float add = 0.f)
{
    u32x4 t;
#pragma unroll
    for (int part = 0; part < SPLIT_PARTS; ++part) split_part<ONES>(part, x, f, t, mul, add);
}

// f(0), f(1), ..., f(N - 1) with the index as a constant: what depends on it is decided before the optimiser sees the code
template <typename F, int... I>
__device__ __forceinline__ void static_for_each(F &&f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) { static_for_each(f, std::make_integer_sequence<int, N>{}); }

// Tile configuration: a block of four wavefronts, WN side by side along n and WK along k, owns a (TM*32) x (WN*32)
// tile of C; every wavefront owns all TM*32 rows of 32 columns.  A slab is KS steps of sixteen k per wavefront.
template <int TM, int WN, int WK>
struct SplitTile {
    static_assert(WN * WK == 4, "four wavefronts");
    static constexpr int BM = TM * 32, BN = WN * 32;
    static constexpr int KS = WK == 1 ? 2 : 1;
    static constexpr int BK = 16 * WK * KS, K8 = BK / 8;
    static constexpr int UNITS = BM * K8;                            // (row of A, eight k) pieces of a slab
    static constexpr int IT = (UNITS + 255) / 256;
    static constexpr int SLAB_VECS = (BK / 16) * 3 * TM * 64;        // 16-byte vectors of a slab of A in LDS
    // two slabs, or the sums that the WK wavefronts of a tile exchange at the end
    static constexpr int EXCHANGE_VECS = WK > 1 ? 4 * TM * 4 * 64 : 0;
    static constexpr int LDS_VECS = 2 * SLAB_VECS > EXCHANGE_VECS ? 2 * SLAB_VECS : EXCHANGE_VECS;
};

template <int TM, int WN, int WK, int A_LAYOUT, int B_LAYOUT, int EPI, bool EARLY = false>
__device__ __forceinline__ void split_block(const GemmArgs &p, const unsigned bid, u32x4 *__restrict__ lds)
{
    typedef SplitTile<TM, WN, WK> T;
    constexpr int BM = T::BM, BN = T::BN, BK = T::BK, K8 = T::K8, IT = T::IT, KS = T::KS;
    BlockTile bt;
    if (!block_tile(p, bid, bt)) return;
    const int w = __builtin_amdgcn_readfirstlane(bt.w);
    const int tile_m = __builtin_amdgcn_readfirstlane(bt.tile_m), tile_n = __builtin_amdgcn_readfirstlane(bt.tile_n);
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, q = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave % WK, wn = wave / WK;
    const int m0 = tile_m * BM, n0 = tile_n * BN + wn * 32;     // n0: the wavefront's columns
    const int k_begin = __builtin_amdgcn_readfirstlane(bt.split) * p.k_per_split, k_end = min(p.K, k_begin + p.k_per_split);
    const float *__restrict__ A = p.A + (size_t)w * p.a_ws;
    const float *__restrict__ B = p.B + (size_t)w * p.b_ws;
    const int a_rows = (A_LAYOUT == K_CONTIG) ? p.M : p.a_lim;        // rows that are stored (the ones vector is not)

    // ---- loader geometry ----
    // Buffer loads: a 32-bit byte offset per lane and a uniform one per load.
    // A: unit u = tid + it*256 is eight k of one row, k8 = 0..K8-1.  An operand that is contiguous along k is read with
    // neighbouring lanes along k (whole cache lines of a row), one that is contiguous along m with neighbouring lanes
    // along m.  In LDS a unit is 16 bytes per plane, at the place where the matrix instruction's lane reads it; for
    // the first kind the rows of a unit's column are permuted so that its eight lanes write to different banks.
    auto rsrc = [](const float *base, unsigned elements) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, (int)(4u * elements), 0x00020000);
    };
    const auto ab = rsrc(A, (unsigned)(A_LAYOUT == K_CONTIG ? p.M : p.K) * (unsigned)p.lda);
    const auto bb = rsrc(B, (unsigned)(B_LAYOUT == K_CONTIG ? p.N : p.K) * (unsigned)p.ldb);
    unsigned a_off[IT];
    int a_dst[IT], a_kept[IT];                                       // a_kept: the unit's first k inside its slab
    // The row of C that multiplies by ones has no row of A; what the clamped address brings is multiplied by 0.  (A value
    // that is not finite makes a sum that is not, see the head of the file.)
    constexpr bool ONES = A_LAYOUT == MN_CONTIG;
    float a_mul[IT], a_add[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int u = tid + it * 256;
        const int row = (A_LAYOUT == K_CONTIG) ? u / K8 : u % BM, k8 = (A_LAYOUT == K_CONTIG) ? u % K8 : u / BM;
        const int swz = (A_LAYOUT == K_CONTIG) ? k8 * (8 / K8) : 0;
        const int m = min(m0 + row, a_rows - 1);
        const bool one = ONES && m0 + row == p.a_ones;
        a_mul[it] = one ? 0.f : SPLIT_SCALE;
        a_add[it] = one ? SPLIT_SCALE : 0.f;
        a_off[it] = (A_LAYOUT == K_CONTIG) ? 4u * ((unsigned)m * (unsigned)p.lda + 8u * k8) : 4u * (8u * k8 * (unsigned)p.lda + (unsigned)m);
        a_kept[it] = 8 * k8;
        a_dst[it] = ((k8 >> 1) * 3 * TM + (row >> 5)) * 64 + (((row & 31) ^ swz) + 32 * (k8 & 1));
    }
    const int bn = min(n0 + l32, p.N - 1);
    const unsigned b_off = (B_LAYOUT == K_CONTIG) ? 4u * ((unsigned)bn * (unsigned)p.ldb + 8u * q) : 4u * (8u * q * (unsigned)p.ldb + (unsigned)bn);

    // What only the last slabs and the epilogue need is worked out there in the forward products, from a thread index that
    // the compiler cannot look through: kept over the loop it costs registers that their kernels would have to spill (up to
    // ten; 256->128, 4 workers, 64 rows 7.4 us -> 7.0 without).
    constexpr bool LATE = A_LAYOUT == K_CONTIG && B_LAYOUT == MN_CONTIG;
    auto thread = [&] {
        int t = tid;
        if constexpr (LATE) keep_loaded(t);
        return t;
    };
    auto a_k = [&](int it) { return LATE ? 8 * ((thread() + it * 256) % K8) : a_kept[it]; };

    struct RawA { f32x8 x[IT]; };
    struct RawB { f32x8 x[KS]; };
    auto k4_vec = [](auto rs, unsigned off, unsigned uni, int half, f32x8 &x) {
        const u32x4 u = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off + 16 * half, (int)uni, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * half + e] = __uint_as_float(u[e]);
    };
    // Slabs that lie inside both operands along k are loaded as they are; in the others every element has an address of
    // its own that is held inside the operand, and is replaced by what it stands for when it is used (cut).
    const int a_klim = (A_LAYOUT == K_CONTIG) ? min(p.a_lim, k_end) : k_end;
    const int n_slabs = (k_end - k_begin + BK - 1) / BK;
    // Without the ones vector along k the last slab may start early, so that it lies inside too: what it then holds of
    // the slab before is replaced by zeros.  (Sums as short as a minibatch have no other slabs to speak of.)
    const bool early = !(A_LAYOUT == K_CONTIG && B_LAYOUT == MN_CONTIG) && k_end - k_begin >= BK;      // uniform
    const int n_fast = early ? n_slabs : (a_klim - k_begin) / BK;
    auto start = [&](int slab) { return early ? min(k_begin + slab * BK, k_end - BK) : k_begin + slab * BK; };
    // what lies below `first` or at or beyond `lim` along k is zero, or one where the ones vector sits
    auto cut = [](f32x8 &x, int k, int first, int lim, int ones) {
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = k + e >= first && k + e < lim ? x[e] : (k + e == ones ? 1.f : 0.f);
    };
    auto whole = [&](int slab) { return early ? start(slab) == k_begin + slab * BK : slab < n_fast; };
    const int k_ones = (A_LAYOUT == K_CONTIG && p.a_ones < k_end) ? p.a_ones : -1;
    // inner (a slab inside the operands): piece 0..7 is one 32-bit load each, or piece 0 both halves of a lane's eight k; otherwise
    // piece 0 is all of them.  The halves go out together: a few slots apart, other wavefronts' loads push the line that
    // they share out of the first-level cache, and where rows start at any element of a line every line is fetched
    // twice (input gradient 2974->1332, 30 workers, 101 rows 266 us against 202; rows of whole lines do not mind).
    auto load_a = [&](int slab, auto inner, int it, int piece, RawA &r) {
        constexpr bool INNER = decltype(inner)::value;
        if (piece > 0 && (!INNER || A_LAYOUT == K_CONTIG)) return;
        const int k0 = start(slab);
        if (INNER || slab < n_fast) {
            if (A_LAYOUT == K_CONTIG) {
                k4_vec(ab, a_off[it], 4u * (unsigned)k0, 0, r.x[it]);
                k4_vec(ab, a_off[it], 4u * (unsigned)k0, 1, r.x[it]);
            } else
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (!INNER || e == piece) r.x[it][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ab, (int)a_off[it], (int)(4u * (unsigned)(k0 + e) * (unsigned)p.lda), 0));
        } else if (!early && slab < n_slabs) {
            const int ku = a_k(it);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const unsigned k = (unsigned)min(k0 + ku + e, a_klim - 1);
                const unsigned off = (A_LAYOUT == K_CONTIG) ? a_off[it] - 4u * (unsigned)ku + 4u * k
                                                            : a_off[it] + 4u * (k - (unsigned)ku) * (unsigned)p.lda;
                r.x[it][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ab, (int)off, 0, 0));
            }
        }
    };
    auto load_b_step = [&](int slab, auto inner, int ks, int piece, RawB &r) {
        constexpr bool INNER = decltype(inner)::value;
        if (piece > 0 && (!INNER || B_LAYOUT == K_CONTIG)) return;
        const int kb = start(slab) + 16 * (wk + ks * WK);
        if (INNER || slab < n_fast) {
            if (B_LAYOUT == K_CONTIG) {
                k4_vec(bb, b_off, 4u * (unsigned)kb, 0, r.x[ks]);
                k4_vec(bb, b_off, 4u * (unsigned)kb, 1, r.x[ks]);
            } else
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (!INNER || e == piece) r.x[ks][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(bb, (int)b_off, (int)(4u * (unsigned)(kb + e) * (unsigned)p.ldb), 0));
        } else if (!early && slab < n_slabs) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const unsigned k = (unsigned)min(kb + 8 * q + e, k_end - 1);
                const unsigned off = (B_LAYOUT == K_CONTIG) ? b_off - 32u * (unsigned)q + 4u * k : b_off + 4u * (k - 8u * (unsigned)q) * (unsigned)p.ldb;
                r.x[ks][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(bb, (int)off, 0, 0));
            }
        }
    };
    auto cut_a = [&](int slab, int it, RawA &r) { cut(r.x[it], start(slab) + a_k(it), k_begin + slab * BK, a_klim, k_ones); };
    auto cut_b = [&](int slab, int ks, RawB &r) { cut(r.x[ks], start(slab) + 16 * (wk + ks * WK) + 8 * q, k_begin + slab * BK, k_end, -1); };
    auto a_here = [&](int it) { return T::UNITS % 256 == 0 || tid + it * 256 < T::UNITS; };
    auto store_plane = [&](int buf, int it, int plane, const SplitFrag &f) {
        if (!a_here(it)) return;
        lds[buf * T::SLAB_VECS + a_dst[it] + plane * TM * 64] = plane == 0 ? f.h : plane == 1 ? f.m : f.l;
    };

    f32x16 hi[TM], lo[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) hi[i][r] = lo[i][r] = 0.f;
    auto mm = [](const u32x4 &x, const u32x4 &y, f32x16 &c) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), c, 0, 0, 0);
    };
    // The fragments of A come from LDS one tile ahead of the products that use them.
    auto fetch = [&](int buf, int ks, int i, int plane, SplitFrag &f) {
        const int step = wk + ks * WK, k8 = 2 * step + q;
        const int swz = (A_LAYOUT == K_CONTIG) ? k8 * (8 / K8) : 0;
        const u32x4 *src = lds + buf * T::SLAB_VECS + (step * 3 * TM + i) * 64 + ((l32 ^ swz) + 32 * q);
        (plane == 0 ? f.h : plane == 1 ? f.m : f.l) = src[plane * TM * 64];
    };
    auto multiply = [&](int part, int i, const SplitFrag &f, const SplitFrag &fb) {
        if (part == 0) mm(f.l, fb.h, lo[i]);
        if (part == 1) mm(f.h, fb.h, hi[i]);
        if (part == 2) mm(f.h, fb.l, lo[i]);
        if (part == 3) mm(f.m, fb.m, lo[i]);
        if (part == 4) mm(f.m, fb.h, lo[i]);
        if (part == 5) mm(f.h, fb.m, lo[i]);
    };

    // Slab s is multiplied from LDS buffer s % 2, tile by tile and step by step ("items" of six matrix instructions, "slots").
    // What prepares the slabs behind it runs between the matrix instructions, spread over them, since a vector instruction takes an
    // eighth of a matrix instruction's time and a wavefront issues in order: each split (the slab's second step of B, slab s+1 of A
    // on its way to the other LDS buffer, slab s+1's first step of B) has a span of slots; the LDS stores and the loads of the raw
    // registers that a split has used up follow in the slots behind it.
    // The large tiles take one split after the other, and load B's first step in the first slots of the next slab.  In bursts (a
    // split within six slots, then its stores and loads) / spread, us: forward 3072->2048, 8 workers, 256 rows 150 / 141; input
    // gradient 2048->2048, 32, 100 199 / 193; forward 784->1024, 16, 128 in 64x128 tiles 27.6 / 26.6, 1024->1024, 16, 128 (input
    // gradient) 32.2 / 31.8.  What the first of these takes over its matrix instructions (83 us) is the loads and LDS stores (in a
    // kernel trace on another box, as built 127): without loads from memory 125, without LDS stores 116, without either and with a
    // third of the LDS reads 102.
    // In the small tiles a slab's twelve or six slots are shorter than a trip to memory, and where the operands come from far or few
    // wavefronts share a compute unit, what counts is that the trips of A and B overlap: both loads go out before either is
    // waited for.  Time over that of the bursts (products of 64 to 3072 inputs, 48 to 2048 outputs, 2 to 32 workers, 16 to 256 rows):
    //   64x64, one after the other   0.84 to 1.11 forward, 0.88 to 1.12 input gradients
    //   64x64, EARLY                 0.95 to 1.01          0.96 to 1.02     (faster where split_early says so)
    //   32x128 forward               0.95 to 1.10 one after the other, 0.97 to 1.03 EARLY      (the same)
    //   32x32 input gradients        0.94 to 1.06 both splits over all six slots, 0.95 to 1.02 in this order
    constexpr int ITEMS = KS * TM, SLOTS = 6 * ITEMS, SPLITS = KS + IT, SPAN = SLOTS / SPLITS;
    constexpr bool FORWARD = A_LAYOUT == K_CONTIG && B_LAYOUT == MN_CONTIG;
    constexpr bool TINY = ITEMS == 1;                                    // the 32x32 tile
    constexpr bool B_BEHIND = TINY || EARLY;                             // B's first step is loaded right behind its split
    constexpr int RATE = SPAN >= 12 ? 1 : 4;                             // pieces of a load per slot, eight in all
    static_assert(!EARLY || SLOTS == 12, "the 64x64 and 32x128 tiles");
    static_assert(SLOTS % SPLITS == 0 && SPAN >= 3, "a split's three stores come before the end of the slab");
    // the splits in order (A's units 0, 1, ..; -1: B's second step, whose registers are in use from the second step on; -2: B's first
    // step, whose registers are free from the second step on, or a second set where there is one step)
    constexpr auto split_at = [](int n) { return n + 1 == SPLITS ? -2 : KS == 1 ? n : n - 1; };
    constexpr auto first_slot = [](int n) { return TINY ? (FORWARD || n == 1 ? 0 : 1) : EARLY ? (KS == 1 ? 6 * n : 3 * n) : SPAN * n; };
    constexpr auto slots_of = [](int) { return TINY ? (FORWARD ? 6 : 5) : EARLY ? (KS == 1 ? 4 : 3) : SPAN; };
    static_assert(KS == 1 || (first_slot(0) + slots_of(0) <= 6 * TM && first_slot(SPLITS - 1) >= 6 * TM), "the two steps of B");
    // (A second set of raw registers, so that a slab's loads have two slabs to arrive in, is slower in every tile: 64x128 DW 38.1 us
    // -> 51.0, 32x32 input gradient 777->333 7.9 -> 8.7.)
    RawA ra;
    RawB rb;
    SplitFrag fb[2];
    // before the loop: slab 0 is split, the raw registers hold what the loop expects to find (A's slab 1, B's second step of slab 0)
#pragma unroll
    for (int u = 0; u < IT; ++u) load_a(0, std::false_type{}, u, 0, ra);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) load_b_step(0, std::false_type{}, ks, 0, rb);
#pragma unroll
    for (int u = 0; u < IT; ++u) {
        SplitFrag f;
        if (!whole(0)) cut_a(0, u, ra);
        split8<ONES>(ra.x[u], f, a_mul[u], a_add[u]);
#pragma unroll
        for (int plane = 0; plane < 3; ++plane) store_plane(0, u, plane, f);
        load_a(1, std::false_type{}, u, 0, ra);
    }
    if (!whole(0)) cut_b(0, 0, rb);
    split8(rb.x[0], fb[0]);
    if constexpr (B_BEHIND) load_b_step(1, std::false_type{}, 0, 0, rb);
    __syncthreads();
    auto slab = [&](int s, auto parity, auto last_slabs) {
        constexpr int buf = decltype(parity)::value;
        constexpr bool LAST = decltype(last_slabs)::value;
        constexpr std::integral_constant<bool, !LAST> inner{};           // every slab that is loaded here lies inside the operands
        // fragments of B: step ks of this slab, and where the first step of the next slab goes
        constexpr int F0 = KS == 1 ? buf : 0, F1 = KS == 1 ? (buf ^ 1) : 0;
        SplitFrag fa[2], fs[IT];
        u32x4 t[SPLITS];
#pragma unroll
        for (int plane = 0; plane < 3; ++plane) fetch(buf, 0, 0, plane, fa[0]);
        static_for<SLOTS>([&](auto slot_) {
            constexpr int slot = decltype(slot_)::value, it = slot / 6, part = slot % 6, ks = it / TM, i = it % TM;
            // a step without a k of its own holds zeros only
            const int k_step = start(s) + 16 * (wk + ks * WK);
            const bool live = !LAST || (k_step < k_end && k_step + 16 > k_begin + s * BK);  // uniform
            if constexpr (LAST)
                static_for<SPLITS>([&](auto n_) {
                    constexpr int n = decltype(n_)::value, u = split_at(n);
                    if constexpr (first_slot(n) == slot) {
                        if constexpr (u == -1) { if (!whole(s)) cut_b(s, KS - 1, rb); }
                        else if constexpr (u == -2) { if (!whole(s + 1)) cut_b(s + 1, 0, rb); }
                        else if (!whole(s + 1)) cut_a(s + 1, u, ra);
                    }
                });
            __builtin_amdgcn_sched_barrier(0);
            if (live) multiply(part, i, fa[it & 1], fb[ks == 0 ? F0 : 1]);
            static_for<(SPLIT_PARTS + slots_of(0) - 1) / slots_of(0)>([&](auto j_) {
                static_for<SPLITS>([&](auto n_) {                        // B's part before A's
                    constexpr int n = SPLITS - 1 - decltype(n_)::value, u = split_at(n), at = slot - first_slot(n), L = slots_of(n);
                    constexpr int q = (at * SPLIT_PARTS + L - 1) / L + decltype(j_)::value;      // split n's parts of this slot: from the first on
                    if constexpr (at >= 0 && at < L && q < SPLIT_PARTS && q * L / SPLIT_PARTS == at) {
                        if constexpr (u == -1) split_part(q, rb.x[KS - 1], fb[1], t[n]);
                        else if constexpr (u == -2) split_part(q, rb.x[0], fb[F1], t[n]);
                        else split_part<ONES>(q, ra.x[u], fs[u], t[n], a_mul[u], a_add[u]);
                    }
                });
            });
            if constexpr (it + 1 < ITEMS && part < 3) fetch(buf, (it + 1) / TM, (it + 1) % TM, part == 0 ? 2 : part - 1, fa[(it + 1) & 1]);
            if constexpr (!B_BEHIND && slot < 8 / RATE)           // the registers that the slab before has used up at its end
                static_for<RATE>([&](auto r_) { load_b_step(s + 1, inner, 0, slot * RATE + decltype(r_)::value, rb); });
            if constexpr (TINY && FORWARD) __builtin_amdgcn_sched_barrier(0);
            static_for<SPLITS>([&](auto n_) {                            // what is left when the slab ends goes into its last slot
                constexpr int n = SPLITS - 1 - decltype(n_)::value, u = split_at(n), end = first_slot(n) + slots_of(n);
                constexpr int after = slot - (end < SLOTS ? end : SLOTS - 1);
                constexpr bool last = slot == SLOTS - 1;
                if constexpr (after >= 0 && u >= 0)
                    static_for<last && after < 3 ? 3 - after : after < 3 ? 1 : 0>([&](auto i_) {
                        if (!LAST || s + 1 < n_slabs) store_plane(buf ^ 1, u, after + decltype(i_)::value, fs[u]);
                    });
                if constexpr (after >= 0 && (u != -2 || B_BEHIND))
                    static_for<last && after * RATE < 8 ? 8 - after * RATE : after * RATE < 8 ? RATE : 0>([&](auto i_) {
                        constexpr int piece = after * RATE + decltype(i_)::value;
                        if constexpr (u == -1) load_b_step(s + 1, inner, KS - 1, piece, rb);
                        else if constexpr (u == -2) load_b_step(s + 2, inner, 0, piece, rb);
                        else load_a(s + 2, inner, u, piece, ra);
                    });
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        __syncthreads();
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    int s = 0;
    for (; s + 3 < n_fast; s += 2) {
        slab(s, even, std::false_type{});
        slab(s + 1, odd, std::false_type{});
    }
    for (; s < n_slabs; s += 2) {
        slab(s, even, std::true_type{});
        if (s + 1 >= n_slabs) break;
        slab(s + 1, odd, std::true_type{});
    }

    // ---- the two sums meet; what went out of the scaled range is summed again (head of the file) ----
    const int late = thread() & 63, c32 = late & 31, cq = late >> 5;         // lane, column and row group of C
    const int n = n0 + c32, nc = min(n, p.N - 1);
    f32x16 acc[TM];
    f32x8 bad = {};                                      // eight chains: NaN as soon as one of a chain's sums is not finite
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float c = hi[i][r] + lo[i][r];
            bad[r % 8] = fmaf(c, 0.f, bad[r % 8]);
            acc[i][r] = c * SPLIT_UNSCALE;
        }
    const float not_finite = ((bad[0] + bad[1]) + (bad[2] + bad[3])) + ((bad[4] + bad[5]) + (bad[6] + bad[7]));
    if (__builtin_expect(__any(not_finite != 0.f), 0)) {  // uniform for the wavefront
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
        // the wavefront's steps of every slab, in pairs of k: lane l holds A[m = l%32][k = l/32] and B[k = l/32][n = l%32]
        for (int st = 0; st < n_slabs * KS; ++st) {
            const int sl = st / KS, kb = start(sl) + 16 * (wk + (st % KS) * WK), first = k_begin + sl * BK;
#pragma unroll 1
            for (int half = 0; half < 16; half += 8) {
                float x[4][TM], y[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int k = kb + half + 2 * u + cq;
                    const bool in = k >= first && k < k_end;
                    const unsigned ka = (unsigned)max(min(k, a_klim - 1), 0), kc = (unsigned)min(k, k_end - 1);
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        const int row = m0 + 32 * i + c32;
                        const unsigned m = (unsigned)min(row, a_rows - 1);
                        const unsigned off = 4u * (A_LAYOUT == K_CONTIG ? m * (unsigned)p.lda + ka : kc * (unsigned)p.lda + m);
                        const float v = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ab, (int)off, 0, 0));
                        const bool one = A_LAYOUT == K_CONTIG ? k == k_ones : row == p.a_ones;
                        x[u][i] = !in ? 0.f : one ? 1.f : A_LAYOUT == K_CONTIG && k >= a_klim ? 0.f : v;
                    }
                    const unsigned off = 4u * (B_LAYOUT == K_CONTIG ? (unsigned)nc * (unsigned)p.ldb + kc : kc * (unsigned)p.ldb + (unsigned)nc);
                    const float v = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(bb, (int)off, 0, 0));
                    y[u] = in ? v : 0.f;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int i = 0; i < TM; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[u][i], y[u], acc[i], 0, 0, 0);
            }
        }
    }

    // ---- epilogue ----
    // Register r of lane l is C[8*(r/4) + 4*q + r%4][l%32] of its 32x32 tile.  Where WK wavefronts share a tile,
    // wavefront wk finishes the register groups r/4 = wk mod WK; the partial sums of the others come through LDS and
    // are added in ascending order of k.
    constexpr bool ELASTIC = (EPI == EPI_ELASTIC || EPI == EPI_ELASTIC_MOM || EPI == EPI_ELASTIC_MOM_BF16);
    constexpr bool MOM = (EPI == EPI_ELASTIC_MOM);
    constexpr bool MOM16 = (EPI == EPI_ELASTIC_MOM_BF16);
    constexpr bool OUT16 = (EPI == EPI_STORE_BF16);
    constexpr int GROUPS = 4 / WK;                       // register groups a wavefront finishes per tile
    float val[TM][GROUPS][4];
    if constexpr (WK > 1) {
        f32x4 *ex = reinterpret_cast<f32x4 *>(lds) + (size_t)wn * (WK * TM * 4 * 64);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                ex[((wk * TM + i) * 4 + g) * 64 + late] = f32x4{acc[i][4 * g], acc[i][4 * g + 1], acc[i][4 * g + 2], acc[i][4 * g + 3]};
        __syncthreads();
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int gg = 0; gg < GROUPS; ++gg) {
                const int g = gg * WK + wk;
                f32x4 v = ex[(i * 4 + g) * 64 + late];
#pragma unroll
                for (int o = 1; o < WK; ++o) v += ex[((o * TM + i) * 4 + g) * 64 + late];
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) val[i][gg][rr] = v[rr];
            }
    } else {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int gg = 0; gg < GROUPS; ++gg)
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) val[i][gg][rr] = acc[i][4 * gg + rr];
    }
    const bool keep = !OUT16 && (!ELASTIC || p.C != nullptr);                         // uniform
    float *__restrict__ C = keep ? p.C + (size_t)w * p.c_ws + (size_t)bt.split * p.c_ss : nullptr;
    unsigned short *__restrict__ C16 = OUT16 ? p.C16 + (size_t)w * p.c_ws : nullptr;
    const float *__restrict__ mask = (EPI == EPI_MASK) ? p.mask + (size_t)w * p.mask_ws : nullptr;
    float *__restrict__ Wr = ELASTIC ? p.Wt + (size_t)w * p.c_ws : nullptr;
    float *__restrict__ Vr = MOM ? p.Vt + (size_t)w * p.c_ws : nullptr;
    unsigned short *__restrict__ Vr16 = MOM16 ? p.Vt16 + (size_t)w * p.c_ws : nullptr;
    const float *__restrict__ Cc = ELASTIC ? p.center : nullptr;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int mt = m0 + 32 * i;                                                   // uniform
        if (mt >= p.M) break;
        const bool rows_in = mt + 32 <= p.M;
        auto row = [&](int gg, int rr) { return mt + 8 * (gg * WK + wk) + 4 * cq + rr; };
        float wv[GROUPS][4], cv[GROUPS][4], vv[GROUPS][4], gate[GROUPS][4];
        unsigned short v16[GROUPS][4];
        (void)wv; (void)cv; (void)vv; (void)gate; (void)v16;
        // all loads of the tile first; a lane whose element lies outside C reads the last row or column instead
#pragma unroll
        for (int gg = 0; gg < GROUPS; ++gg)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int mc = min(row(gg, rr), p.M - 1);
                if constexpr (ELASTIC) {
                    const size_t at = (size_t)mc * p.ldc + nc;
                    wv[gg][rr] = Wr[at];
                    cv[gg][rr] = Cc[at];
                    if constexpr (MOM) vv[gg][rr] = Vr[at];
                    if constexpr (MOM16) v16[gg][rr] = Vr16[at];
                }
                if constexpr (EPI == EPI_MASK) gate[gg][rr] = mask[(size_t)mc * p.ldmask + nc];
            }
        auto finish = [&](auto checked) {
#pragma unroll
            for (int gg = 0; gg < GROUPS; ++gg)
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const int m = row(gg, rr);
                    const size_t at = (size_t)m * p.ldc + n;
                    float v = val[i][gg][rr];
                    if constexpr (MOM16) worker_rule_bf16<true>(wv[gg][rr], v16[gg][rr], v, cv[gg][rr], p.eta, p.rho, p.alpha, p.delta);
                    else if constexpr (ELASTIC) worker_rule<MOM>(wv[gg][rr], vv[gg][rr], v, cv[gg][rr], p.eta, p.rho, p.alpha, p.delta);
                    if (EPI == EPI_RELU) v = fmaxf(v, 0.f);
                    if (EPI == EPI_MASK) v = gate[gg][rr] > 0.f ? v : 0.f;
                    if (decltype(checked)::value && m >= p.M) continue;
                    if constexpr (ELASTIC) {
                        Wr[at] = wv[gg][rr];
                        if constexpr (MOM) Vr[at] = vv[gg][rr];
                        if constexpr (MOM16) Vr16[at] = v16[gg][rr];
                    }
                    if constexpr (OUT16) C16[at] = bf16_narrow(v);
                    else if (keep) C[at] = v;
                }
        };
        if (n < p.N) {
            if (rows_in) finish(std::false_type{});
            else finish(std::true_type{});
        }
    }
}

// Blocks per compute unit that the registers leave room for.
template <int TM> constexpr int split_blocks_per_cu() { return TM == 1 ? 4 : TM == 2 ? 3 : 2; }

template <int TM, int WN, int WK, int A_LAYOUT, int B_LAYOUT, int EPI, bool EARLY = false>
__global__ __launch_bounds__(256, split_blocks_per_cu<TM>()) void gemm_split_kernel(GemmArgs p)
{
    __shared__ u32x4 lds[SplitTile<TM, WN, WK>::LDS_VECS];
    if (A_LAYOUT == K_CONTIG && B_LAYOUT == MN_CONTIG && p.ctr.blocks > 0 && blockIdx.x >= p.ctr.first_block) {         // uniform for the block
        const size_t b = blockIdx.x - p.ctr.first_block;
        center_rule_block(p.ctr.W, p.ctr.Wc, p.ctr.old, p.ctr.P, p.ctr.N, p.ctr.ld, p.ctr.alpha, b, p.ctr.blocks, threadIdx.x);
        return;
    }
    if (A_LAYOUT == MN_CONTIG && p.mean.blocks > 0 && blockIdx.x >= p.mean.first_block) {
        mean_loss_block(p.mean, blockIdx.x - p.mean.first_block);
        return;
    }
    split_block<TM, WN, WK, A_LAYOUT, B_LAYOUT, EPI, EARLY>(p, blockIdx.x, lds);
}

// The weight-gradient products of two layers in one launch (gemm_dw_pair_kernel's purpose).
template <int TM, int WN, int WK, int EPI>
__global__ __launch_bounds__(256, split_blocks_per_cu<TM>()) void gemm_split_dw_pair_kernel(GemmArgs p0, GemmArgs p1, unsigned n0)
{
    __shared__ u32x4 lds[SplitTile<TM, WN, WK>::LDS_VECS];
    if (p0.mean.blocks > 0 && blockIdx.x >= p0.mean.first_block) mean_loss_block(p0.mean, blockIdx.x - p0.mean.first_block);
    else if (blockIdx.x < n0) split_block<TM, WN, WK, MN_CONTIG, MN_CONTIG, EPI>(p0, blockIdx.x, lds);
    else split_block<TM, WN, WK, MN_CONTIG, MN_CONTIG, EPI>(p1, blockIdx.x - n0, lds);
}

// An input-gradient product with the weight-gradient product of a narrow layer, whose few blocks come first: they are a
// chain of round trips to memory, which the blocks of the other product cover.  DW: the form of the narrow product.
enum NarrowForm { DW_128x32 = 0, DW_128x32_VEC = 1, DW_NARROW16 = 2 };

template <int DW>
constexpr int narrow_lds_floats() { return DW == DW_NARROW16 ? 0 : gemm_lds_floats<128, 32, 32, MN_CONTIG, MN_CONTIG>(); }

template <int EPI, int DW>
__device__ __forceinline__ void narrow_dw_any(const GemmArgs &dw, const unsigned bid, float *__restrict__ lds)
{
    if constexpr (DW == DW_NARROW16) narrow_dw_block<1, EPI>(dw, bid);
    else gemm_block<128, 32, 32, 4, 1, MN_CONTIG, MN_CONTIG, DW == DW_128x32_VEC, EPI>(dw, bid, lds);
}

template <int TM, int WN, int WK, int EPI, int DW>
__global__ __launch_bounds__(256, 3) void gemm_split_da_narrow_dw_kernel(GemmArgs da, GemmArgs dw, unsigned n_dw)
{
    constexpr int NARROW = narrow_lds_floats<DW>() / 4, SPLIT = SplitTile<TM, WN, WK>::LDS_VECS;
    __shared__ u32x4 lds[NARROW > SPLIT ? NARROW : SPLIT];
    if (dw.mean.blocks > 0 && blockIdx.x >= dw.mean.first_block) mean_loss_block(dw.mean, blockIdx.x - dw.mean.first_block);
    else if (blockIdx.x < n_dw) narrow_dw_any<EPI, DW>(dw, blockIdx.x, reinterpret_cast<float *>(lds));
    else split_block<TM, WN, WK, K_CONTIG, K_CONTIG, EPI_MASK>(da, blockIdx.x - n_dw, lds);
}

// The same with 64x64 tiles of the fp32 instruction.
template <int EPI, int DW>
__global__ __launch_bounds__(256, 2) void gemm_da_narrow_dw_kernel(GemmArgs da, GemmArgs dw, unsigned n_dw)
{
    constexpr int NARROW = narrow_lds_floats<DW>(), WIDE = gemm_lds_floats<64, 64, 32, K_CONTIG, K_CONTIG>();
    __shared__ __attribute__((aligned(16))) float lds[NARROW > WIDE ? NARROW : WIDE];
    if (dw.mean.blocks > 0 && blockIdx.x >= dw.mean.first_block) mean_loss_block(dw.mean, blockIdx.x - dw.mean.first_block);
    else if (blockIdx.x < n_dw) narrow_dw_any<EPI, DW>(dw, blockIdx.x, lds);
    else gemm_block<64, 64, 32, 2, 2, K_CONTIG, K_CONTIG, true, EPI_MASK>(da, blockIdx.x - n_dw, lds);
}

}  // namespace easgd
