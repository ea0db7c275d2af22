// Step (1) of a Sync EASGD round (Section 5.1): the minibatch gradient of every
// worker at its own weights, for a dense ReLU MLP with softmax cross-entropy
// (forward / backward propagation of Section 2.2), written straight into the
// packed gradient buffer (the packed single-buffer layout of Section 5.2).
//
// Per layer l (d_in = dims[l], d_out = dims[l+1]) the packed block is the
// (d_in+1) x d_out matrix [W_l ; b_l], so with a ones column appended to the
// layer input A_l the three products are
//   forward   Z_l      = [A_l 1] * [W_l ; b_l]                (b x d_out),  A_{l+1} = relu(Z_l)
//   weights   [dW;db]  = [A_l 1]^T * dZ_l                     ((d_in+1) x d_out, contiguous in G)
//   inputs    dZ_{l-1} = (dZ_l * W_l^T) masked by A_l > 0     (b x d_in)
// The last layer's logits are produced as split-K partial sums that the softmax
// kernel adds in ascending split order, so every sum has a fixed order; a last
// layer of at most 16 classes instead takes one launch for its forward product,
// the softmax and its input-gradient product (mlp_head_kernel).
//
// The same sequence of launches also serves the whole round in one call
// (easgd_mlp_round, steps (1)-(5)): Eq. (2) runs ahead of backward propagation
// (on extra blocks of the first forward launch, on a second stream, or as a
// kernel of its own), the input-gradient product of a layer runs before its
// weight-gradient product, and that product applies the worker rule Eq. (1) /
// Eq. (5),(6) to the layer's slice of every replica in its epilogue.
#include "gemm_chain.h"
#include "gemm_split.h"
#include "shared_launches.h"
#include "mlp_head.h"
#include "persistent_round.h"
#include <algorithm>
#include <initializer_list>
#include <mutex>

// The workspace of easgd_grad_static: device memory that belongs to the library, one copy per GPU, held from
// the moment the library is loaded on that GPU until the process ends.  In host code this name is only a
// stand-in for the symbol; the device address is looked up once per device (static_scratch below).
static __device__ __align__(256) unsigned char scratch[EASGD_STATIC_SCRATCH_BYTES];

namespace easgd {

static constexpr int MAX_LAYERS = 8;
static constexpr int MAX_CLASSES = 1024;
static constexpr int MAX_SPLITS = 16;

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

struct GradPlan {
    size_t N = 0;
    size_t off[MAX_LAYERS] = {0};       // packed offset of layer l
    size_t act_off[MAX_LAYERS] = {0};   // workspace offset (bytes) of A_l, l = 1..L-1
    size_t logits_off = 0, rowloss_off = 0, dz_off[3] = {0, 0, 0};
    size_t bytes = 0;
    int splits = 1, k_per_split = 0;
    size_t center_off = 0, round_bytes = 0;
};

// Slab depth of the 128x32 tile (logits, narrow weight gradients).  These products are latency-bound: a block has
// a handful of slabs and little to multiply per slab, so fewer, deeper slabs win (32 against 16: the logits of a
// 2048-wide layer 26 -> 19 us, a whole 784-10 round 25.8 -> 23.2 us).
static constexpr int SPLIT_BK = 32;

static bool make_plan(const int *dims, int L, int P, int b, GradPlan &pl)
{
    if (!dims || L < 1 || L > MAX_LAYERS || P < 1 || b < 1) return false;
    for (int l = 0; l <= L; ++l)
        if (dims[l] < 1) return false;
    size_t n = 0;
    for (int l = 0; l < L; ++l) {
        pl.off[l] = n;
        n += (size_t)dims[l] * dims[l + 1] + dims[l + 1];
    }
    pl.N = n;
    // split the long, skinny logits product over K so that enough blocks run
    const int K = dims[L - 1] + 1;
    int splits = (K + 127) / 128;
    if (splits > MAX_SPLITS) splits = MAX_SPLITS;
    if (splits < 1) splits = 1;
    int kps = (K + splits - 1) / splits;
    kps = (kps + SPLIT_BK - 1) / SPLIT_BK * SPLIT_BK;
    pl.k_per_split = kps;
    pl.splits = (K + kps - 1) / kps;

    size_t o = 0, widest = 0;
    for (int l = 1; l < L; ++l) {
        pl.act_off[l] = o;
        o += align_up((size_t)P * b * dims[l] * sizeof(float), 256);
    }
    for (int l = 1; l <= L; ++l) widest = dims[l] > (int)widest ? dims[l] : widest;
    pl.logits_off = o;
    o += align_up((size_t)pl.splits * P * b * dims[L] * sizeof(float), 256);
    pl.rowloss_off = o;
    o += align_up((size_t)P * b * sizeof(float), 256);
    for (int q = 0; q < 3; ++q) {
        pl.dz_off[q] = o;
        o += align_up((size_t)P * b * widest * sizeof(float), 256);
    }
    pl.bytes = o;
    pl.center_off = o;                   // whole-round call only: the center at time t
    pl.round_bytes = o + align_up(pl.N * sizeof(float), 256);
    return true;
}

// Softmax cross-entropy on the logits of all workers: one wavefront per sample row, the classes
// spread over the lanes.  Sums use fixed shuffle trees and fixed orders.
//   zpart [splits][rows][C] partial logits (added in ascending split order)
//   dz [rows][C] <- (softmax - onehot)/b;   row_loss[rows] <- -log softmax(label)
__global__ __launch_bounds__(256) void softmax_xent_kernel(const float *__restrict__ zpart, const int *__restrict__ y,
                                                           float *__restrict__ dz, float *__restrict__ row_loss,
                                                           int rows, int b, int C, int splits, size_t split_stride)
{
    const int lane = threadIdx.x & 63;
    const size_t row = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= (size_t)rows) return;
    const float inv_b = 1.0f / (float)b;
    const int label = y[row];
    float z[MAX_CLASSES / 64];               // up to 16 classes per lane
    float zmax = -INFINITY;
#pragma unroll
    for (int q = 0; q < MAX_CLASSES / 64; ++q) {
        const int c = lane + 64 * q;
        float v = -INFINITY;
        if (c < C) {
            v = 0.f;
            for (int s = 0; s < splits; ++s) v += zpart[s * split_stride + row * C + c];
        }
        z[q] = v;
        zmax = fmaxf(zmax, v);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, o));
    float sum = 0.f, zlabel = 0.f;           // zlabel: shifted logit of the true class (one lane holds it)
#pragma unroll
    for (int q = 0; q < MAX_CLASSES / 64; ++q) {
        const int c = lane + 64 * q;
        if (c < C) {
            if (c == label) zlabel = z[q] - zmax;
            z[q] = expf(z[q] - zmax);
            sum += z[q];
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) zlabel += __shfl_xor(zlabel, o);
    const float inv_sum = 1.0f / sum;
#pragma unroll
    for (int q = 0; q < MAX_CLASSES / 64; ++q) {
        const int c = lane + 64 * q;
        if (c < C) dz[row * C + c] = (z[q] * inv_sum - (c == label ? 1.f : 0.f)) * inv_b;
    }
    if (lane == 0) row_loss[row] = logf(sum) - zlabel;
}

// One launch for the head of the network; the grid may be extended by blocks that run the center rule (h.ctr).
template <int ROWS, int CP, bool ONE_PASS, int NT = 4>
__global__ __launch_bounds__(256) void mlp_head_kernel(HeadArgs h)
{
    __shared__ float part[4][ROWS * CP];
    __shared__ float dzs[ROWS][CP];
    if (h.ctr.blocks > 0 && blockIdx.x >= h.ctr.first_block) {         // uniform for the block
        const size_t cb = blockIdx.x - h.ctr.first_block;
        center_rule_block(h.ctr.W, h.ctr.Wc, h.ctr.old, h.ctr.P, h.ctr.N, h.ctr.ld, h.ctr.alpha, cb, h.ctr.blocks, threadIdx.x);
        return;
    }
    head_block<ROWS, CP, ONE_PASS, false, NT>(h, blockIdx.x, part, dzs);
}

// Whether the head of a network with these layer widths takes the single-launch path.
static bool head_fits(const int *dims, int L) { return dims[L] <= HEAD_MAX_C; }

template <int CP>
static void launch_head_cp(const HeadArgs &h, unsigned blocks, hipStream_t s)
{
    if (h.d_in <= 1024) EASGD_LAUNCH((mlp_head_kernel<HEAD_ROWS, CP, true>), dim3(blocks), dim3(256), 0, s, h);
    else if (h.d_in <= 2048) EASGD_LAUNCH((mlp_head_kernel<HEAD_ROWS, CP, true, 8>), dim3(blocks), dim3(256), 0, s, h);
    else EASGD_LAUNCH((mlp_head_kernel<HEAD_ROWS, CP, false>), dim3(blocks), dim3(256), 0, s, h);
}

static unsigned head_blocks(int P, int b) { return (unsigned)P * (unsigned)((b + HEAD_ROWS - 1) / HEAD_ROWS); }

static void launch_head(HeadArgs h, hipStream_t s)
{
    unsigned blocks = head_blocks(h.P, h.b);
    if (h.ctr.blocks > 0) {
        h.ctr.first_block = blocks;
        blocks += h.ctr.blocks;
    }
    if (h.C <= 4) launch_head_cp<4>(h, blocks, s);
    else if (h.C <= 8) launch_head_cp<8>(h, blocks, s);
    else if (h.C <= 12) launch_head_cp<12>(h, blocks, s);
    else launch_head_cp<16>(h, blocks, s);
}

// ---- GEMM dispatch -------------------------------------------------------

enum Kind { FWD, DW, DA };

// The weight-gradient products of two layers (64x64 tiles both) in one launch: one launch boundary and one tail less.
template <int EPI>
static void launch_pair_dw_dw(GemmArgs d0, GemmArgs d1, hipStream_t s)
{
    const unsigned n0 = place_blocks<64, 64>(d0), n1 = place_blocks<64, 64>(d1);
    d0.mean.first_block = n0 + n1;
    EASGD_LAUNCH((gemm_dw_pair_kernel<EPI>), dim3(n0 + n1 + d0.mean.blocks), dim3(256), 0, s, d0, d1, n0);
}

template <int BM, int BN, int BK, int WM, int WN, int AL, int BL, int EPI, int MT = 32>
static void launch_tile(const GemmArgs &a_in, bool vec, hipStream_t s)
{
    GemmArgs a = a_in;
    size_t total = place_blocks<BM, BN>(a);
    static_assert(WM * WN * 64 == 256, "the center rule's extra blocks assume 256 threads");
    if (a.ctr.blocks > 0) {
        a.ctr.first_block = (unsigned)total;
        total += a.ctr.blocks;
    }
    a.mean.first_block = (unsigned)total;
    total += a.mean.blocks;
    const dim3 grid((unsigned)total), block(WM * WN * 64);
    if (vec) EASGD_LAUNCH((gemm_mfma_kernel<BM, BN, BK, WM, WN, AL, BL, true, EPI, MT>), grid, block, 0, s, a);
    else if constexpr (AL == K_CONTIG && BL == MN_CONTIG && BN > 32)
        EASGD_LAUNCH((gemm_mfma_kernel<BM, BN, BK, WM, WN, AL, BL, true, EPI, MT, true>), grid, block, 0, s, a);
    else EASGD_LAUNCH((gemm_mfma_kernel<BM, BN, BK, WM, WN, AL, BL, false, EPI, MT>), grid, block, 0, s, a);
}

// A batch that is not a multiple of 32 rows wastes matrix-core time in 32-row MFMA tiles (b = 100: 128 rows are
// multiplied, 28 % more than stored).  The 16x16x4 instruction has the same rate, so a block tile of 3, 5 or 7 x 16
// rows by 128 columns (four wavefronts side by side, 3, 5 or 7 x 2 accumulators each) multiplies 48, 80 or 112
// rows per tile.  It is chosen for the products whose M is the batch (forward, input gradient) when one of the
// three heights covers M with fewer rows than 32-row tiles do and still gives every compute unit about two
// blocks.  Returns that height, or 0.
static int tile16_rows(int M, int N, int P, int splits)
{
    if (N <= 32) return 0;
    long best_rows = (long)((M + 31) / 32) * 32;
    int best = 0;
    for (int bm : {112, 80, 48}) {
        const long rows = (long)((M + bm - 1) / bm) * bm;
        if (rows < best_rows) {
            best_rows = rows;
            best = bm;
        }
    }
    if (best == 0) return 0;
    return (size_t)((M + best - 1) / best) * ((N + 127) / 128) * splits * P >= (size_t)(2 * num_cus()) ? best : 0;
}

// ---- products on the bfloat16 matrix cores (gemm_split.h) ----

static bool split_fits(const GemmArgs &a, bool a_k_contig, bool b_k_contig)
{
    // byte offsets inside an operand of one worker are 32 bits wide
    const size_t ra = a_k_contig ? a.M : a.K, rb = b_k_contig ? a.N : a.K, lim = (size_t)1 << 30;
    return (ra + 128) * (size_t)a.lda < lim && (rb + 128) * (size_t)a.ldb < lim;
}

// The products whose rows are the minibatch (forward, input gradient): the largest tile that still gives every compute unit
// a block.  The smaller the grid, the more a block's own chain of slabs decides, and the more wavefronts share a tile along
// k (the last two numbers of a tile's name in gemm_split.h).  Measured, us per product, 128x128 / 64x128 / 64x64 / 32x32, and
// the fp32 instruction's best tile (forward: d_in -> d_out, workers, minibatch):
//   3072->2048, 32, 100   276 / 291 / 359 / 521     365
//   3072->2048,  8, 256   147 / 150 / 182 / 258     207
//    784->1024, 16, 128    37 /  27 /  29 /  40      32
//   1023-> 777,  6,  37    41 /  28 /  21 /  15      48 (no 128-bit loads)
//    784-> 500,  8,  50    34 /  24 /  17 /  11      18
// SPLIT_NONE where the fp32 instruction is faster: below a length of the sum that depends on the tile and on how full its
// grid is (a block of the split form takes longer to start), and for small tiles whenever the 64x64 tiles of the fp32
// instruction just fill the chip, since the split form then has to multiply in tiles that load more per product.  Time of
// the fp32 instruction over that of the split form at sums of 64, 128, 256, 512 (first the shape as columns, workers, rows):
//                              forward                    input gradient, 128-bit loads
//   128x128  2048, 24, 128     0.90 1.02 1.19 1.22        0.94 1.16 1.27 1.24
//   128x128  1024, 32, 128     0.76 0.88 1.06 1.25        0.80 0.93 1.11 1.29
//   128x128  2048, 20,  80     0.86 0.94 1.08 1.18        0.92 1.05 1.12 1.20     (input gradient 2066, 22, 74, a sum of 92: 18.2 us / 16.9)
//   64x128   1024, 16, 128     0.74 0.82 0.91 1.05        0.80 0.87 1.00 1.12
//   64x128   2048, 32,  64     1.26 1.49 1.79 1.98        0.92 1.06 1.19 1.11
//   64x64     768, 12, 192     0.73 0.83 0.94 1.06        0.81 0.87 1.00 1.10
//   64x64     512, 16, 128     0.67 0.72 0.78 0.87        0.73 0.79 0.84 0.87     (sum of 2048: 0.99, 0.96)
//   32x128   2048, 16,  20     0.80 0.85 0.99 1.15        0.91 1.04 1.15 1.29
//   32x32     512,  8,  50     0.86 0.93 1.10 1.37        1.01 1.10 1.30 1.54
//   32x32     256, 16, 128     0.71 0.75 0.91 1.13        0.84 0.93 1.07 1.22
//   32x32     500, 10, 100     0.66 0.71 0.81 0.94        0.81 0.87 0.94 1.04
//   32x32     500, 15, 100     0.58 0.63 0.69 0.78        0.74 0.77 0.83 0.86     (sum of 2048: 0.92, 0.90)
//   32x32     640, 32,  16     0.80 0.93 1.18 1.48        0.96 1.16 1.37 1.67
// Input gradients whose widths rule out 128-bit loads on the fp32 path (301, 5, 90: 1.28 1.63 2.23; 257, 16, 127: 0.99 1.19
// 1.53; 1023, 16, 128 1.01 at a sum of 49) take the split form from sums of 40 on, or 64 on a large grid of the smallest
// tile; forward products of such widths, whose 128-bit loads straddle cache lines,
// at nine sixteenths of the length (logits of 112 inputs, 106 classes, 3 workers, 162 rows: 8.4 us against 6.8; of 3072, 593,
// 3, 124 in sums of 224: 22.7 against 18.4).  Where the fp32 instruction would multiply in 16-row tiles, whose start is slow,
// the split form takes all but the shortest sums (2048, 32, 100: 1.06 and 1.26 at 48; input gradient of 1224, 18, 234, a sum of
// 68: 28.4 us against 18.0).
static SplitPick split_pick(const GemmArgs &a, bool forward, bool vec, bool any_length = false)
{
    if (options().gemm_tile != 0 || a.N <= 32 || !split_fits(a, true, !forward)) return SPLIT_NONE;
    const size_t cus = (size_t)num_cus();
    auto blocks = [&](int bm, int bn) { return (size_t)((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn) * (size_t)a.P * (size_t)a.splits; };
    constexpr int NEVER = 0x7fffffff;
    const size_t fp32 = blocks(64, 64);                      // the grid of the fp32 instruction's tile
    SplitPick pick;
    int least;                                               // shortest sum
    if (a.M > 64 && blocks(128, 128) >= cus) {
        pick = SPLIT_128x128;
        const size_t n = blocks(128, 128);
        least = forward ? (2 * n >= 3 * cus ? 128 : 192) : (4 * n >= 5 * cus ? 72 : 160);
    } else if (a.M > 32 && blocks(64, 128) >= cus) {
        pick = SPLIT_64x128;
        least = blocks(64, 128) >= 2 * cus ? (forward ? 0 : 96) : (forward ? 384 : 256);
    } else if (a.M > 32 && blocks(64, 64) >= cus) {
        pick = SPLIT_64x64;
        least = fp32 <= cus ? NEVER : (forward ? 384 : 256);
    } else if (a.M <= 32 && blocks(32, 128) >= cus) {
        pick = SPLIT_32x128;
        const size_t n = blocks(32, 128);
        least = !forward ? 112 : n >= 2 * cus ? 0 : 2 * n >= 3 * cus ? 192 : 288;
    } else {
        pick = SPLIT_32x32;
        const size_t n = blocks(32, 32);
        if (n <= cus || fp32 > cus) least = forward ? 192 : 112;
        else if (n <= 2 * cus) least = forward ? 384 : 192;
        else least = 5 * fp32 > 4 * cus && a.M > 32 ? NEVER : (forward ? 768 : 384);
    }
    if (!vec) {
        if (!forward) least = least == NEVER ? 128 : std::min(least, pick == SPLIT_32x32 && blocks(32, 32) > 2 * cus ? 64 : 40);
        else if (least != NEVER) least = least / 16 * 9;
    }
    if (tile16_rows(a.M, a.N, a.P, a.splits) != 0) least = std::min(least, 32);
    return any_length || std::min(a.K, a.k_per_split) >= least ? pick : SPLIT_NONE;
}

// Whether a 64x64 or a forward product's 32x128 split tile requests both operands of a slab before it waits for either (EARLY in
// gemm_split.h): where the trips to memory are long, on operands and results of more than a third of the last-level cache (80 MB), or
// bare, on a single block per compute unit; the 32x128 tile where both hold.  Time of that order over the other one on operands that
// are not in the second-level cache, 64x64: below 80 MB and on more than one block per unit 0.95 to 1.12, elsewhere 0.89 to 1.05;
// 32x128: 0.91 to 1.03 by this rule, 0.96 to 1.04 elsewhere.  us, one after the other / early: 3008->544, 30 workers, 53 rows 91.3 /
// 81.9; input gradients 608->1824, 16, 114 59.8 / 53.3 and 500->641, 16, 128 20.7 / 18.5; 2924->2020, 16, 18 (32x128) 89.4 / 82.6.
static bool split_early(const GemmArgs &a, SplitPick pick)
{
    const bool far = (double)a.P * ((double)a.M * a.K + (double)a.N * a.K + (double)a.M * a.N) > 20e6;
    const int bn = pick == SPLIT_64x64 ? 64 : 128, bm = pick == SPLIT_64x64 ? 64 : 32;
    const bool bare = (size_t)((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn) * (size_t)a.P * (size_t)a.splits <= (size_t)num_cus();
    return pick == SPLIT_64x64 ? far || bare : far && bare;
}

// ---- fp32 products of small grids (gemm_chain.h) ----

// Which tile of gemm_chain.h takes the place of the fp32 instruction's 64x64 tile: rows x columns, or none.
enum ChainPick { CHAIN_NONE, CHAIN_32x32, CHAIN_16x64, CHAIN_32x64 };

// All of them give the same bits, so only time counts: a launch takes a_r + d_r K us, where r is the number of blocks per compute
// unit, rounded up, and K the length of the sum (for the chain tiles in whole slabs of 64).  The constants are fitted to 9 600
// products of forward and backward propagation of up to 900 64x64 tiles, sums of 48 to 3072, each timed in all four tiles
// on operands that are not in the second-level cache.  Half of the times are met to 3 % and nine of ten to 9 % (16x64: 11 %), so a
// chain tile has to promise 1.5 % over the 64x64 tile: it then is more than 2 % slower in one of 160 of the products that come
// here, and 12 % at most (several blocks per unit, sums below 330).  us, 64x64 / 32x32 / 16x64 / 32x64 (64x32 is almost never the best):
//   forward         784-> 500,  8 workers,  50 rows     18.2 /  8.7 /  9.3 / 11.9
//                  1023-> 777,  6,  37                  23.2 / 14.3 / 10.4 / 14.1
//                   784->1520,  4,  64                  18.3 / 13.4 / 14.6 / 12.3
//                  3072-> 427,  7,  38                  59.5 / 20.3 / 21.0 / 33.7
//                   208-> 944, 13, 151                  15.1 / 18.6 / 22.8 / 17.2    (stays)
//                   784-> 640, 12, 100                  18.5 / 22.7 / 25.3 / 21.1    (stays)
//   input gradient   95-> 222,  6, 132                  12.9 /  4.4 /  4.8 /  5.9    (no 128-bit loads for 64x64)
//                  1024-> 100, 32,  64                   9.4 / 14.5 / 18.1 / 13.9    (stays)
static ChainPick chain_pick(const GemmArgs &a, bool forward, bool vec)
{
    if (options().gemm_tile != 0 || a.N <= 32 || !split_fits(a, true, !forward)) return CHAIN_NONE;
    const size_t cus = (size_t)num_cus();
    auto blocks = [&](int bm, int bn) { return (size_t)((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn) * (size_t)a.P * (size_t)a.splits; };
    if (2 * blocks(64, 64) > 5 * cus) return CHAIN_NONE;
    const int sum = std::min(a.K, a.k_per_split), slabs = (sum + 63) / 64 * 64;
    struct Line { double a, d; };
    // input gradients that rule out 128-bit loads on the 64x64 path take about twice as long there
    const bool slow = !forward && !vec;
    // lines: r = 1, 2, ..; beyond the last one in proportion to it
    auto time = [&](int bm, int bn, int K, std::initializer_list<Line> lines) {
        const size_t r = (blocks(bm, bn) + cus - 1) / cus, n = std::min(r, lines.size());
        const Line &l = lines.begin()[n - 1];
        // with more than four blocks per unit the chain tiles' loads, several times the 64x64 tile's per product, decide in long sums
        // (3072->1554, 9 workers, 70 rows: five blocks of 16x64 take a gradient of 212 us to 247)
        if (r > n && bm * bn < 64 * 64 && !slow) return 1e9;
        return (double)r / (double)n * (l.a + l.d * K);
    };
    double best = 0.985 * (slow ? time(64, 64, sum, {{3.54, 0.0437}, {3.19, 0.0744}, {4.91, 0.1050}})
                                : time(64, 64, sum, {{3.74, 0.01756}, {4.66, 0.03255}, {5.94, 0.0467}}));
    ChainPick pick = CHAIN_NONE;
    auto consider = [&](ChainPick t, double us) {
        if (us < best) {
            best = us;
            pick = t;
        }
    };
    consider(CHAIN_32x32, time(32, 32, slabs, {{3.23, 0.00535}, {3.83, 0.01042}, {4.34, 0.01542}, {5.38, 0.01977}}));
    consider(CHAIN_16x64, time(16, 64, slabs, {{3.42, 0.00581}, {4.13, 0.01164}, {4.96, 0.0178}, {6.15, 0.02172}}));
    consider(CHAIN_32x64, time(32, 64, slabs, {{3.42, 0.00991}, {4.34, 0.01825}, {6.2, 0.0277}, {7.5, 0.035}}));
    return pick;
}

template <int WM, int WN, int TM, int BL, int EPI>
static void launch_chain(const GemmArgs &a_in, hipStream_t s)
{
    typedef ChainTile<WM, WN, TM, BL> T;
    GemmArgs a = a_in;
    size_t total = place_blocks<T::BM, T::BN>(a);
    if (a.ctr.blocks > 0) {
        a.ctr.first_block = (unsigned)total;
        total += a.ctr.blocks;
    }
    EASGD_LAUNCH((gemm_chain_kernel<WM, WN, TM, BL, EPI>), dim3((unsigned)total), dim3(256), 0, s, a);
}

template <int TM, int WN, int WK, int AL, int BL, int EPI, bool EARLY = false>
static void launch_split(const GemmArgs &a_in, hipStream_t s)
{
    GemmArgs a = a_in;
    size_t total = place_blocks<TM * 32, WN * 32>(a);
    if (a.ctr.blocks > 0) {
        a.ctr.first_block = (unsigned)total;
        total += a.ctr.blocks;
    }
    a.mean.first_block = (unsigned)total;
    total += a.mean.blocks;
    EASGD_LAUNCH((gemm_split_kernel<TM, WN, WK, AL, BL, EPI, EARLY>), dim3((unsigned)total), dim3(256), 0, s, a);
}

// Weight gradients: whether 64x128 split tiles can take the product (not on grids of less than two blocks per compute unit
// when the fp32 path has 128-bit loads: 784->500, 8 workers, 50 rows 10.2 us against 9.3).
static size_t split_dw_blocks(const GemmArgs &a) { return (size_t)((a.M + 63) / 64) * ((a.N + 127) / 128) * (size_t)a.P; }

static bool split_dw_fits(const GemmArgs &a, bool vec)
{
    return options().gemm_tile == 0 && a.N > 32 && split_fits(a, false, false) && (!vec || split_dw_blocks(a) >= (size_t)(2 * num_cus()));
}

// ... and whether they are faster than the 64x64 tiles of the fp32 instruction: where the products that they multiply for
// nothing, in half empty tiles of columns and in the last slab of 32 rows, leave them the advantage.  The same for all
// epilogues, so that the gradient of a round is that of easgd_grad.  With 128-bit loads on the fp32 path, time of the fp32
// instruction over that of the split form at 24, 32, 50, 64, 100, 128 rows (layer, workers), no worker rule:
//   1024->1024, 16   1.08 1.16 1.00 1.14 1.16 1.29
//   2048->2048,  2   0.97 1.03 0.92 1.04 1.07 1.21
//   1944-> 648,  8   at 135 rows, five slabs and eleven of twelve half tiles: 1.14
//   1024-> 160, 32   0.77 0.89 0.79 0.91 0.88 0.99
//   1024->  48, 32   0.64 0.74 0.67 0.73 0.71 0.83
// With the worker rule in the epilogue both move the replicas as well and there is less to gain; us a round gained or lost
// (784-1024-10, 16 workers: -0.5 -1.4 +3.7 +2.7 +1.9 -1.8; 3072-2048-10, 8: -3.5 -0.0 +7.2 +4.4 +0.4 -16.4; 3072-600, 32, with
// momentum: -20 at 100 rows).
// Without 128-bit loads (no worker rule):
//   1023->1022, 16   1.16 1.32 1.37 1.57 1.68 1.99   (with the rule, at 40 rows: +2.2 us of 70)
//    783->1024,  4   0.98 1.12 1.16 1.40 1.47 1.80   (416 blocks)
//    601-> 641,  4   0.88 0.96 0.97 1.10 1.16 1.39   (240 blocks; with the rule +1.5 +1.0 +1.2 +0.2 -0.5 -2.5 us)
//    255-> 500,  3   0.77 0.83 0.77 0.90 0.90 1.11   (48 blocks; with the rule +0.2 us at 128 rows)
//    783->  35, 20   0.76 0.82 0.81 0.94 0.93 1.12   (260 blocks, the columns of half a tile)
static bool split_dw_pays(const GemmArgs &a, bool vec)
{
    if (!split_dw_fits(a, vec)) return false;
    const size_t cus = (size_t)num_cus(), blocks = split_dw_blocks(a);
    if (vec) {
        if (a.K > 32 && a.K <= 96) return false;
        const long columns = (a.N + 127) / 128 * 2, needed = (a.N + 63) / 64;        // in tiles of 64
        const long multiplied = (a.K + 31) / 32 * 32 * columns, useful = a.K * needed;
        return 100 * multiplied <= (a.K > 96 ? 130 : 134) * useful;
    }
    if (a.N <= 64 || 2 * blocks < cus) return a.K >= 120;
    if (blocks >= 2 * cus) return a.K >= 20 && !(a.K > 32 && a.K < 42);
    return a.K >= (4 * blocks >= 5 * cus ? 44 : 54);
}

// In which form two weight gradients that follow one another are computed, so that they can share a launch; or each in the form
// that pays for it, in a launch of its own.  Where both forms can take both, the split form if it pays for two fifths of the
// work (gradient of 628-1888-816-10, 6, 103: 136 us against 142).  Where only the fp32 form can take both, that one, up to the
// size at which the split form's gain on one of them makes up for a launch (rounds of 3072-512-256-10, 128 rows, one
// launch / two: 4 workers 119.9 / 128.2 us, 8 140.9 / 145.8, 16 184.6 / 181.7; 3072-768-128-10, 16: 265.5 / 256.3).  Where only
// the split form can take both, that one (gradient of 1390-126-205-10, 7, 56: 59.6 us against 65.5 in two launches).
// EASGD_OPT_GEMM_PAIR has no say: it changes no bit.
enum Form { FORM_BY_SIZE, FORM_FP32, FORM_SPLIT };

static Form dw_pair_form(const GemmArgs &a0, bool vec0, const GemmArgs &a1, bool vec1, bool fp32_only)
{
    const long tile = options().gemm_tile;
    if (a0.N <= 32 || a1.N <= 32) return FORM_BY_SIZE;
    const bool fp32 = (tile == 0 || tile == 2) && vec0 && vec1;
    const bool split = !fp32_only && split_dw_fits(a0, vec0) && split_dw_fits(a1, vec1);
    if (!fp32 || fp32_only) return split ? FORM_SPLIT : fp32 ? FORM_FP32 : FORM_BY_SIZE;
    const bool pays0 = split_dw_pays(a0, vec0), pays1 = split_dw_pays(a1, vec1);
    const double size0 = (double)a0.M * a0.N, size1 = (double)a1.M * a1.N;
    if (split) return (pays0 ? size0 : 0) + (pays1 ? size1 : 0) >= 0.4 * (size0 + size1) ? FORM_SPLIT : FORM_FP32;
    const double gain = (pays0 ? size0 * a0.K * a0.P : 0) + (pays1 ? size1 * a1.K * a1.P : 0);
    return gain >= 3.0e9 ? FORM_BY_SIZE : FORM_FP32;
}

template <int EPI>
static void launch_split_pair_dw_dw(GemmArgs d0, GemmArgs d1, hipStream_t s)
{
    const unsigned n0 = place_blocks<64, 128>(d0), n1 = place_blocks<64, 128>(d1);
    d0.mean.first_block = n0 + n1;
    EASGD_LAUNCH((gemm_split_dw_pair_kernel<2, 4, 1, EPI>), dim3(n0 + n1 + d0.mean.blocks), dim3(256), 0, s, d0, d1, n0);
}

// Weight gradients of at most 32 columns: narrow_dw.h or the 128x32 tile (same bits).  A wavefront of the first covers sixteen rows
// and reads all of dZ for them, one of the second thirty-two from LDS: the first wins where the launch is bound by latency, and
// loses where many wavefronts share a compute unit.  us, 128x32 / narrow (layer, workers, rows; plain gradients): 784->10, 4, 64
// 5.9 / 3.5 (with momentum 7.0 / 4.2), 2048->10, 32, 100 15.1 / 9.2, 3072->10, 32, 256 45.2 / 24.8, 2047->17, 20, 77 9.9 / 9.2.
// Time narrow / 128x32 over 2 000 products by blocks of 64 rows per compute unit, at sums below 128 and above:
//   at most 16 columns   128-bit loads ruled out   0.35 to 0.86 everywhere
//                        128-bit loads             up to 1: 0.66 to 0.84, 0.68 to 0.82; above: 0.74 to 0.92, 0.93 to 1.17
//   17 to 32 columns     128-bit loads ruled out   up to 3: 0.57 to 0.99; above: 0.88 to 1.14
//                        128-bit loads             1024->32, 32 workers, 256 rows 13.3 us / 19.7
static bool narrow_dw_fits(const GemmArgs &a, bool vec)
{
    const size_t cus = (size_t)num_cus(), blocks = (size_t)((a.M + 63) / 64) * (size_t)a.P;
    if (a.N <= 16) return !vec || blocks <= cus || a.K <= 128;
    return a.N <= 32 && !vec && blocks <= 3 * cus;
}

template <int TN, int EPI>
static void launch_narrow_dw(const GemmArgs &a_in, hipStream_t s)
{
    GemmArgs a = a_in;
    const unsigned total = place_blocks<64, 16 * TN>(a);
    a.mean.first_block = total;
    EASGD_LAUNCH((narrow_dw_kernel<TN, EPI>), dim3(total + a.mean.blocks), dim3(256), 0, s, a);
}

// Picks the tile shape.  Outputs at most 32 wide use a 128x32 tile of the fp32 matrix instruction, or as weight gradients
// narrow_dw.h; small grids of the products whose rows are the minibatch the tiles of gemm_chain.h; input gradients, a
// wide last layer and weight gradients the tiles of gemm_split.h where split_pick and split_dw_pays say so; everything else, and
// whatever EASGD_OPT_GEMM_TILE forces, tiles of the fp32 instruction: 64x64 blocks (four per compute unit, so that the
// epilogue of one overlaps the products of the others), for the products whose rows are the minibatch the 16-row tiles and
// for the forward products 128x128 where they still give every compute unit about two blocks.
// form: the caller's choice of the instruction (FORM_SPLIT where the product fits it).
template <int AL, int BL, int EPI>
static void launch_gemm(const GemmArgs &a, bool vec, hipStream_t s, Form form = FORM_BY_SIZE)
{
    if (a.N <= 32) {
        if constexpr (AL == MN_CONTIG && BL == MN_CONTIG) {
            if (narrow_dw_fits(a, vec)) {
                if (a.N <= 16) launch_narrow_dw<1, EPI>(a, s);
                else launch_narrow_dw<2, EPI>(a, s);
                return;
            }
        }
        launch_tile<128, 32, SPLIT_BK, 4, 1, AL, BL, EPI>(a, vec, s);
        return;
    }
    constexpr bool forward = AL == K_CONTIG && BL == MN_CONTIG;
    long tile = options().gemm_tile;
    if constexpr (AL == K_CONTIG) {
        const SplitPick pick = form == FORM_FP32 ? SPLIT_NONE : split_pick(a, forward, vec, form == FORM_SPLIT);
        if (pick == SPLIT_128x128) launch_split<4, 4, 1, AL, BL, EPI>(a, s);
        else if (pick == SPLIT_64x128) launch_split<2, 4, 1, AL, BL, EPI>(a, s);
        else if (pick == SPLIT_64x64) {
            if (split_early(a, pick)) launch_split<2, 2, 2, AL, BL, EPI, true>(a, s);
            else launch_split<2, 2, 2, AL, BL, EPI>(a, s);
        } else if (pick == SPLIT_32x128) {
            if constexpr (forward) {
                if (split_early(a, pick)) launch_split<1, 4, 1, AL, BL, EPI, true>(a, s);
                else launch_split<1, 4, 1, AL, BL, EPI>(a, s);
            } else launch_split<1, 4, 1, AL, BL, EPI>(a, s);
        }
        else if (pick == SPLIT_32x32) launch_split<1, 1, 4, AL, BL, EPI>(a, s);
        if (pick != SPLIT_NONE) return;
        int bm16 = (tile == 0) ? tile16_rows(a.M, a.N, a.P, a.splits) : 0;
        if (tile == 4) bm16 = a.M <= 48 ? 48 : a.M <= 80 ? 80 : 112;    // forced: the smallest height that covers M, else 112
        if (bm16 == 112) launch_tile<112, 128, 32, 1, 4, AL, BL, EPI, 16>(a, vec, s);
        else if (bm16 == 80) launch_tile<80, 128, 32, 1, 4, AL, BL, EPI, 16>(a, vec, s);
        else if (bm16 == 48) launch_tile<48, 128, 32, 1, 4, AL, BL, EPI, 16>(a, vec, s);
        if (bm16) return;
        const ChainPick chain = chain_pick(a, forward, vec);
        if (chain == CHAIN_32x32) launch_chain<2, 2, 1, BL, EPI>(a, s);
        else if (chain == CHAIN_16x64) launch_chain<1, 4, 1, BL, EPI>(a, s);
        else if (chain == CHAIN_32x64) launch_chain<1, 4, 2, BL, EPI>(a, s);
        if (chain != CHAIN_NONE) return;
    } else if (form == FORM_SPLIT ? split_dw_fits(a, vec) : form == FORM_BY_SIZE && split_dw_pays(a, vec)) {
        launch_split<2, 4, 1, AL, BL, EPI>(a, s);
        return;
    }
    const size_t big = (size_t)((a.M + 127) / 128) * ((a.N + 127) / 128) * a.splits * a.P;
    if (tile == 4) tile = 0;            // the weight-gradient products have no 16-row form
    if (tile == 0) tile = (forward && big >= (size_t)(2 * num_cus())) ? 1 : 2;
    if (tile == 1) launch_tile<128, 128, 16, 2, 2, AL, BL, EPI>(a, vec, s);
    else if (tile == 2) launch_tile<64, 64, 32, 2, 2, AL, BL, EPI>(a, vec, s);
    else launch_tile<128, 64, 32, 2, 2, AL, BL, EPI>(a, vec, s);
}

static inline bool mult4(size_t x) { return (x & 3u) == 0; }

// Whether the launch of a forward product leaves room on the chip for extra blocks that do bandwidth-bound work beside it.
// Mirrors launch_gemm: the 128x32 and 64x64 tiles use few enough registers and LDS for four blocks per compute unit, the
// 128x128 tile for two, and it is chosen exactly when its blocks already fill those; the split tiles of 64 and 128 rows three
// and two (split_blocks_per_cu).  The 32-row ones leave room whatever their number (rounds with the rule on extra blocks /
// as a launch of its own: 3072-99, 17, 30, 952 blocks 47.0 / 52.3 us; 3072-400, 32, 32, 2048 blocks 158 / 165; 2000-500, 16, 32,
// 1024 blocks 91 / 95); 64x128: 3072-593, 3, 124, 420 blocks 79 / 84; 128x128 more than one per unit: 512-1000, 32, 200 198 / 191.
// The tiles of gemm_chain.h, which a product of at most two and a half 64x64 tiles per unit may take instead, leave two or three
// blocks per unit room and lend the rule's blocks their LDS, and still always have room: 625 drawn rounds that begin
// with one, the rule as a launch of its own over the rule on extra blocks 1.00 to 1.22, median 1.07 (784-112-7, 25, 18 35.7 us /
// 29.3; 3072-1504-1440-10, 3, 42 145.8 / 145.2).
static bool forward_launch_has_room(const GemmArgs &a, bool vec, Form form)
{
    const size_t cus = (size_t)num_cus();
    auto blocks = [&](int bm, int bn) { return (size_t)((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn) * (size_t)a.splits * (size_t)a.P; };
    if (a.N <= 32) return blocks(128, 32) <= 3 * cus;
    switch (form == FORM_FP32 ? SPLIT_NONE : split_pick(a, true, vec, form == FORM_SPLIT)) {
    case SPLIT_128x128: return blocks(128, 128) <= cus;
    case SPLIT_64x128: return blocks(64, 128) <= 2 * cus;
    case SPLIT_64x64: return blocks(64, 64) <= 2 * cus;
    case SPLIT_32x128:
    case SPLIT_32x32: return true;
    case SPLIT_NONE: break;
    }
    long tile = options().gemm_tile;
    if (tile == 4 || (tile == 0 && tile16_rows(a.M, a.N, a.P, a.splits) != 0)) return false;
    if (tile == 0) tile = (blocks(128, 128) >= 2 * cus) ? 1 : 2;
    return tile == 2 && blocks(64, 64) <= 3 * cus;
}

// Elastic update fused into the backward pass.  Eq. (2) runs first and saves the time-t
// center in the workspace for the worker rules; the worker rule is the epilogue of each
// layer's weight-gradient product, which runs after the layer's input-gradient product, the
// last reader of W_l at time t.
struct ElasticStep {
    float *W, *V, *Wc;
    float eta, rho, delta;
    unsigned short *V16;    // momentum buffers stored as bfloat16 (then V is null), or null
};

static int grad_impl(const char *name, const int *dims, int n_layers, const float *W, size_t ld, const float *X,
                     const int32_t *y, int P, int b, float *G, float *loss, void *workspace, size_t workspace_bytes,
                     void *stream, const ElasticStep *step, unsigned short *G16 = nullptr);

// A second stream per device (default priority) with the two events that order it against the caller's
// stream: `fork` is recorded on the caller's stream when the round starts, `join` on the second stream when
// the center rule is done.  Created on first use and kept until the process ends; whole-round calls hold
// `side_mutex`, so that two host threads never interleave their record/wait pairs.
struct SideLane {
    hipStream_t stream = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
    bool tried = false, ok = false;
};
static std::mutex side_mutex;
static constexpr int MAX_DEVICES = 64;
static SideLane side_lanes[MAX_DEVICES];

static SideLane *side_lane()       // call with side_mutex held; nullptr when no lane can be made
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
    SideLane &ln = side_lanes[dev];
    if (!ln.tried) {
        ln.tried = true;
        ln.ok = hipStreamCreateWithFlags(&ln.stream, hipStreamNonBlocking) == hipSuccess &&
                hipEventCreateWithFlags(&ln.fork, hipEventDisableTiming) == hipSuccess &&
                hipEventCreateWithFlags(&ln.join, hipEventDisableTiming) == hipSuccess;
        if (!ln.ok) (void)hipGetLastError();
    }
    return ln.ok ? &ln : nullptr;
}

// Device address of `scratch` on the current device, looked up on the first call per device (with that device
// current) and kept; nullptr (and the error string set) when the lookup fails.
static void *static_scratch(const char *name)
{
    static std::mutex lookup_mutex;
    static void *ptrs[MAX_DEVICES] = {nullptr};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) {
        (void)hipGetLastError();
        fail(EASGD_ELAUNCH, "%s: no current device", name);
        return nullptr;
    }
    std::lock_guard<std::mutex> guard(lookup_mutex);
    if (!ptrs[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            fail(EASGD_ELAUNCH, "%s: address of the static workspace: %s", name, hipGetErrorString(e));
            return nullptr;
        }
        ptrs[dev] = p;
    }
    return ptrs[dev];
}

}  // namespace easgd

extern "C" {

size_t easgd_mlp_num_params(const int *dims, int n_layers)
{
    easgd::GradPlan pl;
    if (!easgd::make_plan(dims, n_layers, 1, 1, pl)) return 0;
    return pl.N;
}

size_t easgd_grad_workspace_bytes(const int *dims, int n_layers, int P, int b)
{
    easgd::GradPlan pl;
    if (!easgd::make_plan(dims, n_layers, P, b, pl)) return 0;
    return pl.bytes;
}

size_t easgd_mlp_round_workspace_bytes(const int *dims, int n_layers, int P, int b)
{
    easgd::GradPlan pl;
    if (!easgd::make_plan(dims, n_layers, P, b, pl)) return 0;
    return pl.round_bytes;
}

int easgd_grad(const int *dims, int n_layers, const float *W, size_t ld, const float *X, const int32_t *y,
               int P, int b, float *G, float *loss, void *workspace, size_t workspace_bytes, void *stream)
{
    return easgd::grad_impl("easgd_grad", dims, n_layers, W, ld, X, y, P, b, G, loss, workspace, workspace_bytes,
                            stream, nullptr);
}

int easgd_grad_static(const int *dims, int n_layers, const float *W, size_t ld, const float *X, const int32_t *y,
                      int P, int b, float *G, float *loss, void *stream)
{
    easgd::GradPlan pl;
    if (!easgd::make_plan(dims, n_layers, P, b, pl))
        return easgd::fail(EASGD_EINVAL, "easgd_grad_static: need 1 <= n_layers <= %d, all dims >= 1, P >= 1, b >= 1", easgd::MAX_LAYERS);
    if (pl.bytes > (size_t)EASGD_STATIC_SCRATCH_BYTES)
        return easgd::fail(EASGD_EWORKSPACE, "easgd_grad_static: this shape needs %zu bytes of workspace, the static workspace holds %zu; "
                           "use easgd_grad with a workspace of the caller", pl.bytes, (size_t)EASGD_STATIC_SCRATCH_BYTES);
    void *ws = easgd::static_scratch("easgd_grad_static");
    if (!ws) return EASGD_ELAUNCH;
    return easgd::grad_impl("easgd_grad_static", dims, n_layers, W, ld, X, y, P, b, G, loss, ws,
                            (size_t)EASGD_STATIC_SCRATCH_BYTES, stream, nullptr);
}

int easgd_grad_bf16(const int *dims, int n_layers, const float *W, size_t ld, const float *X, const int32_t *y,
                    int P, int b, uint16_t *G, float *loss, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!G) return easgd::fail(EASGD_EINVAL, "easgd_grad_bf16: NULL pointer");
    if (reinterpret_cast<uintptr_t>(G) & 1u) return easgd::fail(EASGD_EINVAL, "easgd_grad_bf16: G must be 2-byte aligned");
    return easgd::grad_impl("easgd_grad_bf16", dims, n_layers, W, ld, X, y, P, b, nullptr, loss, workspace,
                            workspace_bytes, stream, nullptr, G);
}

int easgd_mlp_round(const int *dims, int n_layers, float *W, float *V, float *Wc, size_t ld,
                    const float *X, const int32_t *y, int P, int b, float *G, float *loss,
                    float eta, float rho, float delta, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!Wc) return easgd::fail(EASGD_EINVAL, "easgd_mlp_round: NULL pointer");
    const easgd::ElasticStep step = {W, V, Wc, eta, rho, delta, nullptr};
    return easgd::grad_impl("easgd_mlp_round", dims, n_layers, W, ld, X, y, P, b, G, loss, workspace,
                            workspace_bytes, stream, &step);
}

int easgd_mlp_round_bf16v(const int *dims, int n_layers, float *W, uint16_t *V, float *Wc, size_t ld,
                          const float *X, const int32_t *y, int P, int b, float *G, float *loss,
                          float eta, float rho, float delta, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!Wc || !V) return easgd::fail(EASGD_EINVAL, "easgd_mlp_round_bf16v: NULL pointer");
    if (reinterpret_cast<uintptr_t>(V) & 1u) return easgd::fail(EASGD_EINVAL, "easgd_mlp_round_bf16v: V must be 2-byte aligned");
    const easgd::ElasticStep step = {W, nullptr, Wc, eta, rho, delta, V};
    return easgd::grad_impl("easgd_mlp_round_bf16v", dims, n_layers, W, ld, X, y, P, b, G, loss, workspace,
                            workspace_bytes, stream, &step);
}

}  // extern "C"

namespace easgd {

static int grad_impl(const char *name, const int *dims, int n_layers, const float *W, size_t ld, const float *X,
                     const int32_t *y, int P, int b, float *G, float *loss, void *workspace, size_t workspace_bytes,
                     void *stream, const ElasticStep *step, unsigned short *G16)
{
    const int L = n_layers;
    GradPlan pl;
    if (!W || !X || !y || (!G && !G16 && !step)) return fail(EASGD_EINVAL, "%s: NULL pointer", name);
    if (!make_plan(dims, L, P, b, pl))
        return fail(EASGD_EINVAL, "%s: need 1 <= n_layers <= %d, all dims >= 1, P >= 1, b >= 1", name, MAX_LAYERS);
    if (dims[L] > MAX_CLASSES) return fail(EASGD_EINVAL, "%s: at most %d classes, got %d", name, MAX_CLASSES, dims[L]);
    if (ld < pl.N) return fail(EASGD_EINVAL, "%s: ld (%zu) < N (%zu)", name, ld, pl.N);
    if (!aligned16(W) || !aligned16(G) || !aligned16(X)) return fail(EASGD_EINVAL, "%s: W, G, X must be 16-byte aligned", name);
    const size_t need_bytes = step ? pl.round_bytes : pl.bytes;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < need_bytes)
        return fail(EASGD_EWORKSPACE, "%s: workspace must be 256-byte aligned and hold %zu bytes (got %zu)", name, need_bytes, workspace_bytes);
    for (int l = 0; l < L; ++l) {
        const size_t per_worker = (size_t)(dims[l] + 1) * dims[l + 1];
        if (per_worker > 0x3fffffffull || (size_t)b * dims[l] > 0x3fffffffull || (size_t)b * dims[l + 1] > 0x3fffffffull)
            return fail(EASGD_ERANGE, "%s: layer %d exceeds 2^30-1 elements per worker", name, l);
    }
    if ((size_t)P * b * (size_t)pl.splits > 0x7fffffffull) return fail(EASGD_ERANGE, "%s: P*b too large", name);
    clear_error();

    hipStream_t s = static_cast<hipStream_t>(stream);
    char *ws = static_cast<char *>(workspace);
    auto act = [&](int l) -> const float * { return l == 0 ? X : reinterpret_cast<const float *>(ws + pl.act_off[l]); };
    float *logits = reinterpret_cast<float *>(ws + pl.logits_off);
    // dZ_l lives in buffer l % 3: the input-gradient product of layer l reads buffer l % 3 and writes (l-1) % 3
    // while the weight-gradient product of layer l+1, which may share its launch, still reads (l+1) % 3
    float *dz[3] = {reinterpret_cast<float *>(ws + pl.dz_off[0]), reinterpret_cast<float *>(ws + pl.dz_off[1]),
                    reinterpret_cast<float *>(ws + pl.dz_off[2])};

    // Replicas that exceed the last-level cache (256 MB): the weight gradients are bound by the replicas' stream, so
    // gemm_split.h has less to give (3072-2048-2048-10, 32 workers, 100 rows, with momentum: 2 207 us a round -> 2 119), and
    // with so many units its other rounding of the replicas moves a gate of the round after now and then.  All products
    // keep the fp32 instruction there, the logits included.
    const bool fp32 = (size_t)P * pl.N >= ((size_t)1 << 26);
    const Form by_size = fp32 ? FORM_FP32 : FORM_BY_SIZE;

    // a narrow last layer goes through mlp_head_kernel together with the softmax and its own input gradient
    const bool head = options().mlp_head != 0 && head_fits(dims, L);
    if (head && (size_t)P * ((b + HEAD_ROWS - 1) / HEAD_ROWS) > 0x3fffffffull) return fail(EASGD_ERANGE, "%s: P*b too large", name);

    // ---- a single-layer network small enough to be bound by launch boundaries: the whole call in one launch ----
    if (L == 1 && head && options().round_single_launch != 0 &&
        softmax_round_fits(dims[0], dims[1], b, P)) {
        SoftmaxRound r = {};
        r.X = X; r.y = y; r.W_in = W; r.G = G; r.G16 = G16;
        r.dz = dz[0]; r.row_loss = reinterpret_cast<float *>(ws + pl.rowloss_off); r.loss = loss;
        r.ld = ld; r.d_in = dims[0]; r.C = dims[1]; r.b = b; r.P = P;
        if (step) {
            r.W = step->W; r.V = step->V; r.V16 = step->V16; r.Wc = step->Wc;
            r.eta = step->eta; r.rho = step->rho; r.alpha = step->eta * step->rho; r.delta = step->delta;
            r.write_center = step->rho != 0.f;
        }
        if (softmax_round_launch(r, stream) == 0) return check_launch(name);
        // otherwise (stream under capture, no barrier words left): the separate launches below
    }

    // the product of layer l's forward propagation, its loads and its form
    auto forward_args = [&](int l) {
        const int d_in = dims[l], d_out = dims[l + 1];
        const bool last = (l == L - 1);
        GemmArgs a = {};
        a.A = act(l); a.a_ws = (size_t)b * d_in; a.lda = d_in; a.a_lim = d_in; a.a_ones = d_in;
        a.B = W + pl.off[l]; a.b_ws = ld; a.ldb = d_out;
        a.C = last ? logits : const_cast<float *>(act(l + 1)); a.c_ws = (size_t)b * d_out; a.ldc = d_out;
        a.M = b; a.N = d_out; a.K = d_in + 1; a.P = P;
        a.splits = last ? pl.splits : 1;
        a.k_per_split = last ? pl.k_per_split : ((a.K + 63) / 64 * 64);
        a.c_ss = (size_t)P * b * d_out;
        return a;
    };
    auto forward_vec = [&](int l) { return mult4(dims[l]) && mult4(dims[l + 1]); };     // 128-bit loads need the element's alignment only
    auto forward_form = [&](int l) { return l == L - 1 ? by_size : FORM_FP32; };

    // ---- Eq. (2); beside forward propagation when the second stream is in use ----
    // rho == 0: a local step.  Eq. (2) leaves the center as it is and Eq. (1) is a plain (momentum) SGD step, so
    // the center rule is not launched at all and the worker rule reads the center in place (times zero).
    const bool local_step = step && step->rho == 0.f;
    float *old_center = step ? reinterpret_cast<float *>(ws + pl.center_off) : nullptr;
    const float *center_t = local_step ? step->Wc : old_center;
    std::unique_lock<std::mutex> lane_guard;
    SideLane *lane = nullptr;
    bool attach_center = false;
    if (step && !local_step) {
        // Where Eq. (2) runs (EASGD_OPT_ROUND_OVERLAP): 0 = a kernel of its own on the caller's stream, 2 = the
        // same on the library's second stream, beside forward propagation, 3 = on extra blocks of the first
        // forward product's launch.  1 (default) chooses: the extra blocks when that launch leaves room on the
        // chip (they then fill idle wave slots, no stream is involved); else the second stream when the rule has
        // enough to read to be worth the tens of microseconds that ordering two streams costs; else its own kernel.
        const long overlap = options().round_overlap;
        const bool room = (head && L == 1) ? head_blocks(P, b) <= 3u * (unsigned)num_cus()
                                           : forward_launch_has_room(forward_args(0), forward_vec(0), forward_form(0));
        attach_center = (overlap == 3) || (overlap == 1 && room);
        if (!attach_center && (overlap == 2 || (overlap == 1 && (size_t)P * pl.N >= ((size_t)1 << 24)))) {
            lane_guard = std::unique_lock<std::mutex>(side_mutex);
            lane = side_lane();
        }
        const float alpha = step->eta * step->rho;
        int rc;
        if (lane) {
            if (hipEventRecord(lane->fork, s) != hipSuccess || hipStreamWaitEvent(lane->stream, lane->fork, 0) != hipSuccess)
                return check_launch(name) != EASGD_OK ? EASGD_ELAUNCH : fail(EASGD_ELAUNCH, "%s: stream fork failed", name);
            rc = center_range(step->W, step->Wc, old_center, P, pl.N, ld, alpha, lane->stream, true);
            if (rc == EASGD_OK && hipEventRecord(lane->join, lane->stream) != hipSuccess)
                rc = fail(EASGD_ELAUNCH, "%s: stream join failed", name);
        } else if (!attach_center) {
            rc = center_range(step->W, step->Wc, old_center, P, pl.N, ld, alpha, s);
        } else {
            rc = EASGD_OK;
        }
        if (rc != EASGD_OK) return rc;
    }

    // ---- forward propagation ----
    CenterJob center_job = {};           // rides on the first launch of forward propagation when attach_center
    if (attach_center) {
        const size_t cblocks = pl.N / 4 / 256 + 1;
        if (cblocks > 0x3fffffffu) return fail(EASGD_ERANGE, "%s: N too large", name);
        center_job.W = step->W; center_job.Wc = step->Wc; center_job.old = old_center;
        center_job.N = pl.N; center_job.ld = ld; center_job.P = P;
        center_job.alpha = step->eta * step->rho; center_job.blocks = (unsigned)cblocks;
    }
    // The products of the hidden layers keep the fp32 instruction: a unit whose input is within rounding of zero is gated by
    // that rounding, so another sum, however much closer to the exact one, would change which of a round's few such
    // units pass their gradient on.  (The same product without the layers that follow, easgd_layer_product, takes
    // gemm_split.h: 3072->2048, 8 workers, 256 rows 210 us -> 142; the two of a 784-1024-1024-10 round, 16 workers, 128 rows, would gain 9 us of 213.)
    for (int l = 0; l < (head ? L - 1 : L); ++l) {
        GemmArgs a = forward_args(l);
        if (l == 0) a.ctr = center_job;
        if (l == L - 1) launch_gemm<K_CONTIG, MN_CONTIG, EPI_NONE>(a, forward_vec(l), s, forward_form(l));
        else launch_gemm<K_CONTIG, MN_CONTIG, EPI_RELU>(a, forward_vec(l), s, forward_form(l));
    }
    float *row_loss = reinterpret_cast<float *>(ws + pl.rowloss_off);
    const int rows = P * b;
    if (head) {
        HeadArgs h = {};
        h.A = act(L - 1); h.Wl = W + pl.off[L - 1]; h.w_ws = ld; h.y = y;
        h.dz = dz[(L - 1) % 3]; h.row_loss = row_loss; h.da = L >= 2 ? dz[(L - 2) % 3] : nullptr;
        h.d_in = dims[L - 1]; h.C = dims[L]; h.b = b; h.P = P;
        if (L == 1) h.ctr = center_job;
        launch_head(h, s);
    } else {
        EASGD_LAUNCH(softmax_xent_kernel, dim3((rows + 3) / 4), dim3(256), 0, s, logits, y, dz[(L - 1) % 3], row_loss,
                           rows, b, dims[L], pl.splits, (size_t)rows * dims[L]);
    }

    // ---- backward propagation ----
    // The weight-gradient product of a layer is held back until the next product is known, because two
    // independent products can share a launch (launch_pair_*): with the input-gradient product of the layer
    // below when the held one is narrow, or with the weight-gradient product of the layer below.
    const int epi = !step ? (G16 ? EPI_STORE_BF16 : EPI_NONE) : (step->V16 ? EPI_ELASTIC_MOM_BF16 : (step->V ? EPI_ELASTIC_MOM : EPI_ELASTIC));
    const bool pairing = options().gemm_pair != 0;
    const bool tile64 = options().gemm_tile == 0 || options().gemm_tile == 2;   // wide weight gradients use 64x64 or gemm_split.h
    struct Held { bool have = false; GemmArgs a; bool vec = false; Form form = FORM_BY_SIZE; } held;
    // calls f with the epilogue of the weight gradients as a constant
    auto by_rule = [&](auto f) {
        if (epi == EPI_NONE) f(std::integral_constant<int, EPI_NONE>{});
        else if (epi == EPI_STORE_BF16) f(std::integral_constant<int, EPI_STORE_BF16>{});
        else if (epi == EPI_ELASTIC) f(std::integral_constant<int, EPI_ELASTIC>{});
        else if (epi == EPI_ELASTIC_MOM) f(std::integral_constant<int, EPI_ELASTIC_MOM>{});
        else f(std::integral_constant<int, EPI_ELASTIC_MOM_BF16>{});
    };
    auto launch_dw = [&](const Held &h) {
        by_rule([&](auto e) { launch_gemm<MN_CONTIG, MN_CONTIG, decltype(e)::value>(h.a, h.vec, s, h.form); });
    };
    // the first kernel that changes W waits for the center rule, which reads W at time t
    bool joined = lane == nullptr;
    auto join = [&]() {
        if (!joined && hipStreamWaitEvent(s, lane->join, 0) != hipSuccess) return false;
        joined = true;
        return true;
    };
    auto flush = [&]() {
        if (held.have) {
            if (!join()) return false;
            launch_dw(held);
        }
        held.have = false;
        return true;
    };
    for (int l = L - 1; l >= 0; --l) {
        const int d_in = dims[l], d_out = dims[l + 1];
        const float *dz_l = dz[l % 3];
        if (l > 0 && !(head && l == L - 1)) {   // dZ_{l-1} = (dZ_l W_l^T) where A_l > 0
            GemmArgs a = {};
            a.A = dz_l; a.a_ws = (size_t)b * d_out; a.lda = d_out; a.a_lim = d_out; a.a_ones = -1;
            a.B = W + pl.off[l]; a.b_ws = ld; a.ldb = d_out;
            a.C = dz[(l - 1) % 3]; a.c_ws = (size_t)b * d_in; a.ldc = d_in;
            a.mask = act(l); a.mask_ws = (size_t)b * d_in; a.ldmask = d_in;
            a.M = b; a.N = d_in; a.K = d_out; a.P = P;
            a.splits = 1; a.k_per_split = (a.K + 63) / 64 * 64;
            const bool vec = mult4(d_out);
            // A held narrow product shares this launch where the tile leaves a block per compute unit free: not with 128x128
            // tiles, and with the fp32 instruction up to three of its four blocks per compute unit (gradient of 784-256-512-12,
            // 16 workers, 128 rows 73.2 us -> 70.6 with the aligned loader for the narrow product; 784-1024-1024-12, 32, 24
            // 194.6 -> 191.3; 3072-1024-2048-10, 16, 100, all on the fp32 instruction, 479 -> 471).  With the center rule on the
            // second stream it waits, so that the rule has this launch to finish behind as well (rounds of 784-512-2048-12,
            // 16, 128 201.0 us against 202.1, 784-1024-1024-12 206.7 against 207.3).
            bool shared = false;
            const bool narrow = held.have && held.a.N <= 32 && a.N > 32;
            // without 128-bit loads only the split form can share: it is taken whatever the length of the sum (round of
            // 784-254-57-10, 20, 19: 59.7 us against 66.6)
            const Form form = by_size == FORM_BY_SIZE && narrow && !vec ? FORM_SPLIT : by_size;
            if (narrow && pairing && !lane) {
                const SplitPick pick = form == FORM_FP32 ? SPLIT_NONE : split_pick(a, false, vec, form == FORM_SPLIT);
                const size_t blocks = (size_t)((a.M + 63) / 64) * ((a.N + 63) / 64) * P;
                const bool fp32_pair = pick == SPLIT_NONE && vec && tile64 && blocks <= (size_t)3 * num_cus();
                if (fp32_pair || (pick != SPLIT_NONE && pick != SPLIT_128x128)) {
                    by_rule([&](auto e) {
                        constexpr int E = decltype(e)::value;
                        auto launch = [&](auto dw) {
                            constexpr int DW = decltype(dw)::value;
                            if (fp32_pair) launch_pair_da_narrow_dw<E, DW>(a, held.a, s);
                            else launch_split_pair_da_narrow_dw<E, DW>(a, held.a, pick, s);
                        };
                        if (held.a.N <= 16 && narrow_dw_fits(held.a, held.vec)) launch(std::integral_constant<int, DW_NARROW16>{});
                        else if (held.vec) launch(std::integral_constant<int, DW_128x32_VEC>{});
                        else launch(std::integral_constant<int, DW_128x32>{});
                    });
                    shared = true;
                }
            }
            if (shared) held.have = false;
            else {
                launch_gemm<K_CONTIG, K_CONTIG, EPI_MASK>(a, vec, s, form);
                if (!flush()) return fail(EASGD_ELAUNCH, "%s: stream join failed", name);
            }
        }
        // [dW_l ; db_l] = [A_l 1]^T dZ_l, stored at the layer's place in the packed gradient
        GemmArgs d = {};
        d.A = act(l); d.a_ws = (size_t)b * d_in; d.lda = d_in; d.a_lim = d_in; d.a_ones = d_in;
        d.B = dz_l; d.b_ws = (size_t)b * d_out; d.ldb = d_out;
        d.C = G ? G + pl.off[l] : nullptr; d.c_ws = ld; d.ldc = d_out;
        d.C16 = G16 ? G16 + pl.off[l] : nullptr;
        d.M = d_in + 1; d.N = d_out; d.K = b; d.P = P;
        d.splits = 1; d.k_per_split = (d.K + 63) / 64 * 64;
        if (loss && l == L - 1) {            // the first weight-gradient launch also sums the losses up
            d.mean.row_loss = row_loss; d.mean.loss = loss; d.mean.b = b; d.mean.P = P; d.mean.blocks = (unsigned)((P + 3) / 4);
        }
        if (step) {
            d.Wt = step->W + pl.off[l];
            d.Vt = step->V ? step->V + pl.off[l] : nullptr;
            d.Vt16 = step->V16 ? step->V16 + pl.off[l] : nullptr;
            d.center = center_t + pl.off[l];
            d.eta = step->eta; d.rho = step->rho; d.alpha = step->eta * step->rho; d.delta = step->delta;
        }
        const bool vec = mult4(d_in) && mult4(d_out);
        if (held.have) {     // two weight-gradient products in a row (no input-gradient product for layer 0)
            const Form form = dw_pair_form(held.a, held.vec, d, vec, fp32);
            if (form != FORM_BY_SIZE && pairing) {
                if (!join()) return fail(EASGD_ELAUNCH, "%s: stream join failed", name);
                by_rule([&](auto e) {
                    if (form == FORM_FP32) launch_pair_dw_dw<decltype(e)::value>(held.a, d, s);
                    else launch_split_pair_dw_dw<decltype(e)::value>(held.a, d, s);
                });
                held.have = false;
                continue;
            }
            if (form != FORM_BY_SIZE) {
                held.form = form;
                if (!flush()) return fail(EASGD_ELAUNCH, "%s: stream join failed", name);
                held = {true, d, vec, form};
                if (!flush()) return fail(EASGD_ELAUNCH, "%s: stream join failed", name);
                continue;
            }
            if (!flush()) return fail(EASGD_ELAUNCH, "%s: stream join failed", name);
        }
        held = {true, d, vec, by_size};
    }
    if (!flush()) return fail(EASGD_ELAUNCH, "%s: stream join failed", name);
    return check_launch(name);
}

}  // namespace easgd

// One product of forward / backward propagation alone, through the same tile selection and kernels as the gradient.
extern "C" int easgd_layer_product(int kind, int d_in, int d_out, int P, int b, const float *A, const float *Wl, size_t ld,
                                   const float *dZ, float *out, size_t out_ws, int relu, void *stream)
{
    using namespace easgd;
    const char *name = "easgd_layer_product";
    if (kind < 0 || kind > 2 || d_in < 1 || d_out < 1 || P < 1 || b < 1) return fail(EASGD_EINVAL, "%s: bad kind or size", name);
    if (!A || !out || (kind != 1 && !Wl) || (kind != 0 && !dZ)) return fail(EASGD_EINVAL, "%s: NULL pointer", name);
    if (!aligned16(A) || !aligned16(out) || !aligned16(dZ) || !aligned_to(Wl, 4))
        return fail(EASGD_EINVAL, "%s: A, dZ, out must be 16-byte aligned, Wl 4-byte aligned", name);
    const size_t out_need = kind == 0 ? (size_t)b * d_out : kind == 1 ? (size_t)(d_in + 1) * d_out : (size_t)b * d_in;
    if (out_ws < out_need) return fail(EASGD_EINVAL, "%s: out_ws (%zu) below one worker's result (%zu)", name, out_ws, out_need);
    if (kind != 1 && ld < (size_t)(d_in + 1) * d_out) return fail(EASGD_EINVAL, "%s: ld below one layer block", name);
    if ((size_t)(d_in + 1) * d_out > 0x3fffffffull || (size_t)b * d_in > 0x3fffffffull || (size_t)b * d_out > 0x3fffffffull ||
        (size_t)P * b > 0x7fffffffull)
        return fail(EASGD_ERANGE, "%s: an operand exceeds 2^30-1 elements per worker", name);
    clear_error();
    hipStream_t s = static_cast<hipStream_t>(stream);
    GemmArgs a = {};
    a.P = P; a.splits = 1;
    if (kind == 0) {            // Z = [A 1] [W ; b]
        a.A = A; a.a_ws = (size_t)b * d_in; a.lda = d_in; a.a_lim = d_in; a.a_ones = d_in;
        a.B = Wl; a.b_ws = ld; a.ldb = d_out;
        a.C = out; a.c_ws = out_ws; a.ldc = d_out;
        a.M = b; a.N = d_out; a.K = d_in + 1;
        a.k_per_split = (a.K + 63) / 64 * 64;
        const bool vec = mult4(d_in) && mult4(d_out);
        if (relu) launch_gemm<K_CONTIG, MN_CONTIG, EPI_RELU>(a, vec, s);
        else launch_gemm<K_CONTIG, MN_CONTIG, EPI_NONE>(a, vec, s);
    } else if (kind == 1) {     // [dW ; db] = [A 1]^T dZ
        a.A = A; a.a_ws = (size_t)b * d_in; a.lda = d_in; a.a_lim = d_in; a.a_ones = d_in;
        a.B = dZ; a.b_ws = (size_t)b * d_out; a.ldb = d_out;
        a.C = out; a.c_ws = out_ws; a.ldc = d_out;
        a.M = d_in + 1; a.N = d_out; a.K = b;
        a.k_per_split = (a.K + 63) / 64 * 64;
        launch_gemm<MN_CONTIG, MN_CONTIG, EPI_NONE>(a, mult4(d_in) && mult4(d_out), s);
    } else {                    // dA = (dZ W^T) where A > 0
        a.A = dZ; a.a_ws = (size_t)b * d_out; a.lda = d_out; a.a_lim = d_out; a.a_ones = -1;
        a.B = Wl; a.b_ws = ld; a.ldb = d_out;
        a.C = out; a.c_ws = out_ws; a.ldc = d_in;
        a.mask = A; a.mask_ws = (size_t)b * d_in; a.ldmask = d_in;
        a.M = b; a.N = d_in; a.K = d_out;
        a.k_per_split = (a.K + 63) / 64 * 64;
        launch_gemm<K_CONTIG, K_CONTIG, EPI_MASK>(a, mult4(d_out), s);
    }
    return check_launch(name);
}
