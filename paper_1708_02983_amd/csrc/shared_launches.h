// Launches that an input-gradient product shares with the weight-gradient product of a narrow layer, and the numbering of a
// product's blocks.  Their kernels (four split tiles and one of the fp32 instruction, three forms of the narrow product, five
// epilogues) are a source of their own, which is compiled beside the others.
#pragma once
#include "gemm_split.h"

namespace easgd {

// Fills in the tile counts and the die-aware block numbering of a product; returns its number of blocks.
template <int BM, int BN>
inline unsigned place_blocks(GemmArgs &a)
{
    a.tiles_m = (a.M + BM - 1) / BM;
    a.tiles_n = (a.N + BN - 1) / BN;
    size_t total = (size_t)a.tiles_m * a.tiles_n * a.splits * a.P;
    a.xcd_chunk = 0;
    a.die_workers = 0;
    a.band_log2 = 0;
    a.band_tiles = 0;
    if (options().gemm_xcd && total >= 64) {
        total = (total + 7) / 8 * 8;
        a.xcd_chunk = (int)(total / 8);
        // a product with an elastic epilogue (it has a center): interleave the workers of a die
        const long order = options().gemm_xcd;
        if (a.center && a.splits == 1 && a.P % 8 == 0 && (order == 1 || order == 3)) {
            a.die_workers = a.P / 8;
            // bands of 8 (4, 2) tile columns when the tile columns divide into them
            if (order == 1 && a.tiles_m > 1)
                a.band_log2 = a.tiles_n % 8 == 0 ? 3 : a.tiles_n % 4 == 0 ? 2 : a.tiles_n % 2 == 0 ? 1 : 0;
            a.band_tiles = a.tiles_m << a.band_log2;
        }
    }
    // the kernel's divisions by multiplication: exact while dividend * divisor < 2^32
    auto magic = [&](size_t dividend_max, int d) -> unsigned {
        if (d <= 1 || dividend_max * (size_t)d >= ((size_t)1 << 32)) return 0u;
        return (unsigned)((((size_t)1 << 32) + (size_t)d - 1) / (size_t)d);
    };
    const size_t tiles = (size_t)a.tiles_m * a.tiles_n;
    a.magic_tiles = magic(total, (int)tiles);
    a.magic_tiles_n = magic(tiles, a.tiles_n);
    a.magic_die = magic(total / 8 + 1, a.die_workers);
    a.magic_band = magic(tiles, a.band_tiles);
    return (unsigned)total;
}

// Which tile of gemm_split.h a product takes: rows x columns, or none.
enum SplitPick { SPLIT_NONE, SPLIT_128x128, SPLIT_64x128, SPLIT_64x64, SPLIT_32x128, SPLIT_32x32 };

// Blocks of a narrow weight gradient that shares a launch, by its form.
template <int DW>
inline unsigned place_narrow(GemmArgs &dw)
{
    if constexpr (DW == DW_NARROW16) return place_blocks<64, 16>(dw);
    else return place_blocks<128, 32>(dw);
}

// An input-gradient product and the weight-gradient product of a narrow layer in one launch, the first as split tiles of
// `pick`'s shape; false: this tile has none.  DW: the form of the second.
template <int EPI, int DW>
bool launch_split_pair_da_narrow_dw(GemmArgs da, GemmArgs dw, SplitPick pick, hipStream_t s);

// The same with 64x64 tiles of the fp32 instruction.
template <int EPI, int DW>
void launch_pair_da_narrow_dw(GemmArgs da, GemmArgs dw, hipStream_t s);

}  // namespace easgd
