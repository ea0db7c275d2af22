// Launches of an input-gradient product together with the weight-gradient product of a narrow layer (shared_launches.h).
#include "shared_launches.h"

namespace easgd {

template <int EPI, int DW>
bool launch_split_pair_da_narrow_dw(GemmArgs da, GemmArgs dw, SplitPick pick, hipStream_t s)
{
    auto launch = [&](auto tm, auto wn, auto wk) {
        constexpr int TM = decltype(tm)::value, WN = decltype(wn)::value, WK = decltype(wk)::value;
        const unsigned n_dw = place_narrow<DW>(dw), n = place_blocks<TM * 32, WN * 32>(da);
        dw.mean.first_block = n + n_dw;
        EASGD_LAUNCH((gemm_split_da_narrow_dw_kernel<TM, WN, WK, EPI, DW>), dim3(n + n_dw + dw.mean.blocks), dim3(256), 0, s, da, dw, n_dw);
        return true;
    };
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, 2> two{};
    constexpr std::integral_constant<int, 4> four{};
    if (pick == SPLIT_64x128) return launch(two, four, one);
    if (pick == SPLIT_64x64) return launch(two, two, two);
    if (pick == SPLIT_32x128) return launch(one, four, one);
    if (pick == SPLIT_32x32) return launch(one, one, four);
    return false;
}

template <int EPI, int DW>
void launch_pair_da_narrow_dw(GemmArgs da, GemmArgs dw, hipStream_t s)
{
    const unsigned n_dw = place_narrow<DW>(dw), n = place_blocks<64, 64>(da);
    dw.mean.first_block = n + n_dw;
    EASGD_LAUNCH((gemm_da_narrow_dw_kernel<EPI, DW>), dim3(n + n_dw + dw.mean.blocks), dim3(256), 0, s, da, dw, n_dw);
}

#define EASGD_FORMS(EPI)                                                                                                        \
    template bool launch_split_pair_da_narrow_dw<EPI, DW_128x32>(GemmArgs, GemmArgs, SplitPick, hipStream_t);                   \
    template bool launch_split_pair_da_narrow_dw<EPI, DW_128x32_VEC>(GemmArgs, GemmArgs, SplitPick, hipStream_t);               \
    template bool launch_split_pair_da_narrow_dw<EPI, DW_NARROW16>(GemmArgs, GemmArgs, SplitPick, hipStream_t);                 \
    template void launch_pair_da_narrow_dw<EPI, DW_128x32>(GemmArgs, GemmArgs, hipStream_t);                                    \
    template void launch_pair_da_narrow_dw<EPI, DW_128x32_VEC>(GemmArgs, GemmArgs, hipStream_t);                                \
    template void launch_pair_da_narrow_dw<EPI, DW_NARROW16>(GemmArgs, GemmArgs, hipStream_t);
EASGD_FORMS(EPI_NONE)
EASGD_FORMS(EPI_ELASTIC)
EASGD_FORMS(EPI_ELASTIC_MOM)
EASGD_FORMS(EPI_ELASTIC_MOM_BF16)
EASGD_FORMS(EPI_STORE_BF16)
#undef EASGD_FORMS

}  // namespace easgd
