// bf16-split kernel variants, part 2: 5x5 filters and stride 2 (the template is in
// conv_split.h; the parts compile in parallel).  The times are least-squares
// fits of igemm_plan_us's model to graph-replayed calls of 5,000 random layers
// (16-640 channels, 7^2 to 320^2 pixels) and sweeps of tile shapes on one
// MI355X; modelled over measured, 5th to 95th percentile: 0.87-1.09.
#include "conv_split.h"

namespace ilpm {
namespace ig {

int variants_split2(const Variant **table)
{
    //                     KS S  CC MA NB WC WP WK XPIX
    using P128K5 = SplitCfg<5, 1, 8, 1, 2, 1, 2, 2, 240>;
    using P64K5 = SplitCfg<5, 1, 8, 1, 2, 1, 1, 4, 160>;
    using P128S2 = SplitCfg<3, 2, 16, 1, 2, 1, 2, 2, 568>;
    using P64S2 = SplitCfg<3, 2, 16, 1, 2, 1, 1, 8, 304>;
    using P64K5S2 = SplitCfg<5, 2, 8, 1, 2, 1, 1, 4, 368>;
    //                       base  stage1 stage2 round out  part  split flow  piece out_piece
    constexpr Variant::Times tP128K5 = {2.68, 2.04, 3.37, 1.78, 0.25, 0.17, 1.74, 0.15, 0.00051, 0};
    constexpr Variant::Times tP64K5 = {3.13, 1.39, 2.08, 1.20, 0.42, 0.13, 1.68, 0.07, 0.0002, 0.00051};
    constexpr Variant::Times tP128S2 = {1.52, 2.07, 0, 3.43, 0.03, 0.11, 1.91, 0.10, 0.00022, 0.00259};
    constexpr Variant::Times tP64S2 = {1.53, 1.22, 0, 2.51, 0.02, 0.11, 1.88, 0.18, 0.0006, 0.0015};
    constexpr Variant::Times tP64K5S2 = {0, 1.48, 0, 4.67, 0, 0.22, 1.09, 0.07, 0.00028, 0.00043};
    static const Variant t[] = {
        make_split_variant<P128K5>("k5s1_b3_px128_co32", 8, 16, false, tP128K5),
        make_split_variant<P128K5>("k5s1_b3_px128_co32_even", 8, 16, true, tP128K5),
        make_split_variant<P64K5>("k5s1_b3_px64_co32", 8, 8, false, tP64K5),
        make_split_variant<P64K5>("k5s1_b3_px64_co32_even", 8, 8, true, tP64K5),
        make_split_variant<P128S2>("k3s2_b3_px128_co32", 8, 16, false, tP128S2),
        make_split_variant<P128S2>("k3s2_b3_px128_co32_even", 8, 16, true, tP128S2),
        make_split_variant<P64S2>("k3s2_b3_px64_co32", 8, 8, false, tP64S2),
        make_split_variant<P64S2>("k3s2_b3_px64_co32_even", 8, 8, true, tP64S2),
        make_split_variant<P64K5S2>("k5s2_b3_px64_co32", 8, 8, false, tP64K5S2),
        make_split_variant<P64K5S2>("k5s2_b3_px64_co32_even", 8, 8, true, tP64K5S2),
    };
    *table = t;
    return (int)(sizeof(t) / sizeof(t[0]));
}

}  // namespace ig
}  // namespace ilpm
