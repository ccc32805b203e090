// bf16-split kernel variants, part 2: 5x5 filters and stride 2 (the template is in
// conv_split.h; the parts compile in parallel).  The times are least-squares
// fits of igemm_plan_us's model to graph-replayed calls of some 50 layers
// (16-1024 channels, 7^2-300x400 pixels) at 1-32 splits on one MI355X.
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
    //                       base  stage1 stage2 round  out    part   split
    constexpr Variant::Times tP128K5 = {0.91, 2.22, 3.75, 2.74, 0.36, 0.17, 2.4};
    constexpr Variant::Times tP64K5 = {1.66, 1.46, 2.15, 1.92, 0.49, 0.24, 2.3};
    constexpr Variant::Times tP128S2 = {0, 2.50, 0, 5.74, 0, 0.09, 2.1};
    constexpr Variant::Times tP64S2 = {1.65, 1.64, 0, 3.20, 0, 0.15, 1.7};
    constexpr Variant::Times tP64K5S2 = {2.24, 1.49, 0, 2.85, 0.26, 0.21, 1.6};
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
