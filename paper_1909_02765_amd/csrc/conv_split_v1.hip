// bf16-split kernel variants, part 1: 1x1 filters (the template is in
// conv_split.h; the parts compile in parallel).  The times are least-squares
// fits of igemm_plan_us's model to graph-replayed calls of some 50 layers
// (16-1024 channels, 7^2-300x400 pixels) at 1-32 splits on one MI355X.
#include "conv_split.h"

namespace ilpm {
namespace ig {

int variants_split1(const Variant **table)
{
    //                     KS S  CC MA NB WC WP WK XPIX
    using P128 = SplitCfg<1, 1, 64, 1, 2, 2, 2, 2, 128>;
    using P64W = SplitCfg<1, 1, 64, 1, 1, 2, 2, 2, 64>;
    using P64 = SplitCfg<1, 1, 64, 1, 2, 1, 1, 4, 64>;
    //                       base  stage1 stage2 round  out    part   split
    constexpr Variant::Times tP128 = {6.20, 1.61, 0, 0, 0.34, 0.55, 0.1};
    constexpr Variant::Times tP64W = {1.75, 1.30, 0, 2.12, 0.20, 0.55, 0.7};
    constexpr Variant::Times tP64 = {3.15, 1.12, 3.44, 0.93, 0, 0.16, 1.4};
    static const Variant t[] = {
        make_split_variant<P128>("k1s1_b3_px128_co64", 8, 16, false, tP128),
        make_split_variant<P128>("k1s1_b3_px128_co64_even", 8, 16, true, tP128),
        make_split_variant<P64W>("k1s1_b3_px64_co64", 8, 8, false, tP64W),
        make_split_variant<P64W>("k1s1_b3_px64_co64_even", 8, 8, true, tP64W),
        make_split_variant<P64>("k1s1_b3_px64_co32", 8, 8, false, tP64),
        make_split_variant<P64>("k1s1_b3_px64_co32_even", 8, 8, true, tP64),
    };
    *table = t;
    return (int)(sizeof(t) / sizeof(t[0]));
}

}  // namespace ig
}  // namespace ilpm
