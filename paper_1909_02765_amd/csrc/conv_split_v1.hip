// bf16-split kernel variants, part 1: 1x1 filters (the template is in
// conv_split.h; the parts compile in parallel).  The times are least-squares
// fits of igemm_plan_us's model to graph-replayed calls of 5,000 random layers
// (16-640 channels, 7^2 to 320^2 pixels) and sweeps of tile shapes on one
// MI355X; modelled over measured, 5th to 95th percentile: 0.87-1.09.
#include "conv_split.h"

namespace ilpm {
namespace ig {

int variants_split1(const Variant **table)
{
    //                     KS S  CC MA NB WC WP WK XPIX
    using P128 = SplitCfg<1, 1, 64, 1, 2, 2, 2, 2, 128>;
    using P64W = SplitCfg<1, 1, 64, 1, 1, 2, 2, 2, 64>;
    using P64 = SplitCfg<1, 1, 64, 1, 2, 1, 1, 4, 64>;
    //                       base  stage1 stage2 round out  part  split flow  piece out_piece
    constexpr Variant::Times tP128 = {1.69, 1.03, 0, 2.48, 0.06, 0.09, 1.85, 0.47, 0.00037, 0.00182};
    constexpr Variant::Times tP64W = {1.51, 0.89, 0, 1.86, 0.15, 0.17, 1.79, 0.19, 0.00046, 0.00091};
    constexpr Variant::Times tP64 = {2.08, 0.67, 0.84, 1.73, 0.19, 0.15, 1.80, 0.10, 0.00044, 0.00107};
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
