// bf16-split kernel variants, part 0: 3x3 filters (the template is in
// conv_split.h; the parts compile in parallel).  The times are least-squares
// fits of igemm_plan_us's model to graph-replayed calls of 5,000 random layers
// (16-640 channels, 7^2 to 320^2 pixels) and sweeps of tile shapes on one
// MI355X; modelled over measured, 5th to 95th percentile: 0.87-1.09.
#include "conv_split.h"

namespace ilpm {
namespace ig {

int variants_split0(const Variant **table)
{
    //                     KS S  CC MA NB WC WP WK XPIX
    using P256 = SplitCfg<3, 1, 16, 1, 2, 2, 4, 1, 340>;
    using P128 = SplitCfg<3, 1, 16, 1, 2, 2, 2, 2, 192>;
    using P64 = SplitCfg<3, 1, 16, 1, 2, 1, 1, 4, 112>;
    // For maps too small for P128 to fill the chip unsplit: half its output
    // channels per workgroup, so twice the workgroups and no partial sums
    // (256->256 at 56^2: 29.1 us against P128's 30.9 on two splits and the fp32
    // kernels' 31.8).  Its wave runs all 128 pixels, so a weight is split once
    // per workgroup and not once per pixel half, and 32-channel stages halve
    // the barriers (16-channel stages, two waves over the pixels: 30.4 us).
    using P128L = SplitCfg<3, 1, 32, 1, 4, 1, 1, 8, 192>;
    //                       base  stage1 stage2 round out  part  split flow  piece out_piece
    constexpr Variant::Times tP256 = {1.56, 3.57, 0, 1.61, 0.19, 0.16, 2.04, 1.02, 0.00018, 0.00152};
    constexpr Variant::Times tP128 = {1.12, 2.01, 0, 3.05, 0.16, 0.19, 1.56, 0.40, 0.00062, 0.00107};
    constexpr Variant::Times tP64 = {2.38, 1.11, 1.58, 1.49, 0.20, 0.15, 1.78, 0.06, 0.00003, 0.00155};
    constexpr Variant::Times tP128L = {1.33, 2.00, 0, 4.19, 0.09, 0.10, 2.09, 0.46, 0.0007, 0.0013};
    static const Variant t[] = {
        make_split_variant<P256>("k3s1_b3_px256_co64", 16, 16, false, tP256),
        make_split_variant<P256>("k3s1_b3_px256_co64_even", 16, 16, true, tP256),
        make_split_variant<P128>("k3s1_b3_px128_co64", 8, 16, false, tP128),
        make_split_variant<P128>("k3s1_b3_px128_co64_even", 8, 16, true, tP128),
        make_split_variant<P64>("k3s1_b3_px64_co32", 8, 8, false, tP64),
        make_split_variant<P64>("k3s1_b3_px64_co32_even", 8, 8, true, tP64),
        make_split_variant<P128L>("k3s1_b3_px128_co32", 8, 16, false, tP128L),
        make_split_variant<P128L>("k3s1_b3_px128_co32_even", 8, 16, true, tP128L),
    };
    *table = t;
    return (int)(sizeof(t) / sizeof(t[0]));
}

}  // namespace ig
}  // namespace ilpm
