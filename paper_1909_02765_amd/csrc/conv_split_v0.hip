// bf16-split kernel variants, part 0: 3x3 filters (the template is in
// conv_split.h; the parts compile in parallel).  The times are least-squares
// fits of igemm_plan_us's model to graph-replayed calls of some 50 layers
// (16-1024 channels, 7^2-300x400 pixels) at 1-32 splits on one MI355X.
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
    //                       base  stage1 stage2 round  out    part   split
    constexpr Variant::Times tP256 = {2.43, 3.87, 0, 3.36, 0.33, 0.25, 1.6};
    constexpr Variant::Times tP128 = {0.76, 2.31, 0, 4.59, 0.15, 0.20, 1.7};
    constexpr Variant::Times tP64 = {2.65, 1.12, 1.69, 1.71, 0.26, 0.22, 1.7};
    constexpr Variant::Times tP128L = {2.21, 2.42, 0, 4.90, 0.36, 0.30, 0.9};
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
