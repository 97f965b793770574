// Four-step variants: the paper's synthesis rule 2 (Section IV-D) with the
// splits of Section V-D eq. (7)-(8) plus N2 = 2048 alternatives, and the same
// decomposition for lengths beyond one LDS-resident transform (rule 3's
// multi-level case): the column splits N1 x N2 of columns.hpp from 2^15 to
// 2^20, and N = N1 x 16384, the second stage's N1-point DFTs (N1 <= 64) done
// in registers with two-level twiddles.  Without a tuning entry a length
// takes its first split listed here.
#include "columns.hpp"
#include "kernels.hpp"

namespace stockfft {

namespace {
using Sub4096 = Shape<4096, 16, 1, 4, 16, 16, 16>;
using Sub2048 = Shape<2048, 16, 1, 4, 16, 16, 8>;
using Sub16384 = ShapeX<2, false, 4, 16384, 32, 1, 4, 16, 16, 16, 4>;
constexpr const char* kSub16384 = "n16384_e32_c2_b1_p4_r16.16.16.4";
// Column shapes: R0 values per lane, R1 lanes per column.  The 32-value shapes
// exchange real and imaginary parts in turn, which keeps two (1024 points) or
// four (512) workgroups on a CU.
using C128 = Col<16, 8, 32, false, 4>;
using C256 = Col<16, 16, 16, false, 4>;
using C512 = Col<32, 16, 16, true, 4>;
using C1024 = Col<32, 32, 16, true, 4>;

template <class First, class Second>
FourStepVariant column_variant(const char* name, const char* sub_name, int tw_sub_elems, const char* sub2_name) {
  using S = Split<First, Second>;
  return {name, (int)S::N, S::N1, S::N2, sub_name, tw_sub_elems, &launch_columns_first<S>,
          &launch_columns_second<S>, true, sub2_name, S::shape,
          reinterpret_cast<const void*>(&k_columns_first<S, false, 0>),
          reinterpret_cast<const void*>(&k_columns_second<S, false, 0>)};
}
constexpr const char* kSub256 = "n256_e4_b4_p4_r4.4.4.4";
constexpr const char* kSub512 = "n512_e8_b4_p4_r8.8.8";
constexpr const char* kSub1024 = "n1024_e16_b1_p4_r16.16.4";
using Sub256 = Shape<256, 4, 4, 4, 4, 4, 4, 4>;
using Sub512 = Shape<512, 8, 4, 4, 8, 8, 8>;
using Sub1024 = Shape<1024, 16, 1, 4, 16, 16, 4>;
}  // namespace

const FourStepVariant* four_step_variants(int* count) {
  static const FourStepVariant table[] = {
    {"fs8192_2x4096", 8192, 2, 4096, "n4096_e16_b1_p4_r16.16.16", Sub4096::TW_ELEMS,
     &launch_four_step_columns<Sub4096, 2>, &launch_four_step_combine<2, 4096, false>, false},
    {"fs8192_4x2048", 8192, 4, 2048, "n2048_e16_b1_p4_r16.16.8", Sub2048::TW_ELEMS,
     &launch_four_step_columns<Sub2048, 4>, &launch_four_step_combine<4, 2048, false>, false},
    {"fs16384_4x4096", 16384, 4, 4096, "n4096_e16_b1_p4_r16.16.16", Sub4096::TW_ELEMS,
     &launch_four_step_columns<Sub4096, 4>, &launch_four_step_combine<4, 4096, false>, false},
    {"fs16384_8x2048", 16384, 8, 2048, "n2048_e16_b1_p4_r16.16.8", Sub2048::TW_ELEMS,
     &launch_four_step_columns<Sub2048, 8>, &launch_four_step_combine<8, 2048, false>, false},
    column_variant<C256, C128>("fs32768_tile128x256", kSub256, Sub256::TW_ELEMS, nullptr),
    {"fs32768_2x16384", 32768, 2, 16384, kSub16384, Sub16384::TW_ELEMS,
     &launch_four_step_columns<Sub16384, 2>, &launch_four_step_combine<2, 16384, true>, true},
    column_variant<C256, C256>("fs65536_tile256x256", kSub256, Sub256::TW_ELEMS, nullptr),
    {"fs65536_4x16384", 65536, 4, 16384, kSub16384, Sub16384::TW_ELEMS,
     &launch_four_step_columns<Sub16384, 4>, &launch_four_step_combine<4, 16384, true>, true},
    column_variant<C512, C256>("fs131072_tile256x512", kSub512, Sub512::TW_ELEMS, kSub256),
    {"fs131072_8x16384", 131072, 8, 16384, kSub16384, Sub16384::TW_ELEMS,
     &launch_four_step_columns<Sub16384, 8>, &launch_four_step_combine<8, 16384, true>, true},
    column_variant<C512, C512>("fs262144_tile512x512", kSub512, Sub512::TW_ELEMS, nullptr),
    {"fs262144_16x16384", 262144, 16, 16384, kSub16384, Sub16384::TW_ELEMS,
     &launch_four_step_columns<Sub16384, 16>, &launch_four_step_combine<16, 16384, true>, true},
    column_variant<C512, C1024>("fs524288_tile1024x512", kSub512, Sub512::TW_ELEMS, kSub1024),
    {"fs524288_32x16384", 524288, 32, 16384, kSub16384, Sub16384::TW_ELEMS,
     &launch_four_step_columns<Sub16384, 32>, &launch_four_step_combine<32, 16384, true>, true},
    column_variant<C1024, C1024>("fs1048576_tile1024x1024", kSub1024, Sub1024::TW_ELEMS, nullptr),
    {"fs1048576_64x16384", 1048576, 64, 16384, kSub16384, Sub16384::TW_ELEMS,
     &launch_four_step_columns<Sub16384, 64>, &launch_four_step_combine<64, 16384, true>, true},
  };
  *count = (int)(sizeof(table) / sizeof(table[0]));
  return table;
}

}  // namespace stockfft
