// Single-pass shapes for N = 8192 and 16384.  gfx950's 160 KiB LDS holds a
// whole 16384-point complex64 transform (128 KiB + pad), so these sizes need
// no device-memory exchange at all; the four-step path is kept beside them.
#include "variant_maker.hpp"

using stockfft::OrdinaryLoads;
using stockfft::PairedTwiddles;
using stockfft::Shape;
using stockfft::ShapeX;
using stockfft::make_variant;

STOCKFFT_VARIANT_GROUP(variants_large,
  make_variant<Shape<8192, 8, 1, 4, 8, 8, 8, 8, 2>>("n8192_e8_b1_p4_r8.8.8.8.2"),
  make_variant<PairedTwiddles<Shape<8192, 8, 1, 4, 8, 8, 8, 8, 2>>>("n8192_e8_b1_p4_r8.8.8.8.2_pt"),
  make_variant<Shape<8192, 16, 1, 4, 16, 16, 16, 2>>("n8192_e16_b1_p4_r16.16.16.2"),
  make_variant<PairedTwiddles<Shape<8192, 16, 1, 4, 16, 16, 16, 2>>>("n8192_e16_b1_p4_r16.16.16.2_pt"),
  make_variant<Shape<8192, 32, 1, 4, 16, 16, 16, 2>>("n8192_e32_b1_p4_r16.16.16.2"),
  make_variant<PairedTwiddles<Shape<8192, 32, 1, 4, 16, 16, 16, 2>>>("n8192_e32_b1_p4_r16.16.16.2_pt"),
  make_variant<Shape<16384, 16, 1, 4, 16, 16, 16, 4>>("n16384_e16_b1_p4_r16.16.16.4"),
  make_variant<PairedTwiddles<Shape<16384, 16, 1, 4, 16, 16, 16, 4>>>("n16384_e16_b1_p4_r16.16.16.4_pt"),
  make_variant<Shape<16384, 32, 1, 4, 16, 16, 16, 4>>("n16384_e32_b1_p4_r16.16.16.4"),
  make_variant<PairedTwiddles<Shape<16384, 32, 1, 4, 16, 16, 16, 4>>>("n16384_e32_b1_p4_r16.16.16.4_pt"),
  // Two-round exchanges: half the LDS, two (16384) or four (8192) workgroups per CU.
  make_variant<ShapeX<2, false, 4, 16384, 32, 1, 4, 16, 16, 16, 4>>("n16384_e32_c2_b1_p4_r16.16.16.4"),
  make_variant<PairedTwiddles<ShapeX<2, false, 4, 16384, 32, 1, 4, 16, 16, 16, 4>>>("n16384_e32_c2_b1_p4_r16.16.16.4_pt"),
  make_variant<ShapeX<2, false, 4, 8192, 32, 1, 4, 16, 16, 16, 2>>("n8192_e32_c2_b1_p4_r16.16.16.2"),
  make_variant<PairedTwiddles<ShapeX<2, false, 4, 8192, 32, 1, 4, 16, 16, 16, 2>>>("n8192_e32_c2_b1_p4_r16.16.16.2_pt"),
  // Four-round exchanges (a quarter of the LDS): radix 8 before the last
  // pass, so that every exchange splits into four rounds.
  make_variant<ShapeX<4, false, 4, 16384, 32, 1, 4, 8, 8, 8, 8, 4>>("n16384_e32_c4_b1_p4_r8.8.8.8.4"),
  make_variant<ShapeX<4, false, 4, 8192, 32, 1, 4, 8, 8, 8, 16>>("n8192_e32_c4_b1_p4_r8.8.8.16"),
  // Sixteen values per lane with two-round exchanges: radix 8 leaves two
  // butterflies per lane per pass, so each round takes one, and the body fits
  // 64 VGPRs; two 1024-lane workgroups (32 waves) then share a CU.
  make_variant<ShapeX<2, false, 8, 16384, 16, 1, 4, 8, 8, 8, 8, 4>>("n16384_e16_c2_b1_p4_r8.8.8.8.4"),
  make_variant<PairedTwiddles<ShapeX<2, false, 8, 16384, 16, 1, 4, 8, 8, 8, 8, 4>>>("n16384_e16_c2_b1_p4_r8.8.8.8.4_pt"),
  // Radix-32 passes: three passes and two exchanges where the radix-16 and
  // radix-8 plans take four or five and three or four.  us on an MI355X, best
  // shape without / with a radix-32 pass: 8192 x 300 plain 13.4 / 12.1, matched
  // filter 19.6 / 17.0, forward -> adjoint 21.0 / 18.8; 16384 x 300 24.3 / 23.0,
  // 35.4 / 33.3, 38.2 / 35.2.  At 16384 a lane holds 64 values (256 lanes, two
  // workgroups per CU, 210 VGPRs) so that every exchange splits into two rounds.
  make_variant<PairedTwiddles<ShapeX<2, false, 4, 8192, 32, 1, 4, 16, 16, 32>>>("n8192_e32_c2_b1_p4_r16.16.32_pt"),
  make_variant<PairedTwiddles<ShapeX<1, false, 2, 8192, 32, 1, 4, 32, 16, 16>>>("n8192_e32_b1_p4_r32.16.16_pt"),
  make_variant<PairedTwiddles<ShapeX<2, false, 2, 16384, 64, 1, 4, 32, 32, 16>>>("n16384_e64_c2_b1_p4_r32.32.16_pt"),
  make_variant<PairedTwiddles<ShapeX<2, false, 2, 16384, 64, 1, 4, 16, 32, 32>>>("n16384_e64_c2_b1_p4_r16.32.32_pt"),
  make_variant<PairedTwiddles<ShapeX<1, false, 2, 16384, 32, 1, 4, 32, 32, 16>>>("n16384_e32_b1_p4_r32.32.16_pt"),
  // Ordinary row loads.
  make_variant<OrdinaryLoads<PairedTwiddles<ShapeX<2, false, 4, 8192, 32, 1, 4, 16, 16, 32>>>>("n8192_e32_c2_b1_p4_r16.16.32_pt_ol"),
  make_variant<OrdinaryLoads<ShapeX<4, false, 4, 8192, 32, 1, 4, 8, 8, 8, 16>>>("n8192_e32_c4_b1_p4_r8.8.8.16_ol"),
  make_variant<OrdinaryLoads<PairedTwiddles<ShapeX<2, false, 2, 16384, 64, 1, 4, 32, 32, 16>>>>("n16384_e64_c2_b1_p4_r32.32.16_pt_ol"),
  make_variant<OrdinaryLoads<PairedTwiddles<ShapeX<2, false, 8, 16384, 16, 1, 4, 8, 8, 8, 8, 4>>>>("n16384_e16_c2_b1_p4_r8.8.8.8.4_pt_ol"))
