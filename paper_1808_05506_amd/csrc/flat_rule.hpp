// Which calls the flat kernels take from the direct one (their launchers look at
// shapes and alignment besides).
#pragma once

#include "launch.hpp"

namespace dsl {

// Small lattices: several columns a lane and chunks of up to 256 lanes leave the chip idle
// that the direct kernel fills, and a site's links are staged for few columns.  So each
// kind of call has a fewest number of lanes, in units of 1024 (kNever: none); DSLASH_FLAT_LANES
// replaces it.  The lines are where the time on inputs that change from launch to launch
// and on inputs that stay in the caches, averaged, is that of the direct kernel on cubes
// and odd lattices from 4^4 to 32^4; the direct kernel also depends on N_x.  Below: us on
// changing inputs, here and by the direct kernel.
constexpr uint32_t kNever = 0xffffffffu;

inline bool flat_lanes_pay(const Geom& g, int vw, uint32_t fewest) {
  const uint64_t lanes = uint64_t(g.vol) * uint64_t(g.nv / vw);
  if (knobs().flat_lanes.set)
    return knobs().flat_lanes.value >= 0 && lanes >= uint64_t(knobs().flat_lanes.value);
  return fewest != kNever && lanes >= uint64_t(fewest) * 1024;
}

// D_S, vw columns a lane.
inline bool staggered_flat_pays(int dtype, const Geom& g, int vw, bool compressed) {
  const int nv = g.nv;
  const bool bf16 = dtype == DT_BF16;
  uint32_t f;
  if (dtype == DT_C128) {
    f = nv < 4 ? 256 : 0;  // 8^4, N_v = 4 5.8 and 6.2; 16^3 x 16, N_v = 1 26.3 and 18.9
  } else if (dtype == DT_C64) {
    // 12^3 x 24, N_v = 4 11.4 and 14.1, 12^3 x 16 9.9 and 10.1.  Two columns are one piece a colour:
    // 20^3 x 40 91.8 and 74.8, 24^4 71.9 and 79.9; compressed 43.3 and 41.2, 24^3 x 48 74.5 and 83.7.
    // Compressed, N_v = 1 16^3 x 32 18.1 and 15.1, N_v = 4 12^3 x 24 10.3 and 10.1, 16^4 11.1 and 12.8
    f = nv == 2 ? (compressed ? 640 : 320) : compressed && nv == 4 ? 128 : compressed && nv < 4 ? 144 : 80;
  } else if (vw == 1) {
    // N_v = 1 20^4 17.7 and 16.4, 32^4 82.0 and 94.5; N_v = 3 18x14x20x26 18.0 and 17.3, 24^4 36.4 and
    // 40.0; compressed, N_v = 3 24^3 x 48 62.4 and 60.6, N_v = 7 16^4 15.8 and 14.8, 20^3 x 40 60.0 and 65.5
    f = nv < 5 ? (compressed ? kNever : bf16 ? 400 : 256) : (compressed ? 1024 : 80);
  } else if (vw == 2) {
    // N_v = 2 20^4 19.8 and 16.8, 32^4 91.6 and 104; F16 24^3 x 48 64.6 and 70.2
    f = nv == 2 ? (bf16 || compressed ? 768 : 320) : compressed ? 96 : 80;
  } else {
    // N_v = 4 20^4 28.3 and 18.9, 32^4 125 and 121; F16, N_v = 16 12^3 x 24 16.4 and 14.3, 16^4 19.4 and
    // 20.1 (BF16 15.8 and 16.3)
    f = nv == 4 ? kNever : !bf16 && nv < 24 ? 192 : 128;
  }
  return flat_lanes_pay(g, vw, f);
}

// D_W, vw columns a lane.  Left to the direct kernel altogether: N_v = 1 (16^3 x 32 C64 26.6
// against 66.4 us, its site is one contiguous run), and lanes of one 8- or 4-byte word
// where the links are short or few lanes share them (C64 compressed, N_v = 5, 22x20x13x21:
// 93 and 71.5; BF16, N_v = 5, 20x18x14x22: 68 and 59.9).
inline bool wilson_flat_pays(int dtype, const Geom& g, int vw, bool clover, bool compressed) {
  const int nv = g.nv;
  const bool one_word = dtype != DT_C128 && vw == 1, bf16 = dtype == DT_BF16;
  if (nv == 1 || (!clover && one_word && (compressed || nv < 6))) return false;
  uint32_t f;
  // Few columns with the clover term or compressed links (21x16x17x33): C64 clover N_v = 2 171
  // and 128, compressed N_v = 4 106 and 85; BF16 clover N_v = 2 102 and 63, N_v = 8 138 and 102,
  // compressed N_v = 8 103 and 90
  if ((clover && nv <= 2) || ((clover || compressed) && vw == 4 && nv < 16) || (compressed && dtype == DT_C64 && nv < 8)) {
    f = kNever;
  } else if (dtype == DT_C128) {
    // N_v = 4, 110k 27.8 and 20.9; N_v = 12, 172k 30.0 and 30.3; with the clover term, N_v = 4,
    // 17x13x11x19 58.9 and 54.2, 18x14x20x26 165 and 148, 20^4 167 and 182
    f = clover && nv <= 4 ? 640 : 144;
  } else if (one_word) {
    // C64 any (N_v = 5 with the clover term, 8^4 8.5 and 9.9); BF16, N_v = 7 8^4 9.1 and 8.4 (F16 9.0
    // and 10.7), N_v = 9 16 x 8 x 8 x 16 18.1 and 17.1, N_v = 7 17x13x11x19 35.7 and 39.5; with the clover
    // term, N_v = 3 12^4 21.7 and 16.2, 16^3 x 32 63.5 and 60.8, N_v = 5 10^4 14.1 and 11.1, 21x15x13x27
    // 69.2 and 69.7
    f = dtype == DT_C64 ? 0 : nv < 5 ? (bf16 ? 400 : 144) : !bf16 ? 0 : clover ? 232 : 160;
  } else if (vw == 4) {
    // BF16, N_v = 32 16^3 x 32 187 and 180, 12^3 x 24 66.5 and 69.1; with the clover term, N_v = 24
    // 17x13x11x19 76.9 and 65.1, 16^4 104 and 87; compressed, N_v = 24 16^4 81.4 and 77.5, F16 N_v = 28
    // 17x13x11x19 73.1 and 66.9; N_v = 20 20^4 173 and 199
    f = clover && bf16 && nv >= 24 ? 1024 : compressed ? 400 : bf16 && !clover ? 640 : 256;
  } else if (compressed) {
    f = 256;  // C64 N_v = 8 27k sites 1.04 times
  } else if (clover) {
    f = 128;  // C64 N_v = 4, 55k 22.8 and 18.1, 131k 42.4 and 45.3
  } else {
    // BF16, N_v = 2 16^4 21.4 and 21.6, 21x15x13x27 29.7 and 39.1; N_v = 18 8^3 x 16 14.4 and 13.1; N_v = 6
    // 12^3 x 16 18.2 and 22.1
    f = dtype == DT_C64 ? 64 : bf16 && nv == 2 ? 104 : 80;
  }
  return flat_lanes_pay(g, vw, f);
}

}  // namespace dsl
