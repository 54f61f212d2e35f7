// Row-staged D_W kernels (see rows.hpp): a workgroup owns an x-row chunk of
// R sites and all N_v right-hand sides; its inputs are copied into LDS with
// coalesced 16-byte loads, the hops are evaluated from LDS, and the outputs
// leave through LDS with coalesced 16-byte stores.  wilson_rows_kernel
// computes one output row per workgroup; wilson_march_kernel (the default)
// steps one workgroup through several consecutive t of the same (y, z).
#pragma once

#include <stdlib.h>

#include <type_traits>

#include "chunks.hpp"
#include "launch.hpp"
#include "rows.hpp"

namespace dsl {

// LDS layout, in storage words (one complex number each):
//   buf  [(R + HN) * 12 NV] one staged row in slots i + 1: a neighbour row fills
//                           1 .. n, the chunk's own row also the halo slots;
//                           reused for the output
//   lown [(R + HN) * 36]    links in the same slots (of the halo sites V_x of 0 and R + 3)
//   lnb  [R * 9]            V_mu of the backward neighbour row (current mu)
template <int NV, class S, int LW, int HN>
size_t rows_lds_words(int R);

template <class S, class T, int NV>
DSL_HD void lds_spinor(const typename S::word* __restrict__ site, int v, cpx<T> (&p)[4][3]) {
#pragma unroll
  for (int sp = 0; sp < 4; ++sp)
#pragma unroll
    for (int c = 0; c < 3; ++c) p[sp][c] = S::template load<T>(site + (sp * 3 + c) * NV + v);
}

// acc += (1 + C gamma_MU) U' psi with psi and U' read from LDS
template <int MU, int C, bool DAG, int NV, class S, class T, int LW = 9>
__device__ __forceinline__ void lds_hop(const typename S::word* __restrict__ site,
                                       const typename S::word* __restrict__ link, int v, cpx<T> (&acc)[4][3]) {
  cpx<T> p[4][3];
  lds_spinor<S, T, NV>(site, v, p);
  cpx<T> h[2][3];
  project<MU, C, T>(p, h);
  cpx<T> u[3][3];
  if constexpr (LW == 9) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) u[a][b] = S::template load<T>(link + a * 3 + b);
  } else {
    load_link_lw<LW, S, T>(link, u);
  }
  cpx<T> t[2][3];
  su3_mul2<DAG, T>(u, h, t);
  reconstruct_add<MU, C, T>(acc, t);
}

// A storage word (4, 8 or 16 bytes) in the low bytes of a 16-byte register
// group and back, by value (a memcpy through a local can leave the group in
// scratch memory).
template <class W>
__device__ __forceinline__ u32x4 word_to_piece(W w) {
  if constexpr (sizeof(W) == 16) {
    return __builtin_bit_cast(u32x4, w);
  } else if constexpr (sizeof(W) == 8) {
    const u32x2 t = __builtin_bit_cast(u32x2, w);
    return u32x4{t.x, t.y, 0u, 0u};
  } else {
    return u32x4{__builtin_bit_cast(unsigned, w), 0u, 0u, 0u};
  }
}

template <class W>
__device__ __forceinline__ W piece_to_word(u32x4 z) {
  if constexpr (sizeof(W) == 16) {
    return __builtin_bit_cast(W, z);
  } else if constexpr (sizeof(W) == 8) {
    return __builtin_bit_cast(W, u32x2{z.x, z.y});
  } else {
    // 4-byte words are uint32_t pairs of 16-bit halves: a plain conversion
    // (a bit cast of a vector element is miscompiled by this compiler)
    static_assert(__is_same(W, uint32_t), "4-byte storage words are uint32_t");
    return z.x;
  }
}

// One thread's share of a neighbour row in flight: CH 16-byte pieces of the
// spinor run (pieces tid, tid + nth, ...) plus E more 16-byte register groups
// (so that the whole row is one array) for, on a backward hop, the thread's
// ceil(9 / N_v) words of the row's V_mu links, packed, or, on the own row, its
// pieces of the two halo sites.  The piece count per thread does not depend on
// R: a row chunk is R * 12 NV words and the workgroup has R * NV threads.
template <class S>
struct RowPieces {
  static constexpr int CH = 12 * int(sizeof(typename S::word)) / 16;
};

// E for N_v right-hand sides and wb-byte storage words.  The halo needs
// HN * 12 N_v words in R N_v threads, 12 HN wb / (16 R) groups a thread: the
// launcher (halo_fits) takes R >= 16, or 8 above N_v = 16, at HN = 2, and at
// HN = 4 R >= 24 up to N_v = 8, 12 up to N_v = 16 and 8 above.
DSL_HD constexpr int row_extra_groups(int nv, int wb, int hn) {
  const int links = (((9 + nv - 1) / nv) * wb + 15) / 16;
  const int rmin = nv <= 8 ? 24 : (nv <= 16 ? 12 : 8);
  const int halo = hn == 2 ? (nv > 16 ? (24 * wb / 16 + 7) / 8 : 1) : (3 * wb + rmin - 1) / rmin;
  return links > halo ? links : halo;
}
inline bool halo_fits(int R, int nv, int wb, int hn) { return R * 16 * row_extra_groups(nv, wb, hn) >= 12 * hn * wb; }

// Register groups of a row in flight; the functions below take the number RN
// of groups from their argument.
template <int NV, class S, int HN>
struct RowRegs {
  static constexpr int CH = RowPieces<S>::CH;
  static constexpr int E = row_extra_groups(NV, int(sizeof(typename S::word)), HN);
  static constexpr int N = CH + E;
};

// Word i of the thread's link words (i = 0 .. KW - 1) in group i / PER of the
// extra groups, PER = 16 / word bytes words to a group, and back.
template <class W, int KW>
__device__ __forceinline__ u32x4 pack_words(const W (&w)[KW], int i0) {
  constexpr int WB = int(sizeof(W));
  if constexpr (WB == 16) {
    return i0 < KW ? __builtin_bit_cast(u32x4, w[i0]) : u32x4{0u, 0u, 0u, 0u};
  } else if constexpr (WB == 8) {
    const u32x2 a = i0 < KW ? __builtin_bit_cast(u32x2, w[i0]) : u32x2{0u, 0u};
    const u32x2 b = i0 + 1 < KW ? __builtin_bit_cast(u32x2, w[i0 + 1]) : u32x2{0u, 0u};
    return u32x4{a.x, a.y, b.x, b.y};
  } else {
    static_assert(__is_same(W, uint32_t), "4-byte storage words are uint32_t");
    return u32x4{i0 < KW ? w[i0] : 0u, i0 + 1 < KW ? w[i0 + 1] : 0u, i0 + 2 < KW ? w[i0 + 2] : 0u,
                 i0 + 3 < KW ? w[i0 + 3] : 0u};
  }
}

template <class W>
__device__ __forceinline__ W unpack_word(u32x4 z, int k) {
  constexpr int WB = int(sizeof(W));
  if constexpr (WB == 16) {
    return __builtin_bit_cast(W, z);
  } else if constexpr (WB == 8) {
    return __builtin_bit_cast(W, k == 0 ? u32x2{z.x, z.y} : u32x2{z.z, z.w});
  } else {
    return k == 0 ? z.x : (k == 1 ? z.y : (k == 2 ? z.z : z.w));
  }
}

// The backward hop's links V_mu(x - mu) of the chunk's n sites (LW words of
// each): the thread's word i is word
// tid + i nth of the run, clamped to its last word.
template <int MU, int NV, class S, int LW, int HN, int RN>
__device__ __forceinline__ void lnb_issue(const Geom& g, const FlatChunk<HN>& c, const typename S::word* __restrict__ U,
                                          int tid, u32x4 (&r)[RN]) {
  using W = typename S::word;
  constexpr int CH = RowPieces<S>::CH, E = RN - CH;
  constexpr int KW = (LW + NV - 1) / NV, PER = 16 / int(sizeof(W));
  static_assert((KW + PER - 1) / PER <= E, "the link words fit the extra groups");
  const int nth = KW > 1 ? int(blockDim.x * blockDim.y) : 0;
  const int lim = c.n * LW - 1;
  W w[KW];
#pragma unroll
  for (int i = 0; i < KW; ++i) {
    const int q = tid + i * nth, wi = q < lim ? q : lim;
    const int k = wi / LW, e = wi - k * LW;
    w[i] = U[(size_t(flat_nbr<MU, -1>(g, c, uint32_t(k))) * 4 + MU) * LW + e];
  }
#pragma unroll
  for (int s = 0; s < E; ++s) r[CH + s] = pack_words<W, KW>(w, s * PER);
}

template <int NV, class S, int LW, int RN>
__device__ __forceinline__ void lnb_commit(const u32x4 (&r)[RN], typename S::word* lnb, int n,
                                           int tid) {
  using W = typename S::word;
  constexpr int CH = RowPieces<S>::CH, KW = (LW + NV - 1) / NV, PER = 16 / int(sizeof(W));
  const int nth = KW > 1 ? int(blockDim.x * blockDim.y) : 0;
  const int lim = n * LW - 1;
#pragma unroll
  for (int i = 0; i < KW; ++i) {
    const int q = tid + i * nth;
    lnb[q < lim ? q : lim] = unpack_word<W>(r[CH + i / PER], i % PER);
  }
}

template <int NV, class S, int RN>
__device__ __forceinline__ void extra_clear(u32x4 (&r)[RN]) {
  constexpr int CH = RowPieces<S>::CH, E = RN - CH;
#pragma unroll
  for (int s = 0; s < E; ++s) r[CH + s] = u32x4{0u, 0u, 0u, 0u};
}

// The own row's halo sites, SP pieces each: the thread's group s holds piece
// tid + s nth of the HN SP, clamped to the last.
template <int NV, class S, int HN, int RN>
__device__ __forceinline__ void halo_issue(const FlatChunk<HN>& c, const typename S::word* __restrict__ in, int tid,
                                           u32x4 (&r)[RN]) {
  constexpr int SW = 12 * NV, CH = RowPieces<S>::CH, E = RN - CH;
  constexpr int SP = SW * int(sizeof(typename S::word)) / 16;
  const int nth = E > 1 ? int(blockDim.x * blockDim.y) : 0;
#pragma unroll
  for (int s = 0; s < E; ++s) {
    const int q = tid + s * nth, h = q < HN * SP ? q : HN * SP - 1;
    const int k = h / SP;
    const uint32_t hs = halo_site(c, k);
    r[CH + s] = reinterpret_cast<const u32x4*>(in + size_t(c.plane + hs) * SW)[h - k * SP];
  }
}

template <int NV, class S, int HN, int RN>
__device__ __forceinline__ void halo_commit(const FlatChunk<HN>&, const u32x4 (&r)[RN], typename S::word* buf, int tid, int R) {
  constexpr int SW = 12 * NV, CH = RowPieces<S>::CH, E = RN - CH;
  constexpr int SP = SW * int(sizeof(typename S::word)) / 16, SSP = SiteStride<NV, S>::PIECES;
  const int nth = E > 1 ? int(blockDim.x * blockDim.y) : 0;
#pragma unroll
  for (int s = 0; s < E; ++s) {
    const int q = tid + s * nth, h = q < HN * SP ? q : HN * SP - 1;
    const int k = h / SP, slot = k == 0 ? 0 : R + k;
    (reinterpret_cast<u32x4*>(buf) + slot * SSP)[h - k * SP] = r[CH + s];
  }
}

template <int NV, class S, int LW, int HN>
size_t rows_lds_words(int R) {
  return size_t(R + HN) * SiteStride<NV, S>::WORDS + size_t(R + HN) * 4 * LW + size_t(R) * LW;
}

// Piece assignment of a staged row: lane (x, v) of the workgroup moves the
// pieces j * N_v + v (j = 0 .. CH - 1) of site x of the run, so the N_v lanes
// of a site read N_v consecutive 16-byte pieces per instruction and the LDS
// position follows from the site without a division.  Lanes past a partial
// chunk's end repeat the last site (same data to the same place).
template <int MU, int SGN, int NV, class S, int LW = 9, int HN, int RN>
__device__ __forceinline__ void row_issue(const Geom& g, const FlatChunk<HN>& c, const typename S::word* __restrict__ U,
                                          const typename S::word* __restrict__ in, int xl, int v, int tid,
                                          u32x4 (&r)[RN]) {
  using W = typename S::word;
  constexpr int SW = 12 * NV, CH = RowPieces<S>::CH;
  const int xc = xl < c.n ? xl : c.n - 1;
  const u32x4* src = reinterpret_cast<const u32x4*>(in + size_t(flat_nbr<MU, SGN>(g, c, uint32_t(xc))) * SW);
#pragma unroll
  for (int j = 0; j < CH; ++j) r[j] = src[j * NV + v];
  if (SGN < 0) {
    lnb_issue<MU, NV, S, LW>(g, c, U, tid, r);
  } else {
    // every row writes the whole array, so that call sites merged into one
    // array store the same elements (the compiler's store sinking would
    // otherwise make the array addressable and put it in scratch memory)
    extra_clear<NV, S>(r);
  }
}

template <int SGN, int NV, class S, int LW = 9, int HN, int RN>
__device__ __forceinline__ void row_commit(const FlatChunk<HN>& c, const u32x4 (&r)[RN],
                                           typename S::word* row, typename S::word* lnb, int xl, int v, int tid) {
  using W = typename S::word;
  constexpr int CH = RowPieces<S>::CH, SSP = SiteStride<NV, S>::PIECES;
  const int xc = xl < c.n ? xl : c.n - 1;
  u32x4* dst = reinterpret_cast<u32x4*>(row) + xc * SSP;
#pragma unroll
  for (int j = 0; j < CH; ++j) dst[j * NV + v] = r[j];
  if (SGN < 0) lnb_commit<NV, S, LW>(r, lnb, c.n, tid);
}

// The chunk's own row in the same register shape: CH pieces of site x and,
// in the extra groups, the thread's pieces of the halo sites (HN * 12 N_v
// words; the launcher checks that the groups of the workgroup hold them).
template <int NV, class S, int HN, int RN>
__device__ __forceinline__ void own_issue(const FlatChunk<HN>& c, const typename S::word* __restrict__ in, int xl, int v,
                                          int tid, u32x4 (&r)[RN]) {
  using W = typename S::word;
  constexpr int SW = 12 * NV, CH = RowPieces<S>::CH;
  const int xc = xl < c.n ? xl : c.n - 1;
  const u32x4* src = reinterpret_cast<const u32x4*>(in + size_t(c.plane + c.p0 + xc) * SW);
#pragma unroll
  for (int j = 0; j < CH; ++j) r[j] = src[j * NV + v];
  halo_issue<NV, S>(c, in, tid, r);
}

template <int NV, class S, int HN, int RN>
__device__ __forceinline__ void own_commit(const FlatChunk<HN>& c, const u32x4 (&r)[RN],
                                           typename S::word* buf, int xl, int v, int tid, int R) {
  constexpr int CH = RowPieces<S>::CH, SSP = SiteStride<NV, S>::PIECES;
  const int xc = xl < c.n ? xl : c.n - 1;
  u32x4* dst = reinterpret_cast<u32x4*>(buf) + (xc + 1) * SSP;
#pragma unroll
  for (int j = 0; j < CH; ++j) dst[j * NV + v] = r[j];
  halo_commit<NV, S>(c, r, buf, tid, R);
}

// Only the halo sites of the own row (its interior is already
// in LDS), in the extra groups; the spinor slots are cleared so that every
// call site writes the whole register array.
template <int NV, class S, int HN, int RN>
__device__ __forceinline__ void own_halo_issue(const FlatChunk<HN>& c, const typename S::word* __restrict__ in, int tid,
                                               u32x4 (&r)[RN]) {
  constexpr int CH = RowPieces<S>::CH;
#pragma unroll
  for (int j = 0; j < CH; ++j) r[j] = u32x4{0u, 0u, 0u, 0u};
  halo_issue<NV, S>(c, in, tid, r);
}

template <int NV, class S, int HN, int RN>
__device__ __forceinline__ void own_halo_commit(const FlatChunk<HN>& c, const u32x4 (&r)[RN], typename S::word* buf, int tid, int R) {
  halo_commit<NV, S>(c, r, buf, tid, R);
}

template <int MU, int SGN, bool ADJ, int NV, class S, class T, int LW = 9>
__device__ __forceinline__ void row_compute(const typename S::word* nbr, const typename S::word* lown,
                                            const typename S::word* lnb, int xl, int v, cpx<T> (&acc)[4][3]) {
  constexpr int SSW = SiteStride<NV, S>::WORDS;
  if (SGN > 0)
    lds_hop<MU, (ADJ ? 1 : -1), false, NV, S, T, LW>(nbr + xl * SSW, lown + (xl + 1) * 4 * LW + MU * LW, v, acc);
  else
    lds_hop<MU, (ADJ ? -1 : 1), true, NV, S, T, LW>(nbr + xl * SSW, lnb + xl * LW, v, acc);
}

// ---------------------------------------------------------------- half-spinor
// rows (FP32 complex storage).  A hop reads its neighbour only through the
// projection (1 + C gamma_mu) psi, two spin components per colour (eq. def_wils
// with the chiral gamma matrices).  Lane (x, v) of a site loads, for the
// right-hand-side pair q = v mod N_v/2, the two spins that form half-spin
// component s = v div N_v/2 of that projection (spin s and its partner under
// gamma_mu) in all three colours, projects them, and writes the half spinor
// [s][c][N_v] of the site to LDS: half the LDS writes, reads and space of a full
// row.  The projection is the same sum as in project(), so the results are
// bit-identical to staging the full spinor.

// Partner of spin 0 under gamma_mu (spin 1's partner is 5 minus it).
template <int MU> struct HalfPartner { static constexpr int value = MU <= 1 ? 3 : 2; };

// Site stride of a half-spinor row in LDS, padded like SiteStride.
template <int NV, class S>
struct HalfStride {
  static constexpr int WB = int(sizeof(typename S::word));
  static constexpr int SWD = 6 * NV * WB / 4;
  static constexpr int WIN = NV * WB / 4;
  static constexpr int PAD = (((WIN - SWD) % 64) + 64) % 64;
  static constexpr int DW = (PAD <= SWD / 4 && (PAD * 4) % 16 == 0) ? SWD + PAD : SWD;
  static constexpr int WORDS = DW * 4 / WB;
  static constexpr int PIECES = DW * 4 / 16;
};

template <int MU, int SGN, int NV, class S, int LW = 9, int HN, int RN>
__device__ __forceinline__ void half_issue(const Geom& g, const FlatChunk<HN>& c, const typename S::word* __restrict__ U,
                                           const typename S::word* __restrict__ in, int xl, int v, int tid,
                                           u32x4 (&r)[RN]) {
  static_assert(sizeof(typename S::word) == 8 && NV % 2 == 0 && RowPieces<S>::CH == 6,
                "half-spinor rows take FP32 complex storage and an even N_v");
  constexpr int SW = 12 * NV, HP = NV / 2, P0 = HalfPartner<MU>::value;
  const int xc = xl < c.n ? xl : c.n - 1;
  const u32x4* src = reinterpret_cast<const u32x4*>(in + size_t(flat_nbr<MU, SGN>(g, c, uint32_t(xc))) * SW);
  const int hs = v >= HP ? 1 : 0, q = v - hs * HP;
  const int sa = hs, sb = hs ? 5 - P0 : P0;
#pragma unroll
  for (int cc = 0; cc < 3; ++cc) {
    r[cc] = src[(sa * 3 + cc) * HP + q];
    r[3 + cc] = src[(sb * 3 + cc) * HP + q];
  }
  if (SGN < 0)
    lnb_issue<MU, NV, S, LW>(g, c, U, tid, r);
  else
    extra_clear<NV, S>(r);
}

template <int MU, int SGN, bool ADJ, int NV, class S, int LW = 9, int HN, int RN>
__device__ __forceinline__ void half_commit(const FlatChunk<HN>& c, const u32x4 (&r)[RN],
                                            typename S::word* hrow, typename S::word* lnb, int xl, int v, int tid) {
  using W = typename S::word;
  constexpr int HP = NV / 2, HSP = HalfStride<NV, S>::PIECES;
  constexpr int C = SGN > 0 ? (ADJ ? 1 : -1) : (ADJ ? -1 : 1);
  const int xc = xl < c.n ? xl : c.n - 1;
  const int hs = v >= HP ? 1 : 0, q = v - hs * HP;
  // h_s = psi_s + sg X(psi_partner), X = C i (MU = 0, 2) or C (MU = 1, 3)
  const float sg = MU == 0 ? -1.f : (MU == 3 ? 1.f : (hs ? 1.f : -1.f));
  u32x4* dst = reinterpret_cast<u32x4*>(hrow) + xc * HSP + hs * 3 * HP + q;
#pragma unroll
  for (int cc = 0; cc < 3; ++cc) {
    // whole-vector bit casts (a bit cast of a vector element is miscompiled)
    const f32x4 a = __builtin_bit_cast(f32x4, r[cc]), b = __builtin_bit_cast(f32x4, r[3 + cc]);
    f32x4 x;
    if constexpr (MU == 0 || MU == 2) {
      x = f32x4{float(-C) * b.y, float(C) * b.x, float(-C) * b.w, float(C) * b.z};
    } else {
      x = f32x4{float(C) * b.x, float(C) * b.y, float(C) * b.z, float(C) * b.w};
    }
    const f32x4 h = f32x4{a.x + sg * x.x, a.y + sg * x.y, a.z + sg * x.z, a.w + sg * x.w};
    dst[cc * HP] = __builtin_bit_cast(u32x4, h);
  }
  if (SGN < 0) lnb_commit<NV, S, LW>(r, lnb, c.n, tid);
}

template <int MU, int SGN, bool ADJ, int NV, class S, class T, int LW = 9>
__device__ __forceinline__ void half_compute(const typename S::word* hrow, const typename S::word* lown,
                                             const typename S::word* lnb, int xl, int v, cpx<T> (&acc)[4][3]) {
  constexpr int HSW = HalfStride<NV, S>::WORDS;
  constexpr int C = SGN > 0 ? (ADJ ? 1 : -1) : (ADJ ? -1 : 1);
  const typename S::word* site = hrow + xl * HSW;
  cpx<T> h[2][3];
#pragma unroll
  for (int hs = 0; hs < 2; ++hs)
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) h[hs][cc] = S::template load<T>(site + (hs * 3 + cc) * NV + v);
  const typename S::word* link = SGN > 0 ? lown + (xl + 1) * 4 * LW + MU * LW : lnb + xl * LW;
  cpx<T> u[3][3];
  if constexpr (LW == 9) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) u[a][b] = S::template load<T>(link + a * 3 + b);
  } else {
    load_link_lw<LW, S, T>(link, u);
  }
  cpx<T> t[2][3];
  su3_mul2<(SGN < 0), T>(u, h, t);
  reconstruct_add<MU, C, T>(acc, t);
}

// Full or half-spinor staging of a neighbour row, by HALF.
template <bool HALF, int MU, int SGN, bool ADJ, int NV, class S, int LW, int HN, int RN>
__device__ __forceinline__ void o_commit(const FlatChunk<HN>& c, const u32x4 (&r)[RN],
                                         typename S::word* row, typename S::word* lnb, int xl, int v, int tid) {
  if constexpr (HALF)
    half_commit<MU, SGN, ADJ, NV, S, LW>(c, r, row, lnb, xl, v, tid);
  else
    row_commit<SGN, NV, S, LW>(c, r, row, lnb, xl, v, tid);
}

template <bool HALF, int MU, int SGN, bool ADJ, int NV, class S, class T, int LW>
__device__ __forceinline__ void o_compute(const typename S::word* row, const typename S::word* lown,
                                          const typename S::word* lnb, int xl, int v, cpx<T> (&acc)[4][3]) {
  if constexpr (HALF)
    half_compute<MU, SGN, ADJ, NV, S, T, LW>(row, lown, lnb, xl, v, acc);
  else
    row_compute<MU, SGN, ADJ, NV, S, T, LW>(row, lown, lnb, xl, v, acc);
}

// Links of the chunk's sites (4 LW words each), and V_x of the halo sites that a
// lane finds at x - 1 (slot 0, HN = 4: and R + 3): the last piece of the first
// threads.
template <class S, int LW = 9>
struct LinkPieces {
  static constexpr int PER_SITE = 4 * LW * int(sizeof(typename S::word)) / 16;
  static constexpr int XP = (LW * int(sizeof(typename S::word)) + 15) / 16;
};

// Pieces of the chunk's links per thread: ceil(LP / threads per site).
template <class S, int THREADS_PER_SITE, int LW = 9>
struct LinkK {
  static constexpr int value = (LinkPieces<S, LW>::PER_SITE + THREADS_PER_SITE - 1) / THREADS_PER_SITE;
};

template <class S, int K, int LW = 9, int HN>
__device__ __forceinline__ void links_issue(const FlatChunk<HN>& c, const typename S::word* __restrict__ U, int tid, int nth,
                                            u32x4 (&lr)[K + 1]) {
  constexpr int LP = LinkPieces<S, LW>::PER_SITE;
  constexpr int XP = LinkPieces<S, LW>::XP;
  const u32x4* own = reinterpret_cast<const u32x4*>(U + size_t(c.plane + c.p0) * 4 * LW);
  const int pieces = c.n * LP;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const int i = tid + j * nth;
    lr[j] = own[i < pieces ? i : pieces - 1];
  }
  constexpr int HP = HN == 2 ? XP : 2 * XP;
  const int h = tid < HP ? tid : HP - 1, k = h >= XP ? 1 : 0;
  lr[K] = reinterpret_cast<const u32x4*>(U + size_t(c.plane + halo_site(c, k ? HN - 1 : 0)) * 4 * LW)[h - k * XP];
}

template <class S, int K, int LW = 9, int HN>
__device__ __forceinline__ void links_commit(const FlatChunk<HN>& c, const u32x4 (&lr)[K + 1], typename S::word* lown,
                                             int tid, int nth, int R) {
  constexpr int LP = LinkPieces<S, LW>::PER_SITE, XP = LinkPieces<S, LW>::XP;
  u32x4* own = reinterpret_cast<u32x4*>(lown + 4 * LW);
  const int pieces = c.n * LP;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const int i = tid + j * nth;
    own[i < pieces ? i : pieces - 1] = lr[j];
  }
  constexpr int HP = HN == 2 ? XP : 2 * XP;
  const int h = tid < HP ? tid : HP - 1, k = h >= XP ? 1 : 0;
  reinterpret_cast<u32x4*>(lown + (k ? (R + 3) * 4 * LW : 0))[h - k * XP] = lr[K];
}

// Occupancy hint per prefetch depth: deeper prefetch holds more rows in
// registers (about 28 VGPRs per FP32 row) and runs fewer waves per SIMD.
template <int DEPTH> struct RowsWaves { static constexpr int value = DEPTH <= 2 ? 4 : (DEPTH <= 4 ? 3 : 2); };

// CLOV: adds the site-local clover term C(x) in(x) (packed, 36 words per
// site, staged in LDS after lnb).
template <int DEPTH, bool ADJ, bool CLOV, int NV, class S, class T, int HN>
__global__ void __launch_bounds__(256, RowsWaves<DEPTH>::value)
    wilson_rows_kernel(Geom g, FlatMarch m, int xcd, const typename S::word* __restrict__ U,
                       const typename S::word* __restrict__ in, typename S::word* __restrict__ out,
                       const typename S::word* __restrict__ C, T diag) {
  using W = typename S::word;
  constexpr int SW = 12 * NV, CH = RowPieces<S>::CH;
  constexpr int SSW = SiteStride<NV, S>::WORDS, SSP = SiteStride<NV, S>::PIECES;
  extern __shared__ uint4 smem_rows[];
  const int R = int(m.sb);
  W* buf = reinterpret_cast<W*>(smem_rows);
  W* lown = buf + (R + HN) * SSW;
  W* lnb = lown + (R + HN) * 36;
  W* lcl = lnb + ((R * 9 + 3) & ~3);  // [R][36] clover words of the chunk's sites (CLOV), 16-byte aligned

  const uint32_t L = xcd_block(blockIdx.x, gridDim.x, xcd != 0);
  uint32_t seg;
  const FlatChunk<HN> c = flat_chunk<HN>(g, m, L, seg);
  const int v = threadIdx.x, xl = threadIdx.y;
  const int tid = xl * NV + v, nth = R * NV;
  const XSlots xs = x_slots(g, c, R, xl);

  // Seven rows pass through the one LDS row buffer: +y, -y, +z, -z, +t, -t,
  // then the chunk's own row with its halo sites.  Row k is requested DEPTH
  // steps before it is consumed (DEPTH = 7: all at once), each into its own
  // register array.
  constexpr int RN = RowRegs<NV, S, HN>::N;
  u32x4 r0[RN], r1[RN], r2[RN], r3[RN], r4[RN], r5[RN], r6[RN];
#define DSL_ISSUE(K)                                                                   \
  do {                                                                                 \
    if constexpr (K == 0) row_issue<1, +1, NV, S>(g, c, U, in, xl, v, tid, r0);        \
    if constexpr (K == 1) row_issue<1, -1, NV, S>(g, c, U, in, xl, v, tid, r1);        \
    if constexpr (K == 2) row_issue<2, +1, NV, S>(g, c, U, in, xl, v, tid, r2);        \
    if constexpr (K == 3) row_issue<2, -1, NV, S>(g, c, U, in, xl, v, tid, r3);        \
    if constexpr (K == 4) row_issue<3, +1, NV, S>(g, c, U, in, xl, v, tid, r4);        \
    if constexpr (K == 5) row_issue<3, -1, NV, S>(g, c, U, in, xl, v, tid, r5);        \
    if constexpr (K == 6) own_issue<NV, S>(c, in, xl, v, tid, r6);             \
  } while (0)
  // The links (and clover words) are committed first, so they are requested
  // first: loads retire in order.
  constexpr int LK = LinkK<S, NV>::value;
  u32x4 lr[LK + 1], cr[CLOV ? LK : 1];
  links_issue<S, LK>(c, U, tid, nth, lr);
  if constexpr (CLOV) pieces_issue<LK>(cr, C + size_t(c.plane + c.p0) * 36, c.n * LinkPieces<S>::PER_SITE, tid, nth);
  __builtin_amdgcn_sched_barrier(0);
  DSL_ISSUE(0);
  if constexpr (DEPTH > 1) DSL_ISSUE(1);
  if constexpr (DEPTH > 2) DSL_ISSUE(2);
  if constexpr (DEPTH > 3) DSL_ISSUE(3);
  if constexpr (DEPTH > 4) DSL_ISSUE(4);
  if constexpr (DEPTH > 5) DSL_ISSUE(5);
  if constexpr (DEPTH > 6) DSL_ISSUE(6);
  links_commit<S, LK>(c, lr, lown, tid, nth, R);
  if constexpr (CLOV) pieces_commit<LK>(cr, lcl, c.n * LinkPieces<S>::PER_SITE, tid, nth);

  cpx<T> acc[4][3];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) acc[a][b] = zero<T>();

  // Lanes past a partial chunk's end (xl >= n) compute on stale but in-bounds
  // LDS data and their results are never copied out; keeping every lane on
  // the same straight-line path lets the compiler keep the prefetches in
  // flight across the hops.
  W* const row = buf + SSW;  // neighbour rows sit at index 1 .. n
#define DSL_ROW_STEP(K, MU, SGN, CUR)                                         \
  row_commit<SGN, NV, S>(c, CUR, row, lnb, xl, v, tid);                       \
  __syncthreads();                                                            \
  if constexpr (K + DEPTH < 7) DSL_ISSUE(K + DEPTH);                          \
  row_compute<MU, SGN, ADJ, NV, S, T>(row, lown, lnb, xl, v, acc);            \
  __syncthreads();
  DSL_ROW_STEP(0, 1, +1, r0)
  DSL_ROW_STEP(1, 1, -1, r1)
  DSL_ROW_STEP(2, 2, +1, r2)
  DSL_ROW_STEP(3, 2, -1, r3)
  DSL_ROW_STEP(4, 3, +1, r4)
  DSL_ROW_STEP(5, 3, -1, r5)
#undef DSL_ROW_STEP
#undef DSL_ISSUE

  own_commit<NV, S>(c, r6, buf, xl, v, tid, R);
  __syncthreads();
  cpx<T> res[4][3];
  {
    constexpr int CF = ADJ ? +1 : -1, CB = -CF;
    // x hops from the own row (the x - 1 link in the same slot)
    lds_hop<0, CF, false, NV, S, T>(buf + xs.f * SSW, lown + (xl + 1) * 36, v, acc);
    lds_hop<0, CB, true, NV, S, T>(buf + xs.b * SSW, lown + xs.b * 36, v, acc);
    const W* self = buf + (xl + 1) * SSW;
    if constexpr (CLOV) {
      cpx<T> p[4][3];
      lds_spinor<S, T, NV>(self, v, p);
#pragma unroll
      for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
          res[sp][cc].r = fma(diag, p[sp][cc].r, T(-0.5) * acc[sp][cc].r);
          res[sp][cc].i = fma(diag, p[sp][cc].i, T(-0.5) * acc[sp][cc].i);
        }
      clover_madd<S, T>(lcl + xl * 36, p, res);
    } else {
#pragma unroll
      for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
          cpx<T> p = S::template load<T>(self + (sp * 3 + cc) * NV + v);
          res[sp][cc].r = fma(diag, p.r, T(-0.5) * acc[sp][cc].r);
          res[sp][cc].i = fma(diag, p.i, T(-0.5) * acc[sp][cc].i);
        }
    }
  }
  __syncthreads();
  {
    W* o = buf + xl * SSW;
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int cc = 0; cc < 3; ++cc) S::template store<T>(o + (sp * 3 + cc) * NV + v, res[sp][cc]);
  }
  __syncthreads();
  {
    // copy-out with the same site-local piece assignment as the staging
    const int xc = xl < c.n ? xl : c.n - 1;
    const u32x4* src = reinterpret_cast<const u32x4*>(buf) + xc * SSP;
    u32x4* dst = reinterpret_cast<u32x4*>(out + size_t(c.plane + c.p0 + xc) * SW);
    u32x4 r[CH];
#pragma unroll
    for (int j = 0; j < CH; ++j) r[j] = src[j * NV + v];
    // outputs are never read again by this kernel: stream them past the L2
    // so its capacity stays with the input rows that neighbours reuse
#pragma unroll
    for (int j = 0; j < CH; ++j) __builtin_nontemporal_store(r[j], &dst[j * NV + v]);
  }
}

// ---------------------------------------------------------------- t-marching variant
// A workgroup owns the x-row chunk at (y, z) for T consecutive t and steps
// through them.  The -t hop of step t + 1 is U_t(x, t)^dag (1 -/+ gamma_t) psi(x, t),
// formed at step t from the own row already in LDS (a carry of one half
// spinor per lane), so after the first step only six rows are staged per
// output row: +y, -y, +z, -z, +t and the own row, and the +t row of one step
// is the own row of the next, read again while it is still in L2.

// Row K of a step's sequence (0 +y, 1 -y, 2 +z, 3 -z, 4 +t, 5 -t, 6 own, 7 the
// own row's halo sites only) into its register array.
template <int K, int NV, class S, int LW = 9, int HN, int RN>
__device__ __forceinline__ void march_issue(const Geom& g, const FlatChunk<HN>& c, const typename S::word* __restrict__ U,
                                            const typename S::word* __restrict__ in, int xl, int v, int tid, u32x4 (&r0)[RN],
                                            u32x4 (&r1)[RN], u32x4 (&r2)[RN],
                                            u32x4 (&r3)[RN], u32x4 (&r4)[RN],
                                            u32x4 (&r5)[RN], u32x4 (&r6)[RN]) {
  if constexpr (K == 0) row_issue<1, +1, NV, S, LW>(g, c, U, in, xl, v, tid, r0);
  if constexpr (K == 1) row_issue<1, -1, NV, S, LW>(g, c, U, in, xl, v, tid, r1);
  if constexpr (K == 2) row_issue<2, +1, NV, S, LW>(g, c, U, in, xl, v, tid, r2);
  if constexpr (K == 3) row_issue<2, -1, NV, S, LW>(g, c, U, in, xl, v, tid, r3);
  if constexpr (K == 4) row_issue<3, +1, NV, S, LW>(g, c, U, in, xl, v, tid, r4);
  if constexpr (K == 5) row_issue<3, -1, NV, S, LW>(g, c, U, in, xl, v, tid, r5);
  if constexpr (K == 6) own_issue<NV, S>(c, in, xl, v, tid, r6);
  if constexpr (K == 7) own_halo_issue<NV, S>(c, in, tid, r6);
}

// march_issue with the neighbour rows (K = 0 .. 3 and 5) as half spinors.
template <bool HALF, int K, int NV, class S, int LW = 9, int HN, int RN>
__device__ __forceinline__ void march_issue_o(const Geom& g, const FlatChunk<HN>& c, const typename S::word* __restrict__ U,
                                              const typename S::word* __restrict__ in, int xl, int v, int tid, u32x4 (&r0)[RN],
                                              u32x4 (&r1)[RN], u32x4 (&r2)[RN],
                                              u32x4 (&r3)[RN], u32x4 (&r4)[RN],
                                              u32x4 (&r5)[RN], u32x4 (&r6)[RN]) {
  if constexpr (HALF && K == 0) half_issue<1, +1, NV, S, LW>(g, c, U, in, xl, v, tid, r0);
  else if constexpr (HALF && K == 1) half_issue<1, -1, NV, S, LW>(g, c, U, in, xl, v, tid, r1);
  else if constexpr (HALF && K == 2) half_issue<2, +1, NV, S, LW>(g, c, U, in, xl, v, tid, r2);
  else if constexpr (HALF && K == 3) half_issue<2, -1, NV, S, LW>(g, c, U, in, xl, v, tid, r3);
  else if constexpr (HALF && K == 5) half_issue<3, -1, NV, S, LW>(g, c, U, in, xl, v, tid, r5);
  else march_issue<K, NV, S, LW>(g, c, U, in, xl, v, tid, r0, r1, r2, r3, r4, r5, r6);
}

// Sequence of staged rows in a step: all seven in the first step of a
// workgroup, without the -t row (K = 5) afterwards.
template <bool FIRST> struct MarchSeq {
  static constexpr int N = FIRST ? 7 : 6;
  static constexpr int at(int p) { return FIRST ? p : (p < 5 ? p : 6); }
};

// Sequence of the own-buffer step: the own row first and the +t row last, into
// the same buffer, so the +t row of step t is the own row of step t + 1 and a
// later step stages only its halo sites (K = 7).
//   first step: own, +y, -y, +z, -z, -t, +t     later steps: halo, +y, -y, +z, -z, +t
template <bool FIRST> struct MarchSeqO {
  static constexpr int N = FIRST ? 7 : 6;
  static constexpr int at(int p) {
    return p == 0 ? (FIRST ? 6 : 7) : (p <= 4 ? p - 1 : (FIRST ? (p == 5 ? 5 : 4) : 4));
  }
};

template <class T>
__device__ __forceinline__ void hold_acc(cpx<T> (&acc)[4][3]) {
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) hold(acc[a][b]);
}

// Two or three rows in flight fit the 168 VGPRs of three waves per SIMD.
template <int DEPTH> struct MarchWaves { static constexpr int value = DEPTH <= 3 ? 3 : 2; };

template <bool FIRST, int DEPTH, bool ADJ, int NV, class S, class T, int LW, int EPI = EPI_STORE, int HN, int RN>
__device__ __forceinline__ void march_step(const Geom& g, const FlatChunk<HN>& c,
                                           const typename S::word* __restrict__ U,
                                           const typename S::word* __restrict__ in, typename S::word* __restrict__ out,
                                           typename S::word* buf, typename S::word* lown, typename S::word* lnb,
                                           XSlots xs, int R, int xl, int v, int tid, int nth, T diag,
                                           u32x4 (&r0)[RN], u32x4 (&r1)[RN],
                                           u32x4 (&r2)[RN], u32x4 (&r3)[RN],
                                           u32x4 (&r4)[RN], u32x4 (&r5)[RN],
                                           u32x4 (&r6)[RN], u32x4 (&lr)[LinkK<S, NV, LW>::value + 1],
                                           cpx<T> (&carry)[2][3], EpiLane<S>& ep) {
  using W = typename S::word;
  using Q = MarchSeq<FIRST>;
  constexpr int LK = LinkK<S, NV, LW>::value;
  constexpr int SW = 12 * NV, CH = RowPieces<S>::CH;
  constexpr int SSW = SiteStride<NV, S>::WORDS, SSP = SiteStride<NV, S>::PIECES;
  constexpr int CF = ADJ ? +1 : -1, CB = -CF;
  // the first step's leading rows and links were requested by the caller; a
  // later step requests them here, after the previous step's last barrier
  if constexpr (!FIRST) {
    links_issue<S, LK, LW>(c, U, tid, nth, lr);  // (first: see march_step_o)
    __builtin_amdgcn_sched_barrier(0);
#define DSL_SISSUE(P) march_issue<Q::at(P), NV, S, LW>(g, c, U, in, xl, v, tid, r0, r1, r2, r3, r4, r5, r6)
    DSL_SISSUE(0);
    if constexpr (DEPTH > 1) DSL_SISSUE(1);
    if constexpr (DEPTH > 2) DSL_SISSUE(2);
    if constexpr (DEPTH > 3) DSL_SISSUE(3);
    if constexpr (DEPTH > 4) DSL_SISSUE(4);
    if constexpr (DEPTH > 5) DSL_SISSUE(5);
#undef DSL_SISSUE
  }
  links_commit<S, LK, LW>(c, lr, lown, tid, nth, R);

  cpx<T> acc[4][3];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) acc[a][b] = zero<T>();

  W* const row = buf + SSW;
#define DSL_MISSUE(P, CH_)                                                                             \
  march_issue<Q::at(P), NV, S, LW>(g, CH_, U, in, xl, v, tid, r0, r1, r2, r3, r4, r5, r6)
#define DSL_MSTEP(P, MU, SGN, CUR)                                        \
  if constexpr (P < Q::N - 1) {                                           \
    row_commit<SGN, NV, S, LW>(c, CUR, row, lnb, xl, v, tid);                 \
    __syncthreads();                                                      \
    if constexpr (P + DEPTH < Q::N) DSL_MISSUE(P + DEPTH, c);             \
    row_compute<MU, SGN, ADJ, NV, S, T, LW>(row, lown, lnb, xl, v, acc);      \
    hold_acc<T>(acc);                                                     \
    __syncthreads();                                                      \
  }
  DSL_MSTEP(0, 1, +1, r0)
  DSL_MSTEP(1, 1, -1, r1)
  DSL_MSTEP(2, 2, +1, r2)
  DSL_MSTEP(3, 2, -1, r3)
  DSL_MSTEP(4, 3, +1, r4)
  DSL_MSTEP(5, 3, -1, r5)
#undef DSL_MSTEP

  own_commit<NV, S>(c, r6, buf, xl, v, tid, R);
  __syncthreads();
#undef DSL_MISSUE
  cpx<T> res[4][3];
  {
    lds_hop<0, CF, false, NV, S, T, LW>(buf + xs.f * SSW, lown + (xl + 1) * 4 * LW, v, acc);
    lds_hop<0, CB, true, NV, S, T, LW>(buf + xs.b * SSW, lown + xs.b * 4 * LW, v, acc);
    if constexpr (!FIRST) reconstruct_add<3, CB, T>(acc, carry);
    const W* self = buf + (xl + 1) * SSW;
    cpx<T> p[4][3];
    lds_spinor<S, T, NV>(self, v, p);
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int cc = 0; cc < 3; ++cc) {
        res[sp][cc].r = fma(diag, p[sp][cc].r, T(-0.5) * acc[sp][cc].r);
        res[sp][cc].i = fma(diag, p[sp][cc].i, T(-0.5) * acc[sp][cc].i);
      }
    // carry for the next step: U_t(x, t)^dag (1 + CB gamma_t) psi(x, t), projected
    cpx<T> h[2][3];
    project<3, CB, T>(p, h);
    cpx<T> u[3][3];
    load_link_lw<LW, S, T>(lown + (xl + 1) * 4 * LW + 3 * LW, u);
    su3_mul2<true, T>(u, h, carry);
  }
  __syncthreads();
  {
    W* o = buf + xl * SSW;
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int cc = 0; cc < 3; ++cc) S::template store<T>(o + (sp * 3 + cc) * NV + v, res[sp][cc]);
  }
  __syncthreads();
  {
    const int xc = xl < c.n ? xl : c.n - 1;
    const u32x4* src = reinterpret_cast<const u32x4*>(buf) + xc * SSP;
    u32x4* dst = reinterpret_cast<u32x4*>(out + size_t(c.plane + c.p0 + xc) * SW);
    epi_copy_out<EPI, NV, S, CH>(src, dst, v, xl < c.n, ep);
  }
  __syncthreads();
}

// The same step with two row buffers used in turn: row k + 1 is written to
// one buffer while row k is applied from the other, so each staged row costs
// one barrier instead of two.  LDS: buf0, buf1 [(R + HN) SSW], lown, lnb0, lnb1.
template <bool FIRST, int DEPTH, bool ADJ, int NV, class S, class T, int LW, int EPI = EPI_STORE, int HN, int RN>
__device__ __forceinline__ void march_step_pp(const Geom& g, const FlatChunk<HN>& c,
                                              const typename S::word* __restrict__ U,
                                              const typename S::word* __restrict__ in,
                                              typename S::word* __restrict__ out, typename S::word* buf0,
                                              typename S::word* buf1, typename S::word* lown, typename S::word* lnb0,
                                              typename S::word* lnb1, XSlots xs, int R, int xl, int v, int tid, int nth,
                                              T diag, u32x4 (&r0)[RN],
                                              u32x4 (&r1)[RN], u32x4 (&r2)[RN],
                                              u32x4 (&r3)[RN], u32x4 (&r4)[RN],
                                              u32x4 (&r5)[RN], u32x4 (&r6)[RN],
                                              u32x4 (&lr)[LinkK<S, NV, LW>::value + 1], cpx<T> (&carry)[2][3], EpiLane<S>& ep) {
  using W = typename S::word;
  using Q = MarchSeq<FIRST>;
  constexpr int LK = LinkK<S, NV, LW>::value;
  constexpr int SW = 12 * NV, CH = RowPieces<S>::CH;
  constexpr int SSW = SiteStride<NV, S>::WORDS, SSP = SiteStride<NV, S>::PIECES;
  constexpr int CF = ADJ ? +1 : -1, CB = -CF;
  if constexpr (!FIRST) {
#define DSL_SISSUE(P) march_issue<Q::at(P), NV, S, LW>(g, c, U, in, xl, v, tid, r0, r1, r2, r3, r4, r5, r6)
    links_issue<S, LK, LW>(c, U, tid, nth, lr);
    __builtin_amdgcn_sched_barrier(0);
    DSL_SISSUE(0);
    if constexpr (DEPTH > 1) DSL_SISSUE(1);
    if constexpr (DEPTH > 2) DSL_SISSUE(2);
#undef DSL_SISSUE
  }
  links_commit<S, LK, LW>(c, lr, lown, tid, nth, R);

  cpx<T> acc[4][3];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) acc[a][b] = zero<T>();

#define DSL_MISSUE(P) march_issue<Q::at(P), NV, S, LW>(g, c, U, in, xl, v, tid, r0, r1, r2, r3, r4, r5, r6)
  // row P of the sequence goes to buffer P % 2
#define DSL_BUF(P) ((P) % 2 == 0 ? buf0 : buf1)
#define DSL_LNB(P) ((P) % 2 == 0 ? lnb0 : lnb1)
#define DSL_COMMIT(P, SGN, CUR) row_commit<SGN, NV, S, LW>(c, CUR, DSL_BUF(P) + SSW, DSL_LNB(P), xl, v, tid)
  DSL_COMMIT(0, +1, r0);
  __syncthreads();
  // P: the row applied now; then P + 1 is written into the other buffer
#define DSL_PSTEP(P, MU, SGN, NSGN, NCUR)                                             \
  if constexpr (P + DEPTH < Q::N) DSL_MISSUE(P + DEPTH);                              \
  row_compute<MU, SGN, ADJ, NV, S, T, LW>(DSL_BUF(P) + SSW, lown, DSL_LNB(P), xl, v, acc); \
  hold_acc<T>(acc);                                                                   \
  if constexpr (P + 1 < Q::N - 1) DSL_COMMIT(P + 1, NSGN, NCUR);                      \
  if constexpr (P + 1 == Q::N - 1) own_commit<NV, S>(c, r6, DSL_BUF(P + 1), xl, v, tid, R); \
  __syncthreads();
  if constexpr (FIRST) {
    DSL_PSTEP(0, 1, +1, -1, r1)
    DSL_PSTEP(1, 1, -1, +1, r2)
    DSL_PSTEP(2, 2, +1, -1, r3)
    DSL_PSTEP(3, 2, -1, +1, r4)
    DSL_PSTEP(4, 3, +1, -1, r5)
    DSL_PSTEP(5, 3, -1, +1, r0)
  } else {
    DSL_PSTEP(0, 1, +1, -1, r1)
    DSL_PSTEP(1, 1, -1, +1, r2)
    DSL_PSTEP(2, 2, +1, -1, r3)
    DSL_PSTEP(3, 2, -1, +1, r4)
    DSL_PSTEP(4, 3, +1, +1, r0)
  }
#undef DSL_PSTEP
#undef DSL_COMMIT
#undef DSL_MISSUE
  W* const own = DSL_BUF(Q::N - 1);
#undef DSL_BUF
#undef DSL_LNB
  cpx<T> res[4][3];
  {
    lds_hop<0, CF, false, NV, S, T, LW>(own + xs.f * SSW, lown + (xl + 1) * 4 * LW, v, acc);
    lds_hop<0, CB, true, NV, S, T, LW>(own + xs.b * SSW, lown + xs.b * 4 * LW, v, acc);
    if constexpr (!FIRST) reconstruct_add<3, CB, T>(acc, carry);
    cpx<T> p[4][3];
    lds_spinor<S, T, NV>(own + (xl + 1) * SSW, v, p);
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int cc = 0; cc < 3; ++cc) {
        res[sp][cc].r = fma(diag, p[sp][cc].r, T(-0.5) * acc[sp][cc].r);
        res[sp][cc].i = fma(diag, p[sp][cc].i, T(-0.5) * acc[sp][cc].i);
      }
    cpx<T> h[2][3];
    project<3, CB, T>(p, h);
    cpx<T> u[3][3];
    load_link_lw<LW, S, T>(lown + (xl + 1) * 4 * LW + 3 * LW, u);
    su3_mul2<true, T>(u, h, carry);
  }
  // the output leaves through the other buffer (free since the last barrier)
  W* const ob = own == buf0 ? buf1 : buf0;
  {
    W* o = ob + xl * SSW;
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int cc = 0; cc < 3; ++cc) S::template store<T>(o + (sp * 3 + cc) * NV + v, res[sp][cc]);
  }
  __syncthreads();
  {
    const int xc = xl < c.n ? xl : c.n - 1;
    const u32x4* src = reinterpret_cast<const u32x4*>(ob) + xc * SSP;
    u32x4* dst = reinterpret_cast<u32x4*>(out + size_t(c.plane + c.p0 + xc) * SW);
    epi_copy_out<EPI, NV, S, CH>(src, dst, v, xl < c.n, ep);
  }
  __syncthreads();
}

// The step with three buffers: bo holds the own row (with its halo sites)
// and receives the +t row at the end of the step, which is then the next
// step's own row; ba and bb take the other rows in turn (one barrier per staged
// row) and the output.  The own row is gone from bo when the output is formed:
// in BF16, and where N_x lets rows of every block size be made of whole chunks
// (rows_fold), the diagonal term is folded into acc as -2 diag psi at the start (16^3 x
// 32, FP32: 91.8 us against 95.6), elsewhere (late; LATE for chunks of one x-row) the own
// row is read once more before the +t row takes its place and diag psi added last, as
// the direct kernel does (error against FP64, relative: 4.8e-8 against 7.7e-8).
// LDS: bo [(R + HN) SSW], ba, bb [R SSW], lown, lnba, lnbb [R LW].
// HALF: the +-y, +-z and first -t rows go through ba and bb as half spinors
// (ba, bb [R HSW], adjacent), and the output through ba and bb together.
template <bool FIRST, int DEPTH, bool ADJ, int NV, class S, class T, int LW, bool HALF, int EPI, bool LATE, int HN, int RN>
__device__ __forceinline__ void march_step_o(const Geom& g, const FlatChunk<HN>& c, const FlatChunk<HN>& cn,
                                             const typename S::word* __restrict__ U,
                                             const typename S::word* __restrict__ in,
                                             typename S::word* __restrict__ out, typename S::word* bo,
                                             typename S::word* ba, typename S::word* bb, typename S::word* lown,
                                             typename S::word* lnba, typename S::word* lnbb, XSlots xs, int R, int xl,
                                             int v, int tid, int nth, T diag, bool late, u32x4 (&r0)[RN],
                                             u32x4 (&r1)[RN], u32x4 (&r2)[RN],
                                             u32x4 (&r3)[RN], u32x4 (&r4)[RN],
                                             u32x4 (&r5)[RN], u32x4 (&r6)[RN],
                                             u32x4 (&lr)[LinkK<S, NV, LW>::value + 1], cpx<T> (&carry)[2][3], EpiLane<S>& ep) {
  using W = typename S::word;
  using Q = MarchSeqO<FIRST>;
  if constexpr (HN == 2) late = LATE;
  constexpr int LK = LinkK<S, NV, LW>::value;
  constexpr int SW = 12 * NV, CH = RowPieces<S>::CH;
  constexpr int SSW = SiteStride<NV, S>::WORDS, SSP = SiteStride<NV, S>::PIECES;
  constexpr int CF = ADJ ? +1 : -1, CB = -CF;
  // The next step's halo sites, then its links (the last step repeats its own),
  // before the +t row of this one is applied: the links come from HBM, the
  // rows mostly from L2, and loads retire in order, so that links requested in
  // front of the rows hold them up (16^3 x 32: 102 us) and behind them make the
  // step wait for all its leading rows (105 us); from here they have the +t hop
  // and the output to arrive in (91.8 us; between the y rows 94.7; 32^4: 783
  // against 811).  The scheduling barriers keep the compiler to the order.
#define DSL_ONEXT                                                                                             \
  march_issue_o<HALF, 7, NV, S, LW>(g, cn, U, in, xl, v, tid, r0, r1, r2, r3, r4, r5, r6);                    \
  links_issue<S, LK, LW>(cn, U, tid, nth, lr);                                                                \
  __builtin_amdgcn_sched_barrier(0);
#define DSL_OISSUE(P) \
  march_issue_o<HALF, Q::at(P), NV, S, LW>(g, c, U, in, xl, v, tid, r0, r1, r2, r3, r4, r5, r6)
  // The halo sites and links were requested by the previous step (DSL_ONEXT).
  if constexpr (!FIRST) {
    if constexpr (DEPTH > 1) DSL_OISSUE(1);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (DEPTH > 2) DSL_OISSUE(2);
  }
  links_commit<S, LK, LW>(c, lr, lown, tid, nth, R);
  if constexpr (FIRST)
    own_commit<NV, S>(c, r6, bo, xl, v, tid, R);
  else
    own_halo_commit<NV, S>(c, r6, bo, tid, R);
  __syncthreads();
  if constexpr (DEPTH < Q::N) DSL_OISSUE(DEPTH);
  cpx<T> acc[4][3];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) acc[a][b] = zero<T>();
  {
    if constexpr (!FIRST) reconstruct_add<3, CB, T>(acc, carry);
    cpx<T> p[4][3];
    lds_spinor<S, T, NV>(bo + (xl + 1) * SSW, v, p);
    if (!late) {
      const T m2d = T(-2) * diag;
#pragma unroll
      for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) acc[sp][cc] = rmadd(acc[sp][cc], m2d, p[sp][cc]);
    }
    // carry for the next step: U_t(x, t)^dag (1 + CB gamma_t) psi(x, t), projected
    cpx<T> h[2][3];
    project<3, CB, T>(p, h);
    cpx<T> u[3][3];
    load_link_lw<LW, S, T>(lown + (xl + 1) * 4 * LW + 3 * LW, u);
    su3_mul2<true, T>(u, h, carry);
  }
  hold_acc<T>(acc);
  lds_hop<0, CF, false, NV, S, T, LW>(bo + xs.f * SSW, lown + (xl + 1) * 4 * LW, v, acc);
  lds_hop<0, CB, true, NV, S, T, LW>(bo + xs.b * SSW, lown + xs.b * 4 * LW, v, acc);
  hold_acc<T>(acc);
  o_commit<HALF, 1, +1, ADJ, NV, S, LW>(c, r0, ba, lnba, xl, v, tid);
  __syncthreads();
  // row P (in buffer BUF) applied, then row P + 1 written to NBUF
#define DSL_OSTEP(P, MU, SGN, H, BUF, LNB)                                     \
  if constexpr (P + DEPTH < Q::N) DSL_OISSUE(P + DEPTH);                       \
  o_compute<H, MU, SGN, ADJ, NV, S, T, LW>(BUF, lown, LNB, xl, v, acc);        \
  hold_acc<T>(acc);
#define DSL_OCOMMIT(MU, SGN, H, CUR, BUF, LNB)                  \
  o_commit<H, MU, SGN, ADJ, NV, S, LW>(c, CUR, BUF, LNB, xl, v, tid); \
  __syncthreads();
  DSL_OSTEP(1, 1, +1, HALF, ba, lnba)
  DSL_OCOMMIT(1, -1, HALF, r1, bb, lnbb)
  DSL_OSTEP(2, 1, -1, HALF, bb, lnbb)
  DSL_OCOMMIT(2, +1, HALF, r2, ba, lnba)
  DSL_OSTEP(3, 2, +1, HALF, ba, lnba)
  cpx<T> own[4][3];
  if (!FIRST && late) lds_spinor<S, T, NV>(bo + (xl + 1) * SSW, v, own);
  DSL_OCOMMIT(2, -1, HALF, r3, bb, lnbb)
  W* ob;
  if constexpr (FIRST) {
    DSL_OSTEP(4, 2, -1, HALF, bb, lnbb)
    if (late) lds_spinor<S, T, NV>(bo + (xl + 1) * SSW, v, own);
    DSL_OCOMMIT(3, -1, HALF, r5, ba, lnba)
    DSL_OSTEP(5, 3, -1, HALF, ba, lnba)
    DSL_OCOMMIT(3, +1, false, r4, bo + SSW, lnbb)
    DSL_ONEXT
    DSL_OSTEP(6, 3, +1, false, bo + SSW, lnbb)
    ob = HALF ? ba : bb;
  } else {
    DSL_OSTEP(4, 2, -1, HALF, bb, lnbb)
    DSL_OCOMMIT(3, +1, false, r4, bo + SSW, lnba)
    DSL_ONEXT
    DSL_OSTEP(5, 3, +1, false, bo + SSW, lnba)
    ob = ba;
  }
#undef DSL_OSTEP
#undef DSL_OCOMMIT
#undef DSL_OISSUE
#undef DSL_ONEXT
  // out = diag psi - 1/2 (hops) = -1/2 acc, through a free buffer (HALF: ba
  // and bb together, with a site stride of 12 N_v + 4 words where that fits,
  // 12 N_v otherwise)
  constexpr int OSW = HALF ? (12 * NV + 4 <= 2 * HalfStride<NV, S>::WORDS ? 12 * NV + 4 : 12 * NV) : SSW;
  constexpr int OSP = OSW * int(sizeof(W)) / 16;
  static_assert(!HALF || OSW <= 2 * HalfStride<NV, S>::WORDS, "the output fits ba and bb");
  {
    W* o = ob + xl * OSW;
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int cc = 0; cc < 3; ++cc) {
        cpx<T> r;
        r.r = T(-0.5) * acc[sp][cc].r;
        r.i = T(-0.5) * acc[sp][cc].i;
        if (late) r = rmadd(r, diag, own[sp][cc]);
        S::template store<T>(o + (sp * 3 + cc) * NV + v, r);
      }
  }
  __syncthreads();
  {
    const int xc = xl < c.n ? xl : c.n - 1;
    const u32x4* src = reinterpret_cast<const u32x4*>(ob) + xc * OSP;
    u32x4* dst = reinterpret_cast<u32x4*>(out + size_t(c.plane + c.p0 + xc) * SW);
    epi_copy_out<EPI, NV, S, CH>(src, dst, v, xl < c.n, ep);
  }
  __syncthreads();
}

// PP: 0 the one-buffer step (march_step), 1 two buffers in turn
// (march_step_pp), 2 an own-row buffer plus two in turn (march_step_o), 3 the
// same with half-spinor neighbour rows (FP32 storage).
template <int PP, int DEPTH> struct MarchOcc { static constexpr int value = PP ? 2 : MarchWaves<DEPTH>::value; };

template <int DEPTH, bool ADJ, int NV, class S, class T, int LW, int PP, int EPI, int HN, bool LATE>
__global__ void __launch_bounds__(256, (MarchOcc<PP, DEPTH>::value))
    wilson_march_kernel(Geom g, FlatMarch m, int xcd, const typename S::word* __restrict__ U,
                        const typename S::word* __restrict__ in, typename S::word* __restrict__ out, T diag,
                        EpiArgs ea) {
  using W = typename S::word;
  constexpr int CH = RowPieces<S>::CH, LK = LinkK<S, NV, LW>::value;
  constexpr int SSW = SiteStride<NV, S>::WORDS;
  extern __shared__ uint4 smem_march[];
  const int R = int(m.sb);
  W* buf = reinterpret_cast<W*>(smem_march);
  constexpr int BSW = PP == 3 ? HalfStride<NV, S>::WORDS : SSW;  // ba, bb site stride
  W* buf1 = buf + (R + HN) * SSW;  // PP 1: the second buffer; PP 2, 3: ba
  W* buf2 = buf1 + R * BSW;       // PP 2, 3: bb
  W* lown = PP == 1 ? buf1 + (R + HN) * SSW : (PP >= 2 ? buf2 + R * BSW : buf + (R + HN) * SSW);
  W* lnb = lown + (R + HN) * 4 * LW;
  W* lnb1 = lnb + R * LW;  // PP only

  const uint32_t L = xcd_block(blockIdx.x, gridDim.x, xcd != 0);
  uint32_t seg;
  FlatChunk<HN> c = flat_chunk<HN>(g, m, L, seg);
  const int steps = g.n[3] - c.t < int(m.T) ? g.n[3] - c.t : int(m.T);
  const int v = threadIdx.x, xl = threadIdx.y;
  const int tid = xl * NV + v, nth = R * NV;
  const XSlots xs = x_slots(g, c, R, xl);
  FlatChunk<HN> cn = c;  // the chunk of the next step
  if (steps > 1) {
    cn.t += 1;
    cn.plane += uint32_t(g.stride[3]);
  }

  constexpr int RN = RowRegs<NV, S, HN>::N;
  u32x4 r0[RN], r1[RN], r2[RN], r3[RN], r4[RN], r5[RN], r6[RN];
  u32x4 lr[LK + 1];
  cpx<T> carry[2][3];
  EpiLane<S> ep;
  if constexpr (EPI != EPI_STORE) ep.template init<NV>(ea, v, EPI == EPI_AXPY);
  using Q0 = typename std::conditional<PP >= 2, MarchSeqO<true>, MarchSeq<true>>::type;
#define DSL_PISSUE(P) \
  march_issue_o<PP == 3, Q0::at(P), NV, S, LW>(g, c, U, in, xl, v, tid, r0, r1, r2, r3, r4, r5, r6)
  links_issue<S, LK, LW>(c, U, tid, nth, lr);
  DSL_PISSUE(0);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (DEPTH > 1) DSL_PISSUE(1);
  if constexpr (DEPTH > 2) DSL_PISSUE(2);
  if constexpr (DEPTH > 3) DSL_PISSUE(3);
  if constexpr (DEPTH > 4) DSL_PISSUE(4);
#undef DSL_PISSUE
  if constexpr (PP >= 2)
    march_step_o<true, DEPTH, ADJ, NV, S, T, LW, PP == 3, EPI, LATE>(g, c, cn, U, in, out, buf, buf1, buf2, lown, lnb, lnb1, xs,
                                                               R, xl, v, tid, nth, diag, m.late, r0, r1, r2, r3, r4, r5,
                                                               r6, lr, carry, ep);
  else if constexpr (PP == 1)
    march_step_pp<true, DEPTH, ADJ, NV, S, T, LW, EPI>(g, c, U, in, out, buf, buf1, lown, lnb, lnb1, xs, R, xl, v,
                                                       tid, nth, diag, r0, r1, r2, r3, r4, r5, r6, lr, carry, ep);
  else
    march_step<true, DEPTH, ADJ, NV, S, T, LW, EPI>(g, c, U, in, out, buf, lown, lnb, xs, R, xl, v, tid, nth, diag,
                                                    r0, r1, r2, r3, r4, r5, r6, lr, carry, ep);
#pragma nounroll
  for (int k = 1; k < steps; ++k) {
    c = cn;
    if (k + 1 < steps) {
      cn.t += 1;
      cn.plane += uint32_t(g.stride[3]);
    }
    if constexpr (PP >= 2)
      march_step_o<false, DEPTH, ADJ, NV, S, T, LW, PP == 3, EPI, LATE>(g, c, cn, U, in, out, buf, buf1, buf2, lown, lnb, lnb1,
                                                                  xs, R, xl, v, tid, nth, diag, m.late, r0, r1, r2, r3, r4, r5,
                                                                  r6, lr, carry, ep);
    else if constexpr (PP == 1)
      march_step_pp<false, DEPTH, ADJ, NV, S, T, LW, EPI>(g, c, U, in, out, buf, buf1, lown, lnb, lnb1, xs, R, xl,
                                                          v, tid, nth, diag, r0, r1, r2, r3, r4, r5, r6, lr, carry, ep);
    else
      march_step<false, DEPTH, ADJ, NV, S, T, LW, EPI>(g, c, U, in, out, buf, lown, lnb, xs, R, xl, v, tid, nth,
                                                       diag, r0, r1, r2, r3, r4, r5, r6, lr, carry, ep);
  }
  epi_finish<EPI, NV, S>(ea, ep, reinterpret_cast<double*>(smem_march), xl, v, R);
}

// LDS bytes of a march workgroup, without the padding of its site strides.
inline size_t march_lds(int R, int nv, int wb, int pp, int hn) {
  const size_t site = size_t(12) * nv * wb;
  const size_t rows = size_t(R + hn) + (pp == 1 ? R + hn : (pp == 2 ? 2 * R : (pp == 3 ? R : 0)));
  return rows * site + size_t(R + hn) * 36 * wb + size_t(pp ? 2 : 1) * R * 9 * wb;
}

// Rows in flight of a march: three with half-spinor rows, two otherwise.
DSL_HD constexpr int march_depth(int pp) { return pp == 3 ? 3 : 2; }

// The fused epilogues are built for the solver's two forms only (D with
// EPI_NORM, D^dag with EPI_AXPY), on N_v = 12, full links and the default
// prefetch depth of each buffer scheme.
template <int PP, int DEPTH, int LW, int NV, int HN>
struct MarchEpiBuilt {
  static constexpr bool value = NV == 12 && LW == 9 && DEPTH == march_depth(PP);
};

template <int DEPTH, int NV, class S, class T, int LW, int PP, int HN>
static hipError_t march_launch(bool adj, int epi, dim3 grid, dim3 block, size_t lds, hipStream_t st, const Geom& g,
                               const FlatMarch& m, bool xcd, const void* U, const void* in,
                               void* out, T diag, const EpiArgs& ea) {
  using W = typename S::word;
#define DSL_MKL(A, E, LATE)                                                                                   \
  hipLaunchKernelGGL((wilson_march_kernel<DEPTH, A, NV, S, T, LW, PP, E, HN, LATE>), grid, block, lds, st, g, m, \
                     int(xcd), (const W*)U, (const W*)in, (W*)out, diag, ea)
// (BF16 in chunks of one x-row is never late, chunks across row ends read m.late)
#define DSL_MK(A, E)                                    \
  do {                                                  \
    if constexpr (HN == 2 && PP == 3) {                 \
      if (m.late) DSL_MKL(A, E, true); else DSL_MKL(A, E, false); \
    } else {                                            \
      DSL_MKL(A, E, false);                             \
    }                                                   \
  } while (0)
  if (epi == EPI_STORE) {
    if (adj) DSL_MK(true, EPI_STORE); else DSL_MK(false, EPI_STORE);
  } else if constexpr (MarchEpiBuilt<PP, DEPTH, LW, NV, HN>::value) {
    if (epi == EPI_NORM && !adj) DSL_MK(false, EPI_NORM);
    else if (epi == EPI_AXPY && adj) DSL_MK(true, EPI_AXPY);
    else return hipErrorNotSupported;
  } else {
    return hipErrorNotSupported;
  }
#undef DSL_MK
#undef DSL_MKL
  return hipGetLastError();
}

// kb x zb of eight tiles, the split with the smallest cost: N_x / (kb R) for the
// sites with a y neighbour outside the tile (those rows are the nearer ones in
// the order, so they count half) and 2 / zb for z; above N_v = 12 y counts 0.4.  A
// split that does not divide (the XCDs' eighths then cut tiles) costs 1.3 times.
// Rows x planes measured at N_v = 12 on 34^3 x 68: 17 x 9 2226 us, 8 x 17 2116, 7
// of 56 chunks x 34 1994; on 24^3 x 48: 12 x 6 511, 6 x 12 492, 3 x 24 519; N_v =
// 24 there: 6 x 12 1040, 3 x 24 989; N_v = 16 on 30 x 24 x 25 x 36: 6 x 13 642, 3
// x 25 608.
inline void eight_tiles(const Geom& g, FlatMarch& m) {
  const double wy = g.nv > 12 ? 0.8 : 1.0;
  double best = -1;
  for (uint32_t ty = 1; ty <= 8; ty *= 2) {
    const uint32_t tz = 8 / ty, nz = uint32_t(g.n[2]);
    const uint32_t kb = (m.chunks + ty - 1) / ty, zb = (nz + tz - 1) / tz;
    double s = (ty > 1 ? wy * g.n[0] / (double(kb) * m.sb) : 0.0) + (tz > 1 ? 2.0 / zb : 0.0);
    if (m.chunks % ty || nz % tz) s *= 1.3;
    if (best < 0 || s < best) {
      best = s;
      m.kb = kb;
      m.zb = zb;
    }
  }
}

// ONLY_PP >= 0 builds that buffer scheme only (pp must equal it).
template <int DEPTH, int NV, class S, class T, int LW, int ONLY_PP, int HN>
static hipError_t wilson_march_t(bool adj, const Geom& g, int R, int tsteps, int pp, bool late, bool xcd,
                                 const void* U, const void* in, void* out, double mass, hipStream_t st, int epi, EpiArgs& ea) {
  if (ONLY_PP >= 0 && pp != ONLY_PP) return hipErrorInvalidValue;
  using W = typename S::word;
  FlatMarch m = make_flat_march(g, uint32_t(R), uint32_t(tsteps));
  m.late = late;
  const dim3 block(NV, R), grid(m.grid);
  if (epi != EPI_STORE && grid.x > ea.capacity) return hipErrorNotSupported;
  ea.blocks = grid.x;
  size_t lds = rows_lds_words<NV, S, LW, HN>(R) * sizeof(W);
  if (pp == 1) lds += (size_t(R + HN) * SiteStride<NV, S>::WORDS + size_t(R) * LW) * sizeof(W);
  if (pp == 2) lds += (size_t(2 * R) * SiteStride<NV, S>::WORDS + size_t(R) * LW) * sizeof(W);
  if (pp == 3) lds += (size_t(2 * R) * HalfStride<NV, S>::WORDS + size_t(R) * LW) * sizeof(W);
  lds += size_t(knobs().row_lds_extra.get(0));
  const T diag = T(4) + T(mass);
  // Eight tiles of the (x, y) chunks and planes, one per XCD, when the grid runs
  // in more than one round (more than two workgroups per CU); a grid resident
  // at once keeps the plane order.  DSLASH_WMARCH_TILE_Y, _Z override (rows and
  // planes of a tile; 0: plane order).
  if (m.grid > 2u * uint32_t(device_cus())) eight_tiles(g, m);
  if (knobs().wmarch_tile_y.set || knobs().wmarch_tile_z.set)
    flat_march_tile(g, m, knobs().wmarch_tile_y.get(0), knobs().wmarch_tile_z.get(0));
  if constexpr (ONLY_PP >= 0) {
    if constexpr (ONLY_PP == 3 && !(sizeof(W) == 8 && NV % 2 == 0)) return hipErrorInvalidValue;
    else return march_launch<DEPTH, NV, S, T, LW, ONLY_PP, HN>(adj, epi, grid, block, lds, st, g, m, xcd, U, in, out, diag, ea);
  } else {
    switch (pp) {
      case 3:
        if constexpr (sizeof(W) == 8 && NV % 2 == 0)
          return march_launch<DEPTH, NV, S, T, LW, 3, HN>(adj, epi, grid, block, lds, st, g, m, xcd, U, in, out, diag, ea);
        else
          return hipErrorInvalidValue;
      case 2: return march_launch<DEPTH, NV, S, T, LW, 2, HN>(adj, epi, grid, block, lds, st, g, m, xcd, U, in, out, diag, ea);
      case 1: return march_launch<DEPTH, NV, S, T, LW, 1, HN>(adj, epi, grid, block, lds, st, g, m, xcd, U, in, out, diag, ea);
      default: return march_launch<DEPTH, NV, S, T, LW, 0, HN>(adj, epi, grid, block, lds, st, g, m, xcd, U, in, out, diag, ea);
    }
  }
}

// ---------------------------------------------------------------- even-odd hop
// out = c_add add + c_hop H in on the packed sites of parity p (even-odd form
// of D_W, see eo.hip), staged like wilson_rows_kernel on the packed geometry
// (Nx/2 sites per row): the y, z, t neighbours of packed site i sit at packed
// index i of the neighbour rows of `in`; the x neighbours are in the same row
// of `in` at i + r (x + 1) and i - 1 + r (x - 1), r = (p + y + z + t) mod 2.
// Forward links come from Uo (parity p), backward ones from Ui (parity 1 - p).
template <int DEPTH, bool ADJ, int NV, class S, class T, int EPI, int HN>
__global__ void __launch_bounds__(256, RowsWaves<DEPTH>::value)
    wilson_eo_rows_kernel(Geom g, FlatMarch m, int xcd, int p, const typename S::word* __restrict__ Uo,
                          const typename S::word* __restrict__ Ui, const typename S::word* __restrict__ in,
                          typename S::word* __restrict__ out, const typename S::word* __restrict__ add, T c_add,
                          T c_hop, EpiArgs ea) {
  using W = typename S::word;
  constexpr int SW = 12 * NV, CH = RowPieces<S>::CH;
  constexpr int SSW = SiteStride<NV, S>::WORDS, SSP = SiteStride<NV, S>::PIECES;
  extern __shared__ uint4 smem_eo[];
  const int R = int(m.sb);
  W* buf = reinterpret_cast<W*>(smem_eo);
  W* lown = buf + (R + HN) * SSW;  // [R + 4][36], slot i + 1
  W* lnb = lown + (R + HN) * 36;   // [R][9]
  W* lxb = lnb + R * 9;           // [R][9]: V_x(x - 1) from Ui

  const uint32_t L = xcd_block(blockIdx.x, gridDim.x, xcd != 0);
  uint32_t seg;
  const FlatChunk<HN> c = flat_chunk<HN>(g, m, L, seg);
  const int v = threadIdx.x, xl = threadIdx.y;
  const int tid = xl * NV + v, nth = R * NV;
  // packed row of in-plane site q: x + 1 at q + r, x - 1 at q - 1 + r (in the row)
  auto shift_r = [&](uint32_t q) { return (uint32_t(p) + g.dx.div(q) + uint32_t(c.z) + uint32_t(c.t)) & 1u; };
  XSlots xs = x_slots(g, c, R, xl);
  {
    const int i = xl < c.n ? xl : c.n - 1;
    if (shift_r(c.p0 + uint32_t(i))) xs.b = i + 1;
    else xs.f = i + 1;
  }

  constexpr int RN = RowRegs<NV, S, HN>::N;
  u32x4 r0[RN], r1[RN], r2[RN], r3[RN], r4[RN], r5[RN], r6[RN];
#define DSL_ISSUE(K)                                                                   \
  do {                                                                                 \
    if constexpr (K == 0) row_issue<1, +1, NV, S>(g, c, Ui, in, xl, v, tid, r0);       \
    if constexpr (K == 1) row_issue<1, -1, NV, S>(g, c, Ui, in, xl, v, tid, r1);       \
    if constexpr (K == 2) row_issue<2, +1, NV, S>(g, c, Ui, in, xl, v, tid, r2);       \
    if constexpr (K == 3) row_issue<2, -1, NV, S>(g, c, Ui, in, xl, v, tid, r3);       \
    if constexpr (K == 4) row_issue<3, +1, NV, S>(g, c, Ui, in, xl, v, tid, r4);       \
    if constexpr (K == 5) row_issue<3, -1, NV, S>(g, c, Ui, in, xl, v, tid, r5);       \
    if constexpr (K == 6) own_issue<NV, S>(c, in, xl, v, tid, r6);             \
  } while (0)
  // Links of the chunk's own sites (forward hops) and V_x(x - 1) of the x - 1
  // neighbours, which live in the other parity's row: committed first, so
  // requested first (loads retire in order).
  constexpr int LK = LinkK<S, NV>::value, KX = (9 + NV - 1) / NV;
  u32x4 lr[LK];
  W lx[KX];
  pieces_issue<LK>(lr, Uo + size_t(c.plane + c.p0) * 36, c.n * LinkPieces<S>::PER_SITE, tid, nth);
#pragma unroll
  for (int i = 0; i < KX; ++i) {
    const int q = tid + i * nth, w = q < c.n * 9 ? q : c.n * 9 - 1;
    const int k = w / 9, e = w - k * 9;
    const uint32_t pk = c.p0 + uint32_t(k);
    const uint32_t x = pk - g.dx.div(pk) * c.nx;
    const uint32_t q1 = shift_r(pk) ? pk : (x > 0 ? pk - 1 : pk + c.nx - 1);
    lx[i] = Ui[size_t(c.plane + q1) * 36 + e];
  }
  __builtin_amdgcn_sched_barrier(0);
  DSL_ISSUE(0);
  if constexpr (DEPTH > 1) DSL_ISSUE(1);
  if constexpr (DEPTH > 2) DSL_ISSUE(2);
  if constexpr (DEPTH > 3) DSL_ISSUE(3);
  if constexpr (DEPTH > 4) DSL_ISSUE(4);
  if constexpr (DEPTH > 5) DSL_ISSUE(5);
  if constexpr (DEPTH > 6) DSL_ISSUE(6);
  pieces_commit<LK>(lr, lown + 36, c.n * LinkPieces<S>::PER_SITE, tid, nth);
#pragma unroll
  for (int i = 0; i < KX; ++i) {
    const int q = tid + i * nth;
    lxb[q < c.n * 9 ? q : c.n * 9 - 1] = lx[i];
  }

  cpx<T> acc[4][3];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) acc[a][b] = zero<T>();

  W* const row = buf + SSW;
#define DSL_ROW_STEP(K, MU, SGN, CUR)                                         \
  row_commit<SGN, NV, S>(c, CUR, row, lnb, xl, v, tid);                       \
  __syncthreads();                                                            \
  if constexpr (K + DEPTH < 7) DSL_ISSUE(K + DEPTH);                          \
  row_compute<MU, SGN, ADJ, NV, S, T>(row, lown, lnb, xl, v, acc);            \
  hold_acc<T>(acc);                                                           \
  __syncthreads();
  DSL_ROW_STEP(0, 1, +1, r0)
  DSL_ROW_STEP(1, 1, -1, r1)
  DSL_ROW_STEP(2, 2, +1, r2)
  DSL_ROW_STEP(3, 2, -1, r3)
  DSL_ROW_STEP(4, 3, +1, r4)
  DSL_ROW_STEP(5, 3, -1, r5)
#undef DSL_ROW_STEP
#undef DSL_ISSUE

  own_commit<NV, S>(c, r6, buf, xl, v, tid, R);
  __syncthreads();
  cpx<T> res[4][3];
  {
    constexpr int CF = ADJ ? +1 : -1, CB = -CF;
    lds_hop<0, CF, false, NV, S, T>(buf + xs.f * SSW, lown + (xl + 1) * 36, v, acc);
    lds_hop<0, CB, true, NV, S, T>(buf + xs.b * SSW, lxb + xl * 9, v, acc);
    const T ch = T(-0.5) * c_hop;
    const int xc = xl < c.n ? xl : c.n - 1;
    const W* a = add + size_t(c.plane + c.p0 + xc) * SW + v;
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int cc = 0; cc < 3; ++cc) {
        res[sp][cc].r = ch * acc[sp][cc].r;
        res[sp][cc].i = ch * acc[sp][cc].i;
        if (add) {
          const cpx<T> q = S::template load<T>(a + (sp * 3 + cc) * NV);
          res[sp][cc].r = fma(c_add, q.r, res[sp][cc].r);
          res[sp][cc].i = fma(c_add, q.i, res[sp][cc].i);
        }
      }
  }
  __syncthreads();
  {
    W* o = buf + xl * SSW;
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int cc = 0; cc < 3; ++cc) S::template store<T>(o + (sp * 3 + cc) * NV + v, res[sp][cc]);
  }
  __syncthreads();
  {
    const int xc = xl < c.n ? xl : c.n - 1;
    const u32x4* src = reinterpret_cast<const u32x4*>(buf) + xc * SSP;
    u32x4* dst = reinterpret_cast<u32x4*>(out + size_t(c.plane + c.p0 + xc) * SW);
    EpiLane<S> ep;
    if constexpr (EPI != EPI_STORE) ep.template init<NV>(ea, v, EPI == EPI_AXPY);
    epi_copy_out<EPI, NV, S, CH>(src, dst, v, xl < c.n, ep);
    epi_finish<EPI, NV, S>(ea, ep, reinterpret_cast<double*>(smem_eo), xl, v, R);
  }
}

// Order of the one-row D_W kernels: tiles of rows whose spinors at one t take at
// most 1.25 MB, t inside a tile, of those the one with the smallest surface, which counts
// 1.5 times where the tiles do not divide the lattice (the XCDs' eighths then cut them:
// even-odd hop in C64, 32^4, N_v = 4, 204 us in tiles of 14 x 14 rows, 193 of 8 x 16; 24^3 x 48,
// N_v = 12 294 and 272).  DSLASH_ROWS_TILE_Y, _Z override (0: t-planes in turn).
inline FlatMarch one_row_order(const Geom& g, int R, long site_bytes) {
  FlatMarch m = make_flat_march(g, uint32_t(R), 1u);
  double best = -1;
  uint32_t kb = 1, zb = 1;
  for (uint32_t z = 1; z <= uint32_t(g.n[2]); ++z) {
    uint32_t k = uint32_t(1280L * 1024 / (long(z) * R * site_bytes));  // the most chunks have the smallest surface
    if (k > m.chunks) k = m.chunks;
    if (k < 1 && z > 1) break;
    if (k < 1) k = 1;
    // the most chunks, and the most that divide the plane
    for (uint32_t d = k;; --d) {
      const bool divides = m.chunks % d == 0 && uint32_t(g.n[2]) % z == 0;
      if (d < k && !divides) {
        if (d == 1) break;
        continue;
      }
      double s = (d < m.chunks ? 2.0 * g.n[0] / (double(d) * R) : 0.0) + (z < uint32_t(g.n[2]) ? 2.0 / z : 0.0);
      if (!divides) s *= 1.5;
      if (best < 0 || s < best) {
        best = s;
        kb = d;
        zb = z;
      }
      if (divides || d == 1) break;
    }
  }
  m.kb = kb;
  m.zb = zb;
  if (knobs().rows_tile_y.set || knobs().rows_tile_z.set)
    flat_march_tile(g, m, knobs().rows_tile_y.get(0), knobs().rows_tile_z.get(0));
  return m;
}

template <int NV, class S, class T, int HN>
static hipError_t wilson_eo_rows_t(bool adj, const Geom& g, int R, bool xcd, int parity, const void* Uo,
                                   const void* Ui, const void* in, void* out, const void* add, double c_add,
                                   double c_hop, hipStream_t st, int epi, EpiArgs& ea) {
  using W = typename S::word;
  const FlatMarch m = one_row_order(g, R, 12L * NV * long(sizeof(W)));
  const dim3 block(NV, R), grid(m.grid);
  if (epi != EPI_STORE && grid.x > ea.capacity) return hipErrorNotSupported;
  ea.blocks = grid.x;
  const size_t lds = (rows_lds_words<NV, S, 9, HN>(R) + size_t(R) * 9) * sizeof(W);
#define DSL_EK(A, E)                                                                                          \
  hipLaunchKernelGGL((wilson_eo_rows_kernel<3, A, NV, S, T, E, HN>), grid, block, lds, st, g, m, int(xcd), parity, \
                     (const W*)Uo, (const W*)Ui, (const W*)in, (W*)out, (const W*)add, T(c_add), T(c_hop), ea)
  // fused epilogues: the Schur operator M with EPI_NORM, M^dag with EPI_AXPY
  if (epi == EPI_STORE) {
    if (adj) DSL_EK(true, EPI_STORE); else DSL_EK(false, EPI_STORE);
  } else if (epi == EPI_NORM && !adj) {
    DSL_EK(false, EPI_NORM);
  } else if (epi == EPI_AXPY && adj) {
    DSL_EK(true, EPI_AXPY);
  } else {
    return hipErrorNotSupported;
  }
#undef DSL_EK
  return hipGetLastError();
}

template <int DEPTH, int NV, class S, class T, int HN>
static hipError_t wilson_rows_t(bool adj, const Geom& g, int R, bool xcd, const void* U, const void* in,
                                void* out, const void* C, double mass, hipStream_t st) {
  using W = typename S::word;
  const FlatMarch m = one_row_order(g, R, 12L * NV * long(sizeof(W)));
  const dim3 block(NV, R), grid(m.grid);
  size_t lds = (rows_lds_words<NV, S, 9, HN>(R) + (C ? 3 + size_t(R) * 36 : 0)) * sizeof(W);
  // DSLASH_ROW_LDS_EXTRA (bytes) lowers the workgroups per CU (tuning).
  lds += size_t(knobs().row_lds_extra.get(0));
  const T diag = T(4) + T(mass);
#define DSL_RK(A, CL)                                                                                      \
  hipLaunchKernelGGL((wilson_rows_kernel<DEPTH, A, CL, NV, S, T, HN>), grid, block, lds, st, g, m, int(xcd), (const W*)U, \
                     (const W*)in, (W*)out, (const W*)C, diag)
  if (C) {
    if (adj) DSL_RK(true, true); else DSL_RK(false, true);
  } else {
    if (adj) DSL_RK(true, false); else DSL_RK(false, false);
  }
#undef DSL_RK
  return hipGetLastError();
}


// ---------------------------------------------------------------- dispatch
// One launch of this family, as launch_wilson_rows and launch_wilson_eo_rows
// (apply_rows.hip) chose it; each storage is compiled in a file of its own.
struct RowsCall {
  bool eo;                 // the even-odd hop, else D_W on the full lattice
  bool adj;
  const Geom* g;           // (eo: the packed geometry)
  int R, hn;               // sites per chunk, halo sites (2 or 4)
  int tsteps, pp, depth;   // march; tsteps = 0: one output row per workgroup
  bool late;               // march: the diagonal term last
  bool xcd;
  const void *U, *Ub;      // links (eo: of the output and of the input parity)
  const void *in, *add, *clover;
  void* out;
  bool compressed;
  int parity;              // eo
  double mass, c_add, c_hop;
  hipStream_t st;
  int epi;
  EpiArgs* ea;
};

template <int DEPTH, int NV, class S, int LW, int ONLY_PP, int HN>
static hipError_t march_call(const RowsCall& c) {
  return wilson_march_t<DEPTH, NV, S, float, LW, ONLY_PP, HN>(c.adj, *c.g, c.R, c.tsteps, c.pp, c.late, c.xcd, c.U, c.in,
                                                              c.out, c.mass, c.st, c.epi, *c.ea);
}

// N_v = 12: every buffer scheme and depth that the tuning variables reach for
// chunks across row ends, the default ones for chunks of one x-row.
template <class S, int DPP, int HN>
static hipError_t rows_nv12(const RowsCall& c) {
  if (c.eo)
    return wilson_eo_rows_t<12, S, float, HN>(c.adj, *c.g, c.R, c.xcd, c.parity, c.U, c.Ub, c.in, c.out, c.add, c.c_add,
                                              c.c_hop, c.st, c.epi, *c.ea);
  if (c.tsteps > 0 && !c.clover) {
    constexpr int PP6 = sizeof(typename S::word) == 8 ? 3 : 0;  // compressed links
    if constexpr (HN == 2) {
      if (c.compressed) return march_call<march_depth(PP6), 12, S, 6, PP6, 2>(c);
      return march_call<march_depth(DPP), 12, S, 9, DPP, 2>(c);
    } else if (c.compressed) {
      return c.depth <= 2 ? march_call<2, 12, S, 6, -1, 4>(c) : march_call<3, 12, S, 6, -1, 4>(c);
    } else {
      return c.depth <= 2 ? march_call<2, 12, S, 9, -1, 4>(c) : march_call<3, 12, S, 9, -1, 4>(c);
    }
  }
  // one output row per workgroup: chunks across row ends only
  if constexpr (HN == 4) {
#define DSL_RC(D)                                                                                                  \
  return wilson_rows_t<D, 12, S, float, HN>(c.adj, *c.g, c.R, c.xcd, c.U, c.in, c.out, c.clover, c.mass, c.st)
    if (c.depth <= 2) DSL_RC(2);
    if (c.depth <= 3) DSL_RC(3);
    DSL_RC(7);
#undef DSL_RC
  }
  return hipErrorNotSupported;
}

// Other block sizes: the march in the default buffer scheme, and the even-odd hop.
template <class S, int NV, int PP, int HN>
static hipError_t rows_nv(const RowsCall& c) {
  if (c.eo)
    return wilson_eo_rows_t<NV, S, float, HN>(c.adj, *c.g, c.R, c.xcd, c.parity, c.U, c.Ub, c.in, c.out, c.add, c.c_add,
                                              c.c_hop, c.st, c.epi, *c.ea);
  return march_call<march_depth(PP), NV, S, 9, PP, HN>(c);
}

// Storage S, whose default buffer scheme is PP.
template <class S, int PP>
static hipError_t rows_dispatch(const RowsCall& c) {
  const bool h2 = c.hn == 2;
  switch (c.g->nv) {
    case 4: return h2 ? rows_nv<S, 4, PP, 2>(c) : rows_nv<S, 4, PP, 4>(c);
    case 8: return h2 ? rows_nv<S, 8, PP, 2>(c) : rows_nv<S, 8, PP, 4>(c);
    case 12: return h2 ? rows_nv12<S, PP, 2>(c) : rows_nv12<S, PP, 4>(c);
    case 16: return h2 ? rows_nv<S, 16, PP, 2>(c) : rows_nv<S, 16, PP, 4>(c);
    case 24: return h2 ? rows_nv<S, 24, PP, 2>(c) : rows_nv<S, 24, PP, 4>(c);
  }
  return hipErrorNotSupported;
}

hipError_t wilson_rows_c64(const RowsCall& c);
hipError_t wilson_rows_bf16(const RowsCall& c);
hipError_t wilson_rows_f16(const RowsCall& c);
// C64 at the other N_v from 2 to 23, D_W on the full lattice only
hipError_t wilson_rows_c64_any(const RowsCall& c);

}  // namespace dsl
