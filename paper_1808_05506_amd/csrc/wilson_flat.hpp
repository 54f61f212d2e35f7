// Flat D_W kernels: any lattice, any N_v, any storage, also with the clover term or
// compressed links (wilson_flat.hip, wilson_flat16.hip instantiate them).  The
// row-staged kernels (wilson_rows.hpp) have FP32 arithmetic and block sizes and
// chunks that fill their workgroups; these take what is left, but for the calls that
// the direct kernel is faster at (launch_wilson_flat).
//
// A workgroup owns P consecutive sites of an (x, y) plane at one (z, t), across
// row ends, and all N_v right-hand sides: lane (site, group) holds VW columns,
// so that it moves 16 bytes a load where N_v and the alignment allow (C64: two
// columns, C128: one).  Every lane of a wave is used whatever N_x is.  The 72
// words of links a site needs (its four and the four behind it) are staged in
// LDS once, with one coalesced pass; the spinors go straight to registers.
//
// What bounds it: the vector-memory path (short runs per site and component),
// then L2 misses.  A hop loads two halves of six pieces; two or three halves are
// in flight per lane (the register constraints between the halves keep the
// compiler from hoisting all sixteen, which spilled 140 to 490 registers).  L2
// hits are cheap (30 TB/s measured for these access patterns, 9 TB/s from the
// Infinity Cache), so the order of the workgroups decides: tiles of planes x
// chunks, t sweeping inside a tile, each XCD a contiguous eighth of that order
// (flat_shape).  FP64, N_v = 12, 24^3 x 48: 1050 us, 3.3 TB/s algorithmic (1906
// with links and spinors loaded by each lane in (site, column) order).
#pragma once

#include "flat_order.hpp"
#include "stencils.hpp"

namespace dsl {

template <int BYTES> struct FlatPiece;
template <> struct FlatPiece<16> { typedef u32x4 type; };
template <> struct FlatPiece<8> { typedef u32x2 type; };
template <> struct FlatPiece<4> { typedef unsigned int type; };

// VW storage words (one complex number of VW consecutive columns) as one load.
template <class S, int VW>
struct FlatVec {
  using W = typename S::word;
  using V = typename FlatPiece<VW * int(sizeof(W))>::type;
  template <class T>
  static __device__ __forceinline__ void unpack(V z, cpx<T> (&o)[VW]) {
    if constexpr (sizeof(V) == sizeof(W)) {
      W w;
      if constexpr (sizeof(W) == 4) w = z; else w = __builtin_bit_cast(W, z);
      o[0] = S::template load<T>(&w);
    } else if constexpr (sizeof(W) == 8) {
      const f32x4 f = __builtin_bit_cast(f32x4, z);
      o[0] = {f.x, f.y};
      o[1] = {f.z, f.w};
    } else {
      static_assert(__is_same(W, uint32_t), "4-byte storage words are uint32_t");
#pragma unroll
      for (int k = 0; k < VW; ++k) {
        const uint32_t w = z[k];
        o[k] = S::template load<T>(&w);
      }
    }
  }
  template <class T>
  static __device__ __forceinline__ V pack(const cpx<T> (&o)[VW]) {
    W w[VW];
#pragma unroll
    for (int k = 0; k < VW; ++k) S::template store<T>(&w[k], o[k]);
    if constexpr (VW == 1) {
      if constexpr (sizeof(W) == 4) return w[0]; else return __builtin_bit_cast(V, w[0]);
    } else if constexpr (sizeof(W) == 8) {
      return __builtin_bit_cast(V, f32x4{w[0].x, w[0].y, w[1].x, w[1].y});
    } else if constexpr (VW == 2) {
      return V{w[0], w[1]};
    } else {
      return V{w[0], w[1], w[2], w[3]};
    }
  }
};

template <class T>
__device__ __forceinline__ void flat_hold(cpx<T>& z) {
  asm volatile("" : "+v"(z.r), "+v"(z.i));
}

// Half hop H = 0 .. 15: the hops -t, -z, -y, -x, +x, +y, +z, +t, and of each
// the half-spin components 0 and 1 of its projection (1 +- gamma_mu) psi.
template <int H>
struct FlatHalf {
  static constexpr int HOP = H / 2, SP = H % 2;
  static constexpr bool BWD = HOP < 4;
  static constexpr int MU = BWD ? 3 - HOP : HOP - 4;
  static constexpr int PARTNER = SP ? (MU <= 1 ? 2 : 3) : (MU <= 1 ? 3 : 2);  // spin that joins spin SP
};

// The six pieces of a half hop: spin SP and its partner in three colours, at
// byte `voff` of the plane (32 bits: a plane of sites is below 4 GB).
template <int H, class S, int VW>
__device__ __forceinline__ void flat_load(const typename S::word* __restrict__ plane, uint32_t voff, int nv,
                                          typename FlatVec<S, VW>::V (&raw)[6]) {
  using V = typename FlatVec<S, VW>::V;
  using F = FlatHalf<H>;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    raw[c] = *reinterpret_cast<const V*>(reinterpret_cast<const char*>(plane + (F::SP * 3 + c) * nv) + voff);
    raw[3 + c] = *reinterpret_cast<const V*>(reinterpret_cast<const char*>(plane + (F::PARTNER * 3 + c) * nv) + voff);
  }
}

// acc += the half hop's share: h = psi_s + (phase) psi_partner (project in
// stencils.hpp), t = U h or U^dag h, then its two spin components (reconstruct_add).
template <int H, bool ADJ, class S, class T, int VW>
__device__ __forceinline__ void flat_half(const typename FlatVec<S, VW>::V (&raw)[6], const cpx<T> (&u)[3][3],
                                          cpx<T> (&acc)[VW][4][3]) {
  using F = FlatHalf<H>;
  constexpr int MU = F::MU, s = F::SP;
  constexpr int CF = ADJ ? +1 : -1, C = F::BWD ? -CF : CF;
  cpx<T> h[VW][3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    cpx<T> a[VW], b[VW];
    FlatVec<S, VW>::template unpack<T>(raw[c], a);
    FlatVec<S, VW>::template unpack<T>(raw[3 + c], b);
#pragma unroll
    for (int k = 0; k < VW; ++k) {
      if constexpr (MU == 0) h[k][c] = a[k] - ci<C>(b[k]);
      else if constexpr (MU == 1) h[k][c] = s ? a[k] + cs<C>(b[k]) : a[k] - cs<C>(b[k]);
      else if constexpr (MU == 2) h[k][c] = s ? a[k] + ci<C>(b[k]) : a[k] - ci<C>(b[k]);
      else h[k][c] = a[k] + cs<C>(b[k]);
    }
  }
#pragma unroll
  for (int k = 0; k < VW; ++k)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cpx<T> r = zero<T>();
#pragma unroll
      for (int b = 0; b < 3; ++b) r = F::BWD ? cjmadd(r, u[b][a], h[k][b]) : cmadd(r, u[a][b], h[k][b]);
      acc[k][s][a] += r;
      if constexpr (MU == 0) acc[k][3 - s][a] += ci<C>(r);
      else if constexpr (MU == 1 && s == 0) acc[k][3][a] -= cs<C>(r);
      else if constexpr (MU == 1) acc[k][2][a] += cs<C>(r);
      else if constexpr (MU == 2 && s == 0) acc[k][2][a] += ci<C>(r);
      else if constexpr (MU == 2) acc[k][3][a] -= ci<C>(r);
      else acc[k][2 + s][a] += cs<C>(r);
    }
}

// Half hops in flight, and the waves per SIMD whose registers they fit in: three at one
// column a lane in FP32 arithmetic (69 to 85 VGPRs), two elsewhere (C64, two columns, 128,
// 135 with the clover term; FP64 112 to 136; four columns of 16 bits 179 to 238).
template <class S, int VW>
struct FlatDepth {
  static constexpr int LANE = VW * int(sizeof(typename S::real));
  static constexpr int value = LANE >= 8 ? 2 : 3;
  static constexpr int waves = VW >= 4 ? 2 : (LANE >= 8 ? 3 : 4);
};

// out = diag in - 1/2 sum_mu [(1 - gamma_mu) V_mu(x) in(x+mu) + (1 + gamma_mu) V_mu(x-mu)^dag in(x-mu)]
// (+ C(x) in(x) with the clover term), diag = 4 + m0.
template <bool ADJ, bool CLOV, int LW, class S, class T, int VW, int NVC>
__global__ void __launch_bounds__(256, (FlatDepth<S, VW>::waves))
    wilson_flat_kernel(Geom g, FlatOrder o, int xcd, const typename S::word* __restrict__ U,
                       const typename S::word* __restrict__ in, typename S::word* __restrict__ out,
                       const typename S::word* __restrict__ Cl, T diag) {
  using W = typename S::word;
  using V = typename FlatVec<S, VW>::V;
  constexpr int D = FlatDepth<S, VW>::value;
  extern __shared__ uint4 smem_flat[];
  const int P = int(o.P), nv = NVC ? NVC : g.nv;
  W* const lf = reinterpret_cast<W*>(smem_flat);  // [P][4][LW] links of the chunk's sites
  W* const lb = lf + P * 4 * LW;                  // [P][4][LW] V_mu(x - mu)
  W* const lc = lb + P * 4 * LW;                  // [P][36] clover words (CLOV)

  const FlatSite fs = flat_site(g, o, xcd_block(blockIdx.x, gridDim.x, xcd != 0));
  const int z = fs.z, t = fs.t, n = int(fs.n);
  const uint32_t Nx = uint32_t(g.n[0]), Nxy = Nx * uint32_t(g.n[1]), Nz = uint32_t(g.n[2]);
  const uint32_t zp = z + 1 == g.n[2] ? 0u : uint32_t(z + 1), zm = z == 0 ? Nz - 1 : uint32_t(z - 1);
  const uint32_t tp = t + 1 == g.n[3] ? 0u : uint32_t(t + 1), tm = t == 0 ? uint32_t(g.n[3]) - 1 : uint32_t(t - 1);
  const uint32_t plane = Nxy * (uint32_t(z) + Nz * uint32_t(t));
  const uint32_t pl_zp = Nxy * (zp + Nz * uint32_t(t)), pl_zm = Nxy * (zm + Nz * uint32_t(t));
  const uint32_t pl_tp = Nxy * (uint32_t(z) + Nz * tp), pl_tm = Nxy * (uint32_t(z) + Nz * tm);
  const int tid = int(threadIdx.x), nth = int(blockDim.x);

  // in-plane index of the x - 1 neighbour of in-plane site p
  auto x_minus = [&](uint32_t p) -> uint32_t {
    const uint32_t x = p - g.dx.div(p) * Nx;
    return x == 0 ? p + Nx - 1 : p - 1;
  };

  // This lane's site and neighbours; lanes past the chunk's end repeat its last site.
  // (blockIdx.y: blocks of column groups, where a site's do not fit one workgroup)
  const int G = nv / VW, GB = int(o.groups.d);
  const int i = int(o.groups.div(uint32_t(tid)));
  int gq = int(blockIdx.y) * GB + (tid - i * GB);
  const bool live = i < n && gq < G;
  const int ic = i < n ? i : n - 1;
  gq = gq < G ? gq : G - 1;
  const uint32_t p = fs.p0 + uint32_t(ic);
  const uint32_t x = p - g.dx.div(p) * Nx;
  const uint32_t p_xm = x_minus(p), p_xp = x + 1 == Nx ? p + 1 - Nx : p + 1;
  const uint32_t p_yp = p + Nx < Nxy ? p + Nx : p + Nx - Nxy, p_ym = p >= Nx ? p - Nx : p + Nxy - Nx;
  const uint32_t sb = 12u * uint32_t(nv) * uint32_t(sizeof(W)), vb = uint32_t(gq * VW) * uint32_t(sizeof(W));
  const size_t sw = size_t(12) * size_t(nv);
  const uint32_t v_p = p * sb + vb, v_xm = p_xm * sb + vb, v_xp = p_xp * sb + vb, v_ym = p_ym * sb + vb,
                 v_yp = p_yp * sb + vb;
  const W* const in_tm = in + sw * pl_tm;
  const W* const in_zm = in + sw * pl_zm;
  const W* const in_p = in + sw * plane;
  const W* const in_zp = in + sw * pl_zp;
  const W* const in_tp = in + sw * pl_tp;

  V raw[D][6];
  cpx<T> u[3][3];
  cpx<T> acc[VW][4][3];
#pragma unroll
  for (int k = 0; k < VW; ++k)
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) acc[k][a][b] = zero<T>();

  // half hop H into slot H % D; the constraint on the offset keeps the load here
#define DSL_FL(H)                                                                                                 \
  if constexpr ((H) < 16) {                                                                                       \
    constexpr int Hc = (H) < 16 ? (H) : 0, HOP = FlatHalf<Hc>::HOP;                                               \
    uint32_t vo = HOP == 2 ? v_ym : HOP == 3 ? v_xm : HOP == 4 ? v_xp : HOP == 5 ? v_yp : v_p;                     \
    asm volatile("" : "+v"(vo));                                                                                  \
    flat_load<Hc, S, VW>(HOP == 0 ? in_tm : HOP == 1 ? in_zm : HOP == 6 ? in_zp : HOP == 7 ? in_tp : in_p, vo, nv, \
                         raw[Hc % D]);                                                                            \
  }
  {
    // four words in flight a thread and pass; indices past the end repeat the last word
    const int words = n * 4 * LW, last = words - 1;
    const W* const uf = U + size_t(plane + fs.p0) * 4 * LW;
#pragma nounroll
    for (int q0 = tid; q0 < words; q0 += 4 * nth) {
      W a[4], b[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int q = q0 + j * nth < words ? q0 + j * nth : last;
        const int k = q / (4 * LW), e = q - k * 4 * LW, mu = e / LW;
        const uint32_t pk = fs.p0 + uint32_t(k);
        const uint32_t sn = mu == 0 ? plane + x_minus(pk)
                                    : mu == 1 ? plane + (pk >= Nx ? pk - Nx : pk + Nxy - Nx) : (mu == 2 ? pl_zm : pl_tm) + pk;
        a[j] = uf[q];
        b[j] = U[size_t(sn) * 4 * LW + e];
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int q = q0 + j * nth < words ? q0 + j * nth : last;
        lf[q] = a[j];
        lb[q] = b[j];
      }
    }
    if constexpr (CLOV) {
      const W* const cw = Cl + size_t(plane + fs.p0) * 36;
      for (int q = tid; q < n * 36; q += nth) lc[q] = cw[q];
    }
  }
  DSL_FL(0)
  if constexpr (D > 1) { DSL_FL(1) }
  if constexpr (D > 2) { DSL_FL(2) }
  __syncthreads();
  const W* const wf = lf + ic * 4 * LW;
  const W* const wb = lb + ic * 4 * LW;
#define DSL_FH(H)                                                                                      \
  {                                                                                                    \
    if constexpr ((H) % 2 == 0) load_link_lw<LW, S, T>((H) < 8 ? wb + (3 - (H) / 2) * LW : wf + ((H) / 2 - 4) * LW, u); \
    flat_half<H, ADJ, S, T, VW>(raw[(H) % D], u, acc);                                                 \
    _Pragma("unroll") for (int k = 0; k < VW; ++k) _Pragma("unroll") for (int a = 0; a < 4; ++a)       \
        _Pragma("unroll") for (int b = 0; b < 3; ++b) flat_hold(acc[k][a][b]);                         \
    DSL_FL((H) + D)                                                                                    \
  }
  DSL_FH(0) DSL_FH(1) DSL_FH(2) DSL_FH(3) DSL_FH(4) DSL_FH(5) DSL_FH(6) DSL_FH(7)
  DSL_FH(8) DSL_FH(9) DSL_FH(10) DSL_FH(11) DSL_FH(12) DSL_FH(13) DSL_FH(14) DSL_FH(15)
#undef DSL_FH
#undef DSL_FL

  const size_t own = sw * plane;
  char* const op = reinterpret_cast<char*>(out + own) + v_p;
  const char* const ap = reinterpret_cast<const char*>(in_p) + v_p;
  const T hop = T(-0.5);
  const size_t cb = size_t(nv) * sizeof(W);
  if constexpr (CLOV) {
    cpx<T> q[VW][4][3];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        cpx<T> f[VW];
        FlatVec<S, VW>::template unpack<T>(*reinterpret_cast<const V*>(ap + size_t(a * 3 + b) * cb), f);
#pragma unroll
        for (int k = 0; k < VW; ++k) {
          q[k][a][b] = f[k];
          acc[k][a][b].r = fma(diag, f[k].r, hop * acc[k][a][b].r);
          acc[k][a][b].i = fma(diag, f[k].i, hop * acc[k][a][b].i);
        }
      }
#pragma unroll
    for (int k = 0; k < VW; ++k) clover_madd<S, T>(lc + ic * 36, q[k], acc[k]);
    if (live) {
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          cpx<T> f[VW];
#pragma unroll
          for (int k = 0; k < VW; ++k) f[k] = acc[k][a][b];
          *reinterpret_cast<V*>(op + size_t(a * 3 + b) * cb) = FlatVec<S, VW>::template pack<T>(f);
        }
    }
  } else {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const size_t cbo = size_t(a * 3 + b) * cb;
        cpx<T> f[VW];
        FlatVec<S, VW>::template unpack<T>(*reinterpret_cast<const V*>(ap + cbo), f);
#pragma unroll
        for (int k = 0; k < VW; ++k)
          f[k] = {fma(diag, f[k].r, hop * acc[k][a][b].r), fma(diag, f[k].i, hop * acc[k][a][b].i)};
        if (live) *reinterpret_cast<V*>(op + cbo) = FlatVec<S, VW>::template pack<T>(f);
      }
  }
}

struct FlatArgs {
  const void *U, *in, *clover;
  void* out;
  double mass;
};

template <bool ADJ, bool CLOV, int LW, class S, class T, int VW, int NVC>
static hipError_t flat_launch(const Geom& g, const FlatArgs& a, hipStream_t st) {
  using W = typename S::word;
  const FlatShape s = flat_shape(g, 12, int(sizeof(W)), VW, LW, CLOV);
  if (!grid_fits(s.grid, s.block)) return hipErrorNotSupported;
  hipLaunchKernelGGL((wilson_flat_kernel<ADJ, CLOV, LW, S, T, VW, NVC>), s.grid, s.block, s.lds, st, g, s.o,
                     knobs().xcd.get(1), (const W*)a.U, (const W*)a.in, (W*)a.out, (const W*)a.clover, T(4.0 + a.mass));
  return hipGetLastError();
}

// The forms of one (storage, columns per lane): plain, with the clover term and, but
// for one FP32 column a lane (the direct kernel's), with compressed links.
template <class S, class T, int VW, int NVC = 0>
static hipError_t flat_forms(bool adj, const Geom& g, const FlatArgs& a, bool compressed, hipStream_t st) {
  if (a.clover)
    return adj ? flat_launch<true, true, 9, S, T, VW, NVC>(g, a, st) : flat_launch<false, true, 9, S, T, VW, NVC>(g, a, st);
  if (compressed) {
    if constexpr (VW > 1 || sizeof(T) == 8)
      return adj ? flat_launch<true, false, 6, S, T, VW, NVC>(g, a, st)
                 : flat_launch<false, false, 6, S, T, VW, NVC>(g, a, st);
    else
      return hipErrorNotSupported;
  }
  return adj ? flat_launch<true, false, 9, S, T, VW, NVC>(g, a, st) : flat_launch<false, false, 9, S, T, VW, NVC>(g, a, st);
}

// 16-bit storage.
template <class S>
static hipError_t flat_forms16(int vw, bool adj, const Geom& g, const FlatArgs& a, bool compressed, hipStream_t st) {
  switch (vw) {
    case 4: return flat_forms<S, float, 4>(adj, g, a, compressed, st);
    case 2: return flat_forms<S, float, 2>(adj, g, a, compressed, st);
  }
  return flat_forms<S, float, 1>(adj, g, a, compressed, st);
}

// BF16 and F16 storage (wilson_flat16.hip).
hipError_t launch_wilson_flat16(int dtype, int vw, bool adj, const Geom& g, const FlatArgs& a, bool compressed,
                                hipStream_t st);

}  // namespace dsl
