// Flat D_S kernel: any lattice, N_v, storage and alignment, full or compressed
// links, in the order of wilson_flat.hpp and with its links staged in LDS.  A lane
// has VW columns of one site and loads each neighbour's three colours itself.
//
// What bounds it: the short runs of its loads (N_v words a site and colour), most
// of them L2 hits; the order of the tiles moves it by a few percent only.  So the
// lanes stay filled (chunks across row ends, wide pieces), which is what the
// row-staged kernel lacks where its chunks do not divide an x-row: N_v = 12,
// 18x14x20x26 C64 42 us (69 before), 34^4 406 (488); 22x18x20x16 FP64 71 (80);
// 32^4 BF16 206 (269), FP16 200 (275); N_v = 7, 32^4 C64 269 (434), 22x18x20x16
// FP64 54 (107).  Where they do, 32^4 C64 takes 284 us by rows, 300 here.
#include "flat_rule.hpp"
#include "wilson_flat.hpp"

namespace dsl {

namespace {

// Hop H = 0 .. 7: -t, -z, -y, -x, +x, +y, +z, +t.
template <int H>
struct StagHop {
  static constexpr bool BWD = H < 4;
  static constexpr int MU = BWD ? 3 - H : H - 4;
};

// Hops in flight: six where a piece is two FP32 columns or one of FP64, four
// elsewhere (32^4, N_v = 12: C64 300 us, 316 with four, 305 with eight; BF16,
// four columns a lane, 206 with four, 241 with six).
template <class S, int VW>
struct StagDepth {
  static constexpr int value = VW * int(sizeof(typename S::real)) == 8 && sizeof(typename S::word) >= 8 ? 6 : 4;
};

template <bool ADJ, int LW, class S, class T, int VW, int NVC>
__global__ void __launch_bounds__(256, 4)
    staggered_flat_kernel(Geom g, FlatOrder o, int xcd, const typename S::word* __restrict__ U,
                          const typename S::word* __restrict__ in, typename S::word* __restrict__ out, T mass) {
  using W = typename S::word;
  using V = typename FlatVec<S, VW>::V;
  constexpr int D = StagDepth<S, VW>::value;
  extern __shared__ uint4 smem_sflat[];
  const int P = int(o.P), nv = NVC ? NVC : g.nv;
  W* const lf = reinterpret_cast<W*>(smem_sflat);  // [P][4][LW] links of the chunk's sites
  W* const lb = lf + P * 4 * LW;                   // [P][4][LW] V_mu(x - mu)

  const FlatSite fs = flat_site(g, o, xcd_block(blockIdx.x, gridDim.x, xcd != 0));
  const int z = fs.z, t = fs.t, n = int(fs.n);
  const uint32_t Nx = uint32_t(g.n[0]), Nxy = Nx * uint32_t(g.n[1]), Nz = uint32_t(g.n[2]);
  const uint32_t zp = z + 1 == g.n[2] ? 0u : uint32_t(z + 1), zm = z == 0 ? Nz - 1 : uint32_t(z - 1);
  const uint32_t tp = t + 1 == g.n[3] ? 0u : uint32_t(t + 1), tm = t == 0 ? uint32_t(g.n[3]) - 1 : uint32_t(t - 1);
  const uint32_t plane = Nxy * (uint32_t(z) + Nz * uint32_t(t));
  const uint32_t pl_zp = Nxy * (zp + Nz * uint32_t(t)), pl_zm = Nxy * (zm + Nz * uint32_t(t));
  const uint32_t pl_tp = Nxy * (uint32_t(z) + Nz * tp), pl_tm = Nxy * (uint32_t(z) + Nz * tm);
  const int tid = int(threadIdx.x), nth = int(blockDim.x);

  // This lane's site and neighbours; lanes past the chunk's end repeat its last site.
  // (blockIdx.y: blocks of column groups, where a site's do not fit one workgroup)
  const int G = nv / VW, GB = int(o.groups.d);
  const int i = int(o.groups.div(uint32_t(tid)));
  int gq = int(blockIdx.y) * GB + (tid - i * GB);
  const bool live = i < n && gq < G;
  const int ic = i < n ? i : n - 1;
  gq = gq < G ? gq : G - 1;
  const uint32_t p = fs.p0 + uint32_t(ic);
  const uint32_t y = g.dx.div(p), x = p - y * Nx;
  const uint32_t p_xm = x == 0 ? p + Nx - 1 : p - 1, p_xp = x + 1 == Nx ? p + 1 - Nx : p + 1;
  const uint32_t p_yp = p + Nx < Nxy ? p + Nx : p + Nx - Nxy, p_ym = p >= Nx ? p - Nx : p + Nxy - Nx;
  const uint32_t sb = 3u * uint32_t(nv) * uint32_t(sizeof(W)), vb = uint32_t(gq * VW) * uint32_t(sizeof(W));
  const size_t sw = size_t(3) * size_t(nv), cb = size_t(nv) * sizeof(W);
  const uint32_t v_p = p * sb + vb, v_xm = p_xm * sb + vb, v_xp = p_xp * sb + vb, v_ym = p_ym * sb + vb,
                 v_yp = p_yp * sb + vb;
  const char* const in_tm = reinterpret_cast<const char*>(in + sw * pl_tm);
  const char* const in_zm = reinterpret_cast<const char*>(in + sw * pl_zm);
  const char* const in_p = reinterpret_cast<const char*>(in + sw * plane);
  const char* const in_zp = reinterpret_cast<const char*>(in + sw * pl_zp);
  const char* const in_tp = reinterpret_cast<const char*>(in + sw * pl_tp);

  V raw[D][3];
  // sums of the backward and of the forward hops (fewer roundings at full size
  // than one sum of the eight: error against FP64 in C64, relative: 7.3e-8, 7.8e-8)
  cpx<T> acc[2][VW][3];
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int k = 0; k < VW; ++k)
#pragma unroll
      for (int b = 0; b < 3; ++b) acc[f][k][b] = zero<T>();

  // hop H into slot H % D; the constraint on the offset keeps the load here
#define DSL_SL(H)                                                                                          \
  if constexpr ((H) < 8) {                                                                                 \
    constexpr int HOP = (H) < 8 ? (H) : 0;                                                                 \
    uint32_t vo = HOP == 2 ? v_ym : HOP == 3 ? v_xm : HOP == 4 ? v_xp : HOP == 5 ? v_yp : v_p;              \
    asm volatile("" : "+v"(vo));                                                                           \
    const char* const b = HOP == 0 ? in_tm : HOP == 1 ? in_zm : HOP == 6 ? in_zp : HOP == 7 ? in_tp : in_p; \
    _Pragma("unroll") for (int c = 0; c < 3; ++c)                                                          \
        raw[HOP % D][c] = *reinterpret_cast<const V*>(b + size_t(c) * cb + vo);                             \
  }
  {
    // A thread moves one word (link mu, element) of every nth / 4 LW-th site, four
    // or eight (at most 8 bytes a lane: 32^4, C64 N_v = 1 154 us against 186) sites in flight;
    // sites past the end repeat the last one.
    constexpr int SWL = 4 * LW, F = VW * int(sizeof(W)) <= 8 ? 8 : 4;
    const int per = nth / SWL, k0 = tid / SWL, e = tid - k0 * SWL, mu = e / LW;
    if (nth < SWL) {
      for (int q = tid; q < n * SWL; q += nth) {
        const int k = q / SWL, f = q - k * SWL, m = f / LW;
        const uint32_t pk = fs.p0 + uint32_t(k), xk = pk - g.dx.div(pk) * Nx;
        const uint32_t sn = m == 0   ? plane + (xk == 0 ? pk + Nx - 1 : pk - 1)
                            : m == 1 ? plane + (pk >= Nx ? pk - Nx : pk + Nxy - Nx)
                                     : (m == 2 ? pl_zm : pl_tm) + pk;
        lf[q] = U[size_t(plane + fs.p0) * SWL + q];
        lb[q] = U[size_t(sn) * SWL + f];
      }
    } else if (k0 < per) {
      const W* const uf = U + size_t(plane) * SWL + e;
      const W* const ub = U + size_t(mu < 2 ? plane : mu == 2 ? pl_zm : pl_tm) * SWL + e;
#pragma nounroll
      for (int ks = k0; ks < n; ks += F * per) {
        W a[F], b[F];
#pragma unroll
        for (int j = 0; j < F; ++j) {
          const int k = ks + j * per < n ? ks + j * per : n - 1;
          const uint32_t pk = fs.p0 + uint32_t(k);
          uint32_t sn = pk;
          if (mu == 0) {
            const uint32_t xk = pk - g.dx.div(pk) * Nx;
            sn = xk == 0 ? pk + Nx - 1 : pk - 1;
          }
          if (mu == 1) sn = pk >= Nx ? pk - Nx : pk + Nxy - Nx;
          a[j] = uf[pk * uint32_t(SWL)];
          b[j] = ub[sn * uint32_t(SWL)];
        }
#pragma unroll
        for (int j = 0; j < F; ++j) {
          const int k = ks + j * per < n ? ks + j * per : n - 1;
          lf[k * SWL + e] = a[j];
          lb[k * SWL + e] = b[j];
        }
      }
    }
  }
  DSL_SL(0) DSL_SL(1) DSL_SL(2) DSL_SL(3)
  if constexpr (D > 4) {
    DSL_SL(4) DSL_SL(5)
  }
  __syncthreads();
  const W* const wf = lf + ic * 4 * LW;
  const W* const wb = lb + ic * 4 * LW;
  // eta_1 = 1, eta_2 = (-1)^x, eta_3 = (-1)^(x+y), eta_4 = (-1)^(x+y+z)
  const T e1 = x & 1u ? T(-1) : T(1), e2 = (x + y) & 1u ? T(-1) : T(1), e3 = (x + y + uint32_t(z)) & 1u ? T(-1) : T(1);
#define DSL_SH(H)                                                                                       \
  {                                                                                                     \
    using F = StagHop<H>;                                                                               \
    cpx<T> u[3][3];                                                                                     \
    load_link_lw<LW, S, T>((F::BWD ? wb : wf) + F::MU * LW, u);                                         \
    const T eta = F::MU == 0 ? T(1) : F::MU == 1 ? e1 : F::MU == 2 ? e2 : e3;                            \
    cpx<T> h[VW][3];                                                                                    \
    _Pragma("unroll") for (int c = 0; c < 3; ++c) {                                                     \
      cpx<T> a[VW];                                                                                     \
      FlatVec<S, VW>::template unpack<T>(raw[(H) % D][c], a);                                           \
      _Pragma("unroll") for (int k = 0; k < VW; ++k) h[k][c] = a[k];                                    \
    }                                                                                                   \
    _Pragma("unroll") for (int k = 0; k < VW; ++k) _Pragma("unroll") for (int a = 0; a < 3; ++a) {      \
      cpx<T> r = zero<T>();                                                                             \
      _Pragma("unroll") for (int b = 0; b < 3; ++b)                                                     \
          r = F::BWD ? cjmadd(r, u[b][a], h[k][b]) : cmadd(r, u[a][b], h[k][b]);                         \
      acc[!F::BWD][k][a] = rmadd(acc[!F::BWD][k][a], eta, r);                                           \
      flat_hold(acc[!F::BWD][k][a]);                                                                    \
    }                                                                                                   \
    DSL_SL((H) + D)                                                                                     \
  }
  DSL_SH(0) DSL_SH(1) DSL_SH(2) DSL_SH(3) DSL_SH(4) DSL_SH(5) DSL_SH(6) DSL_SH(7)
#undef DSL_SH
#undef DSL_SL
  const T half = ADJ ? T(-0.5) : T(0.5);
  const char* const ap = in_p + v_p;
  char* const op = reinterpret_cast<char*>(out + sw * plane) + v_p;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    cpx<T> f[VW];
    FlatVec<S, VW>::template unpack<T>(*reinterpret_cast<const V*>(ap + size_t(c) * cb), f);
#pragma unroll
    for (int k = 0; k < VW; ++k) {
      f[k].r = fma(mass, f[k].r, half * (acc[1][k][c].r - acc[0][k][c].r));
      f[k].i = fma(mass, f[k].i, half * (acc[1][k][c].i - acc[0][k][c].i));
    }
    if (live) *reinterpret_cast<V*>(op + size_t(c) * cb) = FlatVec<S, VW>::template pack<T>(f);
  }
}

struct StagCall {
  bool adj, compressed;
  const Geom* g;
  const void *U, *in;
  void* out;
  double mass;
  hipStream_t st;
};

template <class S, class T, int VW, int NVC = 0>
hipError_t stag_flat(const StagCall& a) {
  using W = typename S::word;
  const FlatShape s = flat_shape(*a.g, 3, int(sizeof(W)), VW, a.compressed ? 6 : 9, false);
  if (!grid_fits(s.grid, s.block)) return hipErrorNotSupported;
  const int xcd = knobs().xcd.get(1);
#define DSL_SK(A, L)                                                                                             \
  hipLaunchKernelGGL((staggered_flat_kernel<A, L, S, T, VW, NVC>), s.grid, s.block, s.lds, a.st, *a.g, s.o, xcd, \
                     (const W*)a.U, (const W*)a.in, (W*)a.out, T(a.mass))
  if (a.compressed) {
    if (a.adj) DSL_SK(true, 6); else DSL_SK(false, 6);
  } else {
    if (a.adj) DSL_SK(true, 9); else DSL_SK(false, 9);
  }
#undef DSL_SK
  return hipGetLastError();
}

template <class S>
hipError_t stag_flat16(int vw, const StagCall& a) {
  return vw == 4 ? stag_flat<S, float, 4>(a) : vw == 2 ? stag_flat<S, float, 2>(a) : stag_flat<S, float, 1>(a);
}

}  // namespace

hipError_t launch_staggered_flat(bool adj, int dtype, const Geom& g, const void* U, const void* in, void* out,
                                 double mass, hipStream_t st, bool compressed) {
  if (knobs().rows.get(1) == 0 || !flat_covers(g, dtype)) return hipErrorNotSupported;
  const int vw = flat_vw(dtype, g.nv, aligned16(in) && aligned16(out));
  if (!staggered_flat_pays(dtype, g, vw, compressed)) return hipErrorNotSupported;
  const StagCall a{adj, compressed, &g, U, in, out, mass, st};
  // NVC: as in the flat D_W kernels (N_v = 12: C64 24^3 x 48 196 us, 207 without; FP64
  // 22x18x20x16 69 and 71.5)
  switch (dtype) {
    case DT_BF16: return stag_flat16<BF16>(vw, a);
    case DT_F16: return stag_flat16<F16>(vw, a);
    case DT_C128: return g.nv == 12 ? stag_flat<C128, double, 1, 12>(a) : stag_flat<C128, double, 1>(a);
  }
  if (vw == 2) return g.nv == 12 ? stag_flat<C64, float, 2, 12>(a) : stag_flat<C64, float, 2>(a);
  return stag_flat<C64, float, 1>(a);
}

}  // namespace dsl
