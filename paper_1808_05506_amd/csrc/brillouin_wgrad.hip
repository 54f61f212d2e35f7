// Gradient of L = Re sum conj(chi) (D_B psi) with respect to W, each W taken as a
// free complex matrix, for the 40 stored directions d (slot n(d) - 41); any
// lattice and N_v, C64 and C128.  W_d(x) enters the hop of d into out(x) with the
// spin factor S_d = a_k + b_k d.gamma, and, as W_{-d}(x + d) = W_d(x)^dag, the hop of
// -d into out(x + d) with S_{-d}.  Both are Hermitian, so they act on the own field:
//   G_{W_d}(x) = sum_v sum_s [ (S_d chi(x))_s (x) conj(psi(x + d)_s)
//                            + (S_{-d} psi(x))_s (x) conj(chi(x + d)_s) ].
// A workgroup owns a chunk of P sites and NB columns, one lane each (bri_runs.hpp).
// The stored d reach the runs 13 (d = +x only) to 26; each run's psi, then its chi,
// pass through LDS half the spins at a time.  A lane sums the nine elements of the
// run's three directions in registers over both fields, four lanes (two where NB is
// no multiple of four) add theirs, and the rest of a site's N_v shares are summed
// through LDS in a fixed order.
//
// What bounds it: the issue of vector instructions: 144 multiply-adds a hop for
// the products and 24 (7 + kr) a run for the spin factors, which the own field
// shares between the run's hops (24 (5 + 3 kr) with S_d on the neighbour field).
// 16^3 x 32, N_v = 12, C64: 970 us (1417 before, hop by hop, staged through
// registers, the shares of every lane through LDS twice); two waves a SIMD, without
// the spills that three cost: 1140.
#include "bri_runs.hpp"

namespace dsl {

namespace {

// Columns NB, sites P.  RD: lanes whose shares are added in registers.
template <class S, int NB_, int P_, int MODE_>
struct GradBlock {
  using W = typename S::word;
  static constexpr int NB = NB_, P = P_, MODE = MODE_, LANES = NB * P;
  static constexpr int PL = (P + 4) * NB;
  static constexpr int RD = NB % 4 == 0 ? 4 : 2;
  static constexpr int WAVES = MODE == BRI_PAIRS ? 3 : 2;  // per SIMD
};

// x of the lane whose number differs in bit B (0 or 1) of the lane's number
template <int B>
__device__ __forceinline__ float quad_xor(float x) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), B == 0 ? 0xB1 : 0x4E, 0xF, 0xF, true));
}
template <int B>
__device__ __forceinline__ double quad_xor(double x) {
  const auto w = __builtin_bit_cast(uint2, x);
  const uint2 r{uint32_t(__builtin_amdgcn_mov_dpp(int(w.x), B == 0 ? 0xB1 : 0x4E, 0xF, 0xF, true)),
                uint32_t(__builtin_amdgcn_mov_dpp(int(w.y), B == 0 ? 0xB1 : 0x4E, 0xF, 0xF, true))};
  return __builtin_bit_cast(double, r);
}

// gm[dx + 1] += sum over spins q = Q0, Q0 + 1 of (S own)_q (x) conj(f(x + dx)_q), f in
// LDS, S = a + sgn b d.gamma.  gamma_mu takes spin p to (see run_spins of D_B)
//   gamma_4: p ^ 2, 1 (all)         gamma_3: p ^ 2, i (+, -, -, +)
//   gamma_2: 3 - p, (-, +, +, -)    gamma_1: 3 - p, i (+, +, -, -)
// OWN: the own run, dx = +1 only.
template <int Q0, bool OWN, class B, class S, class T>
__device__ __forceinline__ void grad_spins(const typename S::word* buf, const int (&ps)[3], const cpx<T> (&own)[4][3],
                                           T sgn, int dy, int dz, int dt, cpx<T> (&gm)[3][3][3]) {
  const int kr = OWN ? 0 : (dy != 0) + (dz != 0) + (dt != 0);
  const T a0 = T(-0.5) * bri_lambda<T>(kr), a1 = T(-0.5) * bri_lambda<T>(kr + 1);
  const T b0 = sgn * bri_rho<T>(kr == 0 ? 1 : kr), b1 = sgn * bri_rho<T>(kr + 1);
#pragma unroll
  for (int q = Q0; q < Q0 + 2; ++q) {
    const int p = q ^ 2, r = 3 - q;
    const T s3 = (p == 1 || p == 2) ? T(-1) : T(1);
    const T s2 = (r == 1 || r == 2) ? T(1) : T(-1);
    const T s1 = r <= 1 ? T(1) : T(-1);
    cpx<T> base[3], o[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) base[c] = mk(a1 * own[q][c].r, a1 * own[q][c].i);
    if constexpr (!OWN) {
      cpx<T> h[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) h[c] = zero<T>();
      if (dt != 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c) h[c] = rmadd(h[c], T(dt), own[p][c]);
      }
      if (dz != 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c) h[c] = cmadd_i(h[c], s3 * T(dz), own[p][c]);
      }
      if (dy != 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c) h[c] = rmadd(h[c], s2 * T(dy), own[r][c]);
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        o[c] = rmadd(mk(a0 * own[q][c].r, a0 * own[q][c].i), b0, h[c]);
        base[c] = rmadd(base[c], b1, h[c]);
      }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int dx = k == 0 ? 0 : (k == 1 ? -1 : 1);
      if (OWN && dx != 1) continue;
      if (dx != 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c) o[c] = cmadd_i(base[c], T(dx) * s1 * b1, own[r][c]);
      }
      cpx<T> f[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) f[c] = S::template load<T>(buf + ps[dx + 1] + (3 * (q - Q0) + c) * B::PL);
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) gm[dx + 1][a][b] = cmaddj(gm[dx + 1][a][b], o[a], f[b]);
    }
  }
#pragma unroll
  for (int k = OWN ? 2 : 0; k < 3; ++k)
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) hold(gm[k][a][b]);
}

template <class B, class S, class T>
__global__ void __launch_bounds__(B::LANES, B::WAVES)
    brillouin_wgrad_kernel(Geom g, FlatMarch m, int xcd, const typename S::word* __restrict__ chi,
                           const typename S::word* __restrict__ psi, typename S::word* __restrict__ GW) {
  using W = typename S::word;
  constexpr int NB = B::NB, P = B::P, PL = B::PL, LANES = B::LANES, WB = int(sizeof(W)), RD = B::RD;
  constexpr int RL = LANES / RD, RN = NB / RD;  // shares of the workgroup and of a site
  __shared__ __align__(16) char s_half0[6 * PL * WB], s_half1[6 * PL * WB], s_red[27 * RL * WB];
  W* const buf0 = reinterpret_cast<W*>(s_half0);  // [6][P + 4][NB], spins 0, 1
  W* const buf1 = reinterpret_cast<W*>(s_half1);  // spins 2, 3
  W* const red = reinterpret_cast<W*>(s_red);     // [27][P][RN]

  uint32_t seg;
  const FlatChunk<4> c = flat_chunk<4>(g, m, xcd_block(blockIdx.x, gridDim.x, xcd != 0), seg);
  const int nv = g.nv, blocks = (nv + NB - 1) / NB;
  for (int cb = 0; cb < blocks; ++cb) {
    if (cb > 0) __syncthreads();
    RunStage<B, S> st;
    st.init(g, c, cb * NB);
    const int tid = st.tid;
    int ps[3];
    st.slots(g, c, ps);
    const bool col = st.v0 + st.v < nv;
    cpx<T> ox[4][3], op[4][3];  // chi(x), psi(x)
    {
      const size_t base = size_t(c.plane + st.p) * 12 * nv + st.vc;
      load_wspinor<S, T>(chi, base, nv, ox);
      load_wspinor<S, T>(psi, base, nv, op);
    }
    // Halves n = 0 .. 55: run 13 + n / 4, of psi (n / 2 even) and chi, spins 2 (n % 2)
    // and the next.  Half n + 1 is in flight while half n is applied.
    constexpr int N = 4 * (kRuns - 13);
    const auto request = [&](int n, int h, W* dst) {
      const int k = n < N ? n : N - 1;
      st.half(g, c, k & 2 ? chi : psi, 13 + (k >> 2), n < N ? h : 1, dst);
    };
    const auto fetch = [&](int n, int h) {
      W* const dst = h ? buf1 : buf0;
      if constexpr (B::MODE == BRI_WORDS) {
        st.half_commit(dst);
        request(n + 1, h ^ 1, dst);
      } else {
        if (n < N) request(n, h, dst);
      }
    };
#define DSL_BARRIER                                                  \
  if constexpr (B::MODE != BRI_WORDS) __builtin_amdgcn_s_waitcnt(0); \
  __syncthreads();
#define DSL_RUN(RR, OWN)                                                                                    \
  {                                                                                                        \
    const int dy = OWN ? 0 : (RR) % 3 - 1, dz = OWN ? 0 : (RR) / 3 % 3 - 1, dt = OWN ? 0 : (RR) / 9 - 1;      \
    const int n = 4 * ((RR) - 13);                                                                          \
    cpx<T> gm[3][3][3];                                                                                    \
    _Pragma("unroll") for (int k = 0; k < 3; ++k) _Pragma("unroll") for (int a = 0; a < 3; ++a)            \
        _Pragma("unroll") for (int b = 0; b < 3; ++b) gm[k][a][b] = zero<T>();                             \
    DSL_BARRIER                                                                                            \
    fetch(n + 1, 1);                                                                                       \
    grad_spins<0, OWN, B, S, T>(buf0, ps, ox, T(1), dy, dz, dt, gm);                                       \
    DSL_BARRIER                                                                                            \
    fetch(n + 2, 0);                                                                                       \
    grad_spins<2, OWN, B, S, T>(buf1, ps, ox, T(1), dy, dz, dt, gm);                                       \
    DSL_BARRIER                                                                                            \
    fetch(n + 3, 1);                                                                                       \
    grad_spins<0, OWN, B, S, T>(buf0, ps, op, T(-1), dy, dz, dt, gm);                                      \
    DSL_BARRIER                                                                                            \
    fetch(n + 4, 0);                                                                                       \
    grad_spins<2, OWN, B, S, T>(buf1, ps, op, T(-1), dy, dz, dt, gm);                                      \
    _Pragma("unroll") for (int k = OWN ? 2 : 0; k < 3; ++k) _Pragma("unroll") for (int e = 0; e < 9; ++e) { \
      cpx<T> z = gm[k][e / 3][e % 3];                                                                      \
      if (!col) z = zero<T>(); /* columns past N_v repeat the last one */                                  \
      z.r += quad_xor<0>(z.r);                                                                             \
      z.i += quad_xor<0>(z.i);                                                                             \
      if (RD == 4) {                                                                                       \
        z.r += quad_xor<1>(z.r);                                                                           \
        z.i += quad_xor<1>(z.i);                                                                           \
      }                                                                                                    \
      if (tid % RD == 0) S::template store<T>(red + (k * 9 + e) * RL + tid / RD, z);                       \
    }                                                                                                      \
    __syncthreads();                                                                                       \
    constexpr int E = OWN ? 9 : 27;                                                                        \
    W* const gw = GW + size_t(c.plane + c.p0) * 360 + (OWN ? 0 : (3 * (RR) - 41) * 9);                      \
    for (int o = tid; o < c.n * E; o += LANES) {                                                           \
      const int site = o / E, e = o - site * E;                                                            \
      const W* const src = red + (OWN ? e + 18 : e) * RL + site * RN;                                      \
      W* const dst = gw + size_t(site) * 360 + e;                                                          \
      cpx<T> z = cb > 0 ? S::template load<T>(dst) : zero<T>();                                            \
      _Pragma("unroll") for (int l = 0; l < RN; ++l) z += S::template load<T>(src + l);                    \
      S::template store<T>(dst, z);                                                                        \
    }                                                                                                      \
  }
    if constexpr (B::MODE == BRI_WORDS) request(0, 0, buf0);
    fetch(0, 0);
    DSL_RUN(13, true)
#pragma nounroll
    for (int r = 14; r < kRuns; ++r) DSL_RUN(r, false)
#undef DSL_RUN
#undef DSL_BARRIER
  }
}

struct GradCall {
  const Geom* g;
  const void *chi, *psi;
  void* GW;
  hipStream_t st;
};

template <class B, class S, class T>
hipError_t bri_wgrad_t(const GradCall& a) {
  using W = typename S::word;
  const Geom& g = *a.g;
  FlatMarch m = make_flat_march(g, uint32_t(B::P), 1);
  int by, bz;
  pick_tile(g, long(g.n[0]) * 24 * B::NB * long(sizeof(W)), 1280L * 1024, by, bz);
  flat_march_tile(g, m, knobs().bri_tile_y.get(by), knobs().bri_tile_z.get(bz));
  if (!grid_fits(dim3(m.grid), dim3(B::LANES))) return hipErrorNotSupported;
  hipLaunchKernelGGL((brillouin_wgrad_kernel<B, S, T>), dim3(m.grid), dim3(B::LANES), 0, a.st, g, m,
                     int(knobs().xcd.get(1) != 0), (const W*)a.chi, (const W*)a.psi, (W*)a.GW);
  return hipGetLastError();
}

template <int NB, int P>
hipError_t bri_wgrad_c64(const GradCall& a, bool pairs) {
  return pairs ? bri_wgrad_t<GradBlock<C64, NB, P, BRI_PAIRS>, C64, float>(a)
               : bri_wgrad_t<GradBlock<C64, NB, P, BRI_WORDS>, C64, float>(a);
}

template <int NB, int P>
hipError_t bri_wgrad_c128(const GradCall& a) {
  return bri_wgrad_t<GradBlock<C128, NB, P, BRI_WIDE>, C128, double>(a);
}

}  // namespace

// hipErrorNotSupported where the direct kernel is taken: misaligned FP64, planes of 4 GB,
// DSLASH_ROWS=0, and where this one does not pay (brillouin_wgrad_pays).
// DSLASH_ROWS=2: as in D_B, in C64 only.
hipError_t launch_brillouin_wgrad_flat(int dtype, const Geom& g, const void* chi, const void* psi, void* GW,
                                       hipStream_t st) {
  const int rows = knobs().rows.get(1);
  if (rows == 0 || (dtype != DT_C64 && dtype != DT_C128)) return hipErrorNotSupported;
  if (rows == 2 && (dtype != DT_C64 || !brillouin_rows_cover(dtype, g, false))) return hipErrorNotSupported;
  if (rows != 2 && !brillouin_wgrad_pays(dtype, g)) return hipErrorNotSupported;
  const size_t plane = size_t(g.n[0]) * size_t(g.n[1]) * dtype_bytes(dtype);
  if (plane * 12 * size_t(g.nv) >= (size_t(1) << 32)) return hipErrorNotSupported;
  if (dtype == DT_C128 && !(aligned16(chi) && aligned16(psi) && aligned16(GW))) return hipErrorNotSupported;
  const GradCall a{&g, chi, psi, GW, st};
  int nb = bri_block(dtype, g.nv);
  // FP64: four lanes' shares are added in registers or the sums take too much LDS
  if (dtype == DT_C128 && nb == 6) nb = 8;
  if (dtype == DT_C64) {
    const bool pairs = g.nv % 2 == 0 && aligned16(chi) && aligned16(psi);
    switch (nb) {
      case 24: return bri_wgrad_c64<24, 8>(a, pairs);
      case 16: return bri_wgrad_c64<16, 16>(a, pairs);
      case 12: return bri_wgrad_c64<12, 21>(a, pairs);
      case 10: return bri_wgrad_c64<10, 25>(a, pairs);
      case 8: return bri_wgrad_c64<8, 32>(a, pairs);
      case 6: return bri_wgrad_c64<6, 42>(a, pairs);
    }
    return bri_wgrad_c64<4, 64>(a, pairs);
  }
  switch (nb) {
    case 12: return bri_wgrad_c128<12, 16>(a);
    case 8: return bri_wgrad_c128<8, 24>(a);
  }
  return bri_wgrad_c128<4, 40>(a);
}

}  // namespace dsl
