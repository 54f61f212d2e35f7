// D_B on stored off-axis links (Sec. 5), any lattice and N_v, C64 and C128.
//
// A workgroup owns a chunk of P sites (chunks.hpp) and a block of NB right-hand
// sides, one lane each.  The 80 hops reach the 27 runs (y + dy, z + dz, t + dt)
// of the chunk; each run is staged in LDS once, with up to four halo sites, and
// serves the hops dx = -1, 0, 1.  With it come the three link columns of those
// hops: W_d(x) where d is one of the 40 stored directions (runs 14 .. 26, and +x
// of the own run 13), else W_{-d}(x + d), applied as its adjoint.
//   out(x) = (m0 + 15/8) psi(x) + sum_d (-lambda_k / 2 + rho_k d.gamma) W_d(x) psi(x + d)
// (rho_k -> -rho_k for the adjoint) is summed in registers over the 27 runs.
//
// What bounds it: the issue of vector instructions.  The links of the 80 hops are
// 11520 multiply-adds a lane; taken one by one, their spin factors are 7100 more,
// and staging added 3800 (C64) and 13000 (C128).  So
// - the spin factors of the three hops of a run are taken together (run_spins),
//   3900 in all;
// - a run is [component][slot][column] in LDS: a lane's words are at fixed offsets
//   from one address per dx, without bank conflicts;
// - a lane stages the same component, column and link words of every run, so their
//   places are worked out once;
// - the adjoint is a sign of the multiply-add: the runs before and behind the own
//   one are compiled apart;
// - spinors go straight from global memory to LDS (global_load_lds_dwordx4: lane l
//   of a wave writes 16 bytes at b + 16 l for a wave-uniform b), half a run while
//   the other half is applied, so no registers hold them: the links of three hops
//   fit beside the sums at three waves a SIMD (C64) and two (C128).
// 32^4, N_v = 12, C64: 6.28 ms (7.05 before, hop by hop and staged through
// registers; with the staging left out 4.67); 16^3 x 32, C128: 1.38 ms (2.10;
// 1.09).  C64 chunks of 21 sites: 6.23 ms, of 16 6.26 (bri_short_chunks); C128 of 20: 1.41, of 16 1.50.
#include "bri_runs.hpp"

namespace dsl {

namespace {

template <class S, int NB_, int P_, int MODE_>
struct BriBlock {
  using W = typename S::word;
  static constexpr int NB = NB_, P = P_, MODE = MODE_, LANES = NB * P;
  static constexpr int PL = (P + 4) * NB;                     // words per component in LDS
  static constexpr int KL = (9 * P + LANES - 1) / LANES;      // link words per lane and column
  static constexpr int WAVES = MODE == BRI_PAIRS && NB > 4 ? 3 : 2;  // per SIMD
};

template <bool DAG, class S, class T>
__device__ __forceinline__ void lds_link(const typename S::word* link, cpx<T> (&u)[3][3]) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      u[i][j] = S::template load<T>(link + (DAG ? j * 3 + i : i * 3 + j));
      if (DAG) u[i][j].i = -u[i][j].i;
    }
}

// out = in + u psi_q for the lane's spin-q colour triple at psi
template <int PL, class S, class T>
__device__ __forceinline__ void add_link(const cpx<T> (&in)[3], const cpx<T> (&u)[3][3],
                                         const typename S::word* psi, cpx<T> (&out)[3]) {
  cpx<T> p[3];
#pragma unroll
  for (int b = 0; b < 3; ++b) p[b] = S::template load<T>(psi + b * PL);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    out[c] = in[c];
#pragma unroll
    for (int b = 0; b < 3; ++b) out[c] = cmadd(out[c], u[c][b], p[b]);
  }
}

// The hops of one run, spin by spin.  With c-, c0, c+ the products W psi of the
// three dx, and the run's k = kr of (dy, dz, dt) (a_{k+1} = a_k / 2 and b_{k+1} =
// b_k / 4 for a_k = -lambda_k / 2, b_k = rho_k):
//   e = c- + c+, f = c+ - c- = e - 2 c-, m = c0 + e / 2, n = c0 + e / 4 = m - e / 4
//   out += a_k m + b_k (dy g2 + dz g3 + dt g4) n + b_{k+1} g1 f
// where e and m come out of the multiply-adds of the links: 24 (4 + k) operations
// for the spin factors of the three hops, 24 (5 + 3 k) hop by hop.  HALF: the
// links of dx = -1 and +1 are staged times 1/2 (exact), so c-, c+, e, f are halves;
// otherwise e / 2 costs 24 more.  psi_q goes with gamma_mu to the spin
//   gamma_4: q ^ 2, 1 (all)         gamma_3: q ^ 2, i (+, -, -, +)
//   gamma_2: 3 - q, (-, +, +, -)    gamma_1: 3 - q, i (+, +, -, -)
// ps[dx + 1]: the lane's words of the site at x + dx.  OWN: the own run, dx = -1
// adjoint, +1 stored, 0 none; dy, dz, dt are the same for every lane
// (scalar branches).
template <class T>
struct RunLinks {
  cpx<T> m[3][3], o[3][3], p[3][3];  // dx = -1, 0, +1
};

template <bool DAG, bool OWN, int P, class S, class T>
__device__ __forceinline__ void run_links(const typename S::word* link, RunLinks<T>& u) {
  lds_link<OWN || DAG, S, T>(link, u.m);
  lds_link<!OWN && DAG, S, T>(link + 18 * P, u.p);
  if constexpr (!OWN) lds_link<DAG, S, T>(link + 9 * P, u.o);
}

// spins Q0 and Q0 + 1 of psi
template <int Q0, bool ADJ, bool OWN, class B, class S, class T>
__device__ __forceinline__ void run_spins(const typename S::word* buf, const int (&ps)[3], const RunLinks<T>& u, int dy,
                                          int dz, int dt, cpx<T> (&acc)[4][3]) {
  constexpr bool HALF = B::MODE != BRI_WIDE;
  const int kr = OWN ? 0 : (dy != 0) + (dz != 0) + (dt != 0);
  const T s = ADJ ? T(-1) : T(1);
  // OWN: a_1 (c- + c+), of the halves twice that
  const T a = OWN ? T(HALF ? -1 : -0.5) * bri_lambda<T>(1) : T(-0.5) * bri_lambda<T>(kr);
  const T bf = s * T(HALF ? 2 : 1) * bri_rho<T>(kr + 1);
  const T b = s * bri_rho<T>(kr == 0 ? 1 : kr);
  const T by = b * T(dy), bz = b * T(dz), bt = b * T(dt);
#pragma unroll
  for (int q = Q0; q < Q0 + 2; ++q) {
    const int P43 = q ^ 2, P21 = 3 - q;
    const T s3 = (q == 1 || q == 2) ? T(-1) : T(1);
    const T s2 = (q == 1 || q == 2) ? T(1) : T(-1);
    const T s1 = q <= 1 ? T(1) : T(-1);
    cpx<T> z[3], cm[3], e[3], m[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) z[c] = zero<T>();
    add_link<B::PL, S, T>(z, u.m, buf + ps[0] + 3 * (q - Q0) * B::PL, cm);
    add_link<B::PL, S, T>(cm, u.p, buf + ps[2] + 3 * (q - Q0) * B::PL, e);
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[P21][c] = cmadd_i(acc[P21][c], s1 * bf, rmadd(e[c], T(-2), cm[c]));
    if constexpr (OWN) {
#pragma unroll
      for (int c = 0; c < 3; ++c) acc[q][c] = rmadd(acc[q][c], a, e[c]);
    } else {
      if constexpr (HALF) {
        add_link<B::PL, S, T>(e, u.o, buf + ps[1] + 3 * (q - Q0) * B::PL, m);
      } else {
#pragma unroll
        for (int c = 0; c < 3; ++c) z[c] = T(0.5) * e[c];
        add_link<B::PL, S, T>(z, u.o, buf + ps[1] + 3 * (q - Q0) * B::PL, m);
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        acc[q][c] = rmadd(acc[q][c], a, m[c]);
        m[c] = rmadd(m[c], T(HALF ? -0.5 : -0.25), e[c]);
      }
      if (dt != 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[P43][c] = rmadd(acc[P43][c], bt, m[c]);
      }
      if (dz != 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[P43][c] = cmadd_i(acc[P43][c], s3 * bz, m[c]);
      }
      if (dy != 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[P21][c] = rmadd(acc[P21][c], s2 * by, m[c]);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int c = 0; c < 3; ++c) hold(acc[q][c]);
}

template <bool ADJ, bool CLOV, class B, class S, class T>
__global__ void __launch_bounds__(B::LANES, B::WAVES)
    brillouin_flat_kernel(Geom g, FlatMarch m, int xcd, const typename S::word* __restrict__ Wl,
                          const typename S::word* __restrict__ in, typename S::word* __restrict__ out,
                          const typename S::word* __restrict__ C, T diag) {
  using W = typename S::word;
  constexpr int NB = B::NB, P = B::P, PL = B::PL, LANES = B::LANES, WB = int(sizeof(W));
  // arrays of their own: the compiler then knows that reads of one half need not
  // wait for a copy into the other
  __shared__ __align__(16) char s_half0[6 * PL * WB], s_half1[6 * PL * WB], s_links[27 * P * WB];
  W* const buf0 = reinterpret_cast<W*>(s_half0);  // [6][P + 4][NB], spins 0, 1
  W* const buf1 = reinterpret_cast<W*>(s_half1);  // spins 2, 3
  W* const wbuf = reinterpret_cast<W*>(s_links);  // [3][P][9]

  uint32_t seg;
  const FlatChunk<4> c = flat_chunk<4>(g, m, xcd_block(blockIdx.x, gridDim.x, xcd != 0), seg);
  RunStage<B, S> st;
  st.init(g, c, int(blockIdx.y) * NB);
  const int nv = g.nv, tid = st.tid, wave = st.wave;
  const uint32_t nx = c.nx, nxy = c.nxy, p = st.p;
  int ps[3];
  st.slots(g, c, ps);
  const W* const link = wbuf + st.i * 9;

  // link words: element e of chunk site s, and of its x neighbours
  uint32_t lq[B::KL][3], le[B::KL];
#pragma unroll
  for (int k = 0; k < B::KL; ++k) {
    const int h = tid + k * LANES, s0 = h / 9, e = h - s0 * 9, s = s0 < c.n ? s0 : c.n - 1;
    const uint32_t ls = c.p0 + uint32_t(s), x = ls - g.dx.div(ls) * nx;
    lq[k][0] = x > 0 ? ls - 1 : ls + nx - 1;
    lq[k][1] = ls;
    lq[k][2] = x + 1 < nx ? ls + 1 : ls + 1 - nx;
    le[k] = uint32_t(e * WB);
  }

  cpx<T> acc[4][3];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int b = 0; b < 3; ++b) acc[q][b] = zero<T>();

  W lw[B::KL][3];
  // the lane's word k of link column col of run r
  const auto link_word = [&](int r, uint32_t plane, int dy, int col, int k) {
    const bool dag = 3 * r + col <= 40;
    const int slot = dag ? 39 - 3 * r - col : 3 * r + col - 41;  // (-1 at d = 0, unused: slot 0)
    const char* lb = reinterpret_cast<const char*>(Wl) +
                     (size_t(dag ? plane : c.plane) * 360 + size_t((slot > 0 ? slot : 0) * 9)) * WB;
    const uint32_t q = dag ? shift_y(lq[k][col], dy, nx, nxy) : lq[k][1];
    return lb + (q * uint32_t(360 * WB) + le[k]);
  };
  // links of run r: requested (WIDE: into LDS, else into registers) ...
  const auto links = [&](int r) {
    const uint32_t plane = run_plane(g, c, r);
    const int dy = r % 3 - 1;
#pragma unroll
    for (int k = 0; k < B::KL; ++k)
      if (tid + k * LANES < 9 * P) {
#pragma unroll
        for (int col = 0; col < 3; ++col) {
          const char* w = link_word(r, plane, dy, col, k);
          if constexpr (B::MODE == BRI_WIDE) dma16(w, wbuf + col * 9 * P + k * LANES + wave * 64);
          else lw[k][col] = *reinterpret_cast<const W*>(w);
        }
      }
  };
  // ... and from the registers into LDS
  const auto links_commit = [&] {
#pragma unroll
    for (int k = 0; k < B::KL; ++k)
      if (tid + k * LANES < 9 * P) {
#pragma unroll
        for (int col = 0; col < 3; ++col) {
          W w = lw[k][col];
          if (col != 1) {  // halves (run_spins)
            w.x *= T(0.5);
            w.y *= T(0.5);
          }
          wbuf[col * 9 * P + tid + k * LANES] = w;
        }
      }
  };
  // Half a run is in flight while the other one is applied.  Before the first
  // barrier of run r its spins 0, 1 and its links have arrived; then spins 2, 3 are
  // fetched, and after the second barrier (the links are in registers) spins 0, 1
  // and the links of run r + 1 (past the last one: run 26 again, unused).  What
  // passes through registers is requested one half earlier.
#define DSL_FETCH0(r)                              \
  if constexpr (B::MODE == BRI_WORDS) {            \
    st.half_commit(buf0);                              \
    st.half(g, c, in, r, 1, buf1);                              \
  } else {                                         \
    st.half(g, c, in, r, 0, buf0);                              \
  }                                                \
  if constexpr (B::MODE == BRI_WIDE) {             \
    links(r);                                      \
  } else {                                         \
    links_commit();                                \
    links((r) + 1 < kRuns ? (r) + 1 : kRuns - 1);  \
  }
#define DSL_FETCH1(r)                                  \
  if constexpr (B::MODE == BRI_WORDS) {                \
    st.half_commit(buf1);                                  \
    st.half(g, c, in, (r) + 1 < kRuns ? (r) + 1 : kRuns - 1, 0, buf0); \
  } else {                                             \
    st.half(g, c, in, r, 1, buf1);                                  \
  }
#define DSL_BARRIER                                                   \
  if constexpr (B::MODE != BRI_WORDS) __builtin_amdgcn_s_waitcnt(0);  \
  __syncthreads();
#define DSL_APPLY(r, DAG, OWN)                                                                              \
  {                                                                                                         \
    const int dy = OWN ? 0 : (r) % 3 - 1, dz = OWN ? 0 : (r) / 3 % 3 - 1, dt = OWN ? 0 : (r) / 9 - 1;       \
    RunLinks<T> u;                                                                                          \
    DSL_BARRIER                                                                                             \
    run_links<DAG, OWN, P, S, T>(link, u);                                                                  \
    DSL_FETCH1(r)                                                                                           \
    run_spins<0, ADJ, OWN, B, S, T>(buf0, ps, u, dy, dz, dt, acc);                                          \
    DSL_BARRIER                                                                                             \
    DSL_FETCH0((r) + 1 < kRuns ? (r) + 1 : kRuns - 1)                                                       \
    run_spins<2, ADJ, OWN, B, S, T>(buf1, ps, u, dy, dz, dt, acc);                                          \
  }
  if constexpr (B::MODE == BRI_WORDS) st.half(g, c, in, 0, 0, buf0);
  if constexpr (B::MODE != BRI_WIDE) links(0);
  DSL_FETCH0(0)
#pragma nounroll
  for (int r = 0; r < 13; ++r) DSL_APPLY(r, true, false)
  DSL_APPLY(13, false, true)
#pragma nounroll
  for (int r = 14; r < kRuns; ++r) DSL_APPLY(r, false, false)
#undef DSL_APPLY
#undef DSL_BARRIER
#undef DSL_FETCH0
#undef DSL_FETCH1
  // the diagonal term last, from memory: the sums before it stay small (error
  // against FP64 in C64, relative: 6e-8; 1.9e-7 with it between the hops)
  const size_t base = size_t(c.plane + p) * 12 * nv + st.vc;
  cpx<T> own[4][3];
  load_wspinor<S, T>(in, base, nv, own);
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int b = 0; b < 3; ++b) acc[q][b] = rmadd(acc[q][b], diag, own[q][b]);
  if constexpr (CLOV) clover_madd<S, T>(C + size_t(c.plane + p) * 36, own, acc);
  if (st.xl < c.n && st.v0 + st.v < nv) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int b = 0; b < 3; ++b) S::template store<T>(out + base + size_t(q * 3 + b) * nv, acc[q][b]);
  }
}

struct BriCall {
  bool adj;
  const Geom* g;
  const void *Wl, *in, *clover;
  void* out;
  double mass;
  hipStream_t st;
};

template <class B, class S, class T>
hipError_t bri_flat_t(const BriCall& a) {
  using W = typename S::word;
  const Geom& g = *a.g;
  FlatMarch m = make_flat_march(g, uint32_t(B::P), 1);
  int by, bz;
  pick_tile(g, long(g.n[0]) * 12 * B::NB * long(sizeof(W)), 1280L * 1024, by, bz);
  flat_march_tile(g, m, knobs().bri_tile_y.get(by), knobs().bri_tile_z.get(bz));
  const dim3 grid(m.grid, uint32_t((g.nv + B::NB - 1) / B::NB));
  if (!grid_fits(grid, dim3(B::LANES))) return hipErrorNotSupported;
  const T diag = T(a.mass) + T(15.0 / 8.0);
  const int xcd = knobs().xcd.get(1) != 0;
#define DSL_BF(A, CL)                                                                                            \
  hipLaunchKernelGGL((brillouin_flat_kernel<A, CL, B, S, T>), grid, dim3(B::LANES), 0, a.st, g, m, xcd, \
                     (const W*)a.Wl, (const W*)a.in, (W*)a.out, (const W*)a.clover, diag)
  if (a.clover) {
    if (a.adj) DSL_BF(true, true); else DSL_BF(false, true);
  } else {
    if (a.adj) DSL_BF(true, false); else DSL_BF(false, false);
  }
#undef DSL_BF
  return hipGetLastError();
}

template <int NB>
hipError_t bri_flat_c64(const BriCall& a, bool pairs) {
  constexpr int P = bri_sites(DT_C64, NB);
  if constexpr (NB == 12)
    if (bri_short_chunks(*a.g, NB, pairs)) return bri_flat_t<BriBlock<C64, NB, 16, BRI_PAIRS>, C64, float>(a);
  return pairs ? bri_flat_t<BriBlock<C64, NB, P, BRI_PAIRS>, C64, float>(a)
               : bri_flat_t<BriBlock<C64, NB, P, BRI_WORDS>, C64, float>(a);
}

template <int NB>
hipError_t bri_flat_c128(const BriCall& a) {
  return bri_flat_t<BriBlock<C128, NB, bri_sites(DT_C128, NB), BRI_WIDE>, C128, double>(a);
}

}  // namespace

// D_B for C64 and C128; hipErrorNotSupported where the direct kernel is taken: other
// storages, misaligned FP64, planes of 4 GB, DSLASH_ROWS=0, and where this one does not
// pay (brillouin_flat_pays).  DSLASH_ROWS=2: this kernel where brillouin_rows_cover says so.
hipError_t launch_brillouin_flat(bool adj, int dtype, const Geom& g, const void* Wl, const void* in, void* out,
                                 double mass, hipStream_t st, const void* clover) {
  const int rows = knobs().rows.get(1);
  if (rows == 0 || (dtype != DT_C64 && dtype != DT_C128)) return hipErrorNotSupported;
  if (rows == 2 && !brillouin_rows_cover(dtype, g, clover != nullptr)) return hipErrorNotSupported;
  if (rows != 2 && !brillouin_flat_pays(dtype, g)) return hipErrorNotSupported;
  const size_t wb = dtype_bytes(dtype), plane = size_t(g.n[0]) * size_t(g.n[1]) * wb;
  if (plane * 360 >= (size_t(1) << 32) || plane * 12 * size_t(g.nv) >= (size_t(1) << 32)) return hipErrorNotSupported;
  if (dtype == DT_C128 && !(aligned16(Wl) && aligned16(in) && aligned16(out) && aligned16(clover)))
    return hipErrorNotSupported;
  const BriCall a{adj, &g, Wl, in, clover, out, mass, st};
  const int nb = bri_block(dtype, g.nv);
  if (dtype == DT_C64) {
    const bool pairs = g.nv % 2 == 0 && aligned16(in);
    switch (nb) {
      case 24: return bri_flat_c64<24>(a, pairs);
      case 16: return bri_flat_c64<16>(a, pairs);
      case 12: return bri_flat_c64<12>(a, pairs);
      case 10: return bri_flat_c64<10>(a, pairs);
      case 8: return bri_flat_c64<8>(a, pairs);
      case 6: return bri_flat_c64<6>(a, pairs);
    }
    return bri_flat_c64<4>(a, pairs);
  }
  switch (nb) {
    case 12: return bri_flat_c128<12>(a);
    case 8: return bri_flat_c128<8>(a);
    case 6: return bri_flat_c128<6>(a);
  }
  return bri_flat_c128<4>(a);
}

}  // namespace dsl
