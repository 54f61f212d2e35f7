// Row-staged D_B with its off-axis links built on the fly (Sec. 5; see rows.hpp for
// the row staging).  A workgroup
// owns an x-row chunk of R sites and all N_v right-hand sides (thread (x, v)).
// The 80 hops of the 3^4 stencil reach the 27 rows (y + dy, z + dz, t + dt),
// dy, dz, dt in {-1, 0, 1}; each such row is staged once, with the halo sites
// x0 - 1 and x0 + n, through one LDS buffer with coalesced 16-byte loads, and
// serves the hops d = (dx, dy, dz, dt), dx in {-1, 0, 1}; the three link columns
// W_d(x) of those hops are built from V in LDS.  Thread (x, v) accumulates
//   out(x) = (m0 + 15/8) psi(x) + sum_d (-lambda_k / 2 + rho_k d.gamma) W_d(x) psi(x + d)
// (rho_k -> -rho_k for the adjoint) in registers over the 27 rows and writes
// its output once, through LDS with coalesced 16-byte stores.
#include <stdlib.h>

#include "launch.hpp"
#include "rows.hpp"
#include "tiles.hpp"

namespace dsl {

namespace {

constexpr int kBriRows = 27;  // (dy, dz, dt) in {-1, 0, 1}^3, row 13 is the own row

DSL_HD void bri_row_offset(int r, int& dy, int& dz, int& dt) {
  dy = r % 3 - 1;
  dz = (r / 3) % 3 - 1;
  dt = r / 9 - 1;
}

DSL_HD uint32_t bri_row_base(const Geom& g, const RowChunk& c, int dy, int dz, int dt) {
  int y = c.y + dy, z = c.z + dz, t = c.t + dt;
  y = y < 0 ? y + g.n[1] : (y >= g.n[1] ? y - g.n[1] : y);
  z = z < 0 ? z + g.n[2] : (z >= g.n[2] ? z - g.n[2] : z);
  t = t < 0 ? t + g.n[3] : (t >= g.n[3] ? t - g.n[3] : t);
  return uint32_t(g.stride[1] * y + g.stride[2] * z + g.stride[3] * t);
}

template <int NV, class S>
struct BriStage {
  using W = typename S::word;
  static constexpr int SW = 12 * NV;                  // words per site
  static constexpr int SP = SW * int(sizeof(W)) / 16; // 16-byte pieces per site
  static constexpr int CH = SP / NV;                  // pieces per lane
  // halo pieces per thread (2 SP = 12 N_v of them over R N_v threads): one
  // for chunks of at least 12 sites, two for the chunks of 6 .. 11 sites
  // taken at N_v > 16 (the launcher checks R HK >= 12)
  static constexpr int HK = NV > 16 ? 2 : 1;
};

// A staged row in flight: the lane's pieces of its site, one piece of the halo
// sites, and its words of the row's three link columns.
template <int NV, class S>
struct BriRowRegs {
  u32x4 p[BriStage<NV, S>::CH];
  u32x4 halo[BriStage<NV, S>::HK];
};

template <int NV, class S>
__device__ __forceinline__ void bri_issue(const Geom& g, const RowChunk& c, const typename S::word* __restrict__ in, int r,
                                          int xm, int xp, int xl, int v, int tid, int nth, BriRowRegs<NV, S>& q) {
  using St = BriStage<NV, S>;
  int dy, dz, dt;
  bri_row_offset(r, dy, dz, dt);
  const uint32_t nb = bri_row_base(g, c, dy, dz, dt);
  const int xc = xl < c.n ? xl : c.n - 1;
  const u32x4* src = reinterpret_cast<const u32x4*>(in + size_t(nb + c.x0) * St::SW);
#pragma unroll
  for (int j = 0; j < St::CH; ++j) q.p[j] = src[xc * St::SP + j * NV + v];
#pragma unroll
  for (int k = 0; k < St::HK; ++k) {
    int h = tid + k * nth;
    h = h < 2 * St::SP ? h : 2 * St::SP - 1;
    const int hs = h < St::SP ? xm : xp;
    q.halo[k] = reinterpret_cast<const u32x4*>(in + size_t(nb + hs) * St::SW)[h < St::SP ? h : h - St::SP];
  }
}

template <int NV, class S>
__device__ __forceinline__ void bri_commit(const RowChunk& c, const BriRowRegs<NV, S>& q, typename S::word* buf,
                                           int xl, int v, int tid, int nth) {
  using St = BriStage<NV, S>;
  constexpr int SSP = SiteStride<NV, S>::PIECES;
  const int xc = xl < c.n ? xl : c.n - 1;
  u32x4* dst = reinterpret_cast<u32x4*>(buf) + (xc + 1) * SSP;
#pragma unroll
  for (int j = 0; j < St::CH; ++j) dst[j * NV + v] = q.p[j];
#pragma unroll
  for (int k = 0; k < St::HK; ++k) {
    int h = tid + k * nth;
    h = h < 2 * St::SP ? h : 2 * St::SP - 1;
    u32x4* hdst = reinterpret_cast<u32x4*>(buf) + (h < St::SP ? 0 : (c.n + 1) * SSP);
    hdst[h < St::SP ? h : h - St::SP] = q.halo[k];
  }
}

// acc += (a + b d.gamma) chi for chi = W psi, one hop of row (dy, dz, dt)
template <int NV, class S, class T>
__device__ __forceinline__ void bri_hop(const typename S::word* site, const typename S::word* link, int v, T a,
                                        T B1, T B2, T B3, T B4, int d0, int d1, int d2, int d3,
                                        cpx<T> (&acc)[4][3]) {
  cpx<T> u[3][3], p[4][3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) u[i][j] = S::template load<T>(link + i * 3 + j);
#pragma unroll
  for (int sp = 0; sp < 4; ++sp)
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) p[sp][cc] = S::template load<T>(site + (sp * 3 + cc) * NV + v);
  // one colour row of chi = W psi at a time (the spin factor does not mix
  // colours): upper spins += S chi_low, lower += S^dag chi_up with
  // S = sum_mu d_mu s_mu; d_mu is the same for every lane (uniform branches)
#pragma unroll
  for (int cc = 0; cc < 3; ++cc) {
    cpx<T> chi[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      cpx<T> t = zero<T>();
#pragma unroll
      for (int b = 0; b < 3; ++b) t = cmadd(t, u[cc][b], p[q][b]);
      chi[q] = t;
      acc[q][cc] = rmadd(acc[q][cc], a, t);
    }
    if (d3 != 0) {
      acc[0][cc] = rmadd(acc[0][cc], B4, chi[2]);
      acc[1][cc] = rmadd(acc[1][cc], B4, chi[3]);
      acc[2][cc] = rmadd(acc[2][cc], B4, chi[0]);
      acc[3][cc] = rmadd(acc[3][cc], B4, chi[1]);
    }
    if (d2 != 0) {
      acc[0][cc] = cmadd_i(acc[0][cc], -B3, chi[2]);
      acc[1][cc] = cmadd_i(acc[1][cc], B3, chi[3]);
      acc[2][cc] = cmadd_i(acc[2][cc], B3, chi[0]);
      acc[3][cc] = cmadd_i(acc[3][cc], -B3, chi[1]);
    }
    if (d1 != 0) {
      acc[0][cc] = rmadd(acc[0][cc], -B2, chi[3]);
      acc[1][cc] = rmadd(acc[1][cc], B2, chi[2]);
      acc[2][cc] = rmadd(acc[2][cc], B2, chi[1]);
      acc[3][cc] = rmadd(acc[3][cc], -B2, chi[0]);
    }
    if (d0 != 0) {
      acc[0][cc] = cmadd_i(acc[0][cc], -B1, chi[3]);
      acc[1][cc] = cmadd_i(acc[1][cc], -B1, chi[2]);
      acc[2][cc] = cmadd_i(acc[2][cc], B1, chi[1]);
      acc[3][cc] = cmadd_i(acc[3][cc], B1, chi[0]);
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) hold(acc[q][cc]);
}

// On-the-fly links: W_d(x) for the three hops (dx = -1, 0, 1; dy, dz, dt) of
// row r and the chunk's sites, built from V (Tab. 1) straight into the link
// columns, four lanes per (column, site) pair, one per first hop.  Every W_d(x) of the 80
// directions is built where it is used, so no adjoint relation is needed.
template <class S, class T>
__device__ __forceinline__ void bri_build(const Geom& g, const RowChunk& c, const typename S::word* __restrict__ V,
                                          int r, typename S::word* wbuf, int R, int tid, int nth) {
  // GL = 4 consecutive lanes share one (column, site) item: lane `part` sums
  // the orderings that begin with hop number `part` of d, and the partial
  // sums are added in a fixed butterfly (every lane of the group ends with
  // the same bits).  The nth / GL groups step through the 3 n items.
  constexpr int GL = 4;
  int dy, dz, dt;
  bri_row_offset(r, dy, dz, dt);
  const int part = tid % GL;
#pragma unroll 1
  for (int item = tid / GL; item < 3 * c.n; item += nth / GL) {  // uniform over a group
    const int col = item / c.n, site = item - col * c.n;
    const int d[4] = {col - 1, dy, dz, dt};
    if ((d[0] | dy | dz | dt) == 0) continue;  // no hop (a whole group)
    const int x[4] = {c.x0 + site, c.y, c.z, c.t};
    cpx<T> w[3][3];
    const int nperm = brillouin_path_tree_sum<S, T>(g, V, x, d, part, w);
#pragma unroll
    for (int off = 1; off < GL; off *= 2)
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          w[a][b].r += __shfl_xor(w[a][b].r, off);
          w[a][b].i += __shfl_xor(w[a][b].i, off);
        }
    if (part == 0) {
      const T inv = T(1) / T(nperm);
      typename S::word* o = wbuf + col * R * 9 + site * 9;
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) S::template store<T>(o + a * 3 + b, inv * w[a][b]);
    }
  }
}

// The three hops of staged row r (and the diagonal term, with the clover term
// if CLOV, for the own row).
template <bool ADJ, bool CLOV, int NV, class S, class T>
__device__ __forceinline__ void bri_row_compute(int r, const typename S::word* buf, const typename S::word* wbuf,
                                                const typename S::word* lcl, int R, int xl, int v, T diag,
                                                cpx<T> (&acc)[4][3]) {
  constexpr int SSW = SiteStride<NV, S>::WORDS;
  int dy, dz, dt;
  bri_row_offset(r, dy, dz, dt);
#pragma unroll
  for (int dx = -1; dx <= 1; ++dx) {
    const int k = (dx != 0) + (dy != 0) + (dz != 0) + (dt != 0);
    const typename S::word* site = buf + (xl + 1 + dx) * SSW;
    if (k == 0) {
      // own site: the diagonal term
      if constexpr (CLOV) {
        cpx<T> p[4][3];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int cc = 0; cc < 3; ++cc) {
            p[q][cc] = S::template load<T>(site + (q * 3 + cc) * NV + v);
            acc[q][cc] = rmadd(acc[q][cc], diag, p[q][cc]);
          }
        clover_madd<S, T>(lcl + xl * 36, p, acc);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int cc = 0; cc < 3; ++cc)
            acc[q][cc] = rmadd(acc[q][cc], diag, S::template load<T>(site + (q * 3 + cc) * NV + v));
      }
      continue;
    }
    const T a = T(-0.5) * bri_lambda<T>(k);
    const T b = (ADJ ? T(-1) : T(1)) * bri_rho<T>(k);
    const typename S::word* link = wbuf + (dx + 1) * R * 9 + xl * 9;
    bri_hop<NV, S, T>(site, link, v, a, b * T(dx), b * T(dy), b * T(dz),
                      b * T(dt), dx, dy, dz, dt, acc);
  }
}


}  // namespace

// Waves per SIMD: three (168 VGPRs); two below N_v = 8.
template <int NV> struct BriWaves { static constexpr int value = NV < 8 ? 2 : 3; };

// CLOV: adds the site-local clover term (packed, 36 words per site, staged
// in LDS after the link columns).
template <bool ADJ, bool CLOV, int NV, class S, class T>
__global__ void __launch_bounds__(256, BriWaves<NV>::value)
    brillouin_rows_kernel(Geom g, RowTraversal tr, ChunkTiles o, int xcd, const typename S::word* __restrict__ V,
                          const typename S::word* __restrict__ in, typename S::word* __restrict__ out,
                          const typename S::word* __restrict__ C, T diag) {
  using W = typename S::word;
  using St = BriStage<NV, S>;
  constexpr int SSW = SiteStride<NV, S>::WORDS, SSP = SiteStride<NV, S>::PIECES;
  extern __shared__ uint4 smem_bri[];
  const int R = int(tr.sb);
  W* buf = reinterpret_cast<W*>(smem_bri);
  W* wbuf = buf + (R + 2) * SSW;  // [3][R][9]
  W* lcl = wbuf + ((27 * R + 3) & ~3);  // [R][36] (CLOV), 16-byte aligned

  const uint32_t L = xcd_block(blockIdx.x, gridDim.x, xcd != 0);
  const RowChunk c = order_chunk(g, tr, o, L);
  const int v = threadIdx.x, xl = threadIdx.y;
  const int tid = xl * NV + v, nth = R * NV;
  const int xm = wrap_x(g, c.x0 - 1), xp = wrap_x(g, c.x0 + c.n);

  cpx<T> acc[4][3];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) acc[q][cc] = zero<T>();

  // one row in flight while the previous one is applied (three hops of
  // about a thousand instructions per lane hide the load latency); the
  // request after the last row repeats it, unused, so every load is
  // unconditional and in bounds
  constexpr int CLP = 36 * int(sizeof(W)) / 16;  // 16-byte pieces of a site's clover term
  if constexpr (CLOV) copy_pieces<(CLP + NV - 1) / NV>(lcl, C + size_t(c.row_base + c.x0) * 36, c.n * CLP, tid, nth);
  BriRowRegs<NV, S> q;
  bri_issue<NV, S>(g, c, in, 0, xm, xp, xl, v, tid, nth, q);
#pragma nounroll
  for (int r = 0; r < kBriRows; ++r) {
    bri_commit<NV, S>(c, q, buf, xl, v, tid, nth);
    bri_build<S, T>(g, c, V, r, wbuf, R, tid, nth);
    __syncthreads();
    bri_issue<NV, S>(g, c, in, r + 1 < kBriRows ? r + 1 : kBriRows - 1, xm, xp, xl, v, tid, nth, q);
    bri_row_compute<ADJ, CLOV, NV, S, T>(r, buf, wbuf, lcl, R, xl, v, diag, acc);
    __syncthreads();
  }
  // output through LDS, coalesced 16-byte stores
  {
    W* o = buf + xl * SSW;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int cc = 0; cc < 3; ++cc) S::template store<T>(o + (q * 3 + cc) * NV + v, acc[q][cc]);
  }
  __syncthreads();
  {
    const int xc = xl < c.n ? xl : c.n - 1;
    const u32x4* src = reinterpret_cast<const u32x4*>(buf) + xc * SSP;
    u32x4* dst = reinterpret_cast<u32x4*>(out + size_t(c.row_base + c.x0) * St::SW);
    u32x4 o[St::CH];
#pragma unroll
    for (int j = 0; j < St::CH; ++j) o[j] = src[j * NV + v];
#pragma unroll
    for (int j = 0; j < St::CH; ++j) __builtin_nontemporal_store(o[j], &dst[xc * St::SP + j * NV + v]);
  }
}

// Chunk tiles of the D_B row kernels: the largest by x bz rows (by | Ny,
// bz | Nz) whose spinor rows at one t take at most 1.25 MB, the squarer of
// equal sizes, by >= bz on a tie; DSLASH_BRI_TILE_Y, _Z override (0: t-band
// order).  Each output row stages the 27 rows around it, and in the t-band
// order its +-z rows were a band of planes away, gone from the XCD's L2: 32^4,
// N_v = 12, 23.8 against 24.5 ms.
static ChunkTiles bri_tiles(const Geom& g, int R, long site_bytes) {
  int by, bz;
  pick_tile(g, long((g.n[0] + R - 1) / R) * R * site_bytes, 1280L * 1024, by, bz);
  return make_chunk_tiles(g, R, knobs().bri_tile_y.get(by), knobs().bri_tile_z.get(bz));
}

// CLOVER_OK = false builds the form without the clover term only (C must be null).
template <int NV, class S, class T, bool CLOVER_OK = true>
static hipError_t brillouin_rows_t(bool adj, const Geom& g, int R, int bt, bool xcd, const void* V, const void* in,
                                   void* out, const void* C, double mass, hipStream_t st) {
  using W = typename S::word;
  const RowTraversal tr = make_row_traversal(g, uint32_t(R), uint32_t(bt));
  const ChunkTiles o = bri_tiles(g, R, 12L * NV * long(sizeof(W)));
  const dim3 block(NV, R), grid(tr.rows_plane * uint32_t(g.n[2]) * uint32_t(g.n[3]));
  const size_t lds =
      (size_t(R + 2) * SiteStride<NV, S>::WORDS + size_t(3 * R) * 9 + (C ? 3 + size_t(R) * 36 : 0)) * sizeof(W);
  const T diag = T(mass) + T(15.0 / 8.0);
#define DSL_BK(A, CL)                                                                                        \
  hipLaunchKernelGGL((brillouin_rows_kernel<A, CL, NV, S, T>), grid, block, lds, st, g, tr, o, int(xcd), (const W*)V, \
                     (const W*)in, (W*)out, (const W*)C, diag)
  if constexpr (CLOVER_OK) {
    if (C) {
      if (adj) DSL_BK(true, true); else DSL_BK(false, true);
    } else {
      if (adj) DSL_BK(true, false); else DSL_BK(false, false);
    }
  } else {
    if (C) return hipErrorInvalidValue;
    if (adj) DSL_BK(true, false); else DSL_BK(false, false);
  }
#undef DSL_BK
  return hipGetLastError();
}

// Chunk length of the row-staged kernels (C64; N_v = 4, 8, 12, 16, 24), or 0
// when the configuration is not covered.
static int brillouin_rows_sites(int dtype, const Geom& g) {
  // FP32 only: the FP64 variant would not fit in registers
  const int nv = g.nv;
  if (dtype != DT_C64 || (nv != 4 && nv != 8 && nv != 12 && nv != 16 && nv != 24)) return 0;
  int R = row_sites_default(g.n[0], nv);
  R = knobs().row_sites.get(R);
  if (R > g.n[0]) R = g.n[0];
  // the halo sites (2 * 12 N_v words) take HK 16-byte pieces per thread:
  // R HK >= 12; 64 .. 256 threads
  const int hk = nv > 16 ? 2 : 1;
  if (R * hk < 12 || R * nv > 256 || R * nv < 64) return 0;
  return R;
}

// What DSLASH_ROWS=2 asks for: FP32 storage at N_v = 4, 8, 12, 16, 24 (the clover
// term at N_v = 12 only) where a chunk of one x-row holds its halo, FP64 storage
// at N_v = 12.
bool brillouin_rows_cover(int dtype, const Geom& g, bool clover) {
  if (dtype == DT_C128) return g.nv == 12 && !clover;
  return brillouin_rows_sites(dtype, g) > 0 && !(clover && g.nv != 12);
}

// D_B with the off-axis links built from V inside the row-staged kernel (no W
// array).  FP32 storage at N_v = 4, 8, 12, 16, 24 (the clover term at N_v = 12);
// hipErrorNotSupported otherwise.
hipError_t launch_brillouin_fly(bool adj, int dtype, const Geom& g, const void* V, const void* in, void* out,
                                double mass, hipStream_t st, const void* clover) {
  if (!aligned16(V) || !aligned16(in) || !aligned16(out) || !aligned16(clover)) return hipErrorNotSupported;
  const int R = brillouin_rows_sites(dtype, g);
  if (R == 0 || (clover && g.nv != 12)) return hipErrorNotSupported;
  int bt = 2;
  bt = knobs().tband.get(bt);
  bool xcd = true;
  xcd = knobs().xcd.get(xcd) != 0;
  switch (g.nv) {
    case 4: return brillouin_rows_t<4, C64, float, false>(adj, g, R, bt, xcd, V, in, out, nullptr, mass, st);
    case 8: return brillouin_rows_t<8, C64, float, false>(adj, g, R, bt, xcd, V, in, out, nullptr, mass, st);
    case 16: return brillouin_rows_t<16, C64, float, false>(adj, g, R, bt, xcd, V, in, out, nullptr, mass, st);
    case 24: return brillouin_rows_t<24, C64, float, false>(adj, g, R, bt, xcd, V, in, out, nullptr, mass, st);
  }
  return brillouin_rows_t<12, C64, float>(adj, g, R, bt, xcd, V, in, out, clover, mass, st);
}

}  // namespace dsl
