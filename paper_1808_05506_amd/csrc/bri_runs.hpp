// Staging of the 27 runs (y + dy, z + dz, t + dt) of a chunk of sites in LDS, half
// the spins of a run at a time: for D_B and its gradient with respect to W.
#pragma once

#include "bri_shape.hpp"
#include "chunks.hpp"
#include "launch.hpp"
#include "rows.hpp"
#include "stencils.hpp"
#include "tiles.hpp"

namespace dsl {

constexpr int kRuns = 27;  // (dy, dz, dt) in {-1, 0, 1}^3 = r % 3, r / 3 % 3, r / 9; run 13 is the own one

// How a run gets into LDS: C128 words or C64 pairs of columns straight from
// global memory, C64 words through registers (odd N_v, pointers off 16 bytes).
enum { BRI_WIDE, BRI_PAIRS, BRI_WORDS };

DSL_HD uint32_t shift_y(uint32_t p, int dy, uint32_t nx, uint32_t nxy) {
  if (dy > 0) return p + nx < nxy ? p + nx : p + nx - nxy;
  if (dy < 0) return p >= nx ? p - nx : p + nxy - nx;
  return p;
}

// Lane l of a wave writes 16 bytes at lds_wave_base + 16 l.
__device__ __forceinline__ void dma16(const void* src, void* lds_wave_base) {
  __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void*)lds_wave_base, 16, 0, 0);
}

// The plane of run r.
DSL_HD uint32_t run_plane(const Geom& g, const FlatChunk<4>& c, int r) {
  const int dt = r / 9 - 1, dz = r / 3 % 3 - 1;
  int z = c.z + dz, t = c.t + dt;
  z = z < 0 ? z + g.n[2] : (z >= g.n[2] ? z - g.n[2] : z);
  t = t < 0 ? t + g.n[3] : (t >= g.n[3] ? t - g.n[3] : t);
  return c.nxy * (uint32_t(z) + uint32_t(g.n[2]) * uint32_t(t));
}

// What a lane stages of each run, fixed over the runs.  Half a run in LDS is
// [6][P + 4][NB]: component, slot (the chunk's sites, then its halo sites), column.
// B: NB columns, P sites, MODE, LANES = NB P, PL = (P + 4) NB.
template <class B, class S>
struct RunStage {
  using W = typename S::word;
  static constexpr int NB = B::NB, P = B::P, PL = B::PL, LANES = B::LANES, WB = int(sizeof(W));
  static constexpr int HP = 6 * PL / 2, NJ = (HP + LANES - 1) / LANES, HK = (24 * NB + LANES - 1) / LANES;
  static constexpr bool PAIRS = B::MODE == BRI_PAIRS, WORDS = B::MODE == BRI_WORDS, WIDE = B::MODE == BRI_WIDE;

  int nv, tid, wave, lane, v, xl, i, v0, vc;
  uint32_t p, site_bytes, comp_bytes;
  // PAIRS: piece tid + j LANES of a half's pairs of columns, its byte offset at dy =
  // 0 and whether y + 1 (bit j) and y - 1 (bit 16 + j) wrap
  uint32_t pj[PAIRS ? NJ : 1], wrap;
  // else the lane's own column and site, and of the halo sites (4 NB lanes of a wave,
  // component by component; or the lane's share of the 24 NB words of a half)
  uint32_t soff, hq, hoff;
  W row[WORDS ? 6 : 1], halo[WORDS ? HK : 1];

  __device__ __forceinline__ void init(const Geom& g, const FlatChunk<4>& c, int col0) {
    nv = g.nv;
    tid = int(threadIdx.x);
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    lane = tid & 63;
    xl = tid / NB;
    v = tid - xl * NB;
    v0 = col0;
    vc = v0 + v < nv ? v0 + v : nv - 1;  // column of the lane
    i = xl < c.n ? xl : c.n - 1;
    p = c.p0 + uint32_t(i);
    site_bytes = uint32_t(12 * nv * WB);
    comp_bytes = uint32_t(nv * WB);
    wrap = 0;
    if constexpr (PAIRS) {
      static_assert(NJ <= 16, "one mask");
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int h = tid + j * LANES, comp = h / (PL / 2), rem = h - comp * (PL / 2);
        const int slot = rem / (NB / 2), col = v0 + 2 * (rem - slot * (NB / 2));
        const uint32_t q = slot < P ? c.p0 + uint32_t(slot < c.n ? slot : c.n - 1) : halo_site(c, slot - P);
        pj[j] = q * site_bytes + uint32_t(comp < 6 ? comp : 5) * comp_bytes + uint32_t(col < nv ? col : nv - 2) * WB;
        wrap |= (q + c.nx >= c.nxy ? 1u : 0u) << j | (q < c.nx ? 1u : 0u) << (16 + j);
      }
    }
    soff = uint32_t(vc * WB);
    const int hs = lane / NB;
    hq = halo_site(c, hs & 3);
    hoff = uint32_t((v0 + lane - hs * NB < nv ? v0 + lane - hs * NB : nv - 1) * WB);
  }

  // LDS slots of x - 1, x, x + 1, times NB, plus the column (x_slots numbers the
  // chunk from 1, halo site k as 0 or P + k)
  __device__ __forceinline__ void slots(const Geom& g, const FlatChunk<4>& c, int (&ps)[3]) const {
    const XSlots xs = x_slots(g, c, P, i);
    ps[0] = (xs.b == 0 ? P : (xs.b > P ? xs.b : xs.b - 1)) * NB + v;
    ps[1] = i * NB + v;
    ps[2] = (xs.f > P ? xs.f : xs.f - 1) * NB + v;
  }

  // Spins 2 h, 2 h + 1 of run r of `in`: requested (WORDS: into registers, else
  // into LDS at dst) ...
  __device__ __forceinline__ void half(const Geom& g, const FlatChunk<4>& c, const W* __restrict__ in, int r, int h,
                                       W* dst) {
    const int dy = r % 3 - 1;
    const uint32_t nx = c.nx, nxy = c.nxy;
    const char* const src =
        reinterpret_cast<const char*>(in) + size_t(run_plane(g, c, r)) * site_bytes + size_t(6 * h) * comp_bytes;
    if constexpr (PAIRS) {
      const uint32_t step = dy > 0 ? nx * site_bytes : (dy < 0 ? 0u - nx * site_bytes : 0u);
      const uint32_t over = dy > 0 ? (nx - nxy) * site_bytes : (dy < 0 ? (nxy - nx) * site_bytes : 0u);
      const uint32_t bits = dy < 0 ? wrap >> 16 : wrap;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        if (tid + j * LANES < HP)
          dma16(src + uint32_t(pj[j] + (bits >> j & 1 ? over : step)), dst + 2 * (j * LANES + wave * 64));
    } else {
      const char* s0 = src + (shift_y(p, dy, nx, nxy) * site_bytes + soff);
#pragma unroll
      for (int j = 0; j < 6; ++j) {
        if constexpr (WIDE) dma16(s0 + size_t(j) * comp_bytes, dst + j * PL + wave * 64);
        else row[j] = *reinterpret_cast<const W*>(s0 + size_t(j) * comp_bytes);
      }
      if constexpr (WIDE) {
        if (lane < 4 * NB) {
          const char* h0 = src + (shift_y(hq, dy, nx, nxy) * site_bytes + hoff);
          for (int j = wave; j < 6; j += (LANES + 63) / 64) dma16(h0 + size_t(j) * comp_bytes, dst + j * PL + P * NB);
        }
      } else {
#pragma unroll
        for (int k = 0; k < HK; ++k) {
          const int w = tid + k * LANES, comp = w / (4 * NB), rem = w - comp * 4 * NB, hk = rem / NB;
          const int col = v0 + rem - hk * NB;
          halo[k] = *reinterpret_cast<const W*>(src + (shift_y(halo_site(c, hk), dy, nx, nxy) * site_bytes +
                                                       uint32_t(comp < 6 ? comp : 5) * comp_bytes +
                                                       uint32_t((col < nv ? col : nv - 1) * WB)));
        }
      }
    }
  }
  // ... and from the registers into LDS.
  __device__ __forceinline__ void half_commit(W* dst) const {
#pragma unroll
    for (int j = 0; j < 6; ++j) dst[j * PL + i * NB + v] = row[j];
#pragma unroll
    for (int k = 0; k < HK; ++k) {
      const int w = tid + k * LANES, comp = w / (4 * NB);
      if (comp < 6) dst[comp * PL + P * NB + w - comp * 4 * NB] = halo[k];
    }
  }
};

}  // namespace dsl
