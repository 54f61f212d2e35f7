"""Launch shapes, workgroup orders and dispatch rules of the kernels, on the host: the
headers that hold them are compiled into a small library without device code, which
also calls the launchers of libdslash.so where they return before any launch."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else shutil.which("hipcc")

LIB = os.path.join(ROOT, "paper_1808_05506_amd", "libdslash.so")

pytestmark = pytest.mark.skipif(HIPCC is None or not os.path.exists(LIB), reason="no hipcc or libdslash.so not built")

C64, C128, BF16, F16 = 0, 1, 2, 3
NOT_SUPPORTED = 801  # hipErrorNotSupported: left to the direct kernel

SOURCE = r"""
#include "bri_shape.hpp"
#include "flat_order.hpp"
#include "flat_rule.hpp"
#include "rows_shape.hpp"
#include <vector>
using namespace dsl;

static Geom geom(const int* d, int nv) {
  Geom g{};
  for (int i = 0; i < 4; ++i) g.n[i] = d[i];
  g.stride[0] = 1;
  for (int i = 1; i < 4; ++i) g.stride[i] = g.stride[i - 1] * d[i - 1];
  g.vol = uint32_t(d[0]) * d[1] * d[2] * d[3];
  g.nv = nv;
  g.dx = FastDiv::make(d[0]);
  g.dy = FastDiv::make(d[1]);
  g.dz = FastDiv::make(d[2]);
  return g;
}

extern "C" {
void reload() { knob_store() = read_knobs(); }

// out: P, chunks, zb, kb, grid x, grid y, block
void flat(const int* d, int nv, int comps, int wb, int vw, long long* out) {
  const FlatShape s = flat_shape(geom(d, nv), comps, wb, vw, 9, false);
  const long long v[] = {s.o.P, s.o.chunks, s.o.zb, s.o.kb, s.grid.x, s.grid.y, s.block.x};
  for (int i = 0; i < 7; ++i) out[i] = v[i];
}

// how many (chunk, z, t) the order with these tiles does not visit exactly once
int flat_missed(const int* d, int nv, int comps, int wb, int vw) {
  const Geom g = geom(d, nv);
  const FlatShape s = flat_shape(g, comps, wb, vw, 9, false);
  std::vector<int> seen(size_t(s.o.chunks) * d[2] * d[3], 0);
  int bad = 0;
  for (uint32_t L = 0; L < s.grid.x; ++L) {
    const FlatSite f = flat_site(g, s.o, L);
    const long plane = long(d[0]) * d[1];
    if (f.p0 % s.o.P || long(f.p0) >= plane || f.z < 0 || f.z >= d[2] || f.t < 0 || f.t >= d[3] || f.n < 1 ||
        long(f.p0) + f.n > plane) {
      ++bad;
      continue;
    }
    ++seen[(size_t(f.t) * d[2] + f.z) * s.o.chunks + f.p0 / s.o.P];
  }
  for (int n : seen) bad += n != 1;
  return bad;
}

// out: R, halo sites, diagonal term last; 0 where the row-staged D_W march does not apply
int rows(int dtype, const int* d, int nv, int pp, int* out) {
  const bool any = nv != 4 && nv != 8 && nv != 12 && nv != 16 && nv != 24;
  bool late = false;
  const bool ok = rows_shape(geom(d, nv), dtype, pp, any, false, out[0], out[1], late);
  out[2] = late;
  return ok;
}

// out: chunks, planes of a tile of the one-row order; returns the chunks per plane
int one_row(const int* d, int R, int site_bytes, int* out) {
  const FlatMarch m = one_row_order(geom(d, 1), R, site_bytes);
  out[0] = int(m.kb);
  out[1] = int(m.zb);
  return int(m.chunks);
}

int wilson_pays(int dtype, const int* d, int nv, int clover, int compressed) {
  return wilson_flat_pays(dtype, geom(d, nv), flat_vw(dtype, nv, true), clover, compressed);
}
int staggered_pays(int dtype, const int* d, int nv, int compressed) {
  return staggered_flat_pays(dtype, geom(d, nv), flat_vw(dtype, nv, true), compressed);
}
int brillouin_pays(int dtype, const int* d, int nv) { return brillouin_flat_pays(dtype, geom(d, nv)); }
int wgrad_pays(int dtype, const int* d, int nv) { return brillouin_wgrad_pays(dtype, geom(d, nv)); }
int brillouin_block(int dtype, int nv) { return bri_block(dtype, nv); }
int brillouin_short(const int* d, int nv, int pairs) {
  return bri_short_chunks(geom(d, nv), bri_block(DT_C64, nv), pairs != 0);
}

// The launchers on null fields, for calls that they refuse before they launch.
int launch_wilson(int dtype, const int* d, int nv, int clover, int compressed) {
  static float c;
  return launch_wilson_flat(false, dtype, geom(d, nv), nullptr, nullptr, nullptr, 0.1, nullptr, clover ? &c : nullptr,
                            compressed != 0);
}
int launch_staggered(int dtype, const int* d, int nv) {
  return launch_staggered_flat(false, dtype, geom(d, nv), nullptr, nullptr, nullptr, 0.1, nullptr, false);
}
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    d = tmp_path_factory.mktemp("shapes")
    src, lib = d / "shapes.cpp", d / "shapes.so"
    src.write_text(SOURCE)
    csrc = os.path.join(ROOT, "paper_1808_05506_amd", "csrc")
    subprocess.run([HIPCC, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", csrc,
                    str(src), "-x", "none", LIB, "-Wl,-rpath," + os.path.dirname(LIB), "-o", str(lib)],
                   check=True, capture_output=True, timeout=300)
    return ctypes.CDLL(str(lib))


def _dims(d):
    return (ctypes.c_int * 4)(*d)


def _flat(lib, dims, nv, comps, wb, vw):
    out = (ctypes.c_longlong * 7)()
    lib.flat(_dims(dims), nv, comps, wb, vw, out)
    return dict(zip(("P", "chunks", "zb", "kb", "gx", "gy", "block"), out))


@pytest.fixture
def knob(shapes, monkeypatch):
    def set_(**kw):
        for k, v in kw.items():
            monkeypatch.setenv(k, v)
        shapes.reload()
    yield set_
    monkeypatch.undo()
    shapes.reload()


# unset, the whole range (0, text that is no number, negative, too large) and tiles
# that divide nothing: the tile is never empty, and every chunk is visited once
@pytest.mark.parametrize("zb", [None, "0", "-1", "none", "2", "2147483647", "-2147483648"])
@pytest.mark.parametrize("kb", [None, "0", "-3", "3", "2147483647"])
def test_flat_tiles_are_never_empty(shapes, knob, zb, kb):
    knob(**{k: v for k, v in (("DSLASH_FLAT_ZB", zb), ("DSLASH_FLAT_KB", kb)) if v is not None})
    for dims, nv, comps, wb, vw in [((9, 30, 5, 3), 12, 12, 16, 1), ((4, 4, 4, 4), 4, 3, 8, 2), ((34, 34, 3, 2), 6, 12, 4, 2)]:
        s = _flat(shapes, dims, nv, comps, wb, vw)
        assert 1 <= s["zb"] <= dims[2] and 1 <= s["kb"] <= s["chunks"], (s, dims)
        assert shapes.flat_missed(_dims(dims), nv, comps, wb, vw) == 0, (s, dims)


# (site, column) lanes past HIP's 2^32 work-items per grid dimension go to the direct
# kernel, which spreads them over two dimensions
@pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="host only: a shape not refused would be launched")
@pytest.mark.parametrize("dtype,dims,nv", [(BF16, (96, 96, 96, 80), 63), (F16, (64, 64, 64, 64), 514), (C64, (64, 64, 64, 64), 257)])
def test_flat_grids_past_the_launch_limit_are_refused(shapes, dtype, dims, nv):
    vol = dims[0] * dims[1] * dims[2] * dims[3]
    assert vol * nv // (2 if nv % 2 == 0 else 1) >= 2 ** 32
    assert shapes.launch_staggered(dtype, _dims(dims), nv) == NOT_SUPPORTED


# DSLASH_ROWS=0: the direct kernels, not the flat ones
@pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="host only: a call not refused would be launched")
@pytest.mark.parametrize("dtype,nv", [(C64, 5), (C64, 12), (C64, 26), (C128, 7), (C128, 12), (BF16, 12), (F16, 16)])
def test_rows_0_leaves_every_call_to_the_direct_kernels(shapes, dtype, nv, monkeypatch):
    monkeypatch.setenv("DSLASH_ROWS", "0")
    shapes.dslash_reload_tuning()
    try:
        d = _dims((32, 32, 32, 32))
        assert shapes.launch_staggered(dtype, d, nv) == NOT_SUPPORTED
        for clover, compressed in [(0, 0), (1, 0), (0, 1)]:
            assert shapes.launch_wilson(dtype, d, nv, clover, compressed) == NOT_SUPPORTED
    finally:
        monkeypatch.undo()
        shapes.dslash_reload_tuning()


PP = {C64: 3, BF16: 2, F16: 0}


def _rows(lib, dtype, dims, nv):
    out = (ctypes.c_int * 3)()
    return tuple(out) if lib.rows(dtype, _dims(dims), nv, PP[dtype], out) else None


@pytest.mark.parametrize("dtype", [C64, BF16, F16])
@pytest.mark.parametrize("nx", list(range(2, 66)))
def test_the_diagonal_term_does_not_depend_on_the_block_size(shapes, dtype, nx):
    # whether it is added first or last: the same for each block size that has rows at all
    late = {s[2] for s in (_rows(shapes, dtype, (nx, 12, 12, 12), nv) for nv in (4, 8, 12, 16, 24)) if s}
    assert len(late) <= 1
    # (a chunk of one x-row adds it last in C64 only)
    assert late <= ({0, 1} if dtype == C64 else {0})


# Chunk and halo sites, us so and with the shape in brackets (one MI355X)
@pytest.mark.parametrize("dtype,dims,nv,want", [
    (C64, (24, 24, 24, 48), 4, (24, 2)),   # 218 (61, 4: 296; 16, 4: 242)
    (C64, (28, 28, 28, 28), 4, (28, 2)),   # 195 (61, 4: 286; 16, 4: 244)
    (C64, (20, 20, 20, 20), 4, (16, 4)),   # 69 (58, 4: 80; 20, 2: 73)
    (C64, (34, 18, 18, 24), 4, (16, 4)),   # 110 (61, 4: 143)
    (BF16, (24, 24, 24, 48), 4, (16, 4)),  # 126 (64, 4: 154; 24, 2: 162)
    (F16, (14, 13, 12, 16), 4, (16, 4)),   # 15.9 (61, 4: 19.1)
    (BF16, (14, 13, 12, 16), 24, (10, 4)),  # 47 (8, 4: 62)
    (BF16, (34, 18, 18, 24), 24, (10, 4)),  # 304 (8, 4: 346)
    (C64, (16, 16, 16, 32), 12, (16, 2)),
    (C64, (16, 16, 16, 32), 24, (8, 4)),   # 187 (8, 2: 193)
    (BF16, (16, 16, 16, 32), 24, (8, 2)),  # 129 (8, 4: 164)
])
def test_rows_take_the_faster_chunk(shapes, dtype, dims, nv, want):
    assert _rows(shapes, dtype, dims, nv)[:2] == want


# The even-odd hop in C64, us with tiles that divide the lattice and with larger ones:
# 32^4, N_v = 4 193 and 204; 24^3 x 48, N_v = 12 272 and 294
@pytest.mark.parametrize("packed,R,nv", [((16, 32, 32, 32), 16, 4), ((16, 32, 32, 32), 16, 8), ((12, 24, 24, 48), 12, 12)])
def test_one_row_tiles_divide_the_lattice(shapes, packed, R, nv):
    out = (ctypes.c_int * 2)()
    chunks = shapes.one_row(_dims(packed), R, 12 * nv * 8, out)
    assert chunks % out[0] == 0 and packed[2] % out[1] == 0, list(out)
    assert out[0] * out[1] * R * 12 * nv * 8 <= 1280 * 1024


# D_B by the kernel that stages the runs, and by the direct one (us, one MI355X)
@pytest.mark.parametrize("dtype,dims,nv,us,direct", [
    (C128, (4, 4, 4, 4), 12, 73, 59), (C128, (4, 4, 4, 4), 24, 72, 59), (C128, (8, 8, 8, 8), 3, 117, 97),
    (C128, (16, 8, 8, 16), 4, 128, 106), (C128, (12, 12, 12, 12), 4, 166, 195), (C128, (12, 12, 12, 16), 2, 259, 168),
    (C128, (12, 12, 12, 16), 4, 273, 211), (C128, (14, 13, 12, 16), 4, 286, 336), (C128, (16, 16, 16, 16), 2, 362, 494),
    (C128, (18, 14, 20, 26), 2, 780, 1039), (C128, (16, 16, 16, 32), 12, 1317, 2183), (C128, (8, 8, 8, 8), 5, 86, 106),
    (C64, (8, 8, 8, 8), 12, 73, 69), (C64, (12, 12, 12, 16), 4, 155, 101), (C64, (12, 12, 12, 12), 5, 151, 106),
    (C64, (12, 12, 12, 16), 5, 152, 167), (C64, (16, 16, 16, 32), 3, 355, 670), (C64, (12, 12, 12, 24), 1, 250, 172),
    (C64, (32, 32, 32, 32), 12, 6200, 10000),
])
def test_brillouin_takes_the_faster_kernel(shapes, dtype, dims, nv, us, direct):
    assert bool(shapes.brillouin_pays(dtype, _dims(dims), nv)) == (us < direct)


# the gradient with respect to W
@pytest.mark.parametrize("dtype,dims,nv,us,direct", [
    (C128, (4, 4, 4, 4), 4, 147, 6.5), (C128, (4, 4, 4, 4), 20, 746, 25), (C128, (6, 6, 6, 8), 12, 153, 83),
    (C128, (6, 6, 6, 8), 24, 332, 184), (C128, (8, 8, 8, 8), 12, 175, 213), (C128, (8, 8, 8, 8), 24, 372, 461),
    (C128, (8, 8, 8, 8), 8, 163, 115), (C128, (12, 8, 8, 8), 5, 176, 136), (C128, (12, 8, 8, 8), 8, 181, 206),
    (C128, (16, 16, 16, 32), 3, 1955, 2032), (C128, (16, 16, 16, 32), 12, 4092, 7810),
    (C64, (6, 6, 6, 8), 48, 175, 121), (C64, (3, 9, 9, 9), 32, 162, 106), (C64, (8, 8, 8, 8), 20, 165, 131),
    (C64, (8, 8, 8, 8), 24, 105, 150), (C64, (12, 8, 8, 8), 12, 97, 125), (C64, (16, 16, 16, 32), 12, 970, 3100),
])
def test_wgrad_takes_the_faster_kernel(shapes, dtype, dims, nv, us, direct):
    want = us < direct and not (dtype == C128 and nv < 4)  # (below four columns it is the slower one elsewhere)
    assert bool(shapes.wgrad_pays(dtype, _dims(dims), nv)) == want


@pytest.mark.parametrize("dtype,nv,width", [(C128, 4, 4), (C128, 5, 6), (C128, 8, 8), (C128, 12, 12), (C128, 14, 8), (C128, 18, 12),
                                            (C128, 20, 12), (C128, 28, 8), (C64, 4, 4), (C64, 5, 6), (C64, 12, 12), (C64, 24, 24),
                                            (C64, 28, 16), (C64, 40, 8), (C64, 48, 24)])
def test_brillouin_blocks_cost_least(shapes, dtype, nv, width):
    assert shapes.brillouin_block(dtype, nv) == width


# The flat kernels and the direct one (us on inputs that change, one MI355X)
@pytest.mark.parametrize("dtype,dims,nv,compressed,us,direct", [
    (BF16, (20, 20, 20, 20), 4, 0, 28.3, 18.9), (F16, (24, 24, 24, 48), 4, 0, 93.4, 87.2),
    (BF16, (18, 14, 20, 26), 2, 0, 17.4, 13.0), (BF16, (32, 32, 32, 32), 2, 0, 91.6, 104.1),
    (BF16, (20, 20, 20, 20), 1, 0, 17.7, 16.4), (BF16, (24, 24, 24, 24), 12, 0, 55.0, 87.0),
    (C64, (20, 20, 20, 40), 2, 0, 91.8, 74.8), (C64, (24, 24, 24, 24), 2, 0, 71.9, 79.9),
    (C64, (12, 12, 12, 24), 4, 0, 11.4, 14.1), (BF16, (18, 14, 20, 26), 1, 1, 12.5, 8.7),
    (BF16, (24, 24, 24, 48), 3, 1, 62.4, 60.6), (C64, (16, 16, 16, 32), 1, 1, 18.1, 15.1),
    (C64, (20, 20, 20, 40), 2, 1, 43.3, 41.2), (C64, (16, 16, 16, 16), 4, 1, 11.1, 12.8),
    (C128, (8, 8, 8, 8), 4, 0, 5.8, 6.2), (C128, (16, 16, 16, 16), 1, 0, 26.3, 18.9),
])
def test_staggered_flat_takes_what_it_is_faster_at(shapes, dtype, dims, nv, compressed, us, direct):
    assert bool(shapes.staggered_pays(dtype, _dims(dims), nv, compressed)) == (us < direct)


@pytest.mark.parametrize("dtype,dims,nv,clover,compressed,us,direct", [
    (BF16, (16, 8, 8, 16), 32, 0, 0, 29.4, 24.7), (BF16, (8, 8, 8, 8), 7, 0, 0, 9.1, 8.4),
    (F16, (8, 8, 8, 8), 7, 0, 0, 9.0, 10.7), (BF16, (17, 13, 11, 19), 7, 0, 0, 35.7, 39.5),
    (BF16, (16, 8, 8, 16), 9, 0, 0, 18.1, 17.1), (BF16, (21, 15, 13, 27), 2, 0, 0, 29.7, 39.1),
    (BF16, (12, 12, 12, 16), 6, 0, 0, 18.2, 22.1), (BF16, (12, 12, 12, 12), 3, 1, 0, 21.7, 16.2),
    (BF16, (17, 13, 11, 19), 24, 1, 0, 76.9, 65.1), (BF16, (16, 16, 16, 16), 24, 1, 0, 103.8, 86.6),
    (C128, (18, 14, 20, 26), 4, 1, 0, 164.7, 148.1), (C128, (24, 24, 24, 48), 12, 0, 0, 1050, 1906),
    (F16, (17, 13, 11, 19), 28, 0, 1, 73.1, 66.9), (BF16, (20, 20, 20, 20), 20, 0, 1, 173.2, 199.4),
    (C64, (21, 16, 17, 33), 4, 0, 1, 106, 85), (C64, (16, 16, 16, 32), 1, 0, 0, 66.4, 26.6),
])
def test_wilson_flat_takes_what_it_is_faster_at(shapes, dtype, dims, nv, clover, compressed, us, direct):
    assert bool(shapes.wilson_pays(dtype, _dims(dims), nv, clover, compressed)) == (us < direct)


def test_flat_tiles_of_few_planes(shapes):
    # FP64, N_v = 24 on 64 x 4 x 4 x 16: 61 us in tiles of 2 planes x 13 of 26 chunks, 84 in 3 x 7
    s = _flat(shapes, (64, 4, 4, 16), 24, 12, 16, 1)
    assert (s["zb"], s["kb"], s["chunks"]) == (2, 13, 26)
    s = _flat(shapes, (24, 24, 24, 48), 12, 12, 16, 1)  # 1050 us, 3 planes x 7 of 28 chunks
    assert (s["zb"], s["kb"], s["chunks"]) == (3, 7, 28)


# D_B in chunks of 16 sites: 1024 of their workgroups are resident, 768 of those of 21
@pytest.mark.parametrize("dims,nv,pairs,short", [
    ((64, 4, 4, 16), 12, 1, 1), ((16, 8, 8, 16), 12, 1, 1), ((2, 2, 28, 28), 12, 1, 1), ((11, 2, 20, 20), 12, 1, 1),
    ((2, 2, 28, 28), 12, 0, 0), ((2, 2, 28, 28), 10, 1, 0),      # words through registers, other blocks
    ((16, 8, 8, 12), 12, 1, 0), ((2, 2, 24, 32), 12, 1, 0),      # those of 21 are resident too
    ((16, 8, 8, 17), 12, 1, 0), ((32, 32, 32, 32), 12, 1, 0),    # not all of 16
])
def test_brillouin_short_chunks_save_a_round(shapes, dims, nv, pairs, short):
    assert shapes.brillouin_short(_dims(dims), nv, pairs) == short
