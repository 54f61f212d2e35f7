"""The operators where a workgroup's sites run across the ends of x-rows: the
row-staged D_W kernels on lattices whose rows hold no chunk of their own, at every
N_v they take, the direct D_W kernel for FP64, the clover term, compressed links
and 16-bit storage, D_B, and D_S, at the edges of their chunks (planes smaller than
a chunk, a last chunk of one site, N_x = 2, columns past one workgroup) against the
FP64 oracle, with the tolerances of the other operator tests."""
import pytest

import synthetic
from oracle import brillouin, clover, compress, evenodd, grad, staggered, wilson
from tests.gpu_util import compare, down, rounded, say, set_knob, up

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1808_05506_amd import dslash as D  # noqa: E402


@pytest.fixture(autouse=True)
def _small_lattices_too(monkeypatch):
    # lattices of a test's size would take the direct kernels
    set_knob(monkeypatch, "DSLASH_FLAT_LANES", "0")


def _fields(dims, nv, dt, seed):
    u = rounded(synthetic.gauge_links(dims, "haar", seed), dt)
    p = rounded(synthetic.wilson_spinor(dims, nv, seed + 1), dt)
    return u, p


# odd extents, rows shorter and longer than a chunk, a plane that is no multiple of
# a chunk, N_x = 2 and 3 (both x neighbours are wraps), a plane of 4 sites, several
# t segments and a last segment of one step
SHAPES = [(7, 5, 3, 4), (13, 6, 2, 5), (37, 3, 2, 3), (2, 9, 3, 4), (3, 11, 2, 9), (2, 2, 3, 17)]


@pytest.mark.parametrize("nv", [2, 3, 4, 5, 7, 10, 12, 13, 17, 19, 22, 23, 24])
@pytest.mark.parametrize("dims", SHAPES)
def test_wilson_chunks_across_rows(dims, nv):
    say(f"case wilson chunks across rows {dims} nv={nv} c64")
    u, p = _fields(dims, nv, "c64", 700 + nv)
    U, P = up(u, "c64"), up(p, "c64")
    for adj in (False, True):
        compare(down(D.apply("wilson", U, P, 0.1, adjoint=adj)), wilson.apply(u, p, 0.1, adj), "c64",
                f"D_W nv={nv} adj={adj}")


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("nv", [4, 5, 8, 10, 12, 16, 24])
@pytest.mark.parametrize("dims", SHAPES[:4])
def test_wilson_16bit_chunks_across_rows(dims, nv, dt):
    say(f"case wilson chunks across rows {dims} nv={nv} {dt}")
    u, p = _fields(dims, nv, dt, 720 + nv)
    out = D.apply("wilson", up(u, dt), up(p, dt), 0.1)
    compare(down(out), wilson.apply(u, p, 0.1, False), dt, f"D_W nv={nv} {dt}")


@pytest.mark.parametrize("dt", ["c64", "bf16"])
@pytest.mark.parametrize("sites", ["9", "16", "21"])
def test_wilson_chunk_lengths(sites, dt, monkeypatch):
    dims, nv = (14, 5, 2, 9), 12
    say(f"case wilson chunk length {sites} {dt}")
    set_knob(monkeypatch, "DSLASH_ROW_SITES", sites)
    u, p = _fields(dims, nv, dt, 740)
    U, P = up(u, dt), up(p, dt)
    for adj in (False, True):
        compare(down(D.apply("wilson", U, P, 0.1, adjoint=adj)), wilson.apply(u, p, 0.1, adj), dt,
                f"D_W R={sites} adj={adj}")


@pytest.mark.parametrize("nv", [1, 2, 6, 7, 12, 25, 130, 260])
@pytest.mark.parametrize("dims", [(5, 3, 2, 4), (2, 7, 3, 3), (10, 4, 5, 2)])
def test_wilson_fp64_flat(dims, nv):
    say(f"case wilson flat {dims} nv={nv} c128")
    u, p = _fields(dims, nv, "c128", 760 + nv)
    U, P = up(u, "c128"), up(p, "c128")
    for adj in (False, True):
        compare(down(D.apply("wilson", U, P, 0.1, adjoint=adj)), wilson.apply(u, p, 0.1, adj), "c128",
                f"D_W nv={nv} adj={adj}")


@pytest.mark.parametrize("dt,nv", [("c128", 7), ("c64", 5), ("c64", 26), ("f16", 9), ("bf16", 12)])
@pytest.mark.parametrize("dims", [(5, 3, 2, 4), (10, 4, 5, 2)])
def test_wilson_flat_clover_and_compressed(dims, dt, nv):
    say(f"case wilson flat clover and compressed {dims} nv={nv} {dt}")
    u, p = _fields(dims, nv, dt, 780 + nv)
    c = rounded(clover.pack(clover.term(u, 1.3)), dt)
    vc = rounded(compress.compress(synthetic.gauge_links(dims, "smooth", 780)), dt)
    U, P, C, VC = up(u, dt), up(p, dt), up(c, dt), up(vc, dt)
    for adj in (False, True):
        compare(down(D.apply("wilson", U, P, 0.1, adjoint=adj, clover=C)),
                wilson.apply(u, p, 0.1, adj) + clover.apply_term(clover.unpack(c), p), dt, f"clover adj={adj}")
        compare(down(D.apply_compressed("wilson", VC, P, 0.1, adjoint=adj)),
                compress.apply("wilson", vc, p, 0.1, adj), dt, f"compressed adj={adj}")


@pytest.mark.parametrize("tile", [("1", "1"), ("2", "2"), ("5", "3"), ("100", "100")])
def test_wilson_flat_tiles(tile, monkeypatch):
    # every order visits every chunk once, also tiles that divide nothing
    dims, nv = (9, 30, 5, 3), 12
    say(f"case wilson flat tile {tile}")
    set_knob(monkeypatch, "DSLASH_FLAT_ZB", tile[0])
    set_knob(monkeypatch, "DSLASH_FLAT_KB", tile[1])
    u, p = _fields(dims, nv, "c128", 790)
    compare(down(D.apply("wilson", up(u, "c128"), up(p, "c128"), 0.1)), wilson.apply(u, p, 0.1, False), "c128",
            f"tile {tile}")


@pytest.mark.parametrize("dt", ["c64", "c128"])
def test_wilson_misaligned_pointers_take_narrow_words(dt):
    # spinors that begin one complex number past a 16-byte border
    dims, nv = (6, 5, 3, 4), 12
    say(f"case wilson misaligned {dt}")
    u, p = _fields(dims, nv, dt, 800)
    U, P = up(u, dt), up(p, dt)
    hold = torch.zeros(P.numel() + 1, dtype=P.dtype, device=P.device)
    Q = hold[1:].view(P.shape)
    Q.copy_(P)
    compare(down(D.apply("wilson", U, Q, 0.1)), wilson.apply(u, p, 0.1, False), dt, f"misaligned {dt}")


# packed rows of 5, 7, 2 and 1 sites
@pytest.mark.parametrize("dims", [(10, 4, 2, 4), (14, 6, 4, 2), (4, 8, 2, 6), (2, 4, 8, 2)])
@pytest.mark.parametrize("dt,nv", [("c64", 12), ("c64", 4), ("bf16", 12), ("f16", 24), ("f16", 16), ("bf16", 8)])
def test_even_odd_hop_chunks_across_rows(dims, dt, nv):
    say(f"case even-odd chunks across rows {dims} nv={nv} {dt}")
    u, p = _fields(dims, nv, dt, 820 + nv)
    ue, uo = up(evenodd.pack(u, 0), dt), up(evenodd.pack(u, 1), dt)
    for parity in (0, 1):
        pin = evenodd.pack(p, 1 - parity)
        for adj in (False, True):
            compare(down(D.eo_hop(ue, uo, up(pin, dt), parity, adjoint=adj)), evenodd.hop_eo(u, pin, parity, adj), dt,
                    f"eo hop parity={parity} adj={adj}")


# blocks of every width (N_v = 26, 40: several of them; odd N_v: words through
# registers), planes smaller than a chunk, chunks of several rows, N_x = 2 and 3,
# lattices that wrap in every direction within a chunk
@pytest.mark.parametrize("dt,nvs", [("c64", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 13, 16, 18, 22, 24, 26, 40]),
                                    ("c128", [1, 2, 4, 5, 6, 7, 8, 10, 12, 17])])
@pytest.mark.parametrize("dims", [(7, 5, 3, 4), (24, 2, 2, 3), (2, 9, 3, 2), (3, 4, 2, 3)])
def test_brillouin_flat(dims, dt, nvs, monkeypatch):
    set_knob(monkeypatch, "DSLASH_BRI_LANES", "0")  # small lattices would take the direct kernel in C64
    v = synthetic.gauge_links(dims, "haar", 840)
    w = rounded(brillouin.build(v), dt)
    c = rounded(clover.pack(clover.term(v, 1.3)), dt)
    W, C = up(w, dt), up(c, dt)
    for nv in nvs:
        say(f"case brillouin flat {dims} nv={nv} {dt}")
        p = rounded(synthetic.wilson_spinor(dims, nv, 841 + nv), dt)
        P = up(p, dt)
        for adj in (False, True):
            ref = brillouin.apply(w, p, 0.1, adj)
            compare(down(D.apply("brillouin", W, P, 0.1, adjoint=adj)), ref, dt, f"D_B nv={nv} adj={adj}")
        ref = brillouin.apply(w, p, 0.1, False) + clover.apply_term(clover.unpack(c), p)
        compare(down(D.apply("brillouin", W, P, 0.1, clover=C)), ref, dt, f"D_B + C nv={nv}")


@pytest.mark.parametrize("dt,nvs", [("c64", [1, 2, 5, 8, 12, 13, 24, 300]), ("c128", [1, 3, 12, 24]),
                                    ("bf16", [1, 2, 4, 6, 12]), ("f16", [3, 4, 10, 12])])
@pytest.mark.parametrize("dims", [(10, 4, 2, 4), (2, 6, 4, 2), (4, 2, 2, 6), (38, 2, 4, 2)])
def test_staggered_flat(dims, dt, nvs, monkeypatch):
    set_knob(monkeypatch, "DSLASH_ROWS", "0")  # rows of whole chunks as well
    u = rounded(synthetic.gauge_links(dims, "haar", 860), dt)
    vc = rounded(compress.compress(synthetic.gauge_links(dims, "smooth", 861)), dt)
    U, VC = up(u, dt), up(vc, dt)
    for nv in nvs:
        say(f"case staggered flat {dims} nv={nv} {dt}")
        p = rounded(synthetic.staggered_spinor(dims, nv, 862 + nv), dt)
        P = up(p, dt)
        for adj in (False, True):
            compare(down(D.apply("staggered", U, P, 0.1, adjoint=adj)), staggered.apply(u, p, 0.1, adj), dt,
                    f"D_S nv={nv} adj={adj}")
        compare(down(D.apply_compressed("staggered", VC, P, 0.1)), compress.apply("staggered", vc, p, 0.1, False), dt,
                f"D_S compressed nv={nv}")


# blocks of every width (several of them at N_v = 26), planes smaller than a chunk,
# wraps in every direction within a chunk, columns past N_v
@pytest.mark.parametrize("dt,nvs", [("c64", [1, 2, 3, 4, 5, 6, 8, 9, 10, 12, 16, 24, 26]), ("c128", [1, 4, 5, 7, 8, 10, 12, 13])])
@pytest.mark.parametrize("dims", [(7, 5, 3, 4), (24, 2, 2, 3), (2, 9, 3, 2)])
def test_brillouin_wgrad_flat(dims, dt, nvs, monkeypatch):
    set_knob(monkeypatch, "DSLASH_BRI_LANES", "0")  # small lattices would take the direct kernel
    W = up(brillouin.build(synthetic.gauge_links(dims, "haar", 880)), dt)
    for nv in nvs:
        say(f"case brillouin W gradient flat {dims} nv={nv} {dt}")
        chi = rounded(synthetic.wilson_spinor(dims, nv, 881 + nv), dt)
        psi = rounded(synthetic.wilson_spinor(dims, nv, 981 + nv), dt)
        gW, _ = D.backward("brillouin", W, up(chi, dt), up(psi, dt), 0.1, need_grad_in=False)
        compare(down(gW), grad.link_grad_brillouin_W(chi, psi), dt, f"G_W nv={nv}")
