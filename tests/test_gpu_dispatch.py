"""Which kernel family a call takes, and the families that small test lattices reach
only when a tuning variable asks for them, against the FP64 oracle."""
import pytest

import synthetic
from oracle import brillouin, clover, compress, evenodd, staggered, wilson
from tests.gpu_util import compare, down, rounded, say, set_knob, up

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1808_05506_amd import dslash as D  # noqa: E402

NEVER = "2000000000"  # more lanes than any lattice has: the direct kernel


# The direct and the flat kernel add the hops in different orders, so their bits tell
# which one ran.
@pytest.mark.parametrize("op,dt,nv", [("wilson", "c128", 12), ("wilson", "c64", 26), ("staggered", "c128", 12),
                                      ("staggered", "c64", 12), ("staggered", "c128", 7)])
def test_rows_0_selects_the_direct_kernel(op, dt, nv, monkeypatch):
    dims = (10, 4, 6, 4)
    say(f"case direct by DSLASH_ROWS=0 {op} {dt} nv={nv}")
    gen = synthetic.wilson_spinor if op == "wilson" else synthetic.staggered_spinor
    u, p = rounded(synthetic.gauge_links(dims, "haar", 900), dt), rounded(gen(dims, nv, 901), dt)
    U, P = up(u, dt), up(p, dt)
    set_knob(monkeypatch, "DSLASH_FLAT_LANES", "0")
    flat = D.apply(op, U, P, 0.1)
    set_knob(monkeypatch, "DSLASH_FLAT_LANES", NEVER)
    direct = D.apply(op, U, P, 0.1)
    set_knob(monkeypatch, "DSLASH_FLAT_LANES", "0")
    set_knob(monkeypatch, "DSLASH_ROWS", "0")
    got = D.apply(op, U, P, 0.1)
    assert not torch.equal(flat, direct)
    assert torch.equal(got, direct)
    compare(down(got), (wilson if op == "wilson" else staggered).apply(u, p, 0.1, False), dt, f"{op} direct")


# The flat D_S kernel where rows would hold whole chunks as well (these lattices are too
# small for the row-staged one), at its columns per lane and past one workgroup
@pytest.mark.parametrize("dt,nvs", [("c64", [1, 2, 5, 8, 12, 13, 24, 300]), ("c128", [1, 3, 12, 24]),
                                    ("bf16", [1, 2, 4, 6, 12]), ("f16", [3, 4, 10, 12])])
@pytest.mark.parametrize("dims", [(10, 4, 2, 4), (2, 6, 4, 2), (16, 2, 2, 6), (38, 2, 4, 2)])
def test_staggered_flat(dims, dt, nvs, monkeypatch):
    u = rounded(synthetic.gauge_links(dims, "haar", 910), dt)
    vc = rounded(compress.compress(synthetic.gauge_links(dims, "smooth", 911)), dt)
    U, VC = up(u, dt), up(vc, dt)
    for nv in nvs:
        say(f"case staggered flat {dims} nv={nv} {dt}")
        p = rounded(synthetic.staggered_spinor(dims, nv, 912 + nv), dt)
        P = up(p, dt)
        set_knob(monkeypatch, "DSLASH_FLAT_LANES", NEVER)
        direct = D.apply("staggered", U, P, 0.1)
        set_knob(monkeypatch, "DSLASH_FLAT_LANES", "0")
        differ = False
        for adj in (False, True):
            out = D.apply("staggered", U, P, 0.1, adjoint=adj)
            compare(down(out), staggered.apply(u, p, 0.1, adj), dt, f"D_S nv={nv} adj={adj}")
            differ = differ or (not adj and not torch.equal(out, direct))
        assert differ or dt in ("bf16", "f16")  # (16-bit stores round the difference away)
        compare(down(D.apply_compressed("staggered", VC, P, 0.1)), compress.apply("staggered", vc, p, 0.1, False), dt,
                f"D_S compressed nv={nv}")


# Rows of 16 sites add the diagonal term first, rows of 20, 24 and 28 last (C64); the
# blocks of one row take chunks of one x-row or across row ends as their lanes allow
@pytest.mark.parametrize("dt", ["c64", "bf16"])
@pytest.mark.parametrize("nx", [20, 24, 28])
def test_columns_do_not_depend_on_the_block_size(dt, nx, monkeypatch):
    # at a fixed t-segment length and in one buffer scheme, a block of 24 columns equals
    # its blocks of 4, 8, 12 and (the first) 16 columns bit for bit
    dims = (nx, 4, 4, 16)
    say(f"case block-size invariance {dims} {dt}")
    u = rounded(synthetic.gauge_links(dims, "haar", 920), dt)
    p = rounded(synthetic.wilson_spinor(dims, 24, 921), dt)
    U, P = up(u, dt), up(p, dt)
    set_knob(monkeypatch, "DSLASH_ROWS", "1")
    set_knob(monkeypatch, "DSLASH_TSTEPS", "8")
    set_knob(monkeypatch, "DSLASH_MARCH_PP", "3" if dt == "c64" else "2")
    axis = -1 if dt == "c64" else -2
    for adj in (False, True):
        full = D.apply("wilson", U, P, 0.1, adjoint=adj)
        compare(down(full), wilson.apply(u, p, 0.1, adj), dt, f"D_W {dims} adj={adj}")
        for k in (4, 8, 12, 16):
            for c0 in range(0, 24 - k + 1, k):
                sl = [slice(None)] * full.dim()
                sl[axis] = slice(c0, c0 + k)
                part = D.apply("wilson", U, P[tuple(sl)].contiguous(), 0.1, adjoint=adj)
                assert torch.equal(part, full[tuple(sl)]), (k, c0)


# The row-staged kernels on compressed links, which lattices of a test's size take only
# when asked (DSLASH_ROWS=2: those kernels or an error): D_W marches in chunks of one
# x-row (16) and, asked for chunks of 13, across row ends; D_S in rows of 16 and 13 + 13
@pytest.mark.parametrize("op,dt", [("wilson", "c64"), ("wilson", "bf16"), ("wilson", "f16"), ("staggered", "c64"),
                                   ("staggered", "c128")])
@pytest.mark.parametrize("dims", [(16, 4, 2, 8), (26, 2, 2, 4)])
def test_compressed_links_by_rows(op, dt, dims, monkeypatch):
    nv = 12
    say(f"case compressed rows {op} {dims} {dt}")
    vc = rounded(compress.compress(synthetic.gauge_links(dims, "smooth", 930)), dt)
    gen = synthetic.wilson_spinor if op == "wilson" else synthetic.staggered_spinor
    p = rounded(gen(dims, nv, 931), dt)
    VC, P = up(vc, dt), up(p, dt)
    set_knob(monkeypatch, "DSLASH_ROWS", "2")
    for adj in (False, True):
        ref = compress.apply(op, vc, p, 0.1, adj)
        compare(down(D.apply_compressed(op, VC, P, 0.1, adjoint=adj)), ref, dt, f"{op} compressed adj={adj}")
    if op == "wilson":
        set_knob(monkeypatch, "DSLASH_ROW_SITES", "13")
        compare(down(D.apply_compressed(op, VC, P, 0.1)), compress.apply(op, vc, p, 0.1, False), dt, "13 sites")


# D_B on stored links by the kernel that stages the runs, required, and by the direct one
@pytest.mark.parametrize("dims", [(16, 3, 2, 4), (12, 2, 3, 3), (24, 3, 2, 2)])
def test_brillouin_staged_and_direct(dims, monkeypatch):
    nv, dt = 12, "c64"
    say(f"case brillouin staged and direct {dims}")
    w = rounded(brillouin.build(synthetic.gauge_links(dims, "haar", 940)), dt)
    p = rounded(synthetic.wilson_spinor(dims, nv, 941), dt)
    W, P = up(w, dt), up(p, dt)
    out = {}
    for rows in ("2", "0"):
        set_knob(monkeypatch, "DSLASH_ROWS", rows)
        out[rows] = D.apply("brillouin", W, P, 0.1)
        compare(down(out[rows]), brillouin.apply(w, p, 0.1, False), dt, f"D_B DSLASH_ROWS={rows}")
    assert not torch.equal(out["2"], out["0"])


# The even-odd hop by rows, required, against the direct one; packed rows of 27, 16 and 24
@pytest.mark.parametrize("dims,nv", [((54, 2, 4, 2), 12), ((32, 4, 4, 4), 8), ((48, 4, 2, 2), 4)])
def test_even_odd_hop_by_rows_and_direct(dims, nv, monkeypatch):
    dt = "c64"
    say(f"case even-odd rows and direct {dims} nv={nv}")
    u = rounded(synthetic.gauge_links(dims, "haar", 950), dt)
    p = rounded(synthetic.wilson_spinor(dims, nv, 951), dt)
    Ue, Uo = up(evenodd.pack(u, 0), dt), up(evenodd.pack(u, 1), dt)
    pe = evenodd.pack(p, 0)
    out = {}
    for rows in ("2", "0"):
        set_knob(monkeypatch, "DSLASH_ROWS", rows)
        out[rows] = D.eo_hop(Ue, Uo, up(pe, dt), 1)
        compare(down(out[rows]), evenodd.hop_eo(u, pe, 1, False), dt, f"eo hop DSLASH_ROWS={rows}")
    assert not torch.equal(out["2"], out["0"])


# Spinors that begin one complex number past a 16-byte border: one column a lane
@pytest.mark.parametrize("dt,op", [("c64", "wilson"), ("c64", "staggered"), ("bf16", "wilson"), ("f16", "staggered")])
def test_fields_off_a_16_byte_border(dt, op, monkeypatch):
    dims, nv = (6, 4, 2, 4), 12
    say(f"case off a 16-byte border {op} {dt}")
    set_knob(monkeypatch, "DSLASH_FLAT_LANES", "0")
    u = rounded(synthetic.gauge_links(dims, "haar", 960), dt)
    gen = synthetic.wilson_spinor if op == "wilson" else synthetic.staggered_spinor
    p = rounded(gen(dims, nv, 961), dt)
    U, P = up(u, dt), up(p, dt)
    step = 1 if dt == "c64" else 2  # (16-bit fields hold pairs)
    Q, out = (torch.zeros(P.numel() + step, dtype=P.dtype, device=P.device)[step:].view(P.shape) for _ in range(2))
    Q.copy_(P)
    assert Q.data_ptr() % 16 and out.data_ptr() % 16
    ref = (wilson if op == "wilson" else staggered).apply(u, p, 0.1, False)
    compare(down(D.apply(op, U, Q, 0.1, out=out)), ref, dt, f"{op} off a border")


# D_B in chunks of 16 sites (bri_short_chunks): 16 + 6 of a plane of 22, 4 live sites of 16
@pytest.mark.parametrize("dims", [(11, 2, 20, 20), (2, 2, 28, 28)])
def test_brillouin_short_chunks(dims, monkeypatch):
    nv, dt = 12, "c64"
    say(f"case brillouin short chunks {dims}")
    set_knob(monkeypatch, "DSLASH_BRI_LANES", "0")
    u = synthetic.gauge_links(dims, "haar", 970)
    w, c = rounded(brillouin.build(u), dt), rounded(clover.pack(clover.term(u, 1.0)), dt)
    p = rounded(synthetic.wilson_spinor(dims, nv, 971), dt)
    W, P, C = up(w, dt), up(p, dt), up(c, dt)
    for adj in (False, True):
        ref = brillouin.apply(w, p, 0.1, adj)
        compare(down(D.apply("brillouin", W, P, 0.1, adjoint=adj)), ref, dt, f"D_B short chunks adj={adj}")
        ref = ref + clover.apply_term(clover.unpack(c), p)
        compare(down(D.apply("brillouin", W, P, 0.1, adjoint=adj, clover=C)), ref, dt, f"D_B + C short chunks adj={adj}")
