"""GPU parity of the operators (through the C ABI) against the FP64 oracle.

Shapes span several workgroups with a ragged last one, the L = 2 extents
where x + mu and x - mu coincide, a non-cubic lattice and the Ls values of
the workloads.  Bars: FP64 relative 2-norm error <= 1e-13; FP32 <= 1e-6 and
FP16 + scale <= 2e-3 against the oracle applied to the stored input.
"""

import numpy as np
import pytest

import synth
from oracle import codec, lattice as L
from tests.gpu_util import M5, MF, make_operator, pack, rel, rel_per_rhs, unpack

pytestmark = pytest.mark.gpu

SHAPES = [((2, 2, 2, 2), 4), ((4, 4, 4, 4), 8), ((4, 4, 6, 8), 5), ((6, 4, 2, 4), 12)]
F64, F32, F16S = 0, 1, 2
EVEN, ODD, BOTH = 0, 1, 2


def fields(dims, Ls, nrhs, seed):
    return synth.gaussian_fermion_batch(dims, Ls, nrhs, seed)


def stored(op, nat, parity):
    """What the handle's precision stores for ``nat`` (round trip through pack)."""
    return unpack(op, pack(op, nat, parity), nat.shape[0], parity)


@pytest.mark.parametrize("prec", [F64, F32, F16S])
@pytest.mark.parametrize("dims,Ls", SHAPES[:3])
def test_pack_unpack_roundtrip(dims, Ls, prec):
    op, _ = make_operator(dims, Ls, prec=prec)
    nat = fields(dims, Ls, 2, seed=1)
    back = unpack(op, pack(op, nat, BOTH), 2, BOTH)
    if prec == F64:
        assert np.array_equal(back, nat)
    elif prec == F32:
        assert np.array_equal(back, nat.astype(np.complex64).astype(np.complex128))
    else:
        q, s = codec.encode(nat)
        assert np.array_equal(back, codec.decode(q, s))
    # one parity only: the other parity of the output is untouched (zero)
    even = unpack(op, pack(op, nat, EVEN), 2, EVEN)
    expect = np.stack([L.on_parity(back[k], EVEN) for k in range(2)])
    assert np.array_equal(even, expect)


@pytest.mark.parametrize("dims,Ls", SHAPES)
@pytest.mark.parametrize("dagger", [False, True])
@pytest.mark.parametrize("out_parity", [EVEN, ODD])
def test_dhop_f64(dims, Ls, dagger, out_parity):
    nrhs = 3 if Ls <= 8 else 1
    op, U = make_operator(dims, Ls, eps=0.5, seed=2)
    nat = fields(dims, Ls, nrhs, seed=3)
    inp = pack(op, nat, 1 - out_parity)
    out = op.new_field(nrhs)
    op.dhop(inp, out, out_parity, nrhs, dagger)
    got = unpack(op, out, nrhs, out_parity)
    exp = np.stack([L.on_parity(L.dhop(U, L.on_parity(nat[k], 1 - out_parity), dagger), out_parity) for k in range(nrhs)])
    assert rel_per_rhs(got, exp) < 1e-13


def _q(field):
    """The FP16 + scale storage of a natural-layout field, decoded (the oracle's codec)."""
    return codec.decode(*codec.encode(field))


# FP16 + scale against an oracle that rounds to the storage format at the points where the
# kernels store (their output, and the intermediate fields of M_pc^dag M_pc): the kernel adds
# in FP32, so a stored component differs from the oracle's only where the FP32 and FP64 values
# fall on different sides of an FP16 rounding boundary -- one quantum (at most 2^-11 of the
# spinor's largest component) in a small fraction of the components.  One stored rounding
# (D_hop) then leaves a relative 2-norm difference ~ sqrt(fraction) * 2^-11 (measured 4e-6 to
# 1e-5); in M_pc^dag M_pc each of the four roundings' flips is carried through the later
# passes (measured 4.9e-5).  The unrounded comparisons see the rounding itself (1.8e-4 and
# 2.5e-4 measured, bars 2e-3 and 3e-3).
QUANTISED_TOL_HOP = 1e-4
QUANTISED_TOL_MDAGM = 2e-4


@pytest.mark.parametrize("prec,tol", [(F32, 1e-6), (F16S, 2e-3)])
@pytest.mark.parametrize("dims,Ls", SHAPES[1:3])
def test_dhop_low_precision(dims, Ls, prec, tol):
    op, U = make_operator(dims, Ls, eps=0.5, seed=2, prec=prec)
    nat = fields(dims, Ls, 2, seed=4)
    inp = pack(op, nat, EVEN)
    src = unpack(op, inp, 2, EVEN)  # the values the kernel actually reads
    for dagger in (False, True):
        out = op.new_field(2)
        op.dhop(inp, out, ODD, 2, dagger)
        got = unpack(op, out, 2, ODD)
        exp = np.stack([L.on_parity(L.dhop(U, src[k], dagger), ODD) for k in range(2)])
        assert rel_per_rhs(got, exp) < tol
        if prec == F16S:
            assert rel_per_rhs(got, np.stack([_q(e) for e in exp])) < QUANTISED_TOL_HOP


@pytest.mark.parametrize("dims,Ls", SHAPES)
@pytest.mark.parametrize("dagger", [False, True])
def test_m5d_and_inverse_f64(dims, Ls, dagger):
    op, U = make_operator(dims, Ls, seed=5, mf=0.03)
    nat = fields(dims, Ls, 2, seed=6)
    inp = pack(op, nat, EVEN)
    out = op.new_field(2)
    op.m5d(inp, out, 2, dagger)
    got = unpack(op, out, 2, EVEN)
    exp = np.stack([L.m5d(L.on_parity(nat[k], EVEN), M5, 0.03, dag=dagger) for k in range(2)])
    assert rel_per_rhs(got, exp) < 1e-14
    op.m5d_inv(inp, out, 2, dagger)
    got = unpack(op, out, 2, EVEN)
    exp = np.stack([L.m5d_inv(L.on_parity(nat[k], EVEN), M5, 0.03, dag=dagger) for k in range(2)])
    assert rel_per_rhs(got, exp) < 1e-13


@pytest.mark.parametrize("dims,Ls", SHAPES)
@pytest.mark.parametrize("dagger", [False, True])
def test_ddw_f64(dims, Ls, dagger):
    op, U = make_operator(dims, Ls, seed=7)
    nat = fields(dims, Ls, 1, seed=8)
    inp = pack(op, nat, BOTH)
    out = op.new_field(1, both=True)
    op.ddw(inp, out, 1, dagger)
    got = unpack(op, out, 1, BOTH)[0]
    assert rel(got, L.ddw(U, nat[0], M5, MF, dag=dagger)) < 1e-13


@pytest.mark.parametrize("prec,tol", [(F64, 1e-13), (F32, 1e-6), (F16S, 2e-3)])
@pytest.mark.parametrize("dims,Ls,spb", [((2, 2, 2, 2), 4, 1), ((4, 4, 6, 8), 5, 7), ((6, 4, 2, 4), 12, 5), ((4, 4, 4, 4), 8, 16)])
def test_ddw_both_parities_in_one_launch(dims, Ls, spb, prec, tol):
    """The two parities' workgroups share a launch: tile counts that do and do not divide into the
    8 XCDs, ragged last tiles and several right-hand sides, against the oracle on the stored input."""
    nrhs = 3
    op, U = make_operator(dims, Ls, eps=0.5, seed=47, prec=prec)
    op.set_tile(spb)
    inp = pack(op, fields(dims, Ls, nrhs, seed=48), BOTH)
    src = unpack(op, inp, nrhs, BOTH)
    out = op.new_field(nrhs, both=True)
    for dagger in (False, True):
        op.ddw(inp, out, nrhs, dagger)
        exp = np.stack([L.ddw(U, v, M5, MF, dag=dagger) for v in src])
        assert rel_per_rhs(unpack(op, out, nrhs, BOTH), exp) < tol


@pytest.mark.parametrize("prec,tol", [(F64, 1e-13), (F32, 1e-6), (F16S, 2e-3)])
@pytest.mark.parametrize("rpb", [2, 3, 64])
def test_ddw_both_parities_with_rhs_looped_over(rpb, prec, tol):
    """The two-parity launch where a workgroup takes several right-hand sides, the last group short."""
    dims, Ls, nrhs = (4, 4, 6, 8), 5, 5
    op, U = make_operator(dims, Ls, eps=0.5, seed=55, prec=prec, max_nrhs=nrhs)
    op.set_tile(7, 2, rpb)
    inp = pack(op, fields(dims, Ls, nrhs, seed=56), BOTH)
    src = unpack(op, inp, nrhs, BOTH)
    out = op.new_field(nrhs, both=True)
    op.ddw(inp, out, nrhs, True)
    exp = np.stack([L.ddw(U, v, M5, MF, dag=True) for v in src])
    assert rel_per_rhs(unpack(op, out, nrhs, BOTH), exp) < tol


@pytest.mark.parametrize("prec", [F64, F32, F16S])
@pytest.mark.parametrize("Ls", [1, 5, 24, 33, 48, 64, 96])
def test_default_tile_matches_widest(Ls, prec):
    """The default workgroup of a small lattice (one to four waves, by how full Ls leaves them)
    gives bitwise the fields of the widest one, which the parity tests above pin."""
    dims, nrhs = (4, 2, 4, 6), 2
    op, _ = make_operator(dims, Ls, eps=0.5, seed=49, prec=prec)
    inp = pack(op, fields(dims, Ls, nrhs, seed=50), BOTH)
    got = []
    for spb in (0, max(1, min(256 // Ls, 64))):
        op.set_tile(spb)
        pc, full = op.new_field(nrhs), op.new_field(nrhs, both=True)
        op.mpcdagmpc(inp, pc, nrhs)
        op.ddw(inp, full, nrhs, True)
        got.append((pc.cpu(), full.cpu()))
    assert all((a == b).all() for a, b in zip(*got))


@pytest.mark.parametrize("prec", [F64, F32, F16S])
@pytest.mark.parametrize("dims,Ls,nrhs,rpb", [((8, 8, 8, 8), 16, 9, 1), ((8, 8, 8, 8), 16, 9, 4), ((4, 4, 4, 4), 12, 342, 1)])
def test_default_tile_of_many_right_hand_sides(dims, Ls, nrhs, rpb, prec):
    """Past the number of fields where the default workgroup changes (524288 points in a launch,
    262144 for the FP16 + scale M5D; with rhs looped over inside a workgroup, fewer side by side)
    it gives bitwise the fields of one wave and of the widest, which the parity tests above pin."""
    op, _ = make_operator(dims, Ls, eps=0.5, seed=53, prec=prec, max_nrhs=nrhs)
    inp = pack(op, fields(dims, Ls, 3, seed=54), BOTH).view(2, 3, -1)
    both = inp[:, [k % 3 for k in range(nrhs)]].contiguous()
    even, both = both[0].contiguous().view(-1), both.view(-1)
    got = []
    for spb in (0, 64 // Ls, 256 // Ls):
        op.set_tile(spb, 0, rpb)
        pc, m5, full = op.new_field(nrhs), op.new_field(nrhs), op.new_field(nrhs, both=True)
        op.mpcdagmpc(even, pc, nrhs)
        op.m5d_inv(even, m5, nrhs)
        op.ddw(both, full, nrhs)
        got.append((pc, m5, full))
    for other in got[1:]:
        assert all((a == b).all() for a, b in zip(got[0], other))


@pytest.mark.parametrize("dims,Ls", SHAPES)
def test_mpc_and_normal_operator_f64(dims, Ls):
    nrhs = 2
    op, U = make_operator(dims, Ls, seed=9)
    nat = np.stack([L.on_parity(f, EVEN) for f in fields(dims, Ls, nrhs, seed=10)])
    inp = pack(op, nat, EVEN)
    out = op.new_field(nrhs)
    op.mpc(inp, out, nrhs, False)
    assert rel_per_rhs(unpack(op, out, nrhs, EVEN), np.stack([L.mpc(U, v, M5, MF) for v in nat])) < 1e-13
    op.mpc(inp, out, nrhs, True)
    assert rel_per_rhs(unpack(op, out, nrhs, EVEN), np.stack([L.mpc_dag(U, v, M5, MF) for v in nat])) < 1e-13
    op.mpcdagmpc(inp, out, nrhs)
    assert rel_per_rhs(unpack(op, out, nrhs, EVEN), np.stack([L.mpcdagmpc(U, v, M5, MF) for v in nat])) < 1e-13


def test_mpc_chunking_beyond_temporaries():
    """nrhs larger than the operator temporaries: processed in chunks, same result."""
    dims, Ls = (4, 4, 4, 4), 8
    op, U = make_operator(dims, Ls, seed=11, max_nrhs=2)
    nat = np.stack([L.on_parity(f, EVEN) for f in fields(dims, Ls, 5, seed=12)])
    out = op.new_field(5)
    op.mpcdagmpc(pack(op, nat, EVEN), out, 5)
    assert rel_per_rhs(unpack(op, out, 5, EVEN), np.stack([L.mpcdagmpc(U, v, M5, MF) for v in nat])) < 1e-13


@pytest.mark.parametrize("prec,tol", [(F32, 1e-6), (F16S, 3e-3)])
def test_mpcdagmpc_low_precision(prec, tol):
    dims, Ls = (4, 4, 4, 4), 8
    op, U = make_operator(dims, Ls, seed=13, prec=prec)
    nat = np.stack([L.on_parity(f, EVEN) for f in fields(dims, Ls, 2, seed=14)])
    inp = pack(op, nat, EVEN)
    src = unpack(op, inp, 2, EVEN)
    out = op.new_field(2)
    op.mpcdagmpc(inp, out, 2)
    got = unpack(op, out, 2, EVEN)
    assert rel_per_rhs(got, np.stack([L.mpcdagmpc(U, v, M5, MF) for v in src])) < tol
    if prec == F16S:
        # the four passes, each output rounded to FP16 + scale as the kernels store it
        def chain(v):
            t = _q(L.m5d_inv(L.m_oe(U, v), M5, MF))
            u = _q(L.m5d(v, M5, MF) - L.m_eo(U, t))
            t = _q(L.m5d_inv(L.m_eo(U, u, dag=True), M5, MF, dag=True))
            return _q(L.m5d(u, M5, MF, dag=True) - L.m_oe(U, t, dag=True))

        assert rel_per_rhs(got, np.stack([chain(v) for v in src])) < QUANTISED_TOL_MDAGM


def test_repeat_is_bitwise_deterministic():
    dims, Ls = (4, 4, 6, 8), 5
    op, U = make_operator(dims, Ls, seed=15)
    nat = np.stack([L.on_parity(f, EVEN) for f in fields(dims, Ls, 1, seed=16)])
    inp = pack(op, nat, EVEN)
    a, b = op.new_field(1), op.new_field(1)
    op.mpcdagmpc(inp, a, 1)
    op.set_tile(8)  # different workgroup shape, same per-site arithmetic
    op.mpcdagmpc(inp, b, 1)
    import torch

    torch.cuda.synchronize()
    assert torch.equal(a, b)


@pytest.mark.parametrize("order", [1, 2, (1, 2, 2), (2, 1, 4), (1, 4, 1)])
@pytest.mark.parametrize("prec", [F64, F32, F16S])
def test_traversal_order_gives_identical_results(prec, order):
    """The XCD-octant, t-slab and box traversals only permute which workgroup computes a site."""
    dims, Ls = (8, 4, 4, 8), 6
    op, U = make_operator(dims, Ls, seed=17, prec=prec)
    nat = np.stack([L.on_parity(f, EVEN) for f in fields(dims, Ls, 2, seed=18)])
    inp = pack(op, nat, EVEN)
    a, b = op.new_field(2), op.new_field(2)
    op.mpcdagmpc(inp, a, 2)
    if isinstance(order, tuple):
        op.set_order_box(*order)
        assert op.get_order() == (3, order)
    else:
        op.set_order(order)
        assert op.get_order() == (order, (0, 0, 0))
    op.mpcdagmpc(inp, b, 2)
    import torch

    torch.cuda.synchronize()
    assert torch.equal(a, b)
    if prec == F64:
        exp = np.stack([L.mpcdagmpc(U, v, M5, MF) for v in nat])
        assert rel_per_rhs(unpack(op, b, 2, EVEN), exp) < 1e-13


@pytest.mark.parametrize("prec", [F64, F32])
def test_rhs_per_block_identical(prec):
    """Workgroups looping over several rhs with their links staged once compute the
    same values as one rhs per workgroup (5 rhs in groups of 2: a ragged last group)."""
    import torch

    dims, Ls = (4, 4, 6, 8), 5
    op, U = make_operator(dims, Ls, seed=19, prec=prec, max_nrhs=5)
    nat = np.stack([L.on_parity(f, EVEN) for f in fields(dims, Ls, 5, seed=20)])
    inp = pack(op, nat, EVEN)
    a, b = op.new_field(5), op.new_field(5)
    op.mpcdagmpc(inp, a, 5)
    op.set_tile(0, 0, 2)
    op.mpcdagmpc(inp, b, 5)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    fa, fb = inp.clone(), inp.clone()
    op.set_tile(0, 0, 1)
    op.chebyshev_filter(fa, 5, 3, 0.1, 40.0)
    op.set_tile(0, 0, 4)
    op.chebyshev_filter(fb, 5, 3, 0.1, 40.0)
    torch.cuda.synchronize()
    assert torch.equal(fa, fb)


def test_cg_batched_with_rhs_per_block():
    """CG's fused p.Ap partials are per rhs also when a workgroup handles several rhs."""
    from oracle import krylov

    dims, Ls = (4, 4, 4, 4), 8
    op, U = make_operator(dims, Ls, seed=0, max_nrhs=2, max_cg_rhs=2)
    op.set_tile(0, 0, 2)
    b = np.stack([L.on_parity(f, EVEN) for f in fields(dims, Ls, 2, seed=21)])
    x = op.new_field(2)
    code, iters, res = op.cg(pack(op, b, EVEN), x, 2, tol=1e-10)
    xg = unpack(op, x, 2, EVEN)
    for k in range(2):
        ref = krylov.cg(lambda v: L.mpcdagmpc(U, v, M5, MF), b[k], tol=1e-10)
        assert abs(iters[k] - ref.iterations) <= 3 and res[k] < 1.5e-10
        assert rel(xg[k], ref.x) < 1e-6


def test_box_order_rejects_cuts_that_do_not_fit():
    import paper_2103_05034_amd as dwf

    op, _ = make_operator((8, 4, 4, 8), 4, seed=19)
    for cut in ((3, 1, 1), (1, 3, 1), (8, 1, 1), (0, 1, 1), (1, 1, 8)):
        with pytest.raises(dwf.DWFError):
            op.set_order_box(*cut)  # x extent odd, not dividing, or zero
    with pytest.raises(dwf.DWFError):
        op.set_order(3)  # boxes only through set_order_box
    assert op.get_order() == (0, (0, 0, 0))


def test_autotune_cache(tmp_path, monkeypatch):
    """dwf_autotune keeps the shape it found per (architecture, lattice, Ls, nrhs,
    precision, order, occupancy cap, Schur form): a second handle of the same
    configuration gets it without timing (the reported time is the tuned one), a
    different traversal order is tuned afresh, and with DWF_TUNE_CACHE set the shapes
    survive a cleared process cache through the file.  The cached shape computes
    M_pc^dag M_pc bitwise as the tuned one."""
    import torch

    import paper_2103_05034_amd as dwf

    dims, Ls = (8, 4, 4, 8), 6
    monkeypatch.delenv("DWF_TUNE_CACHE", raising=False)
    dwf.tune_cache_clear()
    op1, U = make_operator(dims, Ls, seed=21, max_nrhs=2)
    r1 = op1.autotune(2, 2)
    op2, _ = make_operator(dims, Ls, seed=21, max_nrhs=2)
    r2 = op2.autotune(2, 2)
    assert r1 == r2 and op1.tile == op2.tile
    assert op1.get_order() == op2.get_order()  # the tuned traversal order comes with the cached shape
    nat = np.stack([L.on_parity(f, EVEN) for f in fields(dims, Ls, 2, seed=22)])
    a, b = op1.new_field(2), op2.new_field(2)
    op1.mpcdagmpc(pack(op1, nat, EVEN), a, 2)
    op2.mpcdagmpc(pack(op2, nat, EVEN), b, 2)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    op2.set_order(1)
    spb, depth, ms = op2.autotune(2, 2)
    assert (spb, depth) != (0, 0) and ms > 0
    # through the file
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("DWF_TUNE_CACHE", str(path))
    dwf.tune_cache_clear()
    op3, _ = make_operator(dims, Ls, seed=21, max_nrhs=2)
    r3 = op3.autotune(1, 2)
    assert path.exists() and len(path.read_text().splitlines()) == 1
    dwf.tune_cache_clear()
    op4, _ = make_operator(dims, Ls, seed=21, max_nrhs=2)
    assert op4.autotune(1, 2) == r3
    assert len(path.read_text().splitlines()) == 1  # a hit appends nothing
    dwf.tune_cache_clear()
    for op in (op1, op2, op3, op4):
        op.close()


def test_hop_timing_counts_and_sampling():
    """dwf_enable_timing: 1 times every hop launch (four per M_pc^dag M_pc), n > 1 every
    n-th one; the sums reset on every enable call; timing changes no result."""
    import torch

    dims, Ls = (4, 4, 4, 8), 4
    op, _ = make_operator(dims, Ls, seed=25)
    nat = np.stack([L.on_parity(f, EVEN) for f in fields(dims, Ls, 1, seed=26)])
    v = pack(op, nat, EVEN)
    ref, w = op.new_field(1), op.new_field(1)
    op.mpcdagmpc(v, ref, 1)
    op.enable_timing(True)
    for _ in range(4):
        op.mpcdagmpc(v, w, 1)
    ms, n = op.kernel_time()
    assert n == 16 and ms > 0
    op.enable_timing(True, stride=5)  # launches 0, 5, 10 and 15 of the next sixteen
    for _ in range(4):
        op.mpcdagmpc(v, w, 1)
    ms5, n5 = op.kernel_time()
    assert n5 == 4 and ms5 > 0
    op.enable_timing(False)
    torch.cuda.synchronize()
    assert torch.equal(w, ref)
    import paper_2103_05034_amd as dwf

    with pytest.raises(dwf.DWFError):
        dwf._check(op.lib.dwf_enable_timing(op.h, -1))
