"""GPU parity of the coarse-space transfer (chirality split, block orthonormalisation,
restriction, prolongation) against the oracle, through the C ABI.

The oracle runs on the values the GPU actually holds (the packed input unpacked
again), so restriction differs only by the order of FP64 summation whatever the
storage precision; prolongation and orthonormalisation round their outputs to
the storage precision.  At the paper's 16^3x32, Ls=16 size the checks are the
size-independent identities of an orthonormal blocked basis."""

import numpy as np
import pytest

import synth
from oracle import coarse as C
from oracle import lattice as L
from tests.gpu_util import make_operator, pack, unpack

pytestmark = pytest.mark.gpu

F64, F32, F16S = 0, 1, 2
EVEN = 0
C1 = ((4, 4, 4, 4), 8)


def even_fields(dims, Ls, n, seed):
    return np.stack([L.on_parity(f, L.EVEN) for f in synth.gaussian_fermion_batch(dims, Ls, n, seed)])


def coarse_host(t):
    import torch

    torch.cuda.synchronize()
    return t.cpu().numpy()


def relmax(a, b):
    return np.max(np.abs(a - b)) / np.max(np.abs(b))


@pytest.mark.parametrize("prec,tol", [(F64, 0.0), (F32, 1e-7), (F16S, 2e-3)])
def test_chiral_split(prec, tol):
    dims, Ls = C1
    op, _ = make_operator(dims, Ls, prec=prec, max_nrhs=4)
    v = even_fields(dims, Ls, 2, seed=40)
    buf = pack(op, v, EVEN)
    held = unpack(op, buf, 2, EVEN)
    out = op.chiral_split(buf, 2)
    got = unpack(op, out, 4, EVEN)
    for k in range(2):
        p, m = C.chiral_split(held[k])
        if prec == F64:
            assert np.array_equal(got[2 * k], p) and np.array_equal(got[2 * k + 1], m)
        else:
            assert relmax(got[2 * k], p) <= tol and relmax(got[2 * k + 1], m) <= tol


@pytest.mark.parametrize("prec", [F64, F32, F16S])
@pytest.mark.parametrize("block", [(2, 2, 2, 2), (4, 2, 4, 2), (2, 4, 2, 1)])
def test_restrict_and_prolong(prec, block):
    import torch

    dims, Ls = C1
    op, _ = make_operator(dims, Ls, prec=prec, max_nrhs=8)
    nb = op.set_blocks(block)
    assert nb == C.nblocks(dims, block)
    nvec, nrhs = 5, 3
    basis = pack(op, even_fields(dims, Ls, nvec, seed=41), EVEN)
    v = pack(op, even_fields(dims, Ls, nrhs, seed=42), EVEN)
    B = unpack(op, basis, nvec, EVEN)
    V = unpack(op, v, nrhs, EVEN)
    c = coarse_host(op.restrict(basis, nvec, v, nrhs))
    assert c.shape == (nrhs, nb, nvec)
    for r in range(nrhs):
        assert relmax(c[r], C.restrict(list(B), V[r], dims, block)) < 1e-13
    rng = np.random.default_rng(5)
    cc = rng.standard_normal((nrhs, nb, nvec)) + 1j * rng.standard_normal((nrhs, nb, nvec))
    out = op.prolong(basis, nvec, torch.from_numpy(cc).cuda(), nrhs)
    got = unpack(op, out, nrhs, EVEN)
    tol = {F64: 1e-14, F32: 2e-7, F16S: 2e-3}[prec]
    for r in range(nrhs):
        assert relmax(got[r], C.prolong(list(B), cc[r], dims, block)) < tol


@pytest.mark.parametrize("prec", [F64, F32, F16S])
@pytest.mark.parametrize(
    "dims, Ls, block, nvec, nrhs, both",
    [
        ((4, 4, 4, 4), 5, (2, 2, 2, 2), 1, 1, False),  # one vector, one rhs
        ((4, 4, 4, 4), 8, (2, 2, 2, 2), 9, 1, True),  # three batches of vectors on workgroups of their own
        ((4, 4, 4, 6), 7, (2, 2, 2, 2), 6, 2, True),  # no whole number of vectors in flight, two rhs
        ((4, 4, 4, 4), 12, (4, 4, 4, 2), 8, 5, False),  # two sites a lane; a second tile of rhs with one
        ((8, 8, 16, 32), 1, (2, 2, 2, 1), 3, 2, False),  # 4096 waves: a lane per spinor
    ],
)
def test_restrict_and_prolong_shapes(prec, dims, Ls, block, nvec, nrhs, both):
    import torch

    parity = 2 if both else EVEN
    op, _ = make_operator(dims, Ls, prec=prec, max_nrhs=2)
    nb = op.set_blocks(block, both=both)

    def held(n, seed):
        raw = synth.gaussian_fermion_batch(dims, Ls, n, seed)
        buf = pack(op, raw if both else L.on_parity(raw, EVEN), parity)
        return buf, unpack(op, buf, n, parity)

    basis, B = held(nvec, 53)
    v, V = held(nrhs, 54)
    c = coarse_host(op.restrict(basis, nvec, v, nrhs))
    rng = np.random.default_rng(55)
    cc = rng.standard_normal((nrhs, nb, nvec)) + 1j * rng.standard_normal((nrhs, nb, nvec))
    got = unpack(op, op.prolong(basis, nvec, torch.from_numpy(cc).cuda(), nrhs), nrhs, parity)
    tol = {F64: 1e-14, F32: 2e-7, F16S: 2e-3}[prec]
    for r in range(nrhs):
        assert relmax(c[r], C.restrict(list(B), V[r], dims, block)) < 1e-13
        assert relmax(got[r], C.prolong(list(B), cc[r], dims, block)) < tol


@pytest.mark.parametrize("block", [(2, 2, 2, 2), (4, 2, 4, 2)])
def test_block_orthonormalize_f64(block):
    dims, Ls = C1
    op, _ = make_operator(dims, Ls, prec=F64, max_nrhs=8)
    op.set_blocks(block)
    V = even_fields(dims, Ls, 6, seed=43)
    V[4] = V[4] + 25.0 * V[1]
    buf = pack(op, V, EVEN)
    op.block_orthonormalize(buf, 6)
    Q = unpack(op, buf, 6, EVEN)
    Qo, _ = C.block_orthonormalize(list(V), dims, block)
    for k in range(6):
        assert relmax(Q[k], Qo[k]) < 1e-12
        assert not np.any(L.on_parity(Q[k], L.ODD))


def test_block_orthonormalize_ill_conditioned_and_breakdown():
    import paper_2103_05034_amd as dwf

    dims, Ls = C1
    block = (2, 2, 2, 2)
    op, _ = make_operator(dims, Ls, prec=F64, max_nrhs=8)
    op.set_blocks(block)
    V = even_fields(dims, Ls, 4, seed=44)
    V[2] = V[0] + 1e-6 * V[2]  # kappa ~ 1e6 in every block
    buf = pack(op, V, EVEN)
    op.block_orthonormalize(buf, 4)
    Q = unpack(op, buf, 4, EVEN)
    for j in range(4):
        for k in range(4):
            g = C.block_inner(Q[j], Q[k], dims, block)
            assert np.max(np.abs(g - (1.0 if j == k else 0.0))) < 1e-13
    V[3] = V[1]  # dependent in every block
    buf = pack(op, V, EVEN)
    with pytest.raises(dwf.DWFError) as e:
        op.block_orthonormalize(buf, 4)
    assert e.value.code == dwf.DWF_EBREAKDOWN


@pytest.mark.parametrize("prec,tol", [(F32, 1e-5), (F16S, 3e-3)])
def test_block_orthonormalize_low_precision(prec, tol):
    dims, Ls = C1
    block = (2, 2, 2, 2)
    op, _ = make_operator(dims, Ls, prec=prec, max_nrhs=8)
    op.set_blocks(block)
    buf = pack(op, even_fields(dims, Ls, 5, seed=45), EVEN)
    held = unpack(op, buf, 5, EVEN)
    op.block_orthonormalize(buf, 5)
    Q = unpack(op, buf, 5, EVEN)
    Qo, _ = C.block_orthonormalize(list(held), dims, block)
    for k in range(5):
        assert relmax(Q[k], Qo[k]) < tol
    for j in range(5):
        for k in range(5):
            g = C.block_inner(Q[j], Q[k], dims, block)
            assert np.max(np.abs(g - (1.0 if j == k else 0.0))) < 4 * tol


def test_gamma5_commutes_with_gpu_restriction():
    """GPU chirality split + block orthonormalisation keeps each basis vector chiral, so
    restricting Gamma_5 v flips the sign of the (1 - Gamma_5) rows."""
    dims, Ls = C1
    block = (2, 2, 2, 2)
    op, _ = make_operator(dims, Ls, prec=F64, max_nrhs=8)
    op.set_blocks(block)
    raw = pack(op, even_fields(dims, Ls, 3, seed=46), EVEN)
    basis = op.chiral_split(raw, 3)
    op.block_orthonormalize(basis, 6)
    v = even_fields(dims, Ls, 1, seed=47)
    c = coarse_host(op.restrict(basis, 6, pack(op, v, EVEN), 1))[0]
    cg = coarse_host(op.restrict(basis, 6, pack(op, L.Gamma5(v[0])[None], EVEN), 1))[0]
    sign = np.array([1, -1] * 3)
    assert np.max(np.abs(cg - c * sign[None, :])) < 1e-12 * np.max(np.abs(c))


@pytest.mark.parametrize("block", [(2, 2, 2, 2), (4, 2, 4, 2)])
def test_fullsize_orthonormal_basis_identities(block):
    """16^3x32, Ls=16, FP32 (the Algorithm A / B blocks): after orthonormalisation
    restrict(Q, Q_k) is the k-th unit vector in every block, and restrict o prolong is
    the identity on random coarse vectors."""
    import torch

    dims, Ls = (16, 16, 16, 32), 16
    nvec = 8
    op, _ = make_operator(dims, Ls, eps=0.2, prec=F32, max_nrhs=nvec, max_cg_rhs=0)
    nb = op.set_blocks(block)
    basis = op.new_field(nvec)
    for k in range(nvec):
        op.pack(torch.from_numpy(synth.gaussian_fermion_batch(dims, Ls, 1, 100 + k)).cuda(), EVEN,
                out=basis[k * op.field_bytes(1) : (k + 1) * op.field_bytes(1)])
    op.block_orthonormalize(basis, nvec)
    G = coarse_host(op.restrict(basis, nvec, basis, nvec))  # [r][b][k] = <Q_k, Q_r>
    eye = np.eye(nvec)[:, None, :]
    assert np.max(np.abs(G - eye)) < 2e-6
    rng = np.random.default_rng(6)
    cc = rng.standard_normal((1, nb, nvec)) + 1j * rng.standard_normal((1, nb, nvec))
    back = coarse_host(op.restrict(basis, nvec, op.prolong(basis, nvec, torch.from_numpy(cc).cuda(), 1), 1))
    assert relmax(back, cc) < 1e-6


def test_block_orthonormalize_max_nvec():
    """nvec = 64, the largest basis: the Gram, Cholesky and update kernels hold a full
    64 x 64 complex matrix per block in LDS."""
    dims, Ls = C1
    block = (2, 2, 2, 2)
    op, _ = make_operator(dims, Ls, prec=F64, max_nrhs=64, max_cg_rhs=0)
    op.set_blocks(block)
    V = even_fields(dims, Ls, 64, seed=48)
    buf = pack(op, V, EVEN)
    op.block_orthonormalize(buf, 64)
    G = coarse_host(op.restrict(buf, 64, buf, 64))
    assert np.max(np.abs(G - np.eye(64)[:, None, :])) < 1e-12
    Q = unpack(op, buf, 64, EVEN)
    Qo, _ = C.block_orthonormalize(list(V), dims, block)
    assert max(relmax(Q[k], Qo[k]) for k in range(64)) < 1e-10


@pytest.mark.parametrize("both,block", [(False, (4, 4, 4, 2)), (True, (4, 2, 4, 2))])
def test_blocks_of_1024_5d_sites(both, block):
    """Ls = 16 with 64 sites per block (even sites of 4x4x4x2, or all sites of the
    Algorithm A block 4x2x4x2): 1024 5D sites, two per lane of the per-block kernels."""
    import torch

    dims, Ls = (8, 4, 8, 4), 16
    parity = 2 if both else EVEN
    op, _ = make_operator(dims, Ls, prec=F64, max_nrhs=8, max_cg_rhs=2)
    nb = op.set_blocks(block, both=both)
    assert nb == C.nblocks(dims, block)
    raw = synth.gaussian_fermion_batch(dims, Ls, 3, 50)
    if not both:
        raw = np.stack([L.on_parity(f, L.EVEN) for f in raw])
    split = unpack(op, op.chiral_split(pack(op, raw, parity), 3), 6, parity)
    basis = pack(op, split, parity)
    op.block_orthonormalize(basis, 6)
    Q = unpack(op, basis, 6, parity)
    Qo, _ = C.block_orthonormalize(list(split), dims, block)
    for k in range(6):
        assert relmax(Q[k], Qo[k]) < 1e-12
    W = synth.gaussian_fermion_batch(dims, Ls, 3, 51)
    if not both:
        W = np.stack([L.on_parity(f, L.EVEN) for f in W])
    c = coarse_host(op.restrict(basis, 6, pack(op, W, parity), 3))
    for r in range(3):
        assert relmax(c[r], C.restrict(list(Q), W[r], dims, block)) < 1e-13
    cc = np.random.default_rng(52).standard_normal((2, nb, 6)) + 0.5j
    got = unpack(op, op.prolong(basis, 6, torch.from_numpy(cc).cuda(), 2), 2, parity)
    for r in range(2):
        assert relmax(got[r], C.prolong(list(Q), cc[r], dims, block)) < 1e-14


@pytest.mark.parametrize("prec,unit", [(F64, 2.0**-53), (F32, 2.0**-24), (F16S, 2.0**-11)])
@pytest.mark.parametrize(
    "dims, Ls, block, nvec, both",
    [
        ((4, 4, 4, 4), 3, (2, 2, 2, 2), 1, False),  # one vector; a site of 36 values, no whole number of lines
        ((4, 4, 4, 4), 5, (2, 2, 2, 4), 8, False),  # one full tile of eight vectors
        ((4, 4, 4, 4), 4, (2, 2, 2, 2), 9, True),  # one vector into the second tile; both parities
        ((4, 4, 4, 6), 7, (2, 2, 2, 2), 40, True),  # five full tiles
        ((4, 4, 4, 4), 6, (4, 2, 4, 2), 49, False),  # seven tiles
        ((4, 4, 4, 4), 8, (2, 2, 2, 2), 57, True),  # eight tiles: the products in two launches
        ((4, 4, 4, 4), 16, (2, 2, 2, 2), 64, False),  # the most vectors
    ],
)
def test_block_orthonormalize_tiles(prec, unit, dims, Ls, block, nvec, both):
    parity = 2 if both else EVEN
    op, _ = make_operator(dims, Ls, prec=prec, max_nrhs=2)
    op.set_blocks(block, both=both)
    raw = synth.gaussian_fermion_batch(dims, Ls, nvec, 46)
    buf = pack(op, raw if both else L.on_parity(raw, EVEN), parity)
    held = unpack(op, buf, nvec, parity)
    op.block_orthonormalize(buf, nvec)
    Q = unpack(op, buf, nvec, parity)
    Qo, _ = C.block_orthonormalize(list(held), dims, block)
    # Each of the two rounds rounds every value once to the storage (relative to the spinor's largest for
    # FP16 + scale: sqrt(24) of its norm at most), the first error passing through the second round's R;
    # the FP64 sums over a block's K values add K u.  All of it grows at most with the condition number
    # squared: (1 + r) / (1 - r) with r = sqrt(n / K) for Gaussian vectors, 20 % above it over the blocks.
    K = 12 * Ls * int(np.prod(block)) / (1 if both else 2)
    r = np.sqrt(nvec / K)
    cond = 1.2 * (1 + r) / (1 - r)
    tol = 4 * unit * cond**2 * (np.sqrt(24) if prec == F16S else 1) + K * 2.0**-53 * cond**2
    big = max(float(np.max(np.abs(q))) for q in Qo)
    for k in range(nvec):
        assert np.max(np.abs(Q[k] - Qo[k])) < tol * max(big, 1.0), k


@pytest.mark.parametrize("prec,unit", [(F64, 2.0**-53), (F32, 2.0**-24)])
@pytest.mark.parametrize("dims, Ls, nvec", [((4, 4, 4, 6), 3, 9), ((2, 4, 6, 4), 5, 24), ((4, 4, 6, 4), 7, 56)])
def test_gram_schmidt_ragged_sites(prec, unit, dims, Ls, nvec):
    """Whole-lattice Cholesky QR where a site's values end inside a line and the ranges of sites are unequal."""
    from oracle import krylov

    op, _ = make_operator(dims, Ls, prec=prec, max_nrhs=3)
    buf = pack(op, even_fields(dims, Ls, nvec, seed=47), EVEN)
    held = unpack(op, buf, nvec, EVEN)
    R = op.gram_schmidt(buf, nvec)
    Q = unpack(op, buf, nvec, EVEN)
    Qo, Ro = krylov.gram_schmidt(list(held))
    K = 6 * Ls * int(np.prod(dims))
    r = np.sqrt(nvec / K)
    tol = (4 * unit + K * 2.0**-53) * (1.2 * (1 + r) / (1 - r)) ** 2  # as above
    for k in range(nvec):
        assert np.max(np.abs(Q[k] - Qo[k])) < tol * max(1.0, float(np.max(np.abs(Qo[k]))))
    assert np.max(np.abs(R - Ro)) < tol * np.max(np.abs(Ro))


@pytest.mark.parametrize("offset", [4, 8, 24])
def test_block_orthonormalize_scratch_alignment(offset):
    """Scratch of exactly the stated size at a 4- or 8-byte boundary gives the bits of an aligned
    one, and the bytes on both sides of it stay."""
    import torch
    import paper_2103_05034_amd as dwf

    dims, Ls = C1
    op, _ = make_operator(dims, Ls)
    op.set_blocks((2, 2, 2, 2))
    nvec = 9
    want = pack(op, even_fields(dims, Ls, nvec, seed=56), EVEN)
    got = want.clone()
    op.block_orthonormalize(want, nvec)
    nbytes = op.lib.dwf_block_scratch_bytes(op.h, nvec)
    buf = torch.full((nbytes + 64,), 7, dtype=torch.uint8, device="cuda")
    assert buf.data_ptr() % 64 == 0
    dwf._check(op.lib.dwf_block_orthonormalize(op.h, got.data_ptr(), nvec, buf.data_ptr() + offset, nbytes))
    torch.cuda.synchronize()
    assert (got == want).all()
    assert (buf[:offset] == 7).all() and (buf[offset + nbytes :] == 7).all()


@pytest.mark.parametrize("prec", [F64, F32])
@pytest.mark.parametrize("nvec", [3, 40, 64])
def test_gram_schmidt_of_vectors_at_a_multiple_of_8(prec, nvec):
    """Vectors aligned to 8 bytes only give the bits of aligned ones, and their surroundings stay."""
    import torch

    dims, Ls = (4, 4, 4, 6), 5
    op, _ = make_operator(dims, Ls, prec=prec, max_nrhs=3)
    want = pack(op, even_fields(dims, Ls, nvec, seed=57), EVEN)
    n = want.numel()
    buf = torch.full((n + 64,), 7, dtype=torch.uint8, device="cuda")
    assert buf.data_ptr() % 64 == 0
    got = buf[8 : n + 8]
    got.copy_(want)
    R = op.gram_schmidt(want, nvec)
    assert np.array_equal(op.gram_schmidt(got, nvec), R)
    torch.cuda.synchronize()
    assert (got == want).all()
    assert (buf[:8] == 7).all() and (buf[n + 8 :] == 7).all()


@pytest.mark.parametrize("prec", [F64, F32])
@pytest.mark.parametrize("nvec, nrhs", [(1, 3), (3, 5), (4, 3)])
def test_prolong_of_few_vectors_to_several_right_hand_sides(prec, nvec, nrhs):
    """Both sides of the number of vectors up to which three and more FP32 outputs are formed a
    lane per spinor, two at a time, on a lattice of 4096 waves."""
    test_restrict_and_prolong_shapes(prec, (8, 8, 16, 32), 1, (2, 2, 2, 1), nvec, nrhs, False)
