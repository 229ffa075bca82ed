"""The little Dirac operator's build on the matrix cores, at the edges of its tiles: row groups of 16 and
32 per chirality, several column groups, slice groups of four cut short, faces of extent 1, neighbours
that are the block itself or the same block both ways, and every split of a block's sites."""
import numpy as np
import pytest

import hdcr_inputs as hi
import oracle
import paper_1611_06944_amd as hd
from tests.gpu_util import log, max_rel_elem, to_dev, to_host, torch_dev

pytestmark = pytest.mark.gpu

SHAPES = [
    ((4, 4, 2, 2), 2, (2, 2, 1, 1), 3),     # one stored slice; faces that are the whole block
    ((2, 2, 2, 2), 4, (1, 1, 1, 1), 24),    # single-site blocks: no interior hop, rank 24 of 24
    ((2, 4, 2, 3), 6, (2, 2, 2, 3), 16),    # coarse extent 1 and 2; a full row tile; 3 of 4 slices
    ((3, 2, 4, 2), 10, (3, 1, 2, 2), 17),   # odd block extent, one row past a tile, 5 stored slices
    ((4, 2, 2, 2), 16, (2, 2, 1, 2), 33),   # two row groups, two column groups
    ((2, 2, 2, 4), 8, (2, 2, 2, 2), 49),    # three column groups, ragged
]


@pytest.mark.parametrize("L,Ls,block,nvec", SHAPES)
def test_build_against_oracle(L, Ls, block, nvec):
    """The entries are sums of at most 12 bvol Ls 2^-53-rounded terms of blocks whose columns have norm 1,
    with |H| below 14, so 1e-12 holds for them; the basis itself is orthonormal to the same order times
    the condition of random vectors (below 1e3 here)."""
    torch = torch_dev()
    log(f"build L={L} Ls={Ls} block={block} nvec={nvec}")
    p = oracle.Params(L, Ls, M5=1.8, mf=0.07, bc=(1, -1, 1, -1), b=1.3)
    cs = oracle.Coarse(p, block, nvec)
    U = hi.gauge_field(L, seed=5)
    vecs = np.stack([hi.gaussian_fermion(L, Ls, seed=40 + i) for i in range(nvec)])
    bref, st = oracle.block_basis(vecs, cs)
    assert st == 0
    ref = oracle.coarse_build(U, bref, cs)
    lat = hd.Lattice(L, Ls, M5=p.M5, mf=p.mf, bc=p.bc, b=1.3, block=block, nvec=nvec)
    dv = torch.stack([to_dev(hd.pack_fermion(v)) for v in vecs])
    _, A = hd.build_coarse(lat, to_dev(hd.pack_gauge(U)), dv, hd.C128)
    got = to_host(hd.export_coarse(lat, A, hd.C128)).reshape(ref.shape)
    assert np.abs(got - ref).max() <= 1e-10 * np.abs(ref).max()


@pytest.mark.parametrize("L,Ls,block,nvec", [
    ((2, 2, 2, 2), 2, (1, 1, 1, 1), 1),     # 12 indices to a vector: less than one tile
    ((2, 2, 2, 2), 2, (1, 1, 1, 1), 9),
    ((2, 2, 2, 2), 2, (2, 2, 1, 1), 17),    # 48 indices; a vector past a tile
    ((3, 2, 2, 2), 2, (3, 1, 1, 1), 25),    # 36 indices, four in the last tile; seven groups of vectors
    ((2, 2, 2, 2), 10, (1, 1, 1, 1), 32),   # 60 indices; the most vectors
    ((4, 2, 2, 2), 4, (2, 2, 2, 2), 8),     # several parts; a group of vectors exactly
    ((4, 2, 2, 2), 4, (2, 2, 2, 2), 16),
    ((4, 2, 4, 2), 8, (2, 2, 2, 2), 24),
])
def test_orthonormal_basis_against_oracle(L, Ls, block, nvec):
    """The thin QR factor with a positive diagonal is unique, so the basis equals the oracle's to rounding
    times the condition of the random vectors (below 1e3): 1e-10.  The FP32 and FP16 copies are its
    roundings, so a restriction with either equals the FP64 one within 1e-5 and 2e-2."""
    torch = torch_dev()
    log(f"block basis L={L} Ls={Ls} block={block} nvec={nvec}")
    p = oracle.Params(L, Ls, M5=1.8, mf=0.07)
    cs = oracle.Coarse(p, block, nvec)
    vecs = np.stack([hi.gaussian_fermion(L, Ls, seed=60 + i) for i in range(nvec)])
    ref, st = oracle.block_basis(vecs, cs)
    assert st == 0
    lat = hd.Lattice(L, Ls, M5=p.M5, mf=p.mf, block=block, nvec=nvec)
    dv = torch.stack([to_dev(hd.pack_fermion(v)) for v in vecs])
    basis, _ = hd.build_coarse(lat, to_dev(hd.pack_gauge(hi.gauge_field(L, seed=5))), dv, hd.C128)
    got = np.stack([hd.unpack_fermion(f, L, Ls) for f in to_host(hd.export_basis(lat, basis))])
    assert max_rel_elem(got, ref) <= 1e-10
    psi = to_dev(hd.pack_fermion(hi.gaussian_fermion(L, Ls, seed=7)))
    v64 = hd.restrict(lat, basis, psi)
    v32 = hd.restrict(lat, basis, psi.to(torch.complex64))
    v16 = hd.restrict(lat, basis, psi.to(torch.complex64), half_basis=True)
    assert float((v32 - v64).abs().max()) <= 1e-5 * float(v64.abs().max())
    assert float((v16 - v64).abs().max()) <= 2e-2 * float(v64.abs().max())
