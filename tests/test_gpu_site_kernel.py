"""The fine apply's kernels for fifth dimensions other than 16: the site kernel (links and own spinors
of whole 4d sites in LDS; slice pairs in FP32 on large lattices) and the parity-tile kernel at Ls = 8,
against the oracle, and their fused epilogues against the same smoother on the generic kernel."""
import numpy as np
import pytest

import hdcr_inputs as hi
import oracle
import paper_1611_06944_amd as hd
from tests.gpu_util import log, max_rel_elem, rel_err, to_dev, to_host, torch_dev

pytestmark = pytest.mark.gpu

SHAPES = [
    ((2, 2, 2, 2), 8),      # one tile, extent-2 directions
    ((4, 6, 2, 4), 8),      # parity tiles, ragged over the XCDs
    ((3, 5, 2, 3), 8),      # odd extents at Ls = 8: site kernel, ragged last workgroup
    ((2, 3, 2, 5), 4),      # smallest Ls of the site kernel, workgroups capped by LDS
    ((4, 2, 2, 4), 7),      # odd Ls, work-items past the last whole site
    ((1, 3, 2, 2), 12),     # extent 1
    ((4, 4, 2, 2), 12),
    ((3, 2, 2, 3), 24),
    ((2, 2, 1, 1), 130),    # one site per workgroup, idle lanes
    ((1, 1, 2, 1), 258),    # FP32 pairs by length, FP64 on the generic kernel
]


@pytest.mark.parametrize("L,Ls", SHAPES)
@pytest.mark.parametrize("prec,tol", [("c128", 1e-10), ("c64", 1e-5)])
def test_apply_any_ls(L, Ls, prec, tol):
    torch = torch_dev()
    log(f"site kernel L={L} Ls={Ls} {prec}")
    p = oracle.Params(L, Ls, M5=1.8, mf=0.07, bc=(1, -1, 1, -1), b=1.3)
    lat = hd.Lattice(L, Ls, M5=p.M5, mf=p.mf, bc=p.bc, b=1.3)
    U = hi.gauge_field(L, seed=1)
    psi = hi.gaussian_fermion(L, Ls, seed=0)
    ref = oracle.apply_h(U, psi, p)
    dt = torch.complex128 if prec == "c128" else torch.complex64
    out = hd.apply_fine(lat, to_dev(hd.pack_gauge(U), dt), to_dev(hd.pack_fermion(psi), dt))
    got = hd.unpack_fermion(to_host(out), L, Ls)
    assert max_rel_elem(got, ref) <= tol and rel_err(got, ref) <= tol


@pytest.mark.parametrize("L,Ls", [((4, 4, 2, 6), 8), ((3, 4, 2, 3), 12), ((2, 3, 3, 2), 5)])
@pytest.mark.parametrize("prec,tol", [("c128", 1e-12), ("c64", 2e-5)])
def test_epilogues_match_generic_kernel(L, Ls, prec, tol):
    """An order-5 smoother runs one to three epilogue fields; FP32 rounding (2^-24 per operation, about
    10^2 operations deep, the polynomial's growth below 2) stays under 2e-5."""
    torch = torch_dev()
    log(f"epilogues L={L} Ls={Ls} {prec}")
    lat = hd.Lattice(L, Ls, mf=0.05)
    dt = torch.complex128 if prec == "c128" else torch.complex64
    U = to_dev(hd.pack_gauge(hi.gauge_field(L, seed=4)), dt)
    x = to_dev(hd.pack_fermion(hi.gaussian_fermion(L, Ls, seed=3)), dt)
    got = hd.smooth(lat, U, x, order=5, lo=0.5, hi=64.0)
    ref = hd.smooth(lat.with_tune(dslash_variant=2), U, x, order=5, lo=0.5, hi=64.0)
    assert float((got - ref).abs().max()) <= tol * float(ref.abs().max())


def test_slice_pairs_match_single_slices():
    """16 x 16 x 16 x 24 x 12 is above the size from which FP32 takes slice pairs."""
    torch = torch_dev()
    L, Ls = (16, 16, 16, 24), 12
    log("slice pairs")
    lat = hd.Lattice(L, Ls, mf=0.05)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(5)
    U = to_dev(hd.pack_gauge(hi.gauge_field(L, seed=4)), torch.complex64)
    x = torch.randn((12, lat.V4, Ls), dtype=torch.complex64, device="cuda:0", generator=g)
    got = hd.apply_fine(lat, U, x)
    ref = hd.apply_fine(lat.with_tune(dslash_variant=2), U, x)
    assert float((got - ref).abs().max()) <= 1e-6 * float(ref.abs().max())
    assert torch.equal(got, hd.apply_fine(lat, U, x))


@pytest.mark.parametrize("L,m", [((3, 5, 2, 3), 1), ((2, 4, 2, 2), 2), ((4, 2, 2, 6), 7), ((1, 3, 2, 2), 11),
                                 ((2, 3, 3, 2), 12), ((2, 2, 1, 1), 63)])
def test_continued_fraction_site_kernel(L, m):
    """Ls = 2 (sites capped by LDS), 3, 8, 12, 13 and 64: ragged last workgroups, extent 1, idle
    work-items.  The slice pairs are taken on large lattices only, so they are held against single
    slices there; sums of about 10^2 roundings of 2^-24."""
    torch = torch_dev()
    Ls, bc, M5, R = m + 1, (1, -1, 1, -1), 1.7, 0.35
    log(f"cf site kernel L={L} m={m}")
    beta = list(0.2 + 2.0 * np.random.default_rng(m).random(m))
    U = hi.gauge_field(L, seed=8)
    x = hi.gaussian_fermion(L, Ls, seed=9)
    ref = oracle.apply_cf(U, x, M5, beta, R, bc)
    lat = hd.Lattice(L, Ls, M5=M5, bc=bc)
    for dt, tol in ((torch.complex128, 1e-10), (torch.complex64, 1e-5)):
        out = hd.apply_cf(lat, to_dev(hd.pack_gauge(U), dt), to_dev(hd.pack_fermion(x), dt), beta, R)
        assert max_rel_elem(hd.unpack_fermion(to_host(out), L, Ls), ref) <= tol, dt


def test_continued_fraction_slice_pairs():
    torch = torch_dev()
    L, Ls = (16, 16, 16, 18), 18  # 1.3M 5d sites
    log("cf slice pairs")
    lat = hd.Lattice(L, Ls, M5=1.7, bc=(1, -1, 1, -1))
    U = to_dev(hd.pack_gauge(hi.gauge_field(L, seed=2)))
    g = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn((12, lat.V4, Ls), dtype=torch.complex128, device="cuda", generator=g)
    beta = list(0.3 + 0.1 * np.arange(Ls - 1))
    ref = hd.apply_cf(lat, U, x, beta, 0.35)  # FP64: single slices
    got = hd.apply_cf(lat, U.to(torch.complex64), x.to(torch.complex64), beta, 0.35)
    assert float((got - ref).abs().max()) <= 1e-5 * float(ref.abs().max())


@pytest.mark.parametrize("L,Ls", [((11, 9, 10, 14), 10), ((7, 11, 13, 6), 22)])
def test_slice_pairs_from_ten_slices(L, Ls):
    """Just above 2^17 5d sites, ragged last workgroups: pairs against the generic kernel, and the
    continued fraction's against FP64; rounding as above."""
    torch = torch_dev()
    log(f"slice pairs L={L} Ls={Ls}")
    lat = hd.Lattice(L, Ls, mf=0.05)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(5)
    U = to_dev(hd.pack_gauge(hi.gauge_field(L, seed=4)))
    x = torch.randn((12, lat.V4, Ls), dtype=torch.complex128, device="cuda:0", generator=g)
    U32, x32 = U.to(torch.complex64), x.to(torch.complex64)
    ref = hd.apply_fine(lat.with_tune(dslash_variant=2), U32, x32)
    assert float((hd.apply_fine(lat, U32, x32) - ref).abs().max()) <= 1e-6 * float(ref.abs().max())
    beta = list(0.3 + 0.1 * np.arange(Ls - 1))
    ref = hd.apply_cf(lat, U, x, beta, 0.35)
    assert float((hd.apply_cf(lat, U32, x32, beta, 0.35) - ref).abs().max()) <= 1e-5 * float(ref.abs().max())
