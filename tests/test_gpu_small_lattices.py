"""Kernel choices that depend on the size of the lattice, on both sides of their lines: each call against
the kernels that a tuning value forces, and FP32 against FP64.  Sums of some 10^2 roundings: 2^-53 each
stay under 1e-12 of the largest entry, 2^-24 each under 1e-5."""
import numpy as np
import pytest

import hdcr_inputs as hi
import oracle
import paper_1611_06944_amd as hd
from tests.gpu_util import log, max_rel_elem, to_dev, to_host, torch_dev

pytestmark = pytest.mark.gpu


def _fields(lat, L, seed):
    torch = torch_dev()
    U = to_dev(hd.pack_gauge(hi.gauge_field(L, seed=seed)))
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    return U, torch.randn((12, lat.V4, lat.Ls), dtype=torch.complex128, device="cuda:0", generator=g)


def _err(a, b):
    return float((a - b).abs().max()) / float(b.abs().max())


@pytest.mark.parametrize("L,Ls", [
    ((8, 8, 8, 16), 8),      # 2^13 sites: FP64 on tiles
    ((8, 8, 8, 18), 8),      # above: site kernel
    ((10, 10, 10, 10), 13),  # site kernel would fill the chip once and little more: tiles
    ((8, 8, 16, 16), 6),     # 2^14 sites: FP32 on single-slice tiles, FP64 on the site kernel
    ((8, 8, 16, 16), 12),    # 3 2^16 5d sites
    ((8, 8, 14, 18), 14),    # above: FP32 tiles of slice pairs
    ((12, 12, 12, 14), 11),  # odd Ls above 2^14 sites: FP32 on single-slice tiles
    ((12, 12, 12, 14), 16),
])
def test_continued_fraction_choices(L, Ls):
    torch = torch_dev()
    log(f"cf choices L={L} Ls={Ls}")
    lat = hd.Lattice(L, Ls, M5=1.7, bc=(1, -1, 1, -1))
    U, x = _fields(lat, L, 3)
    beta, R = list(0.3 + 0.1 * np.arange(Ls - 1)), 0.35
    ref = hd.apply_cf(lat.with_tune(dslash_variant=2), U, x, beta, R)
    assert _err(hd.apply_cf(lat.with_tune(dslash_variant=4), U, x, beta, R), ref) <= 1e-12
    assert _err(hd.apply_cf(lat, U, x, beta, R), ref) <= 1e-12
    U32, x32 = U.to(torch.complex64), x.to(torch.complex64)
    for variant in (0, 2, 4):
        assert _err(hd.apply_cf(lat.with_tune(dslash_variant=variant), U32, x32, beta, R), ref) <= 1e-5, variant


@pytest.mark.parametrize("L,Ls", [
    ((2, 2, 2, 2), 5),       # generic kernel below 32 sites
    ((4, 2, 2, 2), 5),       # site kernel from there
    ((4, 4, 4, 8), 64),      # FP64 on the tile kernel (2^15 5d sites)
    ((4, 4, 4, 9), 64),      # on the site kernel
    ((8, 8, 8, 8), 32),      # FP32 on the tile kernel (2^12 sites; 2^13 at Ls = 64)
    ((8, 8, 8, 9), 32),
    ((8, 8, 8, 16), 64),
    ((8, 8, 9, 15), 64),
])
def test_fine_apply_choices(L, Ls):
    torch = torch_dev()
    log(f"apply choices L={L} Ls={Ls}")
    lat = hd.Lattice(L, Ls, mf=0.05, bc=(1, -1, 1, -1))
    U, x = _fields(lat, L, 5)
    ref = hd.apply_fine(lat.with_tune(dslash_variant=2), U, x)
    assert _err(hd.apply_fine(lat, U, x), ref) <= 1e-12
    U32, x32 = U.to(torch.complex64), x.to(torch.complex64)
    assert _err(hd.apply_fine(lat, U32, x32), ref) <= 1e-5


@pytest.mark.parametrize("L,Ls", [
    ((4, 4, 2, 6), 8),       # parity tiles of slice pairs
    ((4, 6, 4, 4), 16),
    ((11, 9, 10, 14), 10),   # site kernels with slice pairs
])
def test_fields_aligned_to_one_entry(L, Ls):
    """FP32 fields need the alignment of an entry, 8 bytes; kernels with 16-byte accesses give the same
    bits for them as for fields on 16 bytes."""
    torch = torch_dev()
    log(f"alignment L={L} Ls={Ls}")
    lat = hd.Lattice(L, Ls, mf=0.05)
    U, x = _fields(lat, L, 7)
    U, x = U.to(torch.complex64), x.to(torch.complex64)

    def shifted(t):
        buf = torch.zeros(t.numel() + 2, dtype=t.dtype, device=t.device)
        view = buf[1:1 + t.numel()].view(t.shape)
        assert view.data_ptr() % 16 == 8
        return view.copy_(t)

    beta = list(0.3 + 0.1 * np.arange(Ls - 1))
    for f in (lambda u, v, o: hd.apply_fine(lat, u, v, out=o), lambda u, v, o: hd.apply_cf(lat, u, v, beta, 0.35, out=o)):
        assert torch.equal(f(shifted(U), shifted(x), shifted(torch.zeros_like(x))), f(U, x, torch.zeros_like(x)))


@pytest.mark.parametrize("Ls", [2, 3, 4, 5, 6, 7, 8, 14, 15, 17, 71, 72, 73])
def test_link_batches(Ls):
    """Site kernels at the work-items per site where their batches of link loads change, and where there
    are as many as link entries; odd extents, a short last workgroup."""
    torch = torch_dev()
    L, bc = (3, 5, 1, 3), (1, -1, 1, -1)
    log(f"link batches Ls={Ls}")
    lat = hd.Lattice(L, Ls, M5=1.8, mf=0.07, bc=bc)
    U, x = hi.gauge_field(L, seed=1), hi.gaussian_fermion(L, Ls, seed=0)
    ref = oracle.apply_h(U, x, oracle.Params(L, Ls, M5=1.8, mf=0.07, bc=bc))
    beta = list(0.2 + np.random.default_rng(Ls).random(Ls - 1))
    cf = oracle.apply_cf(U, x, 1.8, beta, 0.35, bc) if Ls <= 64 else None
    for dt, tol in ((torch.complex128, 1e-10), (torch.complex64, 1e-5)):
        Ud, xd = to_dev(hd.pack_gauge(U), dt), to_dev(hd.pack_fermion(x), dt)
        assert max_rel_elem(hd.unpack_fermion(to_host(hd.apply_fine(lat, Ud, xd)), L, Ls), ref) <= tol, dt
        if cf is not None:
            assert max_rel_elem(hd.unpack_fermion(to_host(hd.apply_cf(lat, Ud, xd, beta, 0.35)), L, Ls), cf) <= tol, dt
