"""The coarse CR's step kernel at the edges of its split: one site, matrices too small for one batch of
loads, rows that do not fill a 16-byte load, more rows than the prefetched rounds, several sites to a
workgroup with a short last one, and partial sums of more than one round."""
import numpy as np
import pytest

import oracle
import paper_1611_06944_amd as hd
from tests.gpu_util import log, max_rel_elem, to_dev, to_host, torch_dev

pytestmark = pytest.mark.gpu

SHAPES = [
    # L, Ls, block, nvec
    ((2, 2, 2, 2), 4, (2, 2, 2, 2), 1),     # one site, every neighbour itself
    ((2, 4, 2, 2), 4, (1, 2, 2, 1), 5),     # Nb = 10
    ((2, 2, 2, 6), 6, (2, 2, 2, 2), 37),    # Nb = 74: two lanes to a row, single-entry loads
    ((4, 2, 2, 2), 8, (2, 2, 2, 2), 64),    # Nb = 128: the largest
    ((7, 7, 7, 3), 4, (1, 1, 1, 1), 3),     # 1029 sites: two to a workgroup, one to the last
    ((8, 8, 8, 6), 4, (1, 1, 1, 1), 8),     # 3072 sites: three and four to a workgroup
]


def _operator(cdims, nb, seed):
    """Hermitian, spectrum in about [2, 4]: A[a, 5+mu] = A[a-mu, 1+mu]^dag."""
    rng = np.random.default_rng(seed)
    C = tuple(reversed(cdims))
    A = rng.standard_normal(C + (9, nb, nb)) + 1j * rng.standard_normal(C + (9, nb, nb))
    A /= 6.0 * np.sqrt(9.0 * nb)
    for mu in range(4):
        A[..., 5 + mu, :, :] = np.roll(A[..., 1 + mu, :, :], 1, axis=3 - mu).conj().swapaxes(-1, -2)
    A[..., 0, :, :] = 0.5 * (A[..., 0, :, :] + A[..., 0, :, :].conj().swapaxes(-1, -2)) + 3.0 * np.eye(nb)
    return A.reshape(-1, 9, nb, nb)


@pytest.mark.parametrize("L,Ls,block,nvec", SHAPES)
def test_steps_match_oracle(L, Ls, block, nvec):
    """Four fixed steps against the oracle's CR on the stored values.  The operator is well conditioned,
    so the iterate carries the rounding of four applies of 9 Nb <= 1152 terms: at most 5e-13 in FP64 and
    3e-4 in FP32 vectors, and some hundredth of that at random signs."""
    torch = torch_dev()
    lat = hd.Lattice(L, Ls, block=block, nvec=nvec)
    cdims = tuple(l // b for l, b in zip(L, block))
    A64 = to_dev(np.ascontiguousarray(_operator(cdims, lat.nb, 3).swapaxes(2, 3)))
    rng = np.random.default_rng(4)
    b = rng.standard_normal((lat.nc, lat.nb)) + 1j * rng.standard_normal((lat.nc, lat.nb))
    for dt, tol in ((hd.C128, 1e-12), (hd.C64, 3e-5), (hd.BF16C, 3e-5)):
        log(f"coarse step L={L} block={block} nvec={nvec} dtype={dt}")
        A = A64 if dt == hd.C128 else hd.convert_coarse(lat, A64, dt)
        vdt = torch.complex128 if dt == hd.C128 else torch.complex64
        bd = to_dev(b, vdt)
        ref = oracle.coarse_cr(to_host(hd.export_coarse(lat, A, dt)), to_host(bd).astype(np.complex128), cdims, tol=0.0,
                               maxiter=4)
        for _ in range(2):  # the workspace of the second solve holds the first one's values
            x, it, code = hd.coarse_solve(lat, A, dt, bd, maxiter=4, tol=0.0, return_status=True)
            assert code == 0 and it == 4 and ref.iters == 4
            assert max_rel_elem(to_host(x), ref.x) <= tol


@pytest.mark.parametrize("L,Ls,block,nvec", [SHAPES[0], SHAPES[2], SHAPES[3], ((4, 6, 2, 2), 4, (2, 2, 2, 2), 24),
                                             ((2, 4, 2, 2), 4, (1, 2, 2, 1), 5)])
def test_apply_every_group_size(L, Ls, block, nvec):
    """Right-hand sides in groups of 1, 2, 3, 4, 6 and 8, full and short, fewer of them where the vectors
    do not fit LDS (Nb = 128 in FP64): against the oracle, and each against its own single apply bit for
    bit.  9 Nb <= 1152 products to an entry: 1e-12 and 3e-5 of the largest entry."""
    torch = torch_dev()
    lat = hd.Lattice(L, Ls, block=block, nvec=nvec)
    cdims = tuple(l // b for l, b in zip(L, block))
    A64 = to_dev(np.ascontiguousarray(_operator(cdims, lat.nb, 5).swapaxes(2, 3)))
    rng = np.random.default_rng(6)
    v = rng.standard_normal((17, lat.nc, lat.nb)) + 1j * rng.standard_normal((17, lat.nc, lat.nb))
    for dt, tol in ((hd.C128, 1e-12), (hd.C64, 3e-5), (hd.BF16C, 3e-5)):
        log(f"coarse apply L={L} block={block} nvec={nvec} dtype={dt}")
        A = A64 if dt == hd.C128 else hd.convert_coarse(lat, A64, dt)
        vd = to_dev(v, torch.complex128 if dt == hd.C128 else torch.complex64)
        A_log = to_host(hd.export_coarse(lat, A, dt))
        ref = np.stack([oracle.coarse_apply(A_log, x.astype(np.complex128), cdims) for x in to_host(vd)])
        one = torch.cat([hd.apply_coarse(lat, A, dt, vd[r:r + 1].contiguous()) for r in range(17)])
        assert max_rel_elem(to_host(one), ref) <= tol
        for n in (2, 3, 4, 5, 6, 7, 8, 9, 12, 17):
            assert torch.equal(hd.apply_coarse(lat, A, dt, vd[:n].contiguous()), one[:n]), (dt, n)
