"""Plain CR step by step: the state after 1 to 41 steps under the oracle's H, over the apply's forms
(inner products taken with the apply at Ls = 8 and 16 on even extents, with and without the summing of
many partials; a pass of their own otherwise), odd and even step counts (x takes two steps at a time)
and counts on both sides of the batches between read-backs."""
import numpy as np
import pytest

import hdcr_inputs as hi
import oracle
import paper_1611_06944_amd as hd
from tests.gpu_util import log, to_dev, to_host, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,Ls,steps", [
    ((4, 4, 4, 4), 16, (1, 2, 3, 8, 9)),
    ((4, 2, 4, 6), 8, (1, 2, 7, 41)),
    ((3, 4, 2, 4), 8, (2, 9)),        # odd extent
    ((4, 4, 2, 4), 12, (1, 10)),
    ((12, 12, 12, 12), 8, (3,)),      # 1296 workgroups of the apply: their partials are summed first
])
def test_cr_iterates(L, Ls, steps):
    torch_dev()
    log(f"CR steps L={L} Ls={Ls}")
    p = oracle.Params(L, Ls, M5=1.8, mf=0.02)
    lat = hd.Lattice(L, Ls, M5=1.8, mf=0.02)
    U = hi.gauge_field(L, seed=1)
    b = hi.gaussian_fermion(L, Ls, seed=0)
    Ud, bd = to_dev(hd.pack_gauge(U)), to_dev(hd.pack_fermion(b))
    ap = lambda f: oracle.apply_h(U, f, p)
    for k in steps:
        x, st, hist = hd.solve(lat, Ud, bd, params=hd.default_params(tol=1e-12, maxiter=k))
        ref = oracle.cr(ap, b, tol=1e-12, maxiter=k, check_true=False)
        assert st["outer_iters"] == k and len(hist) == k
        # x is the iterate whose residual the recurrence carries: each step adds a rounding of a few
        # eps |H| |x| (|H| <= 8, |x| below 10 |b|), under 1e-12 |b| over 41 steps
        true = oracle.norm(b - ap(hd.unpack_fermion(to_host(x), L, Ls))) / oracle.norm(b)
        assert abs(true - hist[-1]) <= 1e-12
        # the same minimal-residual sequence.  (The iterates themselves differ by up to 4e-11 between two
        # FP64 summation orders, for any form of the update: <r, Ar> is near zero for a random source.)
        np.testing.assert_allclose(hist, np.array(ref.history[:k]) / oracle.norm(b), rtol=1e-9)
