"""Plain CR on a lattice with long steps: few applications of H run behind the stop."""
import pytest

import hdcr_inputs as hi
import paper_1611_06944_amd as hd
from tests.gpu_util import log, to_dev, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tol,behind", [(0.9, 2), (0.3, 2), (0.03, 8)])
def test_steps_behind_the_stop(tol, behind):
    """16^4 x 8, the smallest lattice whose steps count as long.  Beside the steps there are the first
    residual and the true one; batches are at most a quarter of the steps before them, or two."""
    torch = torch_dev()
    L, Ls = (16, 16, 16, 16), 8
    log(f"CR steps behind the stop tol={tol}")
    lat = hd.Lattice(L, Ls, M5=1.8, mf=0.05)
    U = to_dev(hd.pack_gauge(hi.gauge_field(L, seed=1)))
    g = torch.Generator(device="cuda:0").manual_seed(3)
    b = torch.randn((12, lat.V4, Ls), dtype=torch.complex128, device="cuda:0", generator=g)
    x, st, hist = hd.solve(lat, U, b, params=hd.default_params(tol=tol, maxiter=200))
    assert st["status"] == 0 and st["true_rel_residual"] <= tol and len(hist) == st["outer_iters"]
    r = b - hd.apply_fine(lat, U, x)
    assert float(r.norm() / b.norm()) == pytest.approx(st["true_rel_residual"], rel=1e-10)
    assert st["outer_iters"] + 2 <= st["fine_applies_f64"] <= st["outer_iters"] + 2 + behind
