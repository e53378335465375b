"""m = 256: the full misfit and the gradient over more patterns than one chunk of the stack buffer
holds (256 and 128), with counts that are no multiple of the XCD count, against the oracle."""
import numpy as np
import pytest

from oracle import emagpie_oracle as O
from gpu_helpers import GRAD32_TOL, MISFIT_TOL, amps, host, init_state, make_rec, problem, rel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("side, minibatch", [(12, 3), (17, 300)])
def test_misfit_and_gradient_over_several_chunks(side, minibatch):
    print("case: m256 chunks", side, minibatch, flush=True)
    p = problem("tiny", n=300, m=256, scan=("raster", side, 2, 1), photons=1e6, B=min(minibatch, side * side),
                L=2, alpha=0.05, seed=91)
    rec = make_rec(p)
    obj, probe = init_state(p, rec)
    rec.epoch(obj, probe, 0)  # leave the phase-free initial guess
    phi = rec.misfit(obj, probe)
    gz, gq, phi_g = rec.grad(obj, probe)
    torch.cuda.synchronize()
    a = amps(p)
    rz, rq, ref = O.gradients(host(probe), host(obj), p.positions, a)
    assert abs(float(phi.item()) - ref) <= MISFIT_TOL * ref
    assert abs(float(phi_g.item()) - ref) <= MISFIT_TOL * ref
    assert rel(host(gz), rz) < GRAD32_TOL and rel(host(gq), rq) < GRAD32_TOL
    rec.close()
