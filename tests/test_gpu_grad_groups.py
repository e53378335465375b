"""The gradient where a patch-stage workgroup takes several patterns (more patterns than
workgroups: 256 at m = 128, 512 at m = 64, 1024 at m = 32), for every FFT plan, and over several
chunks, against the oracle and against sums of parts."""
from types import SimpleNamespace

import pytest

from oracle import emagpie_oracle as O
from gpu_helpers import GRAD32_TOL, GRAD64_TOL, MISFIT_TOL, amps, host, init_state, make_rec, problem, rel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FIELDS = ("n", "minibatch", "levels", "alpha", "alpha_z")
CASES = [(128, 0, 17), (128, 1, 17), (128, 2, 17), (64, 0, 23), (64, 1, 23), (64, 2, 23), (64, 3, 33),
         (32, 0, 33), (32, 1, 33)]


@pytest.mark.parametrize("m, v, side", CASES)
def test_many_patterns_per_workgroup(m, v, side):
    print("case: gradient groups", m, v, side * side, flush=True)
    p = problem("tiny", n=m + side + 3, m=m, scan=("raster", side, 1, 1), photons=1e5, B=8, L=1, alpha=0.05,
                seed=17)
    rec = make_rec(p, fft_plan=v)
    obj, probe = init_state(p, rec)
    rec.epoch(obj, probe, 0)  # leave the phase-free initial guess
    torch.cuda.synchronize()
    rz, rq, ref = O.gradients(host(probe), host(obj), p.positions, amps(p))
    for dtype, tol in ((torch.complex64, GRAD32_TOL), (torch.complex128, GRAD64_TOL)):
        if dtype == torch.complex128 and m == 128:
            continue
        gz, gq, phi = rec.grad(obj.to(dtype), probe.to(dtype))
        torch.cuda.synchronize()
        assert rel(host(gz), rz) < tol and rel(host(gq), rq) < tol, (dtype, rel(host(gz), rz), rel(host(gq), rq))
        assert abs(float(phi.item()) - ref) <= MISFIT_TOL * ref
    rec.close()


@pytest.mark.parametrize("m, side", [(32, 130), (64, 65)])
def test_several_chunks(m, side):
    """More patterns than one chunk holds (16384 at m = 32, 4096 at m = 64): the chunks add up."""
    print("case: gradient chunks", m, side * side, flush=True)
    p = problem("tiny", n=m + side + 3, m=m, scan=("raster", side, 1, 1), photons=1e5, B=8, L=1, alpha=0.05,
                seed=19)
    rec = make_rec(p)
    obj, probe = init_state(p, rec)
    gz, gq, phi = rec.grad(obj, probe)
    gz64, gq64, phi64 = rec.grad(obj.to(torch.complex128), probe.to(torch.complex128))
    # the same sum taken pattern group by pattern group, each in one chunk
    half = len(p.positions) // 2
    sz, sq, sphi = 0, 0, 0.0
    for lo, hi in ((0, half), (half, len(p.positions))):
        part = SimpleNamespace(**{**{k: getattr(p, k) for k in FIELDS}, "positions": p.positions[lo:hi],
                                  "intensities": p.intensities[lo:hi]})
        r = make_rec(part)
        a, b, c = r.grad(obj.to(torch.complex128), probe.to(torch.complex128))
        sz, sq, sphi = sz + host(a), sq + host(b), sphi + float(c.item())
        r.close()
    torch.cuda.synchronize()
    for z, q, f, tol in ((gz, gq, phi, GRAD32_TOL), (gz64, gq64, phi64, GRAD64_TOL)):
        assert rel(host(z), sz) < tol and rel(host(q), sq) < tol
        assert abs(float(f.item()) - sphi) <= MISFIT_TOL * sphi
    rec.close()
