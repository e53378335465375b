"""The misfit total that the gradient's last reduction adds up, at the edges of its 256 threads, alone and with
1024-thread blocks of tiles and probe units beside it."""
import pytest

from gpu_helpers import GRAD64_TOL, problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
E = pytest.importorskip("paper_2511_01793_amd.emagpie")


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("count", [1, 255, 256, 257, 2047, 2049])
def test_total_is_the_sum_of_the_patterns(count, dtype):
    """Against the sum of two halves' totals (float64 sums of the same terms, another order)."""
    print("case: gradient total", count, dtype, flush=True)
    p = problem("tiny", n=32 + 46, m=32, scan=("raster", 46, 1, 1), photons=1e5, B=8, L=1, alpha=0.05, seed=23)

    def total(lo, hi):
        d = torch.from_numpy(p.intensities[lo:hi]).cuda()
        rec = E.Reconstruction(p.positions[lo:hi], d, p.n, minibatch=8, levels=1, alpha=0.05, path="fused")
        obj, probe = torch.from_numpy(p.object_init).cuda(), torch.from_numpy(p.probe_init).cuda()
        out = [rec.grad(obj.to(dtype), probe.to(dtype))[2] for _ in range(3)]
        torch.cuda.synchronize()
        rec.close()
        vals = [float(x.item()) for x in out]
        assert vals[0] == vals[1] == vals[2]
        return vals[0]

    half = count // 2
    parts = (total(0, half) if half else 0.0) + total(half, count)
    assert abs(total(0, count) - parts) <= GRAD64_TOL * parts
