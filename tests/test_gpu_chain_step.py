"""Single minibatch-1 steps on the chain path: the sampled misfit is added to the caller's total."""
import pytest

from gpu_helpers import init_state, problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
E = pytest.importorskip("paper_2511_01793_amd.emagpie")


def small(m):
    n = 2 * m + 9
    return problem("tiny", n=n, m=m, scan=("raster", 3, (m + 4) // 2, 1), photons=1e6, B=1, L=2, alpha=0.05,
                   seed=71)


def steps(p, path, sampled=True):
    d = torch.from_numpy(p.intensities).cuda()
    rec = E.Reconstruction(p.positions, d, p.n, minibatch=1, levels=2, alpha=p.alpha, seed=5, path=path)
    obj, probe = init_state(p, rec)
    total = torch.full((), 3.5, dtype=torch.float64, device="cuda")
    for k in (4, 0, 4):
        rec.step(obj, probe, [k], sampled=total if sampled else None)
    torch.cuda.synchronize()
    rec.close()
    return obj, probe, float(total.item())


@pytest.mark.parametrize("sampled", [True, False])
@pytest.mark.parametrize("m", [32, 64, 128])
def test_steps_add_their_sampled_misfit(m, sampled):
    """Bitwise the fused path's object, probe and total, which starts from the caller's 3.5."""
    print("case: chain step", m, sampled, flush=True)
    p = small(m)
    fused, chain = steps(p, "fused", sampled), steps(p, "chain", sampled)
    assert torch.equal(fused[0], chain[0]) and torch.equal(fused[1], chain[1])
    assert fused[2] == chain[2] and (fused[2] > 3.5 if sampled else fused[2] == 3.5)
