"""The sequential sweep with its workgroups taken to be on several XCDs: packets written through to memory,
bitwise the fused path."""
import numpy as np
import pytest

from gpu_helpers import init_state, problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
E = pytest.importorskip("paper_2511_01793_amd.emagpie")


def sweeps(p, path, positions, apart=False, epochs=2, **kw):
    d = torch.from_numpy(p.intensities).cuda()
    base = dict(minibatch=1, levels=2, alpha=p.alpha, seed=5, path=path)
    base.update(kw)
    rec = E.Reconstruction(positions, d, p.n, **base)
    rec.debug_chain(False, apart)
    obj, probe = init_state(p, rec)
    totals = []
    for e in range(epochs):
        s = torch.zeros((), dtype=torch.float64, device="cuda")
        rec.epoch(obj, probe, e, sampled=s)
        totals.append(s)
    torch.cuda.synchronize()
    rec.debug_chain()
    rec.close()
    return obj, probe, [float(x.item()) for x in totals]


@pytest.mark.parametrize("m, v", [(64, 0), (64, 1), (64, 2), (64, 3), (128, 0), (128, 1), (128, 2)])
@pytest.mark.parametrize("kind", ["raster", "same", "disjoint", "one pixel", "row apart"])
def test_written_through_packets(m, v, kind):
    print("case: chain apart", m, v, kind, flush=True)
    n = 3 * m + 4
    p = problem("tiny", n=n, m=m, scan=("raster", 8, (n - m - 2) // 7, 1), photons=1e6, B=1, L=2, alpha=0.05,
                seed=77)
    pos, N = p.positions.copy(), p.n_pos
    if kind == "same":
        pos[:] = [5, 9]
    elif kind == "disjoint":
        pos[:] = [[0, 0], [m, m], [0, m], [m, 0]] * (N // 4)
    elif kind == "one pixel":
        pos[:] = [[0, 0], [m - 1, m - 1]] * (N // 2)
    elif kind == "row apart":
        pos[:] = [[i % 2, 3] for i in range(N)]
    pos = pos.astype(np.int32)
    for kw in (dict(), dict(levels=3, joint_step=False, zero_phase_memory=True)):
        a, b = sweeps(p, "fused", pos, fft_plan=v, **kw), sweeps(p, "chain", pos, True, fft_plan=v, **kw)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and a[2] == b[2]
