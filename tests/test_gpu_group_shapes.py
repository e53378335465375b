"""The group's finalize reads slots with a bounds check instead of a branch per pixel: every
tile shape and probe side, objects that are no multiple of the tiles, windows at the edges,
and more slots than one scan of 256, bitwise against the members alone."""
import numpy as np
import pytest

from gpu_helpers import init_state, make_rec, problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape", range(4))
def test_group_equals_members_for_every_tile_shape(shape):
    import paper_2511_01793_amd.emagpie as E
    print("case: group finalize shape", shape, flush=True)
    specs = [dict(n=77, m=32, scan=("raster", 18, 2, 1), B=324, L=1), dict(n=131, m=64, scan=("raster", 4, 21, 0), B=5, L=2),
             dict(n=201, m=128, scan=("raster", 3, 36, 0), B=9, L=3), dict(n=33, m=32, scan=("raster", 2, 1, 0), B=3, L=1)]
    ps = [problem("tiny", alpha=0.05, photons=1e6, seed=61 + i, **s) for i, s in enumerate(specs)]
    ends = []
    for grouped in (False, True):
        recs = [make_rec(p, seed=500 + i, finalize_shape=shape) for i, p in enumerate(ps)]
        states = [init_state(p, r) for p, r in zip(ps, recs)]
        if grouped:
            grp = E.Group(recs)
            for e in range(2):
                grp.epoch([o for o, _ in states], [q for _, q in states], e)
        else:
            for r, (o, q) in zip(recs, states):
                for e in range(2):
                    r.epoch(o, q, e)
        torch.cuda.synchronize()
        ends.append([(o.cpu().numpy(), q.cpu().numpy()) for o, q in states])
        if grouped:
            grp.close()
        for r in recs:
            r.close()
    for a, b in zip(*ends):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("with_memory", [(), (1,), (0, 1, 2)])
def test_group_of_members_with_and_without_phase_memory(with_memory):
    """A group without any phase memory runs the kernel that knows none; members with one and
    without share a launch otherwise.  Bitwise the members alone, over three sweeps."""
    import paper_2511_01793_amd.emagpie as E
    print("case: group phase memory", with_memory, flush=True)
    ps = [problem("tiny", n=100 + 20 * i, m=32, scan=("raster", 5, 12, 1), photons=200.0, B=4, L=2, alpha=0.05,
                  seed=71 + i) for i in range(3)]
    ends = []
    for grouped in (False, True):
        recs = [E.Reconstruction(p.positions, torch.from_numpy(p.intensities).cuda(), p.n, minibatch=p.minibatch,
                                 levels=p.levels, alpha=p.alpha, alpha_z=p.alpha_z, path="fused", seed=9 + i,
                                 zero_phase_memory=i in with_memory) for i, p in enumerate(ps)]
        states = [init_state(p, r) for p, r in zip(ps, recs)]
        grp = E.Group(recs) if grouped else None
        for e in range(3):
            if grouped:
                grp.epoch([o for o, _ in states], [q for _, q in states], e)
            else:
                for r, (o, q) in zip(recs, states):
                    r.epoch(o, q, e)
        torch.cuda.synchronize()
        ends.append([(o.cpu().numpy(), q.cpu().numpy()) for o, q in states])
        if grouped:
            grp.close()
        for r in recs:
            r.close()
    for a, b in zip(*ends):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
