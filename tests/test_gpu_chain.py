"""Sequential sweeps (minibatch 1, one launch; several workgroups at m = 64 and 128): bitwise the fused path with
minibatch 1 in every option, window overlaps of every kind, two sweeps at once, and the error path."""
import numpy as np
import pytest

from gpu_helpers import init_state, problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
E = pytest.importorskip("paper_2511_01793_amd.emagpie")


def sweep(p, path, positions=None, epochs=2, sampled=True, n=None, **kw):
    d = torch.from_numpy(p.intensities).cuda()
    base = dict(minibatch=1, levels=2, alpha=p.alpha, alpha_z=p.alpha_z, seed=5, path=path)
    base.update(kw)
    rec = E.Reconstruction(p.positions if positions is None else positions, d, p.n if n is None else n,
                           **base)
    obj, probe = init_state(p, rec)
    if n is not None:
        obj = torch.ones(n, dtype=torch.complex64, device="cuda")
    out = []
    for e in range(epochs):
        s = torch.zeros((), dtype=torch.float64, device="cuda") if sampled else None
        rec.epoch(obj, probe, e, sampled=s)
        out.append(s)
    torch.cuda.synchronize()
    rec.close()
    return obj, probe, [float(x.item()) if x is not None else None for x in out]


def small(m, side=4):
    n = 3 * m + 4
    step = max(1, (n - m - 2) // (side - 1))
    return problem("tiny", n=n, m=m, scan=("raster", side, step, 1), photons=1e6, B=1, L=2, alpha=0.05,
                   seed=67)


def same(a, b):
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and a[2] == b[2]


@pytest.mark.parametrize("m, v", [(32, 0), (32, 1), (64, 0), (64, 1), (64, 2), (64, 3), (128, 0),
                                  (128, 1), (128, 2)])
@pytest.mark.parametrize("kw", [dict(levels=1), dict(levels=3), dict(joint_step=False, levels=1),
                                dict(update_probe=False), dict(alpha_z=0.5), dict(alpha=0.0),
                                dict(zero_phase_memory=True)], ids=str)
def test_every_option_is_bitwise_the_fused_path(m, v, kw):
    print("case: chain option", m, v, kw, flush=True)
    p = small(m, 3)
    same(sweep(p, "fused", fft_plan=v, **kw), sweep(p, "chain", fft_plan=v, **kw))


@pytest.mark.parametrize("m", [32, 64, 128])
@pytest.mark.parametrize("kind", ["same", "disjoint", "one pixel", "row apart", "rectangular", "single"])
def test_window_overlaps(m, kind):
    """Successive windows that coincide, do not meet, share one pixel or all but one row, on a
    rectangular object, and a sweep of one position; without the sampled misfit as well."""
    print("case: chain overlap", m, kind, flush=True)
    p = small(m)
    n, N = None, p.n_pos
    pos = p.positions.copy()
    if kind == "same":
        pos[:] = [5, 9]
    elif kind == "disjoint":
        pos[:] = [[0, 0], [m, m], [0, m], [m, 0]] * (N // 4)
    elif kind == "one pixel":
        pos[:] = [[0, 0], [m - 1, m - 1]] * (N // 2)
    elif kind == "row apart":
        pos[:] = [[i % 2, 3] for i in range(N)]
    elif kind == "rectangular":
        n = (2 * m + 3, 3 * m + 1)
        pos = np.minimum(pos, [m + 3, 2 * m + 1]).astype(np.int32)
    else:
        p.intensities, pos = p.intensities[:1], pos[:1]
    for sampled in (True, False):
        same(sweep(p, "fused", pos, sampled=sampled, n=n), sweep(p, "chain", pos, sampled=sampled, n=n))


def test_two_sweeps_on_two_streams():
    print("case: two chains at once", flush=True)
    ps = [small(64), small(128)]
    ref = [sweep(p, "fused", epochs=3) for p in ps]
    recs, states, streams = [], [], [torch.cuda.Stream(), torch.cuda.Stream()]
    for p in ps:
        d = torch.from_numpy(p.intensities).cuda()
        rec = E.Reconstruction(p.positions, d, p.n, minibatch=1, levels=2, alpha=p.alpha, seed=5, path="chain")
        recs.append(rec)
        states.append(init_state(p, rec))
    torch.cuda.synchronize()
    sums = [[torch.zeros((), dtype=torch.float64, device="cuda") for _ in range(3)] for _ in ps]
    torch.cuda.synchronize()
    for e in range(3):
        for rec, (o, q), s, st in zip(recs, states, sums, streams):
            with torch.cuda.stream(st):
                rec.epoch(o, q, e, sampled=s[e])
    torch.cuda.synchronize()
    for (o, q), s, r in zip(states, sums, ref):
        same((o, q, [float(x.item()) for x in s]), r)
    for rec in recs:
        rec.close()


@pytest.mark.parametrize("sampled", [True, False])
def test_waits_that_give_up_are_reported(sampled):
    """Every wait is made to give up after a few polls: the launch ends normally, the next call
    raises E_HIP once, and the context works again."""
    print("case: chain error path", sampled, flush=True)
    p = small(128, 3)
    d = torch.from_numpy(p.intensities).cuda()
    rec = E.Reconstruction(p.positions, d, p.n, minibatch=1, levels=2, alpha=p.alpha, alpha_z=p.alpha_z,
                           seed=5, path="chain")
    obj, probe = init_state(p, rec)
    rec.debug_barrier(100, 1)
    s = torch.zeros((), dtype=torch.float64, device="cuda")
    rec.epoch(obj, probe, 0, sampled=s if sampled else None)
    torch.cuda.synchronize()
    with pytest.raises(E.EmagpieError) as err:
        rec.epoch(obj, probe, 0)
    assert err.value.name == "E_HIP"
    rec.debug_barrier(0, 0)
    obj, probe = init_state(p, rec)
    out = []
    for e in range(2):
        s = torch.zeros((), dtype=torch.float64, device="cuda")
        rec.epoch(obj, probe, e, sampled=s)
        out.append(s)
    torch.cuda.synchronize()
    rec.close()
    same((obj, probe, [float(x.item()) for x in out]), sweep(p, "fused"))
