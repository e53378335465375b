"""Sequential sweeps whose workgroups do not get to run together: the roll call calls the sharing off and one
workgroup does the sweep, bitwise the fused path; sweeps of few steps, which go there at once."""
import pytest

from gpu_helpers import init_state, problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
E = pytest.importorskip("paper_2511_01793_amd.emagpie")


def small(m, side=4, seed=73):
    n = 3 * m + 4
    step = max(1, (n - m - 2) // (side - 1))
    return problem("tiny", n=n, m=m, scan=("raster", side, step, 1), photons=1e6, B=1, L=2, alpha=0.05,
                   seed=seed)


def rec_for(p, path, count=None, **kw):
    d = torch.from_numpy(p.intensities[:count]).cuda()
    base = dict(minibatch=1, levels=2, alpha=p.alpha, seed=5, path=path)
    base.update(kw)
    return E.Reconstruction(p.positions[:count], d, p.n, **base)


def sweeps(p, path, epochs=2, sampled=True, absent=False, **kw):
    rec = rec_for(p, path, **kw)
    rec.debug_chain(absent)
    obj, probe = init_state(p, rec)
    totals = []
    for e in range(epochs):
        s = torch.full((), -1.0, dtype=torch.float64, device="cuda")
        rec.epoch(obj, probe, e, sampled=s if sampled else None)
        totals.append(s)
    torch.cuda.synchronize()
    rec.debug_chain(False)  # reports a device error, if there was one
    rec.close()
    return obj, probe, [float(x.item()) for x in totals]


def same(a, b):
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and a[2] == b[2]


@pytest.mark.parametrize("m, v", [(32, 0), (32, 1), (64, 0), (64, 1), (64, 2), (64, 3), (128, 0),
                                  (128, 1), (128, 2)])
@pytest.mark.parametrize("kw", [dict(levels=1), dict(levels=3, sampled=False), dict(joint_step=False),
                                dict(update_probe=False), dict(zero_phase_memory=True)], ids=str)
def test_a_sweep_called_off_runs_in_one_workgroup(m, v, kw):
    """At m = 32 from 36 steps, where the sweep is shared (with the summing workgroup) at all."""
    print("case: chain called off", m, v, kw, flush=True)
    p = small(m, 6 if m == 32 else 3)
    ref = sweeps(p, "fused", fft_plan=v, **kw)
    same(ref, sweeps(p, "chain", fft_plan=v, absent=True, **kw))
    if m == 32:
        same(ref, sweeps(p, "chain", fft_plan=v, **kw))


@pytest.mark.parametrize("m", [32, 64, 128])
@pytest.mark.parametrize("count", [1, 2, 3, 15, 16, 31, 32, 33])
def test_sweeps_of_few_steps(m, count):
    print("case: chain steps", m, count, flush=True)
    p = small(m, 6)
    for sampled in (True, False):
        same(sweeps(p, "fused", count=count, sampled=sampled), sweeps(p, "chain", count=count, sampled=sampled))


def test_more_sweeps_at_once_than_fit_one_xcd():
    """Eight sweeps of 17 workgroups on eight streams, three times: all end, all bitwise the fused path."""
    print("case: eight chains at once", flush=True)
    ps = [small(128, seed=80 + i) for i in range(8)]
    refs = [sweeps(p, "fused", epochs=3) for p in ps]
    recs = [rec_for(p, "chain") for p in ps]
    states = [init_state(p, r) for p, r in zip(ps, recs)]
    sums = [[torch.zeros((), dtype=torch.float64, device="cuda") for _ in range(3)] for _ in ps]
    streams = [torch.cuda.Stream() for _ in ps]
    torch.cuda.synchronize()
    for e in range(3):
        for rec, (o, q), s, st in zip(recs, states, sums, streams):
            with torch.cuda.stream(st):
                rec.epoch(o, q, e, sampled=s[e])
    torch.cuda.synchronize()
    for rec, (o, q), s, ref in zip(recs, states, sums, refs):
        rec.debug_chain(False)
        same((o, q, [float(x.item()) for x in s]), ref)
        rec.close()


@pytest.mark.parametrize("absent", [False, True])
def test_captured_sweep_is_decided_at_each_replay(absent):
    """One captured sweep, replayed between eager work: bitwise eager sweeps of the same order."""
    print("case: captured chain", absent, flush=True)
    p = small(64)
    rec = rec_for(p, "chain")
    perm = torch.arange(p.n_pos, dtype=torch.int32, device="cuda").flip(0).contiguous()
    obj, probe = init_state(p, rec)
    s = torch.zeros((), dtype=torch.float64, device="cuda")
    ref = []
    for _ in range(3):
        rec.epoch(obj, probe, 0, perm=perm, sampled=s)
        torch.cuda.synchronize()
        ref.append((obj.clone(), probe.clone(), s.item()))
    rec.debug_chain(absent)
    obj, probe = init_state(p, rec)
    start = obj.clone(), probe.clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        rec.epoch(obj, probe, 0, perm=perm, sampled=s)
    torch.cuda.synchronize()
    obj.copy_(start[0])
    probe.copy_(start[1])
    for want in ref:
        g.replay()
        torch.cuda.synchronize()
        same((obj, probe, s.item()), want)
        (obj.abs().sum() + probe.abs().sum()).item()
    del g
    rec.close()


@pytest.mark.parametrize("m, absent", [(32, False), (64, False), (64, True)])
def test_given_up_waits_leave_the_sweep_together(m, absent):
    """Waits made to give up end the launch normally and are reported once; a sweep that is called
    off has no such wait.  The context works afterwards."""
    print("case: chain give up", m, absent, flush=True)
    p = small(m, 6)
    rec = rec_for(p, "chain")
    rec.debug_barrier(100, 1)
    rec.debug_chain(absent)
    obj, probe = init_state(p, rec)
    s = torch.zeros((), dtype=torch.float64, device="cuda")
    rec.epoch(obj, probe, 0, sampled=s)
    torch.cuda.synchronize()
    if not absent:
        with pytest.raises(E.EmagpieError) as err:
            rec.debug_barrier(0, 0)
        assert err.value.name == "E_HIP"
    rec.debug_barrier(0, 0)
    rec.debug_chain(False)
    obj, probe = init_state(p, rec)
    totals = []
    for e in range(2):
        s = torch.zeros((), dtype=torch.float64, device="cuda")
        rec.epoch(obj, probe, e, sampled=s)
        totals.append(s)
    torch.cuda.synchronize()
    rec.close()
    same((obj, probe, [float(x.item()) for x in totals]), sweeps(p, "fused"))


def test_a_worker_alone_leaves_the_scratch_as_it_is():
    """m = 32 without the sampled misfit is one workgroup's work: nothing is exchanged, and nothing cleared
    for it (the exchange scratch is the end of the workspace)."""
    print("case: chain without scratch", flush=True)
    p = small(32, 6)
    rec = rec_for(p, "chain")
    obj, probe = init_state(p, rec)
    end = rec._ws_ptr - rec._ws.data_ptr() + E.workspace_size(rec.cfg)
    scratch = rec._ws[end - (64 << 10):end]
    scratch.fill_(0x5A)
    rec.epoch(obj, probe, 0)
    torch.cuda.synchronize()
    assert bool((scratch == 0x5A).all())
    rec.epoch(obj, probe, 1, sampled=torch.zeros((), dtype=torch.float64, device="cuda"))
    torch.cuda.synchronize()
    assert not bool((scratch == 0x5A).all())
    rec.close()
