"""Error paths of the C ABI on the GPU: a device allocation that fails
(forced with vam_debug_fail_allocations) must leave every handle either
unchanged or refusing to run, never half-built, and the next call without
the failure must work."""
import math
import sys

import numpy as np
import pytest

import oracle
import synth
from synth.configs import scaled

torch = pytest.importorskip("torch")
import paper_2211_03516_amd as vam

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _p(n=32, n_angles=6):
    F = (n / 2) / math.tan(math.radians(10))
    return scaled(synth.workload("c2"), nx=n, ny=n, nz=n, nu=n, nv=n, focus=F,
                  pupil=F * math.tan(math.radians(6.1)), n_pupil=4, r_outer=0.47 * n,
                  r_inner=0.44 * n, alpha=0.02, n_angles=n_angles)


def _inputs(p, seed):
    rng = synth.SplitMix64(seed)
    n = p["nx"]
    x = torch.from_numpy(rng.uniform(n ** 3).reshape(n, n, n).astype(np.float32)).to(DEV)
    y = torch.from_numpy(rng.uniform(p["n_angles"] * n * n).reshape(p["n_angles"], n, n)
                         .astype(np.float32)).to(DEV)
    return x, y


@pytest.fixture(autouse=True)
def _hook_off():
    yield
    vam.debug_fail_allocations(0)


def test_failed_box_rebuild_refuses_then_recovers():
    p = _p()
    x, y = _inputs(p, 51)
    g = vam.Geometry(p)
    P0, D0 = g.forward(x), g.back(y)
    failed = 0
    for k in range(1, 40):
        say("rebuild with allocation %d failing" % k)
        vam.debug_fail_allocations(k)
        try:
            g.set_box_edge(8)
        except vam.VamError as e:
            vam.debug_fail_allocations(0)
            assert e.status == vam.VAM_ERR_OUT_OF_MEMORY
            failed += 1
            # no box decomposition now: both operators refuse, nothing runs
            with pytest.raises(vam.VamError):
                g.forward(x)
            with pytest.raises(vam.VamError):
                g.back(y)
            g.set_box_edge(12)
            assert torch.equal(g.forward(x), P0)
            assert float((g.back(y) - D0).abs().max()) <= 1e-6 * float(D0.abs().max())
            continue
        vam.debug_fail_allocations(0)
        break   # the rebuild makes fewer than k allocations
    say("%d rebuild allocations failed in turn" % failed)
    assert failed >= 8
    g.close()


def test_failed_setup_and_first_step_allocations():
    p = _p(24, n_angles=4)
    t = torch.zeros((24, 24, 24), device=DEV)
    t[8:16, 8:16, 8:16] = 1.0
    # every allocation of the set-up in turn: an error, and no handle
    for k in range(1, 40):
        vam.debug_fail_allocations(k)
        try:
            g = vam.Geometry(p)
        except vam.VamError as e:
            assert e.status == vam.VAM_ERR_OUT_OF_MEMORY
            continue
        finally:
            vam.debug_fail_allocations(0)
        break
    say("set-up succeeded once %d allocations were allowed to pass" % (k - 1))
    assert k > 5
    # the optimisation step's buffers: each of its four allocations in turn
    proj = g.forward(t)
    ref = proj.clone()
    g.optimize_step(t, ref, lr=0.1, want_loss=False)
    for k in range(1, 5):
        g2 = vam.Geometry(p)
        gp = proj.clone()
        vam.debug_fail_allocations(k)
        with pytest.raises(vam.VamError):
            g2.optimize_step(t, gp, lr=0.1)
        vam.debug_fail_allocations(0)
        assert torch.equal(gp, proj)          # nothing was launched
        g2.optimize_step(t, gp, lr=0.1)
        assert float((gp - ref).abs().max()) <= 1e-5 * float(ref.abs().max())
        g2.close()
    g.close()


def test_failed_first_forward_allocations():
    """The forward's first call allocates its 64-bit fixed-point projections
    and the volume maximum: either allocation failing is an error that writes
    nothing to the output, and the next call gives the same projections as
    a handle whose first call succeeded."""
    p = _p(24, n_angles=4)
    t = torch.zeros((24, 24, 24), device=DEV)
    t[6:18, 8:16, 5:19] = 1.0
    g0 = vam.Geometry(p)
    ref = g0.forward(t)
    g0.close()
    for k in (1, 2):
        g = vam.Geometry(p)
        out = torch.full_like(ref, 7.0)
        vam.debug_fail_allocations(k)
        try:
            with pytest.raises(vam.VamError) as e:
                g.forward(t, out=out)
            assert e.value.status == vam.VAM_ERR_OUT_OF_MEMORY
        finally:
            vam.debug_fail_allocations(0)
        torch.cuda.synchronize()
        assert bool((out == 7.0).all())
        assert torch.equal(g.forward(t), ref)
        g.close()


def test_turned_volumes_only_where_calls_need_them():
    """The volumes of the angles a quarter turn apart: not allocated by calls
    inside one quarter, tried again after an attempt that failed, and given back
    when memory is short at an allocation that a call has to make; the results
    are the same bits throughout."""
    p = _p(24, n_angles=8)
    x, y = _inputs(p, 53)
    g0 = vam.Geometry(p)
    P0, D0 = g0.forward(x), g0.back(y)
    g0.close()
    g = vam.Geometry(p)
    say("inside one quarter")
    vam.debug_fail_allocations(3)              # projections, maximum, then the next one
    assert torch.equal(g.forward(x, angle_begin=2, angle_count=2), P0[2:4])
    with pytest.raises(vam.VamError):
        g.back(y)                              # ... which is the dose accumulator
    say("an attempt that fails")
    vam.debug_fail_allocations(1)
    assert torch.equal(g.forward(x), P0)
    say("tried again")
    vam.debug_fail_allocations(1)
    assert torch.equal(g.forward(x), P0)       # this attempt fails again, so the hook is off now
    assert torch.equal(g.forward(x), P0)       # and this one is made
    say("given back")
    for k in (1, 2):                           # with and without them in the handle
        vam.debug_fail_allocations(1)
        if k == 1:
            assert torch.equal(g.back(y), D0)
            vam.debug_fail_allocations(0)
        else:
            with pytest.raises(vam.VamError):
                g.optimize_step(x, y.clone(), lr=0.1, want_loss=False)
    assert torch.equal(g.forward(x), P0)
    g.close()


def test_forward_of_a_whole_turn_captured_before_its_volumes_exist():
    """A graph captured after calls inside one quarter only: captured calls
    allocate nothing, and every replay gives the eager bits, also with eager
    calls in between that allocate the turned volumes, and after the handle
    was short of memory."""
    p = _p(24, n_angles=8)
    x, y = _inputs(p, 54)
    g = vam.Geometry(p)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        g.forward(x, angle_begin=0, angle_count=2)
        out, out2 = torch.empty((8, 24, 24), device=DEV), torch.empty((8, 24, 24), device=DEV)
        s.synchronize()
        early, late = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
        say("capture before the volumes exist")
        with torch.cuda.graph(early, stream=s):
            g.forward(x, out=out)
        ref = g.forward(x)
        say("capture after")
        with torch.cuda.graph(late, stream=s):
            g.forward(x, out=out2)
        for i in range(4):
            x.mul_(0.5).add_(0.1 * i)
            early.replay()
            late.replay()
            ref = g.forward(x)
            s.synchronize()
            assert torch.equal(out, ref) and torch.equal(out2, ref), i
            if i == 1:                         # a captured call uses the volumes: they stay
                vam.debug_fail_allocations(1)
                with pytest.raises(vam.VamError):
                    g.back(y)
                vam.debug_fail_allocations(0)
            if i == 2:
                g.back(y)
        s.synchronize()
    g.close()


@pytest.mark.parametrize("edge", [8, 12, 16])
def test_deposit_from_segments_not_cut_at_z_cells(edge):
    """Where there is no room for the deposit's segments cut at z cells, it takes
    whole runs of a box: the same operator against the oracle, with rays that
    climb little, much and not at all, in every storage type and over any
    angles; the forward keeps its bits."""
    n, na = 30, 8
    for what, kw in (("thin lens", {}), ("steep", {"projector": 0, "focus": 0.0, "pupil": 0.9, "step": 0.3}),
                     ("long steps", {"projector": 0, "focus": 0.0, "pupil": 0.7, "step": 1.3}),
                     ("along the lattice", {"projector": 0, "focus": 0.0, "pupil": 0.0})):
        p = dict(_p(n, n_angles=na), nz=27, **kw)
        og = oracle.Geometry(p)
        rng = synth.SplitMix64(59)
        x = torch.from_numpy(rng.uniform(27 * n * n).reshape(27, n, n).astype(np.float32)).to(DEV)
        y = torch.from_numpy((rng.uniform(na * n * n).reshape(na, n, n) - 0.3).astype(np.float32))
        g = vam.Geometry(p)
        g.set_box_edge(edge)
        P0, D0 = g.forward(x), g.back(y.to(DEV))
        uncut = 0
        for k in range(9, 40):             # the set-up's allocations after the forward's segments
            vam.debug_fail_allocations(k)
            try:
                g.set_box_edge(edge)
            except vam.VamError as e:
                assert e.status == vam.VAM_ERR_OUT_OF_MEMORY
                continue
            finally:
                vam.debug_fail_allocations(0)
            D = g.back(y.to(DEV))
            if torch.equal(D, D0):
                break                      # the rebuild makes fewer than k allocations
            uncut += 1
            say("%s, edge %d, allocation %d" % (what, edge, k))
            assert torch.equal(g.forward(x), P0)
            if uncut > 1:
                continue
            for dt in (torch.float32, torch.bfloat16, torch.float16):
                for a0, m in ((0, na), (3, 4)):
                    yy = y[a0:a0 + m].to(dt)
                    ref = oracle.adjoint(og, yy.double().numpy(), a0=a0, na=m)
                    got = g.back(yy.to(DEV), angle_begin=a0).cpu().numpy()
                    assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)
                    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()
        assert uncut >= 1 or what == "along the lattice", what
        g.close()
