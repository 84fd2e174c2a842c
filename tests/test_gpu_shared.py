"""GPU: steps with shared halos (every face formed once, by the patch that owns
it, and read from there) against the halo scheme (every patch forms what its
ghosts hold), which `wmb_keep_stages` selects: the same arithmetic on the same
values, so states, counters, stages and ghosts are bitwise equal."""
import numpy as np
import pytest

from paper_1701_07452_amd import inputs as I
from tests.test_gpu_parity import as_f32, gpu_sim, wmb  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

# patch extents, patches along each axis, ghost width, parameters, tuning
PLAIN = {}
SHARED = {
    "one_patch": ((9, 7, 12), (1, 1, 1), 4, PLAIN, None),               # its own neighbour on every side
    "smallest": ((4, 4, 4), (3, 2, 2), 4, PLAIN, None),                 # a halo reaches past half the neighbour
    "odd": ((33, 5, 9), (2, 3, 1), 5, dict(limiter_beta=1.5), None),    # rows that are no whole lines, thin in y
    "whole_lines": ((32, 16, 8), (1, 2, 3), 4, PLAIN, None),
    "separate": ((16, 12, 10), (2, 1, 2), 4, PLAIN, {(6, 0, 0): 0}),    # the corrector as three sweeps
    "fused": ((16, 12, 10), (2, 1, 2), 4, PLAIN, {(6, 0, 0): 4}),
    "marching": ((8, 40, 24), (2, 1, 1), 4, PLAIN, "march"),
    "protected": ((12, 10, 16), (2, 2, 1), 4, dict(rho_protect=0.6, p_protect=0.9), None),
    "protected_march": ((6, 20, 20), (2, 1, 2), 4, dict(rho_protect=0.6, p_protect=0.9, limiter_beta=2.0), "march"),
}


def _setup(case, prec):
    n, nb, g, kw, tun = SHARED[case]
    G = I.uniform_grid(tuple(a * b for a, b in zip(n, nb)), n)
    N = G.shape
    dx = (1.0 / max(N),) * 3
    q, b = I.random_smooth(N, 31, dx=dx, amp=0.4)
    if prec == 1:
        q, b = as_f32(q), as_f32(b)
    if tun == "march":
        tun = {(st, ax, n[ax]): -64 for st in (1, 2) for ax in (1, 2)}
    return G, q, b, dict(kw, ghost=g, dx=dx), tun


def _sim(W, case, prec, shared, tun="case"):
    G, q, b, kw, t = _setup(case, prec)
    sim = gpu_sim(W, G, q, b, prec, **kw)
    if not shared:
        sim.keep_stages(True)
    if t:
        sim.set_tuning(t)
    return G, sim


def _state(G, sim):
    return I.gather(G, [sim.get_state(i) for i in range(G.npatch)])


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("case", sorted(SHARED))
def test_shared_equals_halo(wmb, case, prec):
    """Five graph-replayed steps, with eager steps and reads between them."""
    out = []
    for shared in (True, False):
        G, sim = _sim(wmb, case, prec, shared)
        sim.run_steps(2)
        tot = sim.diagnostics()
        sim.fill_ghosts()
        dt = sim.compute_dt()
        sim.advance(0.0)
        sim.run_steps(2)
        out.append((_state(G, sim), tot, dt, sim.protected_faces(), sim.diagnostics()))
        sim.close()
    for a, c in zip(out[0][0], out[1][0]):
        assert np.array_equal(a, c), float(np.abs(a - c).max())
    assert out[0][2] == out[1][2] and out[0][3] == out[1][3]
    if "protected" in case:
        assert out[0][3] > 0
    for k in (1, 4):  # totals, max div b (normalised, raw), floor activations
        assert np.array_equal(out[0][k][0], out[1][k][0]) and out[0][k][1:] == out[1][k][1:]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("case", ["odd", "separate", "fused"])
def test_stages_and_ghosts_after_shared_steps(wmb, case, prec):
    """wmb_debug_stage after a shared step (with a new dt formed since) gives
    the halo scheme's stages on the ranges a step needs, and wmb_get_stored
    the x-ghosts of interior rows that its update writes."""
    out = []
    for shared in (True, False):
        G, sim = _sim(wmb, case, prec, shared)
        g = int(sim.params.ghost)
        sim.run_steps(3)
        sim.compute_dt()
        got = []
        for ip in range(G.npatch):
            n = G.descs[ip][0]
            rows = (slice(None), slice(g, g + n[2]), slice(g, g + n[1]))
            qs, bs = sim.get_stored(ip)
            got += [qs[rows], bs[rows]]
            box = tuple(slice(g, g + n[2 - a]) for a in range(3))
            for st, lo, hi, tlo, thi in ((1, -2, 2, -3, 2), (5, -1, 1, -1, 0)):
                f = sim.debug_stage(ip, st)
                for d in range(3):
                    sl = tuple(slice(g + (lo if a == d else tlo), g + n[a] + (hi if a == d else thi) + 1) for a in (2, 1, 0))
                    got.append(f[d][(slice(None),) + sl])
            got.append(sim.debug_stage(ip, 3)[(slice(None),) + box])
        sim.run_steps(1)  # the stages formed again leave the next step as it was
        got += list(_state(G, sim))
        out.append(got)
        sim.close()
    for i, (a, c) in enumerate(zip(*out)):
        assert np.array_equal(a, c), (i, float(np.abs(a - c).max()))


@pytest.mark.parametrize("prec", [0, 1])
def test_shared_and_frozen_in_turn(wmb, prec):
    """Steps before a freeze (shared), with a patch frozen and with a slot
    removed (halo scheme), and after both are back (shared again), with a
    retune while frozen."""
    out = []
    for shared in (True, False):
        G, sim = _sim(wmb, "fused", prec, shared)
        sim.run_steps(1)
        sim.set_active(1, False)
        sim.run_steps(2)
        sim.set_tuning({(6, 0, 0): 3, (1, 0, 16): 2})
        sim.set_active(1, True)
        sim.run_steps(2)
        sim.set_present(2, False)
        sim.run_steps(1)
        sim.set_present(2, True)
        sim.run_steps(2)
        out.append(_state(G, sim))
        sim.close()
    for a, c in zip(*out):
        assert np.array_equal(a, c), float(np.abs(a - c).max())


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("how", ["tuning", "schedule"])
def test_lists_rebuilt_while_frozen(wmb, how, prec):
    """Work lists rebuilt between a freeze and the next step (a retune, or
    another schedule and back): the shared steps after the thaw leave out no
    patch."""
    out = []
    for shared in (True, False):
        G, sim = _sim(wmb, "fused", prec, shared)
        sim.run_steps(1)
        sim.set_active(1, False)
        if how == "tuning":
            sim.set_tuning({(6, 0, 0): 3, (1, 0, 16): 2, (1, 1, 12): 4, (2, 2, 10): 4, (3, 0, 0): 13})
        else:
            sim.set_schedule(2)
            sim.set_schedule(1)
        sim.set_active(1, True)
        sim.run_steps(3)
        out.append(_state(G, sim))
        sim.close()
    for a, c in zip(*out):
        assert np.array_equal(a, c), float(np.abs(a - c).max())


def test_fp64_halo_scheme_takes_separate_correctors(wmb):
    """In FP64 the fused x/y corrector serves the shared-halo steps alone (in
    the halo scheme the three sweeps are faster): a profiled shared step has no
    y corrector, one with a frozen patch has it beside those along x and z,
    which each take as long within a factor of four."""
    n, nb = (24, 24, 24), (3, 3, 3)
    G = I.uniform_grid(tuple(a * b for a, b in zip(n, nb)), n)
    q, b = I.random_smooth(G.shape, 5, dx=(1 / 72,) * 3)
    sim = gpu_sim(wmb, G, q, b, 0, dx=(1 / 72,) * 3)
    y = []
    for frozen in (False, True):
        sim.set_active(0, not frozen)
        sim.run_steps(1)
        ms = [sim.profile_step() for _ in range(3)]
        y.append([min(m[k] for m in ms) for k in ("sweep2_x", "sweep2_y", "sweep2_z")])
    sim.close()
    assert y[0][1] < 0.25 * y[0][0]
    assert 0.25 < y[1][1] / y[1][0] < 4 and 0.25 < y[1][1] / y[1][2] < 4


def test_band_rows_set_are_the_ones_that_run(wmb):
    """Every entry (6, 0, 0, r) takes effect in shared steps, whichever rows
    the halo scheme has, and a schedule set and taken back while a patch is
    frozen keeps them.  (wmb_autotune of a shared FP64 batch reports the
    shapes that run and times nothing.)"""
    for r in range(8):
        G, sim = _sim(wmb, "smallest", 0, True)
        sim.set_tuning({(6, 0, 0): r})
        assert sim.autotune()[(6, 0, 0)] == r
        sim.close()
    G, sim = _sim(wmb, "smallest", 0, True)
    before = sim.autotune()
    sim.set_active(1, False)
    sim.set_schedule(2)
    sim.run_steps(1)
    sim.set_schedule(1)
    sim.set_active(1, True)
    sim.run_steps(1)
    assert sim.autotune() == before
    sim.close()


def test_autotune_keeps_the_other_scheme(wmb):
    """Shapes timed for shared-halo steps (FP32) are not forced on the halo
    scheme, which wmb_autotune does not time (the tiles of Steps 3-4 and 8-11
    are common to both)."""
    G, sim = _sim(wmb, "whole_lines", 1, True)
    own = lambda t: {k: v for k, v in t.items() if k[0] in (1, 2, 6)}  # noqa: E731
    sim.keep_stages(True)
    halo = own(sim.autotune())
    sim.keep_stages(False)
    timed = own(sim.autotune(-1))
    sim.keep_stages(True)
    assert own(sim.autotune()) == halo and own(sim.autotune(-1)) == halo
    sim.keep_stages(False)
    assert own(sim.autotune()) == timed  # remembered for shared steps
    sim.close()


def test_stages_after_autotune(wmb):
    """wmb_autotune leaves the intermediates of the steps it timed, which start
    from the current state: its stages are those of the next step (FP32, whose
    shared shapes are timed; one repetition)."""
    G, sim = _sim(wmb, "whole_lines", 1, True)
    g = int(sim.params.ghost)
    sim.run_steps(2)
    sim.autotune(-1)
    got = []
    for _ in range(2):
        stages = []
        for ip in range(G.npatch):
            n = G.descs[ip][0]
            own = (slice(None),) + tuple(slice(g, g + n[a]) for a in (2, 1, 0))
            stages += [sim.debug_stage(ip, 3)[own], sim.debug_stage(ip, 1)[1][own], sim.debug_stage(ip, 5)[2][own]]
        got.append(stages)
        sim.run_steps(1)
    for a, c in zip(*got):
        assert np.isfinite(a).all() and np.array_equal(a, c), float(np.abs(a - c).max())
    sim.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("between", ["nothing", "retune", "schedule", "more"])
def test_stages_after_freeze(wmb, between, prec):
    """The stages of a shared step asked for after one patch was frozen and
    another slot removed, with the work lists rebuilt in between or not, and
    the steps after."""
    out = []
    for shared in (True, False):
        G, sim = _sim(wmb, "fused", prec, shared)
        g = int(sim.params.ghost)
        sim.run_steps(3)
        q, b = sim.get_state(1)
        sim.set_active(1, False)
        sim.set_state(1, q, b)  # copies the frozen patch again
        sim.set_present(2, False)
        if between == "retune":
            sim.set_tuning({(1, 0, 16): 2, (2, 2, 10): 4})
        elif between == "schedule":
            sim.set_schedule(2)
            sim.set_schedule(1)
        elif between == "more":
            sim.set_active(3, False)
            sim.set_active(3, True)
        got = []
        for ip in range(G.npatch):
            n = G.descs[ip][0]
            box = (slice(None),) + tuple(slice(g, g + n[2 - a]) for a in range(3))
            for st, lo, hi, tlo, thi in ((1, -2, 2, -3, 2), (5, -1, 1, -1, 0)):
                f = sim.debug_stage(ip, st)
                for d in range(3):
                    sl = tuple(slice(g + (lo if a == d else tlo), g + n[a] + (hi if a == d else thi) + 1) for a in (2, 1, 0))
                    got.append(f[d][(slice(None),) + sl])
            got.append(sim.debug_stage(ip, 3)[box])
        sim.run_steps(2)
        got += [a for ip in (0, 1, 3) for a in sim.get_state(ip)]
        sim.set_present(2, True)
        sim.set_active(1, True)
        sim.run_steps(2)
        got += list(_state(G, sim))
        out.append(got)
        sim.close()
    for i, (a, c) in enumerate(zip(*out)):
        assert np.array_equal(a, c), (i, float(np.abs(a - c).max()))


# what a shared step can be combined with: the Steps 8-11 launch from queues, a
# dt one step late, other schedules and back, steps launched kernel by kernel
# (from 2^21 zones on), timed shapes (FP32)
OPTIONS = {
    "queue": ((16, 12, 10), (2, 1, 2), {}, {(5, 0, 0): 1}),
    "dt_lag": ((16, 12, 10), (2, 1, 2), dict(dt_lag=1), None),
    "schedules": ((8, 8, 8), (2, 2, 3), {}, None),
    "launched": ((64, 64, 64), (2, 2, 2), {}, None),
    "tuned": ((24, 20, 16), (2, 2, 2), {}, None),
}


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("option", sorted(OPTIONS))
def test_shared_options(wmb, option, prec):
    """Six steps, bitwise those of the halo scheme."""
    n, nb, kw, tun = OPTIONS[option]
    G = I.uniform_grid(tuple(a * b for a, b in zip(n, nb)), n)
    dx = (1.0 / max(G.shape),) * 3
    q, b = I.random_smooth(G.shape, 8, dx=dx, amp=0.4)
    if prec == 1:
        q, b = as_f32(q), as_f32(b)
    out = []
    for shared in (True, False):
        sim = gpu_sim(wmb, G, q, b, prec, dx=dx, **kw)
        if not shared:
            sim.keep_stages(True)
        if tun:
            sim.set_tuning(tun)
        if option == "tuned" and shared:
            sim.autotune(-1)
        for groups in (1, 3, 1, 2, 4, 1):
            if option == "schedules":
                sim.set_schedule(groups)
            sim.run_steps(1)
        out.append((_state(G, sim), sim.diagnostics()))
        sim.close()
    for a, c in zip(out[0][0], out[1][0]):
        assert np.array_equal(a, c), float(np.abs(a - c).max())
    assert np.array_equal(out[0][1][0], out[1][1][0]) and out[0][1][1:] == out[1][1][1:]
