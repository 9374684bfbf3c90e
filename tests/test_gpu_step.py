"""Block steps through the step kernel (nbody_run, nbody_step) against the same
steps through the separate scheduler and corrector kernels, which the phase
timers select.

Both run the same force kernels; the corrector's arithmetic is the same source
compiled into two kernels, so states agree to rounding: after a few tens of
steps, relative 1e-12 on positions and velocities (a few hundred roundings of
1e-16 at most), times and levels exactly.
"""
import numpy as np
import pytest
import torch

import nbody_ics
from helpers import TICKS, say

pytestmark = pytest.mark.gpu


def _sim(model, order=4, precision="fp64", **kw):
    from paper_1312_1789_amd import Simulation
    kw.setdefault("eta", 0.01 if order == 4 else 0.1)
    kw.setdefault("eta_start", 0.1)
    sim = Simulation(model.m, model.x, model.v, order=order, precision=precision, eps2=1e-8, **kw)
    sim.init()
    return sim


def _compare(a, b):
    ha, hb = a.to_numpy(), b.to_numpy()
    np.testing.assert_array_equal(ha["t_tick"], hb["t_tick"])
    np.testing.assert_array_equal(ha["level"], hb["level"])
    for k in ("x", "v"):
        np.testing.assert_allclose(ha[k], hb[k], rtol=1e-12, atol=1e-13)


# one workgroup of 256 particles, its edges, a ragged last one; more than 256
# workgroups (four per thread of the last one) and more than 1024 (sixteen)
@pytest.mark.parametrize("n, order, precision", [
    (2, 4, "fp64"), (3, 6, "mixed"), (255, 4, "fp64"), (256, 8, "fp64"), (257, 6, "fp64"), (1025, 6, "mixed"),
    (5003, 4, "mixed"), (16641, 6, "ds"), (70001, 4, "fp64"), ((1 << 18) + 300, 4, "mixed")])
def test_run_equals_separate_kernels(n, order, precision):
    model = nbody_ics.plummer(n, 2100 + n % 97)
    a, b = _sim(model, order, precision), _sim(model, order, precision)
    b.set_timing(True)
    sizes = []
    for _ in range(12):
        ta, na = a.step()
        tb, nb = b.step()
        assert (ta, na) == (tb, nb)
        sizes.append(na)
    _compare(a, b)
    # a run of several steps, bounded by their number, then by time
    for sim in (a, b):
        assert sim.run(1 << 62, 20)[0] == 20
    _compare(a, b)
    end = (int(a.t_tick.max()) // (TICKS >> 7) + 1) * (TICKS >> 7)
    sa, sb = a.run(end, 200), b.run(end, 200)
    assert sa == sb
    _compare(a, b)
    fa, fb = a.stats(), b.stats()
    say("n=%d order %d %s: %d steps, first active sets %s" % (n, order, precision, fa.steps, sizes))
    assert (fa.steps, fa.sum_n_act, fa.interactions) == (fb.steps, fb.sum_n_act, fb.interactions)


def test_steps_equal_run():
    """The same steps one at a time and in one run, bit for bit: whether the
    next step was enqueued ahead changes nothing."""
    model = nbody_ics.plummer(3000, 2201)
    a, b = _sim(model, 6, "mixed"), _sim(model, 6, "mixed")
    for _ in range(60):
        a.step()
    assert b.run(1 << 62, 60)[0] == 60
    ha, hb = a.to_numpy(), b.to_numpy()
    for k in ("x", "v", "t_tick", "level"):
        np.testing.assert_array_equal(ha[k], hb[k])


def test_synchronised_blocks_are_listed():
    """Active sets larger than the last workgroup lists itself (4096): every
    particle on one level, then half of them a level up."""
    model = nbody_ics.plummer(9001, 2301)
    a, b = _sim(model, 4, "mixed"), _sim(model, 4, "mixed")
    b.set_timing(True)
    lv = torch.full((model.n,), 10, dtype=torch.int32, device=a.device)
    lv[::2] = 9
    for sim in (a, b):
        sim.level.copy_(lv)
    assert a.step() == b.step() == (TICKS >> 10, model.n // 2)
    assert a.step() == b.step()
    _compare(a, b)


# the first candidates of a block come with its time (two, or one when a thread
# has sixteen blocks), those beyond are searched for
@pytest.mark.parametrize("n", [900, 70001, (1 << 18) + 300])
@pytest.mark.parametrize("most", [1, 2, 3, 9])
def test_active_sets_by_block(n, most):
    """Up to `most` due particles in each of a few blocks, the last one among
    them."""
    model = nbody_ics.plummer(n, 2350 + most)
    a, b = _sim(model), _sim(model)
    b.set_timing(True)
    lv = torch.full((n,), 5, dtype=torch.int32)
    due = 0
    for k, base in enumerate([0, 256, 768 if n > 1024 else 512, (n - 1) // 256 * 256]):
        cnt = min(most if k % 2 == 0 else 1, n - base)
        lv[base:base + 3 * cnt:3] = 14
        due = int((lv == 14).sum())
    for sim in (a, b):
        sim.level.copy_(lv.to(sim.device))
    assert a.step() == b.step() == (TICKS >> 14, due)
    for _ in range(3):
        assert a.step() == b.step()
    _compare(a, b)


# the blocks of the last workgroup's four waves: 64 to a wave with one block per
# thread (n <= 65536), 192 with three; 196608 is the largest system of the step kernel
@pytest.mark.parametrize("n, per_wave", [(20000, 64), (60000, 64), (130000, 192), (196608, 192), (196609, 192)])
@pytest.mark.parametrize("where", ["last", "middle", "apart"])
@pytest.mark.parametrize("due", [3, 9, 70])
def test_active_sets_in_late_waves(n, per_wave, where, due):
    """Due particles only in blocks that whole waves without any precede, with
    more of them to a block than come with its time; every other block has all
    its particles at one later time."""
    model = nbody_ics.plummer(n, 2360)
    a, b = _sim(model), _sim(model)
    b.set_timing(True)
    wave = 256 * per_wave
    waves = (n + wave - 1) // wave
    bases = {"last": [(n - 1) // 256 * 256], "middle": [waves // 2 * wave + 256],
             "apart": [0, 2 * wave + 768] if waves > 2 else [512, wave + 768]}[where]
    lv = torch.full((n,), 5, dtype=torch.int32)
    for base in bases:
        lv[base:min(base + due, n)] = 14
    total = int((lv == 14).sum())
    for sim in (a, b):
        sim.level.copy_(lv.to(sim.device))
    assert a.step() == b.step() == (TICKS >> 14, total)
    for _ in range(3):
        assert a.step() == b.step()
    _compare(a, b)


@pytest.mark.parametrize("n_hard", [2, 255, 257])
def test_post_newtonian_steps(n_hard):
    """Post-Newtonian terms added by the step kernel (up to 256 hard
    particles) and by their own kernel (more)."""
    model = nbody_ics.plummer(1200, 2401)
    kw = dict(n_hard=n_hard, c_light=50.0, pn_terms=7)
    a, b = _sim(model, 6, "fp64", **kw), _sim(model, 6, "fp64", **kw)
    b.set_timing(True)
    assert a.run(1 << 62, 25)[0] == b.run(1 << 62, 25)[0] == 25
    _compare(a, b)


def test_run_stops_at_a_nonfinite_value():
    """A NaN stops the run with the steps enqueued ahead left undone; the
    context goes on working once the state is mended."""
    from paper_1312_1789_amd import abi
    model = nbody_ics.plummer(1500, 2501)
    sim = _sim(model, 6, "fp64")
    good = [t.clone() for t in (sim.x, sim.v, *sim.d, sim.t_tick, sim.level)]
    sim.x[0, 7] = float("nan")
    with pytest.raises(abi.NBodyError) as e:
        sim.run(1 << 62, 1000)
    assert e.value.status == abi.NBODY_E_NONFINITE
    assert sim.stats().steps <= 2
    for to, of in zip((sim.x, sim.v, *sim.d, sim.t_tick, sim.level), good):
        to.copy_(of)
    assert sim.run(1 << 62, 10)[0] == 10
    assert torch.isfinite(sim.x).all()


@pytest.mark.parametrize("call", ["run", "step"])
@pytest.mark.parametrize("due", [1, 700])
def test_no_step_after_a_nonfinite_correction(call, due):
    """A non-finite value from the program's own corrector call ends the next
    run or step before it: the call reports it and leaves the state alone
    (due = 1: the first step would be one enqueued before its schedule is
    read).  The call after that goes on."""
    from paper_1312_1789_amd import abi
    model = nbody_ics.plummer(1500, 2601)
    sim = _sim(model, 6, "fp64")
    lv = torch.full((model.n,), 10, dtype=torch.int32)
    lv[:due] = 14
    sim.level.copy_(lv.to(sim.device))
    good = [t.clone() for t in (sim.x, sim.v, *sim.d, sim.t_tick, sim.level)]
    act = torch.tensor([model.n - 1], dtype=torch.int32, device=sim.device)
    f = {k: torch.full((3, 1), float("nan"), dtype=torch.float64, device=sim.device)
         for k in ("acc", "jrk", "snp", "crk")}
    sim.correct(act, TICKS >> 10, f)
    for to, of in zip((sim.x, sim.v, *sim.d, sim.t_tick, sim.level), good):
        to.copy_(of)
    with pytest.raises(abi.NBodyError) as e:
        sim.run(1 << 62, 5) if call == "run" else sim.step()
    assert e.value.status == abi.NBODY_E_NONFINITE
    for now, was in zip((sim.x, sim.v, *sim.d, sim.t_tick, sim.level), good):
        assert torch.equal(now, was)
    assert sim.stats().steps == 0
    assert sim.step() == (TICKS >> 14, due)
    assert sim.run(1 << 62, 5)[0] == 5
    assert torch.isfinite(sim.x).all()
