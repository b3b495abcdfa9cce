"""The GA's generations in one launch (ga_run_kernel) against the oracle's
replay: whole trajectories (final populations, best individuals) bit for bit,
on both fitness tables (option rows under a fixed state; every feasible
configuration otherwise), with one and two pairs per thread, one and two words
of digits, every record layout, ragged populations and no feasible
configuration."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2609_02109_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_02109_amd import mf as mfmod
    return mfmod


CASES = [
    # options, hidden, scenarios, fixed, Eq. 3, GA settings
    ([12, 12, 9, 9, 9], (64, 32), 1, True, True, dict(pop=100, gens=12, p_mut=0.1)),
    ([7, 5, 6], (48, 40), 3, True, False, dict(pop=130, gens=5, tourn_k=1)),
    ([3, 4, 2, 5, 3, 2, 3, 2, 4], (32, 32), 2, True, True, dict(pop=64, gens=6, tourn_k=8, p_mut=0.4)),
    ([12, 12, 9], (32, 32), 2, True, False, dict(pop=4096, gens=3, p_cx=1.0)),
    ([5, 6, 4, 7], (32, 32), 2, True, False, dict(pop=4, gens=0)),
    ([5, 6, 4, 7], (32, 32), 5, False, False, dict(pop=200, gens=9, tourn_k=4, p_mut=0.2)),
    ([4, 3, 5, 3, 4, 2, 3], (64, 64), 3, False, True, dict(pop=2050, gens=4, p_cx=0.9)),
    ([2, 3, 2, 2, 3, 2, 2, 1, 3], (32, 32), 2, False, True, dict(pop=300, gens=5)),
    ([9, 8, 7], (32, 32), 2, False, False, dict(pop=4096, gens=2, tourn_k=2, p_mut=1.0)),
]


@pytest.mark.parametrize("opts,hid,S,fixed,eq3,kw", CASES, ids=[f"{'x'.join(map(str, c[0]))}-{'fixed' if c[3] else 'table'}-p{c[5]['pop']}" for c in CASES])
@pytest.mark.parametrize("cap", ["quantile", "none"])
def test_ga_run_trajectory(mf, orc, opts, hid, S, fixed, eq3, kw, cap):
    inst = synth.make_instance(opts, 8, 4, *hid, seed=6, vram_quantile=0.6, quantise=False)
    if cap == "none":   # no configuration meets the cap
        inst = replace(inst, vram_cap=0.5)
    ob = synth.make_objective(inst, 6, tau_range=(-0.4, 0.2)) if eq3 else None
    st = synth.make_state(inst, 6) if fixed else None
    sc = synth.ga_scenarios(inst.n_models, S, seed=6)
    print(f"[ga run] {opts} fixed={fixed} eq3={eq3} cap={cap} {kw}", flush=True)
    p = mf.Problem(inst, variants=ob)
    g = p.ga(sc.sla, sc.omega, seed=9, final_pop=True, objective=ob, state=st, **kw)
    if not fixed:   # the table: every VRAM-feasible configuration evaluated once
        assert g["forwards"] == p.search(inst.sla, inst.omega, state=synth.make_state(inst, 0))["n_vram"]
    r = orc.Problem(inst, ob, state=st).ga(sc.sla, sc.omega, seed=9, final_pop=True, **kw)
    p.close()
    np.testing.assert_array_equal(g["best_idx"], r["best_idx"])
    assert g["best_J"].tobytes() == r["best_J"].tobytes()
    np.testing.assert_array_equal(g["final_pop"].cpu().numpy().astype(np.uint64), r["final_pop"])


def test_ga_run_spans_of_draws(mf, orc):
    # more generations than one span of draws holds (64 MiB): the population
    # goes from launch to launch
    inst = synth.make_instance([6, 5, 7, 4], 8, 4, 32, 32, seed=3, vram_quantile=0.7)
    sc = synth.ga_scenarios(4, 40, seed=3)
    kw = dict(pop=3000, gens=25, p_mut=0.1, seed=2)
    g = mf.Problem(inst).ga(sc.sla, sc.omega, final_pop=True, **kw)
    r = orc.Problem(inst).ga(sc.sla, sc.omega, final_pop=True, **kw)
    np.testing.assert_array_equal(g["best_idx"], r["best_idx"])
    np.testing.assert_array_equal(g["final_pop"].cpu().numpy().astype(np.uint64), r["final_pop"])


# weights that are not finite: every fitness of a scenario NaN, or some of them,
# or infinite.  The elite is slot 0 when its fitness is NaN; the last case
# carries it from launch to launch
@pytest.mark.parametrize("fixed", [True, False])
@pytest.mark.parametrize("S,kw", [(6, dict(pop=200, gens=6)), (6, dict(pop=300, gens=4)), (40, dict(pop=3000, gens=25))])
def test_ga_run_not_finite_fitness(mf, orc, fixed, S, kw):
    inst = synth.make_instance([6, 5, 7, 4], 8, 4, 32, 32, seed=3, vram_quantile=0.7)
    sc = synth.ga_scenarios(4, S, seed=3)
    sla, om = np.full_like(sc.sla, np.inf), sc.omega.copy()
    om[0] = np.nan
    om[1, :2] = np.inf            # inf - inf where their throughputs differ in sign
    om[2, 0], om[2, 1] = np.inf, -np.inf
    om[3, 2] = -np.inf
    sla[4] = np.nan               # nothing feasible
    st = synth.make_state(inst, 3) if fixed else None
    print(f"[ga run] not finite fixed={fixed} {kw}", flush=True)
    p = mf.Problem(inst)
    g = p.ga(sla, om, seed=5, p_mut=0.1, final_pop=True, state=st, **kw)
    if not fixed:
        assert g["forwards"] == p.search(inst.sla, inst.omega, state=synth.make_state(inst, 0))["n_vram"]
    with np.errstate(invalid="ignore"):
        r = orc.Problem(inst, state=st).ga(sla, om, seed=5, p_mut=0.1, final_pop=True, **kw)
    pop = g["final_pop"].cpu().numpy().astype(np.uint64)
    assert (pop < inst.space_size).all()
    np.testing.assert_array_equal(pop, r["final_pop"])
    np.testing.assert_array_equal(g["best_idx"], r["best_idx"])
    assert g["best_J"].tobytes() == r["best_J"].tobytes()


# few generations of a small population over a space that they outnumber: a
# forward of every configuration by one lane each would take longer than the
# generations do, so every individual is evaluated
@pytest.mark.parametrize("K,hid,gens,table", [([2] * 8, (64, 64), 3, False), ([2] * 8, (64, 64), 60, True),
                                              ([3] * 5, (64, 32), 3, False), ([8, 8], (32, 32), 3, True)])
def test_ga_small_runs_without_the_table(mf, orc, K, hid, gens, table):
    inst = synth.make_instance(K, 8, 4, *hid, seed=8, vram_quantile=0.7)
    sc = synth.ga_scenarios(len(K), 4, seed=8)
    p = mf.Problem(inst)
    n_fl = p.search(inst.sla, inst.omega, state=synth.make_state(inst, 0))["n_vram"]
    g = p.ga(sc.sla, sc.omega, pop=72, gens=gens, seed=4, final_pop=True)
    r = orc.Problem(inst).ga(sc.sla, sc.omega, pop=72, gens=gens, seed=4, final_pop=True)
    assert g["forwards"] == (n_fl if table else 4 * 72 * (gens + 1))
    np.testing.assert_array_equal(g["best_idx"], r["best_idx"])
    assert g["best_J"].tobytes() == r["best_J"].tobytes()
    np.testing.assert_array_equal(g["final_pop"].cpu().numpy().astype(np.uint64), r["final_pop"])
