"""Parity of the HIP path (through the C ABI) with the FP64 oracle.

Integer and index work (Poisson rasters, spike compaction, CSR indexing with
integer weights) must match bit for bit; membrane voltages within 1e-3 mV
RMS over the first 1000 steps; spike counts per neuron are reported.
"""
import math

import numpy as np
import pytest

from oracle import oracle as O
from paper_1412_0595_amd import netgen

pytestmark = pytest.mark.gpu

FIX = 2.0 ** 40


@pytest.fixture(scope="module")
def snn():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1412_0595_amd import snn as S
    S.load()
    return S


def say(*a):
    print(*a, flush=True)


def test_poisson_raster_bitwise(snn):
    say("case: poisson raster, 4 populations, 300 steps")
    inst = dict(g_scale=1.0, seed=(7 << 33) + 5,
                pops=[dict(name="A", kind="poisson", n=1000, rate_hz=300.0, i_ext=0.0),
                      dict(name="B", kind="poisson", n=70, rate_hz=5000.0, i_ext=0.0),
                      dict(name="C", kind="poisson", n=3, rate_hz=20000.0, i_ext=0.0),
                      dict(name="D", kind="poisson", n=1000, rate_hz=300.0, i_ext=0.0)], projs=[])
    spec = dict(dt=0.1, substeps=3, instances=[inst])
    T = 300
    net = snn.Network(spec, raster_steps=T)
    net.step(T)
    orc = O.OracleNet(inst, log_events=True)
    orc.step(T)
    t, p, i = orc.events()
    for pop in range(4):
        ras = net.raster(0, pop, 0, T)
        for k in range(T):
            expect = np.sort(i[(t == k) & (p == pop)])
            assert np.array_equal(ras[k], expect), (pop, k)
        assert np.array_equal(net.spikes(0, pop), orc.counts(pop))
    # two populations of one instance at the same rate draw different streams
    assert not np.array_equal(net.spikes(0, 0), net.spikes(0, 3))
    net.close()


@pytest.mark.parametrize("mode", [0, 3])
@pytest.mark.parametrize("seed", range(6))
def test_propagation_bitwise_integer_weights(snn, seed, mode):
    """G after one step equals the rounded dense product d * (W^T s) on the
    2^-40 uS grid, bit for bit (integer g makes every order exact); by rows
    and in row groups (every projection here is delivered in groups)."""
    say(f"case: propagation seed {seed}, mode {mode}")
    spec = netgen.random_tiny(seed, integer_g=True, max_n=200, p=0.4)
    inst = spec["instances"][0]
    rng = np.random.default_rng(100 + seed)
    flags = {p: (rng.random(pp["n"]) < (1.0 if seed == 1 else 0.3)).astype(np.uint8)
             for p, pp in enumerate(inst["pops"])}
    if seed == 4:
        flags = {p: np.zeros_like(f) for p, f in flags.items()}
    net = snn.Network(spec)
    net.set_launch(mode=mode)
    orc = O.OracleNet(inst)
    for p, f in flags.items():
        net.set_last_spikes(0, p, f)
        orc.set_last_spikes(p, f)
        assert np.array_equal(net.last_spikes(0, p), f)
    net.step(1)
    orc.step(1)
    for q in range(len(inst["projs"])):
        g_gpu = net.conductance(0, q) * FIX
        g_orc = np.rint(orc.G(q) * FIX)
        assert np.array_equal(g_gpu, g_orc), q
    net.close()


@pytest.mark.parametrize("frac", [0.0005, 0.02, 0.3, 1.0])
def test_grouped_delivery_bitwise(snn, frac):
    """Grouped mode with a pre population of 5000 neurons (79 spike words, two
    rounds of the word scan, so groups straddle rounds): projections onto
    1000 and 64 neurons are delivered in row groups, one onto 3000 stays with
    rows; G after one step equals the oracle's bit for bit, at sparse and
    dense activity, in several launch shapes (one block taking every group
    slot in turn, one wavefront per block, eight, the row items split off)."""
    say(f"case: grouped delivery, 5000 pre neurons, {frac:.2%} spiking")
    rng = np.random.default_rng(37)
    n_pre, sizes = 5000, (1000, 3000, 64)
    pops = [dict(name="A", kind="poisson", n=n_pre, rate_hz=0.0, i_ext=0.0)] + \
        [dict(name=f"P{k}", kind="hh", n=m, rate_hz=0.0, i_ext=0.0) for k, m in enumerate(sizes)]
    projs = []
    for k, m in enumerate(sizes):
        mask = rng.random((n_pre, m)) < (0.05 if m > 64 else 0.3)
        rp = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int32)
        ci = np.nonzero(mask)[1].astype(np.int32)
        g = rng.integers(0, 4, ci.size).astype(np.float32)
        projs.append(dict(pre=0, post=k + 1, row_ptr=rp, col_idx=ci, g=g, e_rev=0.0, tau=1.0, stdp=None))
    inst = dict(g_scale=1.0, seed=5, pops=pops, projs=projs)
    spec = dict(dt=0.1, substeps=3, instances=[inst])
    f = (rng.random(n_pre) < frac).astype(np.uint8)
    f[4999] = 1   # the last neuron of the last word
    orc = O.OracleNet(inst)
    orc.set_last_spikes(0, f)
    orc.step(1)
    ref = [np.rint(orc.G(q) * FIX) for q in range(len(projs))]
    for shape in (dict(), dict(prop_blocks=1), dict(prop_block=64, prop_blocks=7), dict(prop_block=512),
                  dict(prop_blocks=8192)):
        net = snn.Network(spec)
        net.set_launch(mode=3, **shape)
        net.set_last_spikes(0, 0, f)
        net.step(1)
        for q in range(len(projs)):
            assert np.array_equal(net.conductance(0, q) * FIX, ref[q]), (shape, q)
        net.close()


def _upstroke_state(n, spiking):
    """V just below 0 with open sodium channels crosses 0 within one step;
    everyone else rests."""
    V0, m0, h0, n0 = O.rest()
    V = np.full(n, V0)
    m = np.full(n, m0)
    h = np.full(n, h0)
    nn = np.full(n, n0)
    V[spiking] = -1.0
    m[spiking] = 0.95
    h[spiking] = 0.6
    nn[spiking] = 0.3
    return V, m, h, nn


@pytest.mark.parametrize("pattern", ["none", "all", "w63", "w64", "w65", "sparse", "last"])
def test_spike_compaction_bitwise(snn, pattern):
    say(f"case: compaction {pattern}")
    n = 200
    idx = {"none": [], "all": list(range(n)), "w63": list(range(63)), "w64": list(range(64, 128)),
           "w65": list(range(128, 193)), "sparse": [0, 63, 64, 127, 150, 199], "last": [199]}[pattern]
    # each spiking neuron projects one synapse onto a counter population so
    # the compacted work items are checked too
    rp = np.arange(n + 1, dtype=np.int32)
    ci = np.arange(n, dtype=np.int32) % 7
    inst = dict(g_scale=1.0, seed=3,
                pops=[dict(name="X", kind="hh", n=n, rate_hz=0.0, i_ext=0.0),
                      dict(name="Y", kind="hh", n=7, rate_hz=0.0, i_ext=0.0)],
                projs=[dict(pre=0, post=1, row_ptr=rp, col_idx=ci, g=np.ones(n, np.float32), e_rev=0.0,
                            tau=5.0, stdp=None)])
    spec = dict(dt=0.1, substeps=3, instances=[inst])
    state = _upstroke_state(n, idx)
    net = snn.Network(spec)
    orc = O.OracleNet(inst)
    for var in range(4):
        net.set_state(0, 0, var, state[var])
        orc.set(0, var, state[var])
    v_prev = net.state(0, 0, snn.V)
    net.step(1)
    orc.step(1)
    v_new = net.state(0, 0, snn.V)
    got = net.last_spikes(0, 0)
    assert np.array_equal(got, ((v_prev < 0) & (v_new >= 0)).astype(np.uint8))
    assert np.array_equal(got, orc.last_spikes(0))
    assert sorted(np.nonzero(got)[0].tolist()) == sorted(idx)
    net.step(1)
    orc.step(1)
    assert np.array_equal(np.rint(net.conductance(0, 0) * FIX), np.rint(orc.G(0) * FIX))
    net.close()


def test_compaction_exact_zero_and_non_finite(snn):
    """Threshold edge cases of the crossing test V(t-1) < 0 <= V(t): a voltage
    landing exactly on 0.0 spikes; one starting at 0.0 or -0.0 does not; a
    NaN or infinite voltage entering the step never spikes and is not counted
    again as a NaN; neighbours at the 64-lane wave boundaries are unaffected.
    The population is a leak-only membrane (g_Na = g_K = 0, g_L = 1 uS,
    E_L = -64 mV, C = 1 nF) with one Euler substep of 0.125 ms and
    I_ext = 64 + 7x nA, x = 2^-10: every operation of the step is then exact,
    and V' = (7V + 7x)/8, so V = -x lands on 0.0 exactly in any evaluation
    order."""
    say("case: compaction edge cases (exact 0.0, -0.0, NaN, +-inf)")
    x = 2.0 ** -10
    n = 200
    V = np.full(n, -2 * x)
    lands = [0, 63, 64, 127, 128, 199]
    V[lands] = -x
    V[[1, 62]] = 0.0
    V[[2, 65]] = -0.0
    V[[3, 66, 129]] = np.nan
    V[[4, 130]] = np.inf
    V[[5, 131]] = -np.inf
    hh = np.array([0.0, 50.0, 0.0, -95.0, 1.0, -64.0, 1.0])
    rp = np.arange(n + 1, dtype=np.int32)
    ci = np.arange(n, dtype=np.int32) % 7
    inst = dict(g_scale=1.0, seed=3,
                pops=[dict(name="X", kind="hh", n=n, rate_hz=0.0, i_ext=64.0 + 7 * x),
                      dict(name="Y", kind="hh", n=7, rate_hz=0.0, i_ext=0.0)],
                projs=[dict(pre=0, post=1, row_ptr=rp, col_idx=ci, g=np.ones(n, np.float32), e_rev=0.0,
                            tau=5.0, stdp=None)])
    spec = dict(dt=0.125, substeps=1, instances=[inst])
    net = snn.Network(spec, hh_params={0: hh})
    orc = O.OracleNet(inst, dt=0.125, substeps=1, hh_params={0: hh})
    net.set_state(0, 0, snn.V, V)
    orc.set(0, O.V, V)
    net.step(1)
    orc.step(1)
    v_new = net.state(0, 0, snn.V)
    assert np.array_equal(v_new[lands], np.zeros(len(lands)))
    assert np.array_equal(orc.get(0, O.V)[lands], np.zeros(len(lands)))
    got = net.last_spikes(0, 0)
    expect = np.zeros(n, np.uint8)
    expect[lands] = 1
    assert np.array_equal(got, expect)
    assert np.array_equal(orc.last_spikes(0), expect)
    assert net.nan_counts()[0] == 0 and orc.nan_count == 0
    net.step(1)
    orc.step(1)
    assert np.array_equal(np.rint(net.conductance(0, 0) * FIX), np.rint(orc.G(0) * FIX))
    assert np.array_equal(net.spikes(0, 0), orc.counts(0))
    net.close()


def test_nan_count_edge_is_the_single_precision_range(snn):
    """The NaN count of Fig. 1 counts a neuron once, at the step its V leaves
    the fp32 state's range: a leak-only neuron whose V lands exactly on
    FLT_MAX + half an ulp (which rounds to infinity) counts, one landing on the
    double just below it does not (the same instance as the oracle's pin of
    this edge).  Only the first step is compared: the stored pair of the value
    just below the edge (hi = FLT_MAX, lo = fl32(rest)) reads back as the edge
    itself, so from there on the two sides may count that neuron differently;
    nothing in the range a network reaches before it overflows is affected."""
    say("case: NaN count at the single-precision range edge")
    from test_oracle_kinetics import nan_edge_instance
    inst, hp, edge, below = nan_edge_instance(O)
    spec = dict(dt=0.125, substeps=1, instances=[inst])
    net = snn.Network(spec, hh_params=hp)
    orc = O.OracleNet(inst, dt=0.125, substeps=1, hh_params=hp)
    for p in (0, 1):
        net.set_state(0, p, snn.V, [-64.0])
        orc.set(p, O.V, [-64.0])
    net.step(1)
    orc.step(1)
    assert orc.nan_count == 1
    assert net.nan_counts()[0] == 1
    assert not np.isfinite(net.state(0, 0, snn.V)[0])
    # the neuron that overflowed is not counted again
    net.step(1)
    assert net.nan_counts()[0] >= 1 and not np.isfinite(net.state(0, 0, snn.V)[0])
    net.close()


def test_one_step_update_from_same_state(snn):
    """From an identical random state (including mid-spike and hyperpolarised
    neurons and nonzero conductances) one step agrees to far below fp32."""
    say("case: one-step update")
    rng = np.random.default_rng(11)
    spec = netgen.make_config(1, scale=0.3)
    inst = spec["instances"][0]
    net = snn.Network(spec)
    orc = O.OracleNet(inst)
    for p in (1, 2):
        n = inst["pops"][p]["n"]
        vals = [rng.uniform(-85, 40, n), rng.uniform(0, 1, n), rng.uniform(0, 1, n), rng.uniform(0, 1, n)]
        vals[0][:4] = [-52.0, -25.0, -50.0, 0.0]    # removable singularities of the rates
        for var in range(4):
            net.set_state(0, p, var, vals[var])
            orc.set(p, var, net.state(0, p, var))   # the stored pair, exactly
    for q, pr in enumerate(inst["projs"]):
        g = rng.uniform(0, 0.02, inst["pops"][pr["post"]]["n"])
        net.set_conductance(0, q, g)
        orc.set_G(q, net.conductance(0, q))
    net.step(1)
    orc.step(1)
    for p in (1, 2):
        for var in range(4):
            a, b = net.state(0, p, var), orc.get(p, var)
            assert np.max(np.abs(a - b)) < 1e-9, (p, var, np.max(np.abs(a - b)))
        assert np.array_equal(net.last_spikes(0, p), orc.last_spikes(p))
    for q in range(3):
        assert np.max(np.abs(net.conductance(0, q) - orc.G(q))) < 2e-12
    net.close()


def _parity_run(snn, spec, T, chunk=50, pops=(1, 2)):
    inst = spec["instances"][0]
    net = snn.Network(spec)
    orc = O.OracleNet(inst)
    se = 0.0
    cnt = 0
    for _ in range(T // chunk):
        net.step(chunk)
        for _k in range(chunk):
            orc.step(1)
        for p in pops:
            d = net.state(0, p, snn.V) - orc.get(p, O.V)
            se += float(np.sum(d * d))
            cnt += d.size
    return net, orc, math.sqrt(se / cnt)


def test_network_parity_workload1(snn):
    """Workload 1 (A=100 Poisson, B=1000, C=100 HH): V RMS over all HH
    neurons, sampled every step of the first 1000, within 1e-3 mV; then spike
    counts per neuron over the full 10000 steps."""
    say("case: workload 1, 1000-step V trace")
    spec = netgen.make_config(1)
    inst = spec["instances"][0]
    net = snn.Network(spec)
    orc = O.OracleNet(inst)
    se, cnt = 0.0, 0
    for t in range(1000):
        net.step(1)
        orc.step(1)
        for p in (1, 2):
            d = net.state(0, p, snn.V) - orc.get(p, O.V)
            se += float(np.sum(d * d))
            cnt += d.size
    rms = math.sqrt(se / cnt)
    c1000 = [(net.spikes(0, p), orc.counts(p)) for p in (1, 2)]
    say(f"workload 1: V RMS over steps 1..1000 = {rms:.3e} mV")
    assert rms <= 1e-3
    for p, (a, b) in zip((1, 2), c1000):
        say(f"  pop {p}: counts identical for {np.mean(a == b) * 100:.2f}% of neurons at step 1000, "
            f"max |diff| {np.max(np.abs(a - b))}")
        assert np.array_equal(a, b)
    say("case: workload 1, steps 1000..10000")
    net.step(9000)
    orc.step(9000)
    assert np.array_equal(net.spikes(0, 0), orc.counts(0))
    for p in (1, 2):
        a, b = net.spikes(0, p), orc.counts(p)
        frac = np.mean(a == b)
        say(f"  pop {p}: counts identical for {frac * 100:.2f}% of neurons at step 10000, "
            f"max |diff| {np.max(np.abs(a - b))}, mean rate {b.mean():.1f} Hz")
        assert frac > 0.9
    assert net.nan_counts()[0] == orc.nan_count == 0
    net.close()


def test_network_parity_workload2_short(snn):
    """Workload 2 (A=1000, B=20000, C=1000; 15M synapses) for 300 steps."""
    say("case: workload 2, 300 steps")
    spec = netgen.make_config(2)
    net, orc, rms = _parity_run(snn, spec, 300)
    say(f"workload 2: V RMS over steps 1..300 (every 50th) = {rms:.3e} mV")
    assert rms <= 1e-3
    assert np.array_equal(net.spikes(0, 0), orc.counts(0))
    for p in (1, 2):
        assert np.mean(net.spikes(0, p) == orc.counts(p)) > 0.999
    net.close()


def test_graph_and_direct_launches_agree(snn):
    """64 steps through the captured graph equal 64 single-step launches."""
    say("case: graph vs direct")
    spec = netgen.make_config(1, scale=0.5)
    a = snn.Network(spec)
    b = snn.Network(spec)
    a.step(64)
    for _ in range(64):
        b.step(1)
    for p in (1, 2):
        for var in range(4):
            assert np.array_equal(a.state(0, p, var), b.state(0, p, var))
        assert np.array_equal(a.spikes(0, p), b.spikes(0, p))
    a.close()
    b.close()


@pytest.mark.parametrize("workload,scale", [(1, 0.5), (3, 0.05)])
def test_profiled_steps_advance_like_steps(snn, workload, scale):
    """snn_profile_steps advances the network exactly as snn_step does (the
    plastic workload included) and reports one launch of each step kernel
    per step with a positive duration."""
    say(f"case: profiled steps, workload {workload} at scale {scale}")
    spec = netgen.make_config(workload, scale=scale)
    a = snn.Network(spec)
    b = snn.Network(spec)
    a.step(150)
    b.step(20)
    prof = b.profile_steps(130)
    assert b.t == a.t == 150
    plastic = any(q.get("stdp") for q in spec["instances"][0]["projs"])
    for k, (ms, n) in prof.items():
        expect = 130 if (k != "potentiate" or plastic) else 0
        assert n == expect, (k, n)
        assert (ms > 0) == (expect > 0), (k, ms)
    for p in (1, 2):
        for var in range(4):
            assert np.array_equal(a.state(0, p, var), b.state(0, p, var))
        assert np.array_equal(a.spikes(0, p), b.spikes(0, p))
    for q in range(len(spec["instances"][0]["projs"])):
        assert np.array_equal(a.conductance(0, q), b.conductance(0, q))
        assert np.array_equal(a.weights(0, q), b.weights(0, q))
    a.close()
    b.close()


def test_launch_shape_does_not_change_results(snn):
    say("case: launch shapes")
    spec = netgen.make_config(1, scale=0.5)
    ref = snn.Network(spec)
    ref.step(200)
    for shape in [dict(neuron_block=64, prop_blocks=7, prop_block=64, chunk=64, mode=0),
                  dict(neuron_block=1024, prop_blocks=4096, prop_block=1024, chunk=2048, mode=0),
                  dict(neuron_block=128, prop_blocks=3, prop_block=256, chunk=256, mode=1),
                  dict(neuron_block=256, prop_blocks=2048, prop_block=256, chunk=256, mode=1)]:
        n = snn.Network(spec)
        n.set_launch(**shape)
        n.step(200)
        for p in (1, 2):
            assert np.array_equal(n.state(0, p, snn.V), ref.state(0, p, snn.V))
            assert np.array_equal(n.spikes(0, p), ref.spikes(0, p))
        for q in range(3):
            assert np.array_equal(n.conductance(0, q), ref.conductance(0, q))
        n.close()
    ref.close()


@pytest.mark.parametrize("workload,scale", [(1, 0.5), (2, 0.25), (3, 0.05)])
def test_delivery_modes_agree_bitwise_with_switches(snn, workload, scale):
    """Row-mode and tile-mode delivery, and switching between them while
    spikes are pending, give the same bits (fixed-point conductances); plastic
    weights included."""
    say(f"case: delivery modes, workload {workload} at scale {scale}")
    spec = netgen.make_config(workload, scale=scale)
    a = snn.Network(spec)
    b = snn.Network(spec)
    b.set_launch(mode=1)
    a.step(150)
    b.step(150)
    a.set_launch(mode=1)      # switch with work pending
    b.set_launch(mode=0)
    a.step(130)
    b.step(130)
    inst = spec["instances"][0]
    for p in range(len(inst["pops"])):
        assert np.array_equal(a.spikes(0, p), b.spikes(0, p))
        if inst["pops"][p]["kind"] == "hh":
            for var in range(4):
                assert np.array_equal(a.state(0, p, var), b.state(0, p, var))
    for q in range(len(inst["projs"])):
        assert np.array_equal(a.conductance(0, q), b.conductance(0, q))
        assert np.array_equal(a.weights(0, q), b.weights(0, q))
    a.close()
    b.close()


def test_pull_delivery_agrees_bitwise(snn):
    """Tile mode delivers the projections of a population with at least 7/8 of
    its neurons spiking by pulling (sliced-ELL column copies, one lane per
    column); the bits equal row mode's, through steps on both sides of the
    threshold, forced all-spiking populations, new weights and a new
    g_scale."""
    say("case: pull delivery against row mode")
    rng = np.random.default_rng(11)
    # A fires with probability 0.875 per step: its count straddles 7/8 of
    # 2000; A->B columns hold about 1000 entries (16 depth chunks); B spans
    # two post tiles and C ends in a partial slice
    inst = netgen.layered_instance(rng, 2000, 1500, 300, rate_hz=8750.0, p_ab=0.5, p_bc=0.3,
                                   g_scale=0.05, seed=(5 << 20) + 1)
    spec = dict(dt=0.1, substeps=3, instances=[inst])
    T = 120
    a = snn.Network(spec, raster_steps=T)
    b = snn.Network(spec)
    b.set_launch(mode=1)
    a.step(T)
    b.step(T)
    thr = (2000 * 7 + 7) // 8
    per_step = np.array([len(r) for r in a.raster(0, 0, 0, T)])
    say(f"  A spikes per step: min {per_step.min()} max {per_step.max()}, "
        f"{np.mean(per_step >= thr) * 100:.0f}% of steps pulled")
    assert 0 < np.sum(per_step >= thr) < T
    _same_network_state(a, b, spec)
    # every B and C neuron spiked at t - 1: their projections are pulled
    for p in (1, 2):
        ones = np.ones(inst["pops"][p]["n"], np.uint8)
        a.set_last_spikes(0, p, ones)
        b.set_last_spikes(0, p, ones)
    a.step(3)
    b.step(3)
    _same_network_state(a, b, spec)
    # new weights (the column-ordered copies follow) and a new g_scale
    import torch
    w = torch.empty(a.weight_count, dtype=torch.float32, device="cuda")
    a.get_weights_device(w)
    w = w * torch.linspace(0.5, 1.5, w.numel(), device="cuda")
    a.set_weights_device(w)
    b.set_weights_device(w)
    a.set_gscale(np.array([0.07], np.float32))
    b.set_gscale(np.array([0.07], np.float32))
    for p in (1, 2):
        ones = np.ones(inst["pops"][p]["n"], np.uint8)
        a.set_last_spikes(0, p, ones)
        b.set_last_spikes(0, p, ones)
    a.step(57)
    b.step(57)
    _same_network_state(a, b, spec)
    # switches with pulled work pending (all B and C neurons spiked at t - 1):
    # rows <-> tiles, then tiles -> fused (the pending pull runs into the
    # fused delivery buffer) against rows -> fused, then back
    plan = [(dict(mode=1), dict(mode=0), 31), (dict(mode=2), dict(mode=2), 17),
            (dict(mode=1), dict(mode=0), 23)]
    for la, lb, n in plan:
        for p in (1, 2):
            ones = np.ones(inst["pops"][p]["n"], np.uint8)
            a.set_last_spikes(0, p, ones)
            b.set_last_spikes(0, p, ones)
        a.set_launch(**la)
        b.set_launch(**lb)
        say(f"  modes {a.launch['mode']} / {b.launch['mode']}, {n} steps")
        a.step(n)
        b.step(n)
        _same_network_state(a, b, spec)
    a.close()
    b.close()


def test_pull_delivery_paths(snn):
    """The pull delivery's other paths against row mode, bitwise: spike words
    looked up in global memory (a pulled population of 70 000 neurons), copied
    into LDS in a loop (65 to 1024 words), single-chunk slices adding into G
    directly, deep slices reduced in one group and in several groups with
    atomics (columns of 5000 entries), a partial last slice, and a projection
    too sparse for one-byte row deltas (no copy: pushed while its population
    is pulled elsewhere)."""
    say("case: pull delivery paths")
    rng = np.random.default_rng(21)
    pops = [dict(name="A", kind="poisson", n=70000, rate_hz=9500.0, i_ext=0.0),
            dict(name="B", kind="hh", n=5000, rate_hz=0.0, i_ext=0.0),
            dict(name="C", kind="hh", n=100, rate_hz=0.0, i_ext=0.0),
            dict(name="D", kind="poisson", n=6000, rate_hz=9500.0, i_ext=0.0)]
    projs = []
    for pre, post, p, tau, erev in [(0, 1, 0.01, netgen.TAU_AB, netgen.E_EXC), (3, 1, 0.02, netgen.TAU_AB, netgen.E_EXC),
                                    (1, 2, 1.0, netgen.TAU_BC, netgen.E_EXC), (2, 2, 1.0, netgen.TAU_CC, netgen.E_INH),
                                    (0, 2, 0.0005, netgen.TAU_AB, netgen.E_EXC)]:
        n_pre, n_post = pops[pre]["n"], pops[post]["n"]
        rp, ci = netgen.bernoulli_csr(rng, n_pre, n_post, p, no_self=(pre == post))
        projs.append(dict(pre=pre, post=post, row_ptr=rp, col_idx=ci,
                          g=netgen.uniform_weights(rng, ci.size, 0.05 / (n_pre * p)),
                          e_rev=erev, tau=tau, stdp=None))
    inst = dict(g_scale=0.05, seed=(6 << 20) + 3, pops=pops, projs=projs)
    spec = dict(dt=0.1, substeps=3, instances=[inst])
    a = snn.Network(spec)
    b = snn.Network(spec)
    b.set_launch(mode=1)
    for n in (40, 20, 20):
        a.step(n)
        b.step(n)
        _same_network_state(a, b, spec)
        for p in (1, 2):       # every B and C neuron spiked at t - 1
            ones = np.ones(pops[p]["n"], np.uint8)
            a.set_last_spikes(0, p, ones)
            b.set_last_spikes(0, p, ones)
    a.step(5)
    b.step(5)
    _same_network_state(a, b, spec)
    assert a.nan_counts()[0] == 0
    a.close()
    b.close()


def _csr_from_columns(n_pre, columns):
    """CSR (ascending columns per row) of the connectivity whose column j
    holds the pre rows columns[j]."""
    pairs = sorted((int(r), j) for j, rows in enumerate(columns) for r in rows)
    counts = np.zeros(n_pre, np.int64)
    for r, _ in pairs:
        counts[r] += 1
    rp = np.zeros(n_pre + 1, np.int64)
    np.cumsum(counts, out=rp[1:])
    return rp.astype(np.int32), np.array([j for _, j in pairs], np.int32)


@pytest.mark.parametrize("n_pre", [3000, 70000])
def test_pull_row_delta_edges(snn, n_pre):
    """The pull copy stores each column's rows as one-byte deltas, gaps above
    255 bridged by weight-0 entries.  With integer weights, one pulled
    delivery equals the oracle's bit for bit on columns built at the edges
    of that encoding: gaps of 254, 255, 256, 510, 511 and 765 rows, a first
    row far from 0, a single entry at the last row, the first and last row
    only, every row (a slice of several pull units), empty columns, and
    random columns of density 0.003 to 0.5 (in LDS and, at 70 000 pre
    neurons, global spike words)."""
    say(f"case: pull delta edges, {n_pre} pre neurons")
    rng = np.random.default_rng(31 + n_pre)
    n_post = 300
    cols = [np.arange(0, n_pre, 255), np.arange(7, n_pre, 256), np.arange(3, n_pre, 254),
            np.cumsum(np.tile([510, 511, 765], n_pre // 1786 + 1))[: n_pre // 600] % n_pre,
            np.array([n_pre - 1]), np.array([0, n_pre - 1]), np.arange(n_pre), np.array([], np.int64),
            np.array([1000, 1255, 1511])]
    while len(cols) < n_post:
        d = 10 ** rng.uniform(np.log10(0.003), np.log10(0.5))
        if rng.random() < 0.05:
            cols.append(np.array([], np.int64))
        else:
            cols.append(np.nonzero(rng.random(n_pre) < d)[0])
    cols = [np.unique(c) for c in cols]
    rp, ci = _csr_from_columns(n_pre, cols)
    # integer weights up to 3 and a 1 ms decay keep the full column's
    # reachable conductance within the library's fixed-point range
    g = rng.integers(0, 4, ci.size).astype(np.float32)
    pops = [dict(name="A", kind="poisson", n=n_pre, rate_hz=0.0, i_ext=0.0),
            dict(name="B", kind="hh", n=n_post, rate_hz=0.0, i_ext=0.0)]
    projs = [dict(pre=0, post=1, row_ptr=rp, col_idx=ci, g=g, e_rev=0.0, tau=1.0, stdp=None)]
    inst = dict(g_scale=1.0, seed=99, pops=pops, projs=projs)
    spec = dict(dt=0.1, substeps=3, instances=[inst])
    net = snn.Network(spec)
    net.set_launch(mode=1)
    orc = O.OracleNet(inst)
    for frac in (1.0, 0.9):
        flags = np.ones(n_pre, np.uint8)
        if frac < 1.0:
            flags[rng.choice(n_pre, int(round((1 - frac) * n_pre)), replace=False)] = 0
        net.set_last_spikes(0, 0, flags)
        orc.set_last_spikes(0, flags)
        net.set_conductance(0, 0, np.zeros(n_post))
        orc.set_G(0, np.zeros(n_post))
        net.step(1)
        orc.step(1)
        g_gpu = net.conductance(0, 0) * FIX
        g_orc = np.rint(orc.G(0) * FIX)
        assert np.array_equal(g_gpu, g_orc), np.nonzero(g_gpu != g_orc)[0][:10]
    net.close()


def _same_network_state(a, b, spec):
    inst = spec["instances"][0]
    for p in range(len(inst["pops"])):
        assert np.array_equal(a.spikes(0, p), b.spikes(0, p))
        assert np.array_equal(a.last_spikes(0, p), b.last_spikes(0, p))
        if inst["pops"][p]["kind"] == "hh":
            for var in range(4):
                assert np.array_equal(a.state(0, p, var), b.state(0, p, var))
    for q in range(len(inst["projs"])):
        assert np.array_equal(a.conductance(0, q), b.conductance(0, q))


@pytest.mark.parametrize("workload,scale", [(1, 0.5), (2, 0.25)])
def test_fused_mode_agrees_bitwise_through_switches(snn, workload, scale):
    """Mode 2 (the neuron update delivers its own spikes into a double-buffered
    delivery buffer) gives the same bits as row mode, also across switches in
    every direction with work pending, with odd step counts (both buffer
    slots) and several launch shapes."""
    say(f"case: fused mode, workload {workload} at scale {scale}")
    spec = netgen.make_config(workload, scale=scale)
    ref = snn.Network(spec)
    fus = snn.Network(spec)
    fus.set_launch(mode=2)
    plan = [(77, dict(mode=2)), (51, dict(mode=1)), (33, dict(mode=2, neuron_block=64, chunk=64)),
            (41, dict(mode=0)), (29, dict(mode=2, neuron_block=1024, chunk=2048)), (64, dict(mode=2, chunk=512))]
    for i, (n, shape) in enumerate(plan):
        ref.step(n)
        fus.step(n)
        say(f"  phase {i}: {n} steps in mode {fus.launch['mode']}, then {shape}")
        _same_network_state(ref, fus, spec)
        fus.set_launch(**shape)
    ref.step(70)
    fus.step(70)
    _same_network_state(ref, fus, spec)
    ref.close()
    fus.close()


@pytest.mark.parametrize("workload,scale", [(1, 0.5), (2, 0.25)])
def test_grouped_mode_agrees_bitwise_through_switches(snn, workload, scale):
    """Mode 3 (small projections delivered in row groups through LDS tiles)
    gives the same bits as row mode, also across switches to and from every
    other mode with work pending, with odd step counts and several launch
    shapes."""
    say(f"case: grouped mode, workload {workload} at scale {scale}")
    spec = netgen.make_config(workload, scale=scale)
    ref = snn.Network(spec)
    grp = snn.Network(spec)
    grp.set_launch(mode=3)
    plan = [(77, dict(mode=0)), (51, dict(mode=3, prop_blocks=1)), (33, dict(mode=2)),
            (41, dict(mode=3, prop_block=64, chunk=64)), (29, dict(mode=1)), (64, dict(mode=3, prop_block=512)),
            (35, dict(mode=3, neuron_block=1024, prop_blocks=8192))]
    for i, (n, shape) in enumerate(plan):
        ref.step(n)
        grp.step(n)
        say(f"  phase {i}: {n} steps in mode {grp.launch['mode']}, then {shape}")
        _same_network_state(ref, grp, spec)
        grp.set_launch(**shape)
    ref.step(70)
    grp.step(70)
    _same_network_state(ref, grp, spec)
    ref.close()
    grp.close()


def test_grouped_mode_rejects_wide_blocks(snn):
    """Grouped mode keeps an 8 KiB LDS tile per wavefront, so blocks of more
    than 512 threads are refused (the launch is left as it was)."""
    spec = netgen.make_config(1, scale=0.5)
    net = snn.Network(spec)
    with pytest.raises(snn.SNNError):
        net.set_launch(mode=3, prop_block=1024)
    net.set_launch(mode=3, prop_block=512)
    net.step(5)
    net.close()


def test_fused_mode_last_spikes_and_rejection(snn):
    """Replacing S(t-1) in fused mode redoes its pending deliveries; a
    network with plastic projections refuses mode 2."""
    say("case: fused mode, set_last_spikes and plastic rejection")
    spec = netgen.make_config(1, scale=0.5)
    a = snn.Network(spec)
    b = snn.Network(spec)
    b.set_launch(mode=2)
    a.step(40)
    b.step(40)
    rng = np.random.default_rng(3)
    for p, pop in enumerate(spec["instances"][0]["pops"]):
        f = (rng.random(pop["n"]) < 0.3).astype(np.uint8)
        a.set_last_spikes(0, p, f)
        b.set_last_spikes(0, p, f)
    a.step(60)
    b.step(60)
    _same_network_state(a, b, spec)
    a.close()
    b.close()
    plastic = snn.Network(netgen.make_config(3, scale=0.05))
    with pytest.raises(RuntimeError, match="fused"):
        plastic.set_launch(mode=2)
    plastic.close()


def test_vbar_accumulates_post_step_voltage(snn):
    say("case: vbar")
    spec = netgen.make_config(1, scale=0.3)
    net = snn.Network(spec, record_vbar=("C",))
    orc = O.OracleNet(spec["instances"][0])
    acc = np.zeros(spec["instances"][0]["pops"][2]["n"])
    for _ in range(100):
        net.step(1)
        orc.step(1)
        acc += net.state(0, 2, snn.V)
    vs = net.vbar_sum(0, 2)
    assert np.allclose(vs, acc, rtol=0, atol=1e-9)
    assert np.max(np.abs(vs - orc.vsum(2))) < 1e-3
    net.close()


def test_network_parity_workload2_1000_steps_autotuned(snn):
    """Workload 2 (A=1000, B=20000, C=1000; 15M synapses), in the launch
    shape the autotuner picks: V RMS over every one of the first 1000 steps
    within 1e-3 mV, spike counts per neuron."""
    say("case: workload 2, autotuned launch, 1000 steps")
    spec = netgen.make_config(2)
    inst = spec["instances"][0]
    net = snn.Network(spec, autotune=True)
    say(f"  launch {net.launch}")
    orc = O.OracleNet(inst)
    se, cnt = 0.0, 0
    for _ in range(1000):
        net.step(1)
        orc.step(1)
        for p in (1, 2):
            d = net.state(0, p, snn.V) - orc.get(p, O.V)
            se += float(np.sum(d * d))
            cnt += d.size
    rms = math.sqrt(se / cnt)
    say(f"  V RMS over every step 1..1000 = {rms:.3e} mV")
    assert rms <= 1e-3
    assert np.array_equal(net.spikes(0, 0), orc.counts(0))
    for p in (1, 2):
        a, b = net.spikes(0, p), orc.counts(p)
        say(f"  pop {p}: counts identical for {np.mean(a == b) * 100:.3f}% of neurons, max |diff| {np.max(np.abs(a - b))}")
        assert np.mean(a == b) > 0.999
    net.close()


@pytest.mark.parametrize("workload", [1, 2])
def test_raster_replay_rms(snn, workload):
    """Raster replay: a GPU network whose hidden and output spikes are
    overwritten after every step by the oracle's own spikes of that step, so
    that both integrate exactly the same synaptic input; the V difference is
    then arithmetic alone.  Reported beside the free-running difference over
    the same first 1000 steps; both within 1e-3 mV RMS."""
    say(f"case: workload {workload}, free-running and raster-replay V RMS over 1000 steps")
    spec = netgen.make_config(workload)
    inst = spec["instances"][0]
    free = snn.Network(spec)
    rep = snn.Network(spec)
    orc = O.OracleNet(inst)
    se = {"free": 0.0, "replay": 0.0}
    cnt = 0
    flips = 0
    for _ in range(1000):
        free.step(1)
        rep.step(1)
        orc.step(1)
        for p in (1, 2):
            vo = orc.get(p, O.V)
            for key, net in (("free", free), ("replay", rep)):
                d = net.state(0, p, snn.V) - vo
                se[key] += float(np.sum(d * d))
            cnt += vo.size
            own = rep.last_spikes(0, p)
            ref = orc.last_spikes(p)
            flips += int(np.count_nonzero(own != ref))
            rep.set_last_spikes(0, p, ref)
    rms = {k: math.sqrt(v / cnt) for k, v in se.items()}
    say(f"  V RMS over steps 1..1000: free-running {rms['free']:.3e} mV, raster replay {rms['replay']:.3e} mV; "
        f"{flips} spikes the replayed network detected differently from the oracle")
    assert rms["free"] <= 1e-3 and rms["replay"] <= 1e-3
    for net in (free, rep):
        net.close()


def _rate_sums(v):
    """alpha + beta of m, h and n at voltages v (mV)."""
    def ratio(x):
        with np.errstate(all="ignore"):
            r = x / np.expm1(x)
        return np.where(np.abs(x) < 1e-6, 1.0 - 0.5 * x, np.where(x > 700.0, 0.0, r))
    with np.errstate(over="ignore"):
        m = 1.28 * ratio((-52.0 - v) / 4.0) + 1.4 * ratio((v + 25.0) / 5.0)
        h = 0.128 * np.exp((-48.0 - v) / 18.0) + 4.0 / (1.0 + np.exp((-25.0 - v) / 5.0))
        n = 0.16 * ratio((-50.0 - v) / 5.0) + 0.5 * np.exp((-55.0 - v) / 40.0)
    return m, h, n


def test_rates_at_the_edges_of_their_forms(snn):
    """One Euler substep at voltages on both sides of every line between the
    forms of the rates (the near range's +-200 mV, the power form's +-1000 mV,
    |x| = 1/64 of each removable singularity), with and without such lanes in
    the same wavefront.  A gate's step is h (a (1 - x) - b x); the rates are
    within 6e-13 relative of the oracle's and the pair holds 48 bits, so the
    gates agree within 1e-12 (1 + h (a + b))."""
    say("case: rates at the edges of their forms")
    edges = [s * e for e in (200.0, 1000.0) for s in (-1.0, 1.0)]
    edges += [c + s * w / 64.0 for c, w in ((-52.0, 4.0), (-25.0, 5.0), (-50.0, 5.0)) for s in (-1.0, 0.0, 1.0)]
    at = np.array([x for e in edges for x in (np.nextafter(np.float32(e), -np.inf, dtype=np.float32), np.float32(e),
                                              np.nextafter(np.float32(e), np.inf, dtype=np.float32))], np.float64)
    plain = np.linspace(-100.3, 59.7, 64 * 3)                      # whole wavefronts without an edge lane
    plain = plain[np.all([np.abs(plain - c) > 0.2 for c in (-52.0, -50.0, -25.0)], axis=0)][:128]
    v = np.concatenate([plain, at, np.array([-900.0, -450.0, 333.0, 1500.0, -1200.0])])
    inst = dict(g_scale=1.0, seed=1, pops=[dict(name="P", kind="hh", n=v.size, rate_hz=0.0, i_ext=0.0)], projs=[])
    spec = dict(dt=0.02, substeps=1, instances=[inst])
    net = snn.Network(spec)
    orc = O.OracleNet(inst, dt=0.02, substeps=1)
    for var, x in ((snn.V, v), (snn.M, np.full(v.size, 0.25)), (snn.H, np.full(v.size, 0.6)), (snn.N, np.full(v.size, 0.4))):
        net.set_state(0, 0, var, x)
        orc.set(0, var, net.state(0, 0, var))
    net.step(1)
    orc.step(1)
    for var, s in zip((snn.M, snn.H, snn.N), _rate_sums(v)):
        a, b = net.state(0, 0, var), orc.get(0, var)
        assert np.all(np.abs(a - b) <= 1e-12 * (1.0 + 0.02 * s)), (var, v[np.argmax(np.abs(a - b) / (1.0 + 0.02 * s))])
    net.close()
