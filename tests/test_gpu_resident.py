"""Resident stepping against the step kernels: the steps that a network takes
by default are bitwise those of an explicitly chosen launch shape, over the
splits of its words that the plan can make, and pending work survives every
change between the two."""
import numpy as np
import pytest

from paper_1412_0595_amd import netgen

pytestmark = pytest.mark.gpu

MODES = (dict(mode=0), dict(mode=1), dict(mode=2), dict(mode=3))


@pytest.fixture(scope="module")
def snn():
    from paper_1412_0595_amd import snn as s
    s.load()
    return s


def layered(n, a, b, c, p_bc=0.5, rate=40.0):
    rng = np.random.default_rng(11)
    return dict(dt=0.1, substeps=3, instances=[
        netgen.layered_instance(rng, a + 3 * i, b + 70 * i, c + i, rate_hz=rate, p_ab=0.3, p_bc=p_bc,
                                seed=netgen.instance_seed(11, i)) for i in range(n)])


def izhikevich():
    return dict(dt=0.1, substeps=3, instances=[
        netgen.izhikevich_instance(100, n_exc=241, n_inh=63, seed=netgen.instance_seed(5, i), conn_seed=5 + i)
        for i in range(3)])


# one block; a few; the blocks of 64-neuron parts and of odd remainders; many
# single blocks (more than the device has compute units); two neuron models
NETS = {
    "tiny": lambda: layered(1, 5, 7, 3, 1.0),
    "word_edges": lambda: layered(1, 64, 128, 65),
    "small": lambda: layered(1, 100, 1000, 100, 1.0),
    "split": lambda: layered(1, 300, 6001, 257),
    "uneven": lambda: layered(5, 130, 500, 40),
    "many": lambda: layered(300, 20, 40, 5),
    "izh": izhikevich,
}


def everything(net, spec):
    """All state that the steps leave, as one list of arrays."""
    out = [net.nan_counts()]
    for b, inst in enumerate(spec["instances"]):
        for p, pop in enumerate(inst["pops"]):
            out += [net.spikes(b, p), net.last_spikes(b, p)]
            if pop["kind"] != "poisson":
                out += [net.state(b, p, v) for v in range(2 if pop["kind"] == "izh" else 4)]
        out += [net.conductance(b, q) for q in range(len(inst["projs"]))]
    return out


def differing(x, y):
    """Indexes of the arrays that differ."""
    assert len(x) == len(y)
    return [k for k, (a, b) in enumerate(zip(x, y)) if not np.array_equal(a, b, equal_nan=a.dtype.kind == "f")]


def by_modes(snn, spec, mode, run):
    net = snn.Network(spec)
    net.set_launch(**mode)
    run(net)
    out = everything(net, spec)
    net.close()
    return out


@pytest.mark.parametrize("name", list(NETS))
def test_default_steps_equal_the_step_kernels(snn, name):
    print(f"case: resident {name}", flush=True)
    spec = NETS[name]()

    def run(net):
        for n in (1, 30, 7, 200, 2):
            net.step(n)
    net = snn.Network(spec)
    run(net)
    got = everything(net, spec)
    net.reset()
    run(net)
    assert not differing(got, everything(net, spec))
    net.close()
    for mode in MODES[:1] if name == "many" else MODES:
        assert not differing(got, by_modes(snn, spec, mode, run)), mode


@pytest.mark.parametrize("name", ["small", "split", "izh"])
@pytest.mark.parametrize("frac", [0.02, 1.0])
def test_given_spikes_and_changes_of_path(snn, name, frac):
    """Spikes set from outside (all at once too: more rows than one listing
    holds), pending when the path changes, in both directions."""
    print(f"case: resident spikes {name} {frac}", flush=True)
    spec = NETS[name]()
    rng = np.random.default_rng(2)
    n_pops = len(spec["instances"][0]["pops"])
    flags = [(rng.random(spec["instances"][0]["pops"][p]["n"]) < frac).astype(np.uint8) for p in range(n_pops)]

    def run(net, change=None):
        net.step(20)
        for p in range(n_pops):
            net.set_last_spikes(0, p, flags[p])
        if change:
            net.set_launch(**change)
        net.step(1)
        net.step(9)
    ref = by_modes(snn, spec, dict(mode=0), run)
    for change in (None, *MODES):
        net = snn.Network(spec)
        run(net, change)
        assert not differing(ref, everything(net, spec)), change
        net.close()


def test_recorded_steps(snn):
    """Raster ring and voltage sums of resident steps."""
    print("case: resident records", flush=True)
    spec = layered(2, 100, 900, 70)

    def run(net):
        net.step(75)
        out = [net.vbar_sum(0, 2), net.vbar_sum(1, 2)]
        for b in range(2):
            for p in range(3):
                out += net.raster(b, p, 25, 75)
        return out
    got = []
    for mode in (None, dict(mode=0)):
        net = snn.Network(spec, record_vbar=("C",), raster_steps=64)
        if mode:
            net.set_launch(**mode)
        got.append(run(net))
        net.close()
    assert not differing(*got)


def test_sources_drawn_ahead(snn):
    """Streams that instances share or not, over calls above and below the
    length from which sources are drawn ahead, longer and shorter than the
    raster ring, and a rate at which every source spikes."""
    print("case: resident sources", flush=True)
    shared = layered(1, 130, 300, 20)["instances"][0]
    other = dict(shared, seed=77, pops=[dict(shared["pops"][0], rate_hz=900.0), *shared["pops"][1:]])
    always = dict(shared, pops=[dict(shared["pops"][0], rate_hz=1e5), *shared["pops"][1:]])
    spec = dict(dt=0.1, substeps=3, instances=[shared, other, dict(shared, g_scale=0.5), always, shared])
    got = []
    for mode in (None, dict(mode=0)):
        net = snn.Network(spec, raster_steps=16)
        if mode:
            net.set_launch(**mode)
        out = []
        for n in (40, 3, 33, 32, 31, 2100):
            net.step(n)
            for b in range(5):
                out += net.raster(b, 0, net.t - min(n, 16), net.t)
            out += everything(net, spec)
        got.append(out)
        net.close()
    assert not differing(*got)


def test_several_networks_step_at_once(snn):
    """Networks on streams and threads of their own, whose blocks together
    are more than the device holds at once."""
    import threading

    import torch
    print("case: resident networks at once", flush=True)
    specs = [layered(1, 300, 5000 + 501 * i, 257) for i in range(4)]

    def run(net, k):
        for _ in range(5):
            net.step(60)
        net.sync()
        got[k] = everything(net, specs[k])
    ref = []
    for spec in specs:
        net = snn.Network(spec)
        net.set_launch(mode=0)
        net.step(300)
        ref.append(everything(net, spec))
        net.close()
    got = {}
    nets = [snn.Network(spec, stream=torch.cuda.Stream()) for spec in specs]
    threads = [threading.Thread(target=run, args=(net, k)) for k, net in enumerate(nets)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k, net in enumerate(nets):
        assert not differing(ref[k], got[k]), k
        net.close()


def test_weights_set_while_tile_mode_waits(snn):
    """Weights set while the steps run resident reach the copies of the mode
    chosen afterwards."""
    import torch
    print("case: resident then tiles", flush=True)
    spec = layered(1, 100, 700, 65)
    out = []
    for first in (None, dict(mode=1)):
        net = snn.Network(spec)
        if first:
            net.set_launch(**first)
        w = torch.empty(net.weight_count, dtype=torch.float32, device="cuda")
        net.get_weights_device(w)
        net.step(30)
        net.set_weights_device(w * 0.5)
        net.step(30)
        net.set_launch(mode=1)
        for p in range(3):
            net.set_last_spikes(0, p, np.ones(spec["instances"][0]["pops"][p]["n"], np.uint8))
        net.step(1)
        net.step(30)
        out.append(everything(net, spec))
        net.close()
    assert not differing(*out)


def test_long_segments_and_groups(snn):
    """The gradient does not depend on how many segments the tape holds: the
    no-allocation entry point's smaller one, and one segment of all steps."""
    import torch
    print("case: adjoint groups", flush=True)
    spec = layered(2, 60, 300, 40)
    for T, K in ((64, 1), (150, 40), (120, 120)):
        net = snn.Network(spec, record_vbar=("C",))
        vb = net.forward_record(2, T, K)
        dg, ds, bad = net.backward(vb, check=True)
        dg2, ds2 = torch.empty_like(dg), torch.empty_like(ds)
        net.backward_noalloc(vb, dg2, ds2)
        assert bad == 0 and torch.equal(dg, dg2) and float(dg.abs().sum()) > 0
        net.close()


@pytest.mark.parametrize("before", (0, 64))
def test_steps_while_the_stream_is_captured(snn, before):
    """A capture does not record steps: they run at once or, after resident
    steps, are refused, and the net goes on as if they had not been asked for."""
    import torch
    print("case: capture", before, flush=True)
    spec = layered(1, 100, 500, 50)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        net, ref = (snn.Network(spec, stream=stream) for _ in range(2))
        for q in (net, ref):
            q.step(before)
            q.sync()
        graph = torch.cuda.CUDAGraph()
        refused = False
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
            try:
                net.step(2)
            except snn.SNNError as e:
                refused = True
                assert e.code == snn.SNN_EINVAL
        assert refused == (before > 0)
        if not refused:
            ref.step(2)
        for q in (net, ref):
            q.step(40)
        assert not differing(everything(net, spec), everything(ref, spec))
        net.close()
        ref.close()


@pytest.mark.parametrize("name", ["uneven", "wide"])
def test_even_calls_keep_the_words_they_begin_with(snn, name):
    """Calls of an even number of steps end in the slot of spike words that
    they begin from.  "wide" has blocks that begin late (bounds of 20 000 rows
    to load) beside blocks that only sources feed.  Calls of 2 to 8 steps at
    every phase of the exchange, and as the last launch of a long call."""
    print(f"case: resident even calls {name}", flush=True)
    rng = np.random.default_rng(12)
    spec = NETS["uneven"]() if name == "uneven" else dict(dt=0.1, substeps=3, instances=[
        netgen.layered_instance(rng, 1000, 20000, 1000, rate_hz=40.0, p_ab=0.2, p_bc=0.5, seed=12)])
    flags = [[(rng.random(p["n"]) < 0.05).astype(np.uint8) for p in spec["instances"][0]["pops"]] for _ in range(4)]
    got = []
    for mode in (None, dict(mode=0)):
        net = snn.Network(spec)
        if mode:
            net.set_launch(**mode)
        out = []
        net.step(64)
        for n in (2, 4, 6, 8):
            for phase in range(8):
                net.step(n)
                net.step(n)
                net.step(9 + (phase - net.t) % 8)        # the next calls begin at step phase + 1 mod 8
                if phase % 2:
                    for p, f in enumerate(flags[n // 2 - 1]):
                        net.set_last_spikes(0, p, f)
            net.step(2048 + n)
            out += everything(net, spec)
        got.append(out)
        net.close()
    assert not differing(*got)


def singles():
    """More networks than compute units, each in a block of its own."""
    base = layered(1, 70, 500, 20)["instances"][0]
    return dict(dt=0.1, substeps=3, instances=[dict(base, seed=netgen.instance_seed(11, i)) for i in range(300)])


@pytest.mark.parametrize("name", ["word_edges", "split", "singles", "izh"])
def test_short_calls_between_long_ones(snn, name):
    """Calls of a few steps go through the step kernels, which take the
    pending work over from resident steps and from spikes set from outside,
    and hand it back."""
    print(f"case: resident short calls {name}", flush=True)
    spec = singles() if name == "singles" else NETS[name]()
    rng = np.random.default_rng(6)
    flags = [(rng.random(p["n"]) < 0.3).astype(np.uint8) for p in spec["instances"][0]["pops"]]

    def run(net):
        for n in (3, 64, 1, 1, 2, 4, 3, 5, 1):
            net.step(n)
        for n in (1, 2, 64):
            for p, f in enumerate(flags):
                net.set_last_spikes(0, p, f)
            net.step(n)
            net.step(3)
    net = snn.Network(spec)
    run(net)
    got = everything(net, spec)
    net.close()
    assert not differing(got, by_modes(snn, spec, dict(mode=0), run))


def test_several_threads_read_one_network(snn):
    """Readers of one network on threads of their own each get their own
    array (small reads share the network's staging memory)."""
    import threading
    print("case: resident readers", flush=True)
    spec = layered(3, 100, 1000, 70)
    net = snn.Network(spec)
    net.step(200)
    reads = [lambda b=b, p=p, v=v: net.state(b, p, v) for b in range(3) for p in (1, 2) for v in range(4)]
    reads += [lambda b=b, p=p: net.spikes(b, p) for b in range(3) for p in range(3)]
    reads += [lambda p=p: net.spike_totals(p) for p in range(3)]
    want = [r() for r in reads]
    wrong = []

    def run(k):
        for i in range(300):
            at = (7 * k + i) % len(reads)
            if not np.array_equal(reads[at](), want[at]):
                wrong.append(at)
    threads = [threading.Thread(target=run, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    net.close()


def steps_resident(snn, net, stream):
    """Whether the network's long calls run resident: stepping while the
    stream is captured is refused after such a call alone."""
    import torch
    net.step(64)
    net.sync()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
        try:
            net.step(1)
        except snn.SNNError:
            return True
    return False


@pytest.mark.parametrize("mode", range(4))
def test_tune_cache_keeps_the_choice(snn, tmp_path, mode):
    """A cached network takes the path that the line names, in every mode of
    its step kernels; a line without that number keeps its shape and gets it."""
    import torch
    print(f"case: resident tune cache {mode}", flush=True)
    spec = layered(1, 100, 500, 50)
    path = tmp_path / "tune.json"
    snn.Network(spec, autotune=True, tune_cache=path).close()
    line = next(x for x in path.read_text().splitlines() if "[" in x)
    key, tuned = line[:line.index("[")], [int(x) for x in line[line.index("[") + 1:line.index("]")].split(",")]
    assert len(tuned) == 6 and tuned[5] in (0, 1)
    shape = [256, 1024, 256, 256, mode]

    def run(net):
        for n in (64, 1, 3, 40, 2):
            net.step(n)
        net.set_last_spikes(0, 1, np.ones(500, np.uint8))
        net.step(1)
        net.step(2)
    ref = by_modes(snn, spec, dict(mode=0), run)
    for numbers, want in ((shape + [0], False), (shape + [1], True), (shape, None)):
        path.write_text("{\n%s%s\n}\n" % (key, numbers))
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            net = snn.Network(spec, autotune=True, tune_cache=path, stream=stream)
            assert list(net.launch.values()) == shape
            run(net)
            assert not differing(ref, everything(net, spec)), numbers
            got = steps_resident(snn, net, stream)
            net.close()
        if want is None:
            now = [int(x) for x in path.read_text().split("[")[1].split("]")[0].split(",")]
            assert now == shape + [int(got)]
        else:
            assert got == want, numbers


def test_tables_given_back(snn, tmp_path):
    """The resident tables (8 bytes per synapse and more) go when the step
    kernels are chosen: by the caller, or by the line of a tune cache."""
    import torch
    print("case: resident tables given back", flush=True)
    spec = layered(1, 300, 3000, 257)
    path = tmp_path / "tune.json"
    used = torch.cuda.memory_allocated
    base = used()
    net = snn.Network(spec, autotune=True, tune_cache=path)
    net.step(40)
    full = used()
    net.set_launch(mode=0)
    assert used() <= full - 8 * net.weight_count
    net.step(40)
    net.set_launch(mode=2)
    net.step(40)
    got = everything(net, spec)
    net.close()
    assert used() == base
    path.write_text(path.read_text().replace(", 1]", ", 0]"))
    net = snn.Network(spec, autotune=True, tune_cache=path)
    assert used() <= base + (full - base) - 8 * net.weight_count
    net.step(120)
    assert not differing(got, everything(net, spec))
    net.close()


def test_tags_begin_anew(snn):
    """The exchange's tags begin anew every 2^20 steps: long calls up to and
    beyond that, short ones, whose sources go through the exchange again, and
    long ones."""
    print("case: resident tags", flush=True)
    spec = layered(1, 70, 130, 20)
    got = []
    for mode in (None, dict(mode=2)):
        net = snn.Network(spec)
        if mode:
            net.set_launch(**mode)
        net.step(30)
        net.step((1 << 20) - 100)
        for n in [5] * 30 + [700, 17, 31]:
            net.step(n)
        got.append(everything(net, spec))
        net.close()
    assert not differing(*got)


def sources_onto(a, b, rate, n=1, p=None):
    base = netgen.layered_instance(np.random.default_rng(3), a, b, 10, rate_hz=rate, p_ab=p or min(0.5, 2e6 / a / b),
                                   p_bc=0.5)
    return dict(dt=0.1, substeps=3, instances=[dict(base, seed=netgen.instance_seed(3, i)) for i in range(n)])


@pytest.mark.parametrize("make,want", [
    (lambda: sources_onto(100000, 1000, 200.0), False),       # each block would walk 2 000 rows a step
    (lambda: sources_onto(300000, 64, 20.0), False),
    (lambda: sources_onto(20000, 1000, 20.0), True),
    (lambda: sources_onto(5000, 1000, 1000.0), True),         # rows of 400 synapses
    (lambda: sources_onto(5000, 100, 1000.0, n=40), True),
    (lambda: layered(1, 100, 1000, 100, 1.0), True),
    (singles, True)])
def test_networks_that_run_resident(snn, make, want):
    """Networks whose sources' deliveries outweigh the shorter chain keep the
    step kernels, which spread them over the chip."""
    import torch
    print("case: resident choice", flush=True)
    spec = make()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        net = snn.Network(spec, stream=stream)
        assert steps_resident(snn, net, stream) == want
        net.close()


def mixed(seed):
    """Instances of populations of all kinds in any order and size, with
    several, no or empty projections, and a step of any length."""
    rng = np.random.default_rng([seed, 9])
    instances = []
    for i in range(rng.integers(1, 4)):
        pops, projs = [], []
        kinds = rng.permutation(["poisson", "hh", *rng.choice(["hh", "izh", "poisson"], rng.integers(1, 4))])
        for k, kind in enumerate(kinds):
            n = int(rng.choice([1, 63, 64, 65, 130, rng.integers(2, 900)]))
            pop = dict(name=f"{kind}{k}", kind=str(kind), n=n, rate_hz=float(rng.choice([0.0, 50.0, 2000.0])) if kind == "poisson" else 0.0,
                       i_ext=float(rng.choice([0.0, 0.2])) if kind == "hh" else 0.0)
            if kind == "izh":
                pop["abcd"] = netgen.izhikevich_params(rng, n, 0)
            pops.append(pop)
        for post, pop in enumerate(pops):
            if pop["kind"] == "poisson":
                continue
            for pre in rng.permutation(len(pops))[:rng.integers(0, 5)]:
                rp, ci = netgen.bernoulli_csr(rng, pops[pre]["n"], pop["n"], float(rng.choice([0.0, 0.02, 0.3, 1.0])))
                projs.append(dict(pre=int(pre), post=post, row_ptr=rp, col_idx=ci, g=netgen.uniform_weights(rng, ci.size, 0.02),
                                  e_rev=float(rng.choice([0.0, -92.0])), tau=float(rng.choice([1.0, 5.0])), stdp=None))
        instances.append(dict(g_scale=float(rng.choice([0.3, 1.0, 4.0])), seed=seed * 10 + i, pops=pops, projs=projs))
    return dict(dt=float(rng.choice([0.02, 0.1])), substeps=int(rng.choice([1, 2, 3, 5])), instances=instances)


@pytest.mark.parametrize("seed", range(16))
def test_mixed_networks(snn, seed):
    """All forms that a network can take, with voltages that run away and
    that are not numbers among them."""
    print(f"case: resident mixed {seed}", flush=True)
    spec = mixed(seed)
    rng = np.random.default_rng([seed, 10])
    state = {}
    for b, inst in enumerate(spec["instances"]):
        for p, pop in enumerate(inst["pops"]):
            if pop["kind"] == "hh":
                v = rng.uniform(-90.0, 40.0, pop["n"])
                odd = rng.random(pop["n"]) < 0.05
                v[odd] = rng.choice([250.0, -1500.0, 3e38, np.nan, -52.0, -25.0], odd.sum())
                state[b, p] = v

    recorded = [f"hh{k}" for k in range(5)] if seed % 2 else []

    def run(mode):
        net = snn.Network(spec, record_vbar=recorded)
        if mode:
            net.set_launch(**mode)
        for (b, p), v in state.items():
            net.set_state(b, p, snn.V, v)
        for n in (5, 40, 1, 33, 8, 2, 12):
            net.step(n)
        out = everything(net, spec) + ([net.vbar_sum(b, p) for b, p in state] if recorded else [])
        net.close()
        return out
    got = run(None)
    for mode in (dict(mode=0), dict(mode=2)):
        assert not differing(got, run(mode)), mode


def test_scales_of_many_projections(snn):
    """g_scale and weights of a batch of more projections than the second
    dimension of a grid holds, the last of them with the largest weight."""
    import torch
    print("case: many projections", flush=True)
    rp, ci = np.array([0, 1], np.int32), np.zeros(1, np.int32)
    pops = [dict(name=f"P{k}", kind="hh", n=1, rate_hz=0.0, i_ext=0.0) for k in range(8)]
    projs = [dict(pre=(p + k) % 8, post=p, row_ptr=rp, col_idx=ci, g=np.array([0.01], np.float32), e_rev=0.0, tau=1.0,
                  stdp=None) for p in range(8) for k in range(4)]
    last = [dict(q) for q in projs]
    last[-1]["g"] = np.array([2.0], np.float32)
    n = 65536 // len(projs) + 2
    spec = dict(dt=0.1, substeps=3, instances=[dict(g_scale=1.0, seed=i, pops=pops, projs=projs if i < n - 1 else last)
                                               for i in range(n)])
    net = snn.Network(spec)
    scales = np.ones(n, np.float32)
    net.set_gscale(scales)
    w = torch.empty(net.weight_count, dtype=torch.float32, device="cuda")
    net.get_weights_device(w)
    assert float(w[-1]) == 2.0
    net.set_weights_device(w)
    # a scale that only the last projection's weight makes too large
    scales[:] = 1e4
    scales[-1] = 1.0
    net.set_gscale(scales)
    scales[-1] = 1e4
    with pytest.raises(snn.SNNError) as e:
        net.set_gscale(scales)
    assert e.value.code == snn.SNN_ERANGE
    net.step(3)
    net.close()
