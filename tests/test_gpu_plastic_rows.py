"""Delivery and potentiation of a plastic network in one launch (rows and
grouped modes) against the two launches of tile mode, bit for bit, with
spikes on both sides of the plastic synapses at once."""
import numpy as np
import pytest

from paper_1412_0595_amd import netgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a,b,c", [(5, 7, 3), (40, 129, 65), (100, 1100, 64), (30, 900, 1030)])
@pytest.mark.parametrize("frac", [0.02, 0.5, 1.0])
def test_rows_of_spiking_pairs(a, b, c, frac):
    from paper_1412_0595_amd import snn
    print(f"case: plastic rows {a} {b} {c} {frac}", flush=True)
    rng = np.random.default_rng(4)
    spec = dict(dt=0.1, substeps=3, instances=[
        netgen.layered_instance(rng, a, b, c, rate_hz=80.0, p_ab=0.4, p_bc=0.5, seed=9, stdp_bc=True) for _ in range(2)])
    flags = [[(rng.random(n) < frac).astype(np.uint8) for n in (a, b, c)] for _ in range(3)]

    def run(**launch):
        net = snn.Network(spec)
        net.set_launch(**launch)
        out = []
        for f in flags:
            for i in range(2):
                for p in range(3):
                    net.set_last_spikes(i, p, f[p])
            net.step(1)
            out += [net.conductance(i, q) for i in range(2) for q in range(3)]
            net.step(20)
        out += [net.weights(i, 1) for i in range(2)] + [net.state(i, p, v) for i in range(2) for p in (1, 2) for v in range(4)]
        net.close()
        return out
    ref = run(mode=1)
    for launch in (dict(mode=0), dict(mode=0, prop_blocks=1, prop_block=64, chunk=64), dict(mode=3)):
        got = run(**launch)
        assert all(np.array_equal(x, y) for x, y in zip(ref, got)), launch
