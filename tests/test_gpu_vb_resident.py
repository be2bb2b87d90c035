"""GPU parity of the LDS-resident VB sweep where its plan changes.

A chunk of 64 positions reads 4, 8, 12 or 15 neighbours, or rows of any length
past that, by its largest degree; the wavefronts are dealt the chunks of a whole
sweep and their number follows the chunks and the units that a CU holds.  All
quantities are integers and equal the oracle's exactly."""
import numpy as np
import pytest

import paper_1906_11195_amd as sg
from tests.gpu_util import assert_instance_equal, oracle_vb, require_gpu

pytestmark = pytest.mark.gpu

FLAGS = sg.MEASURE_OBS | sg.MEASURE_SPINS


def graph(n, degree, seed):
    """Ring with some chords (degrees 2 and 3) and two hubs of the given degree."""
    rng = np.random.default_rng(seed)
    edges = {(i, i + 1) for i in range(2, n - 1)}
    for i in range(2, n - 40, 5):
        edges.add((i, i + int(rng.integers(2, 5)) * 5 + 1))
    for hub in (0, 1):
        for v in rng.choice(np.arange(2, n), size=degree, replace=False):
            edges.add((hub, int(v)))
    e = np.array(sorted(edges), np.int32)
    return e, rng.choice([-1, 1], size=len(e)).astype(np.int8)


@pytest.mark.parametrize("replicas", [1, 2, 3, 5, 8])
@pytest.mark.parametrize("degree", [4, 5, 8, 9, 12, 13, 15, 16, 63])
def test_resident_degrees(degree, replicas):
    require_gpu()
    n = 333
    edges, J = graph(n, degree, degree)
    d = sg.VbDesc(n=n, T=0.9, seed=21, instance_id=degree, edges=edges, J=J, n_replicas=replicas)
    for threads in (0, 64, 1024):
        ctx = sg.sg_create_vb([d], t_max=32, threads_per_unit=threads)
        sg.sg_sweep(ctx, 7)
        sg.sg_sweep(ctx, 33)
        res = sg.sg_measure(ctx, FLAGS)
        sg.sg_free(ctx)
        assert_instance_equal(res, 0, oracle_vb(d, 40, 32), label="degree %d threads %d" % (degree, threads))


@pytest.mark.parametrize("count", [1, 300, 1100])
def test_resident_units_sharing_a_cu(count):
    require_gpu()
    descs = [sg.VbDesc(n=64 + 37 * (i % 29), T=0.7, seed=22, instance_id=i, graph_id=i, c=4.0) for i in range(count)]
    ctx = sg.sg_create_vb(descs, t_max=16)
    sg.sg_sweep(ctx, 20)
    res = sg.sg_measure(ctx, FLAGS)
    sg.sg_free(ctx)
    for i in {0, count // 2, count - 1}:
        n = descs[i].n
        ref = oracle_vb(descs[i], 20, 16)
        assert np.array_equal(res["accepted"][i], ref["accepted"]), i
        assert np.array_equal(res["gram"][i], ref["gram"]), i
        assert np.array_equal(np.asarray(res["spins"][i])[:, :n], ref["spins"]), i
