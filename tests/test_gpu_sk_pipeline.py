"""GPU parity of the SK sweep pipeline at the sizes where its plan changes.

A block is 64 spins and the number of blocks is even; twelve updater wavefronts
hold one field per lane and block, in variants for 1 .. 8, 12, 16, 24, 32 and 48
blocks per wavefront (768 spins per step of 1).  Trajectories, counts and
observables are integers and equal the oracle's exactly."""
import pytest

import paper_1906_11195_amd as sg
from tests.gpu_util import assert_instance_equal, oracle_sk, require_gpu

pytestmark = pytest.mark.gpu

FLAGS = sg.MEASURE_OBS | sg.MEASURE_SPINS


def run_lib(descs, n_sweeps, t_max):
    ctx = sg.sg_create_sk(descs, t_max=t_max)
    try:
        sg.sg_sweep(ctx, n_sweeps)
        return sg.sg_measure(ctx, FLAGS)
    finally:
        sg.sg_free(ctx)


@pytest.mark.parametrize("n", [64, 127, 128, 129, 193, 257, 767, 768, 769, 1537, 2305, 3073, 3841, 4609, 5377, 6144,
                               6145, 9216, 9217, 12289, 18433, 24577])
def test_sk_variant_edges(n):
    require_gpu()
    sweeps = 12 if n < 8000 else 3
    d = sg.SkDesc(n=n, T=0.5, seed=11, instance_id=2, graph_id=n, recompute_period=5)
    res = run_lib([d], sweeps, 8)
    assert_instance_equal(res, 0, oracle_sk(d, sweeps, 8), label="n=%d" % n)


def test_sk_mixed_sizes_in_one_context():
    # the variant is chosen for the largest chain; the smaller ones leave most of
    # its slots unused
    require_gpu()
    descs = [sg.SkDesc(n=n, T=0.3 + 0.1 * i, seed=12, instance_id=i, graph_id=i, n_replicas=3, recompute_period=7)
             for i, n in enumerate((3, 64, 700, 130, 5000, 2049, 7000))]
    res = run_lib(descs, 15, 16)
    for i, d in enumerate(descs):
        assert_instance_equal(res, i, oracle_sk(d, 15, 16), label="n=%d" % d.n)
