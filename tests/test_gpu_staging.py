"""Measurements larger than the largest block of mapped host memory (64 MiB): the
words come over in pieces, they are the same, and no other context's work is waited
for."""
import numpy as np
import pytest
import torch

import paper_1906_11195_amd as sg
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

N, R, COUNT = 1000003, 8, 68     # 544 chains of 125 KB


@pytest.fixture
def large():
    require_gpu()
    ctx = sg.sg_create_vb([sg.VbDesc(n=N, T=0.8, seed=5, instance_id=i, graph_id=1, c=2.0, n_replicas=R)
                           for i in range(COUNT)], t_max=0, split_members=1)
    yield ctx
    sg.sg_free(ctx)


def test_spins_past_the_pool_equal_the_overlaps(large):
    res = sg.sg_measure(large, sg.MEASURE_OBS | sg.MEASURE_SPINS)
    pairs = [(a, b) for a in range(R) for b in range(a + 1, R)]
    for i in range(COUNT):
        s = res["spins"][i]
        assert np.abs(s).min() == 1
        for a in range(0, R, 2):      # every row once
            q = int((s[a] == s[a + 1]).sum()) * 2 - N
            assert q == res["overlap"][i, pairs.index((a, a + 1)), 0], (i, a)
    again = sg.sg_measure(large, sg.MEASURE_SPINS)
    assert all(np.array_equal(a, b) for a, b in zip(res["spins"], again["spins"]))


def test_no_other_context_is_waited_for(large):
    sg.sg_measure(large, sg.MEASURE_SPINS)
    busy = sg.sg_create_vb([sg.VbDesc(n=1024, T=0.8, seed=6, instance_id=0)], t_max=0)
    try:
        side, done = torch.cuda.Stream(), torch.cuda.Event()
        sg.sg_sweep(busy, 1 << 20, stream=side)      # two seconds and more
        done.record(side)
        sg.sg_measure(large, sg.MEASURE_SPINS)
        assert not done.query()
    finally:
        sg.sg_free(busy)


def _vb():
    return sg.sg_create_vb([sg.VbDesc(n=200000, T=0.9, seed=7, instance_id=0)], t_max=0)


def _multispin():
    return sg.sg_create_vb([sg.VbDesc(n=8192, T=0.9, seed=8, instance_id=i, n_replicas=8) for i in range(2)], t_max=0,
                           multispin=True)


def _sk():
    return sg.sg_create_sk([sg.SkDesc(n=2048, T=0.7, seed=9, instance_id=0)], t_max=0)


@pytest.mark.parametrize("create", [_vb, _multispin, _sk])
@pytest.mark.parametrize("sweeps_aside", [False, True])
def test_spins_after_sweeps_on_another_stream(create, sweeps_aside):
    require_gpu()
    side, ref, ctx = torch.cuda.Stream(), create(), create()
    try:
        sg.sg_sweep(ref, 3000)
        want = sg.sg_measure(ref, sg.MEASURE_SPINS)["spins"]
        sg.sg_sweep(ctx, 3000, stream=side if sweeps_aside else None)
        got = sg.sg_measure(ctx, sg.MEASURE_SPINS, stream=None if sweeps_aside else side)["spins"]
        assert all(np.array_equal(a, b) for a, b in zip(want, got))
    finally:
        sg.sg_free(ref)
        sg.sg_free(ctx)
