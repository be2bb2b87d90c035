"""GPU parity of the VB sweep that streams its adjacency, where its plan changes.

A chunk is two blocks of 64 positions of one class; chunks of one degree take their
rows from the first one and read exactly as many words as neighbours, others mask
the lanes past their degree, and rows longer than 8 go on four entries at a time
(with 8 chain slots in bytes past 15).  All quantities are integers and equal the
oracle's exactly, with and without the complemented copy, split or not."""
import numpy as np
import pytest

import paper_1906_11195_amd as sg
from tests.gpu_util import assert_instance_equal, oracle_vb, require_gpu

pytestmark = pytest.mark.gpu

FLAGS = sg.MEASURE_OBS | sg.MEASURE_SPINS


def graph(n, degree, seed):
    """A regular part (ring with second neighbours: even chunks), isolated vertices
    and a few hubs of the given degree."""
    rng = np.random.default_rng(seed)
    m = n - 500
    edges = {(i, i + d) for i in range(3, m - 2) for d in (1, 2)}
    for hub in (0, 1, 2):
        for v in rng.choice(np.arange(3, m), size=degree, replace=False):
            edges.add((hub, int(v)))
    e = np.array(sorted(edges), np.int32)
    return e, rng.choice([-1, 1], size=len(e)).astype(np.int8)


@pytest.mark.parametrize("replicas", [1, 2, 4, 6])
@pytest.mark.parametrize("degree", [7, 8, 9, 12, 13, 15, 16, 63])
def test_streamed_degrees(degree, replicas):
    require_gpu()
    n = 20011
    edges, J = graph(n, degree, degree)
    d = sg.VbDesc(n=n, T=0.9, seed=41, instance_id=degree, edges=edges, J=J, n_replicas=replicas)
    ref = oracle_vb(d, 7, 4)
    for kw in ({}, {"plain_lds": True}, {"split_members": 3}, {"threads_per_unit": 128}):
        ctx = sg.sg_create_vb([d], t_max=4, **kw)
        sg.sg_sweep(ctx, 3)
        sg.sg_sweep(ctx, 4)
        res = sg.sg_measure(ctx, FLAGS)
        sg.sg_free(ctx)
        assert_instance_equal(res, 0, ref, label="degree %d %s" % (degree, kw))
