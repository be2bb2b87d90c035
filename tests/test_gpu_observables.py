"""GPU parity of the Gram and overlap counts where their plan changes.

Rows of a set are staged in tiles of at most 8192 words together: more rows mean
shorter tiles, more words several tiles (added atomically); rows whose length is
no multiple of 16 bytes are staged word by word; the last word ends inside.  The
sums are integers and equal the oracle's exactly."""
import numpy as np
import pytest

import paper_1906_11195_amd as sg
from tests.gpu_util import assert_instance_equal, oracle_vb, require_gpu

pytestmark = pytest.mark.gpu


def check(descs, sweeps, t_max):
    ctx = sg.sg_create_vb(descs, t_max=t_max)
    try:
        for part in (sweeps - sweeps // 3, sweeps // 3):   # the counts are clear again after a measurement
            sg.sg_sweep(ctx, part)
            res = sg.sg_measure(ctx, sg.MEASURE_OBS | sg.MEASURE_SPINS)
    finally:
        sg.sg_free(ctx)
    for i, d in enumerate(descs):
        ref = oracle_vb(d, sweeps, t_max)
        if len(descs) == 1:
            assert_instance_equal(res, i, ref, label="n=%d" % d.n)
        else:
            for key in ("bond", "gram", "overlap", "accepted"):
                assert np.array_equal(res[key][i], ref[key]), (i, key)


@pytest.mark.parametrize("replicas", [1, 2, 3, 8])
@pytest.mark.parametrize("n", [5, 64, 1000, 32768, 65568, 131071])
def test_words_and_replicas(n, replicas):
    require_gpu()
    d = sg.VbDesc(n=n, T=0.9, seed=31, instance_id=n, graph_id=2, c=1.0 if n < 8 else 3.0, n_replicas=replicas)
    check([d], 9, 1 << 12)


def test_many_times():
    require_gpu()
    check([sg.VbDesc(n=33, T=1.5, seed=32, instance_id=1, graph_id=3, c=3.0, n_replicas=2)], 1 << 18, 1 << 30)


def test_sets_of_different_length():
    require_gpu()
    check([sg.VbDesc(n=n, T=0.8, seed=33, instance_id=i, graph_id=i, c=2.0, n_replicas=3)
           for i, n in enumerate([9, 40000, 257, 90001])], 5, 8)
