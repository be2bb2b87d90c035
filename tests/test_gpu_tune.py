"""Autotuned contexts after one another in a process: a workgroup size found for one is
not taken for another that it does not fit.  Resident units of one octave of sizes and
one planned size, whose entries fill the LDS or leave room for twice the wavefronts."""
import numpy as np
import pytest

import paper_1906_11195_amd as sg
from tests.gpu_util import assert_instance_equal, oracle_vb, require_gpu

pytestmark = pytest.mark.gpu


def run(descs, **kw):
    ctx = sg.sg_create_vb(descs, t_max=16, **kw)
    try:
        sg.sg_sweep(ctx, 20)
        return sg.sg_measure(ctx, sg.MEASURE_OBS | sg.MEASURE_SPINS)
    finally:
        sg.sg_free(ctx)


def test_sizes_kept_for_other_groups():
    require_gpu()
    many = [sg.VbDesc(n=2500, T=0.8, seed=11, instance_id=i, graph_id=i, c=4.0) for i in range(300)]
    run(many, autotune=True)
    for n, c in [(3850, 8.0), (3700, 8.0), (2100, 16.0), (3900, 7.5), (4090, 6.0)]:
        few = [sg.VbDesc(n=n, T=0.9, seed=12, instance_id=0, graph_id=0, c=c)]
        assert_instance_equal(run(few, autotune=True), 0, oracle_vb(few[0], 20, 16), label="n=%d c=%g" % (n, c))
    a, b = run(many, autotune=True), run(many)
    for key in ("bond", "gram", "overlap", "accepted"):
        assert np.array_equal(a[key], b[key]), key
