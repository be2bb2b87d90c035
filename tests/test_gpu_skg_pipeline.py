"""GPU parity of the Gaussian SK sweep at the sizes where its plan changes: 13
updater wavefronts hold items of 64, 128 or 256 fields (N <= 832, <= 1664, above),
1 to 5 items each (3328 fields per item); rows are padded to 256 floats.  Spins,
counts, overlaps and Grams equal the oracle's; real bond sums within 1e-9 (about
N^2 / 2 double additions of terms below 1 in another order)."""
import numpy as np
import pytest

import oracle
import paper_1906_11195_amd as sg
from paper_1906_11195_amd.workloads import gaussian_couplings
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

FLAGS = sg.MEASURE_OBS | sg.MEASURE_SPINS


def check(descs, sweeps, t_max):
    ctx = sg.sg_create_sk(descs, t_max=t_max)
    try:
        sg.sg_sweep(ctx, sweeps)
        res = sg.sg_measure(ctx, FLAGS)
    finally:
        sg.sg_free(ctx)
    for i, d in enumerate(descs):
        ref = oracle.skg_run(d.n, d.Jf, d.T, d.seed, d.instance_id, d.n_replicas, sweeps, t_max,
                             period=d.recompute_period, start=d.start, s0=d.s0)
        for key in ("spins", "accepted", "gram", "overlap"):
            assert np.array_equal(res[key][i], ref[key]), "n=%d %s" % (d.n, key)
        assert np.abs(res["bond_real"][i][:, :len(ref["times"])] - ref["bond"]).max() < 1e-9, "n=%d bond" % d.n


@pytest.mark.parametrize("n", [128, 129, 256, 257, 831, 832, 833, 1663, 1664, 1665, 3328, 3329, 6656, 6657, 9984,
                               9985, 13313])
def test_skg_variant_edges(n):
    require_gpu()
    check([sg.SkDesc(n=n, T=0.5, seed=21, instance_id=1, Jf=gaussian_couplings(n, seed=n), recompute_period=3)],
          7 if n < 5000 else 2, 8)


def test_skg_mixed_sizes_in_one_context():
    require_gpu()
    check([sg.SkDesc(n=n, T=0.3 + 0.1 * i, seed=22, instance_id=i, n_replicas=3, Jf=gaussian_couplings(n, seed=n + 7),
                     recompute_period=4) for i, n in enumerate((3, 64, 900, 130, 4000, 2049))], 9, 8)


def test_skg_matrices_of_a_large_context():
    """Couplings that go up in several pieces, rows of several matrices in one piece
    among them: the energies of the start configurations, in 64 bits (n terms of
    variance 1 / n and their sums: rounding far below 1e-9)."""
    require_gpu()
    sizes = [1021, 64, 1021, 1021, 300, 1024, 300, 1021, 63, 1021, 2, 1000]
    descs = []
    for i, n in enumerate(sizes):
        z = np.triu(np.random.default_rng(40 + i).standard_normal((n, n)), 1) / np.sqrt(n)
        Jf = (z + z.T).astype(np.float32)
        descs.append(sg.SkDesc(n=n, T=0.5, seed=14, instance_id=i, n_replicas=2, Jf=Jf))
    ctx = sg.sg_create_sk(descs, t_max=0)
    try:
        res = sg.sg_measure(ctx, sg.MEASURE_OBS | sg.MEASURE_SPINS)
    finally:
        sg.sg_free(ctx)
    for i, d in enumerate(descs):
        for r in range(2):
            s = res["spins"][i][r].astype(np.float64)
            want = 0.5 * s @ (d.Jf.astype(np.float64) @ s)
            assert abs(res["bond_real"][i, r, 0] - want) < 1e-9, (i, r)
