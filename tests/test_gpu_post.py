"""The workgroups of a post launch against the oracle: the energy statistics,
those of M~ and the digest where they are asked for, then the weight blocks of
the resampling or the whole resampling of a small population."""
import numpy as np
import pytest

import oracle
import paper_1704_01888_amd as pa
from paper_1704_01888_amd.workloads import linear_betas

pytestmark = pytest.mark.gpu

OUTPUTS = [0, pa.OUT_MAG, pa.OUT_DIGEST, pa.OUT_MAG | pa.OUT_DIGEST | pa.OUT_HIST | pa.OUT_WIDTHS]
KEYS = ("R_i", "E_sum", "final_spins", "final_E", "last_anc", "hist", "Mt_sum", "mhist", "digest")


@pytest.fixture(scope="module")
def ctx():
    c = pa.Context(0)
    yield c
    c.close()


def _compare(got, want):
    for key in KEYS:
        if key in got and key in want:
            assert (np.asarray(got[key]) == np.asarray(want[key])).all(), key
    np.testing.assert_allclose(got["minus_beta_F"], want["minus_beta_F"], rtol=1e-12)
    for key in ("width_e", "width_m"):
        if key in got:
            np.testing.assert_allclose(got[key], want[key], rtol=1e-12)


def _oracle(kw, outs):
    return oracle.run(oracle.Desc(**kw), final=True, hist=bool(outs & pa.OUT_HIST),
                      magnetisation=bool(outs & pa.OUT_MAG), digest=bool(outs & pa.OUT_DIGEST),
                      widths=bool(outs & pa.OUT_WIDTHS))


@pytest.mark.parametrize("resample", [pa.RESAMPLE_MULTINOMIAL, pa.RESAMPLE_POISSON, pa.RESAMPLE_NONE])
@pytest.mark.parametrize("R", [7, 1000, 5000])
def test_outputs_of_a_post_launch(ctx, R, resample):
    runs = [dict(L=12, q=5, R=R + n, beta=linear_betas(1.3, 5), theta=1, seed=90 + n, resample=resample)
            for n in range(len(OUTPUTS))]
    want = [_oracle(kw, outs) for kw, outs in zip(runs, OUTPUTS)]
    for kw, outs, w in zip(runs, OUTPUTS, want):
        print(f"\nR={kw['R']} outputs={outs} resample={resample}", flush=True)
        _compare(pa.pa_run(ctx, pa.Desc(outputs=outs | pa.OUT_FINAL, **kw)), w)
    got = pa.pa_run_batch(ctx, [pa.Desc(outputs=o | pa.OUT_FINAL, **kw) for kw, o in zip(runs, OUTPUTS)])
    for g, w in zip(got, want):
        _compare(g, w)


LARGE = [
    # Poisson populations on both sides of the size from which the post and count
    # launches work from block histograms and sums (65536); one block of one replica
    dict(L=8, q=4, R=65536, beta=linear_betas(1.2, 12), theta=1, seed=5, resample=0),
    dict(L=4, q=3, R=65537, beta=linear_betas(1.2, 3), theta=1, seed=6, resample=1),
    # equal weights (a repeated beta), strongly skewed ones, and none
    dict(L=8, q=3, R=70001, beta=np.array([0.0, 0.0, 0.5, 1.5, 3.0]), theta=1, seed=7, resample=1),
    dict(L=8, q=3, R=70001, beta=linear_betas(1.2, 3), theta=1, seed=8, resample=2),
    # heating from ground states: one level at first, weights from the largest energy
    dict(L=12, q=6, R=80002, beta=np.array([1.6, 1.3, 1.0, 0.7]), theta=1, seed=9, resample=1, init=pa.INIT_GROUND),
    # the largest side whose blocks fit the scratch, and the next
    dict(L=44, q=10, R=66000, beta=linear_betas(0.9, 2), theta=1, seed=10, resample=0),
    dict(L=46, q=10, R=66000, beta=linear_betas(0.9, 2), theta=1, seed=11, resample=0),
    # several rows a block
    dict(L=8, q=5, R=270003, beta=linear_betas(1.4, 3), theta=1, seed=12, resample=0),
]


@pytest.mark.parametrize("kw", LARGE, ids=lambda c: f"L{c['L']}R{c['R']}r{c['resample']}")
def test_populations_with_block_histograms(ctx, kw):
    outs = OUTPUTS[-1]
    print(f"\nL={kw['L']} q={kw['q']} R={kw['R']} resample={kw['resample']}", flush=True)
    want = _oracle(kw, outs)
    _compare(pa.pa_run(ctx, pa.Desc(outputs=outs | pa.OUT_FINAL, **kw)), want)
    if kw["R"] == 65536:
        assert (want["R_i"] > 65536).any() and (want["R_i"] <= 65536).any()


@pytest.mark.parametrize("R", [1, 2, 3, 5, 33, 34, 2999, 3500])
def test_small_resampling_with_skewed_weights(ctx, R):
    """Draws outside the search window; populations that fill no load of four."""
    kw = dict(L=8, q=3, R=R, beta=np.array([0.0, 0.0, 0.5, 1.5, 3.0, 2.0]), theta=1, seed=70 + R, resample=1)
    print(f"\nR={R}", flush=True)
    _compare(pa.pa_run(ctx, pa.Desc(outputs=OUTPUTS[-1] | pa.OUT_FINAL, **kw)), _oracle(kw, OUTPUTS[-1]))


@pytest.mark.parametrize("L", [8, 64])
def test_small_resampling_in_a_batch(ctx, L):
    """Populations of every remainder of a load of four, each run with a record
    of its own in one post launch."""
    runs = [dict(L=L, q=3, R=R, beta=np.array([0.0, 0.0, 0.5, 1.5, 3.0, 2.0]), theta=1, seed=170 + R, resample=R % 2)
            for R in ((5, 62, 63, 64, 65, 1021, 1024, 2047, 4093, 4094, 4095, 4096) if L == 8 else (30, 31, 33, 200))]
    print(f"\nL={L}", flush=True)
    got = pa.pa_run_batch(ctx, [pa.Desc(outputs=OUTPUTS[-1] | pa.OUT_FINAL, **kw) for kw in runs])
    for g, kw in zip(got, runs):
        _compare(g, _oracle(kw, OUTPUTS[-1]))
