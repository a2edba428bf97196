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
