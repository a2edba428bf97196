"""Batches whose runs of one lattice side take different sweep kernels (q up to 16,
up to 32, above): small launches are joined in one, large ones stay apart; every
run equals the oracle's either way."""
import time

import numpy as np
import pytest
import torch

import oracle
import paper_1704_01888_amd as pa
from paper_1704_01888_amd.workloads import linear_betas

pytestmark = pytest.mark.gpu

ALL = pa.OUT_FINAL | pa.OUT_HIST | pa.OUT_MAG | pa.OUT_DIGEST
KEYS = ("R_i", "final_spins", "final_E", "last_anc", "hist", "Mt_sum", "mhist", "digest")


@pytest.fixture(scope="module")
def ctx():
    c = pa.Context(0)
    yield c
    c.close()


def _check(ctx, runs, outputs):
    got = pa.pa_run_batch(ctx, [pa.Desc(outputs=outputs, **r) for r in runs])
    for r, g in zip(runs, got):
        want = oracle.run(oracle.Desc(**r), final=True, hist=True, magnetisation=True, digest=True)
        for key in KEYS:
            if key in g:
                assert (g[key] == want[key]).all(), (key, r["L"], r["q"], r["R"])


# populations on both sides of the join with the byte kernel (1024 waves at 10 and
# 50), the generic one (2048 at 36 and 100) and the table's (20480)
SIZES = [(10, 21), (10, 1101), (50, 9), (36, 25), (36, 2100), (100, 3), (8, 300), (12, 60), (16, 70), (24, 40), (32, 20),
         (64, 5), (64, 2100), (128, 3), (256, 2)]


@pytest.mark.parametrize("L,R", SIZES, ids=lambda v: str(v))
def test_runs_of_three_kernels_in_one_batch(ctx, L, R):
    small = L * L * R < 200000
    qs = (8, 20, 40, 200, 33, 16, 17, 32) if small else (8, 20, 40)
    runs = [dict(L=L, q=q, R=R + n, beta=linear_betas(1.4, 3 if small else 1), theta=2 if small else 1, seed=600 + q + L,
                 resample=1) for n, q in enumerate(qs)]
    print(f"\nL={L} R={R}", flush=True)
    _check(ctx, runs, ALL)
    if small:
        # only some runs count states; 64-bit thresholds in some steps; both
        # quad forms without a run of another kernel
        runs[0]["beta"] = linear_betas(6.0, 3)
        _check(ctx, [runs[n] for n in (0, 1, 2, 7)], pa.OUT_FINAL | pa.OUT_HIST)
        _check(ctx, [runs[n] for n in (1, 5, 6, 7)], ALL)


@pytest.mark.parametrize("L,R", [(64, 61), (36, 48), (50, 50), (128, 30)])
def test_a_small_mixed_batch_takes_the_time_of_one_kernel(ctx, L, R):
    """Twelve runs with q = 8, 20 and 40 against the same with q = 40 alone, which
    was the time of both when one kernel swept all of them; in a launch per
    kernel 1.3 to 1.6 times it."""
    def descs(qs):
        return [pa.Desc(L=L, q=qs[i % len(qs)], R=R + i, beta=np.linspace(0.0, 1.0, 17), theta=10, seed=7 + i, resample=1)
                for i in range(12)]

    one, mixed = descs((40,)), descs((8, 20, 40))
    ws = torch.empty(max(pa.pa_plan_batch(one), pa.pa_plan_batch(mixed)), dtype=torch.uint8, device="cuda:0")
    best = [1e9, 1e9]
    for _ in range(12):
        for k, d in enumerate((one, mixed)):
            torch.cuda.synchronize()
            t = time.perf_counter()
            pa.pa_run_batch(ctx, d, workspace=ws)
            best[k] = min(best[k], time.perf_counter() - t)
    print(f"\nL={L} R={R}: {best[0] * 1e6:.0f} us, mixed {best[1] * 1e6:.0f} us", flush=True)
    assert best[1] < 1.2 * best[0]
