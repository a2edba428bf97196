"""Populations loaded from host memory (pa_run_load): the look for states of q or
more, after which the run keeps the kernels that take any state."""
import time

import numpy as np
import pytest
import torch

import oracle
import paper_1704_01888_amd as pa
from paper_1704_01888_amd.workloads import linear_betas

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = pa.Context(0)
    yield c
    c.close()


# bytes of the population: 100, 300 (a tail after the 16-byte loads), 65536, and
# a lattice of the tiled path
@pytest.mark.parametrize("L,R", [(10, 1), (10, 3), (32, 64), (264, 2)])
@pytest.mark.parametrize("q,state", [(4, None), (4, 4), (4, 100), (4, 127), (2, 2), (32, 32), (32, 127)])
def test_one_state_of_q_or_more(ctx, L, R, q, state):
    """Nowhere, or at the first, a middle or the last site."""
    kw = dict(L=L, q=q, R=R, beta=linear_betas(1.0, 3), theta=2, seed=9, resample=2)
    n = R * L * L
    for at in (0, n // 2 + 1, n - 1):
        spins = np.random.default_rng(at).integers(0, q, size=(R, L * L), dtype=np.uint8)
        if state is not None:
            spins.reshape(-1)[at] = state
        print(f"\nL={L} R={R} q={q} state={state} at={at}", flush=True)
        run = pa.Run(ctx, pa.Desc(**kw))
        run.load(1, spins, 0.0)
        run.advance(1)
        got = run.read()
        run.finish()
        od = oracle.Desc(**kw)
        for j in range(R):
            assert (got["spins"][j] == oracle.sweep_replica(od, 2, j, spins[j])).all(), j
        if state is None:
            break


def test_a_load_takes_little_more_than_its_upload(ctx):
    """Nothing reads the whole population on the host: 328 MB of 128x128 replicas
    load in the time of their copy to the device (10.8 ms; 18.2 with such a read)."""
    R, N = 20000, 128 * 128
    run = pa.Run(ctx, pa.Desc(L=128, q=10, R=R, beta=linear_betas(1.0, 2), theta=1, seed=1, resample=1))
    spins = np.random.default_rng(0).integers(0, 10, size=(R, N), dtype=np.uint8)
    host, dev = torch.from_numpy(spins), torch.empty((R, N), dtype=torch.uint8, device="cuda:0")
    load, copy = [], []
    for _ in range(8):
        t = time.perf_counter()
        run.load(0, spins, 0.0)
        load.append(time.perf_counter() - t)
        t = time.perf_counter()
        dev.copy_(host)
        torch.cuda.synchronize()
        copy.append(time.perf_counter() - t)
    run.finish()
    print(f"\nload {min(load) * 1e3:.1f} ms, copy {min(copy) * 1e3:.1f} ms", flush=True)
    assert min(load) < 1.4 * min(copy) + 1e-3
