"""The quad sweep kernel (q <= 32, four sites of one colour per dword) against
the oracle, bit for bit: every shape it has, populations that leave the last
lane group and workgroup partly idle, one and several replicas per lane, the
edges of its q range (16, 17, 32 and, on the dword kernel, 33), steps whose
thresholds need 64 bits in the middle of a run, and populations loaded with
spins beyond its range."""
import numpy as np
import pytest

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


def _check(ctx, **kw):
    want = oracle.run(oracle.Desc(**kw), final=True, hist=True, magnetisation=True, digest=True)
    got = pa.pa_run(ctx, pa.Desc(outputs=ALL, **kw))
    for key in KEYS:
        assert (got[key] == want[key]).all(), key
    np.testing.assert_allclose(got["minus_beta_F"], want["minus_beta_F"], rtol=1e-12)


# (L, lanes, waves per workgroup), replicas per lane in the larger population
SHAPES = [(8, 8, 1), (8, 8, 4), (16, 32, 2), (16, 32, 16), (24, 24, 12), (32, 128, 2), (32, 128, 8), (48, 96, 12),
          (64, 512, 8), (96, 384, 6), (96, 384, 12), (128, 512, 8), (128, 1024, 16), (192, 768, 12), (256, 1024, 16)]


@pytest.mark.parametrize("L,G,w", SHAPES, ids=lambda v: str(v))
def test_every_quad_shape_matches_the_oracle(ctx, L, G, w):
    for r_class in range(4):
        ctx.tune_set(L, 0, r_class, G, w)
    small = max(3, 40000 // (L * L)) | 1
    for n, q in enumerate((16, 17, 32, 2)):
        print(f"\nL={L} lanes={G} waves={w} q={q} R={small + n}", flush=True)
        _check(ctx, L=L, q=q, R=small + n, beta=linear_betas(1.7, 3), theta=2, seed=L + q, resample=0)


@pytest.mark.parametrize("L,G,w,R", [(8, 8, 2, 131077), (16, 32, 2, 32771), (24, 24, 12, 21851), (32, 128, 2, 8195),
                                     (48, 96, 12, 5463), (64, 512, 8, 2051), (96, 384, 12, 1367),
                                     (128, 1024, 16, 513)], ids=lambda v: str(v))
def test_several_replicas_per_lane_match_the_oracle(ctx, L, G, w, R):
    for r_class in range(4):
        ctx.tune_set(L, 0, r_class, G, w)
    for q in (10, 20):
        print(f"\nL={L} lanes={G} waves={w} q={q} R={R}", flush=True)
        _check(ctx, L=L, q=q, R=R, beta=linear_betas(0.02, 2), theta=2, seed=L + q, resample=1)


def test_steps_beyond_the_quad_kernel(ctx):
    """q = 33, and beta up to 6, where the dE = 4 threshold is zero: the dword
    kernels, also with a shape that only the quad kernel has."""
    for L, G, w in ((24, 24, 12), (96, 384, 12), (64, 512, 8)):
        for r_class in range(4):
            ctx.tune_set(L, 0, r_class, G, w)
        _check(ctx, L=L, q=33, R=21, beta=linear_betas(1.5, 3), theta=2, seed=5, resample=0)
        _check(ctx, L=L, q=8, R=21, beta=linear_betas(6.0, 4), theta=2, seed=6, resample=0)


def test_batch_of_quad_and_dword_runs(ctx):
    runs = [dict(L=32, q=q, R=R, beta=linear_betas(1.2, 4), theta=2, seed=40 + q, resample=1)
            for q, R in ((8, 5000), (10, 3001), (20, 700), (33, 300), (2, 1))]
    runs += [dict(L=64, q=8, R=1500, beta=linear_betas(1.2, 6), theta=1, seed=50, resample=1),
             dict(L=64, q=5, R=1501, beta=linear_betas(6.0, 5), theta=1, seed=51, resample=1)]
    got = pa.pa_run_batch(ctx, [pa.Desc(outputs=ALL, **r) for r in runs])
    for r, g in zip(runs, got):
        want = oracle.run(oracle.Desc(**r), final=True, hist=True, magnetisation=True, digest=True)
        for key in KEYS:
            assert (g[key] == want[key]).all(), (key, r["q"], r["R"])


def test_loaded_spins_beyond_q_keep_the_dword_kernel(ctx):
    """Spins that no proposal makes (q and above) are states like any other to
    the dword kernels, as before the quad kernel."""
    kw = dict(L=32, q=4, R=64, beta=linear_betas(1.0, 4), theta=3, seed=9, resample=2)
    rng = np.random.default_rng(1)
    spins = rng.integers(0, 120, size=(64, 1024), dtype=np.uint8)
    run = pa.Run(ctx, pa.Desc(**kw))
    run.load(1, spins, 0.0)
    run.advance(1)
    got = run.read()
    run.finish()
    od = oracle.Desc(**kw)
    for j in range(64):
        want = oracle.sweep_replica(od, 2, j, spins[j])
        assert (got["spins"][j] == want).all()


def _any_sides():
    """Sides from 8 on without lane choices (L = 10, 14, 18, 22, 26, 28, ...):
    a small one and a large one of every residue mod 8, and both ends."""
    return [10, 14, 18, 22, 26, 28, 36, 40, 44, 50, 62, 100, 108, 118, 136, 152, 178, 206, 228, 248, 252, 254]


@pytest.mark.parametrize("L", _any_sides())
def test_sides_without_lane_choices_match_the_oracle(ctx, L):
    """Whole and partly idle workgroups, and the smaller workgroups of a small
    launch; the byte and generic kernels of q = 33 on the same side."""
    assert ctx.get_lanes(L)[1] == []
    big = 1200 if L < 40 else max(3, 3000000 // (L * L))
    for q, R in ((3, 5), (16, big), (32, big | 1), (33, 7)):
        print(f"\nL={L} q={q} R={R}", flush=True)
        _check(ctx, L=L, q=q, R=R, beta=linear_betas(1.5, 2), theta=2, seed=L + q, resample=1)


def test_side_without_lane_choices_from_ground_states_to_64_bit_thresholds(ctx):
    for L in (18, 36, 50):
        _check(ctx, L=L, q=6, R=40, beta=np.array([6.0, 5.0, 1.2, 0.8]), theta=2, seed=3, resample=1, init=1)


@pytest.mark.parametrize("L,R,theta", [(260, 5, 2), (264, 4, 3), (300, 3, 1), (308, 3, 2), (512, 3, 2), (1024, 2, 3),
                                       (1028, 2, 1), (2048, 2, 1), (4092, 1, 1), (4096, 1, 1)], ids=lambda v: str(v))
def test_tiled_quads_match_the_oracle(ctx, L, R, theta):
    """Rows of whole and half dwords per colour, ragged last tiles, one to three
    launches per step; with the bonds counted by the last launch (energies and
    spins only) and by the measuring pass (states and digests too)."""
    for q, outputs in ((16, pa.OUT_FINAL | pa.OUT_HIST), (17, ALL), (32, pa.OUT_FINAL | pa.OUT_HIST)):
        print(f"\nL={L} q={q} R={R} theta={theta}", flush=True)
        kw = dict(L=L, q=q, R=R, beta=linear_betas(1.6, 2 if L < 2000 else 1), theta=theta, seed=L + q, resample=1)
        got = pa.pa_run(ctx, pa.Desc(outputs=outputs, **kw))
        want = oracle.run(oracle.Desc(**kw), final=True, hist=True, magnetisation=True, digest=True)
        for key in KEYS:
            if key in got:
                assert (got[key] == want[key]).all(), key


def test_tiled_population_loaded_with_spins_beyond_q(ctx):
    kw = dict(L=264, q=3, R=3, beta=linear_betas(1.0, 4), theta=2, seed=9, resample=2)
    spins = np.random.default_rng(2).integers(0, 100, size=(3, 264 * 264), dtype=np.uint8)
    run = pa.Run(ctx, pa.Desc(**kw))
    run.load(1, spins, 0.0)
    run.advance(1)
    got = run.read()
    run.finish()
    od = oracle.Desc(**kw)
    for j in range(3):
        assert (got["spins"][j] == oracle.sweep_replica(od, 2, j, spins[j])).all()


@pytest.mark.parametrize("L,G,w,R", [(8, 8, 4, 131077), (16, 32, 4, 32771), (32, 128, 2, 9001), (64, 512, 8, 2601)],
                         ids=lambda v: str(v))
def test_launch_of_several_and_single_replicas_per_lane(ctx, L, G, w, R):
    """Populations above the share of a launch that is held one replica per
    lane, alone and as two runs of a batch (the second all single)."""
    for r_class in range(4):
        ctx.tune_set(L, 0, r_class, G, w)
    kw = dict(L=L, q=7, beta=linear_betas(0.05, 2), theta=2, resample=1)
    print(f"\nL={L} R={R}", flush=True)
    _check(ctx, R=R, seed=L, **kw)
    runs = [dict(R=R, seed=L + 1, **kw), dict(R=R // 2, seed=L + 2, **kw)]
    got = pa.pa_run_batch(ctx, [pa.Desc(outputs=ALL, **r) for r in runs])
    for r, g in zip(runs, got):
        want = oracle.run(oracle.Desc(**r), final=True, hist=True, magnetisation=True, digest=True)
        for key in KEYS:
            assert (g[key] == want[key]).all(), (key, r["R"])


def test_batch_takes_the_shape_of_its_replicas_together(ctx):
    """Small runs of one side in one batch sweep with the tuned shape of their
    total population: quad and dword runs, 64-bit thresholds in the middle, M~."""
    for L, one, many in ((8, (16, 2), (8, 4)), (24, (48, 3), (24, 12))):
        for r_class in range(4):
            ctx.tune_set(L, 0, r_class, *(many if r_class else one))
    runs = [dict(L=L, q=q, R=1001 + q, beta=linear_betas(b, 4), theta=2, seed=300 + q + L, resample=1)
            for L in (8, 24) for q, b in ((8, 1.2), (20, 1.2), (33, 1.2), (5, 6.0))]
    got = pa.pa_run_batch(ctx, [pa.Desc(outputs=ALL, **r) for r in runs])
    for r, g in zip(runs, got):
        want = oracle.run(oracle.Desc(**r), final=True, hist=True, magnetisation=True, digest=True)
        for key in KEYS:
            assert (g[key] == want[key]).all(), (key, r["L"], r["q"])
