"""Tuned sweep shapes (pa_tune, pa_tune_set / get, pa_tune_save / load).

Every shape a lattice side has (each lane count with a kernel, each number of
waves per workgroup that fits) gives the oracle's result bit for bit; the
tuner keeps a measured shape per (L, q class, population class); the cache
file round-trips and refuses shapes a side does not have; runs of one kernel
class with different tuned workgroup sizes share a batch correctly."""
import json

import numpy as np
import pytest

import oracle
import paper_1704_01888_amd as pa
from paper_1704_01888_amd.workloads import linear_betas

pytestmark = pytest.mark.gpu

KEYS = ("R_i", "E_sum", "hist", "final_spins", "final_E", "last_anc", "digest")


@pytest.fixture(scope="module")
def ctx():
    c = pa.Context(0)
    yield c
    c.close()


def _same(a, b):
    for k in KEYS:
        assert (a[k] == b[k]).all(), k
    np.testing.assert_allclose(a["minus_beta_F"], b["minus_beta_F"], rtol=1e-12, atol=0)


def _shapes(ctx, L):
    """Every (lanes, waves per workgroup) the library accepts for L."""
    lanes = {ctx.tune_get(L, 8, 300)["lanes"]}
    _, cands = ctx.get_lanes(L)
    lanes.update(c for c in cands if c)
    out = []
    for G in sorted(lanes):
        for w in range(1, 17):
            try:
                ctx.tune_set(L, 0, 0, G, w)
            except pa.PAError:
                continue
            out.append((G, w))
    return out


@pytest.mark.parametrize("L", [4, 6, 8, 12, 16, 20, 24, 32, 64])
def test_every_shape_matches_the_oracle(ctx, L):
    c = dict(L=L, q=8, R=300, beta=linear_betas(1.4, 5), theta=2, seed=60 + L, resample=0)
    want = oracle.run(oracle.Desc(**c), hist=True, final=True, digest=True)
    d = pa.Desc(outputs=pa.OUT_HIST | pa.OUT_FINAL | pa.OUT_DIGEST, **c)
    shapes = _shapes(ctx, L)
    assert len(shapes) >= 1
    print(f"\nL={L}: shapes {shapes}", flush=True)
    for G, w in shapes:
        ctx.tune_set(L, 0, 0, G, w)
        got_shape = ctx.tune_get(L, 8, 300)
        assert (got_shape["lanes"], got_shape["waves_per_block"]) == (G, w)
        _same(pa.pa_run(ctx, d), want)


def test_tune_keeps_the_fastest_shape_and_the_file_round_trips(ctx, tmp_path):
    a = ctx.tune(8, 8, 1000)
    b = ctx.tune(24, 10, 20000)
    print(f"\ntuned {a} {b}", flush=True)
    assert a["attempts_per_ns"] > 0 and b["attempts_per_ns"] > 0
    assert (a["r_class"], b["r_class"]) == (0, 2)
    for e, (L, q, R) in ((a, (8, 8, 1000)), (b, (24, 10, 20000))):
        g = ctx.tune_get(L, q, R)
        assert (g["lanes"], g["waves_per_block"]) == (e["lanes"], e["waves_per_block"])
    path = tmp_path / "tune.jsonl"
    ctx.tune_save(path)
    lines = [json.loads(ln) for ln in path.read_text().splitlines()]
    assert all(ln["arch"].startswith("gfx") for ln in lines)
    other = pa.Context(0)
    try:
        assert other.tune_load(path) == len(lines)
        for e, (L, q, R) in ((a, (8, 8, 1000)), (b, (24, 10, 20000))):
            g = other.tune_get(L, q, R)
            assert (g["lanes"], g["waves_per_block"]) == (e["lanes"], e["waves_per_block"])
        # another architecture's lines are skipped; a shape L does not have is refused
        foreign = dict(lines[0], arch="gfx000", L=16, lanes=64, waves_per_block=2)
        path2 = tmp_path / "foreign.jsonl"
        path2.write_text(json.dumps(foreign) + "\n")
        assert other.tune_load(path2) == 0
        bad = dict(lines[0], lanes=3)
        path3 = tmp_path / "bad.jsonl"
        path3.write_text(json.dumps(bad) + "\n")
        with pytest.raises(pa.PAError) as e:
            other.tune_load(path3)
        assert e.value.status == pa.PA_ERR_INVALID
        path4 = tmp_path / "garbled.jsonl"
        path4.write_text('{"arch": "gfx950", "L": 8\n')
        with pytest.raises(pa.PAError):
            other.tune_load(path4)
    finally:
        other.close()


@pytest.mark.parametrize("mode", ["segmented", "team"])
def test_one_class_with_two_tuned_workgroup_sizes_in_a_batch(ctx, mode):
    # 8x8 runs of population classes 0 and 1 with different waves per workgroup
    ctx.tune_set(8, 0, 0, 16, 1)
    ctx.tune_set(8, 0, 1, 16, 8)
    cases = [dict(L=8, q=8, R=500, beta=linear_betas(1.5, 20), theta=3, seed=70, resample=1),
             dict(L=8, q=8, R=3000, beta=linear_betas(1.5, 25), theta=3, seed=71, resample=0),
             dict(L=8, q=6, R=700, beta=linear_betas(1.2, 12), theta=2, seed=72, resample=0)]
    descs = [pa.Desc(outputs=pa.OUT_HIST | pa.OUT_FINAL | pa.OUT_DIGEST, **c) for c in cases]
    ctx.set_batch_mode(pa.BATCH_TEAM if mode == "team" else pa.BATCH_SEGMENTED)
    try:
        got = pa.pa_run_batch(ctx, descs)
        if mode == "team":
            assert ctx.batch_info() == (3, 2)        # one launch per workgroup size
    finally:
        ctx.set_batch_mode(pa.BATCH_SEGMENTED)
    for d, g in zip(descs, got):
        _same(g, pa.pa_run(ctx, d))


@pytest.fixture()
def plain():
    c = pa.Context(0, tune_cache=False)
    yield c
    c.close()


def _get(c, L, q, R):
    e = c.tune_get(L, q, R)
    return e["lanes"], e["waves_per_block"]


def test_the_kernel_classes_have_entries_of_their_own(plain):
    c = plain
    # without a dword entry: the quad class's shape, or the default where only
    # the quad kernel has it; q above 128 is apart
    c.tune_set(24, 0, 2, 48, 9)
    assert _get(c, 24, 40, 50000) == _get(c, 24, 8, 50000) == (48, 9)
    c.tune_set(24, 0, 2, 24, 12)
    assert _get(c, 24, 8, 50000) == (24, 12) and _get(c, 24, 32, 50000) == (24, 12)
    assert _get(c, 24, 33, 50000) == _get(c, 24, 128, 50000) == _get(c, 24, 129, 50000) == (48, 3)
    c.tune_set(24, 2, 2, 48, 12)
    assert _get(c, 24, 8, 50000) == (24, 12)
    assert _get(c, 24, 33, 50000) == _get(c, 24, 128, 50000) == (48, 12)
    assert _get(c, 24, 129, 50000) == (48, 3)
    # a later entry for every q up to 128 takes its place
    c.tune_set(24, 0, 2, 48, 6)
    assert _get(c, 24, 40, 50000) == _get(c, 24, 8, 50000) == (48, 6)
    # a side without lane choices: the dword kernel's shape above q = 32
    assert _get(c, 50, 8, 3000) != _get(c, 50, 40, 3000) == (64, 4)


@pytest.mark.parametrize("q_large", [1, 2])
@pytest.mark.parametrize("L,lanes,waves", [(24, 24, 12), (32, 128, 8), (64, 512, 16), (96, 384, 12)])
def test_other_classes_refuse_the_quad_kernels_own_shapes(plain, L, lanes, waves, q_large):
    with pytest.raises(pa.PAError) as e:
        plain.tune_set(L, q_large, 1, lanes, waves)
    assert e.value.status == pa.PA_ERR_INVALID
    plain.tune_set(L, 0, 1, lanes, waves)


def test_the_shipped_shapes_of_the_dword_kernel(ctx):
    """Where the two kernels' best shapes differ, each has its own."""
    c = pa.Context(0)
    try:
        assert _get(c, 24, 40, 8000) == _get(c, 24, 40, 50000) == (48, 12)
        assert _get(c, 128, 40, 50000) == (512, 8) and _get(c, 128, 10, 50000) == (1024, 16)
        assert _get(c, 32, 40, 8000) == (256, 4)
    finally:
        c.close()


def test_tuning_above_32_states_leaves_the_quad_class_alone(plain, tmp_path):
    plain.tune_set(32, 0, 1, 128, 4)
    e = plain.tune(32, 40, 4000)
    assert e["q_large"] == 2 and all((t["lanes"], t["waves_per_block"]) in ((256, 4), (128, 2)) for t in e["timed"])
    assert _get(plain, 32, 40, 4000) == (e["lanes"], e["waves_per_block"])
    assert _get(plain, 32, 8, 4000) == (128, 4)
    path = tmp_path / "classes.jsonl"
    plain.tune_save(path)
    other = pa.Context(0, tune_cache=False)
    try:
        assert other.tune_load(path) == 2
        assert _get(other, 32, 40, 4000) == (e["lanes"], e["waves_per_block"])
        assert _get(other, 32, 8, 4000) == (128, 4)
    finally:
        other.close()


def test_steps_of_both_kernels_with_an_entry_each(plain):
    """64-bit thresholds in the middle of a run, q on both sides of 32, alone,
    in a batch (the shape of all replicas together) and in team launches."""
    for r_class in range(4):
        for L, quad, dword in ((24, (24, 12), (48, 9)), (32, (128, 8), (256, 4)), (64, (512, 8), (1024, 16))):
            plain.tune_set(L, 0, r_class, *quad)
            plain.tune_set(L, 2, r_class, *dword)
    runs = [dict(L=L, q=q, R=R, beta=linear_betas(b, 4), theta=2, seed=500 + q + L, resample=1)
            for L, R in ((24, 1500), (32, 900), (64, 300)) for q, b in ((10, 1.2), (20, 6.0), (40, 1.2))]
    want = [oracle.run(oracle.Desc(**r), hist=True, final=True, digest=True) for r in runs]
    descs = [pa.Desc(outputs=pa.OUT_HIST | pa.OUT_FINAL | pa.OUT_DIGEST, **r) for r in runs]
    for d, w in zip(descs, want):
        print(f"\nL={d.L} q={d.q} R={d.R}", flush=True)
        _same(pa.pa_run(plain, d), w)
    for mode in (pa.BATCH_SEGMENTED, pa.BATCH_TEAM):
        plain.set_batch_mode(mode)
        for g, w in zip(pa.pa_run_batch(plain, descs), want):
            _same(g, w)


def test_shapes_whose_launch_the_population_does_not_fill_are_not_timed(plain):
    """Below one round of the 12-wave workgroups such a shape's runs take the
    dword shape, whose rate must not be filed under it; at 24x24 that is every
    population below 2^14."""
    for L, R, lanes, timed in ((24, 8000, 24, False), (24, 17000, 24, True), (48, 2048, 96, False), (48, 5000, 96, True),
                               (96, 1000, 384, False)):
        e = plain.tune(L, 10, R)
        assert ((lanes, 12) in {(t["lanes"], t["waves_per_block"]) for t in e["timed"]}) is timed, (L, R)
    c = pa.Context(0)
    try:
        assert _get(c, 24, 10, 8000) == (48, 12) and _get(c, 24, 10, 50000) == (24, 12)
    finally:
        c.close()
