"""The passes' tile split that an untuned set picks for itself changes no bit:
derivatives, right-hand side and filter of untuned sets equal those of the same
sets tuned to other splits, their reverse modes (whose folds belong to the
nominal split) those of the sets tuned to the nominal one."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_16076_amd import api
    ctx = api.Context(0)
    yield api, ctx, torch
    ctx.sync()


CASES = {
    "one small patch": lambda: synth.config(0, n=48),
    "few short lines": lambda: synth.config(3, n=48),
    "uneven": lambda: synth.config(2, npatch=9, nmax=200),
    "many patches, d = 2": lambda: synth.paper_subpatches(16, 4),
    "long lines": lambda: synth.config(0, n=700),
}


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("name", list(CASES))
def test_untuned_split_changes_no_bit(env, name, layout):
    api, ctx, torch = env
    cfg = CASES[name]()
    ps = cfg.ps
    if name == "long lines":
        ps = synth.unit_square(700, C=28)      # 728 = 2^3 7 13
        cfg.u0 = synth._f32(synth.square_state(ps, np.random.default_rng(0)), ps)
    outs = []
    for tune in (None, (163840, 1024), (24576, 256)):
        s = api.PatchSet.from_layout(ctx, ps, layout)
        if tune:
            s.tune(*tune)
        s.set_filter(10.0, 14)
        u, metric = s.to_device(cfg.u0), s.to_device(ps.metric)
        mu = s.to_device(np.full((1, ps.plane), 1e-3, np.float32))
        rhs, d1, d2, uf = (torch.zeros_like(u) for _ in range(4))
        api.fcsd_rhs(s, u, metric, mu, cfg.ref, 1.4, rhs)
        api.fc_diff(s, 1, u, d1, 4)
        api.fc_diff(s, 2, u, d2, 4)
        api.fcsd_filter(s, u, uf, 1.4)
        outs.append([s.to_host(t) for t in (rhs, d1, d2, uf)])
        s.close()
    for o in outs[1:]:
        for a, b in zip(o, outs[0]):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("name", [k for k in CASES if k != "long lines"])
def test_untuned_split_changes_no_bit_of_the_reverse(env, name, layout):
    api, ctx, torch = env
    cfg = CASES[name]()
    ps = cfg.ps
    rng = np.random.default_rng(4)
    bar = rng.standard_normal((4, ps.plane)).astype(np.float32)
    outs = []
    for tune in (None, (65536, 256)):
        s = api.PatchSet.from_layout(ctx, ps, layout)
        if tune:
            s.tune(*tune)
        s.set_filter(10.0, 14)
        u, metric = s.to_device(cfg.u0), s.to_device(ps.metric)
        mu = s.to_device(np.full((1, ps.plane), 1e-3, np.float32))
        rb = s.to_device(bar)
        ub, e1, e2, d1, d2, fb = (torch.zeros_like(u) for _ in range(6))
        mb = torch.zeros_like(mu)
        api.fcsd_rhs_adj(s, u, metric, mu, cfg.ref, 1.4, rb, ub, mb)
        api.euler_rhs_adj(s, u, metric, cfg.ref, 1.4, rb, e1)
        s.set_schedule(0)
        api.fcsd_rhs_adj(s, u, metric, mu, cfg.ref, 1.4, rb, e2)
        api.fc_diff_adj(s, 1, rb, d1, 4)
        api.fc_diff_adj(s, 2, rb, d2, 4)
        api.fcsd_filter_adj(s, u, rb, fb, 1.4)
        outs.append([s.to_host(t) for t in (ub, e1, e2, d1, d2, fb)] + [s.to_host(mb)])
        s.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


# sets of transforms -> the variants that their untuned split takes
FORMS = {
    "few short lines": dict(transforms=(16, 16), a_two_lines=True, b_four_lines=True, two_rounds=(True, True)),
    "many patches, d = 2": dict(transforms=(64, 64), a_two_lines=True, b_four_lines=False, two_rounds=(True, True)),
    "one small patch": dict(products=(1, 1), transforms=(0, 0)),
    "uneven": dict(products=(9, 9), transforms=(0, 0)),
}


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("name", list(FORMS))
def test_variants_of_the_untuned_split(env, name, layout):
    """The cases that the tests above compare bit for bit do run the variants
    against their one-line forms: the untuned sets the former, the tuned sets
    the latter."""
    api, ctx, torch = env
    s = api.PatchSet.from_layout(ctx, CASES[name]().ps, layout)
    f = s.forms()
    assert {k: f[k] for k in FORMS[name]} == FORMS[name]
    s.tune(65536, 256)
    f = s.forms()
    assert not f["b_four_lines"] and f["two_rounds"] == (False, False)
    s.close()


@pytest.mark.parametrize("layout", [0, 1])
def test_untuned_split_changes_no_bit_of_the_reverse_of_long_lines(env, layout):
    """As for short lines; in blocked storage four complex lines per grid line
    exceed the LDS, so the reverse runs its narrower q2 pass."""
    api, ctx, torch = env
    ps = synth.unit_square(700, C=28)      # 728 = 2^3 7 13
    rng = np.random.default_rng(4)
    u0 = synth._f32(synth.square_state(ps, rng), ps)
    bar = rng.standard_normal((4, ps.plane)).astype(np.float32)
    outs = []
    for tune in (None, (65536, 256)):
        s = api.PatchSet.from_layout(ctx, ps, layout)
        assert s.forms()["transforms"] == (1, 1)
        if tune:
            s.tune(*tune)
        u, metric, rb = s.to_device(u0), s.to_device(ps.metric), s.to_device(bar)
        mu = s.to_device(np.full((1, ps.plane), 1e-3, np.float32))
        ub, d1, d2 = (torch.zeros_like(u) for _ in range(3))
        mb = torch.zeros_like(mu)
        api.fcsd_rhs_adj(s, u, metric, mu, [1.0, 0.0, 0.0, 1.0], 1.4, rb, ub, mb)
        api.fc_diff_adj(s, 1, rb, d1, 4)
        api.fc_diff_adj(s, 2, rb, d2, 4)
        outs.append([s.to_host(t) for t in (ub, d1, d2, mb)])
        s.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("split", ["tuned", "untuned"])
def test_wide_schedule_runs_its_pass(env, split, layout):
    """The wide schedule keeps all eight H fields of a q2 tile in LDS on sets
    of transforms, whatever their tuning, with the bits of the fused one; sets
    of products have one form and report the fused schedule."""
    api, ctx, torch = env
    cfg = CASES["many patches, d = 2"]()
    ps = cfg.ps
    s = api.PatchSet.from_layout(ctx, ps, layout)
    if split == "tuned":
        s.tune(65536, 256)
    outs = []
    for sched in (1, 3):
        s.set_schedule(sched)
        f = s.forms()
        assert f["schedule"] == sched and f["b_four_lines"] == (sched == 3)
        u, metric = s.to_device(cfg.u0), s.to_device(ps.metric)
        rhs = torch.zeros_like(u)
        api.fcsd_rhs(s, u, metric, s.to_device(np.full((1, ps.plane), 1e-3, np.float32)), cfg.ref, 1.4, rhs)
        outs.append(s.to_host(rhs))
    assert np.array_equal(*outs)
    s.close()
    s = api.PatchSet.from_layout(ctx, CASES["uneven"]().ps, layout)
    s.set_schedule(3)
    assert s.forms()["schedule"] == 1
    s.close()


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("name", ["transforms", "products", "both"])
def test_persistent_schedule_runs_on_every_set(env, name, layout):
    """One launch per stage on sets of transforms, of products, and of both
    (lines above 512 points next to short ones, along each direction): the
    schedule reports itself, its waits never give up, and its right-hand side
    has the fused schedule's bits, on short and long queues."""
    api, ctx, torch = env
    if name == "transforms":
        ps = CASES["many patches, d = 2"]().ps
    elif name == "products":
        ps = CASES["uneven"]().ps
    else:
        ps = synth.uneven_sectors(5, 60, 700, 3)
    n1, n2 = np.asarray(ps.n1), np.asarray(ps.n2)
    prod = (0, 0) if name == "transforms" else (int((n1 <= 512).sum()), int((n2 <= 512).sum()))
    rng = np.random.default_rng(8)
    u0 = synth._f32(synth.mach_state(ps, 3.0, synth.draw_perturbation(rng)), ps)
    for tune in (None, ((16384, 16384, 24576), (256, 256, 256))):
        s = api.PatchSet.from_layout(ctx, ps, layout)
        if tune:
            s.tune(*tune)
        f = s.forms()
        assert f["products"] == prod and f["transforms"] == (ps.npatch - prod[0], ps.npatch - prod[1])
        u, metric = s.to_device(u0), s.to_device(ps.metric)
        mu = s.to_device(np.full((1, ps.plane), 1e-3, np.float32))
        outs = []
        for sched in (1, 2):
            s.set_schedule(sched)
            assert s.forms()["schedule"] == sched
            rhs = torch.zeros_like(u)
            api.fcsd_rhs(s, u, metric, mu, [1.4, 3.0, 0.0, 1.0], 1.4, rhs)
            outs.append(s.to_host(rhs))
        assert s.stage_errors() == 0
        assert np.array_equal(*outs)
        s.close()
    if name == "both":
        assert 0 < prod[0] < ps.npatch and 0 < prod[1] < ps.npatch


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("tune", [(65536, 256), (16384, 256), (98304, 1024)])
def test_tuned_set_returns_to_its_picked_split(env, tune, layout):
    """set_split(True) gives a tuned set the variants of an untouched one and
    the bits of its own tuning, reverse mode included; set_split(False) takes
    them back."""
    api, ctx, torch = env
    cfg = CASES["few short lines"]()
    ps = cfg.ps
    rng = np.random.default_rng(6)
    bar = rng.standard_normal((4, ps.plane)).astype(np.float32)
    s = api.PatchSet.from_layout(ctx, ps, layout)
    new = s.forms()
    assert new["picked"]
    s.tune(*tune)
    tuned = s.forms()
    assert not tuned["picked"] and not tuned["b_four_lines"] and tuned["two_rounds"] == (False, False)
    outs = []
    for picked in (False, True, False):
        s.set_split(picked)
        assert s.forms() == (new if picked else tuned)
        u, metric = s.to_device(cfg.u0), s.to_device(ps.metric)
        mu = s.to_device(np.full((1, ps.plane), 1e-3, np.float32))
        rb = s.to_device(bar)
        rhs, ub, d1 = (torch.zeros_like(u) for _ in range(3))
        mb = torch.zeros_like(mu)
        api.fcsd_rhs(s, u, metric, mu, cfg.ref, 1.4, rhs)
        api.fcsd_rhs_adj(s, u, metric, mu, cfg.ref, 1.4, rb, ub, mb)
        api.fc_diff_adj(s, 1, rb, d1, 4)
        outs.append([s.to_host(t) for t in (rhs, ub, d1, mb)])
    for o in outs[1:]:
        for a, b in zip(o, outs[0]):
            assert np.array_equal(a, b)
    s.close()


def test_autotuner_weighs_the_picked_split(env):
    """The split an untouched set runs on is among the autotuner's candidates,
    the fastest candidate is kept, and the set is left on it."""
    from paper_2506_16076_amd import autotune
    api, ctx, torch = env
    cfg = CASES["few short lines"]()
    ps = cfg.ps
    s = api.PatchSet.from_layout(ctx, ps, 1)
    u, metric = s.to_device(cfg.u0), s.to_device(ps.metric)
    mu = s.to_device(np.full((1, ps.plane), 1e-3, np.float32))
    r = autotune.autotune(s, u, metric, mu, cfg.ref, budgets=(24576, 65536), threads=(256, 512), reps=2)
    assert {c["split"] for c in r["stages"]} == {"tuned", "picked"}
    assert r["stage_ms"] == pytest.approx(min(c["ms"] for c in r["stages"]), abs=1e-4)
    assert s.forms()["picked"] == (r["split"] == "picked")
    s.close()


def test_transform_pass_times_what_the_stage_does_not_run(env):
    """fcsd_transform_pass differentiates the state by transforms on each tile
    set, lines of products among them: the FP64 derivative within 1e-5 of its
    largest value (the transform's bar elsewhere), and an aliased output is
    refused."""
    from oracle import fcgram
    api, ctx, torch = env
    cfg = CASES["uneven"]()
    ps = cfg.ps
    s = api.PatchSet.from_layout(ctx, ps, 1)
    assert s.forms()["transforms"] == (0, 0)
    u = s.to_device(cfg.u0)
    for tiles in (0, 1, 2):
        out = torch.zeros_like(u)
        api.fcsd_transform_pass(s, tiles, u, cfg.ref, out)
        got = s.to_host(out)
        for f in (0, 3):
            want = fcgram.diff_plane(cfg.u0[f].astype(np.float64), ps, 1 if tiles == 0 else 2)
            for p in range(ps.npatch):
                w, g = ps.view(want, p), ps.view(got[f], p)
                assert np.abs(g - w).max() <= 1e-5 * max(np.abs(w).max(), np.abs(cfg.u0[f]).max())
    with pytest.raises(api.FcsdError):
        api.fcsd_transform_pass(s, 0, u, cfg.ref, u)
    s.close()


def test_autotuner_times_the_transforms_of_product_sets(env):
    """On sets of products no stage pass runs on the tuned tile sets: each is
    picked by the transforms on it, not by passes that it cannot change."""
    from paper_2506_16076_amd import autotune
    api, ctx, torch = env
    cfg = CASES["uneven"]()
    s = api.PatchSet.from_layout(ctx, cfg.ps, 1)
    u, metric = s.to_device(cfg.u0), s.to_device(cfg.ps.metric)
    mu = s.to_device(np.full((1, cfg.ps.plane), 1e-3, np.float32))
    r = autotune.autotune(s, u, metric, mu, cfg.ref, budgets=(16384, 65536), threads=(256, 512), reps=2)
    for k, key in enumerate(("T0", "T1", "T2")):
        best = min(v[key] for n, v in r["table"].items() if n.startswith(r["order"]))
        assert r["table"]["%s-%dK-%d" % (r["order"], r["budgets"][k] // 1024, r["threads"][k])][key] == best \
            or r["schedule"] == "persistent"
    assert s.forms()["schedule"] == {"split": 0, "fused": 1, "persistent": 2}[r["schedule"]]
    s.close()
