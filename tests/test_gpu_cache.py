"""Parity of the HBM-bound cache kernels (difference refresh, Taylor forecast,
relative-error verification) with the CPU oracle, through the C ABI.

Tolerances.  fp32 cache: both sides hold fp32 values; the kernel's fp32 arithmetic
(a handful of FMAs with O(1) coefficients, a reciprocal instead of a division)
differs from the oracle's float64 by a few fp32 ulps of the largest term, so the
bar is max-abs error / max-abs value <= 1e-5.  bf16 cache: the oracle rounds to
bf16 at the same places the kernel stores, so results agree to 1 bf16 ulp
(2^-8 relative) where fp32-vs-fp64 noise lands on a rounding boundary; against
the unrounded oracle the bar is the end-to-end 2e-2."""
import numpy as np
import pytest

import speca_inputs as si
from oracle import speca_core as core

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _sp():
    import paper_2509_11628_amd as sp
    return sp


def max_abs_rel(a, b):
    a = np.asarray(a, np.float64); b = np.asarray(b, np.float64)
    return float(np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-30))


def _dev(a, dtype):
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda().to(td).contiguous()


def _host(t):
    return t.float().cpu().numpy().astype(np.float64)


def _oracle_caches(B, slots, m, mode, store):
    return [core.FeatureCache(slots, m, mode, store) for _ in range(B)]


CASES = [
    # slots, B, T, D, dtype        (E = T*D: vector path needs E % 8 == 0; 37*13 exercises the scalar tail path)
    (3, 3, 40, 72, "f32"),
    (3, 3, 40, 72, "bf16"),
    (2, 2, 37, 13, "f32"),
    (2, 2, 37, 13, "bf16"),
    (2, 4, 129, 200, "bf16"),     # several blocks per row + ragged last block
]


@pytest.mark.parametrize("slots,B,T,D,dtype", CASES)
@pytest.mark.parametrize("mode", ["taylor", "newton", "adams_bashforth"])
def test_refresh_forecast_parity(slots, B, T, D, dtype, mode):
    sp = _sp()
    from paper_2509_11628_amd import binding as bd
    m = 2
    dt = bd.BF16 if dtype == "bf16" else bd.F32
    ctx = sp.Context(sp.cache_only_desc(slots, T, D, dt))
    ctx.init_cache(sp.make_cfg(order=m, interval=100, coef_mode={"taylor": bd.COEF_TAYLOR, "newton": bd.COEF_NEWTON, "adams_bashforth": bd.COEF_ADAMS_BASHFORTH}[mode]), B)
    oc = _oracle_caches(B, slots, m, mode, dtype)
    # irregular, per-row histories: rows skip some refreshes
    plan = [(0, list(range(B))), (3, list(range(B))), (4, [r for r in range(B) if r % 2 == 0]), (9, list(range(B)))]
    steps_all = [p[0] for p in plan]
    feats = si.feature_trajectory(slots, B, T, D, steps_all, seed=7, dtype=dtype)
    for (s, rows), f in zip(plan, feats):
        sub = np.ascontiguousarray(f[:, rows])
        ctx.refresh(s, rows, _dev(sub, dtype))
        for i, r in enumerate(rows):
            oc[r].refresh(s, [sub[j, i] for j in range(slots)])
    for step in (10, 12):
        rows = list(range(B))
        out = torch.empty((slots, B, T, D), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
        ctx.forecast(step, rows, out)
        got = _host(out)
        exp = np.stack([np.stack([oc[r].forecast(step, j) for r in rows]) for j in range(slots)])
        if dtype == "f32":
            assert max_abs_rel(got, exp) <= 1e-5
        else:
            expb = core.bf16_round(exp)
            ulp = np.abs(expb) * 2.0 ** -7 + 1e-30
            assert np.all(np.abs(got - expb) <= ulp)                       # at most one bf16 step
            assert np.mean(got != expb) < 0.02                             # and almost always identical
    # subset of rows, compact output
    rows = [B - 1]
    out = torch.empty((slots, 1, T, D), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    ctx.forecast(11, rows, out)
    exp = np.stack([np.stack([oc[r].forecast(11, j) for r in rows]) for j in range(slots)])
    assert max_abs_rel(_host(out), exp) <= (1e-5 if dtype == "f32" else 2.0 ** -8)
    ctx.close()


@pytest.mark.parametrize("slots,B,T,D,dtype", [CASES[0], CASES[1], CASES[3], CASES[4]])
@pytest.mark.parametrize("mode", ["taylor", "newton", "adams_bashforth"])
@pytest.mark.parametrize("m", [0, 2, 3])
def test_ring_layout_refresh_forecast_parity(slots, B, T, D, dtype, mode, m):
    """Raw-feature ring layout: per-row histories that differ, more full steps than planes (the
    ring wraps), forecasts during the warm-up; against the oracle's ring cache, which forms the
    differences from the stored features by the recursion's definition."""
    sp = _sp()
    from paper_2509_11628_amd import binding as bd
    dt = bd.BF16 if dtype == "bf16" else bd.F32
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    code = {"taylor": bd.COEF_TAYLOR, "newton": bd.COEF_NEWTON, "adams_bashforth": bd.COEF_ADAMS_BASHFORTH}[mode]
    ctx = sp.Context(sp.cache_only_desc(slots, T, D, dt))
    ctx.init_cache(sp.make_cfg(order=m, interval=100, coef_mode=code, layout=bd.CACHE_RING), B)
    oc = [core.make_cache("ring", slots, m, mode, dtype) for _ in range(B)]
    plan = [(0, list(range(B))), (3, list(range(B))), (4, [r for r in range(B) if r % 2 == 0]), (9, list(range(B))),
            (11, [r for r in range(B) if r % 2 == 1]), (12, list(range(B))), (17, list(range(B)))]
    feats = si.feature_trajectory(slots, B, T, D, [p[0] for p in plan], seed=9, dtype=dtype)
    for n, ((s, rows), f) in enumerate(zip(plan, feats)):
        sub = np.ascontiguousarray(f[:, rows])
        ctx.refresh(s, rows, _dev(sub, dtype))
        for i, r in enumerate(rows):
            oc[r].refresh(s, [sub[j, i] for j in range(slots)])
        for step in (s + 1, s + 3):
            rows_f = list(range(B))
            out = torch.empty((slots, B, T, D), dtype=td, device="cuda")
            ctx.forecast(step, rows_f, out)
            got = _host(out)
            exp = np.stack([np.stack([oc[r].forecast(step, j) for r in rows_f]) for j in range(slots)])
            if dtype == "f32":
                assert max_abs_rel(got, exp) <= 1e-5, (n, step)
            else:
                expb = core.bf16_round(exp)
                # fp32 sum of up to m+1 terms that partly cancel: allow the rounding boundary to move by the
                # fp32 noise of the largest term as well
                ulp = np.abs(expb) * 2.0 ** -7 + 1e-5
                assert np.all(np.abs(got - expb) <= ulp), (n, step)
                assert np.mean(got != expb) < 0.03, (n, step)
    ctx.close()


def test_bf16_cache_vs_unrounded_oracle():
    sp = _sp()
    from paper_2509_11628_amd import binding as bd
    slots, B, T, D, m = 2, 2, 64, 64, 2
    ctx = sp.Context(sp.cache_only_desc(slots, T, D, bd.BF16))
    ctx.init_cache(sp.make_cfg(order=m, interval=4), B)
    oc = _oracle_caches(B, slots, m, "taylor", None)
    feats = si.feature_trajectory(slots, B, T, D, [0, 4, 8], seed=1, dtype="bf16")
    for s, f in zip([0, 4, 8], feats):
        ctx.refresh(s, [0, 1], _dev(f, "bf16"))
        for r in range(B):
            oc[r].refresh(s, [f[j, r] for j in range(slots)])
    out = torch.empty((slots, B, T, D), dtype=torch.bfloat16, device="cuda")
    ctx.forecast(11, [0, 1], out)
    exp = np.stack([np.stack([oc[r].forecast(11, j) for r in range(B)]) for j in range(slots)])
    assert max_abs_rel(_host(out), exp) <= 2e-2


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("E", [8, 1000, 8192, 8192 * 3 + 40, 12345])
def test_verify_parity(dtype, E):
    sp = _sp()
    from paper_2509_11628_amd import binding as bd
    B = 8
    rng = np.random.default_rng(E)
    pred = si._store(rng.standard_normal((B, E)).astype(np.float32), dtype)
    truth = si.perturbed_target(pred, si.VERIFY_DELTAS, seed=3, dtype=dtype)
    ctx = sp.Context(sp.cache_only_desc(1, 1, 8, bd.BF16 if dtype == "bf16" else bd.F32))
    err, acc = ctx.verify(_dev(pred, dtype), _dev(truth, dtype), tau=0.05)
    exp = np.array([core.relative_error(pred[b], truth[b]) for b in range(B)])
    np.testing.assert_allclose(err, exp, rtol=2e-5)          # fp32 accumulation of <= 1e5 terms, pairwise-ish tree
    exp_acc = np.array([core.accept(core.relative_error_f32(pred[b], truth[b]), 0.05) for b in range(B)])
    margin = np.min(np.abs(exp - 0.05) / 0.05)
    if margin > 1e-3:
        assert acc.tolist() == exp_acc.tolist()
    if E >= 1000 and dtype == "f32":
        assert acc.tolist() == [True] * 4 + [False] * 4       # the recipe's 4 accept / 4 reject split
    # identical tensors -> exactly zero; zero truth -> finite thanks to eps
    e0, _ = ctx.verify(_dev(pred, dtype), _dev(pred, dtype))
    assert np.all(e0 == 0.0)
    ez, _ = ctx.verify(_dev(pred, dtype), _dev(np.zeros_like(pred), dtype))
    assert np.all(np.isfinite(ez)) and np.all(ez > 1e6)
    ctx.close()


def test_verify_leaves_the_stream_idle():
    """The errors travel through pinned memory that the host polls; the call still synchronises the stream, as every call that
    returns host results does."""
    import ctypes as C
    sp = _sp()
    from paper_2509_11628_amd import binding as bd
    rows, E = 2, 1024
    p = torch.randn((rows, E), device="cuda"); t = p + 0.1 * torch.randn_like(p)
    ctx = sp.Context(sp.cache_only_desc(1, 1, 8, bd.F32))
    err = np.zeros(rows, np.float32)
    args = (ctx.h, C.c_void_p(p.data_ptr()), C.c_void_p(t.data_ptr()), rows, E, bd.F32, None, 1e-8, bd._p(err, C.c_float), None)
    stream = torch.cuda.current_stream()
    torch.cuda.synchronize()
    idle = 0
    for _ in range(200):
        assert ctx.lib.speca_verify(*args) == bd.OK
        idle += stream.query()
    ctx.close()
    assert idle == 200


@pytest.mark.parametrize("rows", [1023, 1024, 1025, 2100])
def test_verify_of_more_rows_than_one_launch(rows):
    """1024 rows share a launch; the errors of every launch arrive, and the stream is idle after the last one."""
    sp = _sp()
    from paper_2509_11628_amd import binding as bd
    rng = np.random.default_rng(rows)
    E = 24
    truth = rng.standard_normal((rows, E)).astype(np.float32)
    pred = (truth + rng.uniform(0.01, 0.2, (rows, 1)) * rng.standard_normal((rows, E))).astype(np.float32)
    ctx = sp.Context(sp.cache_only_desc(1, 1, 8, bd.F32))
    err, acc = ctx.verify(_dev(pred, "f32"), _dev(truth, "f32"), tau=0.1)
    assert torch.cuda.current_stream().query()
    exp = np.array([core.relative_error(pred[r], truth[r]) for r in range(rows)])
    np.testing.assert_allclose(err, exp, rtol=2e-5)
    clear = np.abs(exp - 0.1) > 1e-5
    assert np.array_equal(acc[clear], (exp <= 0.1)[clear]) and 0 < acc.sum() < rows
    ctx.close()


def test_verify_is_bit_reproducible_and_row_independent():
    sp = _sp()
    from paper_2509_11628_amd import binding as bd
    rng = np.random.default_rng(0)
    B, E = 6, 8192 * 5 + 24
    p = _dev(rng.standard_normal((B, E)), "bf16"); t = _dev(rng.standard_normal((B, E)), "bf16")
    ctx = sp.Context(sp.cache_only_desc(1, 1, 8, bd.BF16))
    e1, _ = ctx.verify(p, t)
    e2, _ = ctx.verify(p, t)
    assert e1.tobytes() == e2.tobytes()
    e3, _ = ctx.verify(p[2:3].contiguous(), t[2:3].contiguous())
    assert e3[0].tobytes() == e1[2].tobytes()                # a row's result does not depend on its neighbours
    ctx.close()


@pytest.mark.parametrize("metric", ["l1", "linf", "cosine"])
def test_verify_other_metrics(metric):
    sp = _sp()
    from paper_2509_11628_amd import binding as bd
    code = {"l1": bd.METRIC_L1, "linf": bd.METRIC_LINF, "cosine": bd.METRIC_COSINE}[metric]
    fn = {"l1": core.relative_error_l1, "linf": core.relative_error_linf, "cosine": core.cosine_distance}[metric]
    rng = np.random.default_rng(5)
    B, E = 3, 8192 + 123
    pred = rng.standard_normal((B, E)).astype(np.float32)
    truth = (pred + 0.1 * rng.standard_normal((B, E))).astype(np.float32)
    ctx = sp.Context(sp.cache_only_desc(1, 1, 8, bd.F32))
    ctx.init_cache(sp.make_cfg(order=0, interval=1, metric=code), 1)
    err, _ = ctx.verify(_dev(pred, "f32"), _dev(truth, "f32"))
    exp = np.array([fn(pred[b], truth[b]) for b in range(B)])
    np.testing.assert_allclose(err, exp, rtol=1e-4, atol=1e-6)
    ctx.close()


def test_error_paths():
    sp = _sp()
    from paper_2509_11628_amd import binding as bd
    ctx = sp.Context(sp.cache_only_desc(2, 4, 8, bd.F32))
    buf = torch.zeros((2, 2, 4, 8), device="cuda")
    with pytest.raises(sp.SpecaError) as e:
        ctx.forecast(1, [0], buf)
    assert e.value.code == bd.ESTATE                      # cache not initialised
    with pytest.raises(sp.SpecaError) as e:
        ctx.init_cache(sp.make_cfg(order=9), 2)
    assert e.value.code == bd.EINVAL
    with pytest.raises(sp.SpecaError) as e:
        ctx.init_cache(sp.make_cfg(interval=0), 2)
    assert e.value.code == bd.EINVAL
    ctx.init_cache(sp.make_cfg(order=1, interval=4), 2)
    with pytest.raises(sp.SpecaError) as e:
        ctx.forecast(1, [0], buf)
    assert e.value.code == bd.ESTATE                      # no reference yet
    ctx.refresh(2, [0, 1], buf)
    for bad in ([2], [-1], [1, 0], [0, 0]):
        with pytest.raises(sp.SpecaError) as e:
            ctx.forecast(3, bad, buf)
        assert e.value.code == bd.EINVAL
    with pytest.raises(sp.SpecaError) as e:
        ctx.forecast(2, [0], buf)                         # not after the reference
    assert e.value.code == bd.ESTATE
    with pytest.raises(sp.SpecaError) as e:
        ctx.refresh(2, [0], buf)
    assert e.value.code == bd.ESTATE
    with pytest.raises(sp.SpecaError) as e:
        ctx.full_step(buf, 3, [0], buf, labels=[0, 0])
    assert e.value.code == bd.EUNSUPPORTED                # cache-only context has no model
    ctx.forecast(3, [0, 1], buf)                          # and a valid call still works afterwards
    torch.cuda.synchronize()
    ctx.close()


@pytest.mark.parametrize("layout", ["differences", "ring"])
def test_config2_full_size_sampled(layout):
    """Configuration 2 at full size (28 slots x 8 x 256 x 1152, bf16, order 2, references at
    steps 0,4,8), in the launch shape the benchmark times (both cache layouts; the benchmark
    runs the ring); checked on sampled positions."""
    sp = _sp()
    from paper_2509_11628_amd import binding as bd
    slots, B, T, D, m = 28, 8, 256, 1152, 2
    ctx = sp.Context(sp.cache_only_desc(slots, T, D, bd.BF16))
    ctx.init_cache(sp.make_cfg(order=m, interval=4, layout=bd.CACHE_RING if layout == "ring" else bd.CACHE_DIFFERENCES), B)
    rows = list(range(B))
    feats = si.feature_trajectory(slots, B, T, D, [0, 4, 8], seed=0, dtype="bf16")
    for s, f in zip([0, 4, 8], feats):
        ctx.refresh(s, rows, _dev(f, "bf16"))
    out = torch.empty((slots, B, T, D), dtype=torch.bfloat16, device="cuda")
    rng = np.random.default_rng(0)
    idx = (rng.integers(0, slots, 4000), rng.integers(0, B, 4000), rng.integers(0, T, 4000), rng.integers(0, D, 4000))
    # include the corners
    for a in idx:
        a[:2] = [0, a.max()]
    F = [f[idx].astype(np.float64) for f in feats]
    for k in (1, 2, 3):
        ctx.forecast(8 + k, rows, out)
        got = _host(out[idx[0], idx[1], idx[2], idx[3]])
        c = core.make_cache(layout, 1, m, "taylor", "bf16")
        for s, f in zip([0, 4, 8], F):
            c.refresh(s, [f])
        expb = core.bf16_round(c.forecast(8 + k, 0))
        assert np.all(np.abs(got - expb) <= np.abs(expb) * 2.0 ** -7 + (1e-5 if layout == "ring" else 1e-30))
        assert np.mean(got != expb) < (0.03 if layout == "ring" else 0.02)
    # verification on the last slot against the recipe's perturbed target: 4 accept / 4 reject at 0.05
    pred = _host(out[slots - 1]).astype(np.float32)
    truth = si.perturbed_target(pred, si.VERIFY_DELTAS, seed=0, dtype="bf16")
    err, acc = ctx.verify(out[slots - 1].contiguous(), _dev(truth, "bf16"), tau=0.05)
    exp = np.array([core.relative_error(pred[b], truth[b]) for b in range(B)])
    np.testing.assert_allclose(err, exp, rtol=2e-5)
    assert acc.tolist() == [True] * 4 + [False] * 4
    assert np.min(np.abs(exp - 0.05) / 0.05) > 0.15
    ctx.close()


def test_row_list_limits():
    """Empty, maximum-size and over-size row lists (one launch carries at most 64 rows)."""
    sp = _sp()
    from paper_2509_11628_amd import binding as bd
    slots, B, T, D = 1, 70, 4, 8
    ctx = sp.Context(sp.cache_only_desc(slots, T, D, bd.F32))
    ctx.init_cache(sp.make_cfg(order=1, interval=4), B)
    rng = np.random.default_rng(0)
    f0 = rng.standard_normal((slots, B, T, D)).astype(np.float32)
    f1 = rng.standard_normal((slots, B, T, D)).astype(np.float32)
    oc = _oracle_caches(B, slots, 1, "taylor", "f32")
    for s_, f in ((0, f0), (3, f1)):
        for lo, hi in ((0, 64), (64, 70)):                # 64 rows: the largest single launch, then the ragged rest
            rows = list(range(lo, hi))
            ctx.refresh(s_, rows, _dev(np.ascontiguousarray(f[:, lo:hi]), "f32"))
        for r in range(B):
            oc[r].refresh(s_, [f[j, r] for j in range(slots)])
    out = torch.empty((slots, 64, T, D), dtype=torch.float32, device="cuda")
    ctx.forecast(5, list(range(64)), out)
    exp = np.stack([np.stack([oc[r].forecast(5, j) for r in range(64)]) for j in range(slots)])
    assert max_abs_rel(_host(out), exp) <= 1e-5
    big = torch.empty((slots, 65, T, D), dtype=torch.float32, device="cuda")
    with pytest.raises(sp.SpecaError) as e:
        ctx.forecast(5, list(range(65)), big)
    assert e.value.code in (bd.EUNSUPPORTED, bd.EINVAL)
    with pytest.raises(sp.SpecaError) as e:
        ctx.forecast(5, [], out)
    assert e.value.code == bd.EINVAL
    with pytest.raises(sp.SpecaError) as e:
        ctx.refresh(6, [], out)
    assert e.value.code == bd.EINVAL
    ctx.close()
