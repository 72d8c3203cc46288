"""Parity of the MMDiT target model (dual- and single-stream blocks, RoPE, QK RMS-norm, joint
attention, rectified-flow sampling) with the CPU oracle, through the C ABI.  Reduced shapes:
the FLUX- and HunyuanVideo-shaped configurations are far beyond a CPU oracle; they are run
at full size by the benchmark and checked there through properties only.

Bars as for the DiT tests: schedules decision by decision, latents 1e-5 (fp32) / 2e-2 (bf16)."""
import numpy as np
import pytest

import branch_tiles
import speca_inputs as si
from oracle import mmdit as ommdit, sampler as osamp, speca_core as core

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from test_gpu_dit import compare_traces, max_abs_rel  # noqa: E402


def make_gpu(shape, weights):
    import paper_2509_11628_amd as sp
    from paper_2509_11628_amd import binding as bd
    dt = bd.BF16 if shape.dtype == "bf16" else bd.F32
    return sp.Context(sp.mmdit_desc(shape), sp.to_device(weights, dt))


def _td(s):
    return torch.bfloat16 if s.dtype == "bf16" else torch.float32


@pytest.fixture(scope="module", params=[("image", "f32"), ("image", "bf16"), ("video", "f32")])
def tiny(request):
    kind, dtype = request.param
    s = si.mmdit_tiny(dtype) if kind == "image" else si.mmdit_tiny_video(dtype)
    w = si.make_mmdit_weights(s, 0)
    return s, w, ommdit.MMDiTOracle(s, w), make_gpu(s, w)


def _tol(s):
    return 1e-5 if s.dtype == "f32" else 2e-2


def test_full_step_matches_oracle_forward(tiny):
    import paper_2509_11628_amd as sp
    s, w, om, ctx = tiny
    B = 2
    x = si.make_video_latents(B, s, 5); txt, vec = si.make_text(B, s, 5)
    ctx.init_cache(sp.make_cfg(order=1, interval=4), B)
    xd = torch.from_numpy(x).cuda()
    td, vd = torch.from_numpy(txt).cuda().to(_td(s)), torch.from_numpy(vec).cuda().to(_td(s))
    out = torch.zeros_like(xd)
    ctx.full_step(xd, 0, [0, 1], out, timestep=640.0, txt=td, pooled=vd)
    exp, feats = om.forward(x, 640.0, (txt, vec))
    assert max_abs_rel(out.cpu().numpy(), exp) <= _tol(s)
    f = torch.empty((s.n_slots, B, s.tokens, s.hidden), dtype=_td(s), device="cuda")
    ctx.forecast(1, [0, 1], f)
    got = f.float().cpu().numpy()
    for j in range(s.n_slots):
        assert max_abs_rel(got[j], feats[j]) <= (1e-5 if s.dtype == "f32" else 1.5e-2), j
    # one row alone gives the same bits
    out1 = torch.zeros_like(xd)
    ctx.init_cache(sp.make_cfg(order=1, interval=4), B)
    ctx.full_step(xd, 0, [1], out1, timestep=640.0, txt=td, pooled=vd)
    assert torch.equal(out1[1], out[1]) and float(out1[0].abs().max()) == 0.0


def _run_both(s, om, ctx, S, B, cfg_kwargs, tau, seed=0):
    import paper_2509_11628_amd as sp
    from paper_2509_11628_amd import binding as bd
    ts, sg = si.flow_tables(S)
    x = si.make_video_latents(B, s, seed); txt, vec = si.make_text(B, s, seed)
    sol = osamp.Solver("flow", ts, sg)
    conds = [(txt[b], vec[b]) for b in range(B)]
    exp, tr = osamp.sample(om, osamp.SpecaConfig(cache_store="bf16" if s.dtype == "bf16" else None, **cfg_kwargs), sol, tau, x, conds)
    mode = bd.COEF_NEWTON if cfg_kwargs.get("mode") == "newton" else bd.COEF_TAYLOR
    kw = {k: v for k, v in cfg_kwargs.items() if k not in ("mode", "cache_layout")}
    layout = bd.CACHE_RING if cfg_kwargs.get("cache_layout") == "ring" else bd.CACHE_DIFFERENCES
    ctx.init_cache(sp.make_cfg(coef_mode=mode, layout=layout, **kw), B)
    xd = torch.from_numpy(x).cuda()
    td, vd = torch.from_numpy(txt).cuda().to(_td(s)), torch.from_numpy(vec).cuda().to(_td(s))
    got = ctx.sample(xd, ts, sg, tau, solver_kind=bd.SOLVER_FLOW, txt=td, pooled=vd)
    return exp, tr, xd.cpu().numpy(), got


def test_flow_trajectory_mixed_schedule(tiny):
    s, w, om, ctx = tiny
    S = 12
    tau = core.tau_linear(0.02, 0.004, S)
    for kw in (dict(order=1, interval=4), dict(order=2, interval=4, mode="newton"), dict(order=2, interval=5, verify_block=0),
               dict(order=2, interval=5, verify_block=s.depth_dual),
               dict(order=2, interval=4, cache_layout="ring"), dict(order=3, interval=5, mode="newton", cache_layout="ring")):
        exp, tr, got, gtr = _run_both(s, om, ctx, S, 2, kw, tau)
        compared, complete = compare_traces(tr, gtr, s.dtype)
        print(f"\n[{s.dtype}] {kw}: kinds {tr.kind.tolist()} compared {compared} complete {complete}")
        assert compared >= 3, kw
        if s.dtype == "f32":
            assert complete, kw
        if complete:
            assert max_abs_rel(got, exp) <= _tol(s), kw


def test_threshold_zero_and_infinite(tiny):
    s, w, om, ctx = tiny
    S = 8
    exp, tr, got, gtr = _run_both(s, om, ctx, S, 2, dict(order=2, interval=3), np.zeros(S, np.float32))
    assert np.all(gtr["kind"] == 0)
    assert max_abs_rel(got, exp) <= _tol(s)
    exp, tr, got, gtr = _run_both(s, om, ctx, S, 2, dict(order=2, interval=3), np.full(S, np.inf, np.float32))
    assert gtr["kind"][0].tolist() == [0, 1, 1, 0, 1, 1, 0, 1]
    assert max_abs_rel(got, exp) <= _tol(s)


def test_mmdit_error_paths(tiny):
    import paper_2509_11628_amd as sp
    from paper_2509_11628_amd import binding as bd
    s, w, om, ctx = tiny
    x = torch.zeros((1, s.in_channels, s.latent_t, s.latent_h, s.latent_w), device="cuda")
    ctx.init_cache(sp.make_cfg(order=1, interval=2), 1)
    with pytest.raises(sp.SpecaError) as e:
        ctx.full_step(x, 0, [0], x, timestep=1.0)                       # text conditioning missing
    assert e.value.code == bd.EINVAL
    bad = dict(w); bad.pop("single0.lin2_w")
    with pytest.raises(sp.SpecaError) as e:
        make_gpu(s, bad)
    assert e.value.code == bd.EINVAL and "single0.lin2_w" in e.value.msg


# rows, text tokens, latent height and width (patch 2), hidden, heads, mlp_hidden: streams of one token, shorter than a tile, that end inside tiles and
# tiles that span rows of the batch; qkv and the first MLP layer on 256x256 tiles; an MLP of 136 features, whose second layer goes row by row and stream by stream
@pytest.mark.parametrize("layout", ["differences", "ring"])
@pytest.mark.parametrize("rows,txt,h,w,D,H,Dm", [(2, 1, 16, 16, 128, 2, 512), (3, 77, 20, 22, 128, 2, 512), (3, 129, 34, 30, 512, 8, 2048),
                                                 (1, 300, 66, 62, 768, 12, 3072), (2, 40, 18, 22, 128, 2, 136), (5, 65, 128, 128, 512, 8, 2048)])
def test_dual_blocks_of_all_rows_in_one_launch(rows, txt, h, w, D, H, Dm, layout):
    """Three reference steps of all rows together leave the bits (output and every cached plane) of the same steps of a row alone, and the
    first one agrees with the oracle's forward of a row (smaller shapes)."""
    import dataclasses
    import paper_2509_11628_amd as sp
    from paper_2509_11628_amd import binding as bd
    s = dataclasses.replace(si.mmdit_tiny("bf16"), depth_dual=2, depth_single=1, hidden=D, heads=H, mlp_hidden=Dm, txt_tokens=txt, latent_h=h, latent_w=w)
    weights = si.make_mmdit_weights(s, 0)
    ctx = make_gpu(s, weights)
    text, vec = si.make_text(rows, s, 3)
    td, vd = torch.from_numpy(text).cuda().bfloat16(), torch.from_numpy(vec).cuda().bfloat16()
    x = {i: torch.from_numpy(si.make_video_latents(rows, s, i)).cuda() for i in range(3)}
    cfg = sp.make_cfg(order=2, interval=100, layout=bd.CACHE_RING if layout == "ring" else bd.CACHE_DIFFERENCES)

    def steps(which):
        ctx.init_cache(cfg, rows)
        out = torch.zeros((3, *x[0].shape), device="cuda")
        for i, step in enumerate((0, 3, 4)):
            ctx.full_step(x[i], step, which, out[i], timestep=900.0 - 100.0 * i, txt=td, pooled=vd)
        f = torch.empty((s.n_slots, len(which), s.tokens, D), dtype=torch.bfloat16, device="cuda")
        ctx.forecast(6, which, f)
        return out, f

    out, f = steps(list(range(rows)))
    for r in {0, rows - 1}:
        out1, f1 = steps([r])
        assert torch.equal(out1[:, r], out[:, r]) and torch.equal(f1[:, 0], f[:, r]), r
    if s.tokens <= 1400:
        r = rows - 1
        exp, _ = ommdit.MMDiTOracle(s, weights).forward(x[0][r:r + 1].cpu().numpy(), 900.0, (text[r:r + 1], vec[r:r + 1]))
        assert max_abs_rel(out[0, r:r + 1].cpu().numpy(), exp) <= 2e-2
    ctx.close()


@pytest.mark.parametrize("layout", ["differences", "ring"])
@pytest.mark.parametrize("case", branch_tiles.STREAMS, ids=lambda c: "x".join(map(str, c[:7])))
def test_both_streams_on_every_tile(case, layout):
    """Launches for both streams of a dual block on every tile that carries them, under every epilogue: after one reference step of all rows the cached
    features and the output of three rows are those of the oracle's forward of the row; after three, and for the errors of an attempt that
    verifies the dual block, rows together leave the bits of a row alone (another tile); the errors are the oracle's."""
    import dataclasses
    import paper_2509_11628_amd as sp
    from paper_2509_11628_amd import binding as bd
    rows, txt, h, w, D, H, Dm, _ = case
    s = dataclasses.replace(si.mmdit_tiny("bf16"), depth_dual=1, depth_single=1, hidden=D, heads=H, mlp_hidden=Dm, txt_tokens=txt, latent_h=h, latent_w=w)
    weights = si.make_mmdit_weights(s, 0)
    om, ctx = ommdit.MMDiTOracle(s, weights), make_gpu(s, weights)
    text, vec = si.make_text(rows, s, 3)
    td, vd = torch.from_numpy(text).cuda().bfloat16(), torch.from_numpy(vec).cuda().bfloat16()
    x = [torch.from_numpy(si.make_video_latents(rows, s, i)).cuda() for i in range(4)]
    cfg = sp.make_cfg(order=2, interval=100, verify_block=0, layout=bd.CACHE_RING if layout == "ring" else bd.CACHE_DIFFERENCES)

    def steps(which):
        ctx.init_cache(cfg, rows)
        out = torch.zeros((4, *x[0].shape), device="cuda")
        f = torch.empty((2, s.n_slots, len(which), s.tokens, D), dtype=torch.bfloat16, device="cuda")
        errors = []
        for i, step in enumerate((0, 3, 4)):
            ctx.full_step(x[i], step, which, out[i], timestep=900.0 - 100.0 * i, txt=td, pooled=vd)
            if i != 1:
                ctx.forecast(step + 2, which, f[i // 2])
                errors.append(ctx.spec_step(x[3], step + 1, which, np.inf, out[3], timestep=500.0, txt=td, pooled=vd)[0])
        return out, f, errors

    out, f, errors = steps(list(range(rows)))
    for r in {0, rows // 2, rows - 1}:
        out1, f1, errors1 = steps([r])
        assert torch.equal(out1[:, r], out[:, r]) and torch.equal(f1[:, :, 0], f[:, :, r]), r
        assert [e[0] for e in errors1] == [e[r] for e in errors]
        cond = text[r:r + 1], vec[r:r + 1]
        exp, feats = om.forward(x[0][r:r + 1].cpu().numpy(), 900.0, cond)
        assert max_abs_rel(out[0, r:r + 1].cpu().numpy(), exp) <= 2e-2
        for j in range(s.n_slots):
            assert max_abs_rel(f[0, j, r].float().cpu().numpy(), feats[j][0]) <= 1.5e-2, j
        # the attempt after one reference: its forecast is the cached feature, the truth the dual block on the new latents
        h0, c0 = om.begin(x[3][r:r + 1].cpu().numpy(), 500.0, cond)
        e = core.relative_error(core.bf16_round(feats[1]), om.block_real(0, h0, c0)[1][-1])
        assert abs(float(errors[0][r]) - e) <= 2e-2 * e, (r, errors[0][r], e)
    ctx.close()


def test_flux_width_slice_matches_oracle():
    """One dual-stream and one single-stream block at the full FLUX width (D 3072, 24 heads of 128,
    MLP 12288) on 128 + 1280 tokens: the large GEMM tiles, the K lengths of
    configuration 4 (3072, 12288, 15360) and the tiled attention over 22 key tiles, against the
    oracle's forward (about a minute of CPU).  The benchmark's model differs in depth and token count."""
    import dataclasses
    import paper_2509_11628_amd as sp
    s = dataclasses.replace(si.mmdit_flux("bf16"), depth_dual=1, depth_single=1, latent_h=64, latent_w=80, txt_tokens=128)
    w = si.make_mmdit_weights(s, 0)
    om = ommdit.MMDiTOracle(s, w)
    ctx = make_gpu(s, w)
    x = si.make_video_latents(1, s, 3); txt, vec = si.make_text(1, s, 3)
    ctx.init_cache(sp.make_cfg(order=2, interval=5), 1)
    xd = torch.from_numpy(x).cuda()
    td, vd = torch.from_numpy(txt).cuda().bfloat16(), torch.from_numpy(vec).cuda().bfloat16()
    out = torch.zeros_like(xd)
    ctx.full_step(xd, 0, [0], out, timestep=0.7, txt=td, pooled=vd)
    exp, feats = om.forward(x, 0.7, (txt, vec))
    assert max_abs_rel(out.cpu().numpy(), exp) <= 2e-2
    f = torch.empty((s.n_slots, 1, s.tokens, s.hidden), dtype=torch.bfloat16, device="cuda")
    ctx.forecast(1, [0], f)
    got = f.float().cpu().numpy()
    rng = np.random.default_rng(0)
    for j in range(s.n_slots):
        idx = (np.zeros(4000, np.int64), rng.integers(0, s.tokens, 4000), rng.integers(0, s.hidden, 4000))
        idx[1][:2] = [0, s.tokens - 1]; idx[2][:2] = [0, s.hidden - 1]
        assert np.max(np.abs(got[j][idx] - feats[j][idx])) <= 2e-2 * np.max(np.abs(feats[j])), j
    ctx.close()
