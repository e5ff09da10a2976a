"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the
same seeded inputs, step by step and end to end.

Bars: bit-exact for bytes, masks, histograms, LUTs, integer moments and flags;
1e-4 relative on the colour matrices; 1e-3 px mean EPE on the flow; 1 LSB
max-abs on every uint8 image.  (The kernels follow the oracle's operation
order, so in practice everything is bit-identical; the test also reports that.)
"""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2308_09209_amd import vstitch as V  # noqa: E402
from paper_2308_09209_amd.scenes import scene_for, small_scene  # noqa: E402
from tests.rigs import crop_rig, smooth_image  # noqa: E402
import bench  # noqa: E402

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def dev(frames):
    return [torch.from_numpy(np.ascontiguousarray(f)).to("cuda:0") for f in frames]


def lsb(a, b):
    return int(np.abs(a.astype(np.int64) - b.astype(np.int64)).max()) if a.size else 0


def check_steps(st, orc, label, full=True, flow=True):
    """Per-step parity of the last frame (the luma pyramid exists only when the
    flow is on)."""
    assert st.n_pairs == orc.n_pairs
    for p in range(orc.n_pairs):
        assert st.strip_box(p) == orc.strip_box(p), (label, p)
        if full:
            for s in (0, 1):
                np.testing.assert_array_equal(st.tap("strip", p, s), orc.tap("strip", p, s), err_msg=f"{label} strip {p}/{s}")
            np.testing.assert_array_equal(st.tap("mask", p), orc.tap("mask", p), err_msg=f"{label} mask {p}")
        np.testing.assert_array_equal(st.tap("hist", p), orc.tap("hist", p), err_msg=f"{label} hist {p}")
        np.testing.assert_array_equal(st.tap("lut", p), orc.tap("lut", p), err_msg=f"{label} lut {p}")
        np.testing.assert_array_equal(st.tap("mom", p), orc.tap("mom", p), err_msg=f"{label} mom {p}")
        if full and flow:
            for cam in (0, 1):
                a, b = st.tap("pyr", p, cam * 8), orc.tap("pyr", p, cam * 8)
                np.testing.assert_array_equal(a, b, err_msg=f"{label} luma {p}/{cam}")
            for lvl in range(st.info.lk_levels):
                need = orc.tap("need", p, lvl)
                np.testing.assert_array_equal(st.tap("need", p, lvl), need,
                                              err_msg=f"{label} flow domain {p}/{lvl}")
                # the plan's domain accounting (the benchmark's flop count)
                assert st.info.flow_px[p][lvl] == int(need.sum()), (label, p, lvl)
                assert st.info.flow_taps[p][lvl] == bench.domain_taps(need, st.params.lk_radius), (label, p, lvl)
        for d in (0, 1):
            a, b = st.tap("flow", p, d), orc.tap("flow", p, d)
            epe = np.sqrt(((a.astype(np.float64) - b) ** 2).sum(-1))
            assert epe.mean() <= 1e-3, (label, p, d, epe.mean(), epe.max())
            if epe.max() > 0:
                say(f"  {label} pair {p} dir {d}: flow not bit-exact, mean EPE {epe.mean():.2e} max {epe.max():.2e}")
    mp, mo = st.tap("mpair"), orc.tap("mpair")
    assert np.max(np.abs(mp - mo)) <= 1e-4 * max(1.0, np.max(np.abs(mo))), (label, mp, mo)
    mk, mko = st.tap("mk"), orc.tap("mk")
    assert np.max(np.abs(mk - mko)) <= 1e-4 * max(1.0, np.max(np.abs(mko))), label
    np.testing.assert_array_equal(st.tap("flags"), orc.tap("flags"))
    np.testing.assert_array_equal(st.tap("quant"), orc.tap("quant"))
    np.testing.assert_array_equal(st.tap("mbar"), orc.tap("mbar"))
    assert lsb(st.tap("bal_lut"), orc.tap("bal_lut")) <= 1, label
    np.testing.assert_array_equal(st.tap("cover"), (orc.tap("cover") > 0).astype(np.uint8))


def run_sequence(rig, frames_fn, n_frames, label, params=None, full=True):
    params = params or {}
    st = V.Stitcher(rig, debug_taps=1, **params)
    orc = O.Oracle(rig, **params)
    exact = 0
    for t in range(n_frames):
        frames = frames_fn(t)
        say(f"[{label}] frame {t}: canvas {orc.canvas} pairs {orc.n_pairs} params {params}")
        pano = st.stitch(dev(frames)).cpu().numpy()
        want = orc.stitch(frames)
        pre, pre_o = st.tap("pano_pre"), orc.tap("pano_pre")
        d_pre, d = lsb(pre, pre_o), lsb(pano, want)
        say(f"  pre-balance max diff {d_pre} LSB, final {d} LSB")
        assert d_pre <= 1 and d <= 1, (label, t, d_pre, d)
        np.testing.assert_array_equal(st.tap("pano_hist"), orc.tap("pano_hist")) if d_pre == 0 else None
        check_steps(st, orc, f"{label} t={t}", full=full, flow=params.get("flow", 1) != 0)
        exact += int(d == 0)
    say(f"[{label}] {exact}/{n_frames} frames bit-identical")
    st.close()


def test_parity_small_chain_with_drift():
    s = small_scene(n_cams=2, W=200, H=120, overlap=0.3, drift=0.05)
    run_sequence(s.rig(), s.frames, 4, "small chain")


def test_parity_small_ring():
    s = small_scene(n_cams=3, W=176, H=100, overlap=0.25, ring=True, drift=0.05)
    run_sequence(s.rig(), s.frames, 3, "small ring")


def test_parity_three_camera_chain_ragged_canvas():
    # canvas width 403 (not a multiple of 4): the byte-store path of the panorama
    s = small_scene(n_cams=3, W=151, H=77, overlap=0.33, drift=0.05)
    rig = s.rig()
    assert rig["canvas_w"] % 4 != 0
    run_sequence(rig, s.frames, 2, "3-cam ragged")


def test_parity_2x640x360_all_frames():
    s = scene_for("2x640x360_chain")
    run_sequence(s.rig(), s.frames, 8, "2x640x360")


@pytest.mark.parametrize("params", [dict(flow=0), dict(color_window=0), dict(balance=0),
                                    dict(color_window=1), dict(lk_levels=1, lk_iters=2),
                                    dict(lk_radius=2, lk_levels=3), dict(lk_iters=0),
                                    dict(lk_lambda=0.25, lambda_pct=10)])
def test_parity_options(params):
    s = small_scene(n_cams=2, W=180, H=100, overlap=0.3, drift=0.05)
    run_sequence(s.rig(), s.frames, 2, "options", params=params)


def test_identity_views_reproduce_texture_exactly():
    tex = smooth_image(96, 460, seed=11)
    rig, frames = crop_rig(tex, 192, 96, [(0, 0), (134, 0), (268, 0)])
    st = V.Stitcher(rig, balance=0)
    pano = st.stitch(dev(frames)).cpu().numpy()
    np.testing.assert_array_equal(pano, tex)
    for p in range(st.n_pairs):
        assert np.all(st.tap("flow", p, 0) == 0) and np.all(st.tap("flow", p, 1) == 0)


def test_identity_views_ring_exact():
    tex = smooth_image(64, 432, seed=12, periodic_x=True)
    rig, frames = crop_rig(tex, 180, 64, [(0, 0), (144, 0), (288, 0)], ring_period=432)
    st = V.Stitcher(rig, balance=0)
    np.testing.assert_array_equal(st.stitch(dev(frames)).cpu().numpy(), tex)


def test_geometry_errors():
    tex = smooth_image(20, 300, seed=3)
    rig, _ = crop_rig(tex, 100, 20, [(0, 0), (40, 0), (80, 0)])      # triple overlap
    with pytest.raises(V.VSError) as e:
        V.Stitcher(rig)
    assert e.value.status == -2
    rig, _ = crop_rig(tex, 100, 20, [(0, 0), (150, 0)])               # no overlap
    with pytest.raises(V.VSError) as e:
        V.Stitcher(rig)
    assert e.value.status == -2


def test_state_save_restore_and_host_state_io():
    """Stopping after frame 2, saving the colour state and resuming in a fresh
    context gives the same frames 3-4 as an uninterrupted run; so does
    passing the state through vs_stitch's in/out arguments."""
    s = small_scene(n_cams=3, W=150, H=90, overlap=0.3, drift=0.08)
    rig = s.rig()
    a = V.Stitcher(rig)
    ref = [a.stitch(dev(s.frames(t))).cpu().numpy() for t in range(5)]
    b = V.Stitcher(rig)
    for t in range(3):
        b.stitch(dev(s.frames(t)))
    saved = V.state_bytes(b.state_get())
    assert b.state_get().frames_seen == 3
    b.close()
    c = V.Stitcher(rig)
    c.state_set(V.state_from_bytes(saved))
    for t in (3, 4):
        np.testing.assert_array_equal(c.stitch(dev(s.frames(t))).cpu().numpy(), ref[t])
    d = V.Stitcher(rig)
    state = None
    for t in range(5):
        pano, state, info = d.stitch(dev(s.frames(t)), state_in=state, want_state=True, want_info=True)
        np.testing.assert_array_equal(pano.cpu().numpy(), ref[t])
        assert info.frames_seen == t + 1 and state.frames_seen == t + 1
    bad = V.state_from_bytes(saved)
    bad.version = 99
    with pytest.raises(V.VSError) as e:
        d.state_set(bad)
    assert e.value.status == -5


def test_deterministic_runs():
    s = small_scene(n_cams=2, W=200, H=120, overlap=0.3, drift=0.05)
    outs = []
    for _ in range(2):
        st = V.Stitcher(s.rig())
        outs.append([st.stitch(dev(s.frames(t))).cpu().numpy() for t in range(3)])
        st.close()
    for a, b in zip(*outs):
        np.testing.assert_array_equal(a, b)


def test_timing_reports_steps():
    s = small_scene(n_cams=2, W=200, H=120, overlap=0.3)
    st = V.Stitcher(s.rig())
    st.set_timing(True)
    for t in range(70):   # more frames than the event ring holds
        st.stitch(dev(s.frames(t % 3)))
    ms, n = st.timing()
    assert n == 70
    assert np.all(ms >= 0) and ms[5] >= ms[:5].sum() * 0.99 and ms[2] > 0


def test_parity_4x1920x1080_ring_full_size():
    """The headline workload at full size (the launch configuration the
    benchmark times): frames 0-2, the first full three-frame window of eqs.
    (2)-(3) and (6)-(7), every output pixel and step against the oracle."""
    s = scene_for("4x1920x1080_ring")
    rig = s.rig()
    st = V.Stitcher(rig, debug_taps=1)
    orc = O.Oracle(rig)
    for t in range(3):
        frames = s.frames(t)
        say(f"[4x1080p ring] frame {t}")
        pano = st.stitch(dev(frames)).cpu().numpy()
        want = orc.stitch(frames)
        d = lsb(pano, want)
        say(f"  final max diff {d} LSB, identical px {np.mean(np.all(pano == want, -1)):.6f}")
        assert d <= 1
        deferred = [int(st.tap("deferred", 0, lvl)[0]) for lvl in range(st.info.lk_levels)]
        say(f"  flow pixels finished by the tail kernel per level: {deferred}")
        check_steps(st, orc, f"4x1080p t={t}", full=True)
        assert st.state_get().frames_seen == t + 1
    st.close()


def test_deferred_flow_pixels_match_oracle():
    """Residual displacements of up to 12 px per camera: flow pixels leave the
    staged tile and finish in the tail kernel (16 lanes per pixel, the sums
    handed down the row lanes, or, with VS_FLOW_INBLOCK, in their own block);
    the flows of every pair and direction bit for bit against the oracle, for
    the staged kernel + tail, the staged kernel finishing its own deferred
    pixels, and the generic kernel, which finishes every pixel itself."""
    sc = small_scene(n_cams=3, W=320, H=160, overlap=0.3, ring=True, seed_config=95, resid=12.0)
    orc = O.Oracle(sc.rig())
    frames = sc.frames(0)
    want = orc.stitch(frames)
    for variant in (4, 11, 28, 25, 0):
        st = V.Stitcher(sc.rig(), debug_taps=1)
        for lvl in range(st.info.lk_levels):
            st.set_flow_variant(lvl, variant)
        pano = st.stitch(dev(frames)).cpu().numpy()
        deferred = [int(st.tap("deferred", 0, lvl)[0]) for lvl in range(st.info.lk_levels)]
        say(f"[12 px residuals, flow variant {variant}] pixels finished by the tail kernel per level: {deferred}, "
            f"panorama max diff {lsb(pano, want)} LSB")
        if variant in (4, 11):
            assert deferred[0] > 0
        else:   # finished in-block or by the generic kernel: no queue
            assert sum(deferred) == 0
        for p in range(orc.n_pairs):
            for d in (0, 1):
                np.testing.assert_array_equal(st.tap("flow", p, d), orc.tap("flow", p, d),
                                              err_msg=f"variant {variant} pair {p} dir {d}")
        assert lsb(pano, want) <= 1
        st.close()


# (the last line's level 0: 1 px per thread, but 601 x 700: 3; 2 and 4 in the test after it)
@pytest.mark.parametrize("w,h,scale,lam,iters", [
    (2, 2, 1.0, 256.0, 5), (17, 5, 1.0, 256.0, 5), (64, 117, 1.0, 1e-3, 6), (120, 125, 1.0, 256.0, 5),   # 4 lanes
    (65, 33, 1e-22, 256.0, 5), (65, 33, 1e12, 1e-12, 5), (97, 61, 1.0, 256.0, 1),      # the plain division
    (121, 125, 1.0, 1e-3, 5), (250, 150, 1.0, 256.0, 5),                               # gradients held
    (251, 150, 1.0, 1e-3, 5), (600, 260, 1e-22, 256.0, 4), (601, 700, 1.0, 1e-3, 5)])  # general, 1 to 4 px per thread
def test_flow_forms_by_level_size_match_oracle(w, h, scale, lam, iters):
    """Level sizes on both sides of each form of the flow kernel, weak
    regularisation (displacements that leave the staged tile) and luma scales
    whose quotients the shortened division does not take: both flows bit for bit
    against the oracle."""
    rng = np.random.default_rng(w * 1000 + h)
    T = np.clip(np.cumsum(rng.normal(size=(h, w)), axis=1) * 12 + 128, 0, 255).round().astype(np.float32)
    M = np.clip(np.roll(T, (1, 2), axis=(0, 1)) + rng.normal(size=T.shape) * 3, 0, 255).round().astype(np.float32)
    T, M = (T * np.float32(scale)).astype(np.float32), (M * np.float32(scale)).astype(np.float32)

    def pyr(a):
        out = [a]
        for _ in range(3):
            out.append(O.pyr_down(out[-1]))
        return out
    say(f"[flow {w}x{h}] scale {scale} lambda {lam} steps {iters}")
    a, b = V.PlainFlow(w, h, lk_lambda=lam, lk_iters=iters)(torch.from_numpy(T).cuda(), torch.from_numpy(M).cuda())
    lf = np.float32(lam)
    np.testing.assert_array_equal(a.cpu().numpy(), O.pyramid_flow(pyr(T), pyr(M), iters=iters, lam=lf))
    np.testing.assert_array_equal(b.cpu().numpy(), O.pyramid_flow(pyr(M), pyr(T), iters=iters, lam=lf))


@pytest.mark.parametrize("w,h,px", [(641, 380, 2), (601, 420, 2), (705, 600, 3), (1001, 529, 4)])
@pytest.mark.parametrize("scale,lam", [(1.0, 1e-3), (1.0, 256.0), (1e-22, 256.0), (1e12, 1e-12), ("stripes", 256.0)])
def test_flow_forms_of_2_to_4_px_per_thread_match_oracle(w, h, px, scale, lam):
    """The default forms with 2, 3 and 4 pixels per thread at level 0 (from 512, 768 and
    1024 tiles of 64 x 16 pixels of both fields): deferred pixels, lumas whose quotients
    the shortened division does not take, and stripes of such lumas beside ordinary ones in
    one wavefront; both flows bit for bit against the oracle."""
    n16 = 2 * -(-w // 64) * -(-h // 16)
    assert px == (4 if n16 >= 1024 else 3 if n16 >= 768 else 2) and n16 >= 512
    rng = np.random.default_rng(w + h)
    T = np.clip(np.cumsum(rng.normal(size=(h, w)), axis=1) * 12 + 128, 0, 255).round().astype(np.float32)
    M = np.clip(np.roll(T, (1, 2), axis=(0, 1)) + rng.normal(size=T.shape) * 3, 0, 255).round().astype(np.float32)
    k = np.where(np.arange(w) // 24 % 2, 1e-22, 1.0) if scale == "stripes" else scale
    T, M = ((a * np.float32(1) * k).astype(np.float32) for a in (T, M))

    def pyr(a):
        out = [a]
        for _ in range(3):
            out.append(O.pyr_down(out[-1]))
        return out
    say(f"[flow {w}x{h}, {px} px per thread] scale {scale} lambda {lam}")
    a, b = V.PlainFlow(w, h, lk_lambda=lam)(torch.from_numpy(T).cuda(), torch.from_numpy(M).cuda())
    it, lf = V.default_params().lk_iters, np.float32(lam)
    np.testing.assert_array_equal(a.cpu().numpy(), O.pyramid_flow(pyr(T), pyr(M), iters=it, lam=lf))
    np.testing.assert_array_equal(b.cpu().numpy(), O.pyramid_flow(pyr(M), pyr(T), iters=it, lam=lf))


@pytest.mark.parametrize("w,h,levels,off", [(5, 3, 1, 0), (17, 9, 2, 1), (64, 16, 4, 2), (129, 33, 4, 3), (1500, 801, 3, 1)])
def test_pair_in_and_out(w, h, levels, off):
    """A luma pair at any word alignment, sizes with and without remainders of the
    copies' words, one level and several, twice on one context: levels 0 and 1 and the
    two flows are the ones of aligned images and of the oracle, words outside the
    outputs stay, and outputs may be left out."""
    rng = np.random.default_rng(w)
    pf = V.PlainFlow(w, h, lk_levels=levels)
    say(f"[pair {w}x{h}] levels {levels} offset {off}")
    for _ in range(2):
        T, M = (rng.integers(0, 256, (h, w)).astype(np.float32) for _ in range(2))
        want = [t.cpu().numpy().ravel() for t in pf(torch.from_numpy(T).cuda(), torch.from_numpy(M).cuda())]
        src = [torch.zeros(h * w + 8, device="cuda") for _ in range(2)]
        for buf, a in zip(src, (T, M)):
            buf[off:off + h * w] = torch.from_numpy(a.ravel()).cuda()
        for use in ((1, 1), (1, 0), (0, 1)):
            dst = [torch.full((2 * h * w + 8,), -7.0, device="cuda") for _ in range(2)]
            ptr = [V._p(d[off:]) if u else None for d, u in zip(dst, use)]
            V.check(V.lib().vs_flow_run(pf.hnd, V._p(src[0][off:]), V._p(src[1][off:]), *ptr, V._stream_handle(None)),
                    "vs_flow_run")
            for d, u, f in zip(dst, use, want):
                got = d.cpu().numpy()
                out = np.full_like(got, -7.0)
                if u:
                    out[off:off + 2 * h * w] = f
                np.testing.assert_array_equal(got, out)
        for l in range(min(levels, 2)):
            for got, a in zip(pf.level(l), (T, M)):
                np.testing.assert_array_equal(got.cpu().numpy(), a if l == 0 else O.pyr_down(a))


@pytest.mark.parametrize("rows", [8, 16])
def test_fused_pyramid_tile_heights(rows):
    """levels 0-2 in one pass at either level-2 tile height: every pyramid
    level of both cameras and the panorama bit for bit against the oracle
    (plain flow), and the fallback path's rebuild of the levels for pairs not
    kept (threshold 0: none kept) equal to the plain path's panorama"""
    s = small_scene(n_cams=3, W=400, H=240, overlap=0.3, ring=True, seed_config=93, drift=0.02)
    rig = s.rig()
    st = V.Stitcher(rig, pyr_tile_rows=rows)
    orc = O.Oracle(rig)
    for t in range(2):
        pano = st.stitch(dev(s.frames(t))).cpu().numpy()
        want = orc.stitch(s.frames(t))
        say(f"[pyramid tiles {rows} rows] frame {t}: max |gpu - oracle| {lsb(pano, want)} LSB")
        assert np.array_equal(pano, want), t
        for p in range(st.n_pairs):
            for cam in (0, 1):
                for lvl in range(st.info.lk_levels):
                    np.testing.assert_array_equal(st.tap("pyr", p, cam * 8 + lvl), orc.tap("pyr", p, cam * 8 + lvl),
                                                  err_msg=f"rows {rows} pair {p} cam {cam} level {lvl}")
    from paper_2308_09209_amd import scenes as S
    fb = V.Stitcher(rig, pyr_tile_rows=rows)
    fb.load_weights(S.nn_blob(*S.random_net(31)))
    fb.set_flow_mode(V.FLOW_SURROGATE_FALLBACK, 0.0)
    ref = V.Stitcher(rig, pyr_tile_rows=rows)
    for t in range(2):
        a = fb.stitch(dev(s.frames(t))).cpu().numpy()
        b = ref.stitch(dev(s.frames(t))).cpu().numpy()
        assert np.array_equal(a, b), t


def test_pyramid_tile_height_parameter_is_checked():
    s = small_scene(n_cams=2, W=160, H=96, overlap=0.3)
    with pytest.raises(V.VSError):
        V.Stitcher(s.rig(), pyr_tile_rows=12)
