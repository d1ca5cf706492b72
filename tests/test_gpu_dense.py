"""Rho maps in the matrix-core form, and top-k lists found with its filter,
against the oracle and against the forms they stand in for, at the edges of
tiles and passes.

SNCC_TEST_DENSE=1 takes the matrix-core form wherever it is possible, 0 never.
Tolerances as everywhere: FP32 rho within 1e-5 of the oracle, FP64 within
1e-9; the uniform-window flags are the same in both forms.
"""

import numpy as np
import pytest

import oracle as O
from workloads import synth

from gpu_util import build_sats

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import paper_2502_01286_amd as S
    return S


@pytest.fixture(scope="module")
def ctx(S):
    import torch
    torch.cuda.init()
    c = S.sncc_ctx_create(0)
    yield c
    S.sncc_ctx_destroy(c)


def _case(seed, M, N, W, H, kind):
    """Frame with a flat patch (uniform windows) and a template."""
    f = synth.scene(seed, M, N)
    f[: min(N, H + 3), : min(M, W + 5)] = 77
    rng = np.random.default_rng(seed + 1)
    x, y = int(rng.integers(0, M - W + 1)), int(rng.integers(0, N - H + 1))
    t = f[y:y + H, x:x + W].astype(np.int64) + rng.integers(-20, 21, (H, W))
    if kind == "spike":  # one bright pixel on a nearly flat ground: four digits in FP32
        t = 20 + rng.integers(0, 2, (H, W))
        t[H // 2, W // 3] = 255
    return f, np.clip(t, 0, 255).astype(np.uint8)


# (M, N, W, H): one-pixel rows and columns, offsets at 1, 127, 128, 129 and
# 257 columns, rows at and around the tiles' 16, 32 and 64, widths around the
# 16-pixel groups, heights around the 8-row steps, a table pitch of exactly
# M + 1, several passes over a tall and over a wide template, windows of more
# than one exact box of squares
SIZES = [(40, 30, 1, 9), (40, 30, 9, 1), (20, 20, 20, 20), (143, 31, 17, 16), (144, 47, 17, 15),
         (145, 48, 17, 17), (191, 90, 64, 25), (320, 97, 63, 33), (321, 160, 65, 97),
         (300, 700, 20, 520), (900, 60, 520, 30), (420, 400, 300, 300), (1023, 140, 31, 12)]


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("kind", ["crop", "spike"])
def test_dense_map(S, ctx, monkeypatch, size, kind):
    import torch
    M, N, W, H = size
    if kind == "spike" and W * H < 64:
        pytest.skip("the spike is not small against the template")
    f, t = _case(M + N, M, N, W, H, kind)
    sigma = 2.0 if kind == "crop" else 0.7  # a single spike must not pass as uniform
    segs, _, _ = S.sncc_segment_template(t, sigma)
    ta = O.precompute_template_approximation(t, sigma)
    want = O.rho_map(f, ta)
    _, s, s2 = build_sats(S, ctx, [f])
    tm = S.sncc_upload_templates(ctx, [segs], [W], [H])
    nu, nv = M - W + 1, N - H + 1
    for prec, dt, tol in ((S.SNCC_FP32_KAHAN, torch.float32, 1e-5),
                          (S.SNCC_FP64, torch.float64, 1e-9)):
        got = []
        for form in "01":
            print("case", size, kind, prec, "form", form, flush=True)
            monkeypatch.setenv("SNCC_TEST_DENSE", form)
            rho = torch.full((nv, nu + 3), 7.0, dtype=dt, device="cuda")
            deg = torch.full((nv, nu + 3), 9, dtype=torch.uint8, device="cuda")
            S.sncc_score(ctx, tm, 0, s[0], s2[0], M, N, prec, rho, deg)
            S.sncc_sync(ctx)
            r, d = rho.cpu().numpy(), deg.cpu().numpy()
            assert (r[:, nu:] == 7).all() and (d[:, nu:] == 9).all()  # nothing past the map
            assert np.abs(r[:, :nu] - want).max() <= tol, (prec, form)
            got.append(d[:, :nu])
        assert (got[0] == got[1]).all()
    S.sncc_tmpl_destroy(tm)


@pytest.mark.parametrize("rows", [16 * 23, 32 * 40, 64 * 38])
def test_dense_map_launch_shapes(S, ctx, monkeypatch, rows):
    """Frames whose tile counts choose two, four and eight rows per wave half:
    both forms agree everywhere."""
    import torch
    M, N, W, H = 1920 + 39, rows + 22, 40, 23
    f, t = _case(rows, M, N, W, H, "crop")
    segs, _, _ = S.sncc_segment_template(t, 3.0)
    _, s, s2 = build_sats(S, ctx, [f])
    tm = S.sncc_upload_templates(ctx, [segs], [W], [H])
    for prec, dt, tol in ((S.SNCC_FP32_KAHAN, torch.float32, 2e-5),
                          (S.SNCC_FP64, torch.float64, 2e-9)):
        got = []
        for form in "01":
            print("case", rows, prec, "form", form, flush=True)
            monkeypatch.setenv("SNCC_TEST_DENSE", form)
            rho = torch.zeros((N - H + 1, M - W + 1), dtype=dt, device="cuda")
            S.sncc_score(ctx, tm, 0, s[0], s2[0], M, N, prec, rho)
            S.sncc_sync(ctx)
            got.append(rho)
        assert float((got[0] - got[1]).abs().max()) <= tol
    S.sncc_tmpl_destroy(tm)


# one-pass templates and their neighbours: heights at the 16-bit sums' limit of
# 257 rows and past it, regions near the LDS limit, odd frame pitches, one
# offset row and column
@pytest.mark.parametrize("size", SIZES[:9] + [(90, 400, 12, 257), (90, 400, 12, 258),
                                              (700, 40, 500, 8), (641, 479, 31, 33),
                                              (1921, 1081, 64, 64), (200, 180, 180, 170)])
def test_dense_frame(S, ctx, monkeypatch, size):
    """The map straight from the frame: rho against the oracle, flags and
    energies exactly."""
    import torch
    M, N, W, H = size
    f, t = _case(M * 3 + N, M, N, W, H, "crop")
    if M * N < 1 << 20:
        f[N // 2:] |= 0xF0  # bright rows: the largest sums
    segs, _, _ = S.sncc_segment_template(t, 2.0)
    ta = O.precompute_template_approximation(t, 2.0)
    tm = S.sncc_upload_templates(ctx, [segs], [W], [H])
    nu, nv = M - W + 1, N - H + 1
    vv, uu = np.meshgrid(np.arange(nv), np.arange(nu), indexing="ij")
    tables = O.sum_tables(f)
    _, _, V = O.window_sums(*tables, W, H, uu, vv)
    d = torch.from_numpy(np.ascontiguousarray(f)).cuda()
    for form in "01":
        print("case", size, "form", form, flush=True)
        monkeypatch.setenv("SNCC_TEST_DENSE", form)
        rho = torch.full((nv, nu + 3), 7.0, dtype=torch.float32, device="cuda")
        deg = torch.full((nv, nu + 3), 9, dtype=torch.uint8, device="cuda")
        en = torch.full((nv, nu + 3), -1, dtype=torch.int64, device="cuda")
        S.sncc_score_frame(ctx, tm, 0, d, rho, form=S.SNCC_FORM_GLOBAL, degen=deg, energy=en)
        S.sncc_sync(ctx)
        r, g, e = rho.cpu().numpy(), deg.cpu().numpy(), en.cpu().numpy()
        assert (r[:, nu:] == 7).all() and (g[:, nu:] == 9).all() and (e[:, nu:] == -1).all()
        assert np.array_equal(e[:, :nu], V) and np.array_equal(g[:, :nu], V == 0)
        us, vs = (uu, vv) if M * N < 1 << 20 else (uu[::37, ::5], vv[::37, ::5])
        want = O.rho_at(*tables, ta, us.ravel(), vs.ravel()).reshape(us.shape)
        assert np.abs(r[vs, us] - want).max() <= 1e-5
    S.sncc_tmpl_destroy(tm)


def test_fp64_map_under_capture(S, monkeypatch):
    """An FP64 map captured before its operands exist, and one after: both
    graphs replay to the oracle's map."""
    import torch
    M, N, W, H = 200, 120, 24, 20
    f, t = _case(5, M, N, W, H, "crop")
    want = O.rho_map(f, O.precompute_template_approximation(t, 2.0))
    segs, _, _ = S.sncc_segment_template(t, 2.0)
    monkeypatch.setenv("SNCC_TEST_DENSE", "1")
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        c = S.sncc_ctx_create(0, st.cuda_stream)
        _, s, s2 = build_sats(S, c, [f])
        tm = S.sncc_upload_templates(c, [segs], [W], [H])
        rho = torch.zeros((N - H + 1, M - W + 1), dtype=torch.float64, device="cuda")
        st.synchronize()
        for _ in range(2):
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=st):
                S.sncc_score(c, tm, 0, s[0], s2[0], M, N, S.SNCC_FP64, rho)
            for _ in range(3):
                rho.fill_(7.0)
                g.replay()
                st.synchronize()
                assert np.abs(rho.cpu().numpy() - want).max() <= 1e-9
            S.sncc_score(c, tm, 0, s[0], s2[0], M, N, S.SNCC_FP64, rho)  # builds the operands
            st.synchronize()
        S.sncc_tmpl_destroy(tm)
        S.sncc_ctx_destroy(c)


def _lists(S, ctx, monkeypatch, form, frames, segs, W, H, pairs, k, prec):
    import torch
    monkeypatch.setenv("SNCC_TEST_DENSE", form)
    B, N, M = len(frames), frames[0].shape[0], frames[0].shape[1]
    _, s, s2 = build_sats(S, ctx, frames)
    tm = S.sncc_upload_templates(ctx, segs, W, H)
    out = torch.full((len(pairs), k, 3), 5, dtype=torch.int32, device="cuda")
    for _ in range(2):  # the second call reuses the plan
        out.fill_(5)
        S.sncc_topk(ctx, tm, s, s2, B, M, N, pairs, k, prec, out)
    S.sncc_sync(ctx)
    S.sncc_tmpl_destroy(tm)
    return out.cpu().numpy()


def _segments(S, t, sigma):
    """Segments at sigma, or below it where that leaves a uniform approximation."""
    while True:
        try:
            return S.sncc_segment_template(t, sigma, t.size)[0]
        except S.SnccError as e:
            assert e.code == S.SNCC_EDEGENERATE and sigma > 1e-3
            sigma *= 0.5


def _frames(kind, M, N):
    if kind == "scene":
        f = synth.scene(M, M, N)
        f[:60, :70] = 90
    elif kind == "uniform":  # every rho 0: the first offsets
        f = np.full((N, M), 31, np.uint8)
    elif kind == "periodic":  # thousands of equal best offsets
        y, x = np.mgrid[0:N, 0:M]
        f = ((x % 7) * 25 + (y % 5) * 13).astype(np.uint8)
    else:  # nearly uniform windows everywhere
        f = np.full((N, M), 100, np.uint8)
        f[np.random.default_rng(3).random((N, M)) < 2e-3] = 101
    return [f, f[::-1].copy()]


@pytest.mark.parametrize("kind", ["scene", "uniform", "periodic", "lowvar"])
@pytest.mark.parametrize("k", [1, 5, 64])
def test_filtered_topk_is_the_direct_topk(S, ctx, monkeypatch, kind, k):
    """Top-k lists with the filter equal, bit for bit in FP32 and in offsets
    and reported rho in FP64, the lists without it: templates of one and
    several LDS passes, of four digits, with windows of more than one exact box
    of squares and as large as the frame; frames whose candidates are few, all
    equal, too many, or of nearly uniform windows."""
    M, N = 420, 330
    frames = _frames(kind, M, N)
    rng = np.random.default_rng(11)
    scene = synth.scene(8, M, N)
    segs, W, H = [], [], []
    for w, h, sigma in ((9, 11, 3), (40, 37, 2), (64, 150, 2), (300, 250, 8), (33, 8, 4),
                        (M, N, 20), (30, 31, 0.7)):
        y, x = int(rng.integers(0, N - h + 1)), int(rng.integers(0, M - w + 1))
        t = frames[0][y:y + h, x:x + w].astype(int) if kind != "uniform" else \
            scene[y:y + h, x:x + w].astype(int)
        t = np.clip(t + rng.integers(-9, 10, t.shape), 0, 255)
        if sigma == 0.7:  # four digits
            t = 20 + rng.integers(0, 2, t.shape)
            t[3, 4] = 255
        if t.std() <= sigma * 1.05:  # no template may be uniform
            sigma = float(t.std()) * 0.5
        segs.append(_segments(S, t.astype(np.uint8), sigma))
        W.append(w)
        H.append(h)
    pairs = [(f, t) for f in (1, 0) for t in range(len(segs))]
    for prec in (S.SNCC_FP32_KAHAN, S.SNCC_FP64):
        print("case", kind, k, prec, flush=True)
        got = _lists(S, ctx, monkeypatch, "1", frames, segs, W, H, pairs, k, prec)
        want = _lists(S, ctx, monkeypatch, "0", frames, segs, W, H, pairs, k, prec)
        if prec == S.SNCC_FP64 and kind == "lowvar":
            # sums of a few doubles in another order: the reported floats
            assert np.allclose(got[..., 2].view(np.float32), want[..., 2].view(np.float32),
                               rtol=0, atol=1e-6, equal_nan=False) or (got == want).all()
        else:
            bad = np.argwhere((got != want).any(axis=(1, 2)))[:, 0]
            assert bad.size == 0, [(pairs[b], got[b][:3].tolist(), want[b][:3].tolist())
                                   for b in bad[:3]]


def test_fp32_lists_of_both_forms_in_one_call(S, ctx, monkeypatch):
    """A call by rule (detailed templates filtered, coarse ones not) gives the
    lists of the segment form."""
    M, N = 1280, 720
    f = synth.scene(77, M, N)
    rng = np.random.default_rng(78)
    segs, W, H = [], [], []
    for w, h, sigma in ((64, 64, 3), (128, 96, 16), (90, 31, 4), (150, 140, 12), (20, 24, 2)):
        t, _, _ = synth.crop_template(rng, f, w, h, sigma_max=sigma)
        a, _, _ = S.sncc_segment_template(t, sigma)
        segs.append(a)
        W.append(w)
        H.append(h)
    pairs = [(0, t) for t in range(5)]
    for k in (1, 10):
        print("case", k, flush=True)
        got = _lists(S, ctx, monkeypatch, "", [f], segs, W, H, pairs, k, S.SNCC_FP32_KAHAN)
        want = _lists(S, ctx, monkeypatch, "0", [f], segs, W, H, pairs, k, S.SNCC_FP32_KAHAN)
        assert (got == want).all()


@pytest.mark.parametrize("M", [420, 640 + 33])
def test_filtered_batch_is_the_direct_batch(S, ctx, monkeypatch, M):
    """A batch with the filter for all its pairs, with none, and by rule gives
    the same lists, refined matches and counts, also in the last tile columns
    that a second launch scores."""
    import torch
    N, k = 300, 12
    frames = [synth.scene(40 + i, M, N) for i in range(3)]
    rng = np.random.default_rng(41)
    coarse, fine, W, H = [], [], [], []
    for w, h in ((21, 30), (33, 33), (64, 90), (150, 40), (40, 24)):
        t, _, _ = synth.crop_template(rng, frames[len(W) % 3], w, h, sigma_max=9)
        coarse.append(S.sncc_segment_template(t, 9)[0])
        fine.append(S.sncc_segment_template(t, 3)[0])
        W.append(w)
        H.append(h)
    pairs = [(f, t) for f in range(3) for t in range(5)]
    got = []
    for form in ("0", "1", ""):
        print("case", M, "form", form, flush=True)
        monkeypatch.setenv("SNCC_TEST_DENSE", form)
        f = torch.from_numpy(np.stack(frames)).cuda()
        s = torch.zeros((3, N + 1, S.sncc_sat_pitch(M)), dtype=torch.int32, device="cuda")
        s2 = torch.zeros_like(s)
        ct = S.sncc_upload_templates(ctx, coarse, W, H)
        ft = S.sncc_upload_templates(ctx, fine, W, H)
        top = torch.zeros((len(pairs), k, 3), dtype=torch.int32, device="cuda")
        best = torch.zeros((len(pairs), 4), dtype=torch.int32, device="cuda")
        count = torch.zeros(len(pairs), dtype=torch.int32, device="cuda")
        b = S.sncc_batch_create(ctx, ct, s, s2, 3, M, N, pairs, k, top, fine=ft, radius=2,
                                best_out=best, count_out=count, frames=f)
        one = []
        for _ in range(3):  # replays with the program's own work between them
            for x in (top, best, count):
                x.fill_(3)
            b.run()
            S.sncc_sync(ctx)
            one.append([x.cpu().numpy() for x in (top, best, count)])
        for x in one[1:]:
            assert all((p == q).all() for p, q in zip(one[0], x))
        got.append(one[0])
        b.destroy()
        S.sncc_tmpl_destroy(ct)
        S.sncc_tmpl_destroy(ft)
    for x in got[1:]:
        assert all((p == q).all() for p, q in zip(got[0], x))


def test_batch_outlives_its_templates(S, ctx, monkeypatch):
    """A batch owns what its launches read of the coarse set: runs after the
    set is destroyed, and others have taken its memory, give the same lists."""
    import torch
    M, N, k = 400, 300, 6
    f = synth.scene(70, M, N)
    rng = np.random.default_rng(71)
    temps = [synth.crop_template(rng, f, w, h, sigma_max=6)[0] for w, h in ((30, 40), (64, 50))]
    segs = [S.sncc_segment_template(t, 6)[0] for t in temps]
    W, H = [30, 64], [40, 50]
    monkeypatch.setenv("SNCC_TEST_DENSE", "1")
    _, s, s2 = build_sats(S, ctx, [f])
    d = torch.from_numpy(f[None]).cuda()
    ct = S.sncc_upload_templates(ctx, segs, W, H)
    top = torch.zeros((2, k, 3), dtype=torch.int32, device="cuda")
    b = S.sncc_batch_create(ctx, ct, s, s2, 1, M, N, [(0, 0), (0, 1)], k, top,
                            frames=d)
    b.run()
    S.sncc_sync(ctx)
    want = top.clone()
    S.sncc_tmpl_destroy(ct)
    others = [S.sncc_upload_templates(ctx, segs[::-1], W[::-1], H[::-1]) for _ in range(8)]
    top.zero_()
    b.run()
    S.sncc_sync(ctx)
    assert torch.equal(top, want) and int(want[0, 0, 0]) >= 0
    b.destroy()
    for o in others:
        S.sncc_tmpl_destroy(o)


@pytest.mark.parametrize("size", [(160, 120), (512, 333), (1920, 700)])
@pytest.mark.parametrize("cand_cap", [1 << 20, 1000])
def test_filtered_threshold_search_is_the_direct_one(S, ctx, monkeypatch, size, cand_cap):
    """The two-threshold search with the slow pass behind the filter finds the
    same survivors and matches as without, thresholds at and between the
    offsets' own values, uniform windows among them, also where the survivor
    list overflows; its replays too."""
    import torch
    M, N = size
    frames = [synth.scene(80 + i, M, N) for i in range(2)]
    frames[1][: N // 3, : M // 2] = 50  # uniform windows: rho is 0 there
    rng = np.random.default_rng(M)
    temps = [synth.crop_template(rng, frames[0], w, h, sigma_max=9)[0]
             for w, h in ((33, 25), (64, 61), (90, 100), (17, 48))]
    fast = [S.sncc_segment_template(t, 9)[0] for t in temps]
    slow = [S.sncc_segment_template(t, 2)[0] for t in temps]
    W, H = [t.shape[1] for t in temps], [t.shape[0] for t in temps]
    _, s, s2 = build_sats(S, ctx, frames)
    pairs = [(1, 3), (0, 0), (1, 1), (0, 2), (1, 0)]
    for lo, hi in ((0.1, 0.3), (-2.0, 0.0), (0.2, -2.0)):
        got = []
        for form in "01":
            print("case", size, cand_cap, lo, hi, "form", form, flush=True)
            monkeypatch.setenv("SNCC_TEST_DENSE", form)
            ft = S.sncc_upload_templates(ctx, fast, W, H)
            st = S.sncc_upload_templates(ctx, slow, W, H)
            cand = torch.zeros((cand_cap, 6), dtype=torch.int32, device="cuda")
            out = torch.zeros((1 << 20, 6), dtype=torch.int32, device="cuda")
            counts = torch.zeros(2, dtype=torch.int32, device="cuda")
            for _ in range(2):
                S.sncc_threshold_match(ctx, ft, st, np.full(4, lo), np.full(4, hi), s, s2, 2, M, N,
                                       pairs, cand, out, counts)
                S.sncc_sync(ctx)
                nc, nm = (int(x) for x in counts.cpu())
                c = S.decode_hits(cand, min(nc, cand_cap))
                o = np.sort(S.decode_hits(out, min(nm, 1 << 20)), order=["pair", "v", "u"])
                got.append((nc, nm, np.sort(c, order=["pair", "v", "u"]), o))
            S.sncc_tmpl_destroy(ft)
            S.sncc_tmpl_destroy(st)
        for g in got[1:]:
            assert g[0] == got[0][0] > 0
            if g[0] > cand_cap:  # which survivors are listed depends on timing
                assert len(g[2]) == cand_cap
                continue
            assert g[1] == got[0][1]
            for f in ("pair", "u", "v"):
                assert np.array_equal(g[2][f], got[0][2][f])
            if g[1] <= 1 << 20:
                for f in ("pair", "u", "v"):
                    assert np.array_equal(g[3][f], got[0][3][f])
                assert np.abs(g[3]["rho"] - got[0][3]["rho"]).max(initial=0) <= 1e-12
