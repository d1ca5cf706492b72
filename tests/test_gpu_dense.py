"""Rho maps in the matrix-core form against the oracle and against the forms
it stands in for, at the edges of its tiles and passes.

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
