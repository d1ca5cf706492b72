"""Frames on which the filter of a top-k search decides nothing (uniform ones,
repeated patterns): the pairs left to the segment form cost that form's time
and the filter's, not a multiple of it, and give its lists."""

import numpy as np
import pytest

from workloads import synth

from gpu_util import build_sats

pytestmark = pytest.mark.gpu

M, N, B, K = 1280 + 40, 720, 2, 5


def _frame(kind):
    if kind == "uniform":
        return np.full((N, M), 31, np.uint8)
    f = np.full((N, M), 240, np.uint8)  # rows of one glyph
    g = np.random.default_rng(4).integers(0, 2, (12, 8))
    for y in range(20, N - 40, 40):
        for x in range(20, M - 40, 16):
            f[y:y + 12, x:x + 8] = np.where(g > 0, 30, 240)
    return f


@pytest.mark.parametrize("kind", ["uniform", "glyphs"])
@pytest.mark.parametrize("batch", [False, True])
def test_undecided_pairs_cost_the_segment_form(monkeypatch, kind, batch):
    import torch
    import paper_2502_01286_amd as S
    torch.cuda.init()
    ctx = S.sncc_ctx_create(0)
    f = _frame(kind)
    src = synth.scene(3, M, N) if kind == "uniform" else f
    rng = np.random.default_rng(7)
    segs, W, H = [], [], []
    for w, h in ((40, 40), (64, 64), (96, 96), (33, 70)):
        x, y = int(rng.integers(0, M - w)), int(rng.integers(60, N - h))
        t = np.clip(src[y:y + h, x:x + w].astype(int) + rng.integers(-9, 10, (h, w)), 0, 255)
        segs.append(S.sncc_segment_template(t.astype(np.uint8), 4)[0])
        W.append(w)
        H.append(h)
    pairs = [(b, t) for b in range(B) for t in range(len(W))]
    d, s, s2 = build_sats(S, ctx, [f, f[::-1]])
    got, ms = [], []
    try:
        for form in ("0", ""):
            monkeypatch.setenv("SNCC_TEST_DENSE", form)
            tm = S.sncc_upload_templates(ctx, segs, W, H)
            top = torch.zeros((len(pairs), K, 3), dtype=torch.int32, device="cuda")
            b = S.sncc_batch_create(ctx, tm, s, s2, B, M, N, pairs, K, top) if batch else None
            best = 1e9
            for _ in range(8):
                e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                top.fill_(3)
                e[0].record()
                if batch:
                    b.run()
                else:
                    S.sncc_topk(ctx, tm, s, s2, B, M, N, pairs, K, S.SNCC_FP32_KAHAN, top)
                e[1].record()
                S.sncc_sync(ctx)
                best = min(best, e[0].elapsed_time(e[1]))
            print("case", kind, batch, "form", form or "by rule", round(best, 3), "ms", flush=True)
            ms.append(best)
            got.append(top.cpu().numpy())
            if b:
                b.destroy()
            S.sncc_tmpl_destroy(tm)
        assert (got[0] == got[1]).all()
        assert ms[1] < 2.0 * ms[0]
    finally:
        S.sncc_ctx_destroy(ctx)


def test_undecided_fp64_pair_costs_the_plain_form(monkeypatch):
    """One FP64 pair of many segments whose every offset is scored: about the
    time of the plain form's map (which has no list to keep), so its lists fill
    the chip."""
    import torch
    import paper_2502_01286_amd as S
    torch.cuda.init()
    ctx = S.sncc_ctx_create(0)
    w = h = 64
    t, _, _ = synth.crop_template(np.random.default_rng(8), synth.scene(3, M, N), w, h, sigma_max=2)
    segs = S.sncc_segment_template(t, 2)[0]
    assert len(segs) > 500
    _, s, s2 = build_sats(S, ctx, [_frame("uniform")])
    rho = torch.zeros((N - h + 1, M - w + 1), dtype=torch.float64, device="cuda")
    top = torch.zeros((1, K, 3), dtype=torch.int32, device="cuda")
    ms = []
    try:
        monkeypatch.setenv("SNCC_TEST_DENSE", "0")
        tm = S.sncc_upload_templates(ctx, [segs], [w], [h])
        for call in (lambda: S.sncc_score(ctx, tm, 0, s[0], s2[0], M, N, S.SNCC_FP64, rho),
                     lambda: S.sncc_topk(ctx, tm, s, s2, 1, M, N, [(0, 0)], K, S.SNCC_FP64, top)):
            best = 1e9
            for _ in range(8):
                e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                e[0].record()
                call()
                e[1].record()
                S.sncc_sync(ctx)
                best = min(best, e[0].elapsed_time(e[1]))
            ms.append(best)
        print("case K", len(segs), "plain map", round(ms[0], 3), "top-k", round(ms[1], 3), flush=True)
        got = S.decode_matches(top)[0]
        assert [(int(m["u"]), int(m["v"])) for m in got] == [(i, 0) for i in range(K)]
        assert ms[1] < 1.5 * ms[0]
        S.sncc_tmpl_destroy(tm)
    finally:
        S.sncc_ctx_destroy(ctx)
