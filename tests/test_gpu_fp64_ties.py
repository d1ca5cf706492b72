"""FP64 top-k where many offsets tie but for the last bits of their doubles:
the lists follow one arithmetic (box sums times c_i added in segment order),
whether the filter finds the candidates or every offset is scored."""

import numpy as np
import pytest

from workloads import synth

from gpu_util import build_sats

pytestmark = pytest.mark.gpu


def _lists(S, ctx, monkeypatch, form, frames, segs, W, H, k):
    import torch
    monkeypatch.setenv("SNCC_TEST_DENSE", form)
    B, N, M = len(frames), frames[0].shape[0], frames[0].shape[1]
    _, s, s2 = build_sats(S, ctx, frames)
    tm = S.sncc_upload_templates(ctx, segs, W, H)
    pairs = [(f, t) for f in range(B) for t in range(len(segs))]
    out = torch.full((len(pairs), k, 3), 5, dtype=torch.int32, device="cuda")
    S.sncc_topk(ctx, tm, s, s2, B, M, N, pairs, k, S.SNCC_FP64, out)
    S.sncc_sync(ctx)
    S.sncc_tmpl_destroy(tm)
    return out.cpu().numpy()


def _shifted_copies(rng, M, N, w, h):
    """A scene with one patch pasted at many places, each a little brighter:
    the windows differ by a constant, so their rho is the same number."""
    f = synth.scene(5, M, N)
    p = rng.integers(40, 160, (h, w))
    d = 0
    for y in range(3, N - h, h + 5):
        for x in range(2, M - w, w + 7):
            f[y:y + h, x:x + w] = p + d
            d = (d + 1) % 90
    return f, p.astype(np.uint8)


@pytest.mark.parametrize("size", [(5, 4, 0.5), (24, 20, 2), (64, 40, 3), (101, 70, 8)])
@pytest.mark.parametrize("k", [1, 10, 64])
def test_fp64_lists_follow_one_arithmetic(monkeypatch, size, k):
    import torch
    import paper_2502_01286_amd as S
    torch.cuda.init()
    ctx = S.sncc_ctx_create(0)
    w, h, sigma = size
    M, N = 900, 500
    rng = np.random.default_rng(w)
    f, p = _shifted_copies(rng, M, N, w, h)
    low = np.full((N, M), 100, np.uint8)  # nearly uniform windows
    low[rng.random((N, M)) < 2e-3] = 101
    low[N // 2:] = np.maximum(low[N // 2:], f[N // 2:] // 64 + 90)
    q = synth.scene(9, w, h)
    segs = [S.sncc_segment_template(t, sigma)[0] for t in (p, q)]
    try:
        print("case", size, k, flush=True)
        got = _lists(S, ctx, monkeypatch, "1", [f, low], segs, [w] * 2, [h] * 2, k)
        want = _lists(S, ctx, monkeypatch, "0", [f, low], segs, [w] * 2, [h] * 2, k)
        assert (want[..., 0] >= 0).all()
        assert (got == want).all(), np.argwhere((got != want).any(axis=2))[:4].tolist()
    finally:
        S.sncc_ctx_destroy(ctx)
