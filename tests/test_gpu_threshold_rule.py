"""The two-threshold search goes without its filter where the thresholds tell
that most survivors match: such a call takes no longer than without it."""

import numpy as np
import pytest

from workloads import synth

from gpu_util import build_sats

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lo,hi", [(0.8, 0.8), (0.8, 0.7)])
def test_close_thresholds_go_without_the_filter(monkeypatch, lo, hi):
    import torch
    import paper_2502_01286_amd as S
    torch.cuda.init()
    M, N, B, T, w = 1920, 1080, 2, 4, 64
    frames = [synth.scene(27 + b, M, N) for b in range(B)]
    rng = np.random.default_rng(2)
    fast, slow = [], []
    for _ in range(T):
        t, _, _ = synth.crop_template(rng, frames[0], w, w, sigma_max=16)
        fast.append(S.sncc_segment_template(t, 16)[0])
        slow.append(S.sncc_segment_template(t, 4)[0])
    pairs = [(b, t) for b in range(B) for t in range(T)]
    cand, out = (torch.zeros((1 << 20, 6), dtype=torch.int32, device="cuda") for _ in range(2))
    counts = torch.zeros(2, dtype=torch.int32, device="cuda")
    calls, ctxs, sets = [], [], []
    try:
        for form in ("0", ""):  # never, by rule: read when the context plans the call
            monkeypatch.setenv("SNCC_TEST_DENSE", form)
            ctx = S.sncc_ctx_create(0)
            ctxs.append(ctx)
            _, s, s2 = build_sats(S, ctx, frames)
            ft, st = (S.sncc_upload_templates(ctx, x, [w] * T, [w] * T) for x in (fast, slow))
            sets += [ft, st]

            def call(ctx=ctx, s=s, s2=s2, ft=ft, st=st):
                S.sncc_threshold_match(ctx, ft, st, [lo] * T, [hi] * T, s, s2, B, M, N, pairs, cand,
                                       out, counts)

            call()
            S.sncc_sync(ctx)
            calls.append(call)
        best = [1e9, 1e9]
        for _ in range(20):  # in turn
            for i, call in enumerate(calls):
                e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                e[0].record()
                call()
                e[1].record()
                torch.cuda.synchronize()
                best[i] = min(best[i], e[0].elapsed_time(e[1]))
        print("case", lo, hi, counts.tolist(), [round(x, 4) for x in best], flush=True)
        assert best[1] < 1.05 * best[0]
    finally:
        for x in sets:
            S.sncc_tmpl_destroy(x)
        for c in ctxs:
            S.sncc_ctx_destroy(c)
