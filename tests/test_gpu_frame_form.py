"""The form that is asked for of sncc_score_frame is the one that runs."""

import numpy as np
import pytest

from workloads import synth

from gpu_util import build_sats

pytestmark = pytest.mark.gpu


def test_global_form_builds_tables(monkeypatch):
    import torch
    import paper_2502_01286_amd as S
    torch.cuda.init()
    M, N, W, H = 640, 480, 32, 32  # the automatic form goes without tables
    f = synth.scene(51, M, N)
    t, _, _ = synth.crop_template(np.random.default_rng(52), f, W, H, sigma_max=6)
    segs = S.sncc_segment_template(t, 6)[0]
    own, ctx = S.sncc_ctx_create(0), S.sncc_ctx_create(0)
    try:
        d, s, s2 = build_sats(S, own, [f])
        tm = S.sncc_upload_templates(ctx, [segs], [W], [H])
        rho = [torch.zeros((N - H + 1, M - W + 1), device="cuda") for _ in range(3)]
        S.sncc_score(own, tm, 0, s[0], s2[0], M, N, S.SNCC_FP32_KAHAN, rho[0])
        S.sncc_score_frame(ctx, tm, 0, d[0], rho[1])
        S.sncc_sync(own)
        S.sncc_sync(ctx)
        monkeypatch.setenv("SNCC_TEST_FAIL_ALLOC", "1")
        S.sncc_score_frame(ctx, tm, 0, d[0], rho[1])  # no tables: no memory
        with pytest.raises(S.SnccError) as e:
            S.sncc_score_frame(ctx, tm, 0, d[0], rho[2], form=S.SNCC_FORM_GLOBAL)
        assert e.value.code == S.SNCC_ENOMEM
        monkeypatch.delenv("SNCC_TEST_FAIL_ALLOC")
        assert S.sncc_score_frame(ctx, tm, 0, d[0], rho[2],
                                  form=S.SNCC_FORM_GLOBAL) == S.SNCC_FORM_GLOBAL
        S.sncc_sync(ctx)
        assert torch.equal(rho[2], rho[0])  # the tables, then sncc_score
        assert float((rho[1] - rho[0]).abs().max()) <= 2e-5
        S.sncc_tmpl_destroy(tm)
    finally:
        for c in (own, ctx):
            S.sncc_ctx_destroy(c)
