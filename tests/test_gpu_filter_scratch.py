"""A program that changes its pair list from call to call holds one filter
scratch per precision, not one per list that the context has not yet dropped."""

import numpy as np
import pytest

from workloads import synth

from gpu_util import build_sats

pytestmark = pytest.mark.gpu


def test_memory_over_many_pair_lists(monkeypatch):
    import torch
    import paper_2502_01286_amd as S
    torch.cuda.init()
    ctx = S.sncc_ctx_create(0)
    M, N, B, T, k = 1280, 720, 2, 4, 5
    frames = [synth.scene(20 + b, M, N) for b in range(B)]
    rng = np.random.default_rng(21)
    segs = [S.sncc_segment_template(synth.crop_template(rng, frames[0], 48, 48, sigma_max=4)[0], 4)[0]
            for _ in range(T)]
    _, s, s2 = build_sats(S, ctx, frames)
    monkeypatch.setenv("SNCC_TEST_DENSE", "1")
    tm = S.sncc_upload_templates(ctx, segs, [48] * T, [48] * T)
    top = torch.zeros((B * T, k, 3), dtype=torch.int32, device="cuda")
    lists = [[(int(f), int(t)) for f, t in zip(rng.integers(0, B, n), rng.integers(0, T, n))]
             for n in [B * T] + [int(x) for x in rng.integers(4, B * T + 1, 40)]]
    try:
        for prec in (S.SNCC_FP32_KAHAN, S.SNCC_FP64):
            S.sncc_topk(ctx, tm, s, s2, B, M, N, lists[0], k, prec, top)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        for pairs in lists[1:]:
            for prec in (S.SNCC_FP32_KAHAN, S.SNCC_FP64):
                S.sncc_topk(ctx, tm, s, s2, B, M, N, pairs, k, prec, top[:len(pairs)])
        torch.cuda.synchronize()
        held = before - torch.cuda.mem_get_info()[0]
        # one list's maps are 15 to 27 MB, 32 lists may be waiting to be dropped
        print("case held", held >> 20, "MB", flush=True)
        assert held < 100 << 20
    finally:
        S.sncc_tmpl_destroy(tm)
        S.sncc_ctx_destroy(ctx)
