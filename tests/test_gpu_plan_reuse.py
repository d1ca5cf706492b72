"""When a context's kept plan may serve the next call: one made under capture,
whose uploads run with the graph, does not; one that had to go without the
filter's memory is made again later."""

import numpy as np
import pytest

from workloads import synth

from gpu_util import build_sats

pytestmark = pytest.mark.gpu

M, N, B, T, K = 640, 480, 2, 4, 5


def _setup(S, ctx):
    frames = [synth.scene(20 + b, M, N) for b in range(B)]
    rng = np.random.default_rng(21)
    segs = [S.sncc_segment_template(synth.crop_template(rng, frames[0], 48, 48, sigma_max=4)[0], 4)[0]
            for _ in range(T)]
    _, s, s2 = build_sats(S, ctx, frames)
    pairs = [(b, t) for b in range(B) for t in range(T)] * 3
    return s, s2, segs, pairs


@pytest.mark.parametrize("prec", [0, 1])
def test_plan_made_under_capture_serves_no_other_call(monkeypatch, prec):
    import torch
    import paper_2502_01286_amd as S
    torch.cuda.init()
    monkeypatch.setenv("SNCC_TEST_DENSE", "1")
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        ctx = S.sncc_ctx_create(0, st.cuda_stream)
        s, s2, segs, pairs = _setup(S, ctx)
        tm = S.sncc_upload_templates(ctx, segs, [48] * T, [48] * T)
        want, got = (torch.full((len(pairs), K, 3), 3, dtype=torch.int32, device="cuda")
                     for _ in range(2))
        other = S.sncc_ctx_create(0, st.cuda_stream)
        S.sncc_topk(other, tm, s, s2, B, M, N, pairs, K, prec, want)
        st.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st, capture_error_mode="relaxed"):
            S.sncc_topk(ctx, tm, s, s2, B, M, N, pairs, K, prec, got)
        st.synchronize()
        assert int(got.min()) == 3 == int(got.max())  # the graph has not run
        for _ in range(3):
            got.fill_(3)
            S.sncc_topk(ctx, tm, s, s2, B, M, N, pairs, K, prec, got)
            st.synchronize()
            assert torch.equal(got, want)
        del g
        S.sncc_tmpl_destroy(tm)
        for c in (ctx, other):
            S.sncc_ctx_destroy(c)


@pytest.mark.parametrize("prec", [0, 1])
def test_filter_returns_when_memory_does(monkeypatch, prec):
    import torch
    import paper_2502_01286_amd as S
    torch.cuda.init()
    monkeypatch.setenv("SNCC_TEST_DENSE", "1")
    ctx = S.sncc_ctx_create(0)
    s, s2, segs, pairs = _setup(S, ctx)
    tm = S.sncc_upload_templates(ctx, segs, [48] * T, [48] * T)
    top = torch.zeros((len(pairs), K, 3), dtype=torch.int32, device="cuda")
    want = None
    try:
        monkeypatch.setenv("SNCC_TEST_FAIL_ALLOC", str(8 << 20))  # the maps: 31 MB
        S.sncc_topk(ctx, tm, s, s2, B, M, N, pairs, K, prec, top)
        torch.cuda.synchronize()
        want = top.clone()
        monkeypatch.delenv("SNCC_TEST_FAIL_ALLOC")
        before = torch.cuda.mem_get_info()[0]
        for i in range(70):
            top.fill_(3)
            S.sncc_topk(ctx, tm, s, s2, B, M, N, pairs, K, prec, top)
        torch.cuda.synchronize()
        assert torch.equal(top, want)
        taken = before - torch.cuda.mem_get_info()[0]
        print("case", prec, "taken", taken >> 20, "MB", flush=True)
        assert taken >= 24 << 20
    finally:
        S.sncc_tmpl_destroy(tm)
        S.sncc_ctx_destroy(ctx)
