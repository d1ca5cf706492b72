"""The matrix-core operands of a new template set are enqueued like all device
work: the call that needs them first does not wait for its stream, and calls on
other streams that follow it see them built."""

import time

import numpy as np
import pytest

import oracle as O
from workloads import synth

from gpu_util import build_sats

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64", "frame"])
def test_first_call_does_not_wait(monkeypatch, prec):
    import torch
    import paper_2502_01286_amd as S
    torch.cuda.init()
    monkeypatch.setenv("SNCC_TEST_DENSE", "1")
    M, N, W, H = 400, 300, 64, 50
    f = synth.scene(31, M, N)
    t, _, _ = synth.crop_template(np.random.default_rng(32), f, W, H, sigma_max=4)
    segs = S.sncc_segment_template(t, 4)[0]
    want = O.rho_map(f, O.precompute_template_approximation(t, 4))
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    streams = [torch.cuda.Stream() for _ in range(2)]
    ctxs = [S.sncc_ctx_create(0, st.cuda_stream) for st in streams]
    d, s, s2 = build_sats(S, ctxs[0], [f])
    dt = torch.float64 if prec == "fp64" else torch.float32
    tm = S.sncc_upload_templates(ctxs[0], [segs], [W], [H])

    def call(i, rho):
        if prec == "frame":
            S.sncc_score_frame(ctxs[i], tm, 0, d[0], rho)
        else:
            S.sncc_score(ctxs[i], tm, 0, s[0], s2[0], M, N,
                         S.SNCC_FP64 if prec == "fp64" else S.SNCC_FP32_KAHAN, rho)

    rho = [torch.zeros((N - H + 1, M - W + 1), dtype=dt, device="cuda") for _ in range(2)]
    with torch.cuda.stream(streams[0]):
        torch.mm(a, a)  # the library's own first-call work
        torch.cuda.synchronize()
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        for _ in range(200):  # about 0.2 s of work ahead of the call
            torch.mm(a, a)
        e[1].record()
    t0 = time.perf_counter()
    call(0, rho[0])
    call(1, rho[1])  # the other stream: its map waits on the device
    host = time.perf_counter() - t0
    pending = not e[1].query()
    torch.cuda.synchronize()
    print("case", prec, "host", round(host * 1e3, 2), "ms, work ahead",
          round(e[0].elapsed_time(e[1]), 1), "ms", flush=True)
    try:
        for r in rho:
            assert np.abs(r.cpu().numpy() - want).max() <= (1e-9 if prec == "fp64" else 1e-5)
        assert pending and host < 0.25e-3 * e[0].elapsed_time(e[1])
    finally:
        S.sncc_tmpl_destroy(tm)
        for c in ctxs:
            S.sncc_ctx_destroy(c)
