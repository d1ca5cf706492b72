"""The matrix-core forms' memory is optional: where the device has none for
their operands or scratch, every call takes the form it had without them, also
after a real failed allocation, whose error the runtime keeps until it is
read."""

import numpy as np
import pytest

from workloads import synth

from gpu_util import build_sats

pytestmark = pytest.mark.gpu

M, N, B = 700, 500, 2
W, H = [128, 120], [128, 110]


def _calls(S, ctx, s, s2, f, tm, fine):
    import torch
    pairs = [(b, t) for b in range(B) for t in range(2)]
    nu, nv = M - W[0] + 1, N - H[0] + 1

    def score(prec, dt):
        rho = torch.zeros((nv, nu), dtype=dt, device="cuda")
        S.sncc_score(ctx, tm, 0, s[0], s2[0], M, N, prec, rho)
        return rho

    def frame():
        rho = torch.zeros((nv, nu), device="cuda")
        S.sncc_score_frame(ctx, tm, 0, f[0], rho)
        return rho

    def topk(prec):
        top = torch.zeros((len(pairs), 4, 3), dtype=torch.int32, device="cuda")
        S.sncc_topk(ctx, tm, s, s2, B, M, N, pairs, 4, prec, top)
        return top

    def batch():
        top = torch.zeros((len(pairs), 4, 3), dtype=torch.int32, device="cuda")
        b = S.sncc_batch_create(ctx, tm, s, s2, B, M, N, pairs, 4, top)
        b.run()
        S.sncc_sync(ctx)
        b.destroy()
        return top

    def threshold():
        cand = torch.zeros((1 << 20, 6), dtype=torch.int32, device="cuda")
        out = torch.zeros((1 << 20, 6), dtype=torch.int32, device="cuda")
        counts = torch.zeros(2, dtype=torch.int32, device="cuda")
        S.sncc_threshold_match(ctx, tm, fine, [0.3] * 2, [0.4] * 2, s, s2, B, M, N, pairs, cand,
                               out, counts)
        S.sncc_sync(ctx)
        o = np.sort(S.decode_hits(out, int(counts[1])), order=["pair", "v", "u"])
        return torch.from_numpy(np.stack([o["pair"], o["v"], o["u"]]))

    return {"score32": lambda: score(S.SNCC_FP32_KAHAN, torch.float32),
            "score64": lambda: score(S.SNCC_FP64, torch.float64), "frame": frame,
            "topk32": lambda: topk(S.SNCC_FP32_KAHAN), "topk64": lambda: topk(S.SNCC_FP64),
            "batch": batch, "threshold": threshold}


@pytest.mark.parametrize("refuse", ["operands", "scratch"])
def test_no_memory_for_the_matrix_core_forms(monkeypatch, refuse):
    """Refused: allocations of 300 kB and more, which are the operands (0.5 to
    2 MB) and the filters' maps, not what the segment forms need here."""
    import torch
    import paper_2502_01286_amd as S
    torch.cuda.init()
    frames = [synth.scene(90 + b, M, N) for b in range(B)]
    rng = np.random.default_rng(91)
    temps = [synth.crop_template(rng, frames[0], w, h, sigma_max=12)[0] for w, h in zip(W, H)]
    coarse = [S.sncc_segment_template(t, 12)[0] for t in temps]
    detail = [S.sncc_segment_template(t, 8)[0] for t in temps]
    ctx, other = S.sncc_ctx_create(0), None
    try:
        f, s, s2 = build_sats(S, ctx, frames)
        want = {}
        monkeypatch.setenv("SNCC_TEST_DENSE", "0")
        tm = S.sncc_upload_templates(ctx, coarse, W, H)
        fine = S.sncc_upload_templates(ctx, detail, W, H)
        for name, call in _calls(S, ctx, s, s2, f, tm, fine).items():
            want[name] = call().cpu()
        monkeypatch.setenv("SNCC_TEST_DENSE", "1")
        new = S.sncc_upload_templates(ctx, coarse, W, H)  # other plans, no operands yet
        fine2 = S.sncc_upload_templates(ctx, detail, W, H)
        calls = _calls(S, ctx, s, s2, f, new, fine2)
        if refuse == "scratch":
            for call in calls.values():
                call()
            S.sncc_sync(ctx)
            other = S.sncc_ctx_create(0)  # without plans; the operands are the templates'
            calls = _calls(S, other, s, s2, f, new, fine2)
        monkeypatch.setenv("SNCC_TEST_FAIL_ALLOC", "300000")
        for name in calls:
            for turn in range(2):
                if name == "frame" and refuse == "operands":
                    continue  # its tables do not fit the limit
                print("case", refuse, name, turn, flush=True)
                got = calls[name]().cpu()
                if name in ("score32", "score64", "frame"):
                    assert (got - want[name]).abs().max() <= 2e-5
                else:
                    assert torch.equal(got, want[name]), name
        monkeypatch.delenv("SNCC_TEST_FAIL_ALLOC")
        for x in (tm, fine, new, fine2):
            S.sncc_tmpl_destroy(x)
    finally:
        monkeypatch.delenv("SNCC_TEST_FAIL_ALLOC", raising=False)
        if other:
            S.sncc_ctx_destroy(other)
        S.sncc_ctx_destroy(ctx)
