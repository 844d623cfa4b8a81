"""Softmax weights of the bf16 models' attention to fp32 accuracy at large
scores, seen through the logits, in decode and in prefill.

In the two-layer decoder below only two tokens of a prompt, A and B, have any
weight (their scores are near 3,700, a fraction of 1 apart, all others' far
below), so an attention output is o = wA vA + wB vB, chosen just off a bf16
rounding boundary.  Layer 0 puts 1 + K (o - t) into residual features, t the
correctly rounded output and K 1/4 over its last place: an output rounded the
other way moves its feature by 1/4.  The decode row shows its own features as
logits, and through layer 1 those of a prompt token, which the prefill made."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_harness import device_setup, upload_pool
from tests.test_gpu_prefill import generic_cfg
from tests.test_gpu_swiglu import bf16, boundary_margin

pytestmark = pytest.mark.gpu
D, HQ, HD = 512, 8, 64
POINTS = 63
C, A, B, T = range(4)      # token types; T is a C that layer 1 looks for


def points():
    """(head, q, alpha, beta, o) of POINTS outputs: vA, vB = alpha +- beta,
    scores q / 8 apart, o on both sides of boundaries; 1e-6 is over the error of
    fp32 weights (a few 2^-24)."""
    out, q = [], 2.0
    i, j = np.meshgrid(np.arange(64, 192), np.arange(1, 64), indexing="ij")
    alpha, beta = i.ravel() / 32.0, j.ravel() / 32.0
    for h in range(HQ):
        pick = []
        while len(pick) < 8:
            q += 1.0 / 16.0
            w_a = 1.0 / (1.0 + np.exp(q / 8.0))
            o = w_a * (alpha + beta) + (1.0 - w_a) * (alpha - beta)
            near = (boundary_margin(o) > 1e-6) & (boundary_margin(o) < 3e-5)
            up = bf16(o) > o
            pick = [*np.flatnonzero(near & up)[:4], *np.flatnonzero(near & ~up)[:4]]
        out += [(h, q, alpha[e], beta[e], o[e]) for e in pick]
    return out[:POINTS]


def weights(cfg, pts):
    z = {name: np.ones(shape) if len(shape) == 1 else np.zeros(shape) for name, shape in W.weight_specs(cfg["model"])}
    e = np.ones((D, D))                    # features 1, 2, 3 tell the types apart, feature 0 is 1 for all
    e[:, 2], e[:, 3] = -1.0, -1.0
    e[A, 2], e[B, 2], e[B, 1], e[T, 3] = 1.0, 1.0, -1.0, 1.0
    z["embed"], z["lm_head"] = e, np.eye(D)
    # layer 0, rotation indices 30 and 31 (which do not turn): k = 240 for A and B, -240 for others; 128 for A, 129 for B
    z["l0.wk"][30, 2] = 240.0
    z["l0.wk"][31, 0], z["l0.wk"][31, 4], z["l0.wk"][31, 1] = 128.0, 0.5, -0.5
    for d, (h, q, alpha, beta, o) in enumerate(pts):
        z["l0.wq"][h * HD + 30, 0], z["l0.wq"][h * HD + 31, 0] = 120.0, q
        z["l0.wv"][d, 0], z["l0.wv"][d, 1] = alpha, beta
        t = bf16(o)
        K = np.ldexp(0.25, 8 - int(np.frexp(t)[1]))
        z["l0.wo"][64 + d, h * HD + d], z["l0.wo"][64 + d, h * HD + 63] = K, -K * t
    z["l0.wv"][63, 0] = 1.0                # an output of exactly 1
    # layer 1: all weight on T; its features 64.. are added to features 128..
    z["l1.wq"][31::HD, 0], z["l1.wk"][31, 3] = 16.0, 64.0
    d = np.arange(POINTS)
    z["l1.wv"][d, 64 + d] = 1.0
    z["l1.wo"][128 + d, d] = 1.0
    return {k: W.f32_to_bf16_bits(np.ascontiguousarray(v, np.float32)) for k, v in z.items()}


# A and B: keys of two waves of a decode split and of two key blocks of the
# prefill; then keys of two decode splits
@pytest.mark.parametrize("b_at,t_at,length", [(80, 100, 110), (200, 220, 230)])
def test_softmax_rounds_as_exact(b_at, t_at, length):
    import torch
    cfg = generic_cfg(D, HQ, 1, HD, 64, [length], layers=2, vocab=D, max_new=4)
    cfg["model"]["rope_theta"] = 1e30      # the last rotation indices turn by < 1e-25
    pts = points()
    ctx, _ = device_setup(cfg, weights(cfg, pts))
    pool = W.pool_with_lengths(cfg, [length])
    pool["tokens"][:] = C
    pool["tokens"][[0, b_at, t_at]] = A, B, T
    d_tok, d_p, _ = upload_pool(pool)
    ctx.sara_begin_step(d_tok, pool["offsets"], d_p, None, 0)
    out = torch.zeros((1, D), dtype=torch.float32, device="cuda")
    ctx.sara_decode_step(None, out)
    got = out.cpu().numpy()[0].astype(np.float64)
    ctx.close()
    d = np.arange(POINTS)
    decode, prefill = got[64 + d] / got[0] - 1.0, got[128 + d] / got[0] - 2.0
    wrong = [int((~(np.abs(x) < 0.06)).sum()) for x in (decode, prefill)]
    assert wrong == [0, 0], (wrong, decode, prefill)
