"""SwiGLU of bf16 models to fp32 accuracy, seen through the logits.

The one-layer decoder below makes each feature's gate g and up u exact in
fp32 (16-bit sums of two weights, normed rows of ones), and each residual
feature h = 1 + K (a - t) with a the layer's bf16 product, t the correctly
rounded one and K 1/4 over t's last place: a product rounded to another bf16
value moves its logit by about 1/4."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_harness import device_setup, upload_pool
from tests.test_gpu_prefill import generic_cfg

pytestmark = pytest.mark.gpu
D, F = 512, 576
# Relative error that the kernel's fp32 arithmetic may have: the exponential
# within 1 ulp, the sum, the quotient and the product each rounded once (silu(g)
# measured within 1.4e-7, the product with u adds 6e-8)
BOUND = 3e-7


def bf16(x):
    """fp64 -> nearest bf16 (half to even), as fp64."""
    m, e = np.frexp(x)
    return np.ldexp(np.round(m * 256.0), e - 8)


def two_bf16(x):
    """(hi + lo, hi, lo): 16 bits of x as the sum of two bf16 values."""
    hi = bf16(x)
    lo = bf16(x - hi)
    return hi + lo, hi, lo


def silu_mul(g, u):
    return g / (1.0 + np.exp(-g)) * u


def boundary_margin(a):
    """Relative distance of a from the nearest bf16 rounding boundary."""
    step = np.ldexp(1.0, np.frexp(a)[1] - 8)
    return np.abs(np.abs(a) / step - np.floor(np.abs(a) / step) - 0.5) * step / np.abs(a)


def near_boundary(lo, hi):
    """D pairs (g, u), lo <= g < hi, whose product lies just off a boundary:
    an error of 1.2e-6 rounds it the other way, one of BOUND does not."""
    r = np.random.default_rng([int(hi) + 100, 5])
    n = 1 << 22
    g = two_bf16(r.uniform(lo, hi, n))[0]
    u = two_bf16(r.uniform(1.0, 2.0, n) * (1.0 + np.exp(-g)) / np.maximum(np.abs(g), 0.5))[0]
    margin = boundary_margin(silu_mul(g, u))
    pick = np.flatnonzero((margin > BOUND) & (margin < 1.2e-6) & (np.abs(g) > 0.5))[:D]
    assert len(pick) == D
    return g[pick], u[pick]


def logits_of(g, u):
    import torch
    cfg = generic_cfg(D, 8, 1, 64, F, [1], layers=1, vocab=D, max_new=4)
    t = bf16(silu_mul(g, u))
    K = np.ldexp(0.25, 8 - np.frexp(t)[1])
    i = np.arange(D)
    gate, up, down = np.zeros((F, D)), np.zeros((F, D)), np.zeros((D, F))
    _, gate[i, 0], gate[i, 1] = two_bf16(g)
    _, up[i, 0], up[i, 1] = two_bf16(u)
    gate[D, 0], up[D, 0] = 64.0, 1.0 / 64.0          # a product of exactly 1
    down[i, i], down[i, D] = K, -K * t
    by_name = {"embed": np.ones((D, D)), "lm_head": np.eye(D), "l0.wg": gate, "l0.wu": up, "l0.wd": down}
    w = {}
    for name, shape in W.weight_specs(cfg["model"]):
        val = by_name.pop(name, np.ones(shape) if len(shape) == 1 else np.zeros(shape))
        w[name] = W.f32_to_bf16_bits(np.ascontiguousarray(val, np.float32))
    assert not by_name
    ctx, _ = device_setup(cfg, w)
    pool = W.pool_with_lengths(cfg, [1])
    d_tok, d_p, _ = upload_pool(pool)
    ctx.sara_begin_step(d_tok, pool["offsets"], d_p, None, 0)
    out = torch.zeros((1, D), dtype=torch.float32, device="cuda")
    ctx.sara_decode_step(None, out)
    got = out.cpu().numpy()[0]
    ctx.close()
    return got


@pytest.mark.parametrize("lo,hi", [(-30.0, -8.0), (-8.0, 8.0), (8.0, 30.0)])
def test_swiglu_rounds_as_exact(lo, hi):
    g, u = near_boundary(lo, hi)
    got = logits_of(g, u)
    wrong = np.flatnonzero(~(np.abs(got - 1.0) < 0.05))
    assert len(wrong) == 0, (len(wrong), list(zip(g[wrong][:4], u[wrong][:4], got[wrong][:4])))


def test_swiglu_large_up():
    """silu(g) u well in range where g u is not."""
    g, u = np.full(D, -50.0), two_bf16(np.linspace(8e36, 6e37, D))[0]
    u = np.where(boundary_margin(silu_mul(g, u)) > BOUND, u, u[0])
    got = logits_of(g, u)
    assert np.all(np.abs(got - 1.0) < 0.05), got[~(np.abs(got - 1.0) < 0.05)][:4]
