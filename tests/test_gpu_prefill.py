"""Prefill of bf16 models: every query-head group size and head width, prompt
lengths at the edges of the attention's key blocks and query tiles."""
import numpy as np
import pytest

import workloads as W
from oracle import run as ORUN
from tests.gpu_harness import compare_logs, device_setup, forced_table, run_gpu_step, slot_rows

pytestmark = pytest.mark.gpu


def generic_cfg(d, hq, hkv, hd, ffn, lengths, layers=2, vocab=512, **alloc):
    """A small bf16 decoder and one probe for each prompt of the given lengths."""
    cfg = W.get_config("qwen1p5b_shape")
    cfg["model"].update(n_layers=layers, d_model=d, n_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ffn=ffn, vocab=vocab,
                        eos_id=vocab - 1)
    U = len(lengths)
    cfg["alloc"].update(B=U, k=2, n0=1, commit_min=2, budget_N=2 * U, pool_U=U, n_slots=U, max_prompt=max(lengths),
                        max_new=2)
    cfg["alloc"].update(alloc)
    return cfg


def check_against_oracle(cfg, lengths):
    """One teacher-forced step: logs bit-exact, every row's logits within the
    2-layer bound of the bf16 slices (3e-2 of the oracle row's rms)."""
    w, pool, seed = W.make_weights(cfg), W.pool_with_lengths(cfg, lengths), W.sampling_seed(cfg)
    ora = ORUN.run_step(cfg, w, pool, seed, keep_logits=lambda u, j, i: True)
    ctx, _ = device_setup(cfg, w)
    gpu = run_gpu_step(ctx, cfg, pool, forced=forced_table(cfg, ora["rollouts_detail"]), capture_logits=True)
    ctx.close()
    compare_logs(gpu["logs"], ora)
    worst = {}
    for (t, s), key in slot_rows(gpu).items():
        o = ora["logits"][key].astype(np.float64)
        rel = float(np.max(np.abs(gpu["logits"][t][s] - o)) / np.sqrt(np.mean(o * o)))
        worst[key[0]] = max(rel, worst.get(key[0], 0.0))
    assert set(worst) == set(range(len(lengths)))
    bad = {lengths[u]: r for u, r in worst.items() if r > 3e-2}
    assert not bad, bad
    return max(worst.values())


@pytest.mark.parametrize("hq,hkv,hd", [(2, 2, 64), (4, 2, 64), (6, 2, 64), (8, 2, 64), (8, 1, 64), (5, 1, 64), (7, 1, 128),
                                       (6, 1, 128), (10, 2, 128), (4, 4, 128), (8, 1, 128)])
def test_prefill_attention_group_sizes(hq, hkv, hd):
    # P - 1 positions are prefilled: none, one, tile and key-block edges (16, 32, 64, 128, 256) and a few blocks
    lengths = [1, 2, 16, 17, 18, 33, 34, 65, 66, 129, 130, 257, 258, 300]
    cfg = generic_cfg(512, hq, hkv, hd, 512, lengths)
    print(f"[prefill] {hq}/{hkv} x {hd}: max |dlogit| / rms {check_against_oracle(cfg, lengths):.4f}", flush=True)


@pytest.mark.parametrize("width,lengths", [
    # 256 x 256 tiles with K splits (o, down) and in one piece (gate|up), ragged last row tile and column tile
    ((1024, 10, 2, 64, 1472), [700, 1301, 33]),
    # as many rows as the q|k|v tiles need (64 tiles), head width 64 and 128
    ((512, 8, 2, 64, 512), [2049] * 3 + [1500]),
    ((512, 4, 2, 128, 448), [1700] * 3),
    # d = 3072: the norm that reads its row twice; rows below any tile
    ((3072, 4, 1, 64, 512), [150, 18, 2]),
    # more rows than one chunk holds: 33,000 rows, the cut inside a prompt
    ((512, 2, 1, 64, 256), [5500] * 6),
])
def test_prefill_gemm_tiles(width, lengths):
    cfg = generic_cfg(*width, lengths)
    print(f"[prefill] {width} {sum(lengths)} tokens: max |dlogit| / rms {check_against_oracle(cfg, lengths):.4f}", flush=True)


@pytest.mark.parametrize("width,lengths,max_new", [
    # rows around the 32- and 64-row blocks, K of one step a wave, odd column-tile counts
    ((64, 1, 1, 64, 64), [1, 2, 17, 40, 65], 3),
    ((192, 3, 1, 128, 320), [33, 64, 66, 5], 4),
    # contexts of several 256-token splits, a tile across the prompt's end; 33 rows
    ((128, 8, 1, 64, 192), [600, 257, 258] + [3] * 30, 20),
])
def test_f32_layers(width, lengths, max_new):
    d, hq, hkv, hd, ffn = width
    cfg = generic_cfg(d, hq, hkv, hd, ffn, lengths, vocab=528, max_new=max_new)
    cfg["model"].update(dtype="f32", eos_id=-1)
    w, pool, seed = W.make_weights(cfg), W.pool_with_lengths(cfg, lengths), W.sampling_seed(cfg)
    ora = ORUN.run_step(cfg, w, pool, seed, keep_logits=lambda u, j, i: True)
    ctx, _ = device_setup(cfg, w)
    gpu = run_gpu_step(ctx, cfg, pool, forced=forced_table(cfg, ora["rollouts_detail"]), capture_logits=True)
    ctx.close()
    compare_logs(gpu["logs"], ora)
    # fp32 against the fp64 oracle: K <= 1024 products a sum and a few layers leave ~1e-6 of the
    # logits' rms; the package's bound for fp32 models is 1e-3
    worst = max(float(np.max(np.abs(gpu["logits"][t][s] - ora["logits"][key]))) for (t, s), key in slot_rows(gpu).items())
    print(f"[f32] {width}: max |dlogit| {worst:.2e}", flush=True)
    assert worst <= 1e-4


def test_prefill_chunk_fits_the_memory_left():
    """Little device memory left: the context takes a smaller prefill chunk
    than it would use otherwise, and its logits agree."""
    import torch

    import paper_2607_26253_amd as sara
    lengths = [600] + [120 + u for u in range(63)]      # 9,900 tokens
    cfg = generic_cfg(512, 8, 1, 64, 65536, lengths, vocab=512)
    pool = W.pool_with_lengths(cfg, lengths)            # of 38,336 at most: a chunk of 32,768 rows would take 4.5 GB
    g = torch.Generator(device="cuda").manual_seed(11)
    w = [(torch.randn(shape, generator=g, device="cuda") * 0.02 if len(shape) == 2 else torch.ones(shape, device="cuda"))
         .to(torch.bfloat16) for _, shape in W.weight_specs(cfg["model"])]
    need = 2 * sum(t.numel() for t in w)      # the context's copy
    out = []
    for short in (False, True):
        torch.cuda.empty_cache()
        hold = None
        if short:
            free = torch.cuda.mem_get_info()[0]
            # 3.5 GB left for the rest: a chunk of about 6,000 rows
            hold = torch.empty(free - need - (7 << 29), dtype=torch.uint8, device="cuda")
        ctx = sara.Sara(cfg["model"], cfg["alloc"], W.sampling_seed(cfg), [t.view(torch.int16) for t in w])
        d_tok, d_p = torch.from_numpy(pool["tokens"]).cuda(), torch.from_numpy(pool["p"]).cuda()
        ctx.sara_begin_step(d_tok, pool["offsets"], d_p, None, 0)
        buf = torch.zeros((cfg["alloc"]["n_slots"], 512), dtype=torch.float32, device="cuda")
        ctx.sara_decode_step(None, buf)
        out.append(buf.cpu().numpy().astype(np.float64))
        ctx.close()
        del hold
    a, b = out
    assert np.isfinite(a).all() and np.abs(a).max() > 0
    # other K splits of the prefill's o and down: other bf16 roundings, as against the oracle
    assert np.linalg.norm(a - b) <= 1e-2 * np.linalg.norm(a)
