"""The stand-alone sampler where its split of the work changes: one row to more
rows than chunks are shared out for, vocabularies around the chunk sizes, rows
that are not 16-byte aligned, masked (-inf) and tied logits."""
import numpy as np
import pytest

from oracle import sampler as OS

pytestmark = pytest.mark.gpu


def tokens(logits, rid, pos, seed, step, temp, top_p, shift=0, noalloc=False):
    import torch

    import paper_2607_26253_amd as sara
    n, V = logits.shape
    flat = torch.empty(n * V + shift, dtype=torch.float32, device="cuda")
    flat[shift:] = torch.from_numpy(logits).cuda().reshape(-1)
    tok = torch.empty(n, dtype=torch.int32, device="cuda")
    f = sara.sara_sample_logits_noalloc if noalloc else sara.sara_sample_logits
    f(flat[shift:].view(n, V), torch.from_numpy(rid).cuda(), torch.from_numpy(pos).cuda(), seed, step, temp, -1, 0, tok,
      top_p=top_p)
    return tok.cpu().numpy()


@pytest.mark.parametrize("n,V,temp,top_p,shift", [
    (1, 5, 1.0, 1.0, 0), (1, 1024, 1.0, 1.0, 0), (1, 1025, 0.7, 1.0, 0), (1, 40001, 1.0, 1.0, 0), (1, 131072, 1.0, 1.0, 1),
    (3, 151936, 1.3, 1.0, 0), (65, 2052, 1.0, 1.0, 2), (70, 20484, 1.0, 1.0, 0), (5, 180000, 1.0, 1.0, 0),
    (1, 4096, 1.0, 0.9, 0), (63, 1000, 1.0, 0.8, 1), (65, 515, 0.7, 0.6, 0), (130, 2048, 1.0, 0.9, 0), (1030, 260, 1.0, 0.5, 0),
    (3, 151936, 1.0, 0.9, 0), (2, 100002, 0.7, 0.95, 0), (1025, 8196, 1.0, 0.9, 0),
])
def test_sampler_split(n, V, temp, top_p, shift):
    g = np.random.default_rng([n, V])
    logits = (g.standard_normal((n, V)) * 2.0).astype(np.float32)
    logits[:, g.integers(0, V, 3)] = -np.inf                 # masked ids
    if n > 1:
        logits[1] = np.float32(0.25)                         # every id tied
        logits[n - 1, V // 2:] = -np.inf                     # the last chunks hold no candidate
    if n > 4 and top_p == 1.0:
        logits[2, [V // 3, V - 2]] = np.inf                  # only infinite scores can win: the lowest of them
    rid, pos = np.arange(n, dtype=np.int32) * 3 + 1, (np.arange(n, dtype=np.int32) * 7) % 1024
    got = tokens(logits, rid, pos, 0x1234567890ABCDEF, 4, temp, top_p, shift)
    if n <= (64 if top_p < 1.0 else 4096):
        again = tokens(logits, rid, pos, 0x1234567890ABCDEF, 4, temp, top_p, shift, noalloc=True)
        assert np.array_equal(got, again)
    skipped = 0
    for i in sorted(set([0, 1, n // 2, n - 1]) & set(range(n))) if n > 100 else range(n):
        tok, sc = OS.sample(logits[i], temp, 0x1234567890ABCDEF, 4, int(rid[i]), int(pos[i]), top_p)
        if got[i] != tok:
            assert OS.near_tie(sc) or (top_p < 1.0 and OS.nucleus_margin(logits[i], temp, top_p) < 1e-8), (i, got[i], tok)
            skipped += 1
    assert skipped <= 1


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("top_p", [1.0, 0.9])
def test_decode_survives_nan_logits(dtype, top_p):
    """A model whose logits are all NaN has no best id; the step still runs to
    its end, with every rollout at the cap."""
    import workloads as W
    from tests.gpu_harness import device_setup, upload_pool
    from tests.test_gpu_prefill import generic_cfg
    lengths = [3, 9, 20]
    cfg = generic_cfg(512, 4, 2, 64, 512, lengths, max_new=5, top_p=top_p)
    cfg["model"].update(dtype=dtype, eos_id=-1)
    w = W.make_weights(cfg)
    w["lm_head"][:] = 0x7FC0 if dtype == "bf16" else np.nan
    ctx, _ = device_setup(cfg, w)
    pool = W.pool_with_lengths(cfg, lengths)
    d_tok, d_p, _ = upload_pool(pool)
    ctx.sara_begin_step(d_tok, pool["offsets"], d_p, None, 0)
    ctx.sara_run(None, graph_iters=4)
    q, r = ctx.sara_query(), ctx.read_rollouts()
    ctx.close()
    assert q["done"] and q["rollouts"] >= 3
    assert set(r["length"].tolist()) <= {0, 5} and (r["length"] == 5).sum() == q["rollouts"]
