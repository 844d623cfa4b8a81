"""Decode attention of many rows: the rollouts of a prompt share the blocks of
its prompt pages, and every row's logits stay bit-identical to a small batch's,
whose rows have blocks of their own."""
import numpy as np
import pytest
import torch

import workloads as W
from tests.gpu_harness import device_setup, slot_rows, upload_pool
from tests.test_gpu_prefill import generic_cfg

pytestmark = pytest.mark.gpu


def logits_by_rollout(cfg, w, pool, slots, forced, steps):
    cfg["alloc"]["n_slots"] = slots
    ctx, _ = device_setup(cfg, w)
    d_tok, d_p, _ = upload_pool(pool)
    ctx.sara_begin_step(d_tok, pool["offsets"], d_p, None, 0)
    k, bufs = cfg["alloc"]["k"], []
    for _ in range(steps):
        buf = torch.full((slots, cfg["model"]["vocab"]), -7.0, dtype=torch.float32, device="cuda")
        ctx.sara_decode_step(forced, buf)
        bufs.append(buf)
        ctx.sara_posterior_decide()
        ctx.sara_refill()
    asg = ctx.read_logs()["assigns"]
    ctx.close()
    return {(u, j): [b[s] for b in bufs] for t, s, u, j in asg if t == 0}, k


@pytest.mark.parametrize("hq,hkv,hd,n0,prompts", [
    (8, 1, 64, 8, 40),      # 2 rows a tile, 8 an item
    (12, 2, 128, 8, 33),    # 6 columns a row
    (10, 2, 64, 7, 40),     # 3 rows a tile, 12 an item
    (8, 2, 128, 5, 60),     # 4 rows a tile
    (2, 2, 64, 9, 30),      # 16 rows a tile, one head a group
    (7, 1, 64, 3, 90),
])
def test_shared_prompt_splits_are_bit_identical(hq, hkv, hd, n0, prompts):
    # prompt pages: none, below a split of 8, exactly 1 and 2 splits, a partial last page, several splits
    lens = [2, 100, 129, 257, 250, 390, 700]
    lengths = [lens[u % len(lens)] for u in range(prompts)]
    cfg = generic_cfg(512, hq, hkv, hd, 512, lengths, k=max(2, n0), n0=n0, budget_N=prompts * max(2, n0), max_new=40)
    w, pool = W.make_weights(cfg), W.pool_with_lengths(cfg, lengths)
    g = np.random.default_rng(3)
    forced = torch.from_numpy(g.integers(0, 500, (prompts * max(2, n0), 40)).astype(np.int32)).cuda()
    steps = 18
    many, _ = logits_by_rollout(cfg, w, pool, prompts * n0, forced, steps)
    few, k = logits_by_rollout(cfg, w, pool, 7 * n0, forced, steps)
    assert len(many) == prompts * n0 > 256 and len(few) == 7 * n0
    for key, rows in few.items():
        for t, (a, b) in enumerate(zip(rows, many[key])):
            assert bool(torch.isfinite(a).all()) and torch.equal(a, b), (key, t)


@pytest.mark.parametrize("top_p,temperature", [(1.0, 1.0), (1.0, 0.7), (0.9, 1.0), (0.9, 0.7)])
@pytest.mark.parametrize("width,n0,prompts", [((1536, 6, 2, 64, 8960), 7, 120), ((1024, 6, 1, 128, 4096), 8, 400)])
def test_many_row_graph_is_bit_identical(width, n0, prompts, top_p, temperature):
    """Many live rows (840 of a wide model, 3,200 of a narrow one): sara_run
    replays the loop with the 256-row tile GEMMs, the eager calls run the
    few-row kernels; sampled tokens, logs and the state both leave behind are
    the same, also once rollouts have ended and few rows are left.  For both
    samplers, with and without a temperature."""
    lengths = [2 + (7 * u) % 60 for u in range(prompts)]
    cfg = generic_cfg(*width, lengths, vocab=1008, k=8, n0=n0, budget_N=prompts * 8, max_new=40, top_p=top_p,
                      temperature=temperature)
    cfg["alloc"].update(n_slots=prompts * n0, commit_min=8, forced_eos_u32=(1 << 32) // 24, pool_U=prompts)
    w, pool, seed = W.make_weights(cfg), W.pool_with_lengths(cfg, lengths), None
    out = []
    for graph in (True, False):
        ctx, _ = device_setup(cfg, w)
        d_tok, d_p, _ = upload_pool(pool)
        ctx.sara_begin_step(d_tok, pool["offsets"], d_p, None, 0)
        if graph:
            ctx.sara_run(None, graph_iters=3)
        else:
            while not ctx.sara_query()["done"]:
                ctx.sara_decode_step()
                ctx.sara_posterior_decide()
                ctx.sara_refill()
        out.append((ctx.read_rollouts(), ctx.read_logs(), ctx.sara_query()))
        ctx.close()
    (ra, la, qa), (rb, lb, qb) = out
    assert qa["tokens"] == qb["tokens"] > 0 and qa["decode_steps"] == qb["decode_steps"]
    for key in ra:
        assert np.array_equal(ra[key], rb[key]), key
    for key in la:
        assert np.array_equal(la[key], lb[key]), key


@pytest.mark.parametrize("graph_iters", [1, 5])
def test_run_follows_the_table_of_each_call(graph_iters):
    """One context, captured loops kept: every sara_run takes the forced table
    (or none) of its own call."""
    lengths = [3 + u for u in range(12)]
    cfg = generic_cfg(512, 4, 2, 64, 512, lengths, k=2, n0=2, budget_N=24, max_new=9)
    cfg["model"]["eos_id"] = -1
    cfg["alloc"].update(n_slots=24)
    w, pool = W.make_weights(cfg), W.pool_with_lengths(cfg, lengths)
    ctx, _ = device_setup(cfg, w)
    d_tok, d_p, _ = upload_pool(pool)
    g = np.random.default_rng(4)
    a, b = (torch.from_numpy(g.integers(0, 500, (24, 9)).astype(np.int32)).cuda() for _ in range(2))

    def tokens(table, graph=True):
        ctx.sara_begin_step(d_tok, pool["offsets"], d_p, None, 0)
        if graph:
            ctx.sara_run(table, graph_iters=graph_iters)
        else:
            while not ctx.sara_query()["done"]:
                ctx.sara_decode_step(table)
                ctx.sara_posterior_decide()
                ctx.sara_refill()
        return ctx.read_rollouts()["tokens"]

    free = tokens(None, graph=False)
    for table in (a, b, None, a, None, b):
        assert np.array_equal(tokens(table), free if table is None else table.cpu().numpy())
    ctx.close()
