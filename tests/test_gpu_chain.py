"""The draft chain (all micro-steps of a step in one launch), and the launch a micro-step that takes what the chain has no room
for, against the batched path's kernels on the same context."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    import paper_2510_25739_amd as H
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return H


# one and sixteen rows, guidance, slices on either side of an entry count of the draw and of a second round of strips,
# micro-steps up to what a context of one layer has room for; top-k of the list and of the dense form; greedy
@pytest.mark.parametrize("cfg,batch,scale,vocab,k,top_k,temperature", [
    (1, 1, 1.0, 16384, 5, 1000, 1.0), (2, 1, 1.0, 16384, 5, 4096, 0.8), (2, 3, 3.0, 8208, 7, 500, 1.0), (1, 16, 1.0, 12288, 2, 1000, 1.0),
    (2, 8, 2.0, 4096, 3, 4096, 1.0), (1, 5, 1.0, 2064, 7, 200, 1.0), (2, 16, 1.0, 4096, 1, 1000, 0.0), (1, 2, 1.0, 12304, 4, 3000, 1.0),
    (2, 9, 1.0, 16384, 2, 1000, 1.0), (1, 3, 1.0, 16384, 2, 1000, 1.0), (2, 4, 1.0, 8192, 1, 1000, 1.0)])
def test_draft_chain(H, cfg, batch, scale, vocab, k, top_k, temperature):
    compare_with_the_batched_path(H, cfg, batch, scale, vocab, k, top_k, temperature, one_launch=1)


# More micro-steps than the exchange slots have places for (at a depth of one layer 10 of sixteen B sequences, 6 of sixteen XL
# ones): slices of one round of the output projection's jobs, with and without idle workgroups, and of two; and the one or two
# micro-steps that stay launches of their own
@pytest.mark.parametrize("cfg,batch,scale,vocab,k", [
    (1, 16, 1.0, 8192, 11), (1, 16, 1.0, 12288, 12), (1, 8, 2.0, 12304, 11), (2, 16, 1.0, 4096, 8), (2, 8, 2.0, 8192, 7), (2, 16, 1.0, 16384, 7),
    (1, 1, 1.0, 16384, 1), (2, 16, 1.0, 16384, 1), (2, 4, 2.0, 8208, 2), (1, 4, 1.0, 12304, 2)])
def test_drafts_that_the_chain_does_not_take(H, cfg, batch, scale, vocab, k):
    compare_with_the_batched_path(H, cfg, batch, scale, vocab, k, 1000, 1.0, one_launch=0)


def compare_with_the_batched_path(H, cfg, batch, scale, vocab, k, top_k, temperature, one_launch):
    s = synth.CONFIGS[cfg].replace(n_layers=1, vocab=vocab, batch=batch, cfg_scale=scale, n_cond=6, grid_h=4, grid_w=max(8, k), k=k, top_k=top_k)
    hk = H.Hawk(H.HawkConfig.from_shape(s))
    hk.load(synth.make_weights(s, seed=5))
    rng = np.random.Generator(np.random.PCG64(9))
    uni = lambda *shp: rng.integers(0, 1 << 24, size=shp).astype(np.float32) / np.float32(1 << 24)  # noqa: E731
    hk.prefill(synth.make_cond(s, seed=2), synth.make_cond(s, seed=3) if s.use_cfg else None, s.grid_h, s.grid_w, temperature, top_k, scale, uni(batch))
    assert hk._L.hawk_draft_in_one_launch(hk._h, k) == one_launch
    N = s.grid_h * s.grid_w
    toks = rng.integers(0, vocab, size=(batch, N)).astype(np.int32)
    at = [1] * batch
    for to in (11, N - k + 1, N):   # in the middle, with the last prompts near the end, with the first ones finished
        goal = [min(to + b % 3, N) for b in range(batch)]
        while at != goal:   # (a prompt that is there gets its last token once more)
            at = [min(x, g - 1) + 1 for x, g in zip(at, goal)]
            hk.force([x - 1 for x in at], np.stack([toks[b, x - 1:x] for b, x in enumerate(at)]))
        n = hk.n()
        ke = [min(k, N - int(x) - 1) if x < N else -1 for x in n]
        u = uni(batch, k)
        d = hk.draft(k, u)
        q = hk.draft_logits(k)
        for b in range(batch):
            assert (d[b, max(ke[b], 0):] == -1).all()
            for i in range(max(ke[b], 0)):
                w, z = oracle.warp(q[b, i], temperature, top_k)
                assert d[b, i] == oracle.inv_cdf(w, z, float(u[b, i])), (b, i)
        fill = np.where(d >= 0, d, 0).astype(np.int32)
        hk.draft_forced(k, fill, False)
        same = hk.draft_logits(k)
        hk.set_path(0)
        hk.draft_forced(k, fill, False)
        other = hk.draft_logits(k)
        hk.set_path(1)
        worst = 0.0
        for b in range(batch):
            m = max(ke[b], 0)
            np.testing.assert_array_equal(q[b, :m], same[b, :m])
            if m:
                worst = max(worst, float(np.abs(q[b, :m] - other[b, :m]).max()))
        # both carry activations as two bf16 planes (16 bits): logits of about 1 from sums of d terms, 2^-17 apart per term
        # and micro-step, guidance weighing two streams
        assert worst <= 2e-4 * max(1.0, 2 * scale - 1), worst
    hk.close()


# Forcing commits any id of the vocabulary; the table of left-neighbour products has the slice's only.  The first micro-step's
# left neighbour below, in and behind the slice, at its edges, and all of them at once; two micro-steps carry it on.
@pytest.mark.parametrize("cfg,batch,scale", [(1, 1, 1.0), (2, 6, 1.0), (1, 8, 2.0), (2, 1, 3.0)])
@pytest.mark.parametrize("where", ["below", "in", "behind", "all"])
def test_draft_chain_behind_forced_tokens_outside_the_slice(H, cfg, batch, scale, where):
    lo, n, vocab, k = 37, 4096, 4800, 4
    s = synth.CONFIGS[cfg].replace(n_layers=1, vocab=vocab, samp_lo=lo, samp_n=n, batch=batch, cfg_scale=scale, n_cond=6, grid_h=4, grid_w=8, k=k, top_k=300)
    hk = H.Hawk(H.HawkConfig.from_shape(s))
    hk.load(synth.make_weights(s, seed=5))
    rng = np.random.Generator(np.random.PCG64(9))
    uni = lambda *shp: rng.integers(0, 1 << 24, size=shp).astype(np.float32) / np.float32(1 << 24)  # noqa: E731
    hk.prefill(synth.make_cond(s, seed=2), synth.make_cond(s, seed=3) if s.use_cfg else None, s.grid_h, s.grid_w, 1.0, s.top_k, scale, uni(batch))
    ids = {"below": [0, lo - 1, 17], "in": [lo, lo + n - 1, lo + 5], "behind": [lo + n, vocab - 1, vocab - 70]}
    ids["all"] = sum(ids.values(), [])
    at, ends = 1, 0
    while at + 2 <= 24:   # (past the first row of the grid, where there is an upper neighbour as well)
        last = [ids[where][(at // 2 + b) % len(ids[where])] for b in range(batch)]
        toks = np.stack([rng.integers(0, vocab, size=batch), last], axis=1).astype(np.int32)
        hk.force([at] * batch, toks)
        at += 2
        u = uni(batch, k)
        d = hk.draft(k, u)
        q = hk.draft_logits(k)
        for b in range(batch):
            for i in range(k):
                w, z = oracle.warp(q[b, i], 1.0, s.top_k)
                assert d[b, i] == lo + oracle.inv_cdf(w, z, float(u[b, i])), (at, b, i)
        hk.set_path(0)
        hk.draft_forced(k, d, False)
        other = hk.draft_logits(k)
        hk.set_path(1)
        worst = float(np.abs(q - other).max())
        # the bound of test_draft_chain; a left block of zeros instead moves these logits (of about 1) by tenths
        assert worst <= 2e-4 * max(1.0, 2 * scale - 1), (at, last, worst)
        ends += 1
    assert ends >= 11
    hk.close()
