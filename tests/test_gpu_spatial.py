"""GPU parity of the spatial drafting structures (Method, "Dual Direction Drafting Heads" and
"Spatial Sampling Pool"; appendix "Draft Heads Structure and Memory Overhead") against the oracle:
the heads' logits within the bf16 tolerance, everything that moves or indexes (cache, pool, counts,
member order) bit-exact, candidates and verification bit-exact on the GPU's own logits.

Inputs are seeded and synthetic: hidden states N(0, 1), head matrices N(0, 0.02^2), output-layer
rows N(0, 0.04^2) (logits of standard deviation about 1.5, as in the other tests), accept lengths
uniform over 0..k, uniforms on the 2^-24 grid.
"""
import numpy as np
import pytest

import oracle
import synth
from oracle import spatial

pytestmark = pytest.mark.gpu

LOGIT_TOL = 2e-2   # max-abs bound on bf16-path logits


@pytest.fixture(scope="module")
def H():
    import torch
    import paper_2510_25739_amd as H
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return H


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def bf16_tensor(bits):
    import torch
    return dev(bits.view(np.int16)).view(torch.bfloat16)


HEAD_CASES = [
    # rows, n_heads, d, V_s
    (6, 4, 1280, 16384),    # the XL shape: two horizontal and two vertical heads on the six rows of a verify pass
    (1, 2, 256, 1008),      # one row, ragged output layer
    (5, 3, 192, 4096),      # d a multiple of 64 only
    (7, 4, 512, 2000),      # more than sixteen (row, head) pairs, ragged output layer
    (12, 4, 4096, 8192),    # the 7B shape: twelve rows (two guidance streams), 8192-entry slice
    (16, 4, 768, 16384),    # 64 (row, head) pairs over a full slice, each weight drawn once
    (24, 4, 1280, 4096),    # two row tiles a weight: (2, 2)
    (65, 4, 256, 16400),    # LDS-staged with row-major weights, ragged both ways: (16, 8)
    (64, 4, 512, 16384),    # (8, 8)
    (150, 4, 512, 16384),   # (20, 12)
]


@pytest.mark.parametrize("rows,n_heads,d,v_s", HEAD_CASES)
def test_heads_match_oracle(H, rows, n_heads, d, v_s):
    h, wh, wo = synth.make_spatial_heads(10 + rows, rows, n_heads, d, v_s)
    q, g = H.spatial_heads(dev(h), bf16_tensor(wh), bf16_tensor(wo), want_g=True)
    q, g = q.cpu().numpy(), g.cpu().numpy()
    o_g, o_q = spatial.spatial_heads(h, synth.bf16_bits_to_f32(wh), synth.bf16_bits_to_f32(wo))
    err_g, err_q = np.abs(g - o_g).max(), np.abs(q.astype(np.float64) - o_q).max()
    print(f"max-abs error: g {err_g:.2e}, logits {err_q:.2e} (logit std {o_q.std():.2f})")
    assert err_g < 2e-3 and err_q < LOGIT_TOL
    assert o_q.std() > 0.5


def scripted_run(H, IW, IH, VSD, HD, v_s, k, temperature, top_k, seed, steps=None, start=0):
    """A raster walk with random accept lengths; every structure compared at every step."""
    import torch
    rng = np.random.Generator(np.random.PCG64(seed))
    n_heads, m_max, n_pos = HD + VSD, VSD + 1, IW * IH
    cache_g = H.SpecCache(IW, IH, VSD, v_s)
    cache_o = spatial.SpecCache(IW, IH, VSD)
    T, step = start, 0
    seen_m = set()
    while T < n_pos and (steps is None or step < steps):
        rows = k + 1
        # logits of all heads on the rows of a verify pass: heads 0..HD-1 horizontal, the rest vertical
        q_all = synth.make_logit_rows(seed * 1000 + step, (rows, n_heads, v_s))
        a = int(rng.integers(0, min(k, n_pos - 1 - T) + 1))     # drafts accepted: positions T .. T + a are committed
        pos = np.array([T + i if i <= a else -1 for i in range(rows)], dtype=np.int32)
        q_dev = dev(q_all)
        cache_g.push(dev(pos), q_dev.view(-1)[HD * v_s:], n_heads * v_s)
        for i in range(a + 1):
            cache_o.push(T + i, [q_all[i, HD + d] for d in range(VSD)])
        Tn = T + a                                              # the last committed position
        # pools for the positions the horizontal heads of row a point to (some beyond the image)
        target = np.array([Tn + j for j in range(1, HD + 1)], dtype=np.int32)
        logits, m, delta = cache_g.pool(dev(target), q_dev.view(-1)[a * n_heads * v_s:], v_s)
        logits, m_h, delta_h = logits.cpu().numpy(), m.cpu().numpy(), delta.cpu().numpy()
        u_draw = synth.make_uniforms(seed * 7919 + step, (HD, m_max))
        u_acc = synth.make_uniforms(seed * 104729 + step, (HD, m_max))
        u_fin = synth.make_uniforms(seed * 1299709 + step, (HD,))
        p_rows = synth.make_logit_rows(seed * 31 + step + 500000, (HD, v_s))
        cand = H.sample_rows(dev(logits.reshape(HD * m_max, v_s)), dev(u_draw.reshape(-1)), temperature, top_k,
                             skip=dev(delta_h.reshape(-1))).view(HD, m_max)
        idx, tok = H.multi_verify(dev(p_rows), dev(logits), cand, dev(u_acc), dev(u_fin), temperature, top_k, m_rows=m)
        ws = torch.empty(H.multi_verify_workspace_bytes(HD, m_max), dtype=torch.uint8, device="cuda:0")
        idx2, tok2 = H.multi_verify(dev(p_rows), dev(logits), cand, dev(u_acc), dev(u_fin), temperature, top_k,
                                    m_rows=m, workspace=ws)
        assert torch.equal(idx, idx2) and torch.equal(tok, tok2)
        cand_h, idx_h, tok_h = cand.cpu().numpy(), idx.cpu().numpy(), tok.cpu().numpy()
        for j in range(HD):
            t = int(target[j])
            if t >= n_pos:
                assert m_h[j] == 0 and (delta_h[j] == -1).all() and (cand_h[j] == -1).all()
                w, z = oracle.warp(p_rows[j], temperature, top_k)
                assert idx_h[j] == 0 and tok_h[j] == oracle.inv_cdf(w, z, float(u_fin[j]))
                continue
            pool = cache_o.pool(t, q_all[a, j])
            seen_m.add(len(pool))
            assert m_h[j] == len(pool)
            assert list(delta_h[j]) == [dv for dv, _ in pool] + [-1] * (m_max - len(pool))
            for i, (dv, row) in enumerate(pool):
                np.testing.assert_array_equal(logits[j, i], row)
                w, z = oracle.warp(row, temperature, top_k)
                assert cand_h[j, i] == oracle.inv_cdf(w, z, float(u_draw[j, i]))
            assert (cand_h[j, len(pool):] == -1).all()
            mm = len(pool)
            o_idx, o_tok = oracle.multi_verify(p_rows[j], logits[j, :mm], cand_h[j, :mm], u_acc[j, :mm], float(u_fin[j]),
                                               temperature, top_k)
            assert (idx_h[j], tok_h[j]) == (o_idx, o_tok)
        T = Tn + 1
        step += 1
    return seen_m, cache_o


@pytest.mark.parametrize("IW,IH,VSD,HD,v_s,k,temperature,top_k", [
    (6, 7, 2, 2, 64, 3, 1.0, 20),        # small image walked from the first to the last position
    (5, 9, 3, 1, 100, 4, 0.8, 100),      # three depths, ragged row, whole vocabulary kept
    (8, 4, 1, 3, 1000, 5, 1.0, 50),      # one depth, three horizontal heads
    (4, 6, 4, 2, 48, 2, 0.0, 10),        # greedy; deeper than the image leaves room for
])
def test_cache_and_pool_walk_matches_oracle(H, IW, IH, VSD, HD, v_s, k, temperature, top_k):
    seen_m, cache_o = scripted_run(H, IW, IH, VSD, HD, v_s, k, temperature, top_k, seed=IW * 10 + VSD)
    assert 1 in seen_m and min(VSD, IH - 1) + 1 in seen_m    # top rows without vertical members, full pools later
    assert cache_o.peak <= spatial.cache_entries(IW, VSD)


def test_cache_and_pool_full_size(H):
    # the XL image (24 x 24, 16384-entry vocabulary, top-k 1000), two depths, two horizontal heads, k = 5
    seen_m, cache_o = scripted_run(H, 24, 24, 2, 2, 16384, 5, 1.0, 1000, seed=99, steps=40)
    assert seen_m == {1, 2, 3}
    assert cache_o.peak == spatial.cache_entries(24, 2)


def test_pipeline_full_size_heads_to_verification(H):
    # heads -> cache -> pool -> candidates -> verification in one go at the XL shape: the logits stay
    # within tolerance of the oracle's, and everything after them is exact on the GPU's own logits
    import torch
    IW, IH, VSD, HD, d, v_s, k = 24, 24, 2, 2, 1280, 16384, 5
    n_heads, m_max = HD + VSD, VSD + 1
    h, wh, wo = synth.make_spatial_heads(5, (k + 1) * 3, n_heads, d, v_s)
    Wh, Wo = bf16_tensor(wh), bf16_tensor(wo)
    fh, fo = synth.bf16_bits_to_f32(wh), synth.bf16_bits_to_f32(wo)
    cache = H.SpecCache(IW, IH, VSD, v_s)
    T = 100
    errs = []
    for step, a in enumerate((5, 2, 0)):
        hs = h[step * (k + 1):(step + 1) * (k + 1)]
        q = H.spatial_heads(dev(hs), Wh, Wo)
        _, o_q = spatial.spatial_heads(hs, fh, fo)
        errs.append(np.abs(q.cpu().numpy().astype(np.float64) - o_q).max())
        pos = np.array([T + i if i <= a else -1 for i in range(k + 1)], dtype=np.int32)
        cache.push(dev(pos), q.view(-1)[HD * v_s:], n_heads * v_s)
        T += a + 1
    assert max(errs) < LOGIT_TOL
    # a line further down the positions pushed above are one row up
    target = np.array([100 + IW, 101 + IW, 105 + IW + 1, 100 + 2 * IW], dtype=np.int32)
    q_h = synth.make_logit_rows(77, (len(target), v_s))
    logits, m, delta = cache.pool(dev(target), dev(q_h), v_s)
    assert delta.cpu().tolist() == [[1, 0, -1], [1, 0, -1], [1, 0, -1], [2, 0, -1]]
    n = len(target)
    u_draw, u_acc, u_fin = (synth.make_uniforms(s, shp) for s, shp in ((1, (n, m_max)), (2, (n, m_max)), (3, (n,))))
    cand = H.sample_rows(logits.view(n * m_max, v_s), dev(u_draw.reshape(-1)), 1.0, 1000, skip=delta.view(-1)).view(n, m_max)
    p_rows = (logits[:, 0] + dev(synth.make_logit_rows(78, (n, v_s), std=1.0))).contiguous()
    idx, tok = H.multi_verify(p_rows, logits, cand, dev(u_acc), dev(u_fin), 1.0, 1000, m_rows=m)
    lg, ch, pr = logits.cpu().numpy(), cand.cpu().numpy(), p_rows.cpu().numpy()
    for j in range(n):
        mm = int(m[j])
        for i in range(mm):
            w, z = oracle.warp(lg[j, i], 1.0, 1000)
            assert ch[j, i] == oracle.inv_cdf(w, z, float(u_draw[j, i]))
        o = oracle.multi_verify(pr[j], lg[j, :mm], ch[j, :mm], u_acc[j, :mm], float(u_fin[j]), 1.0, 1000)
        assert (int(idx[j]), int(tok[j])) == o
