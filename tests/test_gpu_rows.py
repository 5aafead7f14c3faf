"""GPU parity of the many-row passes (prompt rows and teacher-forced step rows of several sequences) against a
plain float64 forward, at sizes that take each of the products' kernels, both attention kernels and ragged
row counts; and of the sampling kernels' selection on rows whose value range it cannot cut linearly.

The bound on hidden states: a cache entry is fp16 (2^-11 relative), activations travel as bf16 pairs (2^-17),
sums are fp32.  The cache dominates: keys and values of relative error 2^-12 (round to nearest, on average half of it) and
weights whose scores of order one shift by as much change an attention output by about 2^-11 of its size, and
the output's share in the residual stream is below one: 2^-11 per layer, 1e-3 for the two layers here.
"""
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


def reference(s, blob, x):
    """Residual stream after all layers for rows x [sequence, position, d], causal, in float64."""
    import torch
    t = lambda name: torch.from_numpy(np.asarray(synth.blob_tensor(s, blob, name), dtype=np.float64))
    x = torch.from_numpy(x.astype(np.float64))
    S, T, d = x.shape
    nh, hd = s.n_heads, s.head_dim
    ang = torch.arange(T, dtype=torch.float64)[:, None] * s.rope_theta ** (-torch.arange(0, hd, 2, dtype=torch.float64) / hd)
    cos, sin = torch.cos(ang), torch.sin(ang)
    norm = lambda v, g: v / torch.sqrt((v * v).mean(-1, keepdim=True) + s.rms_eps) * g

    def heads(v, rotate):
        v = v.view(S, T, nh, hd).transpose(1, 2)
        if not rotate:
            return v
        a, b = v[..., 0::2], v[..., 1::2]
        return torch.stack((a * cos - b * sin, a * sin + b * cos), dim=-1).reshape(S, nh, T, hd)

    hidden = torch.full((T, T), float("-inf"), dtype=torch.float64).triu(1)
    for l in range(s.n_layers):
        a = norm(x, t(f"l{l}.g1"))
        q, k, v = (heads(a @ t(f"l{l}.{w}").T, w != "Wv") for w in ("Wq", "Wk", "Wv"))
        p = torch.softmax(q @ k.transpose(2, 3) / hd ** 0.5 + hidden, dim=-1)
        x = x + (p @ v).transpose(1, 2).reshape(S, T, d) @ t(f"l{l}.Wo").T
        a = norm(x, t(f"l{l}.g2"))
        x = x + (torch.nn.functional.silu(a @ t(f"l{l}.W1").T) * (a @ t(f"l{l}.W3").T)) @ t(f"l{l}.W2").T
    return x.numpy()


def relative(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def hidden_pair(H, s, chunk, want_logits=False, std=0.05):
    """Hidden states of the prompt rows and of a teacher-forced chunk of every sequence, and their reference."""
    blob = synth.make_weights(s, seed=4, std=std)
    hk = H.Hawk(H.HawkConfig.from_shape(s, k_max=max(chunk - 1, 0)))
    hk.load(blob)
    hk.set_path(0)
    cond = synth.make_cond(s, seed=2)
    unc = synth.make_cond(s, seed=3) if s.use_cfg else None
    hk.prefill(cond, unc, s.grid_h, s.grid_w, 1.0, s.top_k, s.cfg_scale, np.full(s.batch, 0.5, np.float32))
    got = [hk.last_hidden(s.n_cond).cpu().numpy().reshape(s.n_seq, s.n_cond, -1)]
    tok = np.zeros((s.batch, chunk), np.int64)
    tok[:, 0] = hk.grid()[:, 0]                  # the chunk's first row is the last committed token
    forced = np.random.Generator(np.random.PCG64(5)).integers(0, s.vocab, size=(s.batch, chunk)).astype(np.int32)
    tok[:, 1:] = forced[:, :-1]
    hk.force([1] * s.batch, forced)
    got.append(hk.last_hidden(chunk).cpu().numpy().reshape(s.n_seq, chunk, -1))
    x0 = cond if unc is None else np.concatenate([cond, unc])
    emb = np.asarray(synth.blob_tensor(s, blob, "E"))[np.tile(tok, (s.n_seq // s.batch, 1))]
    pair = np.concatenate(got, axis=1), reference(s, blob, np.concatenate([x0, emb], axis=1))
    return pair + (hk.logits(chunk), blob) if want_logits else pair


BASE = synth.HawkShape("rows", 2, 256, 4, 704, 1024, 16, 8, 8, 5, top_k=50)
SHAPES = [
    # d_model, heads, d_mlp, prompts, guidance, n_cond, chunk
    (256, 4, 704, 1, 1.0, 1, 1),       # one row everywhere
    (256, 2, 704, 1, 1.0, 65, 17),     # heads of 128; one row past a group of 64 keys and past a tile of 16 step rows
    (256, 4, 704, 3, 1.0, 67, 33),     # ragged tiles of (1, 1), (2, 2), (4, 2); three tiles of step rows
    (256, 4, 704, 10, 1.0, 50, 6),     # (2, 1), (4, 2), (6, 2)
    (256, 4, 704, 32, 1.0, 63, 2),     # (6, 2), LDS-staged (8, 8)
    (512, 4, 1376, 13, 2.0, 50, 3),    # (4, 1), (4, 3), (4, 4), LDS-staged (8, 8); heads of 128
    (512, 8, 1376, 32, 1.0, 63, 2),    # LDS-staged (8, 8) for QKV; (8, 12), weights in registers, for W1|W3
    (768, 12, 2048, 16, 2.0, 100, 2),  # (16, 8) for QKV and (18, 12) for W1|W3, weights in registers, ragged last groups
    (512, 8, 1376, 32, 1.0, 100, 2),   # LDS-staged (10, 8) for QKV and W1|W3
    (256, 4, 1376, 4, 1.0, 84, 5),     # (7, 3) for W1|W3
    (768, 12, 704, 2, 1.0, 56, 9),     # (3, 2) for QKV
    (768, 12, 1376, 13, 1.0, 80, 5),   # (7, 3) for Wo and W2
    # step attention with more cached positions than its waves request at once: eight waves, then four (from 256
    # workgroups on), heads of 64 (three tiles of 16 a wave) and of 128 (two)
    (256, 4, 704, 1, 1.0, 400, 5),
    (256, 2, 704, 1, 1.0, 270, 5),
    (256, 4, 704, 64, 1.0, 210, 2),
    (256, 2, 704, 128, 1.0, 140, 2),
]


@pytest.mark.parametrize("d,heads,mlp,batch,scale,n_cond,chunk", SHAPES)
def test_many_row_passes_match_a_float64_forward(H, d, heads, mlp, batch, scale, n_cond, chunk):
    s = BASE.replace(d_model=d, n_heads=heads, d_mlp=mlp, batch=batch, cfg_scale=scale, n_cond=n_cond, grid_w=max(8, chunk))
    got, ref = hidden_pair(H, s, chunk)
    prompt, step = relative(got[:, :n_cond], ref[:, :n_cond]), relative(got[:, n_cond:], ref[:, n_cond:])
    print(f"rows {s.n_seq * n_cond} + {s.n_seq * chunk}: relative error prompt {prompt:.2e}, step {step:.2e}")
    assert prompt < 1e-3 and step < 1e-3


# With the shapes above: every product kernel with every epilogue that the B, XL and 7B widths take it with, up to 4100 rows
# (asserted, with the library's own choice, in test_rows_dispatch.py).
KERNEL_SHAPES = [
    (768, 12, 352, 13, 1.0, 60, 37),   # (4, 3) two to a unit and (7, 3) for QKV; (3, 2), (4, 2), (6, 2) for Wo and W2
    (128, 2, 704, 20, 1.0, 53, 40),    # (4, 3) for QKV, (4, 3) two to a unit and (4, 4) for W1|W3
    (1024, 16, 704, 8, 1.0, 129, 9),   # (4, 1) for QKV, (2, 1) for W1|W3, (4, 3) two to a unit for Wo and W2
    (1280, 20, 352, 32, 1.0, 103, 4),  # LDS-staged (10, 8) for Wo and W2
    (512, 8, 352, 128, 1.0, 129, 1),   # weights in registers: (20, 12) for QKV, (16, 12) for Wo, (16, 16) for W1|W3, (18, 12) for W2
]


@pytest.mark.parametrize("d,heads,mlp,batch,scale,n_cond,chunk", KERNEL_SHAPES)
def test_every_product_kernel_and_epilogue(H, d, heads, mlp, batch, scale, n_cond, chunk):
    # weights of deviation 0.8 / sqrt(d): scores of order one, which the bound rests on (see the next test)
    s = BASE.replace(d_model=d, n_heads=heads, d_mlp=mlp, batch=batch, cfg_scale=scale, n_cond=n_cond, grid_w=max(8, chunk))
    got, ref = hidden_pair(H, s, chunk, std=0.8 / d ** 0.5)
    prompt, step = relative(got[:, :n_cond], ref[:, :n_cond]), relative(got[:, n_cond:], ref[:, n_cond:])
    print(f"rows {s.n_seq * n_cond} + {s.n_seq * chunk}: relative error prompt {prompt:.2e}, step {step:.2e}")
    assert prompt < 1e-3 and step < 1e-3


@pytest.mark.parametrize("d,heads,mlp,vocab,batch", [
    (256, 8, 704, 1024, 5),       # heads of 32
    (288, 9, 488, 1000, 3),       # hidden features and vocabulary slice in no whole tiles
    (4352, 17, 352, 1008, 2),     # heads of 256, more than 256 partial sums of squares a row
    (32, 2, 2048, 1024, 30),      # one k-step of 32, W1|W3 LDS-staged; heads of 16
])
def test_other_shapes_match_a_float64_forward(H, d, heads, mlp, vocab, batch):
    # Weights of deviation 0.8 / sqrt(d), as 0.05 is at 256: queries and keys of size 0.8 and so scores of order one, which
    # the bound above rests on (0.05 at 4352 gives scores of order ten: 1.5e-3).  Logits, of size 0.8, carry the hidden
    # states' relative error.
    s = BASE.replace(d_model=d, n_heads=heads, d_mlp=mlp, vocab=vocab, batch=batch, n_cond=21)
    got, ref, logits, blob = hidden_pair(H, s, 6, want_logits=True, std=0.8 / d ** 0.5)
    assert relative(got, ref) < 1e-3
    x = ref[:, -6:]
    want = x / np.sqrt((x * x).mean(-1, keepdims=True) + s.rms_eps) * synth.blob_tensor(s, blob, "g_f") @ synth.blob_tensor(s, blob, "W_out").T.astype(np.float64)
    assert relative(logits, want) < 1e-3


def test_queries_beyond_the_range_of_a_half(H):
    # The first feature pair of every head's queries is around 2^20 and meets keys of zero: the scores, and with them the
    # hidden states, are those of the other features.  These are 2^-20 of the row's largest, where a pair of halves moved
    # up to 2^14 still holds 2^-18 of them: within the bound above.
    s = BASE.replace(n_heads=2, n_cond=20)
    blob = synth.make_weights(s, seed=4, std=0.05)
    import torch
    lay = synth.blob_layout(s)
    pairs = [h * s.head_dim + e for h in range(s.n_heads) for e in (0, 1)]
    for l in range(s.n_layers):
        for name, factor in (("Wq", 2.0 ** 21), ("Wk", 0.0)):
            off, shape = lay[f"l{l}.{name}"]
            w = torch.from_numpy(blob[off:off + 2 * shape[0] * shape[1]]).view(torch.bfloat16).view(shape)
            w[pairs] *= factor
    cond = synth.make_cond(s, seed=2)
    hk = H.Hawk(H.HawkConfig.from_shape(s, k_max=3))
    hk.load(blob)
    hk.set_path(0)
    hk.prefill(cond, None, s.grid_h, s.grid_w, 1.0, s.top_k, 1.0, np.full(1, 0.5, np.float32))
    got = [hk.last_hidden(s.n_cond).cpu().numpy().reshape(1, s.n_cond, -1)]
    tok = np.concatenate([hk.grid()[:, :1], [[7, 9, 11]]], axis=1)
    hk.force([1], tok[:, 1:].astype(np.int32))
    got.append(hk.last_hidden(3).cpu().numpy().reshape(1, 3, -1))
    emb = np.asarray(synth.blob_tensor(s, blob, "E"))[tok[:, :3]]
    ref = reference(s, blob, np.concatenate([cond, emb], axis=1))
    assert relative(np.concatenate(got, axis=1), ref) < 1e-3


@pytest.mark.parametrize("heads", [4, 2])   # of 64 and of 128
def test_rows_do_not_feel_what_they_do_not_see(H, heads):
    # a condition row, then a token of a chunk, that is NaN: the rows before it are the same to the bit as without it
    s = BASE.replace(n_heads=heads, n_cond=70, batch=2)
    blob = synth.make_weights(s, seed=4, std=0.05)
    off, shape = synth.blob_layout(s)["E"]
    forced = np.array([[3, 5, 900, 7], [2, 4, 900, 8]], np.int32)
    u = np.full(2, 0.5, np.float32)

    def run(cond, blob, feed):
        hk = H.Hawk(H.HawkConfig.from_shape(s, k_max=3))
        hk.load(blob)
        hk.set_path(0)
        hk.prefill(cond, None, s.grid_h, s.grid_w, 1.0, s.top_k, 1.0, u)
        if not feed:
            return hk.last_hidden(s.n_cond).cpu().numpy().reshape(2, s.n_cond, -1)
        hk.force([1, 1], forced)     # rows: the last token of the prompt pass, then 3, 5, 900 and 2, 4, 900
        return hk.last_hidden(4).cpu().numpy().reshape(2, 4, -1)

    cond = synth.make_cond(s, seed=2)
    clean, bad = run(cond, blob, False), cond.copy()
    bad[0, 66], bad[1, 9] = np.nan, np.nan
    got = run(bad, blob, False)
    np.testing.assert_array_equal(got[0, :66], clean[0, :66])
    np.testing.assert_array_equal(got[1, :9], clean[1, :9])
    assert np.isnan(got[0, 66:]).all() and np.isnan(got[1, 9:]).all()
    clean, holed = run(cond, blob, True), blob.copy()
    holed[off:off + 2 * shape[0] * shape[1]].view(np.uint16).reshape(shape)[900] = 0x7FC0
    got = run(cond, holed, True)
    np.testing.assert_array_equal(got[:, :3], clean[:, :3])
    assert np.isnan(got[:, 3]).all()


HARD_ROWS = {
    "narrower than a bin can resolve": lambda rng, n: (rng.integers(0, 3, n) * 1e-38).astype(np.float32),
    "all equal": lambda rng, n: np.zeros(n, np.float32),
    "few values": lambda rng, n: rng.integers(0, 4, n).astype(np.float32),
    "masked with -inf": lambda rng, n: np.where((rng.random(n) < 0.99) & (np.arange(n) > 3), -np.inf, rng.standard_normal(n)).astype(np.float32),
    "masked with the lowest value": lambda rng, n: np.where((rng.random(n) < 0.99) & (np.arange(n) > 3), np.finfo(np.float32).min, rng.standard_normal(n)).astype(np.float32),
    "one far outlier": lambda rng, n: np.concatenate([[1e6], rng.standard_normal(n - 1)]).astype(np.float32),
}


@pytest.mark.parametrize("n,top_k", [(257, 40), (4097, 64), (8192, 1000), (8193, 2048), (16384, 3000)])
@pytest.mark.parametrize("kind", HARD_ROWS)
def test_selection_on_rows_without_a_useful_linear_cut(H, kind, n, top_k):
    import torch
    rng = np.random.Generator(np.random.PCG64(n))
    rows = np.stack([HARD_ROWS[kind](rng, n) for _ in range(4)])
    u = np.array([0.0, 0.3, 0.77, 1.0 - 2.0 ** -24], np.float32)
    got = H.sample_rows(torch.from_numpy(rows).cuda(), torch.from_numpy(u).cuda(), 1.0, top_k).cpu().numpy()
    want = []
    for r in range(4):
        w, z = oracle.warp(rows[r], 1.0, top_k)
        want.append(oracle.inv_cdf(w, z, float(u[r])))
    np.testing.assert_array_equal(got, want)


def _uniforms(rng, *shape):
    return (rng.integers(0, 1 << 24, size=shape).astype(np.float32) / np.float32(1 << 24)).astype(np.float32)


@pytest.mark.parametrize("n,top_k", [(64, 63), (257, 40), (257, 256), (1200, 1150), (2000, 1990), (2303, 2047), (8192, 1000), (16384, 3000)])
@pytest.mark.parametrize("kind", HARD_ROWS)
def test_candidates_on_rows_without_a_useful_linear_cut(H, kind, n, top_k):
    # every list and dense form of the recursion on such rows; residual masses are sums of fp64 weights of one row's
    # mass (1e-13: rounding of up to n additions of terms below one, in another order)
    import torch
    rng = np.random.Generator(np.random.PCG64(n + top_k))
    rows, m = 4, 2
    p = np.stack([HARD_ROWS[kind](rng, n) for _ in range(rows)])
    q = np.stack([np.stack([HARD_ROWS[kind](rng, n) for _ in range(m)]) for _ in range(rows)])
    cand = rng.integers(0, n, size=(rows, m)).astype(np.int32)
    cand[0] = np.argmax(q[0], axis=1)
    u_acc, u_fin = _uniforms(rng, rows, m), _uniforms(rng, rows)
    want = [oracle.multi_verify(p[r], q[r], cand[r], u_acc[r], float(u_fin[r]), 1.0, top_k, want_resid=True) for r in range(rows)]
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    for ws in (None, torch.empty(H.multi_verify_workspace_bytes(rows, m), dtype=torch.uint8, device="cuda:0")):
        idx, tok, resid = (x.cpu().numpy() for x in H.multi_verify(t(p), t(q), t(cand), t(u_acc), t(u_fin), 1.0, top_k, want_resid=True, workspace=ws))
        np.testing.assert_array_equal(idx, [w[0] for w in want])
        np.testing.assert_array_equal(tok, [w[1] for w in want])
        np.testing.assert_allclose(resid, [w[2] for w in want], rtol=1e-11, atol=1e-13)


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("vocab,top_k", [(200, 40), (200, 199), (256, 255)])
def test_stored_lists_hold_entries_of_the_row_only(H, vocab, top_k, sign):
    # One output row far larger than the others: its logit is the row's largest or smallest, and where it is the
    # largest (one of the signs) all others share the lowest bin of the linear cut with the places past the row's
    # end.  The lists a verify pass leaves are the last arrays of an fp32 context's workspace: lengths, indices, weights.
    s = synth.CONFIGS[0].replace(vocab=vocab, top_k=top_k, k=3)
    blob = synth.make_weights(s, seed=1)
    off, shape = synth.blob_layout(s)["W_out"]
    blob[off:off + 4 * shape[0] * shape[1]].view(np.float32).reshape(shape)[7] *= sign * 1e5
    cfg = H.HawkConfig.from_shape(s)
    hk = H.Hawk(cfg)
    hk.load(blob)
    cap, rows = 2048 + 256, s.k + 1                 # entries of a list, rows of a pass
    up = lambda b: (b + 255) & ~255
    end = H.workspace_bytes(cfg) + hk._ws_ptr - hk._ws.data_ptr()
    lw = end - up(rows * cap * 8)
    lidx = lw - up(rows * cap * 4)
    llen = lidx - up(rows * 4)
    rng = np.random.Generator(np.random.PCG64(3))
    hk.prefill(synth.make_cond(s, seed=2), None, s.grid_h, s.grid_w, 1.0, top_k, 1.0, _uniforms(rng, 1))
    whole = 0
    for _ in range(6):
        hk.draft(s.k, _uniforms(rng, 1, s.k))
        hk.verify(s.k, _uniforms(rng, 1, s.k), _uniforms(rng, 1))
        raw = hk._ws.cpu().numpy()
        length = raw[llen:llen + rows * 4].view(np.int32)
        idx = raw[lidx:lidx + rows * cap * 4].view(np.int32).reshape(rows, cap)
        w = raw[lw:lw + rows * cap * 8].view(np.float64).reshape(rows, cap)
        logits = hk.logits(rows)[0]
        for r in range(rows):
            n, low, high = int(length[r]), logits[r].min(), logits[r].max()
            # without ties the list is everything from the cut's bin up: the whole row where that is the lowest bin
            bins = ((logits[r] - low) * ((1024 - 0.01) / (high - low))).astype(int)
            assert n == (bins >= np.sort(bins)[vocab - top_k]).sum() and n >= top_k
            assert n == vocab or logits[r, 7] < high
            assert (np.diff(idx[r, :n]) > 0).all() and idx[r, 0] >= 0 and idx[r, n - 1] < vocab
            assert (w[r, :n] > 0).sum() <= top_k
            whole += n == vocab
    print("rows listed whole:", whole)
