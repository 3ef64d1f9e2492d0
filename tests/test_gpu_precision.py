"""How much the matrix-core GEMMs lose in their sums, which is far less than the parity tests can see (there the (hi, lo)
split of the activations and the cache's bf16 rows decide).  The weights repeat the first half of K negated in the second
half, the activations repeat it as it is: the exact result is zero, and what comes out is the rounding of the sums alone.

Bound: a matrix instruction adds its 32 products in four groups of eight and rounds the accumulator after each.  An entry's
running sum is a random walk that grows over the first half of K and shrinks over the second; with T groups of eight, C
accumulators that share them and one rounding of half a unit in the last place each, the error relative to the sum at the
middle is sqrt(T / (2 C) * 0.541 * 2^-46 / 12) (0.541: mean of the squared unit over a value's octave); 1.1 times that is allowed."""
import numpy as np
import pytest

from paper_2311_13581_amd import synth

pytestmark = pytest.mark.gpu

D = 4096
bits = synth.f32_to_bf16_bits


def rounded(x):
    return synth.bf16_bits_to_f32(bits(x)).reshape(np.shape(x))


def bound(groups, chains):
    return 1.1 * np.sqrt(groups / (2 * chains) * 0.541 * 2.0 ** -46 / 12)


def weights(shape, k, **given):
    """All zeros (norm gains one) but what is given, as bf16 bits."""
    d, F, V, H = shape.d_model, shape.d_ffn, shape.vocab, shape.n_heads * shape.head_dim
    z = {"tok_emb": (V, d), "lm_head": (V, d), "lookahead": (k, d)}
    W = {n: bits(given.get(n, np.zeros(s, np.float32))).reshape(s) for n, s in z.items()}
    W["final_norm"] = bits(given.get("final_norm", np.ones(d, np.float32)))
    for n, s in (("wq", (H, d)), ("wk", (H, d)), ("wv", (H, d)), ("wo", (d, H)), ("w_gate", (F, d)), ("w_up", (F, d)), ("w_down", (d, F))):
        W[n] = [bits(given.get(n, np.zeros(s, np.float32))).reshape(s)]
    for n in ("attn_norm", "ffn_norm"):
        W[n] = [bits(given.get(n, np.ones(d, np.float32)))]
    return W


@pytest.mark.parametrize("n,chains", [(200, 1), (100, 4)])
@pytest.mark.parametrize("strips", range(6))
def test_sums_of_the_prompt_pass(strips, n, chains):
    """Values of one layer's V projection over a prompt of equal tokens (every tile of the tiled GEMM, whole and in slices; 100
    rows, which add their products step by step, may lose no more than if four accumulators shared K): queries are zero, so the next call's attention output is their mean, and the LM head reads it off feature by feature."""
    from paper_2311_13581_amd import binding
    rng = np.random.default_rng(0)
    lead = 128  # features 0 .. 127 belong to the pending token alone, the rest to the prompt's token
    half = (D - lead) // 2
    shape = synth.ModelShape(1, D, 8, 128, 32, 1040, dtype=synth.BF16)
    H = shape.n_heads * shape.head_dim
    twice = lambda x, sign=1: np.concatenate([np.zeros(x.shape[:-1] + (lead,), np.float32), x, sign * x], -1)
    emb, gain = rng.standard_normal(half), 1 + 0.25 * rng.random(half)
    w = rounded(rng.standard_normal((H, half)).astype(np.float32))
    tok = np.zeros((shape.vocab, D), np.float32)
    tok[0], tok[1, :lead] = twice(emb.astype(np.float32)), 1
    head, wo = np.zeros((shape.vocab, D), np.float32), np.zeros((D, H), np.float32)
    wo[lead + np.arange(H), np.arange(H)] = 1
    head[np.arange(H), lead + np.arange(H)] = 1
    g = binding.Pass(binding.make_config(shape, 0, 1, 256, 64), {"prefill_tiled": 1, "tune.prefill_strips": strips})
    g.load_weights(weights(shape, 0, tok_emb=tok, lm_head=head, wv=twice(w, -1), wo=wo, attn_norm=twice(gain.astype(np.float32))))
    g.prefill(0, np.array([0] * n + [1], np.int32))
    g.draft([0], 0.0, 1)
    logits = g.get_logits(0, 0)[0, :H].astype(np.float64)
    g.close()
    err = logits * np.sqrt(lead / D + shape.rms_eps) * (n + 1) / n
    x = rounded(emb.astype(np.float32)).astype(np.float64)
    mid = (w * (x * rounded(gain.astype(np.float32)))).sum(1) / np.sqrt(2 * (x ** 2).sum() / D + shape.rms_eps)
    rel = np.sqrt((err ** 2).mean() / (mid ** 2).mean())
    print("rows", n, "tile", strips, "error of the sums", rel, "bound", bound(2 * half / 8, chains))
    assert 0 < rel < bound(2 * half / 8, chains)


@pytest.mark.parametrize("slots,k,blocks", [(1, 4, 0), (1, 8, 0), (2, 7, 0), (8, 4, 0), (8, 4, 6), (8, 4, 8), (8, 7, 0), (8, 7, 3), (8, 7, 8)])
def test_sums_of_the_decode_gemm(slots, k, blocks):
    """Logits of a drafting call on a model without layers' contributions: 5, 9, 16, 40 and 64 rows, with the launch shapes'
    own and more blocks per workgroup (pairs of accumulators and products added one by one).  Eight accumulators share K."""
    from paper_2311_13581_amd import binding
    rng = np.random.default_rng(1)
    shape = synth.ModelShape(1, D, 1, 128, 32, 1024, dtype=synth.BF16)
    twice = lambda x, sign=1: np.concatenate([x, sign * x], -1).astype(np.float32)
    w = rounded(rng.standard_normal((shape.vocab, D // 2)).astype(np.float32))
    emb, gain = rng.standard_normal((shape.vocab, D // 2)), 1 + 0.25 * rng.random(D // 2)
    la = rng.standard_normal((k, D // 2))
    g = binding.Pass(binding.make_config(shape, k, slots, 64, 64))
    g.load_weights(weights(shape, k, tok_emb=twice(emb), lm_head=twice(w, -1), lookahead=twice(la), final_norm=twice(gain)))
    if blocks:
        g.set_option("tune.gemm_cfg", 1000000 + 3 * 10000 + 400 + blocks)
    for s in range(slots):
        g.prefill(s, np.array([s], np.int32))
    g.draft(list(range(slots)), 0.0, 1)
    err = np.concatenate([g.get_logits(s, 0) for s in range(slots)]).astype(np.float64)
    g.close()
    x = rounded(np.concatenate([np.concatenate([emb[s:s + 1], la]) for s in range(slots)]).astype(np.float32)).astype(np.float64)
    inv = 1 / np.sqrt(2 * (x ** 2).sum(1) / D + shape.rms_eps)
    mid = (x * rounded(gain.astype(np.float32))) @ w.T.astype(np.float64) * inv[:, None]
    rel = np.sqrt((err ** 2).mean() / (mid ** 2).mean())
    print("rows", slots * (k + 1), "blocks", blocks, "error of the sums", rel, "bound", bound(D / 8, 8))
    assert 0 < rel < bound(D / 8, 8)


def as_splits(v):
    """Sums over the rows of v in 32 bits, as splits of up to 64 keys and a merge in split order give them: sixteen running sums
    of every sixteenth key, added one by one."""
    n = len(v)
    chunk = (-(-n // -(-n // 64)) + 15) // 16 * 16
    chain = lambda parts: np.add.accumulate(np.stack(parts), 0, np.float32)[-1]
    return chain([chain([chain(v[lo + g:min(n, lo + chunk):16]) for g in range(16)]) for lo in range(0, n, chunk)])


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("n", [100, 150, 184])
def test_sums_of_the_generic_attention(n, hd):
    """The generic attention's sums over 65 to 192 keys lose no more than a running sum for every sixteenth key of a split of 64, these
    added one by one, and the splits' after them would.  Queries are zero, so a drafting call's attention output is the mean of the prompt's values (positive ones, each a feature of the token's
    embedding) and the pending token's zeros, and the LM head reads it off; a factor common to all features (the final norm's) is taken
    out.  Bound: the same sums in 32 bits as splits, followed by the three roundings on the way out (division, norm, their product)."""
    from paper_2311_13581_amd import binding
    rng = np.random.default_rng(n)
    lead, H = 128, 1024
    shape = synth.ModelShape(1, lead + H, H // hd, hd, 32, H, dtype=synth.F32)
    z = lambda *s: np.zeros(s, np.float32)
    W = dict(tok_emb=z(H, shape.d_model), lm_head=z(H, shape.d_model), lookahead=z(0, shape.d_model), final_norm=z(shape.d_model) + 1,
             attn_norm=[z(shape.d_model) + 1], ffn_norm=[z(shape.d_model) + 1], wq=[z(H, shape.d_model)], wk=[z(H, shape.d_model)],
             wv=[z(H, shape.d_model)], wo=[z(shape.d_model, H)], w_gate=[z(32, shape.d_model)], w_up=[z(32, shape.d_model)], w_down=[z(shape.d_model, 32)])
    at = np.arange(H)
    W["wv"][0][at, lead + at] = W["wo"][0][lead + at, at] = W["lm_head"][at, lead + at] = 1
    W["tok_emb"][:n, lead:] = rng.integers(64, 128, (n, H)) / 64
    W["tok_emb"][n, :lead] = 1
    g = binding.Pass(binding.make_config(shape, 0, 1, 256, 16))
    g.load_weights(W)
    got, want = [], []
    for _ in range(8):
        order = rng.permutation(n)
        g.prefill(0, np.append(order, n).astype(np.int32))
        g.draft([0], 0.0, 1)
        x = W["tok_emb"][order, lead:].astype(np.float64)
        v = x / np.sqrt((x ** 2).sum(1, keepdims=True) / shape.d_model + shape.rms_eps)
        mean = v.sum(0) / (n + 1)
        norm = np.float32(0.7371)  # any factor: three roundings behind the sums
        for out, y in ((got, g.get_logits(0, 0)[0]), (want, as_splits(v.astype(np.float32)) / np.float32(n + 1) * norm / np.float32(1.217))):
            r = y.astype(np.float64) / mean
            out.append(r / r.mean() - 1)
    g.close()
    got, want = (np.sqrt(np.mean(np.square(e))) for e in (got, want))
    print("keys", n, "head", hd, "error of the sums", got, "as splits", want)
    assert 0 < got < want
