"""The 12-bit copies of the weights (pass_coded_begin): what a product reads back out of them is bit for bit the plain weight, and
the products that read them agree with the plain ones."""
import ctypes as C

import numpy as np
import pytest

from paper_2311_13581_amd import synth

pytestmark = pytest.mark.gpu

bits = synth.f32_to_bf16_bits


def rounded(x):
    return synth.bf16_bits_to_f32(bits(x)).reshape(np.shape(x))


def random_weights(shape, k, seed, spread=0.0):
    """Normal weights; spread > 0: with zeros, weights far below and far above the rest."""
    rng = np.random.default_rng(seed)
    d, F, V, H, L = shape.d_model, shape.d_ffn, shape.vocab, shape.n_heads * shape.head_dim, shape.n_layers

    def m(r, c):
        w = rng.standard_normal((r, c), dtype=np.float32) * np.float32(0.02)
        u = rng.random((r, c), dtype=np.float32)
        w[u < spread] = 0
        w[u > 1 - spread / 8] *= 1e-6
        w[(u > 0.5) & (u < 0.5 + spread / 200)] *= 300
        return bits(w).reshape(r, c)

    one = bits(np.ones(d, np.float32))
    W = {"tok_emb": m(V, d), "lm_head": m(V, d), "final_norm": one, "lookahead": m(max(k, 1), d)[:k], "attn_norm": [one] * L, "ffn_norm": [one] * L}
    for n, (r, c) in (("wq", (H, d)), ("wk", (H, d)), ("wv", (H, d)), ("wo", (d, H)), ("w_gate", (F, d)), ("w_up", (F, d)), ("w_down", (d, F))):
        W[n] = [m(r, c) for _ in range(L)]
    return W


def head_only(d, V, head, k=1, tok=None, la=None):
    """A model of one layer that adds nothing: its logits are the LM head times the normalised embedding."""
    z, one = lambda *s: bits(np.zeros(s, np.float32)).reshape(s), bits(np.ones(d, np.float32))
    return {"tok_emb": z(V, d) if tok is None else bits(tok).reshape(V, d), "lm_head": bits(head).reshape(V, d), "final_norm": one,
            "lookahead": z(k, d) if la is None else bits(la).reshape(k, d), "attn_norm": [one], "ffn_norm": [one], "wq": [z(128, d)],
            "wk": [z(128, d)], "wv": [z(128, d)], "wo": [z(d, 128)], "w_gate": [z(32, d)], "w_up": [z(32, d)], "w_down": [z(d, 32)]}


# strips: one, two, three and four a workgroup of the LM head, the last workgroup with fewer; a tile with one weight more outside the table than a
# copy holds; several slots: 16, 24 and 40 rows through rings of LDS stages; the most k-tiles that either form takes, and one more
@pytest.mark.parametrize("d,V,slots,most,read", [(2048, 2000, 1, 128, True), (2048, 6416, 1, 128, True), (2048, 10000, 1, 128, True), (2048, 15984, 1, 128, True),
                                                 (2048, 2000, 1, 129, False), (4096, 4112, 2, 128, True), (2080, 8208, 3, 128, True), (4096, 12016, 5, 128, True),
                                                 (4096, 4112, 2, 129, False), (16384, 1040, 1, 128, True), (16416, 1040, 1, 128, False), (8192, 2064, 2, 128, True),
                                                 (8224, 2064, 2, 128, False)])
def test_what_is_read_back(d, V, slots, most, read):
    """Rows that are one-hot make a logit a weight of the LM head times the row's norm, which one weight of 2^-5 gives: all 32 columns of tiles with
    1, 2, 3, 60 and `most` weights outside the table, and columns of others."""
    from paper_2311_13581_amd import binding
    k, rng = 7, np.random.default_rng(V)
    head = rng.standard_normal((V, d)).astype(np.float32) * np.float32(0.02)
    ahead = np.array([31, 32, 777, 64, 1024, 1025, d - 1])  # columns of the look-ahead rows
    cols = np.concatenate([np.arange(992, 1024), [0, 1, 63, d - 33, d - 32, d - 2]])  # of the prompts' tokens
    special = np.array([0.0, -0.0, 2.0 ** -126, -2.0 ** -130, 1e30, -3e-20, 5.0, 2.0 ** -133], np.float32)
    strips = V // 16
    for strip, n in ((1, 1), (2, 2), (3, 3), (4, 60), (5, most), (strips - 2, 2), (strips - 1, 4)):
        tile = head[16 * strip:16 * strip + 16, 992:1024]
        tile[(np.abs(tile) < 1e-5) | (np.abs(tile) > 0.12)] = 0.01  # (what the normal distribution has outside)
        at = rng.permutation(512)[:n]
        tile[at // 32, at % 32] = special[rng.integers(0, 8, n)]
    for r in rng.integers(96, V - 32, 60):  # two or so in other tiles
        c = np.append(ahead, cols[32:])
        head[r, c[rng.integers(0, len(c))]] = special[rng.integers(0, 8)]
    head[0, :] = 2.0 ** -5
    tok, la = np.zeros((V, d), np.float32), np.zeros((k, d), np.float32)
    tok[np.arange(len(cols)), cols], la[np.arange(k), ahead] = 1, 1
    g = binding.Pass(binding.make_config(synth.ModelShape(1, d, 1, 128, 32, V, dtype=synth.BF16), k, slots, 64, 64), {"tune.coded": 2})
    g.load_weights(head_only(d, V, head, k, tok, la))
    assert g.coded_use(0, 8 * slots) == read
    stored = rounded(head)
    for first in range(0, len(cols), slots):
        tokens = [min(first + s, len(cols) - 1) for s in range(slots)]
        for s in range(slots):
            g.prefill(s, np.array([tokens[s]], np.int32))
        g.draft(list(range(slots)), 0.0, 1)
        for s in range(slots):
            got, want = g.get_logits(s, 0), stored[:, np.append(cols[tokens[s]], ahead)].T
            assert np.array_equal(got, want * (got[:, :1] * 32)), (first, s)
    g.close()


def test_infinities_and_nan_are_read_back():
    """They stand outside every table: the logits of their rows are not numbers, all others the same bits."""
    from paper_2311_13581_amd import binding
    d, V = 2048, 2000
    head = np.random.default_rng(5).standard_normal((V, d)).astype(np.float32) * np.float32(0.02)
    head[70, 5], head[90, 1000], head[1999, 2047], head[1999, 3] = np.inf, np.nan, -np.inf, np.inf
    tok = np.random.default_rng(6).standard_normal((V, d)).astype(np.float32)
    g = binding.Pass(binding.make_config(synth.ModelShape(1, d, 1, 128, 32, V, dtype=synth.BF16), 1, 1, 64, 64))
    g.load_weights(head_only(d, V, head, 1, tok))
    assert g.coded_use(0, 2)
    g.prefill(0, np.array([3], np.int32))
    g.draft([0], 0.0, 1)
    got = g.get_logits(0, 0)[0]
    g.close()
    want = rounded(tok)[3].astype(np.float64) @ rounded(np.where(np.isfinite(head), head, 0)).T.astype(np.float64)
    want /= np.sqrt((rounded(tok)[3].astype(np.float64) ** 2).mean() + 1e-5)
    bad = np.zeros(V, bool)
    bad[[70, 90, 1999]] = True
    assert not np.isfinite(got[bad]).any() and np.linalg.norm(got[~bad] - want[~bad]) <= 1e-4 * np.linalg.norm(want[~bad])


# blocks a workgroup of QKV (d 2048: 10 and 16 heads, 3072, 5120), of gate/up (F 3200, 5504, 9600, 14400), Wo and down whole on up to 256
# strips, on more (5120), down in slices of K of the plain matrix (d 2048, F 9600)
@pytest.mark.parametrize("d,heads,F,V,k,spread", [(2048, 10, 3200, 1008, 0, 0.002), (2048, 16, 5504, 4800, 4, 0.0), (3072, 24, 9600, 1008, 7, 0.002),
                                                  (5120, 40, 14400, 1008, 4, 0.002), (2048, 16, 9600, 1008, 3, 0.004)])
def test_coded_and_plain_products_agree(d, heads, F, V, k, spread):
    """Both calls' logits on the copies and on the plain matrices.  The weights are the same, so only sums in another order and the
    K/V rows that round the other way for it differ: 1e-4 of the logits, a fifth of what one weight in 2048 gone wrong would make."""
    from paper_2311_13581_amd import binding
    shape = synth.ModelShape(1, d, heads, 128, F, V, dtype=synth.BF16)
    g = binding.Pass(binding.make_config(shape, k, 1, 128, 64), {"graph": 1})
    g.load_weights(random_weights(shape, k, d + F, spread))
    prompt = np.random.default_rng(1).integers(0, V, 40).astype(np.int32)
    out = []
    for coded in (0, 2, 2):
        g.set_option("tune.coded", coded)
        for matrix in range(5):
            assert g.coded_use(matrix, 1 + k) == (coded and (matrix != 2 or heads >= 16))  # (K 1280: no copy of Wo)
        g.prefill(0, prompt)
        g.draft([0], 0.0, 1)
        d0 = g.get_logits(0, 0).copy()
        g.verify([0], 0.0, 1)
        out.append((d0, g.get_logits(0, 1).copy()))
    g.close()
    for a, b, c in zip(*out):
        assert np.linalg.norm(a - b) <= 1e-4 * np.linalg.norm(a)
        assert np.array_equal(b, c)


# 16, 24, 40 and 48 rows: two to eight strips a workgroup, whole and in slices of K, and (d 5120, 32 rows and more) gate/up on the plain matrix
@pytest.mark.parametrize("d,heads,F,V", [(4096, 32, 11008, 8000), (5120, 40, 13760, 4160), (4096, 32, 9632, 33008)])
def test_coded_and_plain_products_agree_in_batches(d, heads, F, V):
    from paper_2311_13581_amd import binding
    shape, slots = synth.ModelShape(1, d, heads, 128, F, V, dtype=synth.BF16), list(range(8))
    g = binding.Pass(binding.make_config(shape, 5, 8, 128, 64))
    g.load_weights(random_weights(shape, 5, d + F, 0.002))
    for rows in (1, 2, 4, 5):
        g.set_option("lookahead_rows", rows)
        out = []
        for coded in (0, 2):
            g.set_option("tune.coded", coded)
            assert rows > 1 or [g.coded_use(matrix, 16) for matrix in range(5)] == 5 * [bool(coded)]
            for s in slots:
                g.prefill(s, np.arange(20 + s, dtype=np.int32))
            g.draft(slots, 0.0, 1)
            out.append(np.stack([g.get_logits(s, 0)[:1 + rows] for s in slots]))
            g.verify(slots, 0.0, 1)  # (the number of rows changes between iterations only)
        assert np.linalg.norm(out[0] - out[1]) <= 1e-4 * np.linalg.norm(out[0]), rows
    g.close()


# calls of 1 to 8 rows, whose activation tiles have room for just those: both register forms, and slices of K through rings of LDS stages
@pytest.mark.parametrize("coded,slices", [(1, 0), (0, 0), (1, 3), (0, 2)])
@pytest.mark.parametrize("d,heads,F", [(2048, 16, 3200), (5120, 40, 8224)])
def test_few_rows_agree_with_a_batch(d, heads, F, coded, slices):
    """A slot's logits in a call of its own and in one of eight slots, of 8 to 64 rows: only sums in another order differ.  1e-4 as above,
    which holds for one layer: a K/V element rounds the other way with the chance of the sums' difference over its last place, 3e-7 / 4e-3, and
    is 4e-3 off then, 3e-5 of the row; in a second layer, whose input differs by that much, ten times as much."""
    from paper_2311_13581_amd import binding
    shape, slots = synth.ModelShape(1, d, heads, 128, F, 1008, dtype=synth.BF16), list(range(8))
    g = binding.Pass(binding.make_config(shape, 7, 8, 128, 64))
    g.load_weights(random_weights(shape, 7, d + F, 0.002))
    g.set_option("tune.coded", 2 * coded)
    g.set_option("tune.gemm_cfg", 2000000 + slices)
    assert g.coded_use(3, 5) == coded
    for ahead in range(8):
        g.set_option("lookahead_rows", ahead)
        out = []
        for of in (slots, [ahead]):
            for s in of:
                g.prefill(s, np.arange(1, 3 + s, dtype=np.int32), seq_id=s)  # (prompts of 1 to 8 rows)
            g.draft(of, 0.0, 1)
            a = g.get_logits(ahead, 0)[:1 + ahead].copy()
            g.verify(of, 0.0, 1)
            out.append((a, g.get_logits(ahead, 1)[:1 + ahead].copy()))
        for a, b in zip(*out):
            assert np.linalg.norm(a - b) <= 1e-4 * np.linalg.norm(a), ahead
    g.close()


@pytest.mark.parametrize("d,heads,F", [(3072, 24, 8192), (4096, 32, 14336)])
def test_down_on_the_copy_stays_whole(d, heads, F):
    """On coded weights the kernel that adds the sums of slices takes longer than slices save here: the same bits as K whole by request."""
    from paper_2311_13581_amd import binding
    shape = synth.ModelShape(1, d, heads, 128, F, 1008, dtype=synth.BF16)
    g = binding.Pass(binding.make_config(shape, 4, 1, 128, 64))
    g.load_weights(random_weights(shape, 4, F))
    assert g.coded_use(4, 5)
    out = []
    for _ in range(2):
        g.prefill(0, np.arange(9, dtype=np.int32))
        g.draft([0], 0.0, 1)
        out.append(g.get_logits(0, 0).copy())
        g.set_option("tune.gemm_cfg", 2000001)
    g.close()
    assert np.array_equal(*out)


@pytest.mark.parametrize("d,reads", [(2048, {16: 1, 32: 1, 40: 1, 48: 0}), (4096, {16: 1, 32: 1, 40: 0, 48: 0}), (5120, {16: 1, 32: 0, 40: 0, 48: 0})])
def test_large_heads_read_the_faster_form(d, reads):
    """An LM head of 32000: from some width on the plain matrix, eight strips a workgroup, is faster than coded strips in two rounds."""
    from paper_2311_13581_amd import binding
    head = np.tile(np.random.default_rng(0).standard_normal((1000, d), dtype=np.float32), (32, 1))
    g = binding.Pass(binding.make_config(synth.ModelShape(1, d, 1, 128, 32, 32000, dtype=synth.BF16), 1, 8, 64, 64))
    g.load_weights(head_only(d, 32000, head))
    assert {rows: g.coded_use(0, rows) for rows in reads} == reads
    g.close()


# one slot: four rows through the register form, its gate/up product keeping the pre-activations; eight: 32 rows and coded transposes
@pytest.mark.parametrize("d,heads,F,slots", [(2048, 16, 5504, 1), (4096, 32, 4416, 8)])
def test_training_on_coded_matrices(d, heads, F, slots):
    """The gradient of a step on the copies and on the plain matrices."""
    from paper_2311_13581_amd import binding
    shape, k = synth.ModelShape(1, d, heads, 128, F, 4096, dtype=synth.BF16), 3
    W = random_weights(shape, k, 5, 0.002)
    target = np.arange(3 * slots, dtype=np.int32).reshape(slots, 3)
    g = binding.Pass(binding.make_config(shape, k, slots, 128, 64))
    g.load_weights(W)
    out = []
    for coded in (0, 2):
        g.set_option("tune.coded", coded)
        g.train_begin(-1)
        for matrix in (0, 1, 3, 4):  # forward, and the transposes of 2^24 weights or more
            assert g.coded_use(matrix, 4 * slots) == bool(coded)
            assert g.coded_use(5 + matrix, 4 * slots) == bool(coded and (d == 4096 or matrix == 3))
        for s in range(slots):
            g.prefill(s, np.arange(30 + s, dtype=np.int32))
        loss = g.train_step(list(range(slots)), target, 0.01)
        out.append((loss, g.train_read(1)))
        g.load_weights(W)
    assert g.train_ws.numel() > g.lib.pass_train_bytes(g.h) + g.lib.pass_coded_bytes(g.h)
    g.close()
    (l0, g0), (l1, g1) = out
    assert abs(l0 - l1) <= 1e-5 * abs(l0) and np.linalg.norm(g0 - g1) <= 2e-4 * np.linalg.norm(g0)


# weights outside the table (2^-24 of the others), and whether calls of 5 and of 16 rows read the copy: none but those of a normal distribution; a tile
# with 12; with 40; a row of one strip; 0.2 and 1 of a tile all over
@pytest.mark.parametrize("where,few,ring", [("none", True, True), ("tile 12", True, True), ("tile 40", False, False), ("row", False, False),
                                            ("all 0.2", True, False), ("all 1", False, False)])
def test_copies_that_would_cost_time_are_not_read(where, few, ring):
    """A copy is read where it saves time: what lies outside its table is put in by one wavefront while the others wait."""
    from paper_2311_13581_amd import binding
    d, V, rng = 2048, 8208, np.random.default_rng(3)
    head = rng.standard_normal((V, d), dtype=np.float32) * np.float32(0.02)
    low = np.zeros((V, d), bool)
    if where.startswith("tile"):
        at = rng.permutation(512)[:int(where[5:])]
        low[160 + at // 32, 992 + at % 32] = True
    elif where == "row":
        low[163] = True
    elif where.startswith("all"):
        low = rng.random((V, d), dtype=np.float32) < float(where[4:]) / 512
    g = binding.Pass(binding.make_config(synth.ModelShape(1, d, 1, 128, 32, V, dtype=synth.BF16), 1, 8, 64, 64))
    with pytest.raises(binding.PassError):
        g.coded_use(0, 5)  # no weights yet
    g.load_weights(head_only(d, V, np.where(low, head * np.float32(2.0 ** -24), head)))
    assert (g.coded_use(0, 5), g.coded_use(0, 16)) == (few, ring)
    g.set_option("tune.coded", 2)  # every copy that holds its matrix
    assert g.coded_use(0, 5) and g.coded_use(0, 16)
    g.set_option("tune.coded", 0)
    assert not g.coded_use(0, 5) and not g.coded_use(0, 16)
    for matrix, rows in ((-1, 5), (10, 5), (0, 0), (0, 65)):  # five matrices, and as many transposes
        assert g.lib.pass_coded_use(g.h, matrix, rows) == -1
    assert g.lib.pass_coded_use(g.h, 9, 5) == 0  # no training
    g.close()


# small products are not coded: of QKV, Wo, gate/up and down those of up to 3 * 2^20 weights (K from 2048) or 11 * 2^20 (shorter K), but narrow ones
# of a long K are; LM heads of a short K from 9000 * 1024 on
@pytest.mark.parametrize("d,heads,F,V,reads", [(1024, 16, 2560, 8016, [0, 0, 0, 0, 0]), (1024, 8, 3072, 9008, [1, 0, 0, 0, 1]), (1536, 16, 4096, 1008, [0, 0, 0, 1, 1]),
                                               (1792, 14, 2048, 1008, [0, 0, 0, 0, 1]), (2048, 4, 2048, 1008, [1, 0, 0, 1, 1])])
def test_small_products_read_the_plain_matrix(d, heads, F, V, reads):
    from paper_2311_13581_amd import binding
    shape = synth.ModelShape(1, d, heads, 128, F, V, dtype=synth.BF16)
    g = binding.Pass(binding.make_config(shape, 1, 1, 64, 64))
    g.load_weights(random_weights(shape, 1, F))
    for rows in (1, 8):
        assert [g.coded_use(matrix, rows) for matrix in range(5)] == reads
    assert (g.lib.pass_coded_bytes(g.h) > 0) == (g.coded is not None) == any(reads)
    g.close()


def test_workspace_of_the_copies():
    """What pass_coded_begin refuses, and that loading weights again ends the use of the old copies (captured graphs too)."""
    import torch
    from paper_2311_13581_amd import binding
    shape, k = synth.ModelShape(1, 2048, 2, 128, 2048, 1008, dtype=synth.BF16), 2
    g = binding.Pass(binding.make_config(shape, k, 1, 128, 64), {"graph": 1})
    assert g.lib.pass_coded_bytes(g.h) == 0 and g.lib.pass_coded_begin(g.h, None, 0) == -2  # no weights yet
    prompt = np.arange(20, dtype=np.int32)

    def logits():
        g.prefill(0, prompt)
        res = []
        for _ in range(3):
            g.draft([0], 0.0, 1)
            g.verify([0], 0.0, 1)
            res.append(g.get_logits(0, 1).copy())
        return res

    g.load_weights(random_weights(shape, k, 1))
    n = g.lib.pass_coded_bytes(g.h)
    ws = torch.empty(n + 512, dtype=torch.uint8, device="cuda")
    base = (ws.data_ptr() + 255) & ~255
    for p, b in ((0, n), (base + 64, n), (base, n - 1)):
        assert g.lib.pass_coded_begin(g.h, C.c_void_p(p), b) == -1
    first = logits()
    g.load_weights(random_weights(shape, k, 2))
    second = logits()
    g.set_option("tune.coded", 0)
    plain = logits()
    g.close()
    assert all(np.linalg.norm(a - b) <= 1e-4 * np.linalg.norm(b) for a, b in zip(second, plain))
    assert not np.allclose(first[0], second[0])
    small = binding.Pass(binding.make_config(synth.ModelShape(1, 512, 4, 128, 1184, 1008, dtype=synth.BF16), k, 1, 128, 64))
    small.load_weights(random_weights(synth.ModelShape(1, 512, 4, 128, 1184, 1008, dtype=synth.BF16), k, 3))
    assert small.coded is None and small.lib.pass_coded_bytes(small.h) == 0
    assert small.lib.pass_coded_begin(small.h, C.c_void_p(base), n) == -2
    small.close()
