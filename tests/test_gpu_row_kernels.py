"""GPU parity of the row kernels (embedding + first norm, RMSNorm, rotary embedding + KV write) where their own shape
rules change: the bits of the rotation, rows that take three and four rounds of a workgroup, more rotary items than a
workgroup has threads, and tables at addresses that only allow narrow loads."""
import numpy as np
import pytest
import torch

import oracle
from hs_inputs import ModelShape, bf16_bits, make_weights, rope_table, make_prompts
from gpu_common import OracleBatch, check_cache, check_last_layer_projections, derived_logit_tol, np_of

pytestmark = pytest.mark.gpu


def test_rotation_is_one_product_and_one_fused_multiply_add():
    """(x, y) -> (fma(x, c, -(y s)), fma(x, s, y c)), every pair of a head alike, bit for bit.  The fp32-activation mode
    keeps keys as floats: with cos = 1 and sin = 0 the cache holds x and y themselves, with any other table the
    rotation of the same values (first layer: its inputs do not depend on the rotation)."""
    from paper_2508_18588_amd.runtime import Engine
    shape = ModelShape(n_layers=1, d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=64, d_ffn=128, vocab=128)
    w, n, half = make_weights(shape, 5), 48, 32
    prompt = make_prompts(1, n + 1, shape.vocab, 6)[0]
    ident = np.zeros((128, half, 2), np.float32)
    ident[:, :, 0] = 1.0
    keys = []
    for rope in (ident, rope_table(128, shape.head_dim)):
        eng = Engine(shape, w, rope, max_batch=1, k_max=15, c_max=1, max_len=n + 1, precise=True)
        eng.load_sequences([prompt], budgets=[9])
        eng.prefill([prompt])
        torch.cuda.synchronize()
        k = np_of(eng.kc).reshape(eng.n_blocks, shape.n_kv_heads, 16, shape.head_dim)
        pages = np_of(eng.block_table)[0]
        keys.append(np.stack([k[pages[t // 16], :, t % 16] for t in range(n)]))
        eng.close()
    x, y = keys[0][..., :half], keys[0][..., half:]
    c, s = rope_table(128, shape.head_dim)[:n, None, :, 0], rope_table(128, shape.head_dim)[:n, None, :, 1]

    def fma(a, b, addend):   # exact product (48 bits) and a sum in extended precision, rounded once more to 24 bits
        return (a.astype(np.longdouble) * b + addend).astype(np.float32)

    assert (x != 0).mean() > 0.9
    assert (keys[1][..., :half] == fma(x, c, -(y * s))).all()
    assert (keys[1][..., half:] == fma(x, s, y * c)).all()


def final_norm_rows(shape, w, tokens):
    """Residual stream and normed rows (fp32-activation mode) of `tokens` as chains of up to 14 rows at positions 0.."""
    from paper_2508_18588_amd.runtime import Engine
    chains = [np.asarray(tokens[i:i + 14], np.int32) for i in range(0, len(tokens), 14)]
    eng = Engine(shape, w, rope_table(64, 64), max_batch=len(chains), k_max=15, c_max=1, max_len=32, precise=True)
    eng.load_sequences([np.array([0], np.int32)] * len(chains), budgets=[9] * len(chains))
    m = eng.set_rows([dict(tok=c, parent=np.arange(-1, len(c) - 1), pos=np.arange(len(c))) for c in chains])
    eng.verify()
    torch.cuda.synchronize()
    x, xn = (np_of(eng.debug_tensor(i).view(torch.float32))[:m * shape.d_model].reshape(m, -1).copy() for i in (4, 0))
    eng.close()
    return x, xn


@pytest.mark.parametrize("d", [64, 4096, 5120])
def test_sum_of_squares_is_a_chain_of_fused_multiply_adds_in_a_fixed_order(d):
    """The final norm of the fp32-activation mode against its own residual stream, bit for bit: a thread's sum of
    squares starts with fma(x, x, y y) and goes on with one fma per element, lanes are added by a butterfly, wavefronts
    left to right (thread t holds elements 4 t .. 4 t + 3 and the same 4096 further on), and the row is x r g with r = 1 / sqrt(sum / d + eps) as the hardware rounds it.  That r is read off a
    second model whose residual stream is its embedding (O and down projection zero), rows of powers of two that square
    and add up, without any rounding, to the sums of the first.  One and two rounds of elements per thread."""
    shape = ModelShape(n_layers=1, d_model=d, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=96)
    w = make_weights(shape, 8, norm_jitter=0.1)
    x, got = final_norm_rows(shape, w, np.random.default_rng(9).integers(0, shape.vocab, 70))
    m = len(x)

    def fma(a, addend):      # a a + addend, rounded once
        return (a.astype(np.longdouble) * a + addend).astype(np.float32)

    rounds = (d // 4 + 1023) // 1024
    threads = max(256, min(1024, (d // 4 + 63) // 64 * 64))
    v = np.zeros((m, rounds * threads, 4), np.float32)
    v[:, :d // 4] = x.reshape(m, d // 4, 4)
    v = v.reshape(m, rounds, threads, 4)
    ss = fma(v[:, 0, :, 0], v[:, 0, :, 1] * v[:, 0, :, 1])
    for it in range(rounds):
        for e in range(2 if it == 0 else 0, 4):
            ss = fma(v[:, it, :, e], ss)
    lanes = ss.reshape(m, threads // 64, 64)
    for o in (32, 16, 8, 4, 2, 1):
        lanes = lanes + lanes[:, :, np.arange(64) ^ o]
    total = lanes[:, 0, 0]
    for i in range(1, threads // 64):
        total = total + lanes[:, i, 0]

    # bit e of a sum: one element 2^(e/2), or two of 2^((e-1)/2); lowest bit first (half of it may be below the sum's last
    # place: its two elements are the first that a thread adds)
    embed = np.zeros((m, d), np.float32)
    for row, t in enumerate(total):
        mant, ex = int(t.view(np.uint32) & 0x7FFFFF) | 0x800000, int(t.view(np.uint32) >> 23) - 150
        el = [2.0 ** ((b + ex) // 2) for b in range(24) if mant >> b & 1 for _ in range(1 + (b + ex) % 2)]
        embed[row, :len(el)] = el
    assert ((embed.astype(np.float64) ** 2).sum(1) == total.astype(np.float64)).all()
    plain = ModelShape(n_layers=1, d_model=d, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=m)
    w2 = make_weights(plain, 8)
    w2["embed"] = bf16_bits(embed)
    w2["wo"], w2["wdown"] = [np.zeros_like(a) for a in w2["wo"]], [np.zeros_like(a) for a in w2["wdown"]]
    x2, xn2 = final_norm_rows(plain, w2, np.arange(m))
    assert (x2 == embed).all()
    at = (np.arange(m), embed.argmax(1))
    r = xn2[at] / embed[at]                       # (a division by a power of two)
    want = x * r[:, None] * w["norm_f"].astype(np.float32)
    assert (got == want).all(), (d, int((got != want).any(1).sum()), m)


def last_row_logits(eng, prompts, how):
    """Logits of every prompt's last token: the text before it by hs_prefill (how = a chunk length) or through hs_verify."""
    eng.load_sequences(list(prompts), budgets=[9] * len(prompts))
    eng.prefill(list(prompts)) if how == "verify" else eng.prefill_chunked(how)
    eng.set_rows([dict(tok=p[-1:], parent=[-1], pos=[len(p) - 1]) for p in prompts])
    eng.verify()
    torch.cuda.synchronize()
    assert eng.poll_error() == 0
    return np_of(eng.logits)[:len(prompts)].astype(np.float64)


@pytest.mark.parametrize("d,hq,hkv,h", [(8256, 1, 1, 64), (12288, 1, 1, 64), (12352, 1, 1, 64), (16384, 2, 1, 64),
                                        (256, 64, 8, 128), (192, 33, 11, 128)])
def test_wide_rows_and_many_heads_against_the_oracle(d, hq, hkv, h):
    """Rows of three and four rounds of a workgroup (d_model beyond 8192 and 12288; the last round full and ragged), and
    heads with more than 1024 rotary items per row: logits and cache against the oracle, in the default and in the
    fp32-activation mode, the prompt written by hs_prefill and by hs_verify."""
    from paper_2508_18588_amd.runtime import Engine
    shape = ModelShape(n_layers=2, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=h, d_ffn=64, vocab=64)
    w, rope = make_weights(shape, d + hq, norm_jitter=0.1), rope_table(64, h)
    prompts = [p[:n] for p, n in zip(make_prompts(3, 21, shape.vocab, 3), (21, 2, 18))]
    ob = OracleBatch(oracle.Model(shape, w, rope), prompts, [9] * 3, 32)
    want = np.stack([ob.seqs[b].tree_logits(p[-1:], np.array([-1], np.int32))[0] for b, p in enumerate(prompts)])
    scale = np.abs(want).max(1, keepdims=True)
    for precise, how in ((False, 16), (False, "verify"), (True, "verify")):
        eng = Engine(shape, w, rope, max_batch=3, k_max=6, c_max=1, max_len=24, shuffle_pages_seed=2, precise=precise)
        got = last_row_logits(eng, prompts, how)
        if precise:
            assert (np.abs(got - want) <= 1e-4 * scale).all()
        else:
            assert np.abs(got - want).max() <= derived_logit_tol(shape, shape.n_layers)
            check_cache(eng, ob, 0, tol=2.0 ** -7 * 0.02 * np.sqrt(d) * 4)
        eng.close()


@pytest.mark.parametrize("d", [8256, 16384])
def test_wide_rows_with_pending_partial_sums(d):
    """A down projection of 8192 columns leaves two or three partial sums per element to a norm of three and four rounds.
    The residual stream after it against fp64 products of the path's own operands, and the norms on either side of it
    against the definition: one rounding to the 8 significant bits of bf16 (half a place is 2^-8 of a power of two) of a value
    computed with a few fp32 roundings."""
    from hs_inputs.device import make_weights_device
    from paper_2508_18588_amd.runtime import Engine
    shape = ModelShape(n_layers=2, d_model=d, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=8192, vocab=64)
    eng = Engine(shape, make_weights_device(shape, 7), rope_table(64, 64), max_batch=3, k_max=15, c_max=1, max_len=32)
    prompts = make_prompts(3, 14, shape.vocab, 3)
    eng.load_sequences(list(prompts), budgets=[9] * 3)
    eng.seq_len.fill_(1)
    m = eng.set_rows([dict(tok=p, parent=np.arange(-1, len(p) - 1), pos=np.arange(len(p))) for p in prompts])
    cap = eng.capture_last_layer()
    eng.verify()
    torch.cuda.synchronize()
    check_last_layer_projections(eng, cap, m, range(m), np.random.default_rng(1))
    for x, xn in ((cap[3], cap[2]), (eng.debug_tensor(4), eng.debug_tensor(0))):
        x = np_of(x.view(torch.float32)[:m * d]).reshape(m, d).astype(np.float64)
        got = np_of(xn.view(torch.bfloat16)[:m * d].double()).reshape(m, d)
        want = x / np.sqrt((x * x).mean(1, keepdims=True) + shape.rms_eps)
        assert (np.abs(got - want) <= (2.0 ** -8 + 2e-6) * np.abs(want)).all()
    eng.close()


def test_tables_that_only_allow_narrow_loads():
    """The header asks no alignment of the embedding and of the rotary table beyond their elements': both one element off a
    16-byte boundary give the bits of the aligned ones."""
    from paper_2508_18588_amd.runtime import Engine
    shape = ModelShape(n_layers=2, d_model=384, n_q_heads=6, n_kv_heads=2, head_dim=64, d_ffn=128, vocab=300)
    w, rope = make_weights(shape, 3, norm_jitter=0.1), rope_table(64, 64)
    prompts = make_prompts(3, 21, shape.vocab, 3)
    shifted = {}
    for name, a in (("embed", torch.from_numpy(w["embed"].view(np.int16))), ("rope", torch.from_numpy(rope))):
        flat = torch.empty(a.numel() + 1, dtype=a.dtype, device="cuda:0")
        flat[1:] = a.flatten().cuda()
        shifted[name] = flat[1:].view(a.shape)
        assert shifted[name].data_ptr() % 16 == a.element_size()
    for precise in (False, True):
        logits = []
        for table, cs in ((w["embed"], rope), (shifted["embed"], rope), (w["embed"], shifted["rope"])):
            eng = Engine(shape, dict(w, embed=table), cs, max_batch=3, k_max=6, c_max=1, max_len=24, precise=precise)
            assert (eng.w["embed"].data_ptr() % 8 != 0) == (table is shifted["embed"])
            assert (eng.rope.data_ptr() % 16 != 0) == (cs is shifted["rope"])
            logits.append(last_row_logits(eng, list(prompts), "verify"))
            eng.close()
        assert (logits[0] == logits[1]).all() and (logits[0] == logits[2]).all()


@pytest.mark.parametrize("vocab", [64, 4096, 16380, 16384, 16386, 16388, 36868])
def test_argmax_is_the_first_of_the_largest_logits(vocab):
    """The largest logit is there three times; widths below, at and above the four loads of 1024 threads that are on their way
    at once, and one that allows no 16-byte loads; with and without an estimate of the rows."""
    from paper_2508_18588_amd.runtime import Engine
    shape = ModelShape(n_layers=1, d_model=64, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=vocab)
    w = make_weights(shape, vocab)
    third = (vocab + 2) // 3
    w["lm_head"] = np.concatenate([w["lm_head"][:third]] * 3)[:vocab].copy()
    rng = np.random.default_rng(vocab)
    eng = Engine(shape, w, rope_table(64, 64), max_batch=70, k_max=0, c_max=1, max_len=32)
    eng.load_sequences([rng.integers(0, vocab, 20).astype(np.int32) for _ in range(70)], [9] * 70)
    eng.set_rows([dict(tok=rng.integers(0, vocab, 1), parent=[-1], pos=[19]) for _ in range(70)])
    for hint in (0, 3, 64, 70):
        eng.c_step.rows_hint = hint
        eng.st["argmax"].fill_(-1)
        eng.verify()
        torch.cuda.synchronize()
        logits = np_of(eng.logits)[:70]
        assert np_of(eng.st["argmax"]).tolist() == logits.argmax(1).tolist(), hint
        assert (logits.argmax(1) < third).all()
    eng.close()
