"""GPU parity of the row kernels (embedding + first norm, RMSNorm, rotary embedding + KV write) where their own shape
rules change: the bits of the rotation, rows that take three and four rounds of a workgroup, more rotary items than a
workgroup has threads, and tables at addresses that only allow narrow loads."""
import numpy as np
import pytest
import torch

import oracle
from hs_inputs import ModelShape, bf16_bits, make_weights, rope_table, make_prompts
from gpu_common import derived_logit_tol, np_of

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
    left to right, and the row is x r g with r = 1 / sqrt(sum / d + eps) as the hardware rounds it.  That r is read off a
    second model whose residual stream is its embedding (O and down projection zero), rows of powers of two that square
    and add up, without any rounding, to the sums of the first.  One and two rounds of elements per thread."""
    shape = ModelShape(n_layers=1, d_model=d, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=96)
    w = make_weights(shape, 8, norm_jitter=0.1)
    x, got = final_norm_rows(shape, w, np.random.default_rng(9).integers(0, shape.vocab, 70))
    m = len(x)

    def fma(a, addend):      # a a + addend, rounded once
        return (a.astype(np.longdouble) * a + addend).astype(np.float32)

    rounds = (d // 4 + 1023) // 1024
    threads = max(256, ((d // 4 + rounds - 1) // rounds + 63) // 64 * 64)
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
