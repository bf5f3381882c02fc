"""GPU parity of the row kernels (embedding + first norm, RMSNorm, rotary embedding + KV write) where their own shape
rules change: the bits of the rotation, rows that take three and four rounds of a workgroup, more rotary items than a
workgroup has threads, and tables at addresses that only allow narrow loads."""
import numpy as np
import pytest
import torch

import oracle
from hs_inputs import ModelShape, make_weights, rope_table, make_prompts
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
