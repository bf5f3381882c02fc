"""The attention's bits, verify and prefill: a change of its layout or schedule leaves every sum in its order (the order of a row's keys
within a page, of its probabilities' sum, of the partitions), so that outputs stay what they were from build to build."""
import hashlib

import numpy as np
import pytest
import torch

from hs_inputs import ModelShape, make_weights, rope_table
from gpu_common import np_of

pytestmark = pytest.mark.gpu

# SHA-256 of the attention output (bf16) of all rows, recorded with 128-key tiles staged through registers (per head size)
BITS = {64: "3bbe7c874c9f1280093ce37281b2961475788b1f951bc4032e2f64d0a1edf1e2",
        128: "2eba43094cc34887f561fc611e17ce99047bf51e1efc514fd8cac3fbc5f25aaf"}

# the same of the prefill's attention (five sequences in two calls, the first layer's output of the last call) and of the K and V
# caches, whose second layer has seen it; recorded with the values in rows of 40 bytes, read in two pieces of 8
PREFILL_BITS = {64: ("d225aeb65f0cf0507590c093de53f6d9152c919436668abb99918e4393bc04e7",
                     "48b60eabd39f9f4255ad909af60353032dfdb4c05ba10d7ae021521340add557",
                     "f2a3ef99cf8b924404c9c2d15d5d5a3b8722b44709bef9f7624d7bc4c5546e6a"),
                128: ("568a54a5b088193367c75c26430764060bab9603e932d4ade14529010ea74f25",
                      "916eade68575597b1d75796d3cfec5353bea2e96dfb7995eed1cced108357037",
                      "c36581751b37330d65960d04dec0dbe95761020f653cc8b1ac612a428536c388")}


def attention_bits(head_dim):
    """One layer, wavefront units (1 and 5 rows of 4 heads) and workgroup units (13 and 23), some past several partitions."""
    from paper_2508_18588_amd.runtime import Engine, Policy
    shape = ModelShape(n_layers=1, d_model=256, n_q_heads=8, n_kv_heads=2, head_dim=head_dim, d_ffn=384, vocab=512)
    rng = np.random.default_rng(31)
    lens, draft_lens = [40, 300, 700, 1100, 1101, 260, 31, 129], [0, 4, 12, 22, 4, 22, 12, 0]
    toks = [rng.integers(0, shape.vocab, n).astype(np.int32) for n in lens]
    none = np.zeros(0, np.int32)
    cands = [[np.concatenate([t[-6:], rng.integers(0, shape.vocab, k)]).astype(np.int32) if k else none] for t, k in zip(toks, draft_lens)]
    eng = Engine(shape, make_weights(shape, 32, norm_jitter=0.1), rope_table(1300, head_dim), max_batch=8, k_max=22, c_max=1, max_len=1200,
                 shuffle_pages_seed=33)
    eng.load_sequences(toks, budgets=[40] * 8)
    eng.set_history(cands)
    eng.prefill_chunked(512)
    eng.draft(Policy(window=6, m_min=3, k_fixed=22, k_max=22))
    eng.verify()
    torch.cuda.synchronize()
    m = int(eng.st["row_off"][8])
    assert m == 8 + sum(draft_lens)
    out = np_of(eng.debug_tensor(2))[:m * 8 * head_dim * 2]
    eng.close()
    return hashlib.sha256(out.tobytes()).hexdigest()


@pytest.mark.parametrize("head_dim", [64, 128])
def test_attention_output_keeps_its_bits(head_dim):
    assert attention_bits(head_dim) == BITS[head_dim]


def prefill_bits(head_dim):
    """Two layers; sequences of 16 to 1136 cached tokens, one cut by the chunk, one by the row limit."""
    from paper_2508_18588_amd.runtime import Engine
    shape = ModelShape(n_layers=2, d_model=256, n_q_heads=8, n_kv_heads=2, head_dim=head_dim, d_ffn=384, vocab=512)
    rng = np.random.default_rng(41)
    toks = [rng.integers(0, shape.vocab, n).astype(np.int32) for n in (34, 300, 1137, 17, 66)]
    eng = Engine(shape, make_weights(shape, 42, norm_jitter=0.1), rope_table(1300, head_dim), max_batch=5, k_max=0, c_max=1, max_len=1200,
                 max_rows=1400, keep_logits=False, shuffle_pages_seed=43)
    eng.load_sequences(toks, budgets=[1] * 5)
    assert eng.prefill_chunked(1024) == 2
    torch.cuda.synchronize()
    m = int(eng.st["row_off"][5])
    out = np_of(eng.debug_tensor(2))[:m * 8 * head_dim * 2], np_of(eng.kc), np_of(eng.vc)
    eng.close()
    return tuple(hashlib.sha256(t.tobytes()).hexdigest() for t in out)


@pytest.mark.parametrize("head_dim", [64, 128])
def test_prefill_attention_keeps_its_bits(head_dim):
    assert prefill_bits(head_dim) == PREFILL_BITS[head_dim]
