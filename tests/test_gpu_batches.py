"""Batches larger than one workgroup of the kernels that lay a step out (draft rows, prefill rows, attention unit lists:
1024 threads, a sequence each): 1100 sequences of mixed lengths and draft lengths, against the plain kernels on the same
cache and the rows that the inputs imply."""
import numpy as np
import pytest
import torch

from hs_inputs import ModelShape, make_weights, rope_table
from gpu_common import np_of

pytestmark = pytest.mark.gpu


def test_eleven_hundred_sequences():
    from paper_2508_18588_amd import HS_FLAG_REFERENCE_KERNELS, HS_K_MATCHLEN
    from paper_2508_18588_amd.runtime import Engine, Policy
    shape = ModelShape(n_layers=2, d_model=256, n_q_heads=8, n_kv_heads=1, head_dim=64, d_ffn=256, vocab=4096)
    B, rng = 1100, np.random.default_rng(4)
    toks = [rng.integers(0, shape.vocab, int(n)).astype(np.int32) for n in rng.integers(2, 60, B)]
    hists, want = [], []
    for b, t in enumerate(toks):
        m = int(rng.integers(0, 9))
        m = 0 if m < 3 or m >= len(t) else m
        text = rng.integers(0, shape.vocab, 40).astype(np.int32)
        if m:
            text[5] = (t[-m - 1] + 1) % shape.vocab
            text[6:6 + m] = t[-m:]
        hists.append([text])
        want.append([int(t[-1])] + text[6 + m:6 + 2 * m].tolist())
    eng = Engine(shape, make_weights(shape, 7), rope_table(128, 64), max_batch=B, k_max=8, c_max=1, max_len=72,
                 shuffle_pages_seed=3)
    eng.load_sequences(toks, [50] * B)
    eng.set_history(hists)
    eng.prefill_chunked(64)                              # more sequences than one workgroup has threads, in several calls
    pol = Policy(window=8, m_min=3, k_mode=HS_K_MATCHLEN, k_max=8)
    eng.draft(pol)
    eng.verify()
    torch.cuda.synchronize()
    assert eng.poll_error() == 0
    ro, tok, r2s, pos = (np_of(eng.st[n]) for n in ("row_off", "tok", "row2seq", "pos"))
    assert np.diff(ro).tolist() == [len(w) for w in want]
    m = int(ro[B])
    assert tok[:m].tolist() == [x for w in want for x in w]
    assert r2s[:m].tolist() == [b for b, w in enumerate(want) for _ in w]
    assert pos[:m].tolist() == [len(toks[b]) - 1 + i for b, w in enumerate(want) for i in range(len(w))]
    assert len({len(w) for w in want}) > 4 and 8 * max(len(w) for w in want) > 32   # both unit lists are in use
    got = eng.logits[:m].clone()
    eng.set_flags(HS_FLAG_REFERENCE_KERNELS)             # rewrites the same cache rows, rounds in other places
    eng.verify()
    torch.cuda.synchronize()
    ref = eng.logits[:m]
    # two bf16 paths through two layers differ by sqrt(2) x their error, 4.5 sqrt(2) + 1 roundings of 2^-9/sqrt(3) rms each
    rel = float((got - ref).double().norm() / ref.double().norm())
    assert rel < 1.5 * 2 ** 0.5 * (4.5 * 2 ** 0.5 + 1) * 2.0 ** -9 / 3 ** 0.5, rel
    worst = (got - ref).double().norm(dim=1) / ref.double().norm(dim=1)
    assert float(worst.max()) < 0.08, float(worst.max())  # a row that saw wrong keys is off by its own size
    eng.close()
