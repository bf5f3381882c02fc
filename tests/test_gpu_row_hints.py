"""The row kernels ask for a row's data before the row count has arrived where the host's estimate covers the row: the result
must not depend on the estimate, and rows that do not exist must leave no trace."""
import numpy as np
import pytest
import torch

from hs_inputs import ModelShape, make_weights, rope_table
from gpu_common import np_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hq,hkv,h,f", [(256, 4, 4, 64, 1024), (1536, 12, 2, 128, 1024), (5120, 8, 8, 128, 8192),
                                          (1024, 4, 2, 128, 4096), (2048, 8, 4, 128, 1024)])
def test_a_step_does_not_depend_on_the_expected_rows(d, hq, hkv, h, f):
    """One and two rounds per row of the norm, with and without pending partial sums (two rounds with six chunks, three of them in
    flight at once; one with sixteen, ten in flight; the rotary kernel with eight, six in flight), heads of 64 and 128; estimates
    of no row, some, exactly all, more (and more than the merge and the other kernels ask ahead for).  A sequence whose page is
    missing writes no K/V, whatever the estimate."""
    from paper_2508_18588_amd.runtime import Engine
    shape = ModelShape(n_layers=2, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=h, d_ffn=f, vocab=512)
    rng, B = np.random.default_rng(d), 5
    toks = [rng.integers(0, 512, n).astype(np.int32) for n in (40, 300, 17, 16, 700)]
    w = make_weights(shape, 3)
    eng = Engine(shape, w, rope_table(1024, h), max_batch=8, k_max=9, c_max=1, max_len=710)
    eng.load_sequences(toks, [9] * B)
    eng.prefill_chunked(256)
    rows = []
    for b, n in enumerate((1, 10, 3, 0, 5)):
        t = np.concatenate([toks[b][-1:], rng.integers(0, 512, max(0, n - 1))]).astype(np.int32)
        rows.append(dict(tok=t, parent=np.arange(-1, n - 1), pos=len(toks[b]) - 1 + np.arange(n)) if n else None)
    m = eng.set_rows(rows)
    assert m == 19
    table = eng.block_table.clone()
    eng.block_table[2, (len(toks[2]) - 1 + 2) // 16] = eng.n_blocks     # (beyond the cache: sequence 2's rows 0.. lie on that page)
    kc, vc = eng.kc.clone(), eng.vc.clone()
    outs = []
    for hint in (0, 1, 7, m, 33, eng.max_rows):
        eng.kc.copy_(kc)
        eng.vc.copy_(vc)
        eng.logits.zero_()
        eng.c_step.rows_hint = hint
        eng.verify()
        torch.cuda.synchronize()
        live = torch.cat([eng.logits[:11], eng.logits[14:m]])           # (the rows whose keys are all there)
        outs.append((live.clone(), eng.kc.clone(), eng.vc.clone(), np_of(eng.st["argmax"])[:11].tolist()))
        assert not eng.logits[m:].any()
    for hint, o in zip((1, 7, m, 33, eng.max_rows), outs[1:]):
        assert torch.equal(o[0], outs[0][0]) and o[3] == outs[0][3], hint
        assert torch.equal(o[1], outs[0][1]) and torch.equal(o[2], outs[0][2]), hint
    # exactly the live rows' slots changed: 16 rows of four sequences, in both layers
    k2 = outs[0][1].view(2, eng.n_blocks, hkv, 16, h) != kc.view(2, eng.n_blocks, hkv, 16, h)
    changed = k2.any(-1).any(2)
    want = torch.zeros_like(changed)
    for b, r in enumerate(rows):
        for i in range(0 if r is None or b == 2 else len(r["tok"])):
            slot = len(toks[b]) - 1 + i
            want[:, int(table[b, slot // 16]), slot % 16] = True
    assert torch.equal(changed, want)
    eng.close()


@pytest.mark.parametrize("shape", [(1536, 12, 2, 128, 8960, 16448), (1024, 8, 2, 128, 1024, 65536)])
def test_more_rows_expected_than_there_are_cost_the_row_kernels_little(shape):
    """64 rows where 1078 are expected: the row kernels take what they take without an estimate.  (Reading a row's data before the
    count for every row expected, they took 1.5 times as long: partial sums, and logits of a wide vocabulary, of a
    thousand rows that do not exist.)"""
    from hs_inputs.device import make_weights_device
    from paper_2508_18588_amd.runtime import Engine
    d, hq, hkv, h, f, v = shape
    sh = ModelShape(n_layers=2, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=h, d_ffn=f, vocab=v)
    eng = Engine(sh, make_weights_device(sh, 1), rope_table(128, h), max_batch=64, k_max=16, c_max=1, max_len=64)
    eng.load_sequences([np.arange(40 + b % 3, dtype=np.int32) for b in range(64)], [9] * 64)
    eng.set_rows([dict(tok=[1], parent=[-1], pos=[39 + b % 3]) for b in range(64)])

    def row_kernels_us(hint):
        eng.c_step.rows_hint = hint
        times = []
        for _ in range(8):
            eng.set_profile(2)
            eng.verify()
            ms, n = eng.get_profile()
            times.append(ms[3] * 1e3)
        eng.set_profile(0)
        return sorted(times[2:])[2]

    none, many = row_kernels_us(0), row_kernels_us(1078)
    eng.close()
    print("row kernels of a pass, us, without an estimate and with one of 1078 rows:", none, many)
    assert many <= 1.2 * none, (none, many)


@pytest.mark.parametrize("hint", [0, 7, 40])
def test_a_sequence_without_tokens_leaves_the_others_alone(hint):
    """It has no partition of keys: the merge reads none of its partial results (with few rows expected and more, counted first)."""
    from paper_2508_18588_amd.runtime import Engine
    shape = ModelShape(n_layers=2, d_model=256, n_q_heads=4, n_kv_heads=4, head_dim=64, d_ffn=512, vocab=512)
    rng = np.random.default_rng(3)
    toks = [rng.integers(0, 512, n).astype(np.int32) for n in (9, 40, 300)]
    eng = Engine(shape, make_weights(shape, 4), rope_table(400, 64), max_batch=3, k_max=4, c_max=1, max_len=310)
    eng.load_sequences(toks, [9] * 3)
    eng.prefill_chunked(512)
    rows = [dict(tok=t[-1:], parent=[-1], pos=[len(t) - 1]) for t in toks]
    outs = []
    for empty in (False, True):
        eng.set_rows(rows)
        if empty:
            eng.seq_len[0] = 0
            eng.st["pos"][0] = -1
        eng.c_step.rows_hint = hint
        eng.verify()
        torch.cuda.synchronize()
        outs.append(eng.logits[1:3].clone())
    eng.close()
    assert torch.equal(*outs) and bool(torch.isfinite(outs[0]).all())
