"""Split-K projections with all K chunks of a tile in one workgroup (many rows): the bits of the split execution and its ordered
reduce, stored and added, against C = A . W^T in fp64 as well.  Widths that end inside a weight unit and inside a group, a last
chunk of one k-tile, and actual row counts from one to more than the launch expects (edges of the 32-row tiles and 256-row
passes).  That nothing of the workspace is written shows that the folded kernel ran."""
import numpy as np
import pytest
import torch

from hs_inputs import ModelShape, make_weights, rope_table
from gpu_common import np_of

pytestmark = pytest.mark.gpu

M_MAX = 4200


@pytest.fixture(scope="module")
def eng():
    from paper_2508_18588_amd.runtime import Engine
    shape = ModelShape(n_layers=1, d_model=1664, n_q_heads=14, n_kv_heads=2, head_dim=128, d_ffn=1664, vocab=4096)
    e = Engine(shape, make_weights(shape, 57), rope_table(64, 128), max_batch=8, k_max=4, c_max=1, max_len=32, max_rows=M_MAX,
               keep_logits=False)
    yield e
    e.close()


# (groups of 2, 2, 3, 4, 3 and 4 units; 26 k-tiles are five chunks of five and one of one, 13 are two of five and one of three)
@pytest.mark.parametrize("n,k,hint", [(2048, 1664, 2000), (1608, 1664, 2000), (1536, 1664, 3000), (1664, 1664, 3000),
                                      (1608, 1664, 4100), (1608, 832, 3000)])
@pytest.mark.parametrize("epi", [0, 1])
def test_folded_chunks_give_the_bits_of_the_split_execution(eng, epi, n, k, hint):
    g = torch.Generator(device="cuda:0").manual_seed(n + k)
    a = torch.randn(M_MAX, k, device="cuda:0", generator=g).to(torch.bfloat16)
    w = (torch.randn(n, k, device="cuda:0", generator=g) * 0.05).to(torch.bfloat16)
    want = a.double() @ w.double().T + (7.0 if epi else 0.0)

    def run(m, rows_hint):
        c = torch.full((M_MAX, n), 7.0, dtype=torch.float32, device="cuda:0")
        m_dev = torch.full((1,), m, dtype=torch.int32, device="cuda:0")
        eng.gemm(epi, a.view(torch.int16), w.view(torch.int16), None, c, m_dev, M_MAX, rows_hint)
        torch.cuda.synchronize()
        return c

    for m in (1, 33, 255, 257, 1000, hint - 1, hint, min(hint + 700, M_MAX)):
        split = run(m, 0)
        eng.workspace.zero_()
        folded = run(m, hint)
        assert not bool(eng.workspace.any()), "the split execution ran"
        assert torch.equal(folded.view(torch.int32), split.view(torch.int32)), (m, hint)
        assert bool((folded[m:] == 7.0).all())
        # fp32 sums over k <= 1664 of products of scale 0.05
        assert float((folded[:m].double() - want[:m]).abs().max()) <= 2e-5 * (float(want.abs().max()) + 1.0)


@pytest.fixture(scope="module")
def wide_eng():
    """QKV of 4608 columns in three chunks, O of 3584 in four, down in two; three and four units to a group."""
    from hs_inputs.device import make_weights_device
    from paper_2508_18588_amd.runtime import Engine
    shape = ModelShape(n_layers=2, d_model=3584, n_q_heads=28, n_kv_heads=4, head_dim=128, d_ffn=512, vocab=512)
    e = Engine(shape, make_weights_device(shape, 58), rope_table(1100, 128), max_batch=80, k_max=16, c_max=1, max_len=1060, seq_caps=[1060] * 2 + [64] * 78)
    yield e
    e.close()


@pytest.mark.parametrize("hint", [1078, 1350])
def test_rows_on_either_side_of_what_is_folded(wide_eng, hint):
    """With fewer rows than expected by a factor the folded launch leaves partial sums after all, one chunk to a workgroup or several
    one after the other: the cache of a prefill call has the bits of a call without an estimate, whatever the row count."""
    from paper_2508_18588_amd import hs_prefill, hs_prefill_args
    eng, rng = wide_eng, np.random.default_rng(hint)
    toks = [rng.integers(0, 512, 1025).astype(np.int32), rng.integers(0, 512, 340).astype(np.int32)]
    for m in (1, 31, 255, 256, 257, 512, 513, 768, 769, 1024, 1025, 1300):
        eng.load_sequences([toks[0][:min(m, 1024) + 1], toks[1][:max(m - 1024, 0) + 1]], [9, 9])
        caches = []
        for h in (0, hint):
            eng.kc.zero_()
            eng.vc.zero_()
            eng.kv_done = torch.zeros(eng.max_batch, dtype=torch.int32, device=eng.dev)
            hs_prefill(eng.ctx, eng.c_cache, eng.c_seq, eng.c_step, hs_prefill_args(1024, h, eng.kv_done.data_ptr()), eng.stream())
            torch.cuda.synchronize()
            assert int(eng.st["row_off"][2]) == m
            caches.append((eng.kc.clone(), eng.vc.clone()))
        assert all(torch.equal(x, y) for x, y in zip(*caches)), m
        assert bool(caches[0][0].any())


def test_a_step_with_fewer_rows_than_expected_costs_little(wide_eng):
    """64 and 192 rows where 1078 are expected: the projections take less than without an estimate, same logits.  (Folded whatever
    the row count, every workgroup of QKV and O along all of K, they took 1.16 to 1.18 times as long; now 0.83 to 0.89.)"""
    eng = wide_eng
    eng.load_sequences([np.arange(20, dtype=np.int32)] * 80, [9] * 80)

    def projections_us(hint):
        eng.c_step.rows_hint = hint
        times = []
        for _ in range(8):
            eng.set_profile(2)
            eng.verify()
            times.append(eng.get_profile()[0][1] * 1e3)
        eng.set_profile(0)
        return sorted(times[2:])[2], eng.logits[:64 * per].clone()

    for per in (1, 3):
        eng.set_rows([dict(tok=[1] * per, parent=np.arange(-1, per - 1), pos=19 + np.arange(per))] * 64 + [None] * 16)
        (none, want), (many, got) = projections_us(0), projections_us(1078)
        print("projections of a pass, us, without an estimate and with one of 1078 rows:", none, many)
        assert torch.equal(want, got)
        assert many <= 1.05 * none, (per, none, many)
