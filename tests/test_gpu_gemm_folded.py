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
