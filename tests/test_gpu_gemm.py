"""GPU parity of the projection GEMM on its own (hs_debug_gemm) against its plain definition, C = A . W^T in fp64 on
the same bf16 operands: every epilogue (store, add to the residual, SwiGLU -> bf16, split-K partial sums + ordered
reduce), row counts that end inside a 32-row tile, on a tile edge and beyond one row pass, a SwiGLU width whose last
weight group is ragged; rows beyond the live count stay untouched, and the row hint -- which selects launch shapes
and row passes -- never changes a bit of the result."""
import numpy as np
import pytest
import torch

from hs_inputs import ModelShape, make_weights, rope_table
from gpu_common import np_of

pytestmark = pytest.mark.gpu

M_MAX = 1100
ROWS = [1, 31, 32, 33, 100, 220, 256, 257, 385, 1054]


def bf16_to_f64(t):
    return (np_of(t).view(np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)


@pytest.fixture(scope="module")
def rig():
    from paper_2508_18588_amd.runtime import Engine
    # d_ffn = 704: 44 SwiGLU units of 16 columns, not a multiple of the 4 or 5 units a workgroup takes
    shape = ModelShape(n_layers=1, d_model=1024, n_q_heads=8, n_kv_heads=2, head_dim=128, d_ffn=704, vocab=16448)
    w = make_weights(shape, 51)
    eng = Engine(shape, w, rope_table(64, shape.head_dim), max_batch=64, k_max=16, c_max=1, max_len=32,
                 max_rows=M_MAX)
    g = torch.Generator(device="cuda:0").manual_seed(5)
    a_d = torch.randn(M_MAX, shape.d_model, device="cuda:0", generator=g).to(torch.bfloat16).view(torch.int16)
    a_f = torch.randn(M_MAX, shape.d_ffn, device="cuda:0", generator=g).to(torch.bfloat16).view(torch.int16)
    yield shape, eng, a_d, a_f
    eng.close()


def run(eng, epi, a, w, w2, m, hint, init=None):
    n = int(w.shape[0])
    c = torch.full((M_MAX, n), 7.0 if init is None else init, dtype=torch.float32, device="cuda:0")
    if epi == 2:
        c = torch.full((M_MAX, n), 0x4170, dtype=torch.int16, device="cuda:0")      # bf16 15.0
    m_dev = torch.full((1,), m, dtype=torch.int32, device="cuda:0")
    eng.gemm(epi, a, w, w2, c, m_dev, M_MAX, hint)
    torch.cuda.synchronize()
    assert eng.poll_error() == 0
    return c


@pytest.mark.parametrize("name", ["qkv", "o", "down", "lm_head", "gate_up"])
def test_projection_equals_its_definition_for_every_row_count_and_hint(rig, name):
    shape, eng, a_d, a_f = rig
    W = eng.w
    qh = shape.n_q_heads * shape.head_dim
    a, w, w2, epi = {"qkv": (a_d, W["wqkv"][0], None, 0), "o": (a_d[:, :qh].contiguous(), W["wo"][0], None, 1),
                     "down": (a_f, W["wdown"][0], None, 1), "lm_head": (a_d, W["lm_head"], None, 0),
                     "gate_up": (a_d, W["wgate"][0], W["wup"][0], 2)}[name]
    af, wf = bf16_to_f64(a), bf16_to_f64(w)
    for m in ROWS:
        want = af[:m] @ wf.T
        if epi == 2:
            up = af[:m] @ bf16_to_f64(w2).T
            want = want / (1.0 + np.exp(-want)) * up
        elif epi == 1:
            want = want + 7.0                                   # added to what the output held
        outs = []
        for hint in (m, 1, 5000):
            c = run(eng, epi, a, w, w2, m, hint)
            got = bf16_to_f64(c) if epi == 2 else np_of(c).astype(np.float64)
            scale = np.abs(want).max() + 1.0
            # fp32 accumulation over k <= 1024 (store/add); one bf16 rounding of the result (SwiGLU)
            tol = 2.0 ** -8 * scale if epi == 2 else 2e-5 * scale
            assert np.abs(got[:m] - want).max() <= tol, (name, m, hint)
            rest = np_of(c)[m:]
            assert (rest == (0x4170 if epi == 2 else 7.0)).all(), (name, m, hint, "rows beyond M were written")
            outs.append(np_of(c)[:m].copy())
        assert (outs[0] == outs[1]).all() and (outs[0] == outs[2]).all(), (name, m, "row hint changed the bits")


@pytest.mark.parametrize("vocab", [4160, 4097])
def test_lm_head_of_a_small_vocabulary_splits_k_and_has_room_for_its_partial_sums(vocab):
    """vocab 4160 with d_model 1024: the LM head runs in 3 K chunks whose partial sums (3 x 4160 columns) are wider
    than those of any layer projection; the workspace must hold them.  One projection against its definition, then a
    few decode steps end to end (the LM head inside hs_verify) against the oracle.  vocab 4097: rows of the partial
    sums and of the logits are not 16-byte aligned (the ordered reduce and the argmax take their scalar paths)."""
    import oracle
    from paper_2508_18588_amd.runtime import Engine, Policy
    from gpu_common import OracleBatch
    from test_gpu_decode import lockstep
    shape = ModelShape(n_layers=1, d_model=1024, n_q_heads=8, n_kv_heads=2, head_dim=128, d_ffn=1024, vocab=vocab)
    w = make_weights(shape, 53)
    rope = rope_table(128, shape.head_dim)
    eng = Engine(shape, w, rope, max_batch=4, k_max=4, c_max=1, max_len=64, max_rows=300)
    g = torch.Generator(device="cuda:0").manual_seed(6)
    a = torch.randn(300, shape.d_model, device="cuda:0", generator=g).to(torch.bfloat16).view(torch.int16)
    want = bf16_to_f64(a) @ bf16_to_f64(eng.w["lm_head"]).T
    for m in (3, 300):
        c = torch.zeros(300, shape.vocab, dtype=torch.float32, device="cuda:0")
        m_dev = torch.full((1,), m, dtype=torch.int32, device="cuda:0")
        eng.gemm(0, a, eng.w["lm_head"], None, c, m_dev, 300, m)
        torch.cuda.synchronize()
        assert np.abs(np_of(c)[:m] - want[:m]).max() <= 2e-5 * (np.abs(want).max() + 1.0)
        assert not np_of(c)[m:].any()
    rng = np.random.default_rng(9)
    prompts = [rng.integers(0, shape.vocab, 20).astype(np.int32) for _ in range(4)]
    eng.load_sequences(prompts, budgets=[6] * 4)
    eng.set_history([[np.zeros(0, np.int32)] for _ in prompts])
    eng.prefill(prompts)
    ob = OracleBatch(oracle.Model(shape, w, rope), prompts, [6] * 4, 64)
    stats = lockstep(eng, ob, [[np.zeros(0, np.int32)] for _ in prompts], Policy(window=8, m_min=3, k_fixed=0, k_max=4),
                     max_steps=6)
    assert stats["emitted"] == 24
    eng.close()


REAL_SHAPES = {
    # the layer projections of the 7B shape (configurations 3 and 4) and of the 14B shape (configuration 5)
    "7b": ModelShape(n_layers=1, d_model=3584, n_q_heads=28, n_kv_heads=4, head_dim=128, d_ffn=18944, vocab=16448),
    "14b": ModelShape(n_layers=1, d_model=5120, n_q_heads=40, n_kv_heads=8, head_dim=128, d_ffn=13824, vocab=16448),
}


@pytest.mark.parametrize("which", ["7b", "14b"])
def test_projections_at_the_real_layer_shapes(which):
    """Each layer projection at its real (N, K) -- 7B: QKV 4608 x 3584, O 3584 x 3584, gate/up 2 x 18944 x 3584, down
    3584 x 18944 (nine K chunks); 14B: 7168 x 5120, 5120 x 5120, 2 x 13824 x 5120, 5120 x 13824 -- at 220, 385, 1054
    and 2176 rows (one short pass, two passes, three, six), against C = A . W^T: every element against an fp64 matrix
    product (library routine on the device), sampled rows and columns against fp64 dot products on the host; rows
    beyond M untouched; bits independent of the row hint."""
    from hs_inputs.device import make_weights_device
    from paper_2508_18588_amd.runtime import Engine
    shape = REAL_SHAPES[which]
    m_max = 2176
    w = make_weights_device(shape, 61, 1)
    eng = Engine(shape, w, rope_table(64, shape.head_dim), max_batch=128, k_max=16, c_max=1, max_len=32,
                 max_rows=m_max, keep_logits=False)
    g = torch.Generator(device="cuda:0").manual_seed(8)
    qh = shape.n_q_heads * shape.head_dim
    a_d = torch.randn(m_max, shape.d_model, device="cuda:0", generator=g).to(torch.bfloat16)
    a_q = torch.randn(m_max, qh, device="cuda:0", generator=g).to(torch.bfloat16)
    a_f = torch.randn(m_max, shape.d_ffn, device="cuda:0", generator=g).to(torch.bfloat16)
    W = eng.w
    rng = np.random.default_rng(12)
    cases = {"qkv": (a_d, W["wqkv"][0], None, 0), "o": (a_q, W["wo"][0], None, 1),
             "gate_up": (a_d, W["wgate"][0], W["wup"][0], 2), "down": (a_f, W["wdown"][0], None, 1)}
    for name, (a, wt, w2, epi) in cases.items():
        n, k = int(wt.shape[0]), int(wt.shape[1])
        ref = a.double() @ wt.double().T                       # [m_max, n] fp64 on the device
        if epi == 2:
            ref = ref / (1.0 + torch.exp(-ref)) * (a.double() @ w2.double().T)
        elif epi == 1:
            ref = ref + 7.0
        scale = float(ref.abs().max()) + 1.0
        for m in (220, 385, 1054, 2176):
            outs = []
            for hint in (m, 1, 5000):
                fill = 0x4170 if epi == 2 else 7.0
                c = torch.full((m_max, n), fill, dtype=torch.int16 if epi == 2 else torch.float32, device="cuda:0")
                m_dev = torch.full((1,), m, dtype=torch.int32, device="cuda:0")
                eng.gemm(epi, a.view(torch.int16), wt, w2, c, m_dev, m_max, hint)
                torch.cuda.synchronize()
                assert eng.poll_error() == 0
                got = c.view(torch.bfloat16).double() if epi == 2 else c.double()
                err = (got[:m] - ref[:m]).abs()
                if epi == 2:   # one bf16 rounding of the result (+ the epilogue's hardware exponential / reciprocal)
                    ok = bool((err <= 1.5 * 2.0 ** -8 * ref[:m].abs() + 4e-5 * scale).all())
                else:          # fp32 accumulation over K in the shape's chunk order
                    ok = float(err.max()) <= 2e-5 * scale
                assert ok, (which, name, m, hint, float(err.max()))
                assert bool((c[m:] == fill).all()), (which, name, m, hint, "rows beyond M were written")
                outs.append(c[:m].clone())
            assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2]), (name, m, "row hint changed bits")
            # sampled outputs against fp64 dot products computed on the host
            rs = np.unique(np.concatenate([rng.integers(0, m, 6), [0, m - 1, min(m - 1, 383), min(m - 1, 384)]]))
            cs = np.unique(np.concatenate([rng.integers(0, n, 12), [0, n - 1, 63, 64, 159, 160]]))
            ah = bf16_to_f64(a.view(torch.int16)[torch.as_tensor(rs, device="cuda:0")])
            want = ah @ bf16_to_f64(wt.view(torch.int16)[torch.as_tensor(cs, device="cuda:0")]).T
            if epi == 2:
                up = ah @ bf16_to_f64(w2.view(torch.int16)[torch.as_tensor(cs, device="cuda:0")]).T
                want = want / (1.0 + np.exp(-want)) * up
            elif epi == 1:
                want = want + 7.0
            sub = outs[0][torch.as_tensor(rs, device="cuda:0")][:, torch.as_tensor(cs, device="cuda:0")]
            sub = bf16_to_f64(sub) if epi == 2 else np_of(sub).astype(np.float64)
            tol = 1.5 * 2.0 ** -8 * np.abs(want) + 4e-5 * scale if epi == 2 else 2e-5 * scale
            assert (np.abs(sub - want) <= tol).all(), (which, name, m, "host dot products")
        del ref
    eng.close()


def test_a_square_projection_of_the_feed_forward_width_has_room_for_its_partial_sums():
    """hs_debug_gemm takes any shape within the model's widths whose partial sums fit the scratch at all of its rows: at the
    1.5B widths 8960 x 8960, in three chunks, does -- however few chunks the model's own down projection runs in."""
    from paper_2508_18588_amd.runtime import Engine
    shape = ModelShape(n_layers=1, d_model=1536, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ffn=8960, vocab=64)
    eng = Engine(shape, make_weights(shape, 5), rope_table(64, shape.head_dim), max_batch=2, k_max=15, c_max=1, max_len=32)
    g = torch.Generator(device="cuda:0").manual_seed(3)
    m, n = eng.max_rows, 8960
    a = torch.randn(m, n, device="cuda:0", generator=g).to(torch.bfloat16)
    w = (torch.randn(n, n, device="cuda:0", generator=g) * 0.02).to(torch.bfloat16)
    c = torch.zeros(m, n, dtype=torch.float32, device="cuda:0")
    eng.gemm(0, a, w, None, c, torch.full((1,), m, dtype=torch.int32, device="cuda:0"), m, m)
    torch.cuda.synchronize()
    want = a.double() @ w.double().T.contiguous()
    assert float((c.double() - want).abs().max()) <= 2e-5 * (float(want.abs().max()) + 1.0)
    eng.close()


@pytest.mark.parametrize("epi,n,k,hint", [(2, 1910, 1088, 4096), (1, 3810, 1088, 4096), (0, 10290, 192, 1280), (1, 10290, 192, 1280),
                                          (2, 12810, 1024, 1280)])
def test_four_wavefront_workgroups_and_passes_of_64_rows(epi, n, k, hint):
    """Shapes at which a hint of many rows selects workgroups of 256 rows x 8 units (from three k-tiles, as many as the rings
    hold, to 17; unsplit and split K; the last unit and the last group ragged), and a hint of one row passes of 64 rows: at
    row counts around the edges of either, the product's definition (fp64 on the same operands) and the bits of the other
    launch shapes, and nothing beyond the live rows."""
    from paper_2508_18588_amd.runtime import Engine
    shape = ModelShape(n_layers=1, d_model=3840, n_q_heads=8, n_kv_heads=2, head_dim=128, d_ffn=1088, vocab=12864)
    eng = Engine(shape, make_weights(shape, 1), rope_table(64, 128), max_batch=1, k_max=0, c_max=1, max_len=32, max_rows=hint, keep_logits=False)
    g = torch.Generator(device="cuda:0").manual_seed(n + epi)
    rnd = lambda r, s: (torch.randn(r, k, device="cuda:0", generator=g) * s).to(torch.bfloat16)
    a, w, w2 = rnd(hint, 1.0), rnd(n, 0.05), rnd(n, 0.05) if epi == 2 else None
    bits = lambda t: None if t is None else t.view(torch.int16)
    for m in (1, 33, 64, 65, 255, 257, 700, hint):
        want = a[:m].double() @ w.double().T
        if epi == 2:
            want = want * torch.sigmoid(want) * (a[:m].double() @ w2.double().T)
        outs = []
        for h in (100, 1, hint):
            c = torch.full((hint, n), 15.0, device="cuda:0", dtype=torch.bfloat16 if epi == 2 else torch.float32)
            m_dev = torch.full((1,), m, dtype=torch.int32, device="cuda:0")
            eng.gemm(epi, bits(a), bits(w), bits(w2), bits(c) if epi == 2 else c, m_dev, hint, h)
            torch.cuda.synchronize()
            assert (c[m:] == 15.0).all(), (m, h, "rows beyond M were written")
            outs.append(c[:m])
        # fp32 sums of at most 1088 products; one bf16 rounding of the result (SwiGLU)
        tol = (2.0 ** -8 if epi == 2 else 2e-5) * (want.abs().max() + 1.0)
        assert (outs[0].double() - want - (15.0 if epi == 1 else 0.0)).abs().max() <= tol, m
        assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2]), (m, "row hint changed the bits")
    eng.close()


def _launch_us(call, n=10):
    """Median time of a launch in microseconds, five times n of them in a row."""
    times = []
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(n):
            call()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) / n * 1e3)
    return sorted(times[1:])[2]


@pytest.mark.parametrize("epi,n,k,m,hint,most", [(0, 16448, 3584, 990, 30, 2.2), (2, 13824, 3584, 990, 30, 2.2),
                                                 (0, 4608, 3584, 220, 990, 1.3), (2, 13824, 3584, 220, 990, 1.5)])
def test_a_wrong_row_hint_costs_little(epi, n, k, m, hint, most):
    """The hint is the caller's guess, and drafting makes the row count swing: launched for `hint` rows, m rows may take at most
    `most` times what they take with the right hint.  (30 for 990: 1.4 as measured, the passes being of 256 rows instead of
    384; 3.6 if they were of 64.  220 for 990: 1.0; 1.5 and 2.4 if the workgroups of the passes without rows
    took no share of the work.)"""
    from paper_2508_18588_amd.runtime import Engine
    shape = ModelShape(n_layers=1, d_model=3584, n_q_heads=28, n_kv_heads=4, head_dim=128, d_ffn=13824, vocab=16448)
    eng = Engine(shape, make_weights(shape, 1), rope_table(64, 128), max_batch=1, k_max=0, c_max=1, max_len=32, max_rows=1024, keep_logits=False)
    g = torch.Generator(device="cuda:0").manual_seed(n)
    rnd = lambda r, s: (torch.randn(r, k, device="cuda:0", generator=g) * s).to(torch.bfloat16).view(torch.int16)
    a, w, w2 = rnd(1024, 1.0), rnd(n, 0.05), rnd(n, 0.05) if epi == 2 else None
    c = torch.zeros(1024, n, device="cuda:0", dtype=torch.int16 if epi == 2 else torch.float32)
    m_dev = torch.full((1,), m, dtype=torch.int32, device="cuda:0")
    right, wrong = (_launch_us(lambda: eng.gemm(epi, a, w, w2, c, m_dev, 1024, h)) for h in (m, hint))
    eng.close()
    print("right and wrong hint, us:", right, wrong)
    assert wrong <= most * right, (right, wrong)


def test_row_maxima_of_more_rows_than_the_hint_of_few():
    """The LM head's keys (epi 3), launched for one row and for 300: the same bits from one row to several passes."""
    from paper_2508_18588_amd import lib
    from paper_2508_18588_amd.runtime import Engine
    n, k = 12810, 1024
    shape = ModelShape(n_layers=1, d_model=k, n_q_heads=8, n_kv_heads=2, head_dim=128, d_ffn=1088, vocab=n)
    eng = Engine(shape, make_weights(shape, 1), rope_table(64, 128), max_batch=1, k_max=0, c_max=1, max_len=32, max_rows=704, keep_logits=False)
    g = torch.Generator(device="cuda:0").manual_seed(8)
    a = torch.randn(704, k, device="cuda:0", generator=g).to(torch.bfloat16)
    w = (torch.randn(n, k, device="cuda:0", generator=g) * 0.05).to(torch.bfloat16)
    groups = lib().hs_debug_rowmax_groups(n)
    for m in (1, 64, 65, 256, 257, 700):
        m_dev = torch.full((1,), m, dtype=torch.int32, device="cuda:0")
        keys = []
        for hint in (1, 300):
            c = torch.zeros(704, groups, dtype=torch.int64, device="cuda:0")
            eng.gemm(3, a.view(torch.int16), w.view(torch.int16), None, c, m_dev, 704, hint)
            torch.cuda.synchronize()
            assert (c[m:] == 0).all()
            keys.append(np_of(c[:m]).view(np.uint64))
        assert (keys[0] == keys[1]).all(), m
        want = (a[:m].float() @ w.float().T)
        best = (0xFFFFFFFF - (keys[0].max(1) & 0xFFFFFFFF)).astype(np.int64)
        got = want[torch.arange(m, device="cuda:0"), torch.from_numpy(best).cuda()]
        # (two fp32 sums of 1024 products in another order: the named column is within their rounding of the largest)
        assert (want.max(1).values - got <= 2e-4).all(), m
    eng.close()


@pytest.mark.parametrize("n", [6380, 10316])
def test_groups_side_by_side(n):
    """Eight and more passes: an XCD runs four groups side by side, and the rest of its groups after them -- seven groups of
    four units (eight wavefronts), six of eight units of which most XCDs have five (four wavefronts).  The product's
    definition and the bits of launches with two passes, with all passes full, the last one ragged, and half of them empty."""
    from paper_2508_18588_amd.runtime import Engine
    k, hint = 192, 3072
    shape = ModelShape(n_layers=1, d_model=192, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=192, vocab=10368)
    eng = Engine(shape, make_weights(shape, 1), rope_table(64, 64), max_batch=1, k_max=0, c_max=1, max_len=32, max_rows=hint, keep_logits=False)
    g = torch.Generator(device="cuda:0").manual_seed(n)
    rnd = lambda r, s: (torch.randn(r, k, device="cuda:0", generator=g) * s).to(torch.bfloat16)
    a, w = rnd(hint, 1.0), rnd(n, 0.05)
    for m in (hint, 2825, 1500):
        want = a[:m].double() @ w.double().T
        outs = []
        for h in (500, hint):
            c = torch.full((hint, n), 15.0, device="cuda:0")
            m_dev = torch.full((1,), m, dtype=torch.int32, device="cuda:0")
            eng.gemm(0, a.view(torch.int16), w.view(torch.int16), None, c, m_dev, hint, h)
            torch.cuda.synchronize()
            assert (c[m:] == 15.0).all(), (m, h, "rows beyond M were written")
            outs.append(c[:m])
        # fp32 sums of 192 products
        assert (outs[1].double() - want).abs().max() <= 2e-5 * (want.abs().max() + 1.0), m
        assert torch.equal(outs[0], outs[1]), (m, "row hint changed the bits")
    eng.close()


@pytest.mark.parametrize("epi,n,k", [(0, 1616, 64), (2, 1616, 128), (0, 1616, 192), (1, 1616, 320), (2, 1616, 448), (0, 28832, 320),
                                     (0, 3600, 18432), (1, 3600, 18432)])
def test_operands_fetched_by_a_wavefront_group_each(epi, n, k):
    """Launches for up to 160 expected rows fetch activations and weights in different wavefronts, each group with waits of its
    own: fewer k-tiles than either ring has stages, as many, more; three and four units to a group, split K; row counts around
    the edges of 8-row blocks, tiles and passes, below and above the hint.  The product's definition in fp64, and the bits of
    the launch for many rows."""
    from paper_2508_18588_amd.runtime import Engine
    rows = 300
    shape = ModelShape(n_layers=1, d_model=3648 if k > 448 else 448, n_q_heads=8, n_kv_heads=2, head_dim=128, d_ffn=max(k, 448),
                       vocab=max(n, 512))
    eng = Engine(shape, make_weights(shape, 1), rope_table(64, 128), max_batch=1, k_max=0, c_max=1, max_len=32, max_rows=rows,
                 keep_logits=False)
    g = torch.Generator(device="cuda:0").manual_seed(n + k)
    rnd = lambda r, s: (torch.randn(r, k, device="cuda:0", generator=g) * s).to(torch.bfloat16)
    a, w, w2 = rnd(rows, 1.0), rnd(n, 0.05), rnd(n, 0.05) if epi == 2 else None
    bits = lambda t: None if t is None else t.view(torch.int16)
    for m in (1, 7, 9, 32, 63, 65, 160, 257, rows):
        want = a[:m].double() @ w.double().T
        if epi == 2:
            want = want * torch.sigmoid(want) * (a[:m].double() @ w2.double().T)
        outs = []
        for h in (300, 1, 32, 33, 160):
            c = torch.full((rows, n), 15.0, device="cuda:0", dtype=torch.bfloat16 if epi == 2 else torch.float32)
            m_dev = torch.full((1,), m, dtype=torch.int32, device="cuda:0")
            eng.gemm(epi, bits(a), bits(w), bits(w2), bits(c) if epi == 2 else c, m_dev, rows, h)
            torch.cuda.synchronize()
            assert (c[m:] == 15.0).all(), (m, h, "rows beyond M were written")
            outs.append(c[:m])
        # fp32 sums of k products of size 0.05: an error of 2^-24 each, at most sqrt(k) of them in a row's favour times ten;
        # one bf16 rounding of the result (SwiGLU)
        tol = 2.0 ** -8 * (want.abs().max() + 1.0) if epi == 2 else 10 * 2.0 ** -24 * k ** 0.5 * (float(want.abs().max()) + 15.0)
        assert (outs[0].double() - want - (15.0 if epi == 1 else 0.0)).abs().max() <= tol, m
        assert all(torch.equal(outs[0], o) for o in outs[1:]), (m, "row hint changed the bits")
    eng.close()
