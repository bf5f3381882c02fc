"""GPU parity of hs_accept in rejection-sampling mode (and greedy mode on given logits) against the oracle.

The acceptance rule is speculative sampling with a point-mass draft (Sec. 2.2 of the paper: the verified tokens
that are valid are kept and the output distribution is preserved).  Both sides get the SAME fp32 logits, the same
seed, sequence ids and positions, so every decision (accepted path, emitted tokens) must be identical; the only
admissible differences are decisions whose uniform lies within rounding distance of its threshold, which the
oracle reports as a margin.  The Philox stream is thereby checked bit for bit as well: one wrong uniform changes
a decision somewhere in thousands of draws."""
import numpy as np
import pytest
import torch

import oracle
from hs_inputs import CONFIG_SHAPES, make_weights, rope_table, make_prompts, config_seed
from gpu_common import LOGIT_TOL, OracleBatch, make_histories, np_of

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def toy():
    shape = CONFIG_SHAPES[1]
    return shape, make_weights(shape, seed=1), rope_table(4096, shape.head_dim)


def random_trees(rng, B, k_max, vocab, two):
    trees = []
    for b in range(B):
        k0 = int(rng.integers(0, k_max + 1))
        c0 = rng.integers(0, vocab, k0)
        chains = [c0]
        if two:
            k1 = int(rng.integers(0, k_max + 1))
            share = int(rng.integers(0, min(k0, k1) + 1))
            chains.append(np.concatenate([c0[:share], rng.integers(0, vocab, k1 - share)]))
        L = int(rng.integers(0, 3000))
        trees.append(oracle.build_tree(chains, int(rng.integers(0, vocab)), L))
    return trees


@pytest.mark.parametrize("two,temperature", [(False, 1.0), (True, 1.0), (True, 0.6)])
def test_rejection_accept_matches_oracle_on_given_logits(toy, two, temperature):
    from paper_2508_18588_amd import HS_ACCEPT_GREEDY, HS_ACCEPT_REJECTION
    from paper_2508_18588_amd.runtime import Engine
    shape, w, rope = toy
    V, B, k_max = shape.vocab, 48, 8
    temperature = float(np.float32(temperature))   # the C ABI carries the temperature as fp32
    rng = np.random.default_rng(5 + int(two) + int(temperature * 10))
    eng = Engine(shape, w, rope, max_batch=B, k_max=k_max, c_max=2, max_len=3200)
    eng.load_sequences([np.array([1], np.int32)] * B, budgets=[100] * B,
                       seq_ids=rng.integers(0, 2 ** 62, B).astype(np.int64))
    seq_ids = np_of(eng.seq_id)[:B].astype(np.uint64)
    n_acc, n_flag, n_dec = 0, 0, 0
    for trial in range(6):
        trees = random_trees(rng, B, k_max, V, two)
        m = eng.set_rows([dict(tok=t["tok"], parent=t["parent"], pos=t["pos"]) for t in trees])
        # peaked synthetic logits: every node's children get a boost so that about half of the drafts are accepted
        lg = rng.normal(0.0, 2.0, size=(m, V)).astype(np.float32)
        r = 0
        for t in trees:
            n = len(t["tok"])
            for i in range(1, n):
                lg[r + t["parent"][i], t["tok"][i]] += rng.choice([0.0, 6.0, 9.0, 12.0])
            r += n
        eng.logits[:m].copy_(torch.from_numpy(lg))
        seed = int(rng.integers(0, 2 ** 63))
        eng.accept(HS_ACCEPT_REJECTION, temperature, seed)
        torch.cuda.synchronize()
        st = {k: np_of(v) for k, v in eng.st.items()}
        r = 0
        for b, t in enumerate(trees):
            n = len(t["tok"])
            a, out, path, margin = oracle.accept_stochastic(t["tok"], t["parent"], t["pos"],
                                                            lg[r:r + n].astype(np.float64), temperature, seed,
                                                            int(seq_ids[b]))
            got = (int(st["accept_len"][b]), st["out_tok"][b, :st["n_out"][b]].tolist(),
                   st["path_row"][b, :st["n_out"][b]].tolist())
            n_dec += 1
            if got != (a, out.tolist(), path.tolist()):
                assert margin < 1e-9, (trial, b, got, (a, out.tolist(), path.tolist()), margin)
                n_flag += 1
            assert st["n_out"][b] == st["accept_len"][b] + 1
            n_acc += a
            r += n
        # greedy mode on the same logits: walk of the per-row argmax (argmax supplied as hs_verify would)
        arg = lg[:m].argmax(1).astype(np.int32)
        eng.st["argmax"][:m].copy_(torch.from_numpy(arg))
        eng.accept(HS_ACCEPT_GREEDY)
        torch.cuda.synchronize()
        st = {k: np_of(v) for k, v in eng.st.items()}
        r = 0
        for b, t in enumerate(trees):
            n = len(t["tok"])
            a, out, path = oracle.accept_greedy(t["tok"], t["parent"], arg[r:r + n])
            assert st["accept_len"][b] == a and st["out_tok"][b, :a + 1].tolist() == out.tolist()
            assert st["path_row"][b, :a + 1].tolist() == path.tolist()
            r += n
    eng.close()
    print("rejection accept: decisions", n_dec, "accepted tokens", n_acc, "flagged", n_flag)
    assert n_acc > 50 and n_flag <= 2


def test_finished_and_empty_sequences(toy):
    """Sequences without rows (budget spent) must report n_out = 0 in both modes."""
    from paper_2508_18588_amd import HS_ACCEPT_GREEDY, HS_ACCEPT_REJECTION
    from paper_2508_18588_amd.runtime import Engine
    shape, w, rope = toy
    eng = Engine(shape, w, rope, max_batch=3, k_max=2, c_max=1, max_len=64)
    eng.load_sequences([np.array([1, 2], np.int32)] * 3, budgets=[5, 0, 5])
    t = oracle.build_tree([[7, 8]], 2, 1)
    eng.set_rows([dict(tok=t["tok"], parent=t["parent"], pos=t["pos"]), None,
                  dict(tok=t["tok"][:1], parent=t["parent"][:1], pos=t["pos"][:1])])
    eng.logits.zero_()
    eng.logits[0, 7] = 50.0   # certain accept of the first draft token
    eng.logits[1, 3] = 50.0   # then certain rejection of 8: token 3 has all the mass
    eng.logits[3, 9] = 50.0
    for mode in (HS_ACCEPT_REJECTION, HS_ACCEPT_GREEDY):
        eng.st["argmax"][:4].copy_(torch.tensor([7, 3, 0, 9], dtype=torch.int32))
        eng.accept(mode, 1.0, 123)
        torch.cuda.synchronize()
        assert np_of(eng.st["n_out"]).tolist() == [2, 0, 1]
        assert np_of(eng.st["out_tok"])[0, :2].tolist() == [7, 3]
        assert np_of(eng.st["out_tok"])[2, 0] == 9
    eng.close()


@pytest.mark.parametrize("precise", [False, True])
def test_tree_rejection_sampling_end_to_end(toy, precise):
    """Two history candidates per sequence, tree-mask verify, rejection sampling at a low temperature (so that
    drafts are accepted with a useful probability), tree commit -- in lock-step with the oracle: logits within the
    tolerance every step.  Default path: the GPU's decisions equal the oracle's rule applied to the GPU's own logits.
    fp32-activation mode: the logits agree to 1e-4 relative, and the GPU's decisions equal the oracle's rule applied
    to the ORACLE's own logits -- the whole stochastic step end to end against an independent computation (a decision
    may differ only where the oracle reports a uniform within 1e-4 of its threshold)."""
    from paper_2508_18588_amd import HS_ACCEPT_REJECTION
    from paper_2508_18588_amd.runtime import Engine, Policy
    from test_gpu_decode import gpu_ar_rollout, check_cache
    shape = CONFIG_SHAPES[1]
    seed = config_seed(5)
    w = make_weights(shape, seed)
    rope = rope_table(512, shape.head_dim)
    model = oracle.Model(shape, w, rope)
    prompts = make_prompts(4, 48, shape.vocab, seed)
    rolls = gpu_ar_rollout(shape, w, rope, list(prompts), 96)
    h0 = make_histories(prompts, rolls, 8, 0.40, 0.0, shape.vocab, seed=90)
    h1 = make_histories(prompts, rolls, 8, 0.60, 0.0, shape.vocab, seed=91)
    cands = [[h0[b][0], h1[b][0]] for b in range(4)]
    pol = Policy(window=8, m_min=3, k_fixed=8, k_max=8)
    T, pseed = float(np.float32(0.02)), 0xABCDEF12345
    eng = Engine(shape, w, rope, max_batch=4, k_max=8, c_max=2, max_len=48 + 96, shuffle_pages_seed=12,
                 precise=precise)
    sids = [11, 2 ** 40 + 5, 7, 2 ** 62 + 1]
    eng.load_sequences(list(prompts), budgets=[96] * 4, seq_ids=sids)
    eng.set_history(cands)
    eng.prefill(list(prompts))
    ob = OracleBatch(model, list(prompts), [96] * 4, 48 + 96 + 24)
    accepted = steps = flagged = 0
    while any(b > 0 for b in ob.budget) and steps < 200:
        eng.draft(pol)
        eng.verify()
        eng.accept(HS_ACCEPT_REJECTION, T, pseed)
        torch.cuda.synchronize()
        st = {k: np_of(v) for k, v in eng.st.items()}
        lg = np_of(eng.logits)
        eng.commit(pol)
        ro = st["row_off"]
        for b in range(4):
            info, tree = ob.draft(b, cands[b], pol)
            if tree is None:
                assert st["n_out"][b] == 0
                continue
            sl = slice(ro[b], ro[b + 1])
            assert st["tok"][sl].tolist() == tree["tok"].tolist()
            assert st["pos"][sl].tolist() == tree["pos"].tolist()
            want = ob.logits(b, tree)
            assert np.abs(lg[sl] - want).max() <= LOGIT_TOL
            if precise:
                assert (np.abs(lg[sl] - want).max(1) <= 1e-4 * np.abs(want).max(1)).all()
            a, out, path, margin = oracle.accept_stochastic(tree["tok"], tree["parent"], tree["pos"],
                                                            want if precise else lg[sl].astype(np.float64), T, pseed,
                                                            sids[b])
            n = st["n_out"][b]
            got = (int(st["accept_len"][b]), st["out_tok"][b, :n].tolist(), st["path_row"][b, :n].tolist())
            near = 1e-4 if precise else 1e-9
            flagged += got != (a, out.tolist(), path.tolist())
            assert got == (a, out.tolist(), path.tolist()) or margin < near, (b, got, a, out, path, margin)
            ob.commit(b, tree, got[0], np.array(got[1]), np.array(got[2]), pol)
            accepted += got[0]
        steps += 1
    torch.cuda.synchronize()
    assert np_of(eng.seq_len)[:4].tolist() == [len(x) for x in ob.x]
    toks = np_of(eng.tokens)
    for b in range(4):
        assert toks[b, :len(ob.x[b])].tolist() == ob.x[b]
    for layer in (0, 1):
        check_cache(eng, ob, layer)
    eng.close()
    print("tree rejection e2e: precise", precise, "steps", steps, "accepted", accepted, "near-threshold", flagged)
    assert flagged <= 2
    assert accepted > 5   # sampling soon leaves the greedy history; the draft path was still exercised


def test_philox_words_equal_the_oracles_on_a_million_counters():
    """The generator itself, GPU against the oracle, bit for bit: all four output words of 2^20 counters -- the
    counter layouts hs_accept uses (position, draw kind 0..7, 64-bit sequence ids) and fully random 128-bit counters
    -- under three keys."""
    import oracle
    from paper_2508_18588_amd import hs_debug_philox
    rng = np.random.default_rng(31)
    n = 1 << 20
    ctr = rng.integers(0, 2 ** 32, (n, 4), dtype=np.uint64).astype(np.uint32)
    half = n // 2
    ctr[:half, 0] = rng.integers(0, 40000, half)      # positions
    ctr[:half, 1] = rng.integers(0, 8, half)          # draw kinds
    ctr[0] = 0
    ctr[1] = 0xFFFFFFFF
    d_ctr = torch.from_numpy(ctr.view(np.int32)).cuda()
    d_out = torch.empty_like(d_ctr)
    for seed in (0, 0xC0FFEE05 * 0x9E3779B1 & (2 ** 63 - 1), 2 ** 64 - 1):
        hs_debug_philox(d_ctr.data_ptr(), seed, d_out.data_ptr(), n, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        got = d_out.cpu().numpy().view(np.uint32)
        want = oracle.philox_batch(ctr, [seed & 0xFFFFFFFF, seed >> 32])
        assert (got == want).all(), seed


@pytest.mark.parametrize("V,B,k,rows_big", [(1, 2, 1, False), (4095, 3, 4, False), (4097, 3, 4, False),
                                            (12290, 5, 8, False), (8192, 70, 31, True)])
def test_rejection_over_several_vocabulary_slices(toy, V, B, k, rows_big):
    """The sampler sums the vocabulary in slices of 4096 tokens: widths at a slice's edge, one that is not a multiple of 4
    (rows then are not 16-byte aligned), rejected tokens in the first, a middle and the last slice, whole slices masked
    with -inf; and more than 2048 rows.  Same logits, seed and ids as the oracle: the same decisions, unless the oracle's margin is below 1e-9."""
    from paper_2508_18588_amd import HS_ACCEPT_REJECTION
    from paper_2508_18588_amd.runtime import Engine
    from hs_inputs import ModelShape
    shape = ModelShape(n_layers=1, d_model=64, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=V)
    rng = np.random.default_rng(V + B)
    eng = Engine(shape, make_weights(shape, 3), rope_table(64, 64), max_batch=B, k_max=k, c_max=1 if rows_big else 2, max_len=80)
    ids = rng.integers(0, 2 ** 62, B)
    eng.load_sequences([np.array([0], np.int32)] * B, budgets=[99] * B, seq_ids=ids.astype(np.int64))
    accepted = 0
    for trial in range(3):
        trees = []
        for b in range(B):
            c0 = rng.choice([0, V // 2, V - 1, int(rng.integers(0, V))], k)
            chains = [c0] if rows_big else [c0, rng.integers(0, V, k)]
            trees.append(oracle.build_tree(chains, 0, int(rng.integers(0, 3000))))
        m = eng.set_rows([dict(tok=t["tok"], parent=t["parent"], pos=t["pos"]) for t in trees])
        assert (m > 2048) == rows_big
        lg = rng.normal(0.0, 2.0, size=(m, V)).astype(np.float32)
        if V > 9000:
            lg[:, 4096:8192] = -np.inf
        r = 0
        for t in trees:
            for i in range(1, len(t["tok"])):
                lg[r + t["parent"][i], t["tok"][i]] = rng.choice([-np.inf, 9.0, 12.0, 30.0], p=[0.1, 0.2, 0.3, 0.4]) if V > 1 else 1.0
            r += len(t["tok"])
        eng.logits[:m].copy_(torch.from_numpy(lg))
        seed = int(rng.integers(0, 2 ** 63))
        eng.accept(HS_ACCEPT_REJECTION, 1.0, seed)
        torch.cuda.synchronize()
        st = {n: np_of(v) for n, v in eng.st.items()}
        r = 0
        for b, t in enumerate(trees):
            n = len(t["tok"])
            a, out, path, margin = oracle.accept_stochastic(t["tok"], t["parent"], t["pos"], lg[r:r + n].astype(np.float64),
                                                            1.0, seed, int(ids[b]))
            g = st["n_out"][b]
            got = (int(st["accept_len"][b]), st["out_tok"][b, :g].tolist(), st["path_row"][b, :g].tolist())
            assert got == (a, out.tolist(), path.tolist()) or margin < 1e-9, (trial, b, got, a, out, path, margin)
            accepted += a
            r += n
    eng.close()
    assert accepted > 0


@pytest.mark.parametrize("temperature", [1e-12, 1e-6, 1e-3, 50.0, 1e30])
def test_rejection_at_extreme_temperatures(toy, temperature):
    """Far below the spacing of fp32 logits (only the largest ones count, ties among them included) and far above their
    range (every token counts alike): same decisions as the oracle, unless its margin is below 1e-9."""
    from paper_2508_18588_amd import HS_ACCEPT_REJECTION
    from paper_2508_18588_amd.runtime import Engine
    shape, w, rope = toy
    V, B, T = shape.vocab, 6, float(np.float32(temperature))
    rng = np.random.default_rng(17)
    eng = Engine(shape, w, rope, max_batch=B, k_max=4, c_max=2, max_len=80)
    eng.load_sequences([np.array([0], np.int32)] * B, budgets=[99] * B)
    trees = [oracle.build_tree([rng.integers(0, V, 4), rng.integers(0, V, 4)], 0, 50) for _ in range(B)]
    m = eng.set_rows([dict(tok=t["tok"], parent=t["parent"], pos=t["pos"]) for t in trees])
    lg = rng.normal(10.0, 2.0, size=(m, V)).astype(np.float32)
    r = 0
    for t in trees:
        top = lg[r:r + len(t["tok"])].max()
        for i in range(1, len(t["tok"])):              # drafted tokens tie with, or lie one spacing off, the largest logit
            lg[r + t["parent"][i], t["tok"][i]] = rng.choice([top, np.nextafter(top, np.float32(0)), 3.0])
        lg[r:r + len(t["tok"]), 7] = top
        r += len(t["tok"])
    eng.logits[:m].copy_(torch.from_numpy(lg))
    eng.accept(HS_ACCEPT_REJECTION, T, 99)
    torch.cuda.synchronize()
    st = {n: np_of(v) for n, v in eng.st.items()}
    r = 0
    for b, t in enumerate(trees):
        n = len(t["tok"])
        a, out, path, margin = oracle.accept_stochastic(t["tok"], t["parent"], t["pos"], lg[r:r + n].astype(np.float64), T, 99, b)
        g = st["n_out"][b]
        got = (int(st["accept_len"][b]), st["out_tok"][b, :g].tolist(), st["path_row"][b, :g].tolist())
        assert got == (a, out.tolist(), path.tolist()) or margin < 1e-9, (b, got, a, out, path, margin)
        r += n
    eng.close()


@pytest.mark.parametrize("V", [4096, 4097, 6000])
def test_rejection_at_an_infinite_temperature_is_uniform_over_the_tokens_that_are_not_excluded(toy, V):
    """Every finite logit weighs the same and an excluded one (-inf) nothing, whether the vocabulary fills its last slice
    of 4096 tokens or not.  Finite logits: the oracle's decisions.  With half the vocabulary excluded: the oracle's
    decisions at a temperature so high that every finite difference is lost, 1e30."""
    from paper_2508_18588_amd import HS_ACCEPT_REJECTION
    from paper_2508_18588_amd.runtime import Engine
    from hs_inputs import ModelShape
    shape = ModelShape(n_layers=1, d_model=64, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=V)
    rng = np.random.default_rng(V)
    B = 40
    eng = Engine(shape, make_weights(shape, 3), rope_table(64, 64), max_batch=B, k_max=3, c_max=2, max_len=60)
    eng.load_sequences([np.array([0], np.int32)] * B, budgets=[99] * B)
    trees = [oracle.build_tree([rng.integers(0, V, 3), rng.integers(0, V, 3)], 0, 50) for _ in range(B)]
    m = eng.set_rows([dict(tok=t["tok"], parent=t["parent"], pos=t["pos"]) for t in trees])
    for excluded in (False, True):
        lg = rng.normal(0.0, 3.0, size=(m, V)).astype(np.float32)
        if excluded:
            lg[:, rng.permutation(V)[:V // 2]] = -np.inf
        eng.logits[:m].copy_(torch.from_numpy(lg))
        eng.accept(HS_ACCEPT_REJECTION, float("inf"), 7)
        torch.cuda.synchronize()
        st = {n: np_of(v) for n, v in eng.st.items()}
        r, last = 0, []
        for b, t in enumerate(trees):
            n = len(t["tok"])
            a, out, path, margin = oracle.accept_stochastic(t["tok"], t["parent"], t["pos"], lg[r:r + n].astype(np.float64),
                                                            1e30 if excluded else float("inf"), 7, b)
            g = st["n_out"][b]
            got = (int(st["accept_len"][b]), st["out_tok"][b, :g].tolist(), st["path_row"][b, :g].tolist())
            assert got == (a, out.tolist(), path.tolist()) or margin < 1e-9, (b, got, a, out, path, margin)
            assert np.isfinite(lg[r + st["path_row"][b, g - 1], got[1][-1]])
            last.append(got[1][-1])
            r += n
        assert len(set(last)) > B // 2
    eng.close()


@pytest.mark.parametrize("V,B,k", [(4096, 5, 4), (4097, 5, 4), (12290, 3, 8), (8192, 70, 31), (24576, 70, 31)])
def test_a_drafted_id_outside_the_vocabulary_is_a_token_of_weight_zero(toy, V, B, k):
    """Histories are the caller's: an id that the model does not know (negative, the vocabulary's size, far beyond) is
    rejected like a token whose logit is -inf, and the other rows of the batch are decided as if it were not there.  The
    oracle gets the logits with one more column, all -inf, and that column's id for every such token.  The last two shapes have
    2240 rows: all summed at once, and, 220 MB of logits, in stages."""
    from paper_2508_18588_amd import HS_ACCEPT_REJECTION
    from paper_2508_18588_amd.runtime import Engine
    from hs_inputs import ModelShape
    shape = ModelShape(n_layers=1, d_model=64, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=V)
    rng = np.random.default_rng(V + 1)
    eng = Engine(shape, make_weights(shape, 3), rope_table(64, 64), max_batch=B, k_max=k, c_max=2 if k < 31 else 1, max_len=80)
    eng.load_sequences([np.array([0], np.int32)] * B, budgets=[99] * B)
    strange = [-1, -5000, V, V + 1, V + 4096, 2 ** 31 - 1, -2 ** 31]
    accepted = 0
    for trial in range(3):
        trees = [oracle.build_tree([rng.integers(0, V, k) for _ in range(eng.c_max)], 0, 50) for _ in range(B)]
        tok, lg = [], rng.normal(0.0, 2.0, size=(sum(len(t["tok"]) for t in trees), V)).astype(np.float32)
        r = 0
        for t in trees:
            x = t["tok"].astype(np.int32).copy()
            for i in range(1, len(x)):
                lg[r + t["parent"][i], x[i]] = 30.0
                if rng.random() < 0.3:
                    x[i] = rng.choice(strange)
            tok.append(x)
            r += len(x)
        m = eng.set_rows([dict(tok=x, parent=t["parent"], pos=t["pos"]) for x, t in zip(tok, trees)])
        eng.logits[:m].copy_(torch.from_numpy(lg))
        eng.accept(HS_ACCEPT_REJECTION, 1.0, 5 + trial)
        torch.cuda.synchronize()
        st = {n: np_of(v) for n, v in eng.st.items()}
        wide = np.concatenate([lg.astype(np.float64), np.full((m, 1), -np.inf)], 1)
        r = 0
        for b, (x, t) in enumerate(zip(tok, trees)):
            n, known = len(x), np.where((x >= 0) & (x < V), x, V).astype(np.int32)
            a, out, path, margin = oracle.accept_stochastic(known, t["parent"], t["pos"], wide[r:r + n], 1.0, 5 + trial, b)
            g = st["n_out"][b]
            got = (int(st["accept_len"][b]), st["out_tok"][b, :g].tolist(), st["path_row"][b, :g].tolist())
            assert got == (a, out.tolist(), path.tolist()) or margin < 1e-9, (trial, b, got, a, out, path, margin)
            accepted += a
            r += n
    eng.close()
    assert accepted > 0


def sampled(eng, step, st, mode_args, stream):
    from paper_2508_18588_amd import hs_accept
    hs_accept(eng.ctx, mode_args, eng.c_seq, step, stream.cuda_stream)
    return st


def results_of(st):
    return [np_of(st[n]).copy() for n in ("accept_len", "n_out", "out_tok", "path_row")]


def test_overlapping_rejection_sampling_of_one_context_on_two_streams(toy):
    """Two calls of one context, each with its own step arrays and logits, are independent of each other also while they
    run side by side: both sum their rows into the same place of the workspace.  And whatever else happens to that place
    during a call (here another stream that keeps filling it with random bits) the call notices and sums for itself: the
    results are those of the same calls one after the other."""
    from paper_2508_18588_amd import HS_ACCEPT_REJECTION, hs_accept_args, hs_step
    from paper_2508_18588_amd.runtime import Engine
    from hs_inputs import ModelShape
    V, B, k = 65540, 16, 8
    shape = ModelShape(n_layers=1, d_model=64, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=V)
    rng = np.random.default_rng(4)
    eng = Engine(shape, make_weights(shape, 3), rope_table(64, 64), max_batch=B, k_max=k, c_max=2, max_len=80)
    eng.load_sequences([np.array([0], np.int32)] * B, budgets=[99] * B, seq_ids=rng.integers(0, 2 ** 62, B).astype(np.int64))
    sides = []
    for temperature in (1.0, 0.5):
        trees = [oracle.build_tree([rng.integers(0, V, k), rng.integers(0, V, k)], 0, 50) for _ in range(B)]
        m = eng.set_rows([dict(tok=t["tok"], parent=t["parent"], pos=t["pos"]) for t in trees])
        lg = torch.randn(eng.max_rows, V, generator=torch.Generator(device="cuda:0").manual_seed(9), device="cuda:0")
        r = 0
        for t in trees:
            for i in range(1, len(t["tok"])):
                lg[r + int(t["parent"][i]), int(t["tok"][i])] = temperature * (np.log(V) + 2.0)
            r += len(t["tok"])
        st = {n: v.clone() for n, v in eng.st.items()}
        step = hs_step(*[st[n].data_ptr() for n in ("draft_start", "match_len", "draft_len", "row_off", "tok", "pos", "parent",
                                                    "anc_mask", "row2seq")], lg.data_ptr(),
                       *[st[n].data_ptr() for n in ("argmax", "accept_len", "n_out", "out_tok", "path_row")], 0,
                       st["draft_src"].data_ptr())
        sides.append((step, st, hs_accept_args(HS_ACCEPT_REJECTION, temperature, 77), lg))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    want = []
    for (step, st, args, _), s in zip(sides, streams):
        torch.cuda.synchronize()
        sampled(eng, step, st, args, s)
        torch.cuda.synchronize()
        want.append(results_of(st))
    assert want[0][0].sum() > 0 and want[1][0].sum() > 0
    for _ in range(60):
        for (step, st, args, _), s in zip(sides, streams):
            sampled(eng, step, st, args, s)
        torch.cuda.synchronize()
        for (step, st, args, _), w_ in zip(sides, want):
            assert all((a == b).all() for a, b in zip(results_of(st), w_))
    # the sums are the workspace's last region: 16 bytes per row and slice of 4096 tokens
    n = eng.max_rows * ((V + 4095) // 4096) * 16
    end = eng._ws_ptr - eng.workspace.data_ptr() + hs_workspace_bytes_of(eng)
    place = eng.workspace[end - (n + 255) // 256 * 256:end].view(torch.int32)
    for _ in range(10):
        with torch.cuda.stream(streams[1]):
            for _ in range(40):
                place.random_()
        sampled(eng, *sides[0][:3], streams[0])
        torch.cuda.synchronize()
        assert all((a == b).all() for a, b in zip(results_of(sides[0][1]), want[0]))
    eng.close()


def hs_workspace_bytes_of(eng):
    from paper_2508_18588_amd import hs_workspace_bytes
    return hs_workspace_bytes(eng.ctx)


@pytest.mark.parametrize("V,B,k,two,drafting", [
    (16401, 70, 31, True, 70), (16404, 70, 31, True, 70),       # rows that are not, and that are 16-byte aligned
    (16400, 1000, 4, False, 1000),                              # chains
    (16400, 1000, 4, False, 100),                               # so few live rows that the first stage sums them all
])
def test_sums_in_stages_equal_the_oracle_and_the_sums_of_all_rows(toy, V, B, k, two, drafting):
    """Many rows (here by the hint) are summed in stages, each for the nodes that the walks have reached: trees of
    every depth from none to k, on which the walks end at every level.  The decisions are the oracle's (unless its
    margin is below 1e-9) and those of one launch for all rows (which a hint of few rows asks for), also in a captured graph
    replayed with other logits, and while another stream overwrites sums and states."""
    from paper_2508_18588_amd import HS_ACCEPT_REJECTION
    from paper_2508_18588_amd.runtime import Engine
    from hs_inputs import ModelShape
    shape = ModelShape(n_layers=1, d_model=64, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=V)
    rng = np.random.default_rng(V)
    eng = Engine(shape, make_weights(shape, 3), rope_table(64, 64), max_batch=B, k_max=k, c_max=2 if two else 1, max_len=80)
    # the host's rule: from 200 MB of logits by the hint, no more than the limits allow; the first stage sums all of up to 100 MB
    many = B * (1 + eng.c_max * k)
    assert many * V * 4e-6 >= 200 > V * 4e-6
    ids = rng.integers(0, 2 ** 62, B)
    eng.load_sequences([np.array([0], np.int32)] * B, budgets=[99] * B, seq_ids=ids.astype(np.int64))
    trees = random_trees(rng, B, k, V, two)
    trees[drafting:] = [oracle.build_tree([np.zeros(0, np.int64)], 1, 50) for _ in range(B - drafting)]
    m = eng.set_rows([dict(tok=t["tok"], parent=t["parent"], pos=t["pos"]) for t in trees])
    assert (m * V * 4e-6 > 100) == (drafting == B)
    at = torch.tensor([(o + int(t["parent"][i])) * V + int(t["tok"][i])
                       for t, o in zip(trees, np.cumsum([0] + [len(t["tok"]) for t in trees])) for i in range(1, len(t["tok"]))],
                      device="cuda:0")
    def logits(seed):
        g = torch.Generator(device="cuda:0").manual_seed(seed)
        eng.logits.copy_(torch.randn(eng.logits.shape, generator=g, device="cuda:0"))
        eng.logits.view(-1)[at] = np.log(V) + 3.0 + torch.randn(len(at), generator=g, device="cuda:0")
    def accept(hint):
        eng.set_rows_hint(hint)
        eng.accept(HS_ACCEPT_REJECTION, 1.0, 1234)
    logits(1)
    accept(many)
    torch.cuda.synchronize()
    want, lg, st, r, depths = results_of(eng.st), np_of(eng.logits[:m]), {n: np_of(v) for n, v in eng.st.items()}, 0, set()
    for b, t in enumerate(trees):
        n = len(t["tok"])
        a, out, path, margin = oracle.accept_stochastic(t["tok"], t["parent"], t["pos"], lg[r:r + n].astype(np.float64), 1.0, 1234, int(ids[b]))
        g = st["n_out"][b]
        got = (int(st["accept_len"][b]), st["out_tok"][b, :g].tolist(), st["path_row"][b, :g].tolist())
        assert got == (a, out.tolist(), path.tolist()) or margin < 1e-9, (b, got, a, out, path, margin)
        depths.add(a)
        r += n
    assert depths >= set(range(min(k, 10)))
    accept(1)
    torch.cuda.synchronize()
    live = lambda res: [(int(n), o[:n].tolist(), q[:n].tolist()) for n, o, q in zip(res[1], res[2], res[3])]
    assert live(results_of(eng.st)) == live(want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        accept(many)
    for seed in (2, 3, 1):
        logits(seed)
        accept(1)
        torch.cuda.synchronize()
        eager = live(results_of(eng.st))
        eng.st["out_tok"].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert live(results_of(eng.st)) == eager
    side = torch.cuda.Stream()
    end = eng._ws_ptr - eng.workspace.data_ptr() + hs_workspace_bytes_of(eng)
    slices = (V + 4095) // 4096
    place = eng.workspace[end - eng.max_rows * slices * 16 - 32 * B - 512 & ~3:end & ~3].view(torch.int32)
    for _ in range(10):
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(40):
                place.random_()
        accept(many)
        torch.cuda.synchronize()
        assert live(results_of(eng.st)) == live(want)
    eng.close()


def test_a_replayed_call_in_stages_while_its_plans_are_overwritten(toy):
    """A call replayed from a graph finds the sums of its earlier replays in the workspace, and their check words are its own.
    Whatever another call overwrites between two workgroups' reads of a plan (here a second stream that keeps rewriting all
    plans), a stage must not leave out a node of it: the walk would take the earlier replay's sum for it.  Two sets of logits
    in turn, so that what is left over is wrong."""
    from paper_2508_18588_amd import HS_ACCEPT_REJECTION
    from paper_2508_18588_amd.runtime import Engine
    from hs_inputs import ModelShape
    V, B, k = 65540, 64, 8
    shape = ModelShape(n_layers=1, d_model=64, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=V)
    rng = np.random.default_rng(12)
    eng = Engine(shape, make_weights(shape, 3), rope_table(64, 64), max_batch=B, k_max=k, c_max=2, max_len=80)
    eng.load_sequences([np.array([0], np.int32)] * B, budgets=[99] * B, seq_ids=rng.integers(0, 2 ** 62, B).astype(np.int64))
    trees = [oracle.build_tree([rng.integers(0, V, k), rng.integers(0, V, k)], 0, 50) for _ in range(B)]
    m = eng.set_rows([dict(tok=t["tok"], parent=t["parent"], pos=t["pos"]) for t in trees])
    at = torch.tensor([(o + int(t["parent"][i])) * V + int(t["tok"][i])
                       for t, o in zip(trees, np.cumsum([0] + [len(t["tok"]) for t in trees])) for i in range(1, len(t["tok"]))],
                      device="cuda:0")
    eng.set_rows_hint(m)
    assert m * V * 4e-6 >= 250            # in stages
    live = lambda res: [(int(n), o[:n].tolist(), q[:n].tolist()) for n, o, q in zip(res[1], res[2], res[3])]
    sets, want = [], []
    for seed in (1, 2):
        g = torch.Generator(device="cuda:0").manual_seed(seed)
        lg = torch.randn(eng.logits.shape, generator=g, device="cuda:0")
        lg.view(-1)[at] = np.log(V) + 2.0 + torch.randn(len(at), generator=g, device="cuda:0")
        eng.logits.copy_(lg)
        eng.accept(HS_ACCEPT_REJECTION, 1.0, 1234)
        torch.cuda.synchronize()
        sets.append(lg)
        want.append(live(results_of(eng.st)))
    assert want[0] != want[1]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        eng.accept(HS_ACCEPT_REJECTION, 1.0, 1234)
    # the plans are 16 bytes per sequence in front of the sums, the workspace's last region
    up = lambda n: (n + 255) // 256 * 256
    end = eng._ws_ptr - eng.workspace.data_ptr() + hs_workspace_bytes_of(eng) - up(eng.max_rows * ((V + 4095) // 4096) * 16)
    plans = eng.workspace[end - up(16 * B):end - up(16 * B) + 16 * B].view(torch.int32)
    noise = torch.randint(-2 ** 31, 2 ** 31, (4 * B,), dtype=torch.int32, device="cuda:0")
    rewrite, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    other = torch.zeros(64, dtype=torch.int32, device="cuda:0")
    with torch.cuda.graph(rewrite):
        for i in range(40):
            torch.add(noise, 7919 * i, out=plans)
            for _ in range(1 + i * 5 % 11):     # (a while without: a stage reads some of its plans before, some after)
                other.add_(1)
    wrong = []
    for trial in range(60):
        eng.logits.copy_(sets[trial % 2])
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            rewrite.replay()
        graph.replay()
        torch.cuda.synchronize()
        got = live(results_of(eng.st))
        wrong += [(trial, b) for b in range(B) if got[b] != want[trial % 2][b]]
    eng.close()
    assert not wrong, (len(wrong), wrong[:10])


def test_few_live_rows_without_a_hint_are_summed_at_once(toy):
    """A context whose limits allow 660 MB of logits, with one row per sequence: without a hint the call may take at most 1.25
    times what it takes with the right one (as measured the same; 1.5 times with four launches that find nothing to do).  Rows
    that the engine lays out itself are a hint, until the next draft."""
    from paper_2508_18588_amd import HS_ACCEPT_REJECTION
    from paper_2508_18588_amd.runtime import Engine, Policy
    from hs_inputs import ModelShape
    V, B, k = 152064, 64, 8
    shape = ModelShape(n_layers=1, d_model=64, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=V)
    eng = Engine(shape, make_weights(shape, 3), rope_table(64, 64), max_batch=B, k_max=k, c_max=2, max_len=80)
    eng.load_sequences([np.array([5, 6, 7], np.int32)] * B, budgets=[99] * B)
    none = np.zeros(0, np.int32)
    eng.set_history([[none, none]] * B)
    assert eng.c_step.rows_hint == 0
    m = eng.set_rows([dict(tok=[7], parent=[-1], pos=[2])] * B)
    assert m == B and eng.c_step.rows_hint == B
    eng.logits.normal_(generator=torch.Generator(device="cuda:0").manual_seed(2))

    def us():
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                eng.accept(HS_ACCEPT_REJECTION, 1.0, 3)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 50)
        return sorted(times[1:])[2], results_of(eng.st)
    right, want = us()
    eng.draft(Policy(window=4, m_min=2, k_fixed=8, k_max=8))
    assert eng.c_step.rows_hint == 0 and int(eng.st["row_off"][B]) == B
    without, got = us()
    assert all((a == b).all() for a, b in zip(got, want))
    eng.set_rows_hint(40)
    eng.set_rows([dict(tok=[7], parent=[-1], pos=[2])] * B)
    eng.draft(Policy(window=4, m_min=2, k_fixed=8, k_max=8))
    assert eng.c_step.rows_hint == 40                # the caller's own stays
    eng.close()
    print("with and without a hint, us:", right, without)
    assert without <= 1.25 * right, (right, without)
