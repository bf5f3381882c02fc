"""GPU parity of hs_draft_group (reward-aware draft over all responses of a prompt, Sec. 5.3 of the paper) against
the oracle: matched length, number of drafted tokens, the drafted tokens themselves and the occurrence the draft is
read from must be identical (integer work: bit-exact), on alphabets small enough to force ties, repeated patterns
and more occurrences than the kernel keeps, on group-of-16 responses of realistic length, and end to end (the
greedy stream with group drafts equals the plain autoregressive stream)."""
import numpy as np
import pytest
import torch

import oracle
from hs_inputs import CONFIG_SHAPES, make_weights, rope_table, make_prompts, mutate, history_with_context, config_seed
from gpu_common import np_of

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def toy():
    shape = CONFIG_SHAPES[1]
    return shape, make_weights(shape, seed=1), rope_table(4096, shape.head_dim)


def run_group_draft(eng, xs, groups, rewards, pol, budgets=None, k_state=None):
    B = len(xs)
    eng.load_sequences(xs, budgets=budgets or [64] * B)
    if k_state is not None:
        eng.k_state[:B].copy_(torch.tensor(k_state, dtype=torch.int32))
    eng.set_group_history(groups, rewards)
    eng.draft_group(pol)
    torch.cuda.synchronize()
    assert eng.poll_error() == 0
    return {k: np_of(v) for k, v in eng.st.items()}


def check_against_oracle(st, xs, groups, rewards, pol, k_req, occ_max=1024):
    ro = st["row_off"]
    for b, x in enumerate(xs):
        want = oracle.reward_draft(groups[b], rewards[b], x, pol.window, pol.m_min, k_req[b], occ_max)
        n = len(want["tok"])
        got = (int(st["match_len"][b]), int(st["draft_len"][b]))
        assert got == (want["m"], n), (b, got, want)
        assert ro[b + 1] - ro[b] == 1 + n
        assert st["tok"][ro[b] + 1:ro[b + 1]].tolist() == want["tok"].tolist(), (b, want)
        assert st["tok"][ro[b]] == x[-1]
        if want["m"] > 0:
            assert (int(st["draft_src"][b]), int(st["draft_start"][b])) == (want["g"], want["p"]), (b, want)
        else:
            assert st["draft_src"][b] == -1 and st["draft_start"][b] == -1
        assert st["parent"][ro[b]:ro[b + 1]].tolist() == list(range(-1, n))


@pytest.mark.parametrize("vocab,G,lh", [(2, 4, 60), (3, 16, 200), (5, 7, 900), (2, 3, 5000), (40, 16, 4100)])
def test_group_draft_matches_oracle_small_alphabets(toy, vocab, G, lh):
    from paper_2508_18588_amd import HS_K_FIXED
    from paper_2508_18588_amd.runtime import Engine, Policy
    shape, w, rope = toy
    B = 24
    rng = np.random.default_rng(vocab * 1000 + G)
    eng = Engine(shape, w, rope, max_batch=B, k_max=16, c_max=1, max_len=2000, g_max=16)
    for trial in range(3):
        win, m_min, k = int(rng.integers(3, 9)), int(rng.integers(1, 4)), int(rng.integers(1, 17))
        pol = Policy(window=win, m_min=min(m_min, win), k_mode=HS_K_FIXED, k_fixed=k, k_max=16)
        xs = [rng.integers(0, vocab, int(rng.integers(1, 40))).astype(np.int32) for _ in range(B)]
        groups = [[rng.integers(0, vocab, int(rng.integers(0, lh + 1))).astype(np.int32) for _ in range(G)]
                  for _ in range(B)]
        rewards = [rng.integers(0, 4, G).astype(np.int32) for _ in range(B)]
        budgets = [int(rng.integers(0, 12)) for _ in range(B)]     # some finished, some short of budget
        st = run_group_draft(eng, xs, groups, rewards, pol, budgets=budgets)
        k_req = [max(0, min(k, budgets[b] - 1)) if budgets[b] > 0 else 0 for b in range(B)]
        for b in range(B):
            if budgets[b] <= 0:
                assert st["row_off"][b + 1] == st["row_off"][b] and st["draft_len"][b] == 0
        live = [b for b in range(B) if budgets[b] > 0]
        sub = lambda a: [a[b] for b in live]
        # compare the live sequences (row offsets are relative: rebuild a compact view)
        ro = st["row_off"]
        for b in live:
            want = oracle.reward_draft(groups[b], rewards[b], xs[b], pol.window, pol.m_min, k_req[b], 1024)
            n = len(want["tok"])
            assert (int(st["match_len"][b]), int(st["draft_len"][b])) == (want["m"], n), (trial, b, want)
            assert st["tok"][ro[b] + 1:ro[b + 1]].tolist() == want["tok"].tolist(), (trial, b, want)
            if want["m"] > 0:
                assert (int(st["draft_src"][b]), int(st["draft_start"][b])) == (want["g"], want["p"]), (trial, b, want)
    eng.close()


def test_group_of_16_realistic_lengths_and_policies(toy):
    """16 responses of ~4k tokens per prompt, each a differently mutated copy of one text, binary rewards; the
    committed tokens follow that text; AIMD and match-length draft lengths."""
    from paper_2508_18588_amd import HS_K_AIMD, HS_K_MATCHLEN
    from paper_2508_18588_amd.runtime import Engine, Policy
    shape, w, rope = toy
    B, G, V = 16, 16, 150000
    rng = np.random.default_rng(77)
    eng = Engine(shape, w, rope, max_batch=B, k_max=32, c_max=1, max_len=6000, g_max=16, w_max=32)
    for mode in (HS_K_AIMD, HS_K_MATCHLEN):
        pol = Policy(window=7, m_min=3, k_mode=mode, k_max=32)
        xs, groups, rewards, kst = [], [], [], []
        for b in range(B):
            text = rng.integers(0, V, 4096).astype(np.int32)
            prompt = rng.integers(0, V, 40).astype(np.int32)
            cut = int(rng.integers(0, 4000))
            xs.append(np.concatenate([prompt, text[:cut]]).astype(np.int32))
            groups.append([history_with_context(prompt, mutate(text, 0.1 + 0.02 * g, 0.03, V, rng), 7)
                           for g in range(G)])
            rewards.append(rng.integers(0, 2, G).astype(np.int32))
            kst.append(int(2 + 2 * rng.integers(0, 16)))
        st = run_group_draft(eng, xs, groups, rewards, pol, budgets=[4096] * B, k_state=kst)
        k_req = []
        for b in range(B):
            m = oracle.reward_draft(groups[b], rewards[b], xs[b], 7, 3, 0)["m"]
            k_req.append(min(32, kst[b] if mode == HS_K_AIMD else max(m, 1)))
        check_against_oracle(st, xs, groups, rewards, pol, k_req)
        assert sum(int(x) for x in st["draft_len"][:B]) > B      # drafts do happen
    eng.close()


def test_group_draft_end_to_end_equals_autoregressive_greedy(toy):
    """Whole iterations with hs_draft_group: the emitted greedy stream equals the plain autoregressive stream of
    the same kernels token for token, and every step's draft equals the oracle's on the same state."""
    from paper_2508_18588_amd import HS_K_AIMD
    from paper_2508_18588_amd.runtime import Engine, Policy
    from test_gpu_decode import gpu_ar_rollout
    shape = CONFIG_SHAPES[1]
    seed = config_seed(1) + 50
    w = make_weights(shape, seed)
    rope = rope_table(512, shape.head_dim)
    B, G, T = 4, 6, 96
    prompts = make_prompts(B, 48, shape.vocab, seed)
    rolls = gpu_ar_rollout(shape, w, rope, list(prompts), T)
    rng = np.random.default_rng(seed)
    groups = [[history_with_context(prompts[b], mutate(np.asarray(rolls[b], np.int32), 0.08 * (g + 1), 0.0,
                                                        shape.vocab, rng), 7) for g in range(G)] for b in range(B)]
    rewards = [rng.integers(0, 2, G).astype(np.int32) for _ in range(B)]
    pol = Policy(window=7, m_min=3, k_mode=HS_K_AIMD, k_max=16)
    eng = Engine(shape, w, rope, max_batch=B, k_max=16, c_max=1, max_len=48 + T, g_max=8, shuffle_pages_seed=5)
    eng.load_sequences(list(prompts), budgets=[T] * B)
    eng.set_group_history(groups, rewards)
    eng.prefill(list(prompts))
    x = [list(map(int, p)) for p in prompts]
    budget, kst = [T] * B, [2] * B
    accepted = steps = 0
    while any(bd > 0 for bd in budget) and steps < 200:
        eng.step_group(pol)
        torch.cuda.synchronize()
        assert eng.poll_error() == 0
        st = {k: np_of(v) for k, v in eng.st.items()}
        ro = st["row_off"]
        for b in range(B):
            if budget[b] <= 0:
                assert st["n_out"][b] == 0
                continue
            k_req = max(0, min(kst[b], 16, budget[b] - 1))
            want = oracle.reward_draft(groups[b], rewards[b], np.asarray(x[b], np.int32), 7, 3, k_req)
            n = len(want["tok"])
            assert st["tok"][ro[b] + 1:ro[b + 1]].tolist() == want["tok"].tolist()
            a, n_out = int(st["accept_len"][b]), int(st["n_out"][b])
            kst[b] = oracle.aimd(kst[b], n > 0, n > 0 and a == n)
            x[b].extend(int(t) for t in st["out_tok"][b, :n_out])
            budget[b] -= n_out
            accepted += a
        assert np_of(eng.k_state)[:B].tolist() == kst
        steps += 1
    for b in range(B):
        assert x[b][48:48 + T] == list(map(int, rolls[b]))
    eng.close()
    print("group draft end to end: steps", steps, "accepted", accepted)
    assert accepted > 40


@pytest.mark.parametrize("B,G", [(128, 16), (64, 16), (3, 16)])
def test_group_draft_with_segments_in_turn(toy, B, G):
    """A workgroup of the scan takes one, two or all of a history's segments of 4096 tokens, by the number of histories:
    lengths around the segments' edges, at every alignment of a history's first and last token, a planted match of every
    length up to the window on either side of an edge."""
    from paper_2508_18588_amd import HS_K_FIXED
    from paper_2508_18588_amd.runtime import Engine, Policy
    shape, w, _ = toy
    rng = np.random.default_rng(1000 * B + G)
    eng = Engine(shape, w, rope_table(16384, shape.head_dim), max_batch=B, k_max=16, c_max=1, max_len=10000, g_max=16)
    pol = Policy(window=16, m_min=2, k_mode=HS_K_FIXED, k_fixed=8, k_max=16)
    xs, groups = [], []
    for b in range(B):
        xs.append(rng.integers(0, 300, 20).astype(np.int32))
        responses = []
        for g in range(G):
            edge = 4096 * int(rng.integers(0, 3))
            n = max(0, edge + int(rng.integers(-5, 24)))
            h = rng.integers(0, 300, n).astype(np.int32)
            m = int(rng.integers(1, 17))
            at = min(n, max(0, 4096 * int(rng.integers(0, 3)) + int(rng.integers(-18, 3)))) - m
            if at >= 0:
                h[at:at + m] = xs[b][-m:]
            responses.append(h)
        groups.append(responses)
    rewards = [rng.integers(0, 4, G).astype(np.int32) for _ in range(B)]
    st = run_group_draft(eng, xs, groups, rewards, pol)
    check_against_oracle(st, xs, groups, rewards, pol, [8] * B)
    assert (st["draft_len"][:B] > 0).any()
    assert B < 64 or len(set(st["draft_start"][:B] // 4096)) == 3        # chosen in each of the segments
    eng.close()


@pytest.mark.parametrize("n_occ", [1, 3, 64, 65, 200])
def test_negative_ids_in_a_response_end_a_walk_alike_for_few_and_many_occurrences(toy, n_occ):
    """A response may hold ids that are no tokens.  They never vote; an occurrence whose next id is -1 drops out, one with
    another negative id next stays live until somebody else votes -- whether the occurrences are walked by one wavefront
    (up to 64) or by the workgroup.  The rule written out in plain Python."""
    from paper_2508_18588_amd import HS_K_FIXED
    from paper_2508_18588_amd.runtime import Engine, Policy
    shape, w, _ = toy
    B, G, k = 24, 4, 6
    rng = np.random.default_rng(n_occ)
    eng = Engine(shape, w, rope_table(16384, shape.head_dim), max_batch=B, k_max=8, c_max=1, max_len=64, g_max=G)
    xs, groups, occs, rewards = [], [], [], []
    for b in range(B):
        x = np.array([100, 101, 102, 103], np.int32)
        resp, occ = [[] for _ in range(G)], []
        for g in np.sort(rng.integers(0, G, n_occ)):
            text = rng.choice([7, 8, -1, -1, -9], 7, p=[0.4, 0.2, 0.2, 0.1, 0.1])
            resp[g] += [50 + len(resp[g]) % 3] + x.tolist()
            occ.append((int(g), len(resp[g])))
            resp[g] += text.tolist()
        xs.append(x)
        groups.append([np.asarray(r + [60], np.int32) for r in resp])
        occs.append(occ)
        rewards.append(rng.integers(0, 3, G).astype(np.int32))
    pol = Policy(window=4, m_min=3, k_mode=HS_K_FIXED, k_fixed=k, k_max=8)
    st = run_group_draft(eng, xs, groups, rewards, pol)
    eng.close()
    ended = 0
    for b in range(B):
        live, draft = {i: True for i in range(n_occ)}, []
        for j in range(k):
            nxt = {}
            for i in [i for i in live if live[i]]:
                g, p = occs[b][i]
                nxt[i] = int(groups[b][g][p + j]) if p + j < len(groups[b][g]) else -2
                live[i] = nxt[i] != -1
            votes = {}
            for i, t in nxt.items():
                if t >= 0:
                    s, v = votes.get(t, (0, 0))
                    votes[t] = (s + int(rewards[b][occs[b][i][0]]), v + 1)
            if not votes:
                break
            best = min(votes, key=lambda t: (-votes[t][0], -votes[t][1], t))
            for i, t in nxt.items():
                live[i] = live[i] and t == best
            draft.append(best)
        left = [i for i in live if live[i]] if draft else [0]
        r0, r1 = st["row_off"][b], st["row_off"][b + 1]
        if left:
            want = (4, len(draft), *occs[b][left[0]], draft)
        else:
            want = (0, 0, -1, -1, [])
            ended += 1
        got = (int(st["match_len"][b]), int(st["draft_len"][b]), int(st["draft_src"][b]), int(st["draft_start"][b]),
               st["tok"][r0 + 1:r1].tolist())
        assert got == want, (b, got, want)
    assert ended > 0 or n_occ > 3
