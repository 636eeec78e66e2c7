"""Selection among candidates with equal scores, by the number of candidates a
level has: few enough to be ranked at once, more than that (all of them pass the
score bound, so the radix select cuts them down), and one to either side.

With item heads of zeros every extension scores the same, so a decode returns the
K lexicographically smallest items in order, each with the log-prob 4 log(1/n)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from _gpu_common import logit_table, upload_tree  # noqa: E402
from oracle.search import extend, path_score, table_scorer, top  # noqa: E402
from oracle.trie import Trie  # noqa: E402
from synth import ModelDims, get_workload, make_catalog, make_prefixes, make_weights  # noqa: E402

# codebook, items, K, N, users
CASES = {
    "one_item": (7, 1, 1, 1, 1),
    "all_items": (9, 64, 64, 64, 2),                # every item is returned
    "level_of_255": (255, 4000, 10, 20, 3),
    "level_of_256": (256, 6000, 33, 34, 3),         # then over 256 of the 33 parents
    "many_equal": (64, 20000, 128, 128, 2),         # 64, 4,096 of 64 parents, then 128 parents
}


@pytest.mark.parametrize("name", list(CASES))
def test_ties_take_the_smallest_items(name):
    from paper_2410_05165_amd.binding import Engine
    codebook, items, K, N, users = CASES[name]
    vocab = 4 * codebook + 8
    w = get_workload("tiny").with_(name=name, target=ModelDims(1, 64, 2, 128, vocab, 8),
                                   draft=ModelDims(1, 64, 2, 128, vocab, 8), codebook=codebook, n_items=items, batch=users,
                                   hist_items=2, prompt_len=0, K=K, N=N)
    cat = make_catalog(w)
    pre = make_prefixes(w, cat)
    tw, dw = make_weights(w, "target"), make_weights(w, "draft")
    for m in (tw, dw):
        m["lm_head_item"] = np.zeros_like(m["lm_head_item"])
    eng = Engine(w, tw, dw, cat)
    out = torch.full((users, K, w.L), -1, dtype=torch.int32, device="cuda:0")
    scores = torch.zeros((users, K), dtype=torch.float32, device="cuda:0")
    n = torch.zeros(users, dtype=torch.int32, device="cuda:0")
    eng.atspeed_decode_topk(torch.from_numpy(pre).cuda(), out, scores, n)
    want = sorted({tuple(int(c) for c in row) for row in cat})[:K]
    for u in range(users):
        got = [tuple(r) for r in out[u, : int(n[u])].cpu().tolist()]
        assert got == want, f"{name}: user {u}"
        np.testing.assert_allclose(scores[u, : len(want)].cpu().numpy(), -w.L * np.log(w.n_item_tokens), rtol=1e-5)
    eng.close()


# copies of beam a, copies of beam b, K, N, items, whether every code scores the same
REPEATS = {
    "few_candidates": (2, 1, 10, 12, 2000, False),       # ranked at once
    "many_candidates": (2, 2, 16, 20, 60000, False),     # cut down by the score bound
    "equal_scores": (2, 2, 16, 20, 60000, True),         # cut down by the radix select
    "full_width": (100, 28, 128, 128, 60000, True),      # 128 of 200 keys up to the last one taken
}


def _repeat_case(name):
    na, nb, K, N, items, flat = REPEATS[name]
    w = get_workload("tiny").with_(name=f"repeat_{name}", n_items=items, batch=2, hist_items=4, K=K, N=N)
    cat = make_catalog(w)
    a, b = sorted({int(r[0]) for r in cat})[3:5]
    paths = np.zeros((2, K, w.L), np.int32)
    paths[0, :na, 0], paths[0, na:na + nb, 0] = a, b
    paths[1, 0, 0], paths[1, 1, 0] = b, a                # the second user holds no beam twice
    scores = np.where(paths[:, :, 0] == a, -1.25, -1.5).astype(np.float32)
    if flat:
        scores[:] = -1.25
    state = (np.ones(2, np.int32), np.array([na + nb, 2], np.int32), paths, scores)
    beams = [[((a,), float(scores[0, 0]))] * na + [((b,), float(scores[0, na]))] * nb,
             [((b,), float(scores[1, 0])), ((a,), float(scores[1, 1]))]]
    return w, cat, state, beams, flat


@pytest.mark.parametrize("name", list(REPEATS))
def test_a_beam_given_twice_counts_twice(name):
    """A state that holds a beam more than once gives equal candidates: the strict
    selection and the draft keep each of them, as the oracle's sort does."""
    from paper_2410_05165_amd.binding import Engine
    w, cat, state, beams, flat = _repeat_case(name)
    tw, dw = make_weights(w, "target"), make_weights(w, "draft")
    if flat:
        dw["lm_head_item"] = np.zeros_like(dw["lm_head_item"])
    trie = Trie(cat)
    eng = Engine(w, tw, dw, cat)
    eng.atspeed_prefill(torch.from_numpy(make_prefixes(w, cat)).cuda())
    # drafting, scored by the draft's own log-probs
    eng.atspeed_set_state(*state)
    eng.atspeed_draft()
    lp = torch.zeros((2, eng.max_nodes, w.n_item_tokens), dtype=torch.float32, device="cuda:0")
    root = torch.zeros((2, w.n_item_tokens), dtype=torch.float32, device="cuda:0")
    eng.atspeed_logprobs(1, lp, root)
    n, token, parent, depth, _ = [x.cpu().numpy() for x in eng.tree_tensors(2)]
    for u in range(2):
        codes = token[u] - w.target.item_base - w.codebook * (depth[u] - 1)
        path = []
        for i in range(n[u]):
            path.append((path[parent[u, i]] if parent[u, i] >= 0 else ()) + (int(codes[i]),))
        lq = table_scorer({(): root[u].cpu().numpy(), **{p: lp[u, i].cpu().numpy() for i, p in reversed(list(enumerate(path)))}})
        got = [p for p in path if len(p) == 2]
        want, margin = top(extend([(p, path_score(lq, p, w.codebook)) for p, _ in beams[u]], lq, trie, w.codebook), w.N)
        assert flat or margin > 1e-5, "the draft's own scores leave no tie at the cut"
        assert sorted(got) == sorted(p for p, _ in want), f"{name}: drafted level of user {u}"
        assert all(trie.is_prefix(p) for p in path)
    # strict selection on given logits over the tree of the beams' paths
    eng.atspeed_set_state(*state)
    nodes = upload_tree(eng, [sorted({p for p, _ in beams[u]}) for u in range(2)], 2)
    rng = np.random.default_rng(3)
    logits = np.zeros((2, eng.max_nodes, w.n_item_tokens), np.float32)
    if not flat:
        logits[:] = rng.normal(size=logits.shape)
    zero = np.zeros((2, w.n_item_tokens), np.float32)
    for call in (eng.atspeed_accept, eng.atspeed_accept_noalloc):
        eng.atspeed_set_state(*state)
        call(torch.from_numpy(logits).cuda(), torch.from_numpy(zero).cuda())
        t, nb, paths, scores = eng.atspeed_get_state(2)
        for u in range(2):
            want, _ = top(extend(beams[u], logit_table(nodes[u], logits[u], zero[u]), trie, w.codebook), w.K)
            assert t[u] == 2 and nb[u] == len(want)
            assert [tuple(int(c) for c in paths[u, k, :2]) for k in range(nb[u])] == [p for p, _ in want], f"{name}: user {u}"
            np.testing.assert_allclose(scores[u, : nb[u]], [s for _, s in want], rtol=0, atol=1e-5)
    eng.close()


@pytest.mark.parametrize("name", list(REPEATS))
def test_a_beam_given_twice_in_the_relaxed_modes(name):
    """The same states through sampled drafting and relaxed verification: every
    drafted node and every beam is a prefix of an item, the beams all different."""
    from paper_2410_05165_amd.binding import RELAXED_EXACT, RELAXED_PAPER, Engine
    w, cat, state, beams, flat = _repeat_case(name)
    trie = Trie(cat)
    tw, dw = make_weights(w, "target"), make_weights(w, "draft")
    for mode in (RELAXED_EXACT, RELAXED_PAPER):
        eng = Engine(w, tw, dw, cat, mode=mode, seed=5)
        eng.atspeed_prefill(torch.from_numpy(make_prefixes(w, cat)).cuda())
        eng.atspeed_set_state(*state)
        eng.atspeed_draft()
        n, token, parent, depth, _ = [x.cpu().numpy() for x in eng.tree_tensors(2)]
        for u in range(2):
            path = []
            for i in range(n[u]):
                code = int(token[u, i]) - w.target.item_base - w.codebook * (int(depth[u, i]) - 1)
                path.append((path[parent[u, i]] if parent[u, i] >= 0 else ()) + (code,))
            assert all(trie.is_prefix(p) for p in path), f"{name}: mode {mode}, user {u}"
            if mode == RELAXED_PAPER:
                cands = sum(len(trie.children(p)) for p, _ in beams[u])
                assert sum(len(p) == 2 for p in path) == min(w.N, cands)
        eng.atspeed_verify()
        t, nb, paths, _ = eng.atspeed_get_state(2)
        for u in range(2):
            got = [tuple(int(c) for c in paths[u, k, : t[u]]) for k in range(nb[u])]
            assert t[u] > 1 and got and len(set(got)) == len(got)
            assert all(trie.is_prefix(p) for p in got), f"{name}: mode {mode}, user {u}"
        eng.close()
