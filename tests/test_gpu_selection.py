"""Selection among candidates with equal scores, by the number of candidates a
level has: few enough to be ranked at once, more than that (all of them pass the
score bound, so the radix select cuts them down), and one to either side.

With item heads of zeros every extension scores the same, so a decode returns the
K lexicographically smallest items in order, each with the log-prob 4 log(1/n)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

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
