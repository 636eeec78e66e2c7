"""bf16 projections across the tile shapes the row count selects, and attention at
the edges of its key and query tiles.

Every shape adds an element's products in the same order, so a user's logits are
bitwise the same however many other users are forwarded with it: the batch sizes
take the projections through their small, four-wave and eight-wave tiles, with row
counts at, below and past tile edges.  One user's logits are also held to the fp64
oracle (the 2e-2 bar of bf16 logits), over prefixes one key below, at and past a
64-key tile."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from _gpu_common import LOGIT_TOL, tokens_of, upload_tree  # noqa: E402
from oracle.model import Decoder  # noqa: E402
from synth import ModelDims, get_workload, make_catalog, make_weights  # noqa: E402

# d_model, heads, d_ffn (the last an odd multiple of 128: the down projection unsplit), prefix tokens, batch sizes
CASES = {
    "d256_dh64_p63": (256, 4, 1024, 63, (2, 5, 16, 41)),
    "d768_dh128_p64": (768, 6, 3072, 64, (2, 3, 10, 30)),
    "d1024_dh64_p65": (1024, 16, 2816, 65, (2, 3, 4, 6, 12, 20, 31)),
    "d1280_dh128_p66": (1280, 10, 3200, 66, (2, 7, 18)),     # norm of a workgroup a row, the others a wave a row
    "d1024_dh128_p129": (1024, 8, 1408, 129, (2, 9, 25)),
    # the shapes that only these widths and row counts take: the largest four-wave tiles of every projection
    "d768_dh64_p64": (768, 12, 3072, 64, (21, 40)),
    "d2048_dh128_p61": (2048, 16, 5504, 61, (6, 7, 9, 16, 22, 34, 51)),
    "d4096_dh128_p61": (4096, 32, 4096, 61, (2, 3, 6, 9, 13)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_logits_do_not_depend_on_the_shape(name):
    from paper_2410_05165_amd.binding import Engine
    d, heads, ffn, P, batches = CASES[name]
    B = max(batches)
    dims = ModelDims(1, d, heads, ffn, 2048, 1024)
    w = get_workload("small").with_(name=name, target=dims, draft=ModelDims(0, 0, 0, 0, 0, 0), n_items=3000, batch=B,
                                    hist_items=1, prompt_len=P - 4, K=10, N=20)
    cat = make_catalog(w)
    rng = np.random.default_rng(11)
    pre = rng.integers(0, 2048, size=(B, P)).astype(np.int32)   # no shared prompt
    tw = make_weights(w, "target")
    eng = Engine(w, tw, None, cat, max_batch=B, max_prefix=P)
    trees = [[tuple(int(c) for c in cat[i]) for i in rng.permutation(len(cat))[:17]] for _ in range(B)]

    def run(n):
        root = torch.full((n, w.n_item_tokens), float("nan"), dtype=torch.float32, device="cuda:0")
        eng.atspeed_prefill(torch.from_numpy(pre[:n]).cuda(), root)
        nodes = upload_tree(eng, trees[:n], n)
        logits = torch.zeros((n, eng.max_nodes, w.n_item_tokens), dtype=torch.float32, device="cuda:0")
        eng.atspeed_tree_logits(logits)
        return root[0].cpu().numpy(), logits[0].cpu().numpy(), nodes[0]

    root1, tree1, nodes = run(1)
    for n in batches:
        root, tree, _ = run(n)
        assert np.array_equal(root, root1), f"{name}: root logits at {n} users"
        assert np.array_equal(tree, tree1), f"{name}: tree logits at {n} users"
    dec = Decoder(dims, tw, "bf16")
    cache = dec.prefill(pre[0])
    np.testing.assert_allclose(root1, cache.last_logits, rtol=0, atol=LOGIT_TOL["bf16"])
    inner = [i for i, p in enumerate(nodes) if len(p) < w.L]
    want = dec.path_logits(cache, [tokens_of(nodes[i], w) for i in inner])
    np.testing.assert_allclose(tree1[inner], want, rtol=0, atol=LOGIT_TOL["bf16"])
    eng.close()


# users, codebook, shared and whole prefix tokens, K, N, gamma, fewest nodes of the largest tree
PLANS = {
    "one_user_one_node": (1, 37, 20, 20, 1, 1, 1, 1),
    "head_148_shared_63": (18, 37, 63, 70, 10, 20, 4, 60),          # 148 head columns, 18 users: two a wave
    "head_1024_shared_all_but_one": (17, 256, 64, 65, 40, 80, 4, 300),
    "trees_past_512_nodes": (70, 255, 65, 69, 100, 100, 4, 560),
    "trees_past_1024_nodes": (3, 256, 0, 64, 128, 128, 6, 1030),     # walked from global memory
}


@pytest.mark.parametrize("name", list(PLANS))
def test_rows_of_many_users_are_planned_as_one_users(name):
    """Shared-prefix length, row planning and the tree walk over many users: each
    user's logits are bitwise those of the user forwarded alone."""
    from paper_2410_05165_amd.binding import Engine
    B, codebook, shared, P, K, N, gamma, fewest = PLANS[name]
    dims = ModelDims(1, 256, 4, 256, 4 * codebook + 8, 8)
    w = get_workload("small").with_(name=name, target=dims, draft=ModelDims(0, 0, 0, 0, 0, 0), n_items=4000, batch=B,
                                    codebook=codebook, hist_items=1, prompt_len=P - 4, K=K, N=N, gamma=gamma)
    cat = make_catalog(w)
    rng = np.random.default_rng(5)
    pre = rng.integers(0, dims.vocab, size=(B, P)).astype(np.int32)
    pre[:, :shared] = pre[0, :shared]
    eng = Engine(w, make_weights(w, "target"), None, cat, max_batch=B, max_prefix=P)
    trees = []
    for u in range(B):
        budget = eng.max_nodes - (37 * u) % (eng.max_nodes // 2 + 1)   # the first user's tree is the largest
        paths, nodes = [], set()
        for i in rng.permutation(len(cat)):
            item = tuple(int(c) for c in cat[i])
            more = {item[:l] for l in range(1, w.L + 1)} - nodes
            if len(nodes) + len(more) > budget:
                break
            nodes |= more
            paths.append(item)
        if not paths:
            paths = [tuple(int(c) for c in cat[0])[:1]]
        trees.append(paths)

    def run(users):
        n = len(users)
        root = torch.full((n, w.n_item_tokens), float("nan"), dtype=torch.float32, device="cuda:0")
        eng.atspeed_prefill(torch.from_numpy(np.ascontiguousarray(pre[users])).cuda(), root)
        nodes = upload_tree(eng, [trees[u] for u in users], n)
        logits = torch.zeros((n, eng.max_nodes, w.n_item_tokens), dtype=torch.float32, device="cuda:0")
        eng.atspeed_tree_logits(logits)
        return root.cpu().numpy(), logits.cpu().numpy(), nodes

    root, logits, nodes = run(list(range(B)))
    assert len(nodes[0]) >= fewest
    for u in sorted({0, 1, B // 2, B - 1} & set(range(B))):
        r1, l1, _ = run([u])
        assert np.array_equal(root[u], r1[0]), f"{name}: root logits of user {u}"
        assert np.array_equal(logits[u], l1[0]), f"{name}: tree logits of user {u}"
    dec = Decoder(dims, make_weights(w, "target"), "bf16")
    cache = dec.prefill(pre[B - 1])
    np.testing.assert_allclose(root[B - 1], cache.last_logits, rtol=0, atol=LOGIT_TOL["bf16"])
    inner = [i for i, p in enumerate(nodes[B - 1]) if len(p) < w.L][:64]
    want = dec.path_logits(cache, [tokens_of(nodes[B - 1][i], w) for i in inner])
    np.testing.assert_allclose(logits[B - 1][inner], want, rtol=0, atol=LOGIT_TOL["bf16"])
    eng.close()
