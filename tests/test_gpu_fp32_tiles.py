"""fp32 models at the edges of the fp32 kernels' tiles: d_ffn an odd multiple
of 16 (the last k-tile of the down projection is half filled, the last gate/up
column group stands alone), an item head of a width that is no multiple of a
tile, every d_head, row counts below, at and past a tile, and the three tile
sizes; in attention one to three key tiles with and without a ragged last one,
and tree rows over and past one query block, against the fp64 oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from _gpu_common import tokens_of, upload_tree  # noqa: E402
from oracle.model import Decoder  # noqa: E402
from synth import ModelDims, get_workload, make_catalog, make_prefixes, make_weights  # noqa: E402

CASES = {
    # name: (d_model, heads, d_ffn, codebook, users, history items)
    "dh32_half_tail": (96, 3, 16 * 21, 50, 1, 4),          # 16 rows, K 336 = 10.5 k-tiles
    "dh64_one_row_over": (128, 2, 16, 33, 1, 16),          # d_ffn 16: half a k-tile; 64 rows, then trees
    "dh128_ragged_rows": (256, 2, 16 * 5, 255, 3, 11),     # 132 rows, 1,020 head columns
    "mid_tiles": (512, 8, 1408, 256, 9, 17),               # 612 rows: 32x64 and 64x64 tiles
    "large_tiles": (1024, 8, 2816, 256, 12, 33),           # 1,584 rows: 64x64 and 128x64 tiles
    "three_key_tiles": (128, 1, 64, 64, 1, 48),            # 192 keys, d_head 128
}


@pytest.mark.parametrize("name", list(CASES))
def test_fp32_logits(name):
    from paper_2410_05165_amd.binding import Engine
    d, heads, ffn, codebook, users, hist = CASES[name]
    dims = ModelDims(1, d, heads, ffn, 4 * codebook + 8, 8)
    w = get_workload("tiny").with_(name=name, target=dims, draft=ModelDims(0, 0, 0, 0, 0, 0), codebook=codebook,
                                   n_items=400, batch=users, hist_items=hist, prompt_len=0, K=16, N=32)
    cat = make_catalog(w)
    pre = make_prefixes(w, cat)
    tw = make_weights(w, "target")
    eng = Engine(w, tw, None, cat)
    root = torch.full((users, w.n_item_tokens), float("nan"), dtype=torch.float32, device="cuda:0")
    eng.atspeed_prefill(torch.from_numpy(pre).cuda(), root)
    torch.cuda.synchronize()
    got = root.cpu().numpy()
    dec = Decoder(dims, tw, "fp32")
    caches = [dec.prefill(pre[u]) for u in range(users)]
    for u in range(users):
        np.testing.assert_allclose(got[u], caches[u].last_logits, rtol=0, atol=1e-4)
    # a tree of random catalog paths per user, wider for each user after the first
    rng = np.random.default_rng(7)
    trees = [[tuple(int(c) for c in cat[i]) for i in rng.permutation(len(cat))[: 8 * (1 + u % 3)]] for u in range(users)]
    nodes = upload_tree(eng, trees, users)
    logits = torch.full((users, eng.max_nodes, w.n_item_tokens), float("nan"), dtype=torch.float32, device="cuda:0")
    eng.atspeed_tree_logits(logits)
    logits = logits.cpu().numpy()
    for u in range(min(users, 3)):
        inner = [i for i, p in enumerate(nodes[u]) if len(p) < w.L]
        want = dec.path_logits(caches[u], [tokens_of(nodes[u][i], w) for i in inner])
        np.testing.assert_allclose(logits[u][inner], want, rtol=0, atol=1e-4)
    eng.close()


# users of the batches; with one user they take every tile size in each kind of call
BATCHES = {"mid_tiles": (2, 5, 9), "large_tiles": (3, 4, 7, 12)}


@pytest.mark.parametrize("name", list(BATCHES))
def test_rows_do_not_depend_on_their_batch(name):
    """A user's logits are bitwise the same alone and in batches of any tile size."""
    from paper_2410_05165_amd.binding import Engine
    d, heads, ffn, codebook, users, hist = CASES[name]
    dims = ModelDims(1, d, heads, ffn, 4 * codebook + 8, 8)
    w = get_workload("tiny").with_(name=name, target=dims, draft=ModelDims(0, 0, 0, 0, 0, 0), codebook=codebook,
                                   n_items=400, batch=users, hist_items=hist, prompt_len=0, K=16, N=32)
    cat = make_catalog(w)
    pre = make_prefixes(w, cat)
    eng = Engine(w, make_weights(w, "target"), None, cat)
    rng = np.random.default_rng(7)
    trees = [[tuple(int(c) for c in cat[i]) for i in rng.permutation(len(cat))[:17]] for _ in range(users)]

    def run(order):
        n = len(order)
        root = torch.full((n, w.n_item_tokens), float("nan"), dtype=torch.float32, device="cuda:0")
        eng.atspeed_prefill(torch.from_numpy(np.ascontiguousarray(pre[order])).cuda(), root)
        upload_tree(eng, [trees[u] for u in order], n)
        logits = torch.zeros((n, eng.max_nodes, w.n_item_tokens), dtype=torch.float32, device="cuda:0")
        eng.atspeed_tree_logits(logits)
        return root.cpu().numpy(), logits.cpu().numpy()

    root1, tree1 = run([users - 1])
    assert np.isfinite(root1).all()
    for n in BATCHES[name]:
        root, tree = run(list(range(users - n, users)))    # the user's rows are the last ones
        assert np.array_equal(root[-1], root1[0]), f"{name}: root logits among {n} users"
        assert np.array_equal(tree[-1], tree1[0]), f"{name}: tree logits among {n} users"
    eng.close()
