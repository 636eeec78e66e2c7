"""Weights that are views into larger buffers: the embedding and fp32 matrices may start
at any element, and the results are bitwise those of aligned copies."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from _gpu_common import upload_tree  # noqa: E402
from synth import ModelDims, get_workload, make_catalog, make_prefixes, make_weights  # noqa: E402


def _engine(w, tw, cat, names, shift):
    """Engine whose weights named by ``names`` start ``shift`` elements into their buffers."""
    from paper_2410_05165_amd.binding import Engine

    class Views(Engine):
        def _upload(self, W, n_layers):
            self._views = {id(a) for k, a in W.items() if names(k)}
            return super()._upload(W, n_layers)

        def _dev(self, a):
            t = super()._dev(a)
            if id(a) not in self._views:
                return t
            buf = torch.empty(t.numel() + shift, dtype=t.dtype, device=t.device)
            buf[shift:] = t.reshape(-1)
            return buf[shift:].view(t.shape)

    return Views(w, tw, None, cat)


def _logits(eng, w, cat, pre):
    root = torch.full((w.batch, w.n_item_tokens), float("nan"), dtype=torch.float32, device="cuda:0")
    eng.atspeed_prefill(torch.from_numpy(pre).cuda(), root)
    rng = np.random.default_rng(7)
    trees = [[tuple(int(c) for c in cat[i]) for i in rng.permutation(len(cat))[:9]] for _ in range(w.batch)]
    upload_tree(eng, trees, w.batch)
    logits = torch.zeros((w.batch, eng.max_nodes, w.n_item_tokens), dtype=torch.float32, device="cuda:0")
    eng.atspeed_tree_logits(logits)
    out = root.cpu().numpy(), logits.cpu().numpy()
    eng.close()
    return out


def _workload(dtype, d, heads, ffn, codebook=50):
    dims = ModelDims(2, d, heads, ffn, 4 * codebook + 8, 8)
    return get_workload("tiny").with_(name="views", dtype=dtype, target=dims, draft=ModelDims(0, 0, 0, 0, 0, 0),
                                      codebook=codebook, n_items=400, batch=3, hist_items=5, K=16, N=32)


# dtype, d_model (1,280: a workgroup a row in the norms, 256: a wave a row), heads, d_ffn
@pytest.mark.parametrize("shift", [1, 2, 3])
@pytest.mark.parametrize("dtype,d,heads,ffn", [("bf16", 256, 4, 256), ("bf16", 1280, 10, 256), ("fp32", 256, 4, 336),
                                               ("fp32", 1280, 10, 128)])
def test_embedding_at_any_element(dtype, d, heads, ffn, shift):
    w = _workload(dtype, d, heads, ffn)
    cat = make_catalog(w)
    pre = make_prefixes(w, cat)
    tw = make_weights(w, "target")
    want = _logits(_engine(w, tw, cat, lambda k: False, 0), w, cat, pre)
    got = _logits(_engine(w, tw, cat, lambda k: k == "tok_emb", shift), w, cat, pre)
    for a, b in zip(got, want):
        assert np.isfinite(b).all() and np.array_equal(a, b)


# d_model, heads, d_ffn (an odd multiple of 16: the down projection's last k-tile is half filled), codebook
@pytest.mark.parametrize("shift", [1, 2, 3])
@pytest.mark.parametrize("d,heads,ffn,codebook", [(64, 2, 16, 7), (96, 3, 336, 50), (512, 4, 1040, 255)])
def test_fp32_matrices_at_any_element(d, heads, ffn, codebook, shift):
    w = _workload("fp32", d, heads, ffn, codebook)
    cat = make_catalog(w)
    pre = make_prefixes(w, cat)
    tw = make_weights(w, "target")
    want = _logits(_engine(w, tw, cat, lambda k: False, 0), w, cat, pre)
    for names in ("wk", "w_up", "w_down", "lm_head", ""):           # one matrix of a call, and all of them
        got = _logits(_engine(w, tw, cat, lambda k: names in k and "norm" not in k, shift), w, cat, pre)
        for a, b in zip(got, want):
            assert np.isfinite(b).all() and np.array_equal(a, b), names
