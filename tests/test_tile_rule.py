"""The row counts of the GPU tests that compare a user's logits alone and in a batch
reach every tile shape that the projections' rules can pick, and the bf16 rule's
picks are near the fastest shapes measured: the rules' own source text, compiled for
the host, is asked which shape a call takes."""
import os
import re
import subprocess

import numpy as np
import pytest

pytest.importorskip("torch")

import test_gpu_fp32_tiles as fp32  # noqa: E402
import test_gpu_tile_shapes as bf16  # noqa: E402
from synth import ModelDims, get_workload, make_catalog  # noqa: E402

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_05165_amd", "csrc")

BF16_HOST = """
#include <algorithm>
#include <cstdio>
typedef int hipError_t;
typedef int hipStream_t;
struct GemmCall {};
enum { EPI_STORE, EPI_RESID, EPI_GU, EPI_QKV };
enum { BMAP_PLAIN, BMAP_QKV, BMAP_GU };
template <int BMAP, int EPI, int WM, int WN, int TM, int TN, int NS = 2>
hipError_t launch_bf16(const GemmCall&, hipStream_t) { return 0; }
%s
int main() {
  char kind;
  int M, N, K, kparts;
  while (scanf(" %%c %%d %%d %%d %%d", &kind, &M, &N, &K, &kparts) == 5)
    printf("%%d\\n", (int)(kind == 'q' ? &pick_shape(kQkvShapes, M, N, K, kparts) - kQkvShapes
                       : kind == 'g' ? &pick_shape(kGuShapes, M, N, K, kparts) - kGuShapes
                       : kind == 'r' ? &pick_shape(kResidShapes, M, N, K, kparts) - kResidShapes
                                     : &pick_shape(kHeadShapes, M, N, K, kparts) - kHeadShapes));
}
"""

FP32_HOST = """
#include <algorithm>
#include <cstdio>
struct Call { int Mmax, N; };
template <int WM, int WN, int TM, int TP, int NS>
int launch_f32(const Call&, int, int) { return WM * TM * 16 * 1000 + WN * TP * 32; }
int pick(const Call& g) {
  const int a = 0, st = 0;
  %s
}
int main() {
  char kind;
  Call g;
  int K, kparts;
  while (scanf(" %%c %%d %%d %%d %%d", &kind, &g.Mmax, &g.N, &K, &kparts) == 5) printf("%%d\\n", pick(g));
}
"""


def _between(name, start, end):
    src = open(os.path.join(CSRC, name)).read()
    a = src.index(start)
    return src[a:src.index(end, a)]


def _indices(tmp_path, source, calls):
    """What the rule in ``source`` answers to each call (kind, M, N, K, parts of k)."""
    (tmp_path / "rule.cpp").write_text(source)
    exe = str(tmp_path / "rule")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-o", exe, str(tmp_path / "rule.cpp")], check=True)
    text = "\n".join("%s %d %d %d %d" % c for c in calls)
    out = subprocess.run([exe], input=text, text=True, capture_output=True, check=True).stdout.split()
    assert len(out) == len(calls)
    return [int(i) for i in out]


def _picks(tmp_path, source, calls):
    return {(c[0], i) for c, i in zip(calls, _indices(tmp_path, source, calls))}


def _block(M, d, ffn, split):
    """q/k/v, gate/up, o and down of a forward of M rows (the last two split in k where the runtime splits them)."""
    return [("q", M, 3 * d, d, 1), ("g", M, 2 * ffn, d, 1), ("r", M, d, d, 2 if split and d % 256 == 0 else 1),
            ("r", M, d, ffn, 2 if split and ffn % 256 == 0 else 1)]


def test_bf16_batches_reach_every_tile_shape(tmp_path):
    rule = _between("gemm.hip", "namespace {\nconstexpr int kCUs", "hipError_t gemm(const GemmCall& g")
    calls = []
    for d, _, ffn, P, batches in bf16.CASES.values():
        B = max(batches)
        w = get_workload("small").with_(target=ModelDims(1, d, 1, ffn, 2048, 1024), n_items=3000, batch=B, hist_items=1,
                                        prompt_len=P - 4)
        cat = make_catalog(w)
        rng = np.random.default_rng(11)
        rng.integers(0, 2048, size=(B, P))       # the prefixes come first
        trees = [[tuple(int(c) for c in cat[i]) for i in rng.permutation(len(cat))[:17]] for _ in range(B)]
        nodes = [len({p[:l] for p in t for l in range(1, w.L)}) for t in trees]
        for n in (1, *batches):
            calls += _block(n * P, d, ffn, True) + [("h", n, w.n_item_tokens, d, 1)]
            calls += _block(sum(nodes[:n]), d, ffn, True) + [("h", sum(nodes[:n]), w.n_item_tokens, d, 1)]
    got = _picks(tmp_path, BF16_HOST % rule, calls)
    for kind, table in (("q", "kQkvShapes"), ("g", "kGuShapes"), ("r", "kResidShapes"), ("h", "kHeadShapes")):
        rows = len(re.findall(r"launch_bf16<", _between("gemm.hip", f"const Shape {table}[]", "};")))
        assert rows > 0 and {i for k, i in got if k == kind} == set(range(rows)), table


def test_fp32_batches_reach_every_tile(tmp_path):
    rule = _between("gemm_f32.hip", "  const long M = std::max(1, g.Mmax);", "}\n\n}  // namespace atspeed")
    tiles = {128064, 64064, 32064}
    calls = []
    for name, batches in fp32.BATCHES.items():
        d, _, ffn, _, _, hist = fp32.CASES[name]
        for n in (1, *batches):
            calls += _block(4 * hist * n, d, ffn, False)
    got = _picks(tmp_path, FP32_HOST % rule, calls)
    assert got == {(kind, t) for kind in "qgr" for t in tiles}


def test_picks_are_near_the_fastest_measured_shape(tmp_path):
    """The rule against the tracked measurements of the shapes: what its picks take
    over the fastest measured shape, on average over the calls of a table."""
    measured, head = {}, None
    for line in open(os.path.join(os.path.dirname(os.path.dirname(CSRC)), "profiles", "gemm_shapes.csv")):
        cells = line.strip().split(";")
        if line.startswith("#"):
            continue
        if cells[0] == "projection":
            head = cells[4:]
        else:
            times = {s: float(t) for s, t in zip(head, cells[4:]) if float(t) > 0}
            measured[(cells[0], *map(int, cells[1:4]))] = times
    rule = _between("gemm.hip", "namespace {\nconstexpr int kCUs", "hipError_t gemm(const GemmCall& g")
    tables = {"qkv": ("q", "kQkvShapes"), "gu": ("g", "kGuShapes"), "o": ("r", "kResidShapes"), "down": ("r", "kResidShapes"),
              "head": ("h", "kHeadShapes")}
    calls, keys = [], []
    for key in measured:
        name, d, ffn, M = key
        k = ffn if name == "down" else d
        n = {"qkv": 3 * d, "gu": 2 * ffn, "head": 1024}.get(name, d)
        calls.append((tables[name][0], M, n, k, 2 if name in ("o", "down") and k % 256 == 0 else 1))
        keys.append(key)
    index = _indices(tmp_path, BF16_HOST % rule, calls)
    over = {}
    for key, i in zip(keys, index):
        kind, table = tables[key[0]]
        rows = re.findall(r"launch_bf16<\w+, \w+, ([\d, ]+)>", _between("gemm.hip", f"const Shape {table}[]", "};"))
        shape = rows[i].replace(" ", "")
        over.setdefault(kind, []).append(np.log(measured[key][shape] / min(measured[key].values())))
    mean = {kind: float(np.mean(v)) for kind, v in over.items()}
    print(mean)
    assert mean["q"] < 0.005 and mean["g"] < 0.005 and mean["r"] < 0.025 and mean["h"] < 0.015, mean
