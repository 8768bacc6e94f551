"""Lazy rounds of exemplar_greedy (large n^2 d): only candidates whose gain of
an earlier round still bounds them above the best score are scored again.
The run must be the one that scores everything: round i picks the lowest
index of the largest exemplar_gain score for its prefix, and f_out is that
score, bit for bit."""
import numpy as np
import pytest

from paper_2101_08763_amd import api, synth
from test_greedy_gpu import run_greedy, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    api.load()
    return torch


def points(kind, n, d, seed):
    if kind == "twice":  # every point twice: exact ties, the lower index first
        X = synth.random_problem(n // 2, d, 1, 1, seed=seed, clusters=12).X
        return np.concatenate([X, X])
    if kind == "unit":
        X = synth.random_problem(n, d, 1, 1, seed=seed, clusters=20).X
        return X / np.linalg.norm(X, axis=1, keepdims=True)
    X = synth.random_problem(n, d, 1, 1, seed=seed, clusters=0 if kind == "iid" else 15).X
    if kind == "heavy":  # norms over five orders of magnitude
        return X * np.exp(1.5 * np.random.default_rng(seed).standard_normal((n, 1)))
    if kind == "far":  # clusters far from the origin: gains small beside f
        return X + 200.0
    return X


@pytest.mark.parametrize("kind,n,d,K", [("mixture", 16_001, 64, 7), ("iid", 16_001, 64, 4), ("iid", 40_000, 8, 4),
                                        ("twice", 16_000, 64, 6), ("unit", 13_003, 100, 5), ("mixture", 9_001, 300, 4),
                                        ("heavy", 16_001, 64, 6), ("far", 16_001, 64, 6)])
@pytest.mark.parametrize("chunked", [False, True])
def test_lazy_rounds_score_as_all(torch_gpu, monkeypatch, kind, n, d, K, chunked):
    torch = torch_gpu
    assert float(n) * n * d >= 1.2e10  # the rule's lazy side
    X = np.ascontiguousarray(points(kind, n, d, 31 + d), dtype=np.float32)
    Vg = torch.from_numpy(X).cuda()
    say(f"  lazy greedy {kind} n={n} d={d} K={K} chunked={chunked}")
    if chunked:
        _, ws = api.exemplar_plan(n, d, n, 1)
        monkeypatch.setenv("EXEMCL_WORKSPACE_LIMIT", str(ws // 2 + 40 * n))
    S, f = run_greedy(torch, Vg, K)
    monkeypatch.delenv("EXEMCL_WORKSPACE_LIMIT", raising=False)
    every = torch.arange(n, dtype=torch.int32, device="cuda")
    for i in range(K):
        sc = api.exemplar_gain(Vg, torch.from_numpy(S[:i].copy()).cuda(), every).cpu().numpy()
        masked = sc.copy()
        masked[S[:i]] = -np.inf
        assert int(np.argmax(masked)) == S[i], f"round {i}"
        assert sc[S[i]] == f[i], f"round {i}: {sc[S[i]]} vs {f[i]}"
