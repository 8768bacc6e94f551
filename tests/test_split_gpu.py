"""fp32 on the bf16 matrix cores (three bf16 parts, six products): every tail
length and number of whole blocks, the changes of row tiles with n, tiles
staged in LDS instead of memory, and the error against 64 bits.

h_s(v) sums d products whose three-part split drops at most 2^-24 of
|v_i||s_i| and is accumulated in fp32, so |f - f64| <= (2 d + 64) 2^-24 (mean of
|v||s| + |s|^2) is a generous bound; EXACT_RTOL (1e-5) is above the errors at
the d tested here and is what the other fp32 tests use.
"""
import numpy as np
import pytest

from paper_2101_08763_amd import api, synth
from test_parity_gpu import check, exact, gpu_eval, say, to_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    api.load()
    return torch


@pytest.fixture(scope="module")
def orc():
    import oracle
    return oracle.load()


@pytest.fixture(autouse=True)
def _plain_env(monkeypatch):
    for v in ("EXEMCL_PATH", "EXEMCL_WG_TARGET", "EXEMCL_PERSIST", "EXEMCL_WORKSPACE_LIMIT"):
        monkeypatch.delenv(v, raising=False)


# every tail of 1 .. 32 coordinates, alone and after 1, 2 and more whole blocks
TAILS = list(range(1, 33)) + [33, 36, 41, 44, 48, 52, 53, 56, 57, 61, 63, 65, 72, 81, 85, 92, 104, 109, 116, 121, 129,
                              140, 148, 157, 165, 170, 180, 185, 193, 196, 197, 209, 224, 230, 257, 301, 333, 352, 400, 447, 449, 480, 496, 500, 512]


@pytest.mark.parametrize("d", TAILS)
def test_every_tail(torch_gpu, orc, d):
    """Odd and even k (lone and paired members), sets past the last group of
    32, rows past the last row tile; scoring of S u {c} on the same rows."""
    n, l = 517, 35
    for k in (1, 4, 5):
        p = synth.random_problem(n, d, l, k, seed=9000 + 10 * d + k, clusters=3)
        say(f"split tail: n={n} d={d} l={l} k={k}")
        Vg, X64 = to_gpu(torch_gpu, p.X, "fp32")
        got = gpu_eval(torch_gpu, Vg, p.sets)
        exact(got, orc.eval(X64, p.sets, 4), f"d={d} k={k}")
    S, C = p.sets[0].copy(), np.arange(0, n, 9, dtype=np.int32)
    g = api.exemplar_gain(Vg, torch_gpu.from_numpy(S).cuda(), torch_gpu.from_numpy(C).cuda())
    torch_gpu.cuda.synchronize()
    exact(g.cpu().numpy(), orc.gain(X64, S, C, 4), f"gain d={d}")


@pytest.mark.parametrize("d", [3, 20, 32, 100, 170])
@pytest.mark.parametrize("n", [127, 1023, 1024, 2047, 2048, 8191, 8192, 32767, 32768, 65_536, 65_537, 99_999, 100_000])
def test_row_tile_rule(torch_gpu, orc, n, d):
    """Both sides of every n at which the row tiles per wavefront change; a
    batch of one set has the bits of the same set in a larger batch."""
    l, k = 70, 3
    p = synth.random_problem(n, d, l, k, seed=9500 + d, clusters=3)
    say(f"row tiles: n={n} d={d}")
    Vg, X64 = to_gpu(torch_gpu, p.X, "fp32")
    got = gpu_eval(torch_gpu, Vg, p.sets)
    idx = np.array([0, 33, 69])
    exact(got[idx], orc.eval(X64, p.sets[idx], 8), f"n={n} d={d}")
    assert np.array_equal(got[33:34], gpu_eval(torch_gpu, Vg, p.sets[33:34]))


@pytest.mark.parametrize("n,d,k", [(300, 8, 200), (9000, 20, 90), (40_000, 100, 300), (120_000, 4, 700), (5000, 300, 60)])
def test_tiles_staged_in_lds(torch_gpu, monkeypatch, n, d, k):
    """A limit that admits the call but not one set group's tiles: the
    evaluation kernel stages them itself, with the same bits."""
    torch = torch_gpu
    l = 40
    p = synth.random_problem(n, d, l, k, seed=9700 + d, clusters=3, replace=True)
    sets = p.sets.copy()
    sets[3, 5:] = -1
    sets[4, 0] = n
    Vg, _ = to_gpu(torch, p.X, "fp32")
    full = gpu_eval(torch, Vg, sets)
    # what one set group is accounted for: 4 bytes per coordinate in blocks of
    # 8 (16 above d = 256), a header, one partial-sum row per 64 (16) points
    if d <= 256:
        blocks = -(-d // 8)
        need = -(-n // 256) * 4 * 32 * 4 + k * ((256 if blocks <= 4 else 128) + blocks * 1024) + 1024
    else:
        blocks = 20   # d = 300 in 16s, rounded up to a compiled count
        need = -(-n // 128) * 8 * 16 * 4 + k * (128 + blocks * 1024) + 1024
    rows = 0 if d % 4 == 0 or d <= 8 else -(-(n * (-(-d // 4) * 4) * 4) // 256) * 256
    say(f"tiles in LDS: n={n} d={d} k={k} limit {need + rows}")
    monkeypatch.setenv("EXEMCL_WORKSPACE_LIMIT", str(need + rows))
    assert np.array_equal(full, gpu_eval(torch, Vg, sets), equal_nan=True)
    assert np.isnan(full[4]) and np.isfinite(np.delete(full, 4)).all()
    monkeypatch.setenv("EXEMCL_WORKSPACE_LIMIT", str(need + rows - 2048))
    with pytest.raises(api.ExemclError) as ei:
        gpu_eval(torch, Vg, sets)
    assert ei.value.status == api.EXEMCL_ENOMEM


def least_limit(monkeypatch, call):
    """The smallest EXEMCL_WORKSPACE_LIMIT under which `call` runs, in steps
    of 256 bytes."""
    lo, hi = 0, 1 << 22
    while hi - lo > 1:
        mid = (lo + hi) // 2
        monkeypatch.setenv("EXEMCL_WORKSPACE_LIMIT", str(256 * mid))
        try:
            call()
            hi = mid
        except api.ExemclError as e:
            assert e.status == api.EXEMCL_ENOMEM
            lo = mid
    return 256 * hi


@pytest.mark.parametrize("n,d,k,l", [(1000, 100, 19, 70), (10_000, 512, 3, 40), (300, 8, 70, 33), (5000, 301, 40, 33),
                                     (513, 52, 1, 1)])
def test_gain_and_greedy_under_tight_limits(torch_gpu, monkeypatch, n, d, k, l):
    """From the smallest limit that is accepted up: tiles of S, of the
    candidates, or both staged by the kernels, or S in several passes -- the
    same bits."""
    torch = torch_gpu
    p = synth.random_problem(n, d, 1, 1, seed=9750 + d, clusters=3)
    Vg, _ = to_gpu(torch, p.X, "fp32")
    rng = np.random.default_rng(d)
    S = torch.from_numpy(rng.choice(n, k, replace=False).astype(np.int32)).cuda()
    C = torch.from_numpy(rng.choice(n, l, replace=False).astype(np.int32)).cuda()

    def gain():
        return api.exemplar_gain(Vg, S, C).cpu().numpy()

    def greedy():
        return np.concatenate([x.cpu().numpy() for x in api.exemplar_greedy(Vg, 3)])

    for name, call in (("gain", gain), ("greedy", greedy)):
        monkeypatch.delenv("EXEMCL_WORKSPACE_LIMIT", raising=False)
        full = call()
        least = least_limit(monkeypatch, call)
        say(f"{name} n={n} d={d} |S|={k}: accepted from {least} bytes")
        for limit in (least, int(1.2 * least), int(1.5 * least), 2 * least, 4 * least):
            monkeypatch.setenv("EXEMCL_WORKSPACE_LIMIT", str(limit))
            assert np.array_equal(full, call()), f"{name} limit {limit}"


@pytest.mark.parametrize("n,d,l,k,rows", [(3000, 20, 40, 30, 0), (2500, 100, 33, 3, 700), (4001, 512, 10, 40, 1000)])
def test_streamed_under_tight_limits(torch_gpu, orc, monkeypatch, n, d, l, k, rows):
    """The smallest accepted limit: the kernel stages the exemplar matrix's
    rows itself."""
    torch = torch_gpu
    p = synth.random_problem(n, d, l, k, seed=9770 + d, clusters=3)
    sets = p.sets.copy()
    sets[2, 1:] = -1
    sets[3, 0] = n
    V, S = torch.from_numpy(np.ascontiguousarray(p.X, np.float32)), torch.from_numpy(sets)
    call = lambda: api.exemplar_eval_streamed(V, S, rows_per_block=rows).numpy()   # noqa: E731
    least = least_limit(monkeypatch, call)
    say(f"streamed n={n} d={d} k={k}: accepted from {least} bytes")
    want = orc.eval(p.X.astype(np.float64), sets, 4)
    for limit in (least, 2 * least):
        monkeypatch.setenv("EXEMCL_WORKSPACE_LIMIT", str(limit))
        exact(call(), want, f"streamed limit {limit}")


@pytest.mark.parametrize("scale", [2.0 ** -30, 1.0, 2.0 ** 30])
def test_error_against_64_bits(torch_gpu, orc, scale):
    """Single-member sets of one point's worth of averaging: the error of
    h_s(v) itself, over magnitudes.  The split keeps 24 bits of every value,
    so scaling by a power of two scales the result exactly."""
    n, d = 900, 100
    p = synth.random_problem(n, d, 64, 1, seed=9800, clusters=5)
    Vg, X64 = to_gpu(torch_gpu, p.X * np.float32(scale), "fp32")
    got = gpu_eval(torch_gpu, Vg, p.sets)
    want = orc.eval(X64, p.sets, 4)
    worst = exact(got, want, f"scale {scale:g}")
    assert worst <= 100 * 2.0 ** -24   # d roundings of 2^-24 each
    V1, _ = to_gpu(torch_gpu, p.X, "fp32")
    assert np.array_equal(got, gpu_eval(torch_gpu, V1, p.sets) * scale * scale)


@pytest.mark.parametrize("d", [49, 52, 81, 84, 40, 68])
def test_small_products_stay_apart(torch_gpu, d):
    """Whole blocks and a tail.  The tail's hi*hi products cancel the bias
    exactly (points hold half of the exemplar's tail); what is left of h is a
    whole block's product with a small one, 64 * j / 8 = 8 j, which is gone
    wherever it is added to the tail's 2^27 (multiples of 16 there).  Every
    value is exact in fp32 if the accumulators stay apart, so f is too, up to
    its sums of 512 terms and its own rounding: 12 roundings of 2^-24."""
    n, r0 = 1001, 32 * (d // 32)
    rng = np.random.default_rng(d)
    X = np.zeros((n, d))
    tail = slice(r0, min(d, r0 + 16))
    X[0, tail] = 2.0 ** 12
    X[1:, tail] = 2.0 ** 11
    X[:, :r0] = 64.0
    X[1:, 0] += rng.choice([1, 3, 5], n - 1) / 8
    X = X.astype(np.float32)
    Vg, X64 = to_gpu(torch_gpu, X, "fp32")
    s = X64[0]
    assert np.float32(0.5 * (s * s).sum()) == 0.5 * (s * s).sum()   # the bias is exact
    want = 2.0 / n * np.maximum(0.0, X64 @ s - 0.5 * (s * s).sum()).sum()
    got = gpu_eval(torch_gpu, Vg, np.zeros((1, 1), np.int32))[0]
    say(f"accumulators apart: d={d} rel err {abs(got - want) / want:.2e}")
    assert abs(got - want) <= 12 * 2.0 ** -24 * want


@pytest.mark.parametrize("n", [128, 256])
def test_wavefront_sums_round_once(torch_gpu, n):
    """Even whole coordinates from 560 to 660: every h is a multiple of 2,
    about 1.5e6 and exact, and so is a wavefront's sum of 16 of them (below
    2^24 twos).  What is left to round is a workgroup's sum and the result:
    2^-24 each (the fp64 sums in between add nothing)."""
    d, l = 8, 512
    rng = np.random.default_rng(n)
    X = (2 * rng.integers(280, 331, (n, d))).astype(np.float32)
    sets = rng.integers(0, n, (l, 2)).astype(np.int32)
    Vg, X64 = to_gpu(torch_gpu, X, "fp32")
    H = X64 @ X64.T - 0.5 * (X64 * X64).sum(1)
    want = 2.0 / n * np.maximum(0.0, np.maximum(H[:, sets[:, 0]], H[:, sets[:, 1]])).sum(0)
    got = gpu_eval(torch_gpu, Vg, sets)
    worst = float((np.abs(got - want) / want).max())
    say(f"sums round once: n={n} worst {worst / 2.0 ** -24:.2f} x 2^-24")
    assert worst <= 2 * 2.0 ** -24


def norm_errors(torch, prec, n, d, seed):
    """The error of the bias -|s|^2 / 2 in units of its last place, for 16
    exemplars: points with one coordinate M at a place where |s_0| is a power
    of two, so <v, s> = M s_0 is exact, just above |s|^2 / 2, and h is their
    difference without rounding."""
    rng = np.random.default_rng(seed)
    worst = 0.0
    for rep in range(16):
        s = rng.standard_normal(d)
        s = s * np.sqrt(d / (s * s).sum())
        s[0] = 2.0 ** -4
        X = np.zeros((n, d))
        X[0] = s
        Xs, X64 = synth.rounded(X.astype(np.float32), prec)
        B = 0.5 * (X64[0] ** 2).sum()
        m = np.exp2(np.ceil(np.log2(B * 16)) - 8)                 # eight bits of M: exact in every storage type
        X64[1:, 0] = np.ceil(B * 16 * 1.02 / m) * m
        V, X64 = to_gpu(torch, X64.astype(np.float32), prec)
        got = gpu_eval(torch, V, np.zeros((1, 1), np.int32))[0]
        h = X64[1, 0] * X64[0, 0]                                # exact; h - B > 0
        want = 2.0 / n * ((n - 1) * (h - B) + B)
        ulp = np.exp2(np.floor(np.log2(B)) - 23)
        worst = max(worst, abs(got - want) * n / 2 / n / ulp)
    return worst


@pytest.mark.parametrize("d", [4, 8, 20, 33, 100, 301, 512])
def test_norms_round_once(torch_gpu, d):
    """Half a unit for the bias, f's own sums (a few percent of a unit: h is
    2 % of B), and above d = 127 the fp32 sums of eight squares, each below a
    tenth of a unit: 0.63 in all when evaluated for these exemplars."""
    worst = norm_errors(torch_gpu, "fp32", 4096, d, 31 + d)
    say(f"norms: d={d} worst {worst:.2f} units")
    assert worst <= 0.75


# ---------------------------------------------------------------------------
# Long fp16/bf16 rows as a tiled product (wide_kernels.hpp).
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("n,d,l,k", [(6144, 1025, 40, 1), (6200, 1056, 17, 2), (9001, 1160, 33, 3), (20_011, 1100, 130, 5),
                                     (6145, 2000, 300, 4)])
def test_long_rows_tiled(torch_gpu, orc, prec, n, d, l, k):
    """Odd and even k-blocks, members and set groups that do not fill a
    column block, ragged rows; the launch shape (row tiles, streams per set
    group) follows l and k, the bits must not."""
    p = synth.random_problem(n, d, l, k, seed=9900 + d, clusters=3)
    say(f"long rows: {prec} n={n} d={d} l={l} k={k}")
    Vg, X64 = to_gpu(torch_gpu, p.X, prec)
    got = gpu_eval(torch_gpu, Vg, p.sets)
    idx = np.unique(np.linspace(0, l - 1, 9).astype(int))
    exact(got[idx], orc.eval(X64, p.sets[idx], 8), f"{prec} d={d}")
    assert np.array_equal(got[5:6], gpu_eval(torch_gpu, Vg, p.sets[5:6])), "batch size 1"
    pad = np.concatenate([p.sets, np.full((l, 3), -1, np.int32), p.sets[:, :1]], axis=1)
    assert np.array_equal(got, gpu_eval(torch_gpu, Vg, pad)), "blank and repeated members"


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
def test_long_rows_through_the_other_calls(torch_gpu, orc, monkeypatch, prec):
    """The tiled product from the fixed scratch, in chunks under a limit, and
    over blocks of rows streamed from host memory."""
    torch = torch_gpu
    n, d, l, k = 13_001, 1100, 300, 3
    p = synth.random_problem(n, d, l, k, seed=9920, clusters=3)
    sets = p.sets.copy()
    sets[7, 1:] = -1
    sets[8, 0] = n
    Vg, X64 = to_gpu(torch, p.X, prec)
    s = torch.from_numpy(sets).cuda()
    full = api.exemplar_eval(Vg, s).cpu().numpy()
    out = torch.empty(l, dtype=torch.float32, device="cuda")
    api.exemplar_eval_noalloc(Vg, s, out)
    assert np.array_equal(full, out.cpu().numpy(), equal_nan=True), "noalloc"
    _, ws = api.exemplar_plan(n, d, l, k, {"fp16": api.EXEMCL_FP16, "bf16": api.EXEMCL_BF16}[prec])
    rows = n * 1104 * 2   # the padded copy stays whole
    monkeypatch.setenv("EXEMCL_WORKSPACE_LIMIT", str(rows + (ws - rows) // 4 + 4096))
    assert np.array_equal(full, api.exemplar_eval(Vg, s).cpu().numpy(), equal_nan=True), "chunked"
    monkeypatch.delenv("EXEMCL_WORKSPACE_LIMIT")
    idx = np.array([0, 7, 8, 150, 299])
    want = orc.eval(X64, sets[idx], 8)
    exact(full[idx], want, "in memory")
    for block in (6200, 0, 1000):   # tiled, one block, split coordinates
        got = api.exemplar_eval_streamed(Vg.cpu(), torch.from_numpy(sets), rows_per_block=block).numpy()
        exact(got[idx], want, f"streamed, {block} rows a block")


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("n,d", [(6144, 1025), (6300, 1100)])
def test_long_rows_bias_seeds(torch_gpu, prec, n, d):
    """1 024 coordinates whose product with the exemplar is exactly
    |s|^2 / 2 = 2^25, and a last one that adds 3: exact when the accumulator
    starts at the bias, a multiple of 4 when the bias comes last.  f sums
    h = 3 over all points but the exemplar (2^25, exact): 12 roundings of
    2^-24, and the last coordinate's share of |s|^2 / 2, 2^-25 in h."""
    X = np.zeros((n, d))
    X[0, :1024], X[1:, :1024] = 256.0, 128.0
    X[0, d - 1], X[1:, d - 1] = 2.0 ** -12, 3 * 2.0 ** 12
    Vg, X64 = to_gpu(torch_gpu, X.astype(np.float32), prec)
    assert np.array_equal(X64, X)
    want = 2.0 / n * np.maximum(0.0, X64 @ X64[0] - 0.5 * (X64[0] ** 2).sum()).sum()
    got = gpu_eval(torch_gpu, Vg, np.zeros((1, 1), np.int32))[0]
    say(f"long rows, bias: {prec} n={n} d={d} rel err {abs(got - want) / want:.2e}")
    assert abs(got - want) <= 13 * 2.0 ** -24 * want


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("n,d", [(4096, 1025), (6144, 1025), (6144, 1536)])
def test_long_norms_round_once(torch_gpu, prec, n, d):
    """Long rows' biases, on both kernels: half a unit, and f's own sums."""
    worst = norm_errors(torch_gpu, prec, n, d, 31 + d)
    say(f"norms: {prec} n={n} d={d} worst {worst:.2f} units")
    assert worst <= 0.6


# ---------------------------------------------------------------------------
# Small fp32 calls: tiles staged by the evaluation kernel, results written by
# the workgroup that ends last.
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("n,d,l,k", [(1, 3, 1, 1), (130, 3, 64, 8), (1000, 8, 16, 5), (1000, 8, 65, 5), (1000, 8, 64, 9),
                                     (8191, 128, 33, 8), (5000, 40, 64, 1), (30_000, 20, 20, 4),
                                     (1000, 32, 16, 16), (1000, 32, 16, 17), (1000, 33, 17, 16), (30_000, 8, 16, 3)])
def test_one_launch(torch_gpu, orc, n, d, l, k):
    """Both sides of the rules (k <= 8, 16 up to d = 32; one launch up to
    l = 16): the bits of a set do not
    depend on whether its batch is small enough; calls repeat on one block."""
    p = synth.random_problem(n, d, 80, k, seed=9950 + d, clusters=0, replace=True)
    sets = p.sets.copy()
    sets[3 % l, 0] = n          # invalid: NaN
    sets[2 % l, 1:] = -1        # blanks
    Vg, X64 = to_gpu(torch_gpu, p.X, "fp32")
    full = gpu_eval(torch_gpu, Vg, np.tile(sets, (1, 17)))    # more than 16 tiles: staged by a launch of its own
    say(f"one launch: n={n} d={d} l={l} k={k}")
    for _ in range(3):
        got = gpu_eval(torch_gpu, Vg, sets[:l])
        assert np.array_equal(got, full[:l], equal_nan=True)
    idx = np.arange(0, l, max(1, l // 5))
    check(got[idx], orc.eval(X64, sets[idx], 4), orc.loss_e0(X64), "fp32", "one launch")


@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("n,d,l,k", [(1, 1, 1, 1), (5000, 16, 64, 8), (5000, 17, 20, 3),
                                     (6001, 32, 16, 31), (6001, 33, 16, 15), (6001, 64, 17, 16),
                                     (10_000, 70, 48, 8), (9000, 80, 65, 8), (20_011, 96, 5, 4), (7000, 109, 33, 7), (12_345, 128, 16, 8)])
def test_one_launch_16_bit(torch_gpu, orc, prec, n, d, l, k):
    """Every compiled row length (32 x 32 tiles up to d = 16, then 1 .. 4
    k-blocks, the last one whole or half) of the 16-bit kernels: as above."""
    p = synth.random_problem(n, d, 80, k, seed=9970 + d, clusters=0, replace=True)
    sets = p.sets.copy()
    sets[3 % l, 0] = n
    sets[2 % l, 1:] = -1
    Vg, X64 = to_gpu(torch_gpu, p.X, prec)
    full = gpu_eval(torch_gpu, Vg, np.tile(sets, (1, 17)))   # more than 16 tiles: staged by a launch of its own
    say(f"one launch: {prec} n={n} d={d} l={l} k={k}")
    for _ in range(3):
        got = gpu_eval(torch_gpu, Vg, sets[:l])
        assert np.array_equal(got, full[:l], equal_nan=True)
    idx = np.arange(0, l, max(1, l // 5))
    check(got[idx], orc.eval(X64, sets[idx], 4), orc.loss_e0(X64), prec, "one launch")
