"""GPU k-means against the oracle, bit for bit, where the kernels' paths meet:
element type, channel widths on both sides of each padded width (odd ones for
fp32), one centroid to more than the LDS holds, all iterations in one block
(320 rows), several blocks of fused iterations, and the separate launches
(sums beyond the LDS, or 48 MiB of rows), few and many row blocks per head
(the finish kernel shares a row's sums among four waves from 8 blocks on),
exact ties, fp32 values outside the range of the matrix-core filter, and rows
that start at any element of a buffer.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_2608_12780_amd import binding as B  # noqa: E402
from paper_2608_12780_amd.inputs import bf16_bits, bf16_widen  # noqa: E402
from paper_2608_12780_amd.layer import ScopeLayer  # noqa: E402

import gpu_harness as G  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    oracle.lib()


def _rows(rng, heads, n, d, dtype):
    """Clustered rows (so that near-ties are rare but present)."""
    centres = rng.standard_normal((heads, 23, d))
    x = np.stack([centres[h][rng.integers(0, 23, n)] for h in range(heads)])
    x = (x + 0.4 * rng.standard_normal(x.shape)).astype(np.float32)
    return bf16_widen(bf16_bits(x)) if dtype == "bf16" else x


def _device(x, dtype):
    t = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    return t.to(torch.bfloat16) if dtype == "bf16" else t


def _init(rng, n, c, *lead):
    return np.stack([np.sort(rng.choice(n, c, replace=False)).astype(np.int32)
                     for _ in range(int(np.prod(lead)))]).reshape(*lead, c)


def _check(x, dtype, split, c_q, c_m, iters, init_q, init_k):
    heads, n, d = x.shape
    off = np.concatenate([[0], np.cumsum(split)[:-1]])
    ranges = (tuple(int(o) for o in off), tuple(split))
    G.say(f"[kmeans] {dtype} heads={heads} n={n} split={split} c_q={c_q} c_m={c_m}")
    layer = ScopeLayer(heads, n, d, ranges, c_q, c_m, iters, 0.9, 1, dtype=dtype)
    dev = _device(x, dtype)
    layer.cluster_queries(dev, torch.from_numpy(init_q).cuda())
    layer.cluster_keys(dev, torch.from_numpy(init_k).cuda())
    torch.cuda.synchronize()
    q = oracle.cluster_queries(x, c_q, iters, init_q)
    k = oracle.cluster_key_subspaces(x, ranges, c_m, iters, init_k)
    assert np.array_equal(layer.assign.cpu().numpy(), q["assign"])
    assert np.array_equal(layer.perm.cpu().numpy(), q["perm"])
    assert np.array_equal(layer.codes.cpu().numpy().view(np.uint32), k["codes"])
    return layer, q, k


@pytest.mark.parametrize("dtype,heads,n,split,c_q,c_m", [
    ("f32", 2, 256, (16, 24, 24), 8, (8, 8, 8)),        # one row block
    ("f32", 1, 2311, (17, 31, 33), 31, (33, 1, 32)),    # odd widths, many blocks
    ("f32", 5, 777, (15, 47, 49), 96, (40, 7, 64)),
    ("f32", 3, 1500, (16, 56, 56), 65, (33, 32, 31)),   # fused iterations
    ("f32", 2, 1200, (44, 42, 42), 300, (333, 20, 5)),  # beyond one block's LDS
    ("bf16", 1, 2311, (10, 2, 52), 1, (3, 2, 70)),
    ("bf16", 40, 300, (44, 42, 42), 33, (17, 64, 31)),  # few blocks per head
    ("bf16", 2, 1999, (16, 24, 24), 129, (32, 33, 16)),
    ("bf16", 3, 320, (16, 56, 56), 31, (9, 33, 32)),    # one block, ten slices
    ("bf16", 3, 321, (16, 56, 56), 31, (9, 33, 32)),    # eleven
    ("f32", 1, 29, (43, 42, 43), 7, (5, 29, 1)),        # one slice, odd pairs
    ("bf16", 300, 330, (8, 4, 4), 5, (3, 2, 7)),        # one block of 11 slices
    ("bf16", 260, 700, (44, 42, 42), 5, (3, 2, 7)),     # one block each: an iteration, and all
    ("bf16", 100, 1100, (8, 4, 4), 5, (3, 2, 7)),       # an iteration, 35 slices
    ("f32", 60, 1100, (8, 4, 4), 5, (3, 2, 7)),         # all, 35 slices
    ("f32", 45, 1100, (8, 4, 4), 5, (3, 2, 7)),         # separate
    ("bf16", 1, 700, (44, 42, 42), 86, (64, 90, 128)),  # sums about as large as the LDS
    # separate launches, sums beyond the LDS: queries and a lone fitting subspace
    # by themselves, the three in one pass, several in one launch
    ("f32", 2, 1100, (44, 42, 42), 160, (700, 20, 720)),
    ("f32", 2, 1100, (16, 24, 24), 224, (32, 480, 448)),
    ("f32", 2, 1100, (16, 56, 56), 129, (192, 220, 220)),
    ("f32", 2, 1100, (44, 42, 42), 255, (320, 160, 150)),
    ("f32", 2, 1100, (44, 42, 42), 130, (333, 300, 260)),
    ("bf16", 2, 1100, (16, 56, 56), 161, (333, 260, 300)),
    ("f32", 2, 98304, (16, 24, 24), 9, (8, 8, 8)),      # either side of 48 MiB
    ("bf16", 2, 98305, (44, 42, 42), 9, (8, 8, 8)),
])
def test_clustering_matches_the_oracle(dtype, heads, n, split, c_q, c_m):
    rng = np.random.default_rng(n + heads)
    x = _rows(rng, heads, n, sum(split), dtype)
    layer, q, k = _check(x, dtype, split, c_q, c_m, 4, _init(rng, n, c_q, heads),
                         _init(rng, n, max(c_m), heads, 3))
    assert np.array_equal(layer.q_centroids.cpu().numpy().view(np.uint32),
                          q["centroids"].view(np.uint32))
    assert np.array_equal(layer.k_centroids.cpu().numpy().view(np.uint32).reshape(-1),
                          k["centroids"].view(np.uint32).reshape(-1))


def test_fp32_exact_ties_take_the_lowest_centroid():
    # rows on a coarse dyadic grid, every starting row three times: exact ties
    rng = np.random.default_rng(5)
    proto = rng.integers(-4, 5, (40, 64)).astype(np.float32) / 4
    x = proto[rng.integers(0, 40, 900)][None]
    init = np.repeat(rng.choice(900, 12, replace=False), 3).astype(np.int32)[None]
    _check(x, "f32", (16, 24, 24), 36, (36, 36, 36), 1, init, np.repeat(init[:, None], 3, 1))


@pytest.mark.parametrize("share", [1.0, 0.5, 0.06])
@pytest.mark.parametrize("n,split,c_q,c_m", [
    (300, (16, 56, 56), 37, (8, 33, 70)),          # all iterations in one block
    (1500, (17, 31, 33), 70, (33, 70, 32)),        # fused iterations, odd widths
    (1100, (44, 42, 42), 300, (333, 130, 90)),     # separate launches, a chunked codebook
])
def test_fp32_rows_with_many_tied_centroids(n, split, c_q, c_m, share):
    # a share of the rows are the same, and so are the centroids that start from
    # them: few, many or all points of a wave need the canonical scan
    rng = np.random.default_rng(n)
    x = _rows(rng, 2, n, sum(split), "f32")
    same = rng.random((2, n)) < share
    x[same] = 0.0 if share < 1.0 else x[0, 0]
    init_q, init_k = _init(rng, n, c_q, 2), _init(rng, n, max(c_m), 2, 3)
    ties = np.flatnonzero(same[0])[:12]
    init_q[:, :len(ties)] = ties      # a dozen centroids that tie, whatever the share
    init_k[:, :, :min(len(ties), min(c_m))] = ties[:min(c_m)]
    layer, q, k = _check(x, "f32", split, c_q, c_m, 3, init_q, init_k)
    assert np.array_equal(layer.q_centroids.cpu().numpy().view(np.uint32), q["centroids"].view(np.uint32))
    assert np.array_equal(layer.k_centroids.cpu().numpy().view(np.uint32).reshape(-1),
                          k["centroids"].view(np.uint32).reshape(-1))


@pytest.mark.parametrize("c_q", [20, 300])
def test_fp32_values_outside_the_filter(c_q):
    # one assignment (the status word reports such inputs, and their sums are
    # not defined): rows that overflow the filter, are not finite or denormal
    rng = np.random.default_rng(c_q)
    x = _rows(rng, 1, 1100, 128, "f32")
    bad = [1e20, 3e38, -3e38, np.inf, -np.inf, np.nan, 1e-42, 0.0]
    for i, v in enumerate(bad):
        x[0, 10 * i + 3, i] = v
        x[0, 10 * i + 5] = v
    ordinary = _init(rng, 1000, c_q, 1) + 100
    extreme = ordinary.copy()
    extreme[0, 4], extreme[0, 7], extreme[0, 11] = 5, 13, 53  # 1e20, 3e38 and NaN
    for init in (ordinary, extreme):
        G.say(f"[kmeans] extreme fp32 rows, c_q={c_q}")
        layer = ScopeLayer(1, 1100, 128, ((0, 16, 72), (16, 56, 56)), c_q, (9, 9, 9), 1, 0.9, 1,
                           dtype="f32")
        layer.cluster_queries(_device(x, "f32"), torch.from_numpy(init).cuda())
        want = oracle.cluster_queries(x, c_q, 1, init)["assign"]
        got = layer.assign.cpu().numpy()
        assert np.array_equal(got, want), np.flatnonzero(got != want)[:20]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,c_q,c_m", [
    (300, 9, (8, 8, 8)),           # all iterations in one block
    (1500, 33, (33, 32, 31)),      # fused iterations
    (1500, 160, (200, 224, 224)),  # separate launches
])
def test_rows_from_any_element_on(dtype, n, c_q, c_m):
    """Rows that start one element into their buffer give the same bits."""
    heads, split, iters = 2, (16, 56, 56), 3
    rng = np.random.default_rng(n)
    x = _device(_rows(rng, heads, n, 128, dtype), dtype)
    buf = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")
    y = buf[1:].view(x.shape)
    y.copy_(x)
    assert y.data_ptr() % 16 == x.element_size()
    init_q = torch.from_numpy(_init(rng, n, c_q, heads)).cuda()
    init_k = torch.from_numpy(_init(rng, n, max(c_m), heads, 3)).cuda()
    G.say(f"[kmeans] rows at an odd element, {dtype} n={n} c_q={c_q}")
    got = []
    for t in (x, y):
        layer = ScopeLayer(heads, n, 128, ((0, 16, 72), split), c_q, c_m, iters, 0.9, 1, dtype=dtype)
        layer.cluster_queries(t, init_q)
        layer.cluster_keys(t, init_k)
        torch.cuda.synchronize()
        got.append((layer.q_centroids, layer.assign, layer.perm, layer.k_centroids, layer.codes))
    for a, b in zip(*got):
        assert torch.equal(a, b)
