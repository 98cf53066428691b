"""CPU: the torch reference of the canonical clustering against the C library's
fmaf and the oracle."""
import ctypes
import ctypes.util

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import canonical  # noqa: E402
import oracle  # noqa: E402


def test_fma_rounds_once():
    libm = ctypes.CDLL(ctypes.util.find_library("m"))
    libm.fmaf.restype, libm.fmaf.argtypes = ctypes.c_float, [ctypes.c_float] * 3
    rng = np.random.default_rng(3)
    a, b = (rng.standard_normal(20000).astype(np.float32) for _ in range(2))
    c = (rng.standard_normal(20000) * 2.0 ** rng.integers(-60, 40, 20000)).astype(np.float32)
    c[:4000] = -(a[:4000] * b[:4000])              # cancellation
    # sums next to the midpoint of two floats, by far less than float64 keeps
    a[4000:8000] = 1 + 2.0 ** -12
    b[4000:8000] = (1 + rng.integers(0, 2, 4000) * 2.0 ** -23) * 2.0 ** -60
    c[4000:8000] = 1 + rng.integers(0, 1 << 20, 4000) * 2.0 ** -22
    b[8000:9000] *= 2.0 ** -24
    a[8000:9000] = 1
    b[8000:9000] = 2.0 ** -24
    c[8000:9000] = np.nextafter(np.float32(1), np.float32(2)) * rng.choice([-1, 1], 1000)
    got = canonical.fma32(*map(torch.from_numpy, (a, b, c))).numpy()
    want = np.array([libm.fmaf(*v) for v in zip(a, b, c)], np.float32)
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("dyadic", [False, True])
def test_assignment_and_update_match_the_oracle(dyadic):
    rng = np.random.default_rng(4)
    n, d, C = 1500, 24, 40
    if dyadic:  # many exact ties
        x = rng.integers(-2, 3, (1, n, d)).astype(np.float32) / 2
    else:
        x = (rng.standard_normal((1, 9, d))[:, rng.integers(0, 9, n)]
             + 1e-5 * rng.standard_normal((1, n, d))).astype(np.float32)
    init = rng.choice(n, C, replace=False).astype(np.int32)[None]
    q = oracle.cluster_queries(x, C, 1, init)
    t = torch.from_numpy(x[0])
    u = t[torch.from_numpy(init[0]).long()]
    g, scored = canonical.assign(t, u)
    assert np.array_equal(g.numpy(), q["assign"][0]) and scored > 50
    assert np.array_equal(canonical.update(t, g, u).numpy().view(np.uint32),
                          q["centroids"][0].view(np.uint32))
