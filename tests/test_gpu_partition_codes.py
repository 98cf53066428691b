"""GPU selection from code planes: planes of up to three subspaces are packed
into one word per key where the workspace has the room, and the selection then
runs over the distinct codes.  Compared bit for bit with the selection from
the planes themselves (the smallest workspace that the call takes) and from
the materialised logits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2608_12780_amd import binding as B  # noqa: E402

import gpu_harness as G  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


# 1024 is the largest codebook (10 bits); 3000 keys of 1024^3 codes are all
# distinct; 4 subspaces stay on the planes
@pytest.mark.parametrize("heads,n,c_m", [
    (2, 1, (1,)), (1, 257, (64,)), (2, 3001, (1024,)),
    (1, 1023, (7, 300)), (3, 2050, (1024, 1024)),
    (2, 3000, (1024, 1024, 1024)), (1, 4099, (5, 1, 9)), (1, 40000, (40, 30, 20)),
    (2, 1500, (6, 5, 4, 3)),
])
@pytest.mark.parametrize("values", ["spread", "zeros"])
def test_planes_packed_or_not_select_the_same_keys(heads, n, c_m, values):
    G.say(f"[planes] heads={heads} n={n} c_m={c_m} {values}")
    M, c_q, d = len(c_m), 3 if n > 2 else 1, 64
    rng = np.random.default_rng(n + M)
    c_m = tuple(min(c, n) for c in c_m)
    bounds = np.linspace(0, d, M + 1).astype(int)
    part = B.make_partition([range(bounds[m], bounds[m + 1]) for m in range(M)], c_m)
    shape = B.make_shape(heads, n, d, B.BF16, ((0, 16, 40), (16, 24, 24)))
    # a few codes lie beyond their codebooks, up to 65535: clamped on the device
    codes = np.stack([rng.integers(0, c_m[m], (heads, n)) for m in range(M)], 1)
    codes[:, :, n // 2] = 65535
    clamped = np.stack([np.minimum(codes[:, m], c_m[m] - 1) for m in range(M)], 1)
    col = np.concatenate([[0], np.cumsum(c_m)]).astype(int)
    tables = rng.standard_normal((heads, c_q, col[-1])).astype(np.float32) * 2
    if values == "zeros":  # logits of both zeros and of equal sums
        tables = np.where(rng.random(tables.shape) < 0.5, np.float32(-0.0), np.float32(0.0))
        tables[:, :, 0] = 3.0
    s = np.zeros((heads, c_q, n), np.float32)
    for h in range(heads):
        for m in range(M):
            t = tables[h][:, col[m] + clamped[h, m]]
            s[h] = t if m == 0 else s[h] + t
    s = (s * np.float32(0.125) + np.float32(0.0)).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    tables_d, scores_d = dev(tables.astype(np.float32)), dev(s)
    codes_d = dev(codes.astype(np.uint16).view(np.int16))
    counts = dev(rng.integers(1, 9, (heads, c_q)).astype(np.int32))
    size = B.alloc_partition_workspace(shape, c_q, part, "cuda").numel()

    def select(scores, ws):
        e = lambda *sh: torch.full(sh, -1, dtype=torch.int32, device="cuda")
        o = dict(base=e(heads, c_q), topp=e(heads, c_q), k_head=e(heads), cnt=e(heads, c_q),
                 idx=e(heads, c_q, n))
        B.scope_select_partition(shape, c_q, part, scores, tables_d, codes_d, counts, 0.8,
                                 (n + 9) // 10, o["base"], o["topp"], o["k_head"], o["cnt"],
                                 o["idx"], ws)
        torch.cuda.synchronize()
        return o

    # the smallest workspace that the call takes (too small ones are refused
    # on the host) has no room to pack
    full = torch.empty(size, dtype=torch.uint8, device="cuda")
    lo, hi = 0, size
    while lo + 1 < hi:
        mid = (lo + hi) // 2
        try:
            select(scores_d, full[:mid])
            hi = mid
        except Exception:
            lo = mid
    assert hi < size or M > 3
    want = select(scores_d, full)
    for got in (select(None, full), select(None, full[:hi])):
        for key in ("base", "topp", "k_head", "cnt", "idx"):
            assert torch.equal(got[key], want[key]), key
