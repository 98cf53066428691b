"""GPU: attention calls of few work slots, which run in an order of their own
with their last slots cut along the keys and joined from partial results.
Every row is checked against plain torch attention in float64 on the inputs
rounded to bf16, and against the same call with room for the work list alone
(whole slots, K and V rounded row by row)."""
import math

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


# (heads, cluster sizes, keys per cluster, d, dtype)
def _uneven(n):
    # one long cluster, then hundreds of cheap slots: an equal-cost queue would
    # overflow, so the queues are cut by number
    sizes = [2048] + [(n - 2048) // 299] * 299
    sizes[-1] += n - sum(sizes)
    return sizes, [n] + [1 + (7 * i) % 64 for i in range(299)]


CASES = {
    "dense_4096": (2, [4096], [4096], 128, "bf16"),            # shortest list that splits
    "dense_4161_d64": (1, [4161], [4161], 64, "bf16"),         # a ragged last tile
    "dense_4500_f32": (1, [4500], [4500], 128, "f32"),
    "sparse_ragged": (1, [5000, 40, 300, 1, 0, 6000, 129, 4914], [16384, 4097, 4032, 1, 9, 8191, 16000, 5000],
                      128, "bf16"),
    "sparse_pairs_d64": (2, [100] * 60 + [4200, 6200], [4096 + 64 * (i % 7) for i in range(60)] + [0, 9000],
                         64, "bf16"),
    "sparse_f32_d64": (1, [16400 - 3 * 700] + [700] * 3, [4200, 16400, 4100, 64], 64, "f32"),
    "uneven": (1, *_uneven(16500), 128, "bf16"),
    "whole_slots": (20, [26214 // 9] * 9, [6000] * 9, 64, "bf16"),  # no pieces: eight rounds and more
}


@pytest.mark.parametrize("name", list(CASES))
def test_split_slots(name):
    heads, sizes, keys, d, dtype = CASES[name]
    n, c_q = sum(sizes), len(sizes)
    G.say(f"[split] {name}: heads={heads} n={n} clusters={c_q} d={d} {dtype}")
    g = torch.Generator(device="cuda").manual_seed(n + d)
    rand = lambda s: s * torch.randn(heads, n, d, generator=g, device="cuda")
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v = (rand(s).to(tdt) for s in (1.5, 1.5, 1.0))
    offsets = torch.zeros(heads, c_q + 1, dtype=torch.int32, device="cuda")
    offsets[:, 1:] = torch.tensor(np.cumsum(sizes), device="cuda")
    perm = torch.stack([torch.randperm(n, generator=g, device="cuda") for _ in range(heads)])
    counts = torch.tensor(keys, dtype=torch.int32, device="cuda").repeat(heads, 1)
    sel = torch.full((heads, c_q, n), -1, dtype=torch.int32, device="cuda")
    for h in range(heads):
        for c, r in enumerate(keys):
            sel[h, c, :r] = torch.randperm(n, generator=g, device="cuda")[:r].sort()[0]
    off = (0, d // 4, d // 2)
    shape = B.make_shape(heads, n, d, B.BF16 if dtype == "bf16" else B.F32, (off, (d // 4, d // 4, d // 2)))
    full = B.alloc_workspace(shape, c_q, (1, 1, 1))
    lists = torch.empty(2 * heads * (-(-n // 256) + c_q) * 16 + 256, dtype=torch.uint8, device="cuda")
    out = []
    for ws in (full, lists):
        o = torch.full_like(q, float("nan"))
        B.scope_sparse_attention(shape, q, k, v, c_q, offsets, perm.int(), counts, sel, 0.0, o, ws)
        out.append(o.double())
    torch.cuda.synchronize()
    ref = torch.zeros(heads, n, d, dtype=torch.float64, device="cuda")
    for h in range(heads):
        qd, kd, vd = (x[h].to(torch.bfloat16).double() for x in (q, k, v))
        for c, r in enumerate(keys):
            rows = perm[h, offsets[h, c]:offsets[h, c + 1]]
            if r == 0 or rows.numel() == 0:
                continue
            kk = sel[h, c, :r].long()
            for a in range(0, rows.numel(), 2048):
                p = torch.softmax(qd[rows[a:a + 2048]] @ kd[kk].T / math.sqrt(d), 1)
                ref[h, rows[a:a + 2048]] = p @ vd[kk]
    for o in out:
        err = (o - ref).abs()
        assert float(err.max()) <= G.MAX_ABS
        assert float(err.sum() / ref.abs().sum()) <= G.MEAN_REL
    # both round the weights to bf16 against running maxima of their own
    assert float((out[0] - out[1]).norm() / out[1].norm()) <= 5e-3
