"""GPU: attention calls that run in a block order of their own, some of their
slots as two halves.  Every row is checked against plain torch attention in
float64 on the inputs rounded to bf16, and must be bit for bit that of the same
call with room for the work list alone (list order, whole slots, fp32 K and V
rounded row by row): a result depends neither on the workspace nor on the other
heads of the call, nor do NaN and infinities spread further."""
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
    "dense_4096": (2, [4096], [4096], 128, "bf16"),            # shortest call with an order
    "dense_4161_d64": (1, [4161], [4161], 64, "bf16"),         # a ragged last tile
    "dense_4500_f32": (1, [4500], [4500], 128, "f32"),
    "sparse_ragged": (1, [5000, 40, 300, 1, 0, 6000, 129, 4914], [16384, 4097, 4032, 1, 9, 8191, 16000, 5000],
                      128, "bf16"),
    "sparse_pairs_d64": (2, [100] * 60 + [4200, 6200], [4096 + 64 * (i % 7) for i in range(60)] + [0, 9000],
                         64, "bf16"),
    "sparse_f32_d64": (1, [16400 - 3 * 700] + [700] * 3, [4200, 16400, 4100, 64], 64, "f32"),
    "uneven": (1, *_uneven(16500), 128, "bf16"),
    "whole_slots": (20, [26214 // 9] * 9, [6000] * 9, 64, "bf16"),  # no halves
    "round_and_halves": (5, [14401], [14401], 128, "bf16"),    # a round of whole slots, the rest halved
}


def _problem(heads, sizes, keys, d, dtype):
    n, c_q = sum(sizes), len(sizes)
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
    return shape, q, k, v, offsets, perm, counts, sel


def _attend(shape, q, k, v, offsets, perm, counts, sel):
    """The call with the whole workspace, and with room for the list alone."""
    heads, n, c_q = shape.heads, shape.n, counts.shape[1]
    full = B.alloc_workspace(shape, c_q, (1, 1, 1))
    lists = torch.empty(2 * heads * (-(-n // 256) + c_q) * 16 + 256, dtype=torch.uint8, device="cuda")
    out = []
    for ws in (full, lists):
        o = torch.full_like(q, float("nan"))
        B.scope_sparse_attention(shape, q, k, v, c_q, offsets, perm.int(), counts, sel, 0.0, o, ws)
        out.append(o)
    torch.cuda.synchronize()
    return out


def _bits(o):
    return o.view(torch.int16 if o.dtype == torch.bfloat16 else torch.int32)


@pytest.mark.parametrize("name", list(CASES))
def test_split_slots(name):
    heads, sizes, keys, d, dtype = CASES[name]
    n, c_q = sum(sizes), len(sizes)
    G.say(f"[split] {name}: heads={heads} n={n} clusters={c_q} d={d} {dtype}")
    shape, q, k, v, offsets, perm, counts, sel = _problem(heads, sizes, keys, d, dtype)
    out = _attend(shape, q, k, v, offsets, perm, counts, sel)
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
    err = (out[0].double() - ref).abs()
    assert float(err.max()) <= G.MAX_ABS
    assert float(err.sum() / ref.abs().sum()) <= G.MEAN_REL
    assert torch.equal(_bits(out[0]), _bits(out[1]))


# few slots and waves run a block each, more of them in pairs: of these heads one
# alone is on the one side and `heads` of them on the other
@pytest.mark.parametrize("heads,sizes,d,dtype", [
    (60, [100] * 13, 64, "bf16"),
    (9, [300, 1, 0, 256, 33, 517, 64] * 2, 64, "bf16"),
    (2, [3] * 700, 64, "bf16"),
    (3, [2] * 1024, 64, "bf16"),                # paired either way
    (6, [64] * 50, 128, "f32"),
    (13, [24] * 45, 128, "f32"),                # copies of K and V for the many chunks
    (9, [12] * 92, 64, "f32"),
    (4, [300, 1, 0, 256, 33, 517, 64], 128, "bf16"),
])
def test_remainders_alone_or_paired(heads, sizes, d, dtype):
    n, c_q = sum(sizes), len(sizes)
    G.say(f"[split] alone or paired: heads={heads} n={n} clusters={c_q} d={d} {dtype}")
    keys = [(37 * i + 5) % n + 1 for i in range(c_q)]
    shape, q, k, v, offsets, perm, counts, sel = _problem(heads, sizes, keys, d, dtype)
    many = _attend(shape, q, k, v, offsets, perm, counts, sel)
    off = (0, d // 4, d // 2)
    shape1 = B.make_shape(1, n, d, shape.dtype, (off, (d // 4, d // 4, d // 2)))
    for h in (0, heads - 1):
        one = _attend(shape1, *(x[h:h + 1].contiguous() for x in (q, k, v, offsets, perm, counts, sel)))
        for o in one:
            assert torch.equal(_bits(o[0]), _bits(many[0][h]))
    qd, kd, vd = (x[0].to(torch.bfloat16).double() for x in (q, k, v))
    for c in range(0, c_q, max(1, c_q // 20)):
        rows, kk = perm[0, offsets[0, c]:offsets[0, c + 1]], sel[0, c, :keys[c]].long()
        if rows.numel():
            ref = torch.softmax(qd[rows] @ kd[kk].T / math.sqrt(d), 1) @ vd[kk]
            assert float((many[0][0, rows].double() - ref).abs().max()) <= G.MAX_ABS


@pytest.mark.parametrize("d,dtype", [(128, "bf16"), (64, "bf16"), (128, "f32")])
def test_not_finite_values_stay_where_they_are(d, dtype):
    heads, n = 2, 4608
    G.say(f"[split] NaN and infinite logits, d={d} {dtype}")
    shape, q, k, v, offsets, perm, counts, sel = _problem(heads, [n], [n], d, dtype)
    # head 0: the logits of the second half of the keys overflow to -inf, a
    # whole number of tiles: weights of exactly zero
    q[0, :, 0] = 4.0
    k[0, n // 2:, 0] = -3e38
    # head 1: one NaN value in V, one in Q
    v[1, 3000, 5] = float("nan")
    q[1, 77, 1] = float("nan")
    out = _attend(shape, q, k, v, offsets, perm, counts, sel)
    assert torch.equal(_bits(out[0]), _bits(out[1]))
    o = out[0].double()
    r16 = lambda x: x.to(torch.bfloat16).double()
    p = torch.softmax(r16(q[0]) @ r16(k[0, :n // 2]).T / math.sqrt(d), 1)
    ref = p @ r16(v[0, :n // 2])
    assert float((o[0] - ref).abs().max()) <= G.MAX_ABS
    nan = torch.zeros(n, d, dtype=torch.bool, device="cuda")
    nan[:, 5] = nan[77] = True
    assert torch.equal(torch.isnan(o[1]), nan)
