"""GPU selection with the distinct-code build at the edges of its table sizes:
512 to 16384 slots per part, one part to the most, tables as full as they get
(every key its own code) and nearly empty (a handful of codes), against the
selection from the same logits materialised."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2608_12780_amd import binding as B  # noqa: E402

import gpu_harness as G  # noqa: E402


# heads x n: slots per part / parts of the build
@pytest.mark.parametrize("heads,n", [
    (1, 1), (2, 409), (1, 410),       # 512 slots: one part full to 80%, then two
    (3, 13107), (3, 13108),           # 32 parts of 512, then 17 of 1024
    (30, 26214), (40, 32760),         # 4 parts of 8192 and 5
    (150, 9000),                      # 16384: a block per head, no room for more
])
@pytest.mark.parametrize("distinct", [True, False])
def test_selection_from_codes_equals_selection_from_scores(heads, n, distinct):
    G.say(f"[codes] heads={heads} n={n} distinct={distinct}")
    rng = np.random.default_rng(heads * n + distinct)
    c_q, c_m, d = 3, (61, 53, 47), 64
    if distinct:  # a third of all triples, each once
        flat = np.stack([rng.permutation(61 * 53 * 47)[:n] for _ in range(heads)])
    else:
        flat = rng.integers(0, 5, (heads, n)) * 7919 % (61 * 53 * 47)
    codes = (flat % 61) | (flat // 61 % 53 << 10) | (flat // (61 * 53) << 20)
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    tables = torch.from_numpy(rng.standard_normal((heads, c_q, sum(c_m))).astype(np.float32) * 2).cuda()
    counts = i32(rng.integers(1, 9, (heads, c_q)))
    codes = i32(codes)
    shape = B.make_shape(heads, n, d, B.BF16, ((0, 16, 40), (16, 24, 24)))
    # the logits of the tables, in the order that the selection sums them
    z = [(codes.long() >> (10 * m)) & 1023 for m in range(3)]
    col = [0, 61, 114]
    pick = [torch.gather(tables, 2, (z[m] + col[m])[:, None].expand(-1, c_q, -1)) for m in range(3)]
    scores = ((pick[0] + pick[1]) + pick[2]) * np.float32(1.0 / 8.0) + 0.0
    ws = torch.empty(B.scope_workspace_size(shape, min(c_q, n), (min(61, n), min(53, n), min(47, n)))
                     + (1 << 20), dtype=torch.uint8, device="cuda")
    if n < 61:
        c_q, c_m = 1, (1, 1, 1)
        tables, scores, counts = tables[:, :1, :3].contiguous(), scores[:, :1].contiguous(), counts[:, :1].contiguous()
        codes = torch.zeros_like(codes)
        scores = ((tables[:, :, :1] + tables[:, :, 1:2]) + tables[:, :, 2:3]) * np.float32(0.125) + 0.0
        scores = scores.contiguous()
    got = []
    for s in (None, scores.contiguous()):
        e = lambda *sh: torch.full(sh, -1, dtype=torch.int32, device="cuda")
        o = dict(base=e(heads, c_q), topp=e(heads, c_q), k_head=e(heads), cnt=e(heads, c_q),
                 idx=e(heads, c_q, n))
        B.scope_select(shape, c_q, c_m, s, tables, codes, counts, 0.8, (n + 9) // 10, o["base"],
                       o["topp"], o["k_head"], o["cnt"], o["idx"], ws)
        got.append(o)
    torch.cuda.synchronize()
    for key in got[0]:
        assert torch.equal(got[0][key], got[1][key]), key


@pytest.mark.parametrize("cnt", [1, 2, 127, 128, 129, 130])
@pytest.mark.parametrize("ties", [False, True])
def test_crossing_lists_around_the_direct_limit(cnt, ties):
    """All logits within one coarse bin (1/64): the crossing list holds `cnt`
    distinct codes, resolved directly up to 128 of them; with `ties` several
    codes share a logit.  Both crossings (Top-p and rank) against the oracle."""
    G.say(f"[codes] crossing list of {cnt}, ties={ties}")
    rng = np.random.default_rng(cnt + 1000 * ties)
    c_q, d, n = 3, 64, 3 * cnt + 5
    step = np.arange(cnt) // 3 if ties else np.arange(cnt)
    tables = np.zeros((1, c_q, cnt + 2), np.float32)
    for c in range(c_q):
        tables[0, c, :cnt] = rng.permutation(step).astype(np.float32) * 2.0 ** -11
    codes = np.concatenate([np.arange(cnt), rng.integers(0, cnt, n - cnt)])[rng.permutation(n)]
    counts = rng.integers(1, 50, (1, c_q)).astype(np.int32)
    for rho, k_fix in ((0.5, 1), (0.05, max(1, n // 3)), (0.9, n - 1)):
        G.select_from_codes(tables, codes[None].astype(np.uint32), counts, d, (cnt, 1, 1), rho, k_fix)
