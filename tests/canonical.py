"""The canonical k-means assignment and update in plain torch, on any device:
a reference for whole problems that shares no code with the library.

The argmin of fl(|u_r|^2 - 2 <x, u_r>), with fp32 fma chains in channel order,
is decided by float64 scores wherever they differ by more than the chains can
err; the few points left are scored by the chains themselves."""
import torch


def fma32(a, b, c):
    """fp32 a * b + c with one rounding.  The product is exact in float64; the
    sum is rounded to odd there, which makes the rounding to fp32 the only one
    that counts (Boldo and Melquiond, "Emulation of a FMA and correctly rounded
    sums: proved algorithms using rounding to odd", 2008)."""
    p, c = a.double() * b.double(), c.double()
    s = p + c
    t = s - p
    err = (p - (s - t)) + (c - t)
    bits = s.view(torch.int64)
    outward = (err > 0) == (s > 0)  # the exact sum lies further from zero
    odd = torch.where((err != 0) & (bits & 1 == 0), torch.where(outward, bits + 1, bits - 1), bits)
    return odd.view(torch.float64).float()


def chain(x, u):
    """<x, u> of the rows of x and u as an fp32 fma chain."""
    acc = torch.zeros(x.shape[0], dtype=torch.float32, device=x.device)
    for c in range(x.shape[1]):
        acc = fma32(x[:, c], u[:, c], acc)
    return acc


def assign(x, u):
    """The canonical centroid of every row of x [n, d] among u [C, d] (fp32),
    and how many rows took the chains."""
    d = x.shape[1]
    nu = chain(u, u)
    x64, u64 = x.double(), u.double()
    s = torch.addmm(nu.double()[None], x64, u64.T.contiguous(), alpha=-2.0)
    # |chain - exact| <= d 2^-24 sum |x_c u_c| (and terms of second order), one
    # rounding of the last fma, and the float64 sum's own, far below
    reach = x64.norm(dim=1) * u64.norm(dim=1).max()
    err = 1.01 * (2 * d * 2.0 ** -24 * reach + 2.0 ** -24 * (nu.max().double() + 2 * reach))
    near = s <= (s.min(1).values + 2 * err)[:, None]
    out = s.argmin(1)
    rows = torch.nonzero(near.sum(1) > 1)[:, 0]
    if rows.numel():
        i, r = torch.nonzero(near[rows], as_tuple=True)
        two = torch.full((i.numel(),), -2.0, device=x.device)
        score = fma32(two, chain(x[rows[i]], u[r]), nu[r])
        best = torch.full((rows.numel(),), float("inf"), device=x.device)
        best = best.scatter_reduce(0, i, score, "amin")
        first = torch.full((rows.numel(),), u.shape[0], dtype=torch.int64, device=x.device)
        out[rows] = first.scatter_reduce(0, i, torch.where(score == best[i], r, u.shape[0]), "amin")
    return out, rows.numel()


def update(x, g, u):
    """The means of the rows of x by label g: exact int64 sums of rint(x 2^24),
    one float64 division, rounded to fp32; an empty cluster keeps its row of u."""
    total = torch.zeros(u.shape, dtype=torch.int64, device=x.device)
    total.index_add_(0, g, torch.round(x.double() * 2.0 ** 24).long())
    count = torch.bincount(g, minlength=u.shape[0])
    mean = (total.double() / (count.double() * 2.0 ** 24)[:, None]).float()
    return torch.where((count > 0)[:, None], mean, u)
