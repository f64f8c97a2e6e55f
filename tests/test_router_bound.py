"""How far the fp64 router's logits can be from the exact sums: the bounds by which large batches decide whether exact integer
sums give a token the same experts and weights (route_exact_kernel), against the fp64 chain itself in its order of summation.
The products of two bf16 values are exact in fp64, and math.fsum rounds their exact sum once."""
import math

import numpy as np
import pytest
import torch


def rows(n, H, spread, seed):
    """[n, H] bf16 values: normally distributed, each times a power of two from a range of `spread`."""
    g = torch.Generator().manual_seed(seed)
    scale = 2.0 ** -torch.randint(0, spread + 1, (n, H), generator=g).double()
    return (torch.randn((n, H), generator=g, dtype=torch.float64) * scale).bfloat16()


def chain(x, w):
    """The fp64 sums of row pairs, in the kernel's order: 32-wide chunk c belongs to partial sum c % 16; in a chunk, value j of its
    four quarters for j = 0 .. 7; partial sums p, p + 4, p + 8, p + 12 in order, then those four."""
    n, H = x.shape
    part = np.zeros((16, n))
    for c in range((H + 31) // 32):
        for j in range(8):
            for q in range(4):
                k = c * 32 + q * 8 + j
                if k < H:
                    part[c % 16] += x[:, k] * w[:, k]
    z = None
    for p in range(4):
        s = part[p]
        for i in (4, 8, 12):
            s = s + part[p + i]
        z = s if z is None else z + s
    return z


def heads(a):
    """2-norm, largest 2-norm of the values of one partial sum, and the last place of the smallest value."""
    v = a.double().numpy()
    of = np.arange(v.shape[1]) // 32 % 16
    part = np.max([np.sqrt((v[:, of == p] ** 2).sum(1)) for p in range(16)], axis=0)
    e = (a.view(torch.int16).int().numpy() & 0x7fff) >> 7
    last = np.where(v == 0, 512, e).min(1) - 134
    return np.sqrt((v ** 2).sum(1)), part, last


@pytest.mark.parametrize("H", [8, 72, 1000, 2048, 4104])
@pytest.mark.parametrize("spread", [0, 4, 8, 16, 22])
def test_the_chain_stays_within_the_bounds(H, spread):
    n = 300
    bx, bw = rows(n, H, spread, H + spread), rows(n, H, spread, H + spread + 1)
    bx[:, :: 7] = 0
    x, w = bx.double().numpy(), bw.double().numpy()
    got = chain(x, w)
    exact = np.array([math.fsum(a * b) for a, b in zip(x, w)])
    (nx, px, lx), (nw, pw, lw) = heads(bx), heads(bw)
    fits = 2.0 ** (53 + lx + lw)
    how = np.where(nx * nw < fits, 0, np.where(px * pw < fits, 1, 2))
    terms = ((H + 31) // 32 + 15) // 16 * 32
    bound = np.choose(how, [0 * nx, 8 * nx * nw * 2.0 ** -53, (terms + 40) * nx * nw * 2.0 ** -52])
    assert (np.abs(got - exact) <= bound).all()
    if H == 2048 and spread in (4, 8):
        assert set(how) == {0, 1, 2}
    if H >= 1000 and spread >= 16:
        assert (got != exact).any()            # (the bounds are about something)
