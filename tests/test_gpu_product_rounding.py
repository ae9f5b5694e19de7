"""Rounding of complex64 products along the launch shapes taken by default.

A chain of c multiply-adds of random terms leaves a relative error of about
0.42 2^-24 sqrt(c / 2) (rms of a rounding to nearest, the partial sums growing
as the square root of their terms); a complex product of K terms is a chain of
2 K per component.  K cut into r parts leaves the chains 2 K / r long and adds
log2 r (lanes of a wave, added in a tree) or r / 2 (ranges added in turn).
Bounds take 0.5 for 0.42.  The sizes are ones that a shape chosen for speed
alone would round more: a tile's whole K where sums can go in lanes, fewer
ranges of K, three real products for four."""
import numpy as np
import pytest
import torch

from paper_2108_06831_amd import contract_pair

pytestmark = pytest.mark.gpu


def _product(a, b):
    got = contract_pair(a, [0, 1, 2], b, [0, 2, 3], [0, 1, 3])
    want = torch.stack([torch.mm(x, y) for x, y in zip(a.to(torch.complex128), b.to(torch.complex128))])
    return got.to(torch.complex128), want


# (batch, m, n, k as powers of two), lanes or ranges, what adding them up counts
LONG = [((3, 3, 9, 8), 32, 5), ((3, 3, 10, 10), 16, 4), ((0, 3, 12, 10), 32, 5), ((3, 9, 4, 7), 16, 4),
        ((7, 6, 3, 9), 16, 4), ((0, 9, 9, 9), 8, 4), ((0, 11, 7, 8), 8, 4), ((0, 8, 11, 9), 4, 2), ((0, 7, 12, 7), 4, 2)]


@pytest.mark.parametrize("size,parts,adds", LONG)
def test_long_sums_stay_short_chains(size, parts, adds):
    b, m, n, k = size
    gen = torch.Generator(device="cuda").manual_seed(sum(size))
    x, y = (torch.randn(s, dtype=torch.complex64, device="cuda", generator=gen)
            for s in ((1 << b, 1 << m, 1 << k), (1 << b, 1 << k, 1 << n)))
    got, want = _product(x, y)
    err = float((got - want).norm() / want.norm())
    bound = 0.5 * 2.0 ** -24 * np.sqrt((1 << k) / parts + adds)
    print(f"{size}: {err:.2e}, bound {bound:.2e}", flush=True)
    assert err < bound


@pytest.mark.parametrize("size", [(0, 10, 10, 7), (0, 9, 9, 9), (2, 10, 9, 8), (7, 5, 12, 2), (10, 5, 5, 5), (12, 5, 3, 5),
                                  (7, 4, 5, 9), (10, 4, 10, 4), (0, 5, 17, 3)])
def test_small_imaginary_parts_keep_their_own_precision(size):
    """Operands whose imaginary parts are 2^-12 of their real ones: formed from products of its own, the
    result's imaginary part is right to its own magnitude; as a difference of three products it is
    right to that of the real part only, 2^12 times as far off."""
    b, m, n, k = size
    gen = torch.Generator(device="cuda").manual_seed(sum(size))

    def operand(*s):
        re, im = (torch.randn(s, device="cuda", generator=gen) for _ in range(2))
        return torch.complex(re, im * 2.0 ** -12)
    got, want = _product(operand(1 << b, 1 << m, 1 << k), operand(1 << b, 1 << k, 1 << n))
    err = float((got.imag - want.imag).norm() / want.imag.norm())
    bound = 0.5 * 2.0 ** -24 * np.sqrt((1 << k) + 8)
    print(f"{size}: {err:.2e}, bound {bound:.2e}", flush=True)
    assert err < bound
