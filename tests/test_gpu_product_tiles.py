"""Matrix-core products over bit layouts in which the indices interleave: edges of tiles, ranges of K, batches."""
import numpy as np
import pytest
import torch

from paper_2108_06831_amd import contract_pair

pytestmark = pytest.mark.gpu

# (b, m, n, k) as powers of two: fewer rows or columns than a tile, whole and several tiles, less than a K tile, more
# K tiles than the kernel tabulates (K / ranges > 1024), packed batches and columns
SIZES = [(0, 5, 7, 6), (0, 6, 5, 9), (0, 6, 6, 3), (0, 7, 6, 4), (1, 7, 9, 5), (0, 6, 7, 13), (6, 5, 5, 5), (7, 5, 4, 4),
         (0, 5, 17, 3), (4, 4, 13, 4), (3, 6, 10, 2), (0, 10, 10, 6), (1, 11, 8, 8), (0, 3, 12, 9)]


def _layout(rng, b, m, n, k, interleave):
    """Modes of extent 2 in shuffled order in each tensor, or (not interleaved) in blocks."""
    ids = {"b": list(range(b)), "m": list(range(100, 100 + m)), "n": list(range(200, 200 + n)),
           "k": list(range(300, 300 + k))}
    sides = [ids["b"] + ids["m"] + ids["k"], ids["b"] + ids["k"] + ids["n"], ids["b"] + ids["m"] + ids["n"]]
    if interleave:
        sides = [[int(v) for v in rng.permutation(s)] for s in sides]
    return ids, sides


def _product(ids, sides, a, b):
    """The product in complex128 on the CPU, in C's layout."""
    pos = lambda side, what: [side.index(v) for v in ids[what]]
    size = lambda what: 1 << len(ids[what])
    A = a.permute(pos(sides[0], "b") + pos(sides[0], "m") + pos(sides[0], "k")).reshape(size("b"), size("m"), size("k"))
    B = b.permute(pos(sides[1], "b") + pos(sides[1], "k") + pos(sides[1], "n")).reshape(size("b"), size("k"), size("n"))
    C = np.matmul(A.numpy(), B.numpy()).reshape([2] * len(sides[2]))
    order = ids["b"] + ids["m"] + ids["n"]
    return C.transpose([order.index(v) for v in sides[2]])


@pytest.mark.parametrize("precision", ["c64", "bf16x3"])
@pytest.mark.parametrize("interleave", [True, False])
@pytest.mark.parametrize("size", SIZES)
def test_products_of_any_layout(size, interleave, precision):
    rng = np.random.default_rng(sum(v * 17 ** i for i, v in enumerate(size)) + interleave)
    ids, sides = _layout(rng, *size, interleave)
    gen = torch.Generator().manual_seed(7)
    a, b = (torch.randn([2] * len(s), dtype=torch.complex64, generator=gen) for s in sides[:2])
    got = contract_pair(a.cuda(), sides[0], b.cuda(), sides[1], sides[2], precision=precision).cpu().numpy()
    want = _product(ids, sides, a.to(torch.complex128), b.to(torch.complex128))
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    # rounding of K sums in FP32 (three-product form: a few units per term); split precision: each operand to 2^-17,
    # the product of the low parts (2^-18) dropped, over the four real products of a complex one
    K = 1 << size[3]
    bound = 2.0 ** -24 * (8 + 2 * np.sqrt(K)) if precision == "c64" else 2.0 ** -14 + 2.0 ** -24 * 2 * np.sqrt(K)
    assert err < bound, (size, interleave, precision, err, bound)
    assert np.abs(got - want).max() < 64 * bound * np.abs(want).max()
