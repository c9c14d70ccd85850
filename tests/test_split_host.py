"""The arithmetic of the three-part split of float32 operands (h the upper half
of the bits, m and l the remainders rounded to bf16), in numpy: what the parts
leave of an operand and the six products of a product."""
import numpy as np

import workloads


def bf16(x):
    return workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(x.astype(np.float32)))


def split(x):
    h = (x.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
    m = bf16(x - h)
    return h, m, bf16((x - h) - m)


def operands(scale=1.0):
    """Every lower half under a few upper halves, and normal values."""
    low = np.arange(65536, dtype=np.uint32)
    high = [(np.float32(s).view(np.uint32) & np.uint32(0xFFFF0000)) for s in (1.0, 1.0078125, 1.5, 1.9921875)]
    x = np.concatenate([(h | low).view(np.float32) for h in high]
                       + [np.random.default_rng(1).standard_normal(100_000).astype(np.float32)])
    return (x * np.float32(scale)).astype(np.float32)


def test_parts_add_up_to_the_operand():
    """Exact down to 2^-110 (the last bit of such an operand is 2^-133, bf16's
    smallest value); below, up to half of that is lost."""
    for k in (0, 60, 110, 114, 120, 124):
        x = operands(2.0 ** -k)
        lost = np.abs(sum(p.astype(np.float64) for p in split(x)) - x.astype(np.float64))
        assert not lost[np.abs(x) >= 2.0 ** -110].any()
        assert lost.max() <= 2.0 ** -134
        assert k < 111 or lost.any()


def test_six_products_are_the_product_up_to_2_to_the_minus_22():
    """ml, lm and ll are left out: under 2^-22 of the product (2^-23 is passed),
    and 2^-25 in the mean square."""
    x = operands()
    worst = x[np.argmax(np.abs(x.astype(np.float64) - sum(p.astype(np.float64) for p in split(x)[:2]))
                        / np.abs(x))]
    rng = np.random.default_rng(2)
    errs = []
    for y in (x, np.full_like(x, worst), rng.permutation(x)):
        a, b = [[p.astype(np.float64) for p in split(q)] for q in (x, y)]
        six = a[0] * (b[0] + b[1] + b[2]) + a[1] * (b[0] + b[1]) + a[2] * b[0]
        exact = x.astype(np.float64) * y.astype(np.float64)
        ok = exact != 0
        errs.append(np.abs(six - exact)[ok] / np.abs(exact)[ok])
    e = np.concatenate(errs)
    assert 2.0 ** -23 < e.max() < 2.0 ** -22
    normal = errs[2]
    assert np.sqrt(np.mean(normal ** 2)) < 2.0 ** -25
