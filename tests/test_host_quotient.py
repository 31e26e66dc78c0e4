"""The kernels' division by the host's reciprocals (gemm_device.h: Divisor, quotient), the same arithmetic in Python."""
import random


def quotient(n, d):
    r = 0xFFFFFFFF if d == 1 else 2 ** 32 // d
    q = n * r >> 32
    return q + 1 if n - q * d >= d else q


def test_quotient_is_exact_below_2_to_31():
    rng = random.Random(7)
    divisors = [1, 2, 3, 4, 7, 8, 2 ** 31 - 1, 2 ** 30, 2 ** 16 + 1] + [rng.randrange(1, 2 ** rng.randrange(1, 32)) for _ in range(3000)]
    for d in divisors:
        top = (2 ** 31 - 1) // d * d
        for n in {0, 1, d - 1, d, 2 * d - 1, 2 * d, top - 1, top, 2 ** 31 - 1, rng.randrange(2 ** 31)}:
            if 0 <= n < 2 ** 31:
                assert quotient(n, d) == n // d, (n, d)
