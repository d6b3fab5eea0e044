"""The float32 quotients by a shared reciprocal (divisor, exact_div in rk_model.h) are the correctly rounded ones for the
divisors and dividends they are used with.  The fused multiply-adds are emulated: the product of two float32 is exact in
float64, the sum is rounded to odd there and then to float32.  The hardware's approximate reciprocal may be off by one unit
either way, so every case starts from all three."""
import numpy as np

F = np.float32


def fma(a, b, c):
    x, y = a.astype(np.float64) * b.astype(np.float64), c.astype(np.float64)
    s = x + y
    t = s - x
    err = (x - (s - t)) + (y - t)                                # what the sum lost
    even = (s.view(np.int64) & 1) == 0
    s = np.where((err != 0) & even, np.nextafter(s, np.where(err > 0, np.inf, -np.inf)), s)
    return s.astype(F)


def approximate(b):
    r = (1.0 / b.astype(np.float64)).astype(F)
    return [r, np.nextafter(r, F(0)), np.nextafter(r, F(np.inf))]


def reciprocal(b, r):                                            # divisor
    return fma(fma(-b, r, np.ones_like(b)), r, r)


def quotient(a, b, r):                                           # exact_div
    q = (a * r).astype(F)
    return fma(fma(-q, b, a), r, q)


def test_fused_multiply_add_is_emulated_right():
    """1 + 2^-24 + 2^-60 lies above the midpoint of two float32, though its float64 does not."""
    one = np.ones(1, F)
    assert fma(F([2.0 ** -24 + 2.0 ** -47]), F([1.0]), one)[0] == F(1.0 + 2.0 ** -23)
    assert fma(F([2.0 ** -30]), F([2.0 ** -30]), F([1.0 + 2.0 ** -23]))[0] == F(1.0 + 2.0 ** -23)
    assert fma(F([1.0 - 2.0 ** -24]), F([2.0 ** -24]), one)[0] == one[0]
    assert fma(F([1.0 + 2.0 ** -23]), F([2.0 ** -24]), one)[0] == F(1.0 + 2.0 ** -23)


def test_quotients_by_a_number_of_replicas():
    d = np.arange(1, 65536).astype(F)
    for r in approximate(d):
        inv = reciprocal(d, r)
        assert np.array_equal(inv, F(1) / d)
        assert np.array_equal(F(8) * inv, F(8) / d)
        for a in (6.0, 7.0):
            assert np.array_equal(quotient(np.full_like(d, a), d, inv), F(a) / d)


def test_quotients_by_the_shards_of_a_model():
    """d = t*p, t a power of two: every p below 4,096, and every t at some of them, with dividends over the mantissas and the
    exponents that the kernels hand over (1e-20 to 1e30)."""
    rng = np.random.default_rng(5)
    p = np.arange(1, 4096)
    mantissas = np.concatenate([[0, 1, 2, 3, 2 ** 23 - 1, 2 ** 23 - 2, 2 ** 22], rng.integers(0, 2 ** 23, 100)])
    a = np.ldexp(1.0 + mantissas / 2.0 ** 23, rng.integers(-66, 99, len(mantissas))).astype(F)
    for t in (1, 8):
        b, x = (m.reshape(-1) for m in np.meshgrid((t * p).astype(F), a))
        for r in approximate(b):
            assert np.array_equal(quotient(x, b, reciprocal(b, r)), x / b)
    every = np.arange(2 ** 23, 2 ** 24, dtype=np.int64).astype(F)        # every mantissa, at a few p
    for k in (3, 4095):
        b = np.full_like(every, k)
        for r in approximate(b[:1]):
            inv = reciprocal(b[:1], r)
            assert np.array_equal(quotient(every, b, np.broadcast_to(inv, b.shape)), every / b)
