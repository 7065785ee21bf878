"""The DRAM time of the searches whose bandwidth or array count is no power of two is formed without a
division (dram_time_general): restated here with exact rational arithmetic, it has the bits of
c_lat * fl(fl(words * word) / dram_bw) for word counts and bandwidths over their whole ranges."""
import math
import random
from fractions import Fraction


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))        # one rounding


def dram_time(words, word, bw, c_lat):
    b, k = math.frexp(bw)
    b, k = 2.0 * b, k - 1
    y, c = 1.0 / b, math.ldexp(c_lat, -k)
    x = words * word
    q = x * y
    q = fma(fma(-b, q, x), y, q)
    q = fma(fma(-b, q, x), y, q)
    return c * q


def test_same_bits_as_the_division():
    rng = random.Random(5)
    worst = [1.0 + 2.0 ** -52, 2.0 - 2.0 ** -52, 1.0 + 2.0 ** -26, 1.5, 60.0, 3.0, 2.0 ** -40 * 3, 1e300, 1e-200]
    for n in range(30000):
        bw = rng.choice(worst) if n % 3 == 0 else rng.choice([rng.uniform(0.1, 1000.0), float(rng.randrange(1, 4096)),
                                                              math.ldexp(1.0 + rng.random(), rng.randrange(-60, 60))])
        word = float(rng.choice([1, 2, 3, 4, 8]))
        words = float(rng.choice([rng.randrange(1, 1 << 12), rng.randrange(1, 1 << 32), rng.randrange(1, 1 << 50)]))
        if n % 5 == 0 and 1.0 <= bw < 1e9:        # quotients next to a whole number or a midpoint
            words = float(max(1, int(bw * rng.randrange(1, 1 << 20)) + rng.randrange(-1, 2)))
        c_lat = rng.randrange(1, 129) / rng.choice([1.0, 2.0, 3.0, 5.0])
        assert dram_time(words, word, bw, c_lat) == c_lat * ((words * word) / bw), (words, word, bw, c_lat)
