"""The primality test behind every entry point's check of p, against a Miller-Rabin
with other bases: all small numbers, the divisors of its own bases, strong
pseudoprimes to the first prime bases, squares and products of close primes, and the
top of the accepted range."""
import pytest

import paper_2505_24256_amd as zr
import synth

BASES = (325, 9375, 28178, 450775, 9780504, 1795265022)


def _divisors_that_are_prime(n):
    out, d = set(), 2
    while d * d <= n:
        while n % d == 0:
            out.add(d)
            n //= d
        d += 1
    return out | ({n} if n > 1 else set())


def _numbers(kind):
    if kind == "small":
        return range(0, 20_000)
    if kind == "bases":
        ps = sorted(set().union(*map(_divisors_that_are_prime, BASES)))
        return [a * b for a in ps for b in ps + [1]] + list(BASES)
    if kind == "pseudoprimes":
        return [2047, 1373653, 25326001, 3215031751, 2152302898747, 3474749660383, 341550071728321,
                3825123056546413051, 561, 1105, 1729, 2465, 8911, 825265, 321197185]
    if kind == "squares":
        ps = [p for p in range(3_037_000_000 - 500, 3_037_000_000, 1) if synth.is_prime(p)]
        return [a * b for a in ps for b in ps]
    return list(range((1 << 63) - 600, (1 << 63))) + list(range((1 << 61) - 300, (1 << 61) + 300))


@pytest.mark.parametrize("kind", ["small", "bases", "pseudoprimes", "squares", "top"])
def test_prime_check(kind):
    for n in _numbers(kind):
        assert bool(zr.lib().zr_is_prime(n)) == synth.is_prime(n), n


def test_prime_check_beyond_the_field_range():
    for n in (1 << 63, (1 << 63) + 29, (1 << 64) - 59):
        assert not zr.lib().zr_is_prime(n)
