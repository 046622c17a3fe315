"""The primality test behind the rule that a1 and a2 are distinct primes, against
trial division: small numbers, pseudoprimes of its bases, squares of primes
and the ends of the 32-bit range."""
import pytest

from paper_2609_37538_amd import avsg as A


@pytest.fixture(scope="module", autouse=True)
def _lib():
    try:
        A.load()
    except ImportError:
        pytest.skip("libavsg.so not built")


def _prime(v):
    return v > 1 and all(v % d for d in range(2, min(v, int(v ** 0.5) + 2)))


HARD = [2047, 3277, 4033, 4681, 25326001, 314821, 46657, 252601, 1194649, 12327121, 3215031751, 2654435761,
        2246822519, 4294967291, 4294967295, 4294967279, 65521 * 65521, 65521 * 65519, 2147483647, 4294836225]


def test_prime_rule_matches_trial_division():
    other = 1000003
    for v in list(range(0, 2500)) + [p * p for p in (61, 67, 251, 40009)] + HARD:
        ok = A.avsg_check_config(A.make_config(2, 64, 1, 256, a1=v, a2=other)) == A.AVSG_OK
        assert ok == _prime(v), v
