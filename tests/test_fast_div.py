"""Division by a product and a shift (the work split of the products): the constants, built for the CPU, against integer division."""
import ctypes as C
import random

import host_shim


class FastDiv(C.Structure):
    _fields_ = [("m", C.c_uint32), ("s", C.c_uint32)]


def test_quotients_are_exact_below_two_to_the_31():
    lib = host_shim.build("""
#include "fast_div.hpp"
extern "C" void make_into(uint32_t d, FastDiv* out) { *out = make_fast_div(d); }
extern "C" uint32_t quotient(uint32_t n, const FastDiv* d) { return fast_div(n, *d); }
""")

    def make(d):
        f = FastDiv()
        lib.make_into(C.c_uint32(d), C.byref(f))
        return f

    rng = random.Random(1)
    top = 2 ** 31 - 1
    divisors = list(range(1, 3000)) + [2 ** k + e for k in range(1, 31) for e in (-1, 0, 1)] + [top - 1, top] + \
        [rng.randrange(1, 2 ** 31) for _ in range(2000)]
    for d in divisors:
        f = make(d)
        assert 0 < f.m < 2 ** 32 and f.s < 64
        q = top // d   # the error grows with the quotient and shows first just below a multiple
        for k in {0, 1, q - 1, q, rng.randrange(q + 1), rng.randrange(q + 1), rng.randrange(q + 1)}:
            for n in (k * d - 1, k * d, k * d + 1, k * d + d - 1):
                if 0 <= n <= top:
                    assert n * f.m < 2 ** 64 and n * f.m >> f.s == n // d, (n, d)
        assert lib.quotient(C.c_uint32(top), C.byref(f)) == q
