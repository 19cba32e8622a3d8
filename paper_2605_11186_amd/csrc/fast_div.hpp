// Division by a number that only the launch knows, as a product and a shift.  Plain C++ (constexpr: host and device).
#pragma once
#include <stdint.h>

// n / d for n < 2^31: m = floor(2^(31 + l) / d) + 1 with d <= 2^l exceeds 2^(31 + l) / d by at most 2^l / 2^(31 + l) of it,
// less than 1 / n.  The division itself is some 35 instructions on the device, about 2 ns each at the head of a launch, and a
// workgroup of a product did four to ten of them.
struct FastDiv {
    uint32_t m = 1, s = 0;   // d = 1
};
constexpr FastDiv make_fast_div(uint32_t d) {
    if (d <= 1) return FastDiv{};
    uint32_t l = 1;
    while (l < 31 && (1u << l) < d) ++l;
    return FastDiv{static_cast<uint32_t>((uint64_t{1} << (31 + l)) / d + 1), 31 + l};
}
constexpr uint32_t fast_div(uint32_t n, FastDiv d) { return static_cast<uint32_t>((static_cast<uint64_t>(n) * d.m) >> d.s); }
