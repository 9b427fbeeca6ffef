// The encoder's rounded brackets, evaluated on the CPU by the code the kernel compiles (CornerGrid of csrc/octopus_encode.hpp).  Per
// number of direction bits 3, 4, 5 one line: the bits, near_axis(), the bracket of a coordinate 0 and of 1, whether the bracket never
// falls as the coordinate grows (every fp32 difference to 1 / 2 that is a multiple of 2^-25), and the first coordinate of each further bracket.
// Built by tests/test_encoder_brackets.py.
#include <cmath>
#include <cstdio>
#include <cstring>

#include "octopus_encode.hpp"

template <int BD>
static void show() {
    using G = octopus::CornerGrid<BD>;
    auto at = [](float w) {
        return static_cast<int>(G::bracket_within(std::fmin(std::fmax(w, -G::kReach), G::kReach)) - G::kOne) - G::H;
    };
    const int first = at(-0.5f);
    std::printf("%d %.9g %d %d", BD, static_cast<double>(G::near_axis()), first, at(0.5f));
    int last = first;
    bool rises = true;
    double steps[64];
    int n = 0;
    for (long k = -(1L << 24); k <= (1L << 24); ++k) {
        const float w = std::ldexp(static_cast<float>(k), -25);
        const int b = at(w);
        rises = rises && b >= last;
        for (; last < b && n < 64; ++last) steps[n++] = 0.5 + static_cast<double>(w);
        last = b;
    }
    std::printf(" %d", rises ? 1 : 0);
    for (int i = 0; i < n; ++i) std::printf(" %.17g", steps[i]);
    std::printf("\n");
}

int main() {
    show<3>();
    show<4>();
    show<5>();
    return 0;
}
