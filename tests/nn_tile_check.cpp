// Host check of the LDS convolution's slice arithmetic (csrc/nn_tile.hpp) against the plain
// k -> (tap, channel) decode, for every channel count and tile shape that is instantiated.
#include <cstdio>
#include "nn_tile.hpp"
using namespace casclb::nn;
static long bad = 0, n = 0;
#define CHECK(c) do { ++n; if (!(c)) { if (bad++ < 10) printf("FAIL %s line %d CI %d TW %d T %d\n", #c, __LINE__, CI, TW, T); } } while (0)

template <int CI, int TW, int T> void tile() {
    using G = Tile<CI, TW, T>;
    CHECK(G::TH * TW == 4 * 16 * T && G::R * G::TPR == T && G::HW == TW + 2 && G::HH == G::TH + 2);
    CHECK(G::KPAD >= 9 * CI && G::KPAD - 9 * CI < 32 && G::KPAD == 32 * G::S);
    for (int s = 0; s < G::S; ++s) {
        const int first = G::offset(4 * s), second = G::offset(4 * s + 3), at = G::split(s), live = G::live(s);
        for (int g = 0; g < 4; ++g) {
            const int k = 32 * s + 8 * g;
            CHECK((g < live) == (k < 9 * CI));
            if (k >= 9 * CI) continue;   // zeros, whatever is read
            const int tap = k / CI, c = k - tap * CI;
            CHECK(G::tap_of(4 * s + g) == tap && c % 8 == 0 && c + 8 <= CI);
            // as the kernel reads it: 8 g of the lane's base, one of two offsets
            const int off = 8 * g + (first == second ? first : (g >= at ? second : first));
            CHECK(off == ((tap / 3) * G::HW + tap % 3) * G::PS + c);
        }
        // past the end of K too the addresses lie in the workgroup's LDS
        for (int g = 0; g < 4; ++g) {
            const int off = 8 * g + (first == second ? first : (g >= at ? second : first));
            const int last = ((3 * G::R + (T - 1) / G::TPR) * G::HW + 16 * ((T - 1) % G::TPR) + 15) * G::PS + off;
            CHECK(off >= 0 && last + 8 <= G::LDS);
        }
    }
}

int main() {
    tile<16, 32, 4>(); tile<32, 32, 4>(); tile<48, 32, 4>(); tile<64, 32, 4>(); tile<80, 32, 4>(); tile<96, 32, 4>();
    tile<16, 16, 2>(); tile<32, 16, 2>(); tile<48, 16, 2>(); tile<64, 16, 2>(); tile<80, 16, 2>(); tile<96, 16, 2>();
    tile<112, 16, 2>(); tile<128, 16, 2>(); tile<160, 16, 2>(); tile<192, 16, 2>();
    printf("%ld checks, %ld failures\n", n, bad);
    return bad != 0;
}
