// Tile shapes and K slices of the LDS convolution (nn_conv.hip), host and device.
#pragma once

namespace casclb {
namespace nn {

// A workgroup's TH x TW pixels of CI channels with their halo, T matrix-core tiles of 16
// pixels per wavefront; K = tap CI + channel in slices of 32, "piece" q = 8 values of K.
template <int CI, int TW, int T>
struct Tile {
    static constexpr int TPR = TW / 16;            // matrix-core tiles per pixel row
    static constexpr int R = T / TPR;              // pixel rows per wavefront
    static constexpr int TH = 4 * R;
    static constexpr int HW = TW + 2, HH = TH + 2, NP = HW * HH;
    static constexpr int PS = CI + 8;              // LDS elements per pixel
    static constexpr int CPP = CI / 8;             // 8-channel pieces per pixel
    static constexpr int S = (9 * CI + 31) / 32;   // K slices
    static constexpr int KPAD = 32 * S;
    // LDS elements: the lanes past the end of K read up to 8 values behind the last pixel
    // (which become zeros)
    static constexpr int LDS = NP * PS + 8;
    static constexpr int tap_of(int q) { return q / CPP > 8 ? 8 : q / CPP; }
    // LDS offset of piece q minus 8 (q mod 4), a function of its tap only within a slice
    static constexpr int offset(int q) {
        const int tap = tap_of(q), slice = q / 4;
        return ((tap / 3) * HW + tap % 3) * PS + 32 * slice - CI * tap;
    }
    static constexpr int split(int s) {            // first lane group of slice s in its second tap (4: none)
        for (int g = 1; g < 4; ++g)
            if (tap_of(4 * s + g) != tap_of(4 * s)) return g;
        return 4;
    }
    static constexpr int live(int s) {             // lane groups of slice s before the end of K
        const int left = 9 * CPP - 4 * s;
        return left < 4 ? left : 4;
    }
};

}  // namespace nn
}  // namespace casclb
