// Types shared by the host API and the kernels of the casclb library.
#pragma once

#include <stdint.h>

namespace casclb {

enum Lattice : int { kD2Q9 = 0, kD2Q9D2Q5 = 1, kD3Q27 = 2, kD3Q15 = 3 };
enum Storage : int { kF64 = 0, kF32Dev = 1, kF16Dev = 2 };

// du2, u2, drho, momentum x/y/z, scalar, non-finite count, dphi2, phi2
constexpr int kDiagSlots = 10;
constexpr int kMaxBlock = 256;  // largest block of any kernel

// Division of n < 2^31 by a fixed divisor d >= 1 as a multiply-high and a
// shift (round-up method for invariant divisors): q = (mulhi(n, m) + n) >> s
// with s = ceil(log2 d), m = floor(2^32 (2^s - d) / d) + 1.  Lets a kernel
// decode its block index with scalar integer ops instead of an emulated
// division.
struct FastDiv {
    uint32_t d, m, s;
    FastDiv() : d(1), m(1), s(0) {}
    explicit FastDiv(uint32_t div) : d(div), m(0), s(0) {
        while ((1ull << s) < div) ++s;
        m = (uint32_t)((((1ull << s) - div) << 32) / div + 1);
    }
#ifdef __HIPCC__
    __host__ __device__
#endif
    uint32_t div(uint32_t n) const {
        const uint32_t hi = (uint32_t)(((uint64_t)n * m) >> 32);
        return (hi + n) >> s;
    }
};

// Lattice geometry seen by a kernel.
struct Geometry {
    int32_t nx, ny, nz;
    int32_t bb[3];        // 1: halfway bounce-back walls at both ends of the axis
    int64_t plane;        // elements between population planes
    int32_t x_blocks;     // blocks along x per row
    int32_t xcd_remap;    // 1: give each XCD a contiguous range of rows
    int64_t grid_blocks;  // total blocks of the launch (< 2^31)
    int32_t rows;         // rows per thread (1 or 2): a thread updates node x of `rows` consecutive rows
    int32_t nrows;        // ny * nz
    int32_t xpair;        // 1: 16-bit storage, a thread updates nodes 2t, 2t+1 (x_blocks counts pairs)
    FastDiv div_xb;       // division by x_blocks
    FastDiv div_ny;       // division by ny
    int32_t flat;         // 1: threads take consecutive flat nodes (casclb_step_flat), not rows
};

// Arguments of the fused step kernel (passed by value).
struct StepArgs {
    Geometry geo;
    const void* src;   // stored state (flow planes, then scalar planes)
    void* dst;         // next state
    double rho0;
    double w_shear, w_bulk, w_third, w_fourth;  // flow relaxation rates
    double w_phi, w_phi_high;                    // scalar relaxation rates
    // force: uniform components or a [dims][plane] field in the arithmetic type
    double fx, fy, fz;   // separate fields: an indexed array here ends up in scratch
    const void* force_field;
    double f_pre, f_tot;   // time factors: pre-collision half step, whole step
    // source (scalar lattice only)
    double source;
    const void* source_field;
    double s_pre, s_tot;
    // residual check (DIAG kernels only)
    void* u_prev;          // [dims][plane] previous check's velocity, arithmetic type
    double* partials;      // [grid_blocks][kDiagSlots]
    // walls of 2D lattices (EXT kernels only), side index 2*axis + (0 low,
    // 1 high), axis 0 = x, 1 = y, as a device table (indexed by a run-time
    // side; an array among the kernel arguments would be copied to scratch):
    // [0..8) wall velocity (x, y) per side, [8..12) 1 = scalar held fixed,
    // [12..16) the fixed scalar value
    const double* walls;
    double heat;           // viscous-heating coefficient c_h of the scalar source c_h (S:S)
    int32_t ext;           // walls move, a scalar wall is fixed, or heat != 0
    // float16 storage: 1 = stores rounded stochastically with random bits from a
    // hash of (node, population, sr_seed), sr_seed a hash of the step number;
    // 0 = rounded to nearest
    int32_t sr;
    uint32_t sr_seed;
    FastDiv div_nx;        // division by nx (flat launches)
    double lorentz;        // 2D lattices: s of the velocity-dependent x-force -s u_x (0: none)
};
constexpr int kWallTable = 16;

// Relaxation rates and time factors of a step in the arithmetic type.
template <class Real>
struct NodeRates {
    Real rho0, shear, bulk, third, fourth, phi, phi_high, lorentz;
    Real f_pre, f_tot, s_pre, s_tot, heat;
};

template <class Real>
#ifdef __HIPCC__
__host__ __device__
#endif
inline NodeRates<Real> node_rates(const StepArgs& a) {
    return {Real(a.rho0), Real(a.w_shear), Real(a.w_bulk), Real(a.w_third), Real(a.w_fourth), Real(a.w_phi),
            Real(a.w_phi_high), Real(a.lorentz), Real(a.f_pre), Real(a.f_tot), Real(a.s_pre), Real(a.s_tot),
            Real(a.heat)};
}

// Several steps of a 2D lattice per launch (casclb_multistep).
constexpr int kMultiMaxSteps = 16;

// Tiling of one slice: a workgroup of `block` threads owns tx x ty nodes and
// steps the region w x h = (tx + 2 hx) x (ty + 2 hy) <= block around them, the
// halo hx, hy being steps - 1 nodes, or 0 on an axis the tile covers whole.
struct MultiShape {
    int32_t tx, ty, hx, hy, w, h, steps, block;
    uint32_t tiles, per_slice, tiles_x;   // workgroups in all, per slice and along x
    FastDiv div_w, div_per_slice, div_tiles_x;
};

struct MultiArgs {
    StepArgs step;               // src, dst, fields and settings; the factors of the first step
    MultiShape shape;
    NodeRates<float> rates32;    // the step's rates in the arithmetic type
    NodeRates<double> rates64;
    int32_t varying;             // 1: factors[s] = f_pre, f_tot, s_pre, s_tot of step s
    double factors[kMultiMaxSteps][4];
    uint32_t seeds[kMultiMaxSteps];   // stochastic rounding: sr_seed of step s
};

}  // namespace casclb
