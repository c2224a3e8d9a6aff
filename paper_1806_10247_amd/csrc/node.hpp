// Device code of one lattice node shared by the step kernels: streaming loads,
// the pull with its wall rules, the force and source of the node, and the
// collision with both half steps.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "common.hpp"
#include "lattice.hpp"

// Multiply-adds are fused only within one source expression.  With fusion
// across statements the backend decides per basic block, so the kernel
// variants of one lattice (rows or x-adjacent nodes per thread, residual
// steps) would round differently; this way every launch shape gives
// bit-identical results.
#pragma clang fp contract(on)

namespace casclb {

template <class T>
__device__ __forceinline__ T ld_stream(const T* p) {
    return __builtin_nontemporal_load(p);
}
template <class T>
__device__ __forceinline__ void st_stream(T* p, T v) {
    __builtin_nontemporal_store(v, p);
}

template <class Real, class Store>
__device__ __forceinline__ Real to_real(Store v) {
    return static_cast<Real>(v);
}
template <class Store, class Real>
__device__ __forceinline__ Store to_store(Real v) {
    return static_cast<Store>(v);
}

// ---------------------------------------------------------------------------
// float16 storage with stochastic rounding
// ---------------------------------------------------------------------------
// The per-step force kick F.e/<e_x|e_x> of a weakly forced lattice (5.6e-9 on
// D3Q27 at F = 1e-7) lies far below half a float16 unit of the stored
// deviations (the smallest subnormal is 6e-8), so rounding to nearest drops it
// at every store and a lattice started from rest never moves.  Stochastic
// rounding takes the float16 neighbour above or below with probabilities in
// proportion to the distances, so the expected stored value is the float32
// value and the kicks survive on average.  The random bits come from a
// counter-based hash of (node, population, step), so every launch shape gives
// the same result.
__device__ __forceinline__ uint32_t mix32(uint32_t x) {
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

// Per-population salt added to a node's key (distinct odd multiples of the
// 32-bit golden ratio): over the nodes every bit of key + salt stays uniform.
__device__ __forceinline__ constexpr uint32_t sr_salt(int plane) { return (uint32_t)(plane + 1) * 0x9E3779B9u; }

// float32 -> float16 with stochastic rounding in one instruction
// (v_cvt_sr_f16_f32): the neighbour above or below with probabilities in
// proportion to the distances, the random 32 bits r choosing; exact on
// float16 values, subnormals included (spacing 2^-24).  The pair form packs
// two (low, high) into one word.
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_halves_sr(float lo, float hi, uint32_t rlo, uint32_t rhi) {
    half2_t o = {(_Float16)0.0f, (_Float16)0.0f};
    o = __builtin_amdgcn_cvt_sr_f16_f32(o, lo, rlo, false);
    o = __builtin_amdgcn_cvt_sr_f16_f32(o, hi, rhi, true);
    return __builtin_bit_cast(uint32_t, o);
}
__device__ __forceinline__ _Float16 half_sr(float v, uint32_t r) {
    half2_t o = {(_Float16)0.0f, (_Float16)0.0f};
    o = __builtin_amdgcn_cvt_sr_f16_f32(o, v, r, false);
    return o[0];
}

__device__ __forceinline__ _Float16 half_lo(uint32_t w) { return __builtin_bit_cast(_Float16, (uint16_t)w); }
__device__ __forceinline__ _Float16 half_hi(uint32_t w) {
    return __builtin_bit_cast(_Float16, (uint16_t)(w >> 16));
}

__device__ __forceinline__ uint32_t pack_halves(float lo, float hi) {
    const uint16_t a = __builtin_bit_cast(uint16_t, static_cast<_Float16>(lo));
    const uint16_t b = __builtin_bit_cast(uint16_t, static_cast<_Float16>(hi));
    return (uint32_t)a | ((uint32_t)b << 16);
}

struct RowPos {
    int y, z;            // block-uniform
    int64_t row;         // block-uniform: nx*(y + ny*z)
    bool active;
    uint32_t x, xm, xp;  // per lane: x (clamped), x-1 and x+1 wrapped periodically
    int64_t node;        // row + x
};

__device__ __forceinline__ uint32_t logical_block(const Geometry& g) {
    const uint32_t b = blockIdx.x;
    if (g.xcd_remap) {
        // blocks are dispatched to the 8 XCDs round-robin; hand XCD k the
        // contiguous range [k*G/8, (k+1)*G/8) of logical blocks
        const uint32_t per = (uint32_t)(g.grid_blocks >> 3);
        return (b & 7u) * per + (b >> 3);
    }
    return b;
}

// Position of this thread's node in row k (0 <= k < g.rows) of the group of
// rows of logical block lb.  A row past the last one is clamped and marked
// inactive.
__device__ __forceinline__ RowPos row_position_at(const Geometry& g, uint32_t lb, int k = 0) {
    RowPos p;
    const uint32_t group = g.div_xb.div(lb);
    const int xb = (int)(lb - group * (uint32_t)g.x_blocks);
    uint32_t row = group * (uint32_t)g.rows + (uint32_t)k;
    const bool row_ok = row < (uint32_t)g.nrows;
    if (!row_ok) row = (uint32_t)g.nrows - 1;
    const uint32_t z = g.div_ny.div(row);
    p.y = (int)(row - z * (uint32_t)g.ny);
    p.z = (int)z;
    p.row = (int64_t)g.nx * row;
    const int x = xb * (int)blockDim.x + (int)threadIdx.x;
    p.active = row_ok && x < g.nx;
    const int xc = p.active ? x : g.nx - 1;
    p.x = (uint32_t)xc;
    p.xm = (uint32_t)(xc == 0 ? g.nx - 1 : xc - 1);
    p.xp = (uint32_t)(xc == g.nx - 1 ? 0 : xc + 1);
    p.node = p.row + xc;
    return p;
}

// Position of this thread's node in row k of its own block's group of rows.
__device__ __forceinline__ RowPos row_position(const Geometry& g, int k = 0) {
    return row_position_at(g, logical_block(g), k);
}

// Pull of the population in plane `plane_self` with velocity (EX, EY, EZ)
// (eq. 22b): read node x - e of the stored state, wrapped on periodic axes.
// A link whose source lies in a wall returns the opposite population
// (`plane_opp`) of the same node (halfway bounce-back).  The row part of the
// address and the y/z wall decisions are block-uniform, so each load is a
// uniform base pointer plus one of the three per-lane offsets x, x-1, x+1.
// XWALL: walls on the x axis too (then the x decision is per lane).
template <int EX, int EY, int EZ, bool XWALL, class Store>
__device__ __forceinline__ Store pull(const Store* __restrict__ src, const Geometry& g, const RowPos& p,
                                      int plane_self, int plane_opp) {
    bool wall = false;
    int sy = p.y - EY, sz = p.z - EZ;
    if constexpr (EY != 0) {
        if (sy < 0) { wall |= g.bb[1] != 0; sy += g.ny; }
        if (sy >= g.ny) { wall |= g.bb[1] != 0; sy -= g.ny; }
    }
    if constexpr (EZ != 0) {
        if (sz < 0) { wall |= g.bb[2] != 0; sz += g.nz; }
        if (sz >= g.nz) { wall |= g.bb[2] != 0; sz -= g.nz; }
    }
    const int64_t src_row = (int64_t)g.nx * ((int64_t)sy + (int64_t)g.ny * sz);
    const Store* own = src + (int64_t)plane_opp * g.plane + p.row;       // bounce-back source row
    const Store* base = wall ? own : src + (int64_t)plane_self * g.plane + src_row;
    uint32_t off = EX == 0 ? p.x : (EX > 0 ? p.xm : p.xp);
    if (wall) off = p.x;
    if constexpr (XWALL && EX != 0) {
        const bool lane_wall = g.bb[0] != 0 && (EX > 0 ? p.x == 0 : p.x == (uint32_t)g.nx - 1);
        const Store* q = lane_wall ? own + p.x : base + off;
        return ld_stream(q);
    } else {
        return ld_stream(base + off);
    }
}

template <int D, bool XWALL, class Real, class Store>
__device__ __forceinline__ void gather_flow(const Store* __restrict__ src, const Geometry& g, const RowPos& p,
                                            Real (&m)[Flow<D>::Q]) {
    static_for<Flow<D>::Q>([&](auto aa) {
        constexpr int A = decltype(aa)::value;
        constexpr int EX = Flow<D>::velocity(A, 0), EY = Flow<D>::velocity(A, 1), EZ = Flow<D>::velocity(A, 2);
        m[Flow<D>::grid_of(A)] = to_real<Real>(pull<EX, EY, EZ, XWALL>(src, g, p, A, Flow<D>::opposite(A)));
    });
}

template <bool XWALL, class Real, class Store>
__device__ __forceinline__ void gather_scalar(const Store* __restrict__ src, int first_plane, const Geometry& g,
                                              const RowPos& p, Real (&s)[5]) {
    static_for<5>([&](auto aa) {
        constexpr int A = decltype(aa)::value;
        s[A] = to_real<Real>(pull<d2q5_velocity(A, 0), d2q5_velocity(A, 1), 0, XWALL>(
            src, g, p, first_plane + A, first_plane + d2q5_opposite(A)));
    });
}

template <int D, class Real>
__device__ __forceinline__ void node_force(const StepArgs& a, const RowPos& p, Real (&fb)[3]) {
    // uniform components first, then the field (if any) replaces them; written
    // without a branch between two stores into fb, which would keep fb (and the
    // force argument) in private memory for float64
    const Real* ff = reinterpret_cast<const Real*>(a.force_field);
    const bool field = ff != nullptr;
    const int64_t off = p.row + p.x;
    const Real f0 = field ? ld_stream(ff + off) : Real(a.fx);
    const Real f1 = field ? ld_stream(ff + a.geo.plane + off) : Real(a.fy);
    Real f2 = Real(0);
    if constexpr (D == 3) f2 = field ? ld_stream(ff + 2 * a.geo.plane + off) : Real(a.fz);
    fb[0] = f0;
    fb[1] = f1;
    fb[2] = f2;
}

// ---------------------------------------------------------------------------
// per-lattice constants: dimension, populations per node, and the velocity /
// opposite of population a in the ABI order
// ---------------------------------------------------------------------------
template <int LAT>
struct Lat {
    static constexpr int D = LAT == kD2Q9 || LAT == kD2Q9D2Q5 ? 2 : 3;
    static constexpr int Q = LAT == kD3Q15 ? 15 : Flow<D>::Q;
    __device__ static constexpr int velocity(int a, int axis) {
        if constexpr (LAT == kD3Q15) return D3Q15::velocity(a, axis);
        else return Flow<D>::velocity(a, axis);
    }
    __device__ static constexpr int opposite(int a) {
        if constexpr (LAT == kD3Q15) return D3Q15::opposite(a);
        else return Flow<D>::opposite(a);
    }
};

// ---------------------------------------------------------------------------
// walls with a velocity / a fixed scalar value, viscous heating (2D lattices)
// ---------------------------------------------------------------------------
// Side crossed first (axis x, then y) by the pull of velocity (EX, EY) at p:
// 2*axis + (0 low, 1 high), or -1 when the link stays in the fluid.
template <int EX, int EY>
__device__ __forceinline__ int crossed_side(const Geometry& g, const RowPos& p) {
    int side = -1;
    if constexpr (EY != 0) {
        const int sy = p.y - EY;
        if (g.bb[1] && sy < 0) side = 2;
        if (g.bb[1] && sy >= g.ny) side = 3;
    }
    if constexpr (EX != 0) {
        const int sx = (int)p.x - EX;
        if (g.bb[0] && sx < 0) side = 0;
        if (g.bb[0] && sx >= g.nx) side = 1;
    }
    return side;
}

__device__ __forceinline__ double wall_u_of(const StepArgs& a, int side, int c) { return a.walls[2 * side + c]; }
__device__ __forceinline__ bool phi_fixed_of(const StepArgs& a, int side) { return a.walls[8 + side] != 0.0; }
__device__ __forceinline__ double phi_wall_of(const StepArgs& a, int side) { return a.walls[12 + side]; }

// Moving-wall bounce-back: a link from a wall of velocity u_w brings the
// opposite population plus 6 w_a rho0 (e_a . u_w) (m in grid order).
template <class Real>
__device__ __forceinline__ void moving_walls(const StepArgs& a, const RowPos& p, Real (&m)[9]) {
    static_for<9>([&](auto aa) {
        constexpr int A = decltype(aa)::value;
        constexpr int EX = Flow<2>::velocity(A, 0), EY = Flow<2>::velocity(A, 1);
        const int side = crossed_side<EX, EY>(a.geo, p);
        if (side >= 0) {
            const double eu = EX * wall_u_of(a, side, 0) + EY * wall_u_of(a, side, 1);
            m[Flow<2>::grid_of(A)] += Real(6.0 * rest_weight<2>(A) * a.rho0 * eu);
        }
    });
}

// S:S of the strain rate from the second raw moments (deviations kxx, kyy,
// kxy of the streamed populations) and the half-forced velocity: with
// Pi_ab = sum f e_a e_b - rho u_a u_b - rho/3 delta_ab,
// S_xy = -3 w_shear/(2 rho0) Pi_xy, S_xx - S_yy = -3 w_shear/(2 rho0)(Pi_xx - Pi_yy),
// S_xx + S_yy = -3 w_bulk/(2 rho0)(Pi_xx + Pi_yy) (Sec. 6, thermal Couette flow).
template <class Real>
__device__ __forceinline__ Real strain_rate_squared(const StepArgs& a, Real kxx, Real kyy, Real kxy, Real rho,
                                                    const Real (&u)[3]) {
    const Real drho3 = (rho - Real(a.rho0)) * Real(1.0 / 3.0);
    const Real pxx = kxx - rho * u[0] * u[0] - drho3;
    const Real pyy = kyy - rho * u[1] * u[1] - drho3;
    const Real pxy = kxy - rho * u[0] * u[1];
    const Real cs = Real(-1.5 * a.w_shear / a.rho0), cb = Real(-1.5 * a.w_bulk / a.rho0);
    const Real sxy = cs * pxy, dif = cs * (pxx - pyy), tr = cb * (pxx + pyy);
    const Real sxx = Real(0.5) * (tr + dif), syy = Real(0.5) * (tr - dif);
    return sxx * sxx + syy * syy + Real(2) * sxy * sxy;
}

// Fixed-value scalar walls (anti-bounce-back with the source the collision
// adds to every population, S_tot/5, restored on the reflected link):
// g_a = -g^p_opp(a) + phi_w (1/3 + u_w,k^2) + 2 S_tot/5, k the axis of a.
template <class Real>
__device__ __forceinline__ void scalar_walls(const StepArgs& a, const RowPos& p, Real stot, Real (&sc)[5]) {
    static_for<5>([&](auto aa) {
        constexpr int A = decltype(aa)::value;
        constexpr int EX = d2q5_velocity(A, 0), EY = d2q5_velocity(A, 1);
        if constexpr (EX != 0 || EY != 0) {
            const int side = crossed_side<EX, EY>(a.geo, p);
            if (side >= 0 && phi_fixed_of(a, side)) {
                const double uk = wall_u_of(a, side, EX != 0 ? 0 : 1);
                sc[A] = -sc[A] + Real(phi_wall_of(a, side) * (1.0 / 3.0 + uk * uk)) + Real(0.4) * stot;
            }
        }
    });
}

// A value the optimiser may not move computations on ahead of this point: the
// products with it are formed (and fused with the sums they enter) in the
// collision, as in the kernels of one step, not once outside a loop over steps.
template <class Real>
__device__ __forceinline__ Real pinned(Real v) {
    asm volatile("" : "+v"(v));
    return v;
}

// What a node's collision leaves besides its populations.
template <class Real>
struct NodeResult {
    Real rho, u[3];            // density, half-forced velocity
    Real fpre[3], ftot[3];     // force over the pre-collision half step and the whole step
    Real phi_post, phi_star;   // scalar of the written state, half-sourced scalar
};

// Collision with both half steps of one node: m (grid order, ABI order for
// D3Q15) and sc hold the streamed populations in, the ones to store out; fb
// is the node's force, source() its scalar source.
template <int LAT, class Real, bool EXT, class Source>
__device__ __forceinline__ void collide_values(const StepArgs& a, const NodeRates<Real>& k, const RowPos& p,
                                               const Real (&fb)[3], Source source, Real (&m)[Lat<LAT>::Q],
                                               Real (&sc)[5], NodeResult<Real>& r) {
    constexpr int D = Lat<LAT>::D;
    constexpr int Q = Lat<LAT>::Q;
    Real kxx = Real(0), kyy = Real(0), kxy = Real(0);
    if constexpr (EXT && D == 2) {
        moving_walls<Real>(a, p, m);
        if constexpr (LAT == kD2Q9D2Q5) {
            static_for<Q>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                constexpr int EX = grid_velocity(K, 0), EY = grid_velocity(K, 1);
                if constexpr (EX != 0) kxx += m[K];
                if constexpr (EY != 0) kyy += m[K];
                if constexpr (EX * EY != 0) kxy += Real(EX * EY) * m[K];
            });
        }
    }
    r.fpre[0] = k.f_pre * fb[0];
    r.fpre[1] = k.f_pre * fb[1];
    r.fpre[2] = k.f_pre * fb[2];
    r.ftot[0] = k.f_tot * fb[0];
    r.ftot[1] = k.f_tot * fb[1];
    r.ftot[2] = k.f_tot * fb[2];
    if constexpr (D == 2) {
        if (a.lorentz != 0.0) {
            // velocity-dependent x-force F_x - s u_x (Hartmann flow, Sec. 6) by the implicit midpoint
            // rule: rho u_x = j_x + (F_pre,x - s u_x)/2, the step's force F_x - s u_x with that u_x
            Real drho = Real(0), jx = Real(0);
            static_for<Q>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                drho += m[K];
                jx += Real(grid_velocity(K, 0)) * m[K];
            });
            const Real rho = k.rho0 + drho, sl = k.lorentz;
            const Real ux = (jx + Real(0.5) * r.fpre[0]) / (rho + Real(0.5) * sl);
            r.fpre[0] = r.fpre[0] - sl * ux;
            r.ftot[0] = r.ftot[0] - sl * ux;
        }
    }
    const FlowRates<Real> w{k.shear, k.bulk, k.third, k.fourth};
    if constexpr (LAT == kD3Q15)
        collide_d3q15<Real>(m, k.rho0, r.fpre, r.ftot, w, r.rho, r.u);   // m in ABI order
    else
        collide_flow<D, Real>(m, k.rho0, r.fpre, r.ftot, w, r.rho, r.u);

    r.phi_post = Real(0);
    r.phi_star = Real(0);
    if constexpr (LAT == kD2Q9D2Q5) {
        const Real sb = source();
        Real spre = k.s_pre * sb, stot = k.s_tot * sb;
        if constexpr (EXT) {
            const Real sr = k.heat * strain_rate_squared<Real>(a, kxx, kyy, kxy, r.rho, r.u);
            spre += sr;
            stot += sr;
            scalar_walls<Real>(a, p, stot, sc);
        }
        const ScalarRates<Real> ws{k.phi, k.phi_high};
        const Real phi_o = collide_scalar<Real>(sc, r.u, spre, stot, ws);
        r.phi_post = phi_o + stot;                  // scalar of the written state
        r.phi_star = phi_o + Real(0.5) * spre;      // half-sourced scalar (the u* analogue)
    }
}

// Collision, both half steps and (DIAG) residual terms of one node whose
// streamed populations `raw` / `raw_sc` have been loaded: m (grid order, ABI
// order for D3Q15) and sc receive the populations to store.
template <int LAT, class Real, class Store, bool DIAG, bool EXT = false>
__device__ __forceinline__ void collide_node(const StepArgs& a, const RowPos& p, const Store (&raw)[Lat<LAT>::Q],
                                             const Store (&raw_sc)[5], double (&v)[kDiagSlots],
                                             Real (&m)[Lat<LAT>::Q], Real (&sc)[5]) {
    constexpr int D = Lat<LAT>::D;
    constexpr int Q = Lat<LAT>::Q;
    const Geometry& g = a.geo;
    static_for<Q>([&](auto kk) {
        constexpr int K = decltype(kk)::value;
        m[K] = to_real<Real>(raw[K]);
    });
    if constexpr (LAT == kD2Q9D2Q5) {
        static_for<5>([&](auto kk) {
            constexpr int K = decltype(kk)::value;
            sc[K] = to_real<Real>(raw_sc[K]);
        });
    }
    Real fb[3];
    node_force<D, Real>(a, p, fb);
    NodeResult<Real> r;
    collide_values<LAT, Real, EXT>(
        a, node_rates<Real>(a), p, fb,
        [&] {
            Real sb = Real(a.source);
            if (a.source_field) sb = ld_stream(reinterpret_cast<const Real*>(a.source_field) + p.row + p.x);
            return sb;
        },
        m, sc, r);

    if constexpr (DIAG) {
        if (p.active) {
            Real* up = reinterpret_cast<Real*>(a.u_prev) + p.row;
            double du2 = 0.0, u2 = 0.0;
            bool finite = isfinite((double)r.rho);
            static_for<D>([&](auto ax) {
                constexpr int AX = decltype(ax)::value;
                Real* slot = up + (int64_t)AX * g.plane + p.x;
                const double old = (double)*slot;
                const double now = (double)r.u[AX];
                *slot = r.u[AX];
                du2 += (now - old) * (now - old);
                u2 += now * now;
                finite = finite && isfinite(now);
            });
            v[0] += du2;
            v[1] += u2;
            v[2] += (double)(r.rho - Real(a.rho0));
            // momentum of the written state: j + F_tot = rho u - F_pre/2 + F_tot
            static_for<D>([&](auto ax) {
                constexpr int AX = decltype(ax)::value;
                v[3 + AX] += (double)r.rho * (double)r.u[AX] - 0.5 * (double)r.fpre[AX] + (double)r.ftot[AX];
            });
            v[6] += (double)r.phi_post;
            if constexpr (LAT == kD2Q9D2Q5) {
                Real* slot = up + (int64_t)D * g.plane + p.x;
                const double old = (double)*slot;
                const double now = (double)r.phi_star;
                *slot = r.phi_star;
                v[8] += (now - old) * (now - old);
                v[9] += now * now;
                finite = finite && isfinite(now);
            }
            v[7] += finite ? 0.0 : 1.0;
        }
    }
}

// Random key of one node's stores in this step (stochastic rounding).
__device__ __forceinline__ uint32_t sr_node_key(const StepArgs& a, const RowPos& p) {
    return mix32(((uint32_t)p.node * 0x9E3779B1u) ^ a.sr_seed);
}

// FP64 sum over the block of kDiagSlots values; thread 0 of the block gets the result.
__device__ __forceinline__ void block_sum(double (&v)[kDiagSlots], double* out) {
    __shared__ double red[kMaxBlock / 64][kDiagSlots];
    static_for<kDiagSlots>([&](auto cc) {
        constexpr int C = decltype(cc)::value;
        double s = v[C];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        v[C] = s;
    });
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0)
        static_for<kDiagSlots>([&](auto cc) {   // compile-time indices keep v in registers
            constexpr int C = decltype(cc)::value;
            red[wave][C] = v[C];
        });
    __syncthreads();
    if (threadIdx.x < kDiagSlots) {
        double s = 0.0;
        const int nw = (blockDim.x + 63) >> 6;
        for (int w = 0; w < nw; ++w) s += red[w][threadIdx.x];
        out[threadIdx.x] = s;
    }
}

}  // namespace casclb
