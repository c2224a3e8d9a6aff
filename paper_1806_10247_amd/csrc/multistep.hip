// Several steps of a 2D lattice per launch (D2Q9, D2Q9 + D2Q5).
//
// One step per launch costs a small lattice the launch and one round trip to
// memory per step, and a large one a read and a write of every population per
// step.  Here a workgroup owns a tile of nodes with a halo of K - 1 nodes: the
// first of K steps pulls the tile and halo from global memory, the states
// between steps live in LDS, and the last step writes the tile; after step s
// the nodes at least s away from the edge of the region are valid, so the halo
// is recomputed, not exchanged.  A thread keeps the same node for all K steps:
// its LDS source addresses (periodic wraps and wall reflections included), its
// force and its source are formed once.  An axis the tile covers whole needs no
// halo; a lattice that fits one tile runs all its steps on chip.
//
// The arithmetic per node is that of the one-step kernels (collide_values), so
// results are bit-identical to stepping one launch at a time.
//
// What bounds it: a small lattice its launch and the chain of one node's step
// (about 0.6 us a step at one wavefront per SIMD: 230 vector instructions, two
// barriers, one LDS round trip), a large one vector issue, the halo's share
// included.  Plain loads and stores: the halo is read by up to four workgroups,
// and a tile's row ends are completed in L2 by the neighbouring tile.  Measured
// (MI355X, us per step, one step per launch -> this kernel): D2Q9 4 x 64 float64
// 3.46 -> 0.64; D2Q9 + D2Q5 float32 64^2 3.27 -> 1.27, 256^2 4.3 -> 2.2, 4096^2
// 356 -> 168 (42 -> 99 billion node updates per second); float64 1531 x 1021
// 79.6 -> 36, 4096^2 784 -> 356; float16 4096^2 216 -> 159; D2Q9 2000^2 float32
// 58 -> 29.
#include <hip/hip_runtime.h>
#include <math.h>

#include "common.hpp"
#include "kernels.hpp"
#include "lattice.hpp"
#include "node.hpp"

#pragma clang fp contract(on)   // see node.hpp

namespace casclb {

namespace {

template <class T>
__device__ __forceinline__ T load_at(const void* base, uint32_t byte_offset) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + byte_offset);
}

template <int LAT, class Real, class Store, bool EXT, bool SR, int BLOCK>
__global__ void __launch_bounds__(BLOCK) casclb_multistep(const MultiArgs ma) {
    constexpr int Q = Lat<LAT>::Q;
    constexpr int QS = LAT == kD2Q9D2Q5 ? 5 : 0;
    constexpr uint32_t E = sizeof(Store);
    extern __shared__ __align__(16) unsigned char lds_raw[];
    Store* lds = reinterpret_cast<Store*>(lds_raw);   // [Q + QS][BLOCK]
    const StepArgs& a = ma.step;
    const Geometry& g = a.geo;
    const MultiShape& t = ma.shape;
    const int l = (int)threadIdx.x;
    const bool in_region = l < t.w * t.h;
    const int lc = in_region ? l : 0;
    const int ly = (int)t.div_w.div((uint32_t)lc), lx = lc - ly * t.w;
    // each of the 8 XCDs takes a contiguous range of tiles: neighbours share its L2
    const uint32_t b = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (b >= t.tiles) return;   // the grid is rounded up to a multiple of 8
    const uint32_t slice = t.div_per_slice.div(b), in_slice = b - slice * t.per_slice;
    const uint32_t tyi = t.div_tiles_x.div(in_slice), txi = in_slice - tyi * t.tiles_x;
    const int rx = (int)txi * t.tx - t.hx + lx, ry = (int)tyi * t.ty - t.hy + ly;   // unwrapped coordinates
    const bool out_x = rx < 0 || rx >= g.nx, out_y = ry < 0 || ry >= g.ny;
    const bool exists = in_region && !(out_x && g.bb[0]) && !(out_y && g.bb[1]);
    // steps after which the node's value is still valid: its distance from the region's edge on cut axes
    const int dx = t.hx == 0 ? t.steps : min(lx, t.w - 1 - lx), dy = t.hy == 0 ? t.steps : min(ly, t.h - 1 - ly);
    const int valid = exists ? min(dx, dy) : -1;
    const bool owned = exists && !out_x && !out_y && valid >= t.steps - 1;
    auto wrapped = [](int v, int n) {   // -n <= v < 3n
        v = v < 0 ? v + n : v;
        v = v >= n ? v - n : v;
        return v >= n ? v - n : v;
    };
    RowPos p;
    const int x = exists ? wrapped(rx, g.nx) : 0, y = exists ? wrapped(ry, g.ny) : 0;
    p.x = (uint32_t)x;
    p.xm = (uint32_t)(x == 0 ? g.nx - 1 : x - 1);
    p.xp = (uint32_t)(x == g.nx - 1 ? 0 : x + 1);
    p.y = y;
    p.z = (int)slice;
    p.active = owned;
    const uint32_t slice_row = slice * (uint32_t)g.ny;
    const uint32_t row = (slice_row + (uint32_t)y) * (uint32_t)g.nx;
    const uint32_t rowm = (slice_row + (uint32_t)(y == 0 ? g.ny - 1 : y - 1)) * (uint32_t)g.nx;
    const uint32_t rowp = (slice_row + (uint32_t)(y == g.ny - 1 ? 0 : y + 1)) * (uint32_t)g.nx;
    p.row = row;
    p.node = row + p.x;
    const uint32_t node = row + p.x, plane = (uint32_t)g.plane;

    // a link whose source lies in a wall returns the opposite population of the node itself
    auto blocked = [&](int ex, int ey) {
        return (g.bb[0] && (x - ex < 0 || x - ex >= g.nx)) || (g.bb[1] && (y - ey < 0 || y - ey >= g.ny));
    };
    // ---- first step: pull from global memory
    Real m[Q], sc[5];
    uint32_t from[Q + QS];   // LDS element each population is pulled from in the later steps
    auto neighbour = [&](int ex, int ey) {   // LDS index of the node at (x - ex, y - ey)
        int nx = lx - ex, ny = ly - ey;
        nx = nx < 0 ? nx + t.w : (nx >= t.w ? nx - t.w : nx);
        ny = ny < 0 ? ny + t.h : (ny >= t.h ? ny - t.h : ny);
        return (uint32_t)(nx + ny * t.w);
    };
    Store raw[Q + QS];
    static_for<Q + QS>([&](auto aa) {
        constexpr int A = decltype(aa)::value;
        constexpr int EX = A < Q ? Flow<2>::velocity(A < Q ? A : 0, 0) : d2q5_velocity(A < Q ? 0 : A - Q, 0);
        constexpr int EY = A < Q ? Flow<2>::velocity(A < Q ? A : 0, 1) : d2q5_velocity(A < Q ? 0 : A - Q, 1);
        constexpr int OPP = A < Q ? Flow<2>::opposite(A < Q ? A : 0) : Q + d2q5_opposite(A < Q ? 0 : A - Q);
        const uint32_t sx = EX == 0 ? p.x : (EX > 0 ? p.xm : p.xp);
        const uint32_t sr = EY == 0 ? row : (EY > 0 ? rowm : rowp);
        uint32_t src = (uint32_t)A * plane + sr + sx;
        from[A] = (uint32_t)(A * BLOCK) + neighbour(EX, EY);
        if constexpr (EX != 0 || EY != 0) {
            const bool wall = blocked(EX, EY);
            src = wall ? (uint32_t)OPP * plane + node : src;
            from[A] = wall ? (uint32_t)(OPP * BLOCK + l) : from[A];
        }
        raw[A] = load_at<Store>(a.src, src * E);
    });
    Real fb[3] = {Real(a.fx), Real(a.fy), Real(0)}, sb = Real(a.source);
    if (a.force_field) {
        fb[0] = load_at<Real>(a.force_field, node * (uint32_t)sizeof(Real));
        fb[1] = load_at<Real>(a.force_field, (plane + node) * (uint32_t)sizeof(Real));
    }
    if constexpr (QS > 0)
        if (a.source_field) sb = load_at<Real>(a.source_field, node * (uint32_t)sizeof(Real));
    for (int s = 0;; ++s) {
        static_for<Q>([&](auto aa) {
            constexpr int A = decltype(aa)::value;
            m[Flow<2>::grid_of(A)] = to_real<Real>(raw[A]);
        });
        if constexpr (QS > 0)
            static_for<5>([&](auto aa) {
                constexpr int A = decltype(aa)::value;
                sc[A] = to_real<Real>(raw[Q + A]);
            });
        NodeRates<Real> k;
        if constexpr (sizeof(Real) == 8) k = ma.rates64;
        else k = ma.rates32;
        if (ma.varying) {
            k.f_pre = Real(ma.factors[s][0]);
            k.f_tot = Real(ma.factors[s][1]);
            k.s_pre = Real(ma.factors[s][2]);
            k.s_tot = Real(ma.factors[s][3]);
        }
        const Real fs[3] = {pinned(fb[0]), pinned(fb[1]), Real(0)}, ss = pinned(sb);
        NodeResult<Real> r;
        collide_values<LAT, Real, EXT>(a, k, p, fs, [&] { return ss; }, m, sc, r);
        // the stored values, as the one-step kernels store them
        if constexpr (SR) {
            const uint32_t key = mix32(((uint32_t)p.node * 0x9E3779B1u) ^ ma.seeds[s]);
            static_for<Q + QS>([&](auto aa) {
                constexpr int A = decltype(aa)::value;
                raw[A] = half_sr(A < Q ? m[Flow<2>::grid_of(A < Q ? A : 0)] : sc[A < Q ? 0 : A - Q], key + sr_salt(A));
            });
        } else {
            static_for<Q + QS>([&](auto aa) {
                constexpr int A = decltype(aa)::value;
                raw[A] = to_store<Store>(A < Q ? m[Flow<2>::grid_of(A < Q ? A : 0)] : sc[A < Q ? 0 : A - Q]);
            });
        }
        if (s == t.steps - 1) break;
        // ---- exchange through LDS
        if (valid >= s)
            static_for<Q + QS>([&](auto aa) {
                constexpr int A = decltype(aa)::value;
                lds[A * BLOCK + l] = raw[A];
            });
        __syncthreads();
        static_for<Q + QS>([&](auto aa) {
            constexpr int A = decltype(aa)::value;
            raw[A] = lds[from[A]];
        });
        __syncthreads();
    }
    if (owned)
        static_for<Q + QS>([&](auto aa) {
            constexpr int A = decltype(aa)::value;
            *reinterpret_cast<Store*>(reinterpret_cast<char*>(a.dst) + ((uint32_t)A * plane + node) * E) = raw[A];
        });
}

template <int LAT, class Real, class Store, bool EXT, bool SR, int BLOCK>
hipError_t launch_b(const MultiArgs& a, hipStream_t s) {
    constexpr size_t lds = (size_t)(Lat<LAT>::Q + (LAT == kD2Q9D2Q5 ? 5 : 0)) * BLOCK * sizeof(Store);
    if constexpr (lds > 65536) {   // above the default dynamic LDS limit
        const hipError_t e = hipFuncSetAttribute((const void*)casclb_multistep<LAT, Real, Store, EXT, SR, BLOCK>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((casclb_multistep<LAT, Real, Store, EXT, SR, BLOCK>), dim3((a.shape.tiles + 7) / 8 * 8), dim3(BLOCK), lds, s,
                       a);
    return hipGetLastError();
}

template <int LAT, class Real, class Store, bool EXT, bool SR>
hipError_t launch_r(const MultiArgs& a, hipStream_t s) {
    switch (a.shape.block) {
        case 256: return launch_b<LAT, Real, Store, EXT, SR, 256>(a, s);
        case 512: return launch_b<LAT, Real, Store, EXT, SR, 512>(a, s);
        case 1024: return launch_b<LAT, Real, Store, EXT, SR, 1024>(a, s);
    }
    return hipErrorInvalidValue;
}

template <int LAT, class Real, class Store>
hipError_t launch_t(const MultiArgs& a, hipStream_t s) {
    if constexpr (sizeof(Store) == 2) {
        if (a.step.sr)
            return a.step.ext ? launch_r<LAT, Real, Store, true, true>(a, s) : launch_r<LAT, Real, Store, false, true>(a, s);
    }
    return a.step.ext ? launch_r<LAT, Real, Store, true, false>(a, s) : launch_r<LAT, Real, Store, false, false>(a, s);
}

}  // namespace

hipError_t launch_multistep(int lat, int storage, const MultiArgs& a, hipStream_t s) {
    switch (lat * 3 + storage) {
        case kD2Q9 * 3 + kF64: return launch_t<kD2Q9, double, double>(a, s);
        case kD2Q9 * 3 + kF32Dev: return launch_t<kD2Q9, float, float>(a, s);
        case kD2Q9 * 3 + kF16Dev: return launch_t<kD2Q9, float, _Float16>(a, s);
        case kD2Q9D2Q5 * 3 + kF64: return launch_t<kD2Q9D2Q5, double, double>(a, s);
        case kD2Q9D2Q5 * 3 + kF32Dev: return launch_t<kD2Q9D2Q5, float, float>(a, s);
        case kD2Q9D2Q5 * 3 + kF16Dev: return launch_t<kD2Q9D2Q5, float, _Float16>(a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace casclb
