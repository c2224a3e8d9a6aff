// One step of a 3D lattice whose rows do not fit the row kernels' blocks
// (D3Q27, D3Q15): threads take consecutive nodes of the flat index, whatever
// row they fall in.
//
// The row kernels (kernels.hip) give every wavefront 64 nodes of one row, so
// that coordinates and walls are scalar; rows shorter than 64 nodes leave lanes
// idle, and rows that are not whole 128-byte lines make every wave's stores end
// in partial lines.  Here every wave stores 64 consecutive nodes (lines are
// whole), and coordinates, wraps and walls are per lane: about 100 vector
// instructions more per node, which these memory-bound kernels have room for.
// Addresses are 32-bit byte offsets from the buffer (the host checks they fit).
// Bound by HBM: 250 x 203 x 190 float32 379 us per step (5.5 TB/s of algorithmic
// traffic, 69% of 8 TB/s; 538 us by rows), float64 747 (922), float16 205 (328);
// 3 x 45 x 45, a launch's latency, 4.3 us (11.9).  Ordinary loads: a wave's
// shifted load shares its first and last line with the neighbouring waves, and
// keeping them in L2 beats non-temporal loads (float32 379 against 418 us);
// giving each XCD a contiguous range of nodes is slower (420 us).
// The arithmetic per node is that of the row kernels: results are bit-identical.
#include <hip/hip_runtime.h>
#include <math.h>

#include "common.hpp"
#include "kernels.hpp"
#include "lattice.hpp"
#include "node.hpp"

#pragma clang fp contract(on)   // see node.hpp

namespace casclb {

namespace {

// Position of flat node n and its neighbours: x offsets and row offsets (in
// nodes) of the three values along each axis, wrapped periodically; index 0, 1,
// 2 for velocity component 0, +1 (source at the lower neighbour), -1.
struct FlatPos {
    RowPos p;
    uint32_t node;
    uint32_t xs[3], ys[3], zs[3];   // source x; y * nx; z * nx * ny
    bool wall[3][3];                // [axis][1 or 2]: that source lies in a wall
};

__device__ __forceinline__ void axis_sources(uint32_t c, uint32_t n, uint32_t scale, bool walls, uint32_t (&s)[3],
                                             bool (&wall)[3]) {
    s[0] = c * scale;
    s[1] = (c == 0 ? n - 1 : c - 1) * scale;
    s[2] = (c == n - 1 ? 0 : c + 1) * scale;
    wall[0] = false;
    wall[1] = walls && c == 0;
    wall[2] = walls && c == n - 1;
}

__device__ __forceinline__ FlatPos flat_position(const StepArgs& a, uint32_t n, bool active) {
    const Geometry& g = a.geo;
    FlatPos f;
    const uint32_t row = a.div_nx.div(n), x = n - row * (uint32_t)g.nx;
    const uint32_t z = g.div_ny.div(row), y = row - z * (uint32_t)g.ny;
    axis_sources(x, (uint32_t)g.nx, 1, g.bb[0], f.xs, f.wall[0]);
    axis_sources(y, (uint32_t)g.ny, (uint32_t)g.nx, g.bb[1], f.ys, f.wall[1]);
    axis_sources(z, (uint32_t)g.nz, (uint32_t)(g.nx * g.ny), g.bb[2], f.zs, f.wall[2]);
    f.node = n;
    f.p.x = x;
    f.p.xm = f.xs[1];
    f.p.xp = f.xs[2];
    f.p.y = (int)y;
    f.p.z = (int)z;
    f.p.row = (int64_t)(row * (uint32_t)g.nx);
    f.p.node = n;
    f.p.active = active;
    return f;
}

// Logical block of this workgroup: with xcd_remap each of the 8 XCDs, to which
// workgroups go round-robin, takes a contiguous range (the grid is then rounded
// up to a multiple of 8 and the surplus returns).
__device__ __forceinline__ uint32_t flat_block(const Geometry& g) {
    const uint32_t b = blockIdx.x;
    return g.xcd_remap ? (b & 7u) * (gridDim.x >> 3) + (b >> 3) : b;
}

__host__ __device__ constexpr int side(int e) { return e == 0 ? 0 : (e > 0 ? 1 : 2); }

template <class T>
__device__ __forceinline__ T load_at(const void* base, uint32_t byte_offset) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + byte_offset);
}

template <int LAT, class Real, class Store, bool DIAG, bool SR>
__global__ void __launch_bounds__(kMaxBlock) casclb_step_flat(const StepArgs a) {
    constexpr int Q = Lat<LAT>::Q;
    constexpr int D = Lat<LAT>::D;
    constexpr uint32_t E = sizeof(Store);
    const Geometry& g = a.geo;
    const uint32_t lb = flat_block(g), total = (uint32_t)g.nx * (uint32_t)g.nrows;
    if (lb >= (uint32_t)g.grid_blocks) return;
    const uint32_t n = lb * blockDim.x + threadIdx.x;
    const FlatPos f = flat_position(a, n < total ? n : total - 1, n < total);
    const uint32_t plane = (uint32_t)g.plane;
    Store raw[Q], raw_sc[5];
    static_for<Q>([&](auto aa) {
        constexpr int A = decltype(aa)::value;
        constexpr int X = side(Lat<LAT>::velocity(A, 0)), Y = side(Lat<LAT>::velocity(A, 1)),
                      Z = side(Lat<LAT>::velocity(A, 2));
        constexpr int slot = LAT == kD3Q15 ? A : Flow<D>::grid_of(A);
        uint32_t src = (uint32_t)A * plane + f.xs[X] + f.ys[Y] + f.zs[Z];
        if constexpr (X || Y || Z) {
            const bool wall = f.wall[0][X] || f.wall[1][Y] || f.wall[2][Z];
            src = wall ? (uint32_t)Lat<LAT>::opposite(A) * plane + f.node : src;
        }
        raw[slot] = load_at<Store>(a.src, src * E);
    });
    double v[kDiagSlots] = {};
    Real m[Q], sc[5];
    collide_node<LAT, Real, Store, DIAG>(a, f.p, raw, raw_sc, v, m, sc);
    if (f.p.active) {
        char* out = reinterpret_cast<char*>(a.dst) + f.node * E;
        const uint32_t key = SR ? sr_node_key(a, f.p) : 0u;
        static_for<Q>([&](auto aa) {
            constexpr int A = decltype(aa)::value;
            constexpr int slot = LAT == kD3Q15 ? A : Flow<D>::grid_of(A);
            Store* to = reinterpret_cast<Store*>(out + (int64_t)A * g.plane * E);
            if constexpr (SR) st_stream(to, half_sr(m[slot], key + sr_salt(A)));
            else st_stream(to, to_store<Store>(m[slot]));
        });
    }
    if constexpr (DIAG) block_sum(v, a.partials + (int64_t)lb * kDiagSlots);
}

// Two x-adjacent nodes 2t, 2t + 1 per thread in 16-bit storage (even nx, x
// periodic, even plane stride), read and written as 32-bit words as in
// casclb_step_xpair.
template <int LAT, bool DIAG, bool SR>
__global__ void __launch_bounds__(kMaxBlock) casclb_step_flat_pair(const StepArgs a) {
    using Real = float;
    using Store = _Float16;
    constexpr int Q = Lat<LAT>::Q;
    constexpr int D = Lat<LAT>::D;
    const Geometry& g = a.geo;
    const uint32_t lb = flat_block(g), total = ((uint32_t)g.nx >> 1) * (uint32_t)g.nrows;
    if (lb >= (uint32_t)g.grid_blocks) return;
    const uint32_t t = lb * blockDim.x + threadIdx.x;
    const bool active = t < total;
    const uint32_t word = active ? t : total - 1;
    const FlatPos f = flat_position(a, 2 * word, active);
    RowPos p1 = f.p;
    p1.x += 1;
    p1.xm = f.p.x;
    p1.xp = p1.x == (uint32_t)g.nx - 1 ? 0 : p1.x + 1;
    p1.node += 1;
    const uint32_t half_plane = (uint32_t)(g.plane >> 1), words = (uint32_t)g.nx >> 1;
    const uint32_t w0 = f.p.x >> 1, wm = w0 == 0 ? words - 1 : w0 - 1, wp = w0 == words - 1 ? 0 : w0 + 1;
    Store raw0[Q], raw1[Q], raw_sc[5];
    static_for<Q>([&](auto aa) {
        constexpr int A = decltype(aa)::value;
        constexpr int X = side(Lat<LAT>::velocity(A, 0)), Y = side(Lat<LAT>::velocity(A, 1)),
                      Z = side(Lat<LAT>::velocity(A, 2));
        constexpr int slot = LAT == kD3Q15 ? A : Flow<D>::grid_of(A);
        const bool wall = f.wall[1][Y] || f.wall[2][Z];
        const uint32_t row = (uint32_t)A * half_plane + ((f.ys[Y] + f.zs[Z]) >> 1);   // rows hold an even number of nodes
        const uint32_t own = (uint32_t)Lat<LAT>::opposite(A) * half_plane + word;
        const bool w = (Y || Z) && wall;
        if constexpr (X == 0) {
            const uint32_t v = load_at<uint32_t>(a.src, (w ? own : row + w0) * 4u);
            raw0[slot] = half_lo(v);
            raw1[slot] = half_hi(v);
        } else {
            // e_x = +1: nodes 2t - 1, 2t; e_x = -1: 2t + 1, 2t + 2; at a wall both nodes' own
            const uint32_t va = load_at<uint32_t>(a.src, (w ? own : row + (X == 1 ? wm : w0)) * 4u);
            const uint32_t vb = load_at<uint32_t>(a.src, (w ? own : row + (X == 1 ? w0 : wp)) * 4u);
            raw0[slot] = w ? half_lo(va) : half_hi(va);
            raw1[slot] = w ? half_hi(vb) : half_lo(vb);
        }
    });
    double v[kDiagSlots] = {};
    Real m0[Q], m1[Q], sc[5];
    collide_node<LAT, Real, Store, DIAG>(a, f.p, raw0, raw_sc, v, m0, sc);
    collide_node<LAT, Real, Store, DIAG>(a, p1, raw1, raw_sc, v, m1, sc);
    if (active) {
        uint32_t* out = reinterpret_cast<uint32_t*>(a.dst) + word;
        const uint32_t key0 = SR ? sr_node_key(a, f.p) : 0u, key1 = SR ? sr_node_key(a, p1) : 0u;
        static_for<Q>([&](auto aa) {
            constexpr int A = decltype(aa)::value;
            constexpr int slot = LAT == kD3Q15 ? A : Flow<D>::grid_of(A);
            uint32_t* to = out + (int64_t)A * half_plane;
            if constexpr (SR) st_stream(to, pack_halves_sr(m0[slot], m1[slot], key0 + sr_salt(A), key1 + sr_salt(A)));
            else st_stream(to, pack_halves(m0[slot], m1[slot]));
        });
    }
    if constexpr (DIAG) block_sum(v, a.partials + (int64_t)lb * kDiagSlots);
}

template <int LAT, class Real, class Store, bool SR>
hipError_t launch_flat_r(const StepArgs& a, int block, bool diag, hipStream_t s) {
    const int64_t blocks = a.geo.xcd_remap ? (a.geo.grid_blocks + 7) / 8 * 8 : a.geo.grid_blocks;
    const dim3 grid((unsigned)blocks), blk((unsigned)block);
    if constexpr (sizeof(Store) == 2) {
        if (a.geo.xpair) {
            if (diag) hipLaunchKernelGGL((casclb_step_flat_pair<LAT, true, SR>), grid, blk, 0, s, a);
            else hipLaunchKernelGGL((casclb_step_flat_pair<LAT, false, SR>), grid, blk, 0, s, a);
            return hipGetLastError();
        }
    }
    if (diag) hipLaunchKernelGGL((casclb_step_flat<LAT, Real, Store, true, SR>), grid, blk, 0, s, a);
    else hipLaunchKernelGGL((casclb_step_flat<LAT, Real, Store, false, SR>), grid, blk, 0, s, a);
    return hipGetLastError();
}

template <int LAT>
hipError_t launch_flat_t(int storage, const StepArgs& a, int block, bool diag, hipStream_t s) {
    switch (storage) {
        case kF64: return launch_flat_r<LAT, double, double, false>(a, block, diag, s);
        case kF32Dev: return launch_flat_r<LAT, float, float, false>(a, block, diag, s);
        case kF16Dev:
            return a.sr ? launch_flat_r<LAT, float, _Float16, true>(a, block, diag, s)
                        : launch_flat_r<LAT, float, _Float16, false>(a, block, diag, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_step_flat(int lat, int storage, const StepArgs& a, int block, bool diag, hipStream_t s) {
    if (lat == kD3Q27) return launch_flat_t<kD3Q27>(storage, a, block, diag, s);
    if (lat == kD3Q15) return launch_flat_t<kD3Q15>(storage, a, block, diag, s);
    return hipErrorInvalidValue;
}

}  // namespace casclb
