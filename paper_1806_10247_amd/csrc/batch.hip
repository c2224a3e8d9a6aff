// Batched solver: thousands of independent small D2Q9 channels (x periodic,
// halfway bounce-back walls on y) with a uniform driving force F_b and the
// velocity-dependent Lorentz force -s u_x (Hartmann flow, Sec. 6), advanced
// to a steady residual by one persistent launch.
//
// Each workgroup takes domains from a work queue (one global atomic counter)
// and runs a domain to completion by itself: domains are independent, so the
// only synchronisation between time steps is a workgroup barrier.  A domain
// that fits in the workgroup's LDS is copied in once, stepped entirely in LDS (in
// place if its threads can hold what they pull, else between two buffers) and
// copied back; a larger one is stepped in its two global-memory buffers, several
// steps per sweep where LDS holds the states between them.  Every K steps the workgroup reduces the residual
// r = ||u^n - u^{n-K}|| / (K ||u^n||) of the half-forced velocity and stops
// the domain when r < tol, when u did not change at all in K steps (storage
// precision reached), at max_steps, or on a non-finite value.  Finished
// domains retire; when the queue is empty every wave of the grid exits.
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "batch.hpp"
#include "lattice.hpp"

namespace casclb {

namespace {

// Where a thread's node lies and what it pulls from: element offsets into one
// [9][n] buffer.  A link whose source lies in a wall (both y ends) returns the
// node's own opposite population; x is periodic.
struct NodePos {
    uint32_t node;
    bool lo, hi;        // next to the lower / upper wall
    uint32_t xm, xp;    // the node's index with x - 1, x + 1 (wrapped, mod 2^32)
};
__device__ __forceinline__ NodePos node_pos(uint32_t node, int x, int y, int nx, int ny) {
    return {node, y == 0, y == ny - 1, x == 0 ? node + (uint32_t)nx - 1u : node - 1u,
            x == nx - 1 ? node - (uint32_t)nx + 1u : node + 1u};
}
template <int A>
__device__ __forceinline__ uint32_t pull_index(const NodePos& p, uint32_t n, uint32_t nx) {
    constexpr int EX = Flow<2>::velocity(A, 0), EY = Flow<2>::velocity(A, 1);
    const uint32_t at = EX == 0 ? p.node : (EX > 0 ? p.xm : p.xp);
    if constexpr (EY == 0) return A * n + at;
    else return (EY > 0 ? p.lo : p.hi) ? Flow<2>::opposite(A) * n + p.node : A * n + at - EY * nx;
}

// The element at a 32-bit byte or element offset (a domain's buffer is at most 2^20 x 9 values).
template <class T>
__device__ __forceinline__ T& at_byte(T* base, uint32_t i) {
    using B = std::conditional_t<std::is_const_v<T>, const char, char>;
    return *reinterpret_cast<T*>(reinterpret_cast<B*>(base) + i);
}
template <class T>
__device__ __forceinline__ T& element(T* base, uint32_t i) {
    return at_byte(base, i * (uint32_t)sizeof(T));
}

// Implicit Lorentz half step and collision of one D2Q9 node: raw (order of eq.
// 15) holds the streamed deviations, out receives the ones to store.  Returns the
// half-forced velocity.
template <class Real, class Store>
__device__ __forceinline__ void batch_collide(const Store (&raw)[9], const BatchParams& bp, const BatchDomain& dom,
                                              Store (&out)[9], Real (&u)[3]) {
    constexpr int Q = 9;
    Real m[Q];
    static_for<Q>([&](auto aa) {
        constexpr int A = decltype(aa)::value;
        m[Flow<2>::grid_of(A)] = static_cast<Real>(raw[A]);
    });
    // implicit half step of the velocity-dependent force:
    // rho u_x = j_x + (F_b - s u_x)/2, the step's force is F_b - s u_x
    Real drho = Real(0), jx = Real(0);
    static_for<Q>([&](auto kk) {
        constexpr int K = decltype(kk)::value;
        drho += m[K];
        jx += Real(grid_velocity(K, 0)) * m[K];
    });
    const Real rho = Real(bp.rho0) + drho;
    const Real s = Real(dom.lorentz), fb = Real(dom.force_x);
    const Real ux = (jx + Real(0.5) * fb) / (rho + Real(0.5) * s);
    const Real fx = fb - s * ux;
    const Real f[3] = {fx, Real(0), Real(0)};
    const FlowRates<Real> w{Real(dom.w_shear), Real(bp.w_bulk), Real(bp.w_third), Real(bp.w_fourth)};
    Real rho_out;
    collide_flow<2, Real>(m, Real(bp.rho0), f, f, w, rho_out, u);
    static_for<Q>([&](auto aa) {
        constexpr int A = decltype(aa)::value;
        out[A] = static_cast<Store>(m[Flow<2>::grid_of(A)]);
    });
}

template <class Store>
__device__ __forceinline__ void batch_pull(const Store* src, const NodePos& p, uint32_t n, uint32_t nx, Store (&raw)[9]) {
    static_for<9>([&](auto aa) {
        constexpr int A = decltype(aa)::value;
        raw[A] = element(src, pull_index<A>(p, n, nx));
    });
}

// The same from global memory: every population plane's base is uniform (scalar
// registers), so a node's byte offsets are all the vector arithmetic: 26 instructions
// with the loop's own instead of 53.  Opposites of the links that move along y are two
// planes apart, which makes one base serve a link's source and its wall value.
template <class Store>
__device__ __forceinline__ void batch_pull_global(const Store* src, uint32_t node, uint32_t x, uint32_t n, uint32_t nx,
                                                  Store (&raw)[9]) {
    constexpr uint32_t B = sizeof(Store);
    const uint32_t at = B * node, up = B * (2u * n + nx);
    const uint32_t xm = at + (x == 0u ? B * (nx - 1u) : 0u - B), xp = at + (x == nx - 1u ? 0u - B * (nx - 1u) : B);
    const bool lo = node < nx, hi = node >= n - nx;
    static_for<9>([&](auto aa) {
        constexpr int A = decltype(aa)::value;
        constexpr int EX = Flow<2>::velocity(A, 0), EY = Flow<2>::velocity(A, 1);
        const uint32_t from = EX == 0 ? at : (EX > 0 ? xm : xp);
        if constexpr (EY == 0) {
            raw[A] = at_byte(src + A * (int64_t)n, from);
        } else if constexpr (EY > 0) {
            static_assert(Flow<2>::opposite(A) == A + 2);
            raw[A] = at_byte(src + (A * (int64_t)n - nx), lo ? at + up : from);
        } else {
            static_assert(Flow<2>::opposite(A) == A - 2);
            raw[A] = at_byte(src + (A - 2) * (int64_t)n, hi ? at : from + up);
        }
    });
}

// One D2Q9 node of one domain from `src` to `dst` ([9][n] deviations).
template <class Real, class Store>
__device__ __forceinline__ void batch_node(const Store* src, Store* dst, int n, int nx, int ny, int x, int y,
                                           const BatchParams& bp, const BatchDomain& dom, Real (&u)[3]) {
    const uint32_t node = (uint32_t)(x + nx * y);
    Store raw[9], out[9];
    batch_pull(src, node_pos(node, x, y, nx, ny), (uint32_t)n, (uint32_t)nx, raw);
    batch_collide<Real, Store>(raw, bp, dom, out, u);
    static_for<9>([&](auto aa) {
        constexpr int A = decltype(aa)::value;
        element(dst, (uint32_t)A * (uint32_t)n + node) = out[A];
    });
}

// FP64 workgroup sum of two values; every thread gets the result.
__device__ __forceinline__ void wg_sum2(double& a, double& b, double* red) {
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off, 64);
        b += __shfl_xor(b, off, 64);
    }
    // every lane of a wave holds the wave's sums after the butterfly; all of
    // them store it (same value, same address): no lane-divergent branch in a
    // loop that contains barriers
    const int wave = threadIdx.x >> 6;
    __syncthreads();
    red[2 * wave] = a;
    red[2 * wave + 1] = b;
    __syncthreads();
    a = 0.0;
    b = 0.0;
    const int nw = (blockDim.x + 63) >> 6;
    for (int w = 0; w < nw; ++w) {
        a += red[2 * w];
        b += red[2 * w + 1];
    }
}

// A node's share of the residual check.
struct CheckSums {
    double du2 = 0.0, u2 = 0.0;
    bool finite = true;
    template <class Real>
    __device__ __forceinline__ void add(const Real (&u)[3], Real* uprev, uint32_t node, uint32_t n) {
        const double ux = (double)u[0], uy = (double)u[1];
        const double ox = (double)uprev[node], oy = (double)uprev[n + node];
        uprev[node] = u[0];
        uprev[n + node] = u[1];
        du2 += (ux - ox) * (ux - ox) + (uy - oy) * (uy - oy);
        u2 += ux * ux + uy * uy;
        finite = finite && isfinite(ux) && isfinite(uy);
    }
};

// The stop decision after a check step (0: go on), from every thread's sums.
__device__ __forceinline__ int check_stop(CheckSums c, bool& have_prev, double& res, const BatchParams& bp, double* red) {
    double bad = c.finite ? 0.0 : 1.0, unused = 0.0;
    wg_sum2(c.du2, c.u2, red);
    wg_sum2(bad, unused, red + 64);
    int stop = 0;
    if (bad > 0.0) {
        stop = kBatchNonFinite;
    } else if (have_prev) {
        res = sqrt(c.du2) / ((double)bp.check_interval * sqrt(c.u2));
        if (c.du2 == 0.0)
            stop = kBatchStationary;
        else if (res < bp.tol)
            stop = kBatchConverged;
    }
    have_prev = true;
    // Every lane holds the same sums; broadcasting the decision from lane 0
    // makes the loop exit a scalar branch.  Left as a per-lane value the
    // compiler may build an exec-mask loop around the barriers that re-runs
    // without the work-queue atomic of the enclosing loop (a hang).
    return __builtin_amdgcn_readfirstlane(stop);
}

template <class T>
using LdsPtr = __attribute__((address_space(3))) T*;
__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return (uint32_t)(uintptr_t)(LdsPtr<const char>)reinterpret_cast<const char*>(p);
}
template <class T>
__device__ __forceinline__ LdsPtr<T> lds_pointer(uint32_t address) {
    return (LdsPtr<T>)(uintptr_t)address;
}

constexpr uint32_t kNoRings = 0xffffffffu;

// Byte address in the ring plane at `base` of a byte offset.  Float rings start at a
// multiple of the plane's size (batch_ring_align), so the base is or-ed in: one
// instruction (a later step's vector instructions per node 233 -> 205-214, 5.0 -> 4.8 ms below).
template <class Store>
__device__ __forceinline__ uint32_t ring_address(uint32_t offset, uint32_t base) {
    constexpr uint32_t MB = kBatchRing * sizeof(Store) - 1;
    uint32_t a = sizeof(Store) == 4 ? (offset & MB) | base : (offset & MB) + base;
    asm("" : "+v"(a));   // planes as immediate offsets of one address, not an address each
    return a;
}

// batch_fused steps of a domain in global memory in one sweep over it, the states
// between them in LDS rings.  Step k of the sweep is 2 nx nodes behind step k - 1, whose
// last kBatchRing nodes its ring holds: a pull reaches at most 2 nx - 1 nodes (a row and
// the wrap along x), so blockDim.x + 4 nx nodes must fit.  Every node is stepped
// once, so one read and one write of the state serve all the steps; the same
// arithmetic on the same values as one step at a time.  One barrier between a step and the
// next covers both hazards from three steps on: a ring is overwritten two barriers after
// it was read; with two steps one more is needed.
//
// One step at a time, 256 workgroups' domains overflow the caches and run at the memory's
// rate: 512 float domains of 4-64 x 16-256 nodes, 200 steps, 6.8 ms = 5 TB/s.  In
// sweeps 4.8 ms, of which the largest domain (16,384 nodes, started first) takes 4.5 on its
// CU, bound by vector arithmetic.  129 such domains, whose states the caches hold: 3.9 ms
// either way; 149 double ones: 7.0 and 5.6.
template <class Real, class Store>
__device__ __forceinline__ void batch_sweep(const Store* cur, Store* nxt, uint32_t rings, uint32_t x, uint32_t n, uint32_t nx,
                                            const BatchParams& bp, const BatchDomain& dom) {
    constexpr uint32_t T = batch_fused<Real>, B = sizeof(Store), P = kBatchRing * B, two = 2u * P;
    const uint32_t threads = blockDim.x, dx = threads % nx;
    Store raw[9];
    if (threadIdx.x < n) batch_pull_global<Store>(cur, threadIdx.x, x, n, nx, raw);
    for (uint32_t base = 0; base < n + (T - 1) * 2u * nx; base += threads) {
        const uint32_t node = base + threadIdx.x;
        const uint32_t to_xm = x == 0u ? B * (nx - 1u) : 0u - B, to_xp = x == nx - 1u ? 0u - B * (nx - 1u) : B;
        Store now[9], out[9];
        Real u[3];
        static_for<9>([&](auto aa) { now[decltype(aa)::value] = raw[decltype(aa)::value]; });
        x += dx;
        x = min(x, x - nx);   // less nx where x >= nx (unsigned)
        if (node + threads < n) batch_pull_global<Store>(cur, node + threads, x, n, nx, raw);
        if (node < n) {
            batch_collide<Real, Store>(now, bp, dom, out, u);
            const uint32_t to = ring_address<Store>(B * node, rings);
            static_for<9>([&](auto aa) {
                constexpr int A = decltype(aa)::value;
                *lds_pointer<Store>(to + A * P) = out[A];
            });
        }
        for (uint32_t k = 1; k < T; ++k) {
            __syncthreads();
            uint32_t from = rings + (k - 1) * 9u * P, from2 = from + two;
            asm("" : "+v"(from), "+v"(from2));   // one scalar operand per instruction: the mask
            const uint32_t at = node - k * 2u * nx;   // (before the domain's first node: past its last, mod 2^32)
            if (at < n) {
                // as in batch_pull_global one base per link serves source and wall value
                const uint32_t here = B * at, xm = here + to_xm, xp = here + to_xp;
                const bool lo = at < nx, hi = at >= n - nx;
                const uint32_t own = ring_address<Store>(here, from), own2 = ring_address<Store>(here, from2);
                static_for<9>([&](auto aa) {
                    constexpr int A = decltype(aa)::value;
                    constexpr int EX = Flow<2>::velocity(A, 0), EY = Flow<2>::velocity(A, 1);
                    const uint32_t src = (EX == 0 ? here : (EX > 0 ? xm : xp)) - EY * (B * nx);
                    const uint32_t link = A == 0 ? own : ring_address<Store>(src, EY < 0 ? from2 : from);
                    if constexpr (EY == 0) now[A] = *lds_pointer<const Store>(link + A * P);
                    else if constexpr (EY > 0) now[A] = *lds_pointer<const Store>((lo ? own2 : link) + A * P);
                    else now[A] = *lds_pointer<const Store>((hi ? own : link) + (A - 2) * P);
                });
                batch_collide<Real, Store>(now, bp, dom, out, u);
                if (k + 1 < T) {
                    const uint32_t to = ring_address<Store>(here, from + 9u * P);
                    static_for<9>([&](auto aa) {
                        constexpr int A = decltype(aa)::value;
                        *lds_pointer<Store>(to + A * P) = out[A];
                    });
                } else {
                    static_for<9>([&](auto aa) {
                        constexpr int A = decltype(aa)::value;
                        at_byte(nxt + A * (int64_t)n, here) = out[A];
                    });
                }
            }
        }
        if constexpr (T == 2) __syncthreads();
    }
}

// Runs one domain to completion with buffers `b0` (holding the state) and
// `b1`; returns which of the two holds the final state.  GLOBAL: the buffers are in
// global memory, a thread's next node is loaded while it computes the present one.
template <class Real, class Store, bool GLOBAL>
__device__ int run_domain(Store* b0, Store* b1, uint32_t rings, Real* uprev, const BatchParams& bp, const BatchDomain& dom,
                          double* red, int64_t& steps_out, double& res_out, int& status_out) {
    const uint32_t nx = (uint32_t)dom.nx, ny = (uint32_t)dom.ny, n = nx * ny, threads = blockDim.x;
    // a thread's nodes are `threads` apart: (dx, dy) further, with one carry
    const uint32_t dy = threads / nx, dx = threads - dy * nx;
    const uint32_t y_first = threadIdx.x / nx, x_first = threadIdx.x - y_first * nx;
    Store* cur = b0;
    Store* nxt = b1;
    int which = 0;
    bool have_prev = false;
    double res = INFINITY;
    int status = kBatchMaxSteps;
    int64_t s = 0;
    int32_t since = 0;   // steps since the last check
    for (; s < bp.max_steps;) {
        if constexpr (GLOBAL)
            // as many steps at once as there are before the next check
            if (rings != kNoRings && since < bp.check_interval - batch_fused<Real> && s + batch_fused<Real> <= bp.max_steps) {
                batch_sweep<Real, Store>(cur, nxt, rings, x_first, n, nx, bp, dom);
                __syncthreads();  // the sweep's writes are visible before the next reads them
                Store* t = cur;
                cur = nxt;
                nxt = t;
                which ^= 1;
                s += batch_fused<Real>;
                since += batch_fused<Real>;
                continue;
            }
        const bool check = ++since == bp.check_interval;
        if (check) since = 0;
        CheckSums sums;
        uint32_t x = x_first, y = y_first;
        Store raw[9];
        if (GLOBAL && threadIdx.x < n) batch_pull_global<Store>(cur, threadIdx.x, x, n, nx, raw);
        for (uint32_t node = threadIdx.x; node < n; node += threads) {
            Store now[9], out[9];
            if constexpr (GLOBAL) {
                static_for<9>([&](auto aa) { now[decltype(aa)::value] = raw[decltype(aa)::value]; });
                x += dx;
                x = min(x, x - nx);   // less nx where x >= nx (unsigned)
                if (node + threads < n) batch_pull_global<Store>(cur, node + threads, x, n, nx, raw);
            } else {
                batch_pull<Store>(cur, node_pos(node, (int)x, (int)y, (int)nx, (int)ny), n, nx, now);
                x += dx;
                y += dy;
                if (x >= nx) {
                    x -= nx;
                    ++y;
                }
            }
            Real u[3];
            batch_collide<Real, Store>(now, bp, dom, out, u);
            static_for<9>([&](auto aa) {
                constexpr int A = decltype(aa)::value;
                if constexpr (GLOBAL) at_byte(nxt + A * (int64_t)n, node * (uint32_t)sizeof(Store)) = out[A];
                else element(nxt, A * n + node) = out[A];
            });
            if (check) sums.add(u, uprev, node, n);
        }
        __syncthreads();  // the step's writes are visible before the next step reads them
        Store* t = cur;
        cur = nxt;
        nxt = t;
        which ^= 1;
        ++s;
        if (check) {
            const int stop = check_stop(sums, have_prev, res, bp, red);
            if (stop) {
                status = stop;
                break;
            }
        }
    }
    steps_out = s;
    res_out = res;
    status_out = status;
    return which;
}

// The same for a domain of at most R nodes per thread whose one buffer fits in
// LDS: stepped in place, a step's reads all taken before its writes, with the
// addresses of every pull formed once.
template <class Real, class Store, int R>
__device__ __forceinline__ void run_resident(Store* lds, Real* uprev, const BatchParams& bp, const BatchDomain& dom,
                                             double* red, int64_t& steps_out, double& res_out, int& status_out) {
    const int nx = dom.nx, ny = dom.ny, n = nx * ny;
    uint32_t from[R][9];
    static_for<R>([&](auto rr) {
        constexpr int r = decltype(rr)::value;
        int node = (int)threadIdx.x + r * (int)blockDim.x;
        node = node < n ? node : n - 1;
        const int y = node / nx, x = node - y * nx;
        const NodePos p = node_pos((uint32_t)node, x, y, nx, ny);
        static_for<9>([&](auto aa) {
            constexpr int A = decltype(aa)::value;
            from[r][A] = pull_index<A>(p, (uint32_t)n, (uint32_t)nx);
        });
    });
    bool have_prev = false;
    double res = INFINITY;
    int status = kBatchMaxSteps;
    int64_t s = 0;
    for (; s < bp.max_steps;) {
        const bool check = ((s + 1) % bp.check_interval) == 0;
        CheckSums sums;
        Store raw[R][9];
        static_for<R>([&](auto rr) {
            constexpr int r = decltype(rr)::value;
            static_for<9>([&](auto aa) {
                constexpr int A = decltype(aa)::value;
                raw[r][A] = lds[from[r][A]];
            });
        });
        __syncthreads();
        static_for<R>([&](auto rr) {
            constexpr int r = decltype(rr)::value;
            const int node = (int)threadIdx.x + r * (int)blockDim.x;
            Store out[9];
            Real u[3];
            batch_collide<Real, Store>(raw[r], bp, dom, out, u);
            if (node < n) {
                static_for<9>([&](auto aa) {
                    constexpr int A = decltype(aa)::value;
                    lds[A * n + node] = out[A];
                });
                if (check) sums.add(u, uprev, (uint32_t)node, (uint32_t)n);
            }
        });
        __syncthreads();
        ++s;
        if (check) {
            const int stop = check_stop(sums, have_prev, res, bp, red);
            if (stop) {
                status = stop;
                break;
            }
        }
    }
    steps_out = s;
    res_out = res;
    status_out = status;
}

}  // namespace

// SMALL: domains of at most one node per thread, or no LDS and at most four: nothing to sweep
// and little to load ahead, and without that code the registers (float 123 -> 80, double 128
// and 40 bytes of scratch -> 115) leave room for a third workgroup of 512 threads per CU.
// 2000 domains of 1-8 x 4-64 nodes without LDS, 100 steps: 524 -> 288 us in float, 584 -> 448
// in double; with larger domains loading ahead is worth more (600 domains of up to 16,384
// nodes, workgroups of 256 threads: 3.2 ms against 4.1).
template <class Real, class Store, bool SMALL>
__global__ void __launch_bounds__(1024, SMALL && sizeof(Real) == 4 ? 6 : 4) casclb_batch(BatchParams bp) {
    extern __shared__ unsigned char lds_raw[];
    __shared__ int s_next;
    __shared__ double red[160];
    Store* lds = reinterpret_cast<Store*>(lds_raw);
    // Control flow of this loop is kept scalar (wave-uniform in registers the
    // compiler can see): a lane-divergent branch in a loop that holds barriers
    // lets the compiler split it into nested exec-mask loops in which the other
    // lanes re-enter the barriers without the work-queue atomic (a hang).
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    for (;;) {
        if (wave == 0) {
            // every lane executes the atomic, only lane 0 adds 1; lane 0's
            // result is the index this workgroup took
            const int v = atomicAdd(bp.queue, threadIdx.x == 0 ? 1 : 0);
            s_next = __builtin_amdgcn_readfirstlane(v);
        }
        __syncthreads();
        const int d = __builtin_amdgcn_readfirstlane(s_next);
        __syncthreads();
        if (d >= bp.ndomains) break;
        const BatchDomain dom = bp.domains[bp.order[d]];
        const int n = dom.nx * dom.ny;
        Store* g0 = reinterpret_cast<Store*>(bp.pool) + dom.offset;
        Store* g1 = g0 + (int64_t)9 * n;
        Real* uprev = reinterpret_cast<Real*>(bp.uprev) + dom.uprev_offset;
        int64_t steps = 0;
        double res = INFINITY;
        int status = 0;
        if (n <= bp.resident_nodes) {
            for (int i = threadIdx.x; i < 9 * n; i += blockDim.x) lds[i] = g0[i];
            __syncthreads();
            const int per = (n + (int)blockDim.x - 1) / (int)blockDim.x;
            if (SMALL || per <= 1) run_resident<Real, Store, 1>(lds, uprev, bp, dom, red, steps, res, status);
            else if constexpr (batch_resident_per_thread<Real> == 2)
                run_resident<Real, Store, 2>(lds, uprev, bp, dom, red, steps, res, status);
            for (int i = threadIdx.x; i < 9 * n; i += blockDim.x) g0[i] = lds[i];
            __syncthreads();
        } else if (!SMALL && n <= bp.lds_nodes) {
            Store* l0 = lds;
            Store* l1 = lds + (int64_t)9 * n;
            for (int i = threadIdx.x; i < 9 * n; i += blockDim.x) l0[i] = g0[i];
            __syncthreads();
            const int which = run_domain<Real, Store, false>(l0, l1, kNoRings, uprev, bp, dom, red, steps, res, status);
            const Store* fin = which ? l1 : l0;
            for (int i = threadIdx.x; i < 9 * n; i += blockDim.x) g0[i] = fin[i];
            __syncthreads();
        } else {
            constexpr uint32_t align = batch_ring_align<Real>;
            const uint32_t rings = dom.nx <= bp.fused_nx ? (lds_address(lds) + align - 1) / align * align : kNoRings;
            const int which = run_domain<Real, Store, !SMALL>(g0, g1, rings, uprev, bp, dom, red, steps, res, status);
            if (which) {
                for (int i = threadIdx.x; i < 9 * n; i += blockDim.x) g0[i] = g1[i];
                __syncthreads();
            }
        }
        if (wave == 0) {  // all lanes of wave 0 store the same values
            const int id = bp.order[d];
            bp.out_steps[id] = steps;
            bp.out_residual[id] = res;
            bp.out_status[id] = status;
        }
    }
}

__global__ void casclb_batch_reset(int* queue) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *queue = 0;
}

// Half-forced velocity and density of every node of one domain.
template <class Real, class Store>
__global__ void casclb_batch_moments(BatchParams bp, int id, double* rho_out, double* u_out) {
    const BatchDomain dom = bp.domains[id];
    const int nx = dom.nx, ny = dom.ny, n = nx * ny;
    const int node = blockIdx.x * blockDim.x + threadIdx.x;
    if (node >= n) return;
    const int y = node / nx, x = node - y * nx;
    const Store* src = reinterpret_cast<const Store*>(bp.pool) + dom.offset;
    const int xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
    Real drho = Real(0), jx = Real(0), jy = Real(0);
    static_for<9>([&](auto aa) {
        constexpr int A = decltype(aa)::value;
        constexpr int EX = Flow<2>::velocity(A, 0), EY = Flow<2>::velocity(A, 1);
        const int sy = y - EY;
        const bool wall = sy < 0 || sy >= ny;
        const int sx = EX == 0 ? x : (EX > 0 ? xm : xp);
        const Real v = static_cast<Real>(src[wall ? Flow<2>::opposite(A) * n + node : A * n + sx + nx * sy]);
        drho += v;
        jx += Real(EX) * v;
        jy += Real(EY) * v;
    });
    const Real rho = Real(bp.rho0) + drho;
    rho_out[node] = (double)rho;
    u_out[node] = (double)((jx + Real(0.5) * Real(dom.force_x)) / (rho + Real(0.5) * Real(dom.lorentz)));
    u_out[n + node] = (double)(jy / rho);
}

// Rest state (deviations zero) of every domain's first buffer.
template <class Store>
__global__ void casclb_batch_zero(Store* pool, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        pool[i] = Store(0);
}

// ---- routed domains: one ordinary launch per step over all of them

template <class Real, class Store, bool CHECK>
__global__ void __launch_bounds__(kWideBlock) casclb_batch_wide(WideParams p, int parity) {
    // the routed domains are the batch's longest chains of steps: their waves take
    // precedence in issue over the persistent launch's, which runs beside them
    __builtin_amdgcn_s_setprio(3);
    __shared__ double red[3][kWideBlock / 64];
    const int4 t = p.tiles[blockIdx.x];
    if (p.state[t.x] >= 2) return;   // the slot stopped: uniform over the workgroup
    const BatchDomain dom = p.domains[p.ids[t.x]];
    const int nx = dom.nx, ny = dom.ny, n = nx * ny;
    Store* g0 = reinterpret_cast<Store*>(p.pool) + dom.offset;
    Store* g1 = g0 + (int64_t)9 * n;
    const Store* src = parity ? g1 : g0;
    Store* dst = parity ? g0 : g1;
    BatchParams bp{};
    bp.rho0 = p.rho0;
    bp.w_bulk = p.w_bulk;
    bp.w_third = p.w_third;
    bp.w_fourth = p.w_fourth;
    const int node = t.y + (int)threadIdx.x;
    double du2 = 0.0, u2 = 0.0, bad = 0.0;
    if (node < n) {
        const int y = node / nx, x = node - y * nx;
        Real u[3];
        batch_node<Real, Store>(src, dst, n, nx, ny, x, y, bp, dom, u);
        if (CHECK) {
            Real* uprev = reinterpret_cast<Real*>(p.uprev) + dom.uprev_offset;
            const double ux = (double)u[0], uy = (double)u[1];
            const double ox = (double)uprev[node], oy = (double)uprev[n + node];
            uprev[node] = u[0];
            uprev[n + node] = u[1];
            du2 = (ux - ox) * (ux - ox) + (uy - oy) * (uy - oy);
            u2 = ux * ux + uy * uy;
            bad = (isfinite(ux) && isfinite(uy)) ? 0.0 : 1.0;
        }
    }
    if (CHECK) {
        // wave butterflies, then the waves in order: a fixed summation order
        for (int off = 32; off > 0; off >>= 1) {
            du2 += __shfl_xor(du2, off, 64);
            u2 += __shfl_xor(u2, off, 64);
            bad += __shfl_xor(bad, off, 64);
        }
        const int wave = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) {
            red[0][wave] = du2;
            red[1][wave] = u2;
            red[2][wave] = bad;
        }
        __syncthreads();
        if (threadIdx.x < 3) {
            double s = 0.0;
            for (int w = 0; w < kWideBlock / 64; ++w) s += red[threadIdx.x][w];
            p.partials[(int64_t)blockIdx.x * 3 + threadIdx.x] = s;
        }
    }
}

__global__ void casclb_wide_init(WideParams p) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r == 0) *p.step = 0;
    if (r >= p.nslots) return;
    const int id = p.ids[r];
    p.state[r] = 0;
    p.out_steps[id] = 0;
    p.out_residual[id] = INFINITY;
    p.out_status[id] = kBatchNotRun;
}

// One thread per slot: the slot's tile partials in tile order, then the
// stopping rule of the persistent kernel.  The step counter is advanced by a
// separate launch, after every slot has read it.
__global__ void casclb_wide_check(WideParams p) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= p.nslots) return;
    const int st = p.state[r];
    if (st >= 2) return;
    double du2 = 0.0, u2 = 0.0, bad = 0.0;
    const int t0 = p.tile_first[r], nt = p.tile_count[r];
    for (int t = t0; t < t0 + nt; ++t) {
        du2 += p.partials[(int64_t)t * 3];
        u2 += p.partials[(int64_t)t * 3 + 1];
        bad += p.partials[(int64_t)t * 3 + 2];
    }
    const int id = p.ids[r];
    int stop = 0;
    if (bad > 0.0) {
        stop = kBatchNonFinite;
    } else if (st == 1) {
        const double res = sqrt(du2) / ((double)p.check_interval * sqrt(u2));
        p.out_residual[id] = res;
        if (du2 == 0.0)
            stop = kBatchStationary;
        else if (res < p.tol)
            stop = kBatchConverged;
    }
    if (stop) {
        p.state[r] = 2;
        p.out_status[id] = stop;
        p.out_steps[id] = *p.step + p.check_interval;
    } else {
        p.state[r] = 1;
        atomicAdd(p.active, 1);   // an integer count: exact in any order
    }
}

__global__ void casclb_wide_advance(WideParams p) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *p.step += p.check_interval;
}

__global__ void casclb_wide_reset_active(WideParams p) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *p.active = 0;
}

__global__ void casclb_wide_close(WideParams p, int64_t steps) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= p.nslots || p.state[r] >= 2) return;
    const int id = p.ids[r];
    p.state[r] = 2;
    p.out_status[id] = kBatchMaxSteps;
    p.out_steps[id] = steps;
}

template <class Store>
__global__ void __launch_bounds__(kWideBlock) casclb_wide_gather(WideParams p) {
    const int4 t = p.tiles[blockIdx.x];
    const int id = p.ids[t.x];
    if ((p.out_steps[id] & 1) == 0) return;
    const BatchDomain dom = p.domains[id];
    const int n = dom.nx * dom.ny;
    const int node = t.y + (int)threadIdx.x;
    if (node >= n) return;
    Store* g0 = reinterpret_cast<Store*>(p.pool) + dom.offset;
    const Store* g1 = g0 + (int64_t)9 * n;
    for (int a = 0; a < 9; ++a) g0[(int64_t)a * n + node] = g1[(int64_t)a * n + node];
}

hipError_t launch_wide_step(bool f64, const WideParams& p, int ntiles, int parity, bool check, hipStream_t s) {
    if (ntiles < 1) return hipSuccess;
    if (f64) {
        if (check)
            hipLaunchKernelGGL((casclb_batch_wide<double, double, true>), dim3(ntiles), dim3(kWideBlock), 0, s, p, parity);
        else
            hipLaunchKernelGGL((casclb_batch_wide<double, double, false>), dim3(ntiles), dim3(kWideBlock), 0, s, p, parity);
    } else {
        if (check)
            hipLaunchKernelGGL((casclb_batch_wide<float, float, true>), dim3(ntiles), dim3(kWideBlock), 0, s, p, parity);
        else
            hipLaunchKernelGGL((casclb_batch_wide<float, float, false>), dim3(ntiles), dim3(kWideBlock), 0, s, p, parity);
    }
    return hipGetLastError();
}

static int slot_blocks(const WideParams& p) { return (p.nslots + 255) / 256; }

hipError_t launch_wide_init(const WideParams& p, hipStream_t s) {
    hipLaunchKernelGGL(casclb_wide_init, dim3(slot_blocks(p)), dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_wide_check(const WideParams& p, hipStream_t s) {
    hipLaunchKernelGGL(casclb_wide_reset_active, dim3(1), dim3(64), 0, s, p);
    hipLaunchKernelGGL(casclb_wide_check, dim3(slot_blocks(p)), dim3(256), 0, s, p);
    hipLaunchKernelGGL(casclb_wide_advance, dim3(1), dim3(64), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_wide_close(const WideParams& p, int64_t steps, hipStream_t s) {
    hipLaunchKernelGGL(casclb_wide_close, dim3(slot_blocks(p)), dim3(256), 0, s, p, steps);
    return hipGetLastError();
}

hipError_t launch_wide_gather(bool f64, const WideParams& p, int ntiles, hipStream_t s) {
    if (ntiles < 1) return hipSuccess;
    if (f64)
        hipLaunchKernelGGL(casclb_wide_gather<double>, dim3(ntiles), dim3(kWideBlock), 0, s, p);
    else
        hipLaunchKernelGGL(casclb_wide_gather<float>, dim3(ntiles), dim3(kWideBlock), 0, s, p);
    return hipGetLastError();
}

template <class Real>
static auto batch_kernel(bool small) {
    return small ? casclb_batch<Real, Real, true> : casclb_batch<Real, Real, false>;
}

hipError_t launch_batch(bool f64, bool small, const BatchParams& bp, int grid, int block, size_t lds_bytes, hipStream_t s) {
    hipLaunchKernelGGL(casclb_batch_reset, dim3(1), dim3(64), 0, s, bp.queue);
    hipLaunchKernelGGL(f64 ? batch_kernel<double>(small) : batch_kernel<float>(small), dim3(grid), dim3(block), lds_bytes, s, bp);
    return hipGetLastError();
}

hipError_t batch_set_lds_limit(bool f64, bool small, size_t lds_bytes) {
    const auto kernel = f64 ? batch_kernel<double>(small) : batch_kernel<float>(small);
    return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
}

hipError_t launch_batch_moments(bool f64, const BatchParams& bp, int id, int n, double* rho, double* u,
                                hipStream_t s) {
    const int blocks = (n + 255) / 256;
    if (f64)
        hipLaunchKernelGGL((casclb_batch_moments<double, double>), dim3(blocks), dim3(256), 0, s, bp, id, rho, u);
    else
        hipLaunchKernelGGL((casclb_batch_moments<float, float>), dim3(blocks), dim3(256), 0, s, bp, id, rho, u);
    return hipGetLastError();
}

hipError_t launch_batch_zero(bool f64, void* pool, int64_t n, hipStream_t s) {
    int64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    if (f64)
        hipLaunchKernelGGL(casclb_batch_zero<double>, dim3((unsigned)blocks), dim3(256), 0, s, (double*)pool, n);
    else
        hipLaunchKernelGGL(casclb_batch_zero<float>, dim3((unsigned)blocks), dim3(256), 0, s, (float*)pool, n);
    return hipGetLastError();
}

}  // namespace casclb
