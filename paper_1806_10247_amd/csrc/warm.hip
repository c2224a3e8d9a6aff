// Field operations of the warm start (include/casclb_warm.h): restriction and
// prolongation between lattices, the two-level Richardson combination, the
// projection that removes the mean and the Nyquist lines, packing of the
// network's NHWC input and unpacking of its output, and the initial moments.
// All are bandwidth-bound passes over float64 planes, run once per problem;
// the plane-wide sums are done by one workgroup per plane in a fixed order so
// results do not depend on timing.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "casclb_warm.h"

namespace casclb_warm {

constexpr int kBlock = 256;

__device__ __forceinline__ int wrap(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// fixed-order sum over the block: each thread's partial, then a tree in LDS
__device__ double block_sum(double v, double* lds) {
    lds[threadIdx.x] = v;
    __syncthreads();
    for (int s = kBlock / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) lds[threadIdx.x] += lds[threadIdx.x + s];
        __syncthreads();
    }
    const double r = lds[0];
    __syncthreads();
    return r;
}

__global__ void __launch_bounds__(kBlock) restrict_k(const double* __restrict__ src, int64_t planes, int L,
                                                     double scale, double* __restrict__ dst) {
    const int Lc = L / 2;
    const int64_t total = planes * (int64_t)Lc * Lc;
    for (int64_t k = blockIdx.x * (int64_t)kBlock + threadIdx.x; k < total; k += (int64_t)gridDim.x * kBlock) {
        const int64_t p = k / ((int64_t)Lc * Lc);
        const int r = (int)(k - p * (int64_t)Lc * Lc);
        const int Y = r / Lc, X = r - Y * Lc;
        const double* a = src + p * (int64_t)L * L + (int64_t)(2 * Y) * L + 2 * X;
        dst[k] = scale * (0.25 * ((a[0] + a[1]) + (a[L] + a[L + 1])));
    }
}

// Catmull-Rom weights of the four taps at t = 1/4 (odd fine nodes, taps X-1..X+2)
// and t = 3/4 (even fine nodes, taps X-2..X+1): exact binary fractions.
__constant__ double kW[2][4] = {{-0.0234375, 0.2265625, 0.8671875, -0.0703125},
                                {-0.0703125, 0.8671875, 0.2265625, -0.0234375}};

// Scale of a plane: that of its field when the planes are density, velocity (two
// components) and scalar of `batch` problems.
struct PlaneScales {
    double s[3];
    int batch;   // 0: every plane has scale s[0]
};
__device__ __forceinline__ double plane_scale(const PlaneScales& f, int plane) {
    if (f.batch == 0) return f.s[0];
    return plane < f.batch ? f.s[0] : (plane < 3 * f.batch ? f.s[1] : f.s[2]);
}

__global__ void __launch_bounds__(kBlock) prolong_k(const double* __restrict__ src, int plane0, int Lc,
                                                    PlaneScales scales, double* __restrict__ dst) {
    const int L = 2 * Lc, plane = plane0 + (int)blockIdx.y;
    const uint32_t r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= (uint32_t)L * (uint32_t)L) return;
    const int y = (int)(r / (uint32_t)L), x = (int)(r - (uint32_t)y * (uint32_t)L);
    // first tap and weight row per axis
    const int ox = x & 1, oy = y & 1;
    const int x0 = (x >> 1) - 2 + ox, y0 = (y >> 1) - 2 + oy;
    const double* a = src + (int64_t)plane * Lc * Lc;
    double acc = 0.0;
    for (int j = 0; j < 4; ++j) {
        const double* row = a + wrap(y0 + j, Lc) * Lc;
        double s = 0.0;
        for (int i = 0; i < 4; ++i) s += kW[ox][i] * row[wrap(x0 + i, Lc)];
        acc += kW[oy][j] * s;
    }
    dst[(int64_t)plane * L * L + r] = plane_scale(scales, plane) * acc;
}

// out = a x + b y + c z over the planes of the fields, a, b, c per field
__global__ void __launch_bounds__(kBlock) combine_k(int64_t n, int plane0, PlaneScales a, const double* __restrict__ x, PlaneScales b,
                                                    const double* __restrict__ y, PlaneScales c,
                                                    const double* __restrict__ z, double* __restrict__ out) {
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r >= n) return;
    const int plane = plane0 + (int)blockIdx.y;
    const int64_t i = (int64_t)plane * n + r;
    double v = plane_scale(a, plane) * x[i] + plane_scale(b, plane) * y[i];
    if (z) v = v + plane_scale(c, plane) * z[i];
    out[i] = v;
}

__global__ void __launch_bounds__(kBlock) axpby_k(int64_t n, double a, const double* x, double b, const double* y,
                                                  double* out) {
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock)
        out[i] = a * x[i] + b * y[i];
}

// One workgroup of kProjBlock threads per plane, two passes over it.
//
// With R[y] = mean over x of (-1)^x A(x, y) and C[x] = mean over y of
// (-1)^y A(x, y), the Nyquist lines of the plane are (-1)^x R[y] +
// (-1)^y (C[x] - (-1)^x c), c = mean over y of (-1)^y R[y] (the (pi, pi)
// coefficient, shared by both lines); the mean and the low modes (0 <
// kx^2 + ky^2 <= k2max, one of each +-k pair, kx in 0..2, |ky| <= 2) are
// orthogonal to both lines and to each other, so every coefficient comes from
// the original plane and one second pass subtracts them all.
//
// Both passes take the columns in groups of 64 J (J per lane) and the rows
// two or four at a time, their loads in flight together; wave w takes rows w, w +
// 16, ...  Pass 1: a row's (-1)^x sum is reduced across the wave by a butterfly
// and kept in LDS; everything else is summed along the columns in registers: the
// (-1)^y sums and, for the low modes, the sums against 1, cos / sin(ky y 2 pi /
// L), ky = 1, 2, whose factors are the same for every lane.  The waves' column
// sums are added in wave order through LDS, and the low-mode coefficients (the
// modes are separable) are formed one per wave from them.  Pass 2 subtracts, per
// row, R[y], the column terms and the low modes regrouped as a_kx(y) cos(kx x ..)
// + b_kx(y) sin(kx x ..), one row's coefficients per thread beforehand.  Every sum
// has a fixed order: results do not depend on timing.  Bound by one CU's memory
// latency: four planes of 256^2 take 32 us without and 53 us with the low
// modes (40 and 140 with six row sums by butterflies and one row's loads at a time).
constexpr int kProjBlock = 1024;
constexpr int kProjWaves = kProjBlock / 64;
constexpr int kMaxLowModes = 12;   // half-plane modes with kx^2 + ky^2 <= 8
constexpr int kProjSums = 2 + 2 * kMaxLowModes;
constexpr int kProjRows = 4;

__device__ __forceinline__ double wave_sum(double v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// index of the twiddle for wave number k at position i (|k| <= 2, 0 <= i < L)
__device__ __forceinline__ int twiddle_index(int k, int i, int L) {
    int m = k * i;
    m = m < 0 ? m + 2 * L : m;   // -2 L < k i < 2 L
    m = m >= L ? m - L : m;
    return m >= L ? m - L : m;
}

// columns per lane: the largest lattices keep the LDS for their row and column sums,
// and six column sums of four columns do not fit the 128 registers of a lane
int project_columns(int L, int nmodes) { return L <= 64 || L > 1024 ? 1 : (L <= 128 || nmodes > 0 ? 2 : 4); }

size_t project_lds_bytes(int L, int nmodes) {
    return (size_t)((nmodes > 0 ? 9 : 2) * L + project_columns(L, nmodes) * kProjWaves * 64 + kProjWaves + kProjSums) *
           sizeof(double);
}

template <int J, bool LOW>
__global__ void __launch_bounds__(kProjBlock) project_k(double* data, int L, int nmodes, int4 modes_a, int4 modes_b,
                                                        int4 modes_c, int4 modes_d, int4 modes_e, int4 modes_f) {
    constexpr int KR = LOW && J > 1 ? 2 : kProjRows, NC = LOW ? 6 : 1;   // column sums: (-1)^y, then 1, cos y, sin y, cos 2y, sin 2y
    extern __shared__ double lds[];
    double* red = lds;                              // [J][kProjWaves][64] wave partials
    double* totals = red + J * kProjWaves * 64;     // [kProjWaves]
    double* fin = totals + kProjWaves;              // [kProjSums] plane sums
    double* rowR = fin + kProjSums;                 // R[y]
    double* cols = rowR + L;                        // [NC][L] column sums; [1..5] later the low modes' row coefficients
    double* ct = cols + NC * L;                     // with low modes: cos(2 pi m / L)
    double* st = ct + L;                            //   sin(2 pi m / L)
    double* A = data + (int64_t)blockIdx.x * L * L;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const double inv = 1.0 / (double)L;
    __shared__ int mkx[kMaxLowModes], mky[kMaxLowModes];   // wave numbers of the low modes
    if constexpr (LOW) {
        if (threadIdx.x == 0) {
            const int4 packed[6] = {modes_a, modes_b, modes_c, modes_d, modes_e, modes_f};
#pragma unroll
            for (int i = 0; i < 6; ++i) {   // constant indexes: stays in registers
                mkx[2 * i] = packed[i].x;
                mky[2 * i] = packed[i].y;
                mkx[2 * i + 1] = packed[i].z;
                mky[2 * i + 1] = packed[i].w;
            }
        }
        for (int m = threadIdx.x; m < L; m += kProjBlock) sincospi(2.0 * (double)m / (double)L, &st[m], &ct[m]);
        __syncthreads();
    }
    const double sx0 = (lane & 1) ? -1.0 : 1.0;   // x is even exactly when lane is
    auto load_rows = [&](int y0, int g, double (&v)[KR][J]) {
#pragma unroll
        for (int i = 0; i < KR; ++i)
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int y = y0 + i * kProjWaves, x = g + lane + 64 * j;
                v[i][j] = y < L && x < L ? A[(int64_t)y * L + x] : 0.0;
            }
    };
    // ---- pass 1
    double total = 0.0;
    for (int g = 0; g < L; g += 64 * J) {
        double acc[NC][J];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < J; ++j) acc[c][j] = 0.0;
        for (int y0 = wave; y0 < L; y0 += KR * kProjWaves) {
            double v[KR][J], alt[KR];
            load_rows(y0, g, v);
#pragma unroll
            for (int i = 0; i < KR; ++i) {
                const int y = y0 + i * kProjWaves;
                const double sy = (y & 1) ? -1.0 : 1.0;
                alt[i] = 0.0;
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    alt[i] += v[i][j];
                    acc[0][j] += sy * v[i][j];
                }
                if constexpr (LOW) {
                    const int yc = y < L ? y : 0, y2 = twiddle_index(2, yc, L);   // (rows past the end are zeros)
                    const double c1 = ct[yc], s1 = st[yc], c2 = ct[y2], s2 = st[y2];
#pragma unroll
                    for (int j = 0; j < J; ++j) {
                        acc[1][j] += v[i][j];
                        acc[2][j] += v[i][j] * c1;
                        acc[3][j] += v[i][j] * s1;
                        acc[4][j] += v[i][j] * c2;
                        acc[5][j] += v[i][j] * s2;
                    }
                }
                total += alt[i];
                alt[i] *= sx0;
            }
#pragma unroll
            for (int i = 0; i < KR; ++i) alt[i] = wave_sum(alt[i]);
            if (lane == 0)
#pragma unroll
                for (int i = 0; i < KR; ++i) {
                    const int y = y0 + i * kProjWaves;
                    if (y < L) rowR[y] = (g == 0 ? 0.0 : rowR[y]) + alt[i] * inv;
                }
        }
        // the waves' column sums, added in wave order
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            __syncthreads();
#pragma unroll
            for (int j = 0; j < J; ++j) red[(j * kProjWaves + wave) * 64 + lane] = acc[c][j];
            __syncthreads();
            const int x = g + (int)threadIdx.x;
            if (threadIdx.x < 64 * J && x < L) {
                double s = 0.0;
                for (int w = 0; w < kProjWaves; ++w) s += red[(wave * kProjWaves + w) * 64 + lane];
                cols[c * L + x] = s;
            }
        }
    }
    total = wave_sum(total);
    if (lane == 0) totals[wave] = total;
    __syncthreads();
    // ---- plane sums, one per wave: q = 0 mean, 1 (-1)^y R[y], 2 + 2 i and 3 + 2 i the
    // cos and sin coefficients of low mode i
    for (int q = wave; q < 2 + 2 * nmodes; q += kProjWaves) {
        double s = 0.0;
        if (q == 0) {
            for (int w = 0; w < kProjWaves; ++w) s += totals[w];
        } else if (q == 1) {
            for (int y = lane; y < L; y += 64) s += (y & 1) ? -rowR[y] : rowR[y];
            s = wave_sum(s);
        } else if constexpr (LOW) {
            const int kx = mkx[(q - 2) >> 1], ky = mky[(q - 2) >> 1], k = ky < 0 ? -ky : ky;
            const double sgn = ky < 0 ? -1.0 : 1.0;
            const double* cy = cols + (k == 0 ? 1 : 2 * k) * L;   // sums against cos(k y ..), sin(k y ..)
            const double* sn = cols + (2 * k + 1) * L;
            for (int x = lane; x < L; x += 64) {
                const int t = twiddle_index(kx, x, L);
                const double pc = cy[x], ps = k == 0 ? 0.0 : sgn * sn[x];
                s += (q & 1) ? pc * st[t] + ps * ct[t] : pc * ct[t] - ps * st[t];
            }
            s = wave_sum(s);
        }
        if (lane == 0) fin[q] = q == 0 ? s * inv * inv : (q == 1 ? s * inv : 2.0 * s * inv * inv);
    }
    __syncthreads();
    const double mean = fin[0], cnn = fin[1];
    if constexpr (LOW) {
        // row coefficients a0 (with the mean), a1, b1, a2, b2 over the sums no longer needed
        for (int y = threadIdx.x; y < L; y += kProjBlock) {
            double a0 = mean, a1 = 0.0, b1 = 0.0, a2 = 0.0, b2 = 0.0;
            for (int m = 0; m < nmodes; ++m) {
                const int kx = mkx[m], t = twiddle_index(mky[m], y, L);
                const double mc = fin[2 + 2 * m], ms = fin[3 + 2 * m];
                const double a = mc * ct[t] + ms * st[t], b = ms * ct[t] - mc * st[t];
                if (kx == 0) {
                    a0 += a;
                } else if (kx == 1) {
                    a1 += a;
                    b1 += b;
                } else {
                    a2 += a;
                    b2 += b;
                }
            }
            cols[1 * L + y] = a0;
            cols[2 * L + y] = a1;
            cols[3 * L + y] = b1;
            cols[4 * L + y] = a2;
            cols[5 * L + y] = b2;
        }
        __syncthreads();
    }
    // ---- pass 2
    for (int g = 0; g < L; g += 64 * J) {
        double col[J];   // C[x] - (-1)^x c of this lane's columns
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int x = g + lane + 64 * j;
            col[j] = x < L ? cols[x] * inv - sx0 * cnn : 0.0;
        }
        for (int y0 = wave; y0 < L; y0 += KR * kProjWaves) {
            double v[KR][J];
            load_rows(y0, g, v);
#pragma unroll
            for (int i = 0; i < KR; ++i) {
                const int y = y0 + i * kProjWaves;
                if (y >= L) break;
                const double sy = (y & 1) ? -1.0 : 1.0, ry = rowR[y];
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const int x = g + lane + 64 * j;
                    if (x < L) {
                        double low = mean;
                        if constexpr (LOW) {
                            const int x2 = twiddle_index(2, x, L);
                            low = cols[1 * L + y] + cols[2 * L + y] * ct[x] + cols[3 * L + y] * st[x] +
                                  cols[4 * L + y] * ct[x2] + cols[5 * L + y] * st[x2];
                        }
                        A[(int64_t)y * L + x] = v[i][j] - sx0 * ry - sy * col[j] - low;
                    }
                }
            }
        }
    }
}

struct Channels {
    lb_warm_channel c[LB_WARM_MAX_CHANNELS];
};

// The channel loops run over the compile-time maximum with a guard, so every
// access to the argument struct has a constant index (no private-memory copy).
__global__ void __launch_bounds__(kBlock) pack_k(Channels ch, int nc, int64_t total, float* out) {
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < total; i += (int64_t)gridDim.x * kBlock) {
#pragma unroll
        for (int c = 0; c < LB_WARM_MAX_CHANNELS; ++c) {
            if (c < nc) {
                const double v = ch.c[c].src ? ch.c[c].scale * ch.c[c].src[i] + ch.c[c].offset : ch.c[c].offset;
                out[i * nc + c] = (float)v;
            }
        }
    }
}

__global__ void __launch_bounds__(kBlock) unpack_k(const float* y, Channels ch, int nc, int64_t total) {
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < total; i += (int64_t)gridDim.x * kBlock) {
#pragma unroll
        for (int c = 0; c < LB_WARM_MAX_CHANNELS; ++c)
            if (c < nc)
                ch.c[c].dst[i] = (ch.c[c].src ? ch.c[c].src[i] : 0.0) + ch.c[c].scale * (double)y[i * nc + c];
    }
}

// One workgroup of kProjBlock threads per problem b; the momentum sums are
// reduced per wave by a butterfly and then added in wave order (deterministic).
__global__ void __launch_bounds__(kProjBlock) initial_state_k(const double* drho, const double* u, const double* phi,
                                                              const double* F, const double* S, int batch, int64_t n,
                                                              double rho0, int zero_momentum, double* rho_out,
                                                              double* u_out, double* phi_out) {
    __shared__ double red[3][kProjWaves];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t b = blockIdx.x;
    const int64_t o = b * n, comp = (int64_t)batch * n;
    double shift_x = 0.0, shift_y = 0.0;
    if (zero_momentum) {
        double sr = 0.0, sx = 0.0, sy = 0.0;
#pragma unroll 4
        for (int64_t i = threadIdx.x; i < n; i += kProjBlock) {
            const double r = rho0 + drho[o + i];
            sr += r;
            sx += r * u[o + i];
            sy += r * u[comp + o + i];
        }
        sr = wave_sum(sr);
        sx = wave_sum(sx);
        sy = wave_sum(sy);
        if (lane == 0) {
            red[0][wave] = sr;
            red[1][wave] = sx;
            red[2][wave] = sy;
        }
        __syncthreads();
        double tr = 0.0, tx = 0.0, ty = 0.0;
        for (int w = 0; w < kProjWaves; ++w) {
            tr += red[0][w];
            tx += red[1][w];
            ty += red[2][w];
        }
        shift_x = tx / tr;
        shift_y = ty / tr;
    }
#pragma unroll 4
    for (int64_t i = threadIdx.x; i < n; i += kProjBlock) {
        const double r = rho0 + drho[o + i];
        rho_out[o + i] = r;
        u_out[o + i] = (u[o + i] - shift_x) - F[o + i] / (2.0 * r);
        u_out[comp + o + i] = (u[comp + o + i] - shift_y) - F[comp + o + i] / (2.0 * r);
        if (phi_out) phi_out[o + i] = phi[o + i] - (S ? 0.5 * S[o + i] : 0.0);
    }
}

// The same in three launches that use the whole chip, for problems of many nodes
// and outputs apart from the inputs: partial sums (kInitParts workgroups per
// problem, left in the first kInitParts nodes of the outputs), every other node,
// then those first nodes.  One problem of 64^2: 9.7 us in one launch, 9.9 in
// three; 90^2: 18 and 10; 256^2: 109 and 10 (launch-bound: the kernels take 4 + 4 + 2).
constexpr int kInitParts = 64;
struct InitArgs {
    const double *drho, *u, *phi, *F, *S;
    int64_t n, comp;   // nodes per problem, stride between the components
    double rho0;
    double *rho_out, *u_out, *phi_out;
};

__device__ __forceinline__ void initial_node(const InitArgs& a, int64_t i, double shift_x, double shift_y) {
    const double r = a.rho0 + a.drho[i];
    a.rho_out[i] = r;
    a.u_out[i] = (a.u[i] - shift_x) - a.F[i] / (2.0 * r);
    a.u_out[a.comp + i] = (a.u[a.comp + i] - shift_y) - a.F[a.comp + i] / (2.0 * r);
    if (a.phi_out) a.phi_out[i] = a.phi[i] - (a.S ? 0.5 * a.S[i] : 0.0);
}

__global__ void __launch_bounds__(kBlock) initial_sums_k(InitArgs a) {
    __shared__ double lds[kBlock];
    const int64_t o = (int64_t)blockIdx.y * a.n;
    double sr = 0.0, sx = 0.0, sy = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < a.n; i += kInitParts * kBlock) {
        const double r = a.rho0 + a.drho[o + i];
        sr += r;
        sx += r * a.u[o + i];
        sy += r * a.u[a.comp + o + i];
    }
    sr = block_sum(sr, lds);
    sx = block_sum(sx, lds);
    sy = block_sum(sy, lds);
    if (threadIdx.x == 0) {
        a.rho_out[o + blockIdx.x] = sr;
        a.u_out[o + blockIdx.x] = sx;
        a.u_out[a.comp + o + blockIdx.x] = sy;
    }
}

// u's shift of problem o / n from the partial sums (every wavefront adds them in the same order)
__device__ __forceinline__ void initial_shift(const InitArgs& a, int64_t o, double& shift_x, double& shift_y) {
    static_assert(kInitParts == 64, "one partial sum per lane");
    const int lane = threadIdx.x & 63;
    const double tr = wave_sum(a.rho_out[o + lane]), tx = wave_sum(a.u_out[o + lane]),
                 ty = wave_sum(a.u_out[a.comp + o + lane]);
    shift_x = tx / tr;
    shift_y = ty / tr;
}

__global__ void __launch_bounds__(kBlock) initial_rest_k(InitArgs a) {
    const int64_t o = (int64_t)blockIdx.y * a.n;
    double shift_x, shift_y;
    initial_shift(a, o, shift_x, shift_y);
    const int64_t i = kInitParts + (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < a.n) initial_node(a, o + i, shift_x, shift_y);
}

__global__ void __launch_bounds__(kInitParts) initial_first_k(InitArgs a) {
    const int64_t o = (int64_t)blockIdx.x * a.n;
    double shift_x, shift_y;
    initial_shift(a, o, shift_x, shift_y);   // one wavefront: read before any of it is overwritten
    initial_node(a, o + threadIdx.x, shift_x, shift_y);
}

int grid_for(int64_t total) {
    const int64_t blocks = (total + kBlock - 1) / kBlock;
    return (int)(blocks < 65536 ? (blocks > 0 ? blocks : 1) : 65536);
}

constexpr int kMaxPlanes = 65535;   // of one launch (grid.y)

int done(hipError_t e) { return e == hipSuccess ? LB_OK : LB_EHIP; }

int launch_prolong(const double* src, int planes, int Lc, const PlaneScales& scales, double* dst, hipStream_t s) {
    const unsigned blocks = ((unsigned)(2 * Lc) * (unsigned)(2 * Lc) + kBlock - 1) / kBlock;
    for (int p0 = 0; p0 < planes; p0 += kMaxPlanes)
        hipLaunchKernelGGL(prolong_k, dim3(blocks, (unsigned)std::min(kMaxPlanes, planes - p0)), dim3(kBlock), 0, s, src, p0,
                           Lc, scales, dst);
    return done(hipGetLastError());
}

// Whether [a, a + n) and [b, b + m) share an element.
bool overlap(const double* a, int64_t n, const double* b, int64_t m) {
    return a && b && (uintptr_t)a < (uintptr_t)(b + m) && (uintptr_t)b < (uintptr_t)(a + n);
}

}  // namespace casclb_warm

using namespace casclb_warm;

extern "C" {

int lb_warm_restrict(const double* src, int32_t planes, int32_t L, double scale, double* dst, void* stream) {
    if (!src || !dst || planes < 1 || L < 2 || L > LB_WARM_MAX_L || (L & 1)) return LB_EINVAL;
    const int64_t total = (int64_t)planes * (L / 2) * (L / 2);
    hipLaunchKernelGGL(restrict_k, dim3(grid_for(total)), dim3(kBlock), 0, (hipStream_t)stream, src, (int64_t)planes,
                       (int)L, scale, dst);
    return done(hipGetLastError());
}

int lb_warm_prolong(const double* src, int32_t planes, int32_t Lc, double scale, double* dst, void* stream) {
    if (!src || !dst || planes < 1 || Lc < 2 || 2 * Lc > LB_WARM_MAX_L) return LB_EINVAL;
    return launch_prolong(src, planes, Lc, PlaneScales{{scale, scale, scale}, 0}, dst, (hipStream_t)stream);
}

int lb_warm_prolong_fields(const double* src, int32_t batch, int32_t Lc, const double scales[3], double* dst,
                           void* stream) {
    if (!src || !dst || !scales || batch < 1 || batch > (1 << 28) || Lc < 2 || 2 * Lc > LB_WARM_MAX_L) return LB_EINVAL;
    return launch_prolong(src, 4 * batch, Lc, PlaneScales{{scales[0], scales[1], scales[2]}, batch}, dst, (hipStream_t)stream);
}

int lb_warm_combine_fields(int32_t batch, int64_t n, const double a[3], const double* x, const double b[3],
                           const double* y, const double c[3], const double* z, double* out, void* stream) {
    if (batch < 1 || batch > (1 << 28) || n < 1 || n > (int64_t)LB_WARM_MAX_L * LB_WARM_MAX_L || !a || !x || !b || !y ||
        (z && !c) || !out)
        return LB_EINVAL;
    const PlaneScales pa{{a[0], a[1], a[2]}, batch}, pb{{b[0], b[1], b[2]}, batch};
    PlaneScales pc{{0.0, 0.0, 0.0}, batch};
    if (z) pc = PlaneScales{{c[0], c[1], c[2]}, batch};
    for (int p0 = 0; p0 < 4 * batch; p0 += kMaxPlanes)
        hipLaunchKernelGGL(combine_k, dim3((unsigned)((n + kBlock - 1) / kBlock), (unsigned)std::min(kMaxPlanes, 4 * batch - p0)),
                           dim3(kBlock), 0, (hipStream_t)stream, n, p0, pa, x, pb, y, pc, z, out);
    return done(hipGetLastError());
}

int lb_warm_axpby(int64_t n, double a, const double* x, double b, const double* y, double* out, void* stream) {
    if (n < 0 || (n > 0 && (!x || !y || !out))) return LB_EINVAL;
    if (n == 0) return LB_OK;
    hipLaunchKernelGGL(axpby_k, dim3(grid_for(n)), dim3(kBlock), 0, (hipStream_t)stream, n, a, x, b, y, out);
    return done(hipGetLastError());
}

int lb_warm_project(double* data, int32_t planes, int32_t L, int32_t k2max, void* stream) {
    if (!data || planes < 1 || L < 2 || L > LB_WARM_MAX_L || (L & 1)) return LB_EINVAL;
    if (k2max < 0 || k2max > LB_WARM_MAX_K2) return LB_EINVAL;
    // one mode of each +-k pair: kx > 0, or kx = 0 and ky > 0; |k| far below the Nyquist lines
    int m[2 * kMaxLowModes] = {0};
    int n = 0;
    for (int kx = 0; kx * kx <= k2max; ++kx)
        for (int ky = -3; ky <= 3; ++ky) {
            if (kx * kx + ky * ky == 0 || kx * kx + ky * ky > k2max) continue;
            if (kx == 0 && ky <= 0) continue;
            if (2 * kx >= L || 2 * (ky < 0 ? -ky : ky) >= L) return LB_EINVAL;
            m[2 * n] = kx;
            m[2 * n + 1] = ky;
            ++n;
        }
    const size_t lds = project_lds_bytes(L, n);
    const int4 ma = make_int4(m[0], m[1], m[2], m[3]), mb = make_int4(m[4], m[5], m[6], m[7]),
               mc = make_int4(m[8], m[9], m[10], m[11]), md = make_int4(m[12], m[13], m[14], m[15]),
               me = make_int4(m[16], m[17], m[18], m[19]), mf = make_int4(m[20], m[21], m[22], m[23]);
    const int J = project_columns(L, n);
    auto plain = J == 1 ? project_k<1, false> : J == 2 ? project_k<2, false> : project_k<4, false>;
    auto low = J == 1 ? project_k<1, true> : project_k<2, true>;
    auto kernel = n > 0 ? low : plain;
    if (lds > 65536) {   // the largest lattices need more than the default dynamic LDS limit
        const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return LB_EHIP;
    }
    hipLaunchKernelGGL(kernel, dim3(planes), dim3(kProjBlock), lds, (hipStream_t)stream, data, (int)L, n, ma, mb, mc,
                       md, me, mf);
    return done(hipGetLastError());
}

static int channels_of(const lb_warm_channel* in, int32_t nc, bool unpack, Channels* out) {
    if (!in || nc < 1 || nc > LB_WARM_MAX_CHANNELS) return LB_EINVAL;
    for (int c = 0; c < nc; ++c) {
        if (unpack && !in[c].dst) return LB_EINVAL;
        out->c[c] = in[c];
    }
    return LB_OK;
}

int lb_warm_pack(const lb_warm_channel* channels, int32_t nchannels, int32_t batch, int64_t n, float* out,
                 void* stream) {
    Channels ch{};
    if (channels_of(channels, nchannels, false, &ch) || !out || batch < 1 || n < 1) return LB_EINVAL;
    const int64_t total = (int64_t)batch * n;
    hipLaunchKernelGGL(pack_k, dim3(grid_for(total)), dim3(kBlock), 0, (hipStream_t)stream, ch, (int)nchannels, total,
                       out);
    return done(hipGetLastError());
}

int lb_warm_unpack(const float* y, const lb_warm_channel* channels, int32_t nchannels, int32_t batch, int64_t n,
                   void* stream) {
    Channels ch{};
    if (channels_of(channels, nchannels, true, &ch) || !y || batch < 1 || n < 1) return LB_EINVAL;
    const int64_t total = (int64_t)batch * n;
    hipLaunchKernelGGL(unpack_k, dim3(grid_for(total)), dim3(kBlock), 0, (hipStream_t)stream, y, ch, (int)nchannels,
                       total);
    return done(hipGetLastError());
}

int lb_warm_initial_state(const double* drho, const double* u, const double* phi, const double* F, const double* S,
                          int32_t batch, int64_t n, double rho0, int32_t zero_momentum, double* rho_out,
                          double* u_out, double* phi_out, void* stream) {
    if (!drho || !u || !F || !rho_out || !u_out || batch < 1 || n < 1) return LB_EINVAL;
    if ((phi == nullptr) != (phi_out == nullptr)) return LB_EINVAL;
    const int64_t all = (int64_t)batch * n;
    const InitArgs a{drho, u, phi, F, S, n, all, rho0, rho_out, u_out, phi_out};
    // outputs that share memory with an input are written only after every sum: one workgroup each
    bool apart = true;
    for (const double* in : {drho, phi, S})
        apart = apart && !overlap(in, all, rho_out, all) && !overlap(in, all, u_out, 2 * all) && !overlap(in, all, phi_out, all);
    for (const double* in : {u, F})
        apart = apart && !overlap(in, 2 * all, rho_out, all) && !overlap(in, 2 * all, u_out, 2 * all) && !overlap(in, 2 * all, phi_out, all);
    // from where three launches cost less than one: 64^2 nodes
    if (zero_momentum && apart && n >= 4096 && batch <= kMaxPlanes) {
        hipLaunchKernelGGL(initial_sums_k, dim3(kInitParts, (unsigned)batch), dim3(kBlock), 0, (hipStream_t)stream, a);
        hipLaunchKernelGGL(initial_rest_k, dim3((unsigned)((n - kInitParts + kBlock - 1) / kBlock), (unsigned)batch),
                           dim3(kBlock), 0, (hipStream_t)stream, a);
        hipLaunchKernelGGL(initial_first_k, dim3((unsigned)batch), dim3(kInitParts), 0, (hipStream_t)stream, a);
        return done(hipGetLastError());
    }
    hipLaunchKernelGGL(initial_state_k, dim3(batch), dim3(kProjBlock), 0, (hipStream_t)stream, drho, u, phi, F, S,
                       (int)batch, n, rho0, (int)(zero_momentum != 0), rho_out, u_out, phi_out);
    return done(hipGetLastError());
}

}  // extern "C"
