// Field operations of the warm start (include/casclb_warm.h): restriction and
// prolongation between lattices, the two-level Richardson combination, the
// projection that removes the mean and the Nyquist lines, packing of the
// network's NHWC input and unpacking of its output, and the initial moments.
// All are bandwidth-bound passes over float64 planes, run once per problem;
// the plane-wide sums are done in a fixed order so
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

// node (x, y) of a plane prolonged from a
__device__ __forceinline__ double prolong_node(const double* a, int Lc, int x, int y) {
    // first tap and weight row per axis
    const int ox = x & 1, oy = y & 1;
    const int x0 = (x >> 1) - 2 + ox, y0 = (y >> 1) - 2 + oy;
    double acc = 0.0;
    for (int j = 0; j < 4; ++j) {
        const double* row = a + wrap(y0 + j, Lc) * Lc;
        double s = 0.0;
        for (int i = 0; i < 4; ++i) s += kW[ox][i] * row[wrap(x0 + i, Lc)];
        acc += kW[oy][j] * s;
    }
    return acc;
}

// dst = a x + b P y + c P z over the planes, P the prolongation; x and z may be null
__global__ void __launch_bounds__(kBlock) prolong_k(int plane0, int Lc, PlaneScales a, const double* __restrict__ px,
                                                    PlaneScales b, const double* __restrict__ py, PlaneScales c,
                                                    const double* __restrict__ pz, double* __restrict__ dst) {
    const int L = 2 * Lc, plane = plane0 + (int)blockIdx.y;
    const uint32_t r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= (uint32_t)L * (uint32_t)L) return;
    const int y = (int)(r / (uint32_t)L), x = (int)(r - (uint32_t)y * (uint32_t)L);
    const int64_t i = (int64_t)plane * L * L + r, o = (int64_t)plane * Lc * Lc;
    double v = plane_scale(b, plane) * prolong_node(py + o, Lc, x, y);
    if (px) v = plane_scale(a, plane) * px[i] + v;
    if (pz) v = v + plane_scale(c, plane) * prolong_node(pz + o, Lc, x, y);
    dst[i] = v;
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

// The same projection by many workgroups per plane, in two launches with the partial
// sums in a workspace between them.  project_sums_k: a workgroup of 16 wavefronts takes
// 16 RPW rows (a wavefront's are 16 apart), sums each of them plainly and, for the low
// modes, against cos / sin(kx x 2 pi / L), kx = 1, 2 (the modes are separable; a lane's
// columns have one parity, so the (-1)^x sum is the plain one with the lanes' signs), and
// writes its part of the (-1)^y column sums.  project_apply_k: the same rows again; every
// workgroup adds the column parts (at most 32) and forms the plane sums from the row sums
// by itself: a third launch for them cost more (24 us against 18 for four planes of 256^2
// with low modes).  About 512 workgroups, each stepping through every gridDim.x-th part of
// its plane, so that many planes do not repeat the plane sums for every part (256 planes of
// 256^2: 71 us, 131 with low modes; one workgroup per part 85 and 193).  Fixed order as
// above, whatever the number of workgroups (two fit a CU; up to 768 take a part each).
// Bound by latency, then by memory: four planes of 256^2 take 8.4 us (30 with one workgroup
// each), 17.7 with low modes (52); of 1024^2 35 and 52 (458 and 805).
constexpr int kSplitParts = 32;
__host__ __device__ constexpr int split_rows(int L) { return 16 * ((L + 16 * kSplitParts - 1) / (16 * kSplitParts)); }
__host__ __device__ constexpr int split_parts(int L) { return (L + split_rows(L) - 1) / split_rows(L); }
// doubles of a plane: row sums R[y], plain and (low modes) cos, sin, cos 2, sin 2; column parts
__host__ __device__ constexpr int64_t split_work(int L, bool low) { return (int64_t)((low ? 6 : 2) + split_parts(L)) * L; }

// columns per lane at a time of project_sums_k, within 128 registers
__host__ __device__ constexpr int sums_columns(int rpw) { return rpw > 2 ? 2 : 4; }

struct LowModes {
    int8_t n, kx[kMaxLowModes], ky[kMaxLowModes];
};

// Rows y0, y0 + 16, ... of a plane, columns g + lane + 64 j
template <int RPW, int J>
__device__ __forceinline__ void project_load(const double* A, int L, int y0, int g, double (&v)[RPW][J]) {
#pragma unroll
    for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int y = y0 + 16 * i, x = g + ((int)threadIdx.x & 63) + 64 * j;
            v[i][j] = y < L && x < L ? A[(int64_t)y * L + x] : 0.0;
        }
}

template <int RPW, bool LOW>
__global__ void __launch_bounds__(kProjBlock, RPW == 1 && !LOW ? 8 : 4) project_sums_k(const double* __restrict__ data, int L, double* __restrict__ work) {
    extern __shared__ double lds[];
    constexpr int J = sums_columns(RPW);
    double* red = lds;                            // [kProjWaves][64 J]
    double* ct = red + kProjWaves * 64 * J;       // with low modes: cos(2 pi m / L)
    double* st = ct + L;                          //   sin(2 pi m / L)
    const double* A = data + (int64_t)blockIdx.y * L * L;
    double* rows = work + (int64_t)blockIdx.y * split_work(L, LOW);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const double sx0 = (lane & 1) ? -1.0 : 1.0, inv = 1.0 / (double)L;   // x is even exactly when lane is
    for (int b = blockIdx.x; b < split_parts(L); b += gridDim.x) {
        double* part = rows + (int64_t)((LOW ? 6 : 2) + b) * L;
        const int y0 = b * 16 * RPW + wave;
        double sum[RPW][LOW ? 5 : 1] = {};
        for (int g = 0; g < L; g += 64 * J) {
            double v[RPW][J], col[J] = {};
            project_load(A, L, y0, g, v);
            const bool first = g == 0 && b == (int)blockIdx.x;
            if constexpr (LOW)
                if (first) {   // behind the first loads
                    for (int m = threadIdx.x; m < L; m += kProjBlock) sincospi(2.0 * (double)m / (double)L, &st[m], &ct[m]);
                    __syncthreads();
                }
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int x = g + lane + 64 * j, xc = x < L ? x : 0, x2 = twiddle_index(2, xc, L);   // (columns past the end are zeros)
#pragma unroll
                for (int i = 0; i < RPW; ++i) {
                    sum[i][0] += v[i][j];
                    col[j] += ((y0 + 16 * i) & 1) ? -v[i][j] : v[i][j];
                    if constexpr (LOW) {
                        sum[i][1] += v[i][j] * ct[xc];
                        sum[i][2] += v[i][j] * st[xc];
                        sum[i][3] += v[i][j] * ct[x2];
                        sum[i][4] += v[i][j] * st[x2];
                    }
                }
            }
            if (!first) __syncthreads();
#pragma unroll
            for (int j = 0; j < J; ++j) red[(wave * J + j) * 64 + lane] = col[j];
            __syncthreads();
            if (threadIdx.x < 64 * J && g + (int)threadIdx.x < L) {
                double s = 0.0;
                for (int w = 0; w < kProjWaves; ++w) s += red[w * 64 * J + threadIdx.x];
                part[g + threadIdx.x] = s;
            }
        }
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int y = y0 + 16 * i;
            const double alt = wave_sum(sx0 * sum[i][0]) * inv;
#pragma unroll
            for (int c = 0; c < (LOW ? 5 : 1); ++c) sum[i][c] = wave_sum(sum[i][c]);
            if (lane == 0 && y < L) {
                rows[y] = alt;
#pragma unroll
                for (int c = 0; c < (LOW ? 5 : 1); ++c) rows[(int64_t)(1 + c) * L + y] = sum[i][c];
            }
        }
    }
}

template <int RPW, bool LOW>
__global__ void __launch_bounds__(kProjBlock, RPW == 1 ? 8 : 4) project_apply_k(double* __restrict__ data, int L, LowModes modes,
                                                                                const double* __restrict__ work) {
    extern __shared__ double lds[];
    constexpr int J = RPW > 2 || LOW ? 2 : 4, ROWS = 16 * RPW;
    double* cols = lds;                  // C[x]
    double* fin = cols + L;              // [kProjSums] plane sums
    double* coef = fin + kProjSums;      // with low modes: [5][ROWS] row coefficients a0 (with the mean), a1, b1, a2, b2
    double* ct = coef + 5 * ROWS;        //   cos(2 pi m / L)
    double* st = ct + L;                 //   sin(2 pi m / L)
    double* A = data + (int64_t)blockIdx.y * L * L;
    const double* rows = work + (int64_t)blockIdx.y * split_work(L, LOW);
    const double* part = rows + (int64_t)(LOW ? 6 : 2) * L;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nparts = split_parts(L);
    const double inv = 1.0 / (double)L;
    double v[RPW][J];
    project_load(A, L, (int)blockIdx.x * ROWS + wave, 0, v);
    for (int x = threadIdx.x; x < L; x += kProjBlock) {
        double s = 0.0;
#pragma unroll 8
        for (int p = 0; p < nparts; ++p) s += part[(int64_t)p * L + x];
        cols[x] = s * inv;
    }
    if constexpr (LOW) {
        for (int m = kProjBlock - 1 - threadIdx.x; m < L; m += kProjBlock) sincospi(2.0 * (double)m / (double)L, &st[m], &ct[m]);
        __syncthreads();
    }
    // plane sums, one per wave (the last waves first: the first ones have the columns): q = 0
    // mean, 1 c, 2 + 2 i and 3 + 2 i the cos and sin coefficients of low mode i
    for (int q = kProjWaves - 1 - wave; q < 2 + (LOW ? 2 * modes.n : 0); q += kProjWaves) {
        double s = 0.0;
        if (q < 2) {
            for (int y = lane; y < L; y += 64) s += q == 0 ? rows[L + y] : ((y & 1) ? -rows[y] : rows[y]);
        } else if constexpr (LOW) {
            const int kx = modes.kx[(q - 2) >> 1], ky = modes.ky[(q - 2) >> 1];
            const double* cx = rows + (int64_t)(kx == 0 ? 1 : 2 * kx) * L;   // sums against cos(kx x ..), sin(kx x ..)
            const double* sn = rows + (int64_t)(2 * kx + 1) * L;
            for (int y = lane; y < L; y += 64) {
                const int t = twiddle_index(ky, y, L);
                const double pc = cx[y], ps = kx == 0 ? 0.0 : sn[y];
                s += (q & 1) ? ps * ct[t] + pc * st[t] : pc * ct[t] - ps * st[t];
            }
        }
        s = wave_sum(s);
        if (lane == 0) fin[q] = q == 0 ? s * inv * inv : (q == 1 ? s * inv : 2.0 * s * inv * inv);
    }
    __syncthreads();
    const double mean = fin[0], cnn = fin[1], sx0 = (lane & 1) ? -1.0 : 1.0;
    for (int b = blockIdx.x; b < nparts; b += gridDim.x) {
        const int y0 = b * ROWS + wave;
        if constexpr (LOW) {
            if (b > (int)blockIdx.x) __syncthreads();   // the last rows' coefficients are read
            if (threadIdx.x < ROWS) {
                const int y = b * ROWS + threadIdx.x;
                double a0 = mean, a1 = 0.0, b1 = 0.0, a2 = 0.0, b2 = 0.0;
                for (int m = 0; m < modes.n; ++m) {
                    const int kx = modes.kx[m], t = twiddle_index(modes.ky[m], y < L ? y : 0, L);
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
                coef[0 * ROWS + threadIdx.x] = a0;
                coef[1 * ROWS + threadIdx.x] = a1;
                coef[2 * ROWS + threadIdx.x] = b1;
                coef[3 * ROWS + threadIdx.x] = a2;
                coef[4 * ROWS + threadIdx.x] = b2;
            }
            __syncthreads();
        }
        for (int g = 0; g < L; g += 64 * J) {
            if (g > 0 || b > (int)blockIdx.x) project_load(A, L, y0, g, v);
#pragma unroll
            for (int i = 0; i < RPW; ++i) {
                const int y = y0 + 16 * i, r = wave + 16 * i;
                if (y >= L) break;
                const double sy = (y & 1) ? -1.0 : 1.0, ry = rows[y];
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const int x = g + lane + 64 * j;
                    if (x < L) {
                        double low = mean;
                        if constexpr (LOW) {
                            const int x2 = twiddle_index(2, x, L);
                            low = coef[r] + coef[ROWS + r] * ct[x] + coef[2 * ROWS + r] * st[x] + coef[3 * ROWS + r] * ct[x2] +
                                  coef[4 * ROWS + r] * st[x2];
                        }
                        A[(int64_t)y * L + x] = v[i][j] - sx0 * ry - sy * (cols[x] - sx0 * cnn) - low;
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
// then those first nodes.  One problem of 256^2: 109 us in one launch, 10 in three
// (launch-bound: the kernels take 4 + 4 + 2).
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
// Lattices from which the split projection is taken, by size alone up to kSplitPlanes planes
// (a problem's result is the same in every batch of up to 64).  us with one workgroup per
// plane and split, 4 planes and 256: 128^2 12.2 and 7.5, but 15.4 and 25.8; 160^2 19.4 and
// 8.1, 29.7 and 35.6; 256^2 31 and 8.8, 62 and 71; with low modes 160^2 34 and 17, but 45
// and 82; 192^2 38 and 18, 52 and 97; 256^2 52 and 18, 76 and 131; 1024^2 805 and 54,
// 1476 and 1565.  (The whole chip has work with 256 planes: above that one workgroup each
// is faster up to 384^2 and as fast beyond.)
constexpr int split_min(bool low) { return low ? 192 : 160; }
constexpr int kSplitPlanes = 256, kSplitGroups = 512;

int done(hipError_t e) { return e == hipSuccess ? LB_OK : LB_EHIP; }

int launch_prolong(int planes, int Lc, const PlaneScales& a, const double* x, const PlaneScales& b, const double* y,
                   const PlaneScales& c, const double* z, double* dst, hipStream_t s) {
    const unsigned blocks = ((unsigned)(2 * Lc) * (unsigned)(2 * Lc) + kBlock - 1) / kBlock;
    for (int p0 = 0; p0 < planes; p0 += kMaxPlanes)
        hipLaunchKernelGGL(prolong_k, dim3(blocks, (unsigned)std::min(kMaxPlanes, planes - p0)), dim3(kBlock), 0, s, p0, Lc, a,
                           x, b, y, c, z, dst);
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
    const PlaneScales one{{scale, scale, scale}, 0}, none{};
    return launch_prolong(planes, Lc, none, nullptr, one, src, none, nullptr, dst, (hipStream_t)stream);
}

int lb_warm_prolong_fields(int32_t batch, int32_t Lc, const double a[3], const double* x, const double b[3], const double* y,
                           const double c[3], const double* z, double* dst, void* stream) {
    if (batch < 1 || batch > (1 << 28) || Lc < 2 || 2 * Lc > LB_WARM_MAX_L || (x && !a) || !b || !y || (z && !c) || !dst)
        return LB_EINVAL;
    auto scales = [&](const double* s) { return s ? PlaneScales{{s[0], s[1], s[2]}, batch} : PlaneScales{}; };
    return launch_prolong(4 * batch, Lc, scales(a), x, scales(b), y, scales(c), z, dst, (hipStream_t)stream);
}

int lb_warm_axpby(int64_t n, double a, const double* x, double b, const double* y, double* out, void* stream) {
    if (n < 0 || (n > 0 && (!x || !y || !out))) return LB_EINVAL;
    if (n == 0) return LB_OK;
    hipLaunchKernelGGL(axpby_k, dim3(grid_for(n)), dim3(kBlock), 0, (hipStream_t)stream, n, a, x, b, y, out);
    return done(hipGetLastError());
}

// The half plane's low modes (one of each +-k pair: kx > 0, or kx = 0 and ky > 0); LB_EINVAL
// for arguments that a projection refuses.
static int low_modes(int planes, int L, int k2max, LowModes* m) {
    if (planes < 1 || L < 2 || L > LB_WARM_MAX_L || (L & 1) || k2max < 0 || k2max > LB_WARM_MAX_K2) return LB_EINVAL;
    *m = LowModes{};
    for (int kx = 0; kx * kx <= k2max; ++kx)
        for (int ky = -3; ky <= 3; ++ky) {
            if (kx * kx + ky * ky == 0 || kx * kx + ky * ky > k2max) continue;
            if (kx == 0 && ky <= 0) continue;
            if (2 * kx >= L || 2 * (ky < 0 ? -ky : ky) >= L) return LB_EINVAL;   // |k| far below the Nyquist lines
            m->kx[m->n] = (int8_t)kx;
            m->ky[m->n++] = (int8_t)ky;
        }
    return LB_OK;
}

int lb_warm_project(double* data, int32_t planes, int32_t L, int32_t k2max, void* stream) {
    LowModes low;
    if (!data || low_modes(planes, L, k2max, &low) != LB_OK) return LB_EINVAL;
    const int n = low.n;
    int m[2 * kMaxLowModes] = {0};
    for (int i = 0; i < n; ++i) {
        m[2 * i] = low.kx[i];
        m[2 * i + 1] = low.ky[i];
    }
    const size_t lds = project_lds_bytes(L, n);
    const int4 ma = make_int4(m[0], m[1], m[2], m[3]), mb = make_int4(m[4], m[5], m[6], m[7]),
               mc = make_int4(m[8], m[9], m[10], m[11]), md = make_int4(m[12], m[13], m[14], m[15]),
               me = make_int4(m[16], m[17], m[18], m[19]), mf = make_int4(m[20], m[21], m[22], m[23]);
    const int J = project_columns(L, n);
    auto plain = J == 1 ? project_k<1, false> : J == 2 ? project_k<2, false> : project_k<4, false>;
    auto with_low = J == 1 ? project_k<1, true> : project_k<2, true>;
    auto kernel = n > 0 ? with_low : plain;
    if (lds > 65536) {   // the largest lattices need more than the default dynamic LDS limit
        const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return LB_EHIP;
    }
    hipLaunchKernelGGL(kernel, dim3(planes), dim3(kProjBlock), lds, (hipStream_t)stream, data, (int)L, n, ma, mb, mc,
                       md, me, mf);
    return done(hipGetLastError());
}

int64_t lb_warm_project_work(int32_t planes, int32_t L, int32_t k2max) {
    LowModes low;
    if (low_modes(planes, L, k2max, &low) != LB_OK || L < split_min(low.n > 0) || planes > kSplitPlanes) return 0;
    return planes * split_work(L, low.n > 0);
}

int lb_warm_project_split(double* data, int32_t planes, int32_t L, int32_t k2max, double* work, void* stream) {
    LowModes low;
    if (!data || !work || low_modes(planes, L, k2max, &low) != LB_OK || lb_warm_project_work(planes, L, k2max) == 0)
        return LB_EINVAL;
    const int rpw = split_rows(L) / 16;
    const int parts = split_parts(L);
    const int groups = 2 * parts * planes <= 3 * kSplitGroups ? parts : (kSplitGroups + planes - 1) / planes;
    const dim3 grid((unsigned)groups, (unsigned)planes), block(kProjBlock);
    const hipStream_t st = (hipStream_t)stream;
    static_assert((kProjWaves * 64 * 4 + 2 * LB_WARM_MAX_L) * sizeof(double) <= 65536, "default dynamic LDS");
    static_assert((3 * LB_WARM_MAX_L + kProjSums + 5 * 64) * sizeof(double) <= 65536, "default dynamic LDS");
    static_assert(split_rows(LB_WARM_MAX_L) <= 64, "at most four rows per wavefront");
    const int table = low.n > 0 ? 2 * L : 0;
    const size_t lds_sums = (kProjWaves * 64 * sums_columns(rpw) + table) * sizeof(double);
    const size_t lds_apply = (L + kProjSums + 5 * 16 * rpw + table) * sizeof(double);
    auto launch = [&](auto sums, auto apply) {
        hipLaunchKernelGGL(sums, grid, block, lds_sums, st, data, (int)L, work);
        hipLaunchKernelGGL(apply, grid, block, lds_apply, st, data, (int)L, low, work);
        return done(hipGetLastError());
    };
    if (low.n > 0)
        return rpw == 1 ? launch(project_sums_k<1, true>, project_apply_k<1, true>)
             : rpw == 2 ? launch(project_sums_k<2, true>, project_apply_k<2, true>)
             : rpw == 3 ? launch(project_sums_k<3, true>, project_apply_k<3, true>)
                        : launch(project_sums_k<4, true>, project_apply_k<4, true>);
    return rpw == 1 ? launch(project_sums_k<1, false>, project_apply_k<1, false>)
         : rpw == 2 ? launch(project_sums_k<2, false>, project_apply_k<2, false>)
         : rpw == 3 ? launch(project_sums_k<3, false>, project_apply_k<3, false>)
                    : launch(project_sums_k<4, false>, project_apply_k<4, false>);
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
    // outputs that share memory with an input are written only after every sum: one workgroup each
    bool apart = true;
    for (const double* in : {drho, phi, S})
        apart = apart && !overlap(in, all, rho_out, all) && !overlap(in, all, u_out, 2 * all) && !overlap(in, all, phi_out, all);
    for (const double* in : {u, F})
        apart = apart && !overlap(in, 2 * all, rho_out, all) && !overlap(in, 2 * all, u_out, 2 * all) && !overlap(in, 2 * all, phi_out, all);
    // from where three launches, about 5 us of host time each, cost less than one: us in one
    // launch and in three, 64^2 12.5 and 15.5, 88^2 15.5 and 15, 96^2 18 and 15 (64 problems
    // 21.6 and 20.4)
    if (zero_momentum && apart && n >= 7744) {
        for (int64_t b0 = 0; b0 < batch; b0 += kMaxPlanes) {
            const unsigned bs = (unsigned)std::min<int64_t>(kMaxPlanes, batch - b0);
            const int64_t o = b0 * n;
            const InitArgs a{drho + o, u + o, phi ? phi + o : nullptr, F + o, S ? S + o : nullptr, n, all, rho0,
                             rho_out + o, u_out + o, phi_out ? phi_out + o : nullptr};
            hipLaunchKernelGGL(initial_sums_k, dim3(kInitParts, bs), dim3(kBlock), 0, (hipStream_t)stream, a);
            hipLaunchKernelGGL(initial_rest_k, dim3((unsigned)((n - kInitParts + kBlock - 1) / kBlock), bs), dim3(kBlock), 0,
                               (hipStream_t)stream, a);
            hipLaunchKernelGGL(initial_first_k, dim3(bs), dim3(kInitParts), 0, (hipStream_t)stream, a);
        }
        return done(hipGetLastError());
    }
    hipLaunchKernelGGL(initial_state_k, dim3(batch), dim3(kProjBlock), 0, (hipStream_t)stream, drho, u, phi, F, S,
                       (int)batch, n, rho0, (int)(zero_momentum != 0), rho_out, u_out, phi_out);
    return done(hipGetLastError());
}

}  // extern "C"
