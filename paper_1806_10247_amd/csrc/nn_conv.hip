// The network's 3x3 convolutions with the input tile in LDS (forward and input
// gradient), bf16 matrix cores, fp32 accumulation.
//
// Workgroup = 4 wavefronts = one TH x TW pixel tile of one image and NU
// 16-channel output tiles.  The tile and its one-pixel circular halo are staged
// in LDS as bf16 (pixel stride CI + 8 elements: 16-byte reads of consecutive
// pixels hit distinct banks).  A wavefront owns T matrix-core tiles of 16
// consecutive pixels.  The products are D = W X: the rows of D are output
// channels, its columns pixels, so that a lane ends with four consecutive
// channels of one pixel and the epilogue works on them as one 8- or 16-byte
// piece: bias, ReLU and the 2 x 2 means forward; the ReLU mask of the next
// gradient and the adjoints of the upsampling (2 x 2 sums) and of the pooling (a
// quarter added to four pixels) backward.
//
// Everything but the tensors' sizes is a template argument (channels CI, tile,
// input and output kind), so that the K loop is straight code: K runs over
// k = tap * CI + c in slices of 32, lane group g taking the 8 channels at
// 32 s + 8 g; a slice spans at most two taps, so its LDS offset is one constant
// or a choice of two by g, and the T tiles differ by constants in the
// instructions.  The slices and their order are those of conv3x3_mfma: the same
// float32 sums.  What bounds it: at 256^2 memory and the staging (a 16-channel
// layer does 20 products per wavefront for 680 staged 16-byte pieces) and, with
// one output tile, the LDS reads (one 1 KB fragment per product); at the coarse
// levels one workgroup's latency; there T = 2 and one output tile per workgroup
// spread the layer over more CUs.  Measured at batch 16, 256^2 (us): 13 raw inputs
// to 16 channels 28, 16 to 16 20 (72 MB, 3.6 TB/s), 48 to 16 42, 16 to 4 15;
// 64^2 and coarser 6-8 a layer.  A workgroup that steps through several tiles with
// the next one's loads in flight was slower (48 to 16 50): its registers cost more
// workgroups per CU than it overlaps.  Whole inference: batch 16 384 -> 245 us,
// batch 1 183 -> 94 us against the kernel before it (run-time channel counts,
// two-byte stores, the input and output copied).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "nn.hpp"
#include "nn_tile.hpp"

namespace casclb {
namespace nn {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;

template <int N, class F>
__device__ __forceinline__ void unrolled(F&& f) {
    if constexpr (N > 0) {
        unrolled<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

__device__ __forceinline__ int wrap(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

__device__ __forceinline__ float shuffle_x1(float v) {   // the value of lane ^ 1
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));
}

// v with 0 where channels c .. c + 3 of pixel px of the bf16 view m are not > 0.
__device__ __forceinline__ f32x4 masked(f32x4 v, const View& m, size_t px, int c) {
    if (m.base) {
        const bf16x4 a = *reinterpret_cast<const bf16x4*>(reinterpret_cast<const bf16_t*>(m.base) +
                                                          px * (uint32_t)m.cs + (uint32_t)(m.co + c));
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (!((float)a[j] > 0.0f)) v[j] = 0.0f;
    }
    return v;
}

enum Input { kBf16 = 0, kF32 = 1, kRaw = 2 };

// Pieces of one tile's input held in registers between their loads and their
// LDS stores: all of a thread's pieces, loads issued together.
template <int CI, int TW, int T, int XM>
struct Staged {
    using G = Tile<CI, TW, T>;
    static constexpr int PIECES = G::NP * G::CPP;
    static constexpr int N = (PIECES + 255) / 256;
    bf16x8 v[XM == kBf16 ? N : 1];
    f32x4 f[XM == kF32 ? 2 * N : 1];

    __device__ __forceinline__ void load(const ConvArgs& a, uint32_t img_row, int y0, int x0) {
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const uint32_t e = r * 256 + threadIdx.x;
            if (e < (uint32_t)PIECES) {
                const uint32_t q = e / G::CPP, c0 = 8 * (e - q * G::CPP);
                const uint32_t qy = q / G::HW, qx = q - qy * G::HW;
                const uint32_t yy = (uint32_t)wrap(y0 - 1 + (int)qy, a.h), xx = (uint32_t)wrap(x0 - 1 + (int)qx, a.w);
                const size_t px = (size_t)((img_row + yy) * (uint32_t)a.w + xx);
                if constexpr (XM == kF32) {
                    const float* p = reinterpret_cast<const float*>(a.x.base) + px * (uint32_t)a.x.cs + (uint32_t)a.x.co + c0;
                    f[2 * r] = *reinterpret_cast<const f32x4*>(p);
                    f[2 * r + 1] = *reinterpret_cast<const f32x4*>(p + 4);
                } else if ((int)c0 < a.c_split) {
                    v[r] = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const bf16_t*>(a.x.base) +
                                                           px * (uint32_t)a.x.cs + (uint32_t)a.x.co + c0);
                } else {
                    const size_t p2 = ((img_row >> 1) + (yy >> 1)) * (uint32_t)(a.w >> 1) + (xx >> 1);
                    v[r] = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const bf16_t*>(a.x2.base) +
                                                           p2 * (uint32_t)a.x2.cs + (uint32_t)a.x2.co + c0 -
                                                           (uint32_t)a.c_split);
                }
            }
        }
    }
    __device__ __forceinline__ void store(const ConvArgs&, bf16_t* tile, uint32_t, int, int) {
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const uint32_t e = r * 256 + threadIdx.x;
            if (e < (uint32_t)PIECES) {
                const uint32_t q = e / G::CPP, c0 = 8 * (e - q * G::CPP);
                bf16x8 w;
                if constexpr (XM == kF32) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        w[c] = (__bf16)f[2 * r][c];
                        w[c + 4] = (__bf16)f[2 * r + 1][c];
                    }
                } else {
                    w = v[r];
                }
                *reinterpret_cast<bf16x8*>(tile + q * G::PS + c0) = w;
            }
        }
    }
};

// Raw fp32, cin_raw floats per pixel: copied to LDS as it lies in memory (16-byte
// pieces; the two halo columns apart), then each thread packs whole pixels.
template <int TW, int T>
struct Staged<16, TW, T, kRaw> {
    using G = Tile<16, TW, T>;
    static constexpr int N = (G::HH * TW * 16 / 4 + 255) / 256, NE = (2 * G::HH * 16 + 255) / 256;   // at most 16 floats
    f32x4 in[N];
    float out[NE];

    __device__ __forceinline__ void load(const ConvArgs& a, uint32_t img_row, int y0, int x0) {
        const uint32_t cr = (uint32_t)a.cin_raw, per_row = TW / 4 * cr;
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const uint32_t i = r * 256 + threadIdx.x;
            if (i < G::HH * per_row) {
                const uint32_t row = a.div_raw.div(i), k = i - row * per_row;
                const uint32_t yy = (uint32_t)wrap(y0 - 1 + (int)row, a.h);
                in[r] = *reinterpret_cast<const f32x4*>(
                    a.xin + (((size_t)(img_row + yy) * (uint32_t)a.w + (uint32_t)x0) * cr + 4 * k));
            }
        }
#pragma unroll
        for (int r = 0; r < NE; ++r) {
            const uint32_t i = r * 256 + threadIdx.x;
            if (i < 2 * G::HH * cr) {
                const uint32_t px = a.div_cin.div(i), c = i - px * cr;
                const uint32_t yy = (uint32_t)wrap(y0 - 1 + (int)(px >> 1), a.h);
                const uint32_t xx = (uint32_t)wrap(px & 1 ? x0 + TW : x0 - 1, a.w);
                out[r] = a.xin[((size_t)(img_row + yy) * (uint32_t)a.w + xx) * cr + c];
            }
        }
    }
    __device__ __forceinline__ void store(const ConvArgs& a, bf16_t* tile, uint32_t img_row, int y0, int x0) {
        const uint32_t cr = (uint32_t)a.cin_raw, inner_n = G::HH * (TW / 4) * cr;
        float* inner = reinterpret_cast<float*>(tile + G::LDS);          // [HH][TW * cr]
        float* edge = inner + G::HH * TW * cr;                           // [HH][2][cr]
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const uint32_t i = r * 256 + threadIdx.x;
            if (i < inner_n) *reinterpret_cast<f32x4*>(inner + 4 * i) = in[r];
        }
#pragma unroll
        for (int r = 0; r < NE; ++r) {
            const uint32_t i = r * 256 + threadIdx.x;
            if (i < 2 * G::HH * cr) edge[i] = out[r];
        }
        __syncthreads();
        for (uint32_t q = threadIdx.x; q < (uint32_t)G::NP; q += 256) {
            const uint32_t qy = q / G::HW, qx = q - qy * G::HW;
            const float* src = qx == 0 ? edge + 2 * qy * cr
                                       : (qx == G::HW - 1 ? edge + (2 * qy + 1) * cr : inner + (qy * TW + qx - 1) * cr);
            bf16x8 lo, hi;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                lo[c] = (__bf16)(c < (int)cr ? src[c] : 0.0f);
                hi[c] = (__bf16)(c + 8 < (int)cr ? src[c + 8] : 0.0f);
            }
            *reinterpret_cast<bf16x8*>(tile + q * G::PS) = lo;
            *reinterpret_cast<bf16x8*>(tile + q * G::PS + 8) = hi;
            if (a.pack.base && blockIdx.y == 0 && qx >= 1 && qx <= (uint32_t)TW && qy >= 1 && qy <= (uint32_t)G::TH) {
                const size_t px = (size_t)(img_row + (uint32_t)y0 + qy - 1) * (uint32_t)a.w + (uint32_t)x0 + qx - 1;
                bf16_t* to = reinterpret_cast<bf16_t*>(a.pack.base) + px * (uint32_t)a.pack.cs + (uint32_t)a.pack.co;
                *reinterpret_cast<bf16x8*>(to) = lo;
                *reinterpret_cast<bf16x8*>(to + 8) = hi;
            }
        }
    }
};

template <int CI, int TW, int T, int XM, bool YF32, int NU, int PF>
__global__ void __launch_bounds__(256) conv3x3_lds(ConvArgs a) {
    using G = Tile<CI, TW, T>;
    static_assert(T % G::TPR == 0 && G::R % 2 == 0, "whole pairs of pixel rows per wavefront");
    extern __shared__ __align__(16) unsigned char lds_raw[];
    bf16_t* tile = reinterpret_cast<bf16_t*>(lds_raw);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, grp = lane >> 4, col = lane & 15;
    const uint32_t tiles_x = (uint32_t)(a.w / TW), tiles_y = (uint32_t)(a.h / G::TH);
    const uint32_t trow = a.div_w.div(blockIdx.x), tx = blockIdx.x - trow * tiles_x;
    const uint32_t img = a.div_h.div(trow), ty = trow - img * tiles_y;
    const uint32_t img_row = img * (uint32_t)a.h;
    const int x0 = (int)tx * TW, y0 = (int)ty * G::TH;
    const int cg = (int)blockIdx.y * NU, co16 = (a.co + 15) >> 4;

    // weights of the first PF slices, in flight while the tile is staged
    const bf16_t* wrow = a.wt + (uint32_t)(cg * 16 + col) * (uint32_t)G::KPAD + 8 * grp;
    bf16x8 bq[PF][NU];
    auto load_weights = [&](auto ss) {
        constexpr int s = decltype(ss)::value;
#pragma unroll
        for (int u = 0; u < NU; ++u)
            if (cg + u < co16) bq[s % PF][u] = *reinterpret_cast<const bf16x8*>(wrow + u * 16 * G::KPAD + 32 * s);
    };

    Staged<CI, TW, T, XM> staged;
    staged.load(a, img_row, y0, x0);
    unrolled<(PF < G::S ? PF : G::S)>(load_weights);
    staged.store(a, tile, img_row, y0, x0);
    __syncthreads();

    // ---- products
    f32x4 acc[T][NU];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int u = 0; u < NU; ++u) acc[t][u] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16_t* mine = tile + (wave * G::R * G::HW + col) * G::PS + 8 * grp;
    unrolled<G::S>([&](auto ss) {
        constexpr int s = decltype(ss)::value;
        bf16x8 bc[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) bc[u] = bq[s % PF][u];
        if constexpr (s + PF < G::S) load_weights(std::integral_constant<int, s + PF>{});
        constexpr int first = G::offset(4 * s), second = G::offset(4 * s + 3), at = G::split(s), live = G::live(s);
        const int off = first == second ? first : (grp >= at ? second : first);
        bf16x8 av[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            av[t] = *reinterpret_cast<const bf16x8*>(mine + off + ((t / G::TPR) * G::HW + 16 * (t % G::TPR)) * G::PS);
            if constexpr (live < 4) {   // past the end of K: zeros, whatever the pixel holds
                if (grp >= live)
#pragma unroll
                    for (int c = 0; c < 8; ++c) av[t][c] = (__bf16)0.0f;
            }
        }
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int t = 0; t < T; ++t)
                acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bc[u], av[t], acc[t][u], 0, 0, 0);
    });

    // ---- epilogue: channels o .. o + 3 of pixel (row, x0 + 16 (t % TPR) + col)
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int o = (cg + u) * 16 + 4 * grp;
        if (cg + u >= co16 || o >= a.co) continue;
        float bias[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) bias[j] = a.bias && o + j < a.co ? a.bias[o + j] : 0.0f;
        f32x4 v[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const uint32_t row = img_row + (uint32_t)(y0 + wave * G::R + t / G::TPR);
            const size_t px = row * (uint32_t)a.w + (uint32_t)(x0 + 16 * (t % G::TPR) + col);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[t][j] = acc[t][u][j] + bias[j];
                if (a.relu) v[t][j] = fmaxf(v[t][j], 0.0f);
            }
            if constexpr (YF32) {
                if (a.add.base) {
                    const uint32_t fw = 2 * (uint32_t)a.w;   // the finer level's width
                    const size_t fine = (size_t)(2 * row) * fw + 2 * (uint32_t)(x0 + 16 * (t % G::TPR) + col);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const size_t q = fine + (k >> 1) * fw + (k & 1);
                        float* d = reinterpret_cast<float*>(a.add.base) + q * (uint32_t)a.add.cs + (uint32_t)(a.add.co + o);
                        const f32x4 sum = *reinterpret_cast<const f32x4*>(d) + 0.25f * v[t];
                        *reinterpret_cast<f32x4*>(d) = masked(sum, a.add_mask, q, o);
                    }
                } else if (!(a.sum.base && o >= a.sum_from)) {
                    v[t] = masked(v[t], a.mask, px, o);
                    float* d = reinterpret_cast<float*>(a.y.base) + px * (uint32_t)a.y.cs + (uint32_t)(a.y.co + o);
                    if (o + 4 <= a.co && a.y_vec) {
                        *reinterpret_cast<f32x4*>(d) = v[t];
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (o + j < a.co) d[j] = v[t][j];
                    }
                }
            } else {
                bf16x4 h;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    h[j] = (__bf16)v[t][j];
                    v[t][j] = (float)h[j];
                }
                *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16_t*>(a.y.base) + px * (uint32_t)a.y.cs +
                                           (uint32_t)(a.y.co + o)) = h;
            }
        }
        if constexpr (YF32) {
            if (a.sum.base && o >= a.sum_from) {   // 2 x 2 sums, in the order of upsample_bwd_k
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    if ((t / G::TPR) % 2) continue;   // the upper row of each pair
                    f32x4 sum;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        sum[j] = (v[t][j] + shuffle_x1(v[t][j])) + (v[t + G::TPR][j] + shuffle_x1(v[t + G::TPR][j]));
                    if ((col & 1) == 0) {
                        const uint32_t row = (img_row >> 1) + (uint32_t)((y0 + wave * G::R + t / G::TPR) >> 1);
                        const size_t px = row * (uint32_t)(a.w >> 1) + (uint32_t)((x0 + 16 * (t % G::TPR) + col) >> 1);
                        const int c = o - a.sum_from;
                        *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.sum.base) + px * (uint32_t)a.sum.cs +
                                                  (uint32_t)(a.sum.co + c)) = masked(sum, a.sum_mask, px, c);
                    }
                }
            }
        } else {
            if (a.pool.base) {   // 2 x 2 means of the bf16 outputs, in the order of avgpool_k
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    if ((t / G::TPR) % 2) continue;   // the upper row of each pair
                    bf16x4 h;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float top = v[t][j] + shuffle_x1(v[t][j]);
                        const float bottom = v[t + G::TPR][j] + shuffle_x1(v[t + G::TPR][j]);
                        h[j] = (__bf16)(0.25f * (top + bottom));
                    }
                    if ((col & 1) == 0) {
                        const uint32_t row = (img_row >> 1) + (uint32_t)((y0 + wave * G::R + t / G::TPR) >> 1);
                        const size_t px = row * (uint32_t)(a.w >> 1) + (uint32_t)((x0 + 16 * (t % G::TPR) + col) >> 1);
                        *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16_t*>(a.pool.base) + px * (uint32_t)a.pool.cs +
                                                   (uint32_t)(a.pool.co + o)) = h;
                    }
                }
            }
        }
    }
}

template <int CI, int TW, int T, int XM, bool YF32, int NU>
hipError_t launch_nu(const ConvArgs& a, hipStream_t s) {
    using G = Tile<CI, TW, T>;
    constexpr int PF = T == 2 ? (G::S < 6 ? G::S : 6) : 2;
    ConvArgs b = a;
    b.div_w = FastDiv((uint32_t)(a.w / TW));
    b.div_h = FastDiv((uint32_t)(a.h / G::TH));
    b.y_vec = a.y.cs % 4 == 0 && a.y.co % 4 == 0 && ((uintptr_t)a.y.base & 15) == 0;
    size_t lds = (size_t)G::LDS * sizeof(bf16_t);
    if (XM == kRaw) {
        b.div_raw = FastDiv((uint32_t)(TW / 4 * a.cin_raw));
        b.div_cin = FastDiv((uint32_t)a.cin_raw);
        lds += (size_t)G::HH * (TW + 2) * a.cin_raw * sizeof(float);
    }
    const auto kernel = conv3x3_lds<CI, TW, T, XM, YF32, NU, PF>;
    if (lds > 65536) {   // above the default dynamic LDS limit
        const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    const int co16 = (a.co + 15) / 16;
    const int64_t tiles = (int64_t)a.n * (a.h / G::TH) * (a.w / TW);
    const dim3 grid((unsigned)tiles, (unsigned)((co16 + NU - 1) / NU));
    hipLaunchKernelGGL(kernel, grid, dim3(256), lds, s, b);
    return hipGetLastError();
}

// Launches of at least this many 32 x 8 tiles fill the chip with them (two
// workgroups per CU); smaller ones take 16 x 8 tiles, one output tile each.
constexpr int64_t kWideTiles = 512;

template <int CI, int XM, bool YF32>
hipError_t launch_ci(const ConvArgs& a, hipStream_t s) {
    const int co16 = (a.co + 15) / 16;
    if constexpr (CI <= 96) {
        if (a.w % 32 == 0 && (int64_t)a.n * (a.h / 8) * (a.w / 32) >= kWideTiles) {
            if (co16 == 1) return launch_nu<CI, 32, 4, XM, YF32, 1>(a, s);
            if (co16 % 3 == 0) return launch_nu<CI, 32, 4, XM, YF32, 3>(a, s);
            return launch_nu<CI, 32, 4, XM, YF32, 2>(a, s);
        }
    }
    return launch_nu<CI, 16, 2, XM, YF32, 1>(a, s);
}

template <int XM, bool YF32>
hipError_t launch_xm(const ConvArgs& a, hipStream_t s) {
    switch (a.ci_pad) {
        case 16: return launch_ci<16, XM, YF32>(a, s);
        case 32: return launch_ci<32, XM, YF32>(a, s);
        case 48: return launch_ci<48, XM, YF32>(a, s);
        case 64: return launch_ci<64, XM, YF32>(a, s);
        case 80: return launch_ci<80, XM, YF32>(a, s);
        case 96: return launch_ci<96, XM, YF32>(a, s);
        case 112: return launch_ci<112, XM, YF32>(a, s);
        case 128: return launch_ci<128, XM, YF32>(a, s);
        case 160: return launch_ci<160, XM, YF32>(a, s);
        case 192: return launch_ci<192, XM, YF32>(a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

bool conv_lds_fits(const ConvArgs& a) {
    const int32_t ci = a.ci_pad;
    if (!(ci >= 16 && ci % 16 == 0 && (ci <= 128 || ci == 160 || ci == 192))) return false;
    if (a.w % 16 || a.h % 8 || a.kpad != (9 * ci + 31) / 32 * 32) return false;
    // pixel numbers and element offsets within an image row are 32-bit
    return (int64_t)a.n * a.h * a.w < ((int64_t)1 << 31);
}

hipError_t launch_conv_lds(const ConvArgs& a, bool x_f32, bool y_f32, hipStream_t s) {
    if (!conv_lds_fits(a)) return hipErrorInvalidValue;
    if (a.xin) {
        // 16-byte pieces of the raw input
        if (a.ci_pad != 16 || a.cin_raw < 1 || a.cin_raw > 16 || y_f32 || ((uintptr_t)a.xin & 15)) return hipErrorInvalidValue;
        return launch_ci<16, kRaw, false>(a, s);
    }
    if (x_f32) return y_f32 ? launch_xm<kF32, true>(a, s) : hipErrorInvalidValue;
    if (!y_f32) return launch_xm<kBf16, false>(a, s);
    return launch_xm<kBf16, true>(a, s);
}

}  // namespace nn
}  // namespace casclb
