// Weight and bias gradients of the network's 3x3 convolutions with the pixel
// tiles transposed in LDS: dW[o][tap][c] = sum_p g[p][o] x[p shifted by tap][c],
// db[o] = sum_p g[p][o].
//
// The contraction runs over pixels, so a matrix-core fragment is 8 consecutive
// pixels of one channel, while memory holds consecutive channels of one pixel.
// A workgroup stages a 256-pixel tile (32 x 8, or 16 x 16 at width 16) of the
// gradient's 16 outputs o and of the input's 16 CT channels c with its circular
// halo, transposed: a thread loads two neighbouring pixels in 16-byte pieces
// and writes one word (both pixels) per channel, so that a fragment is one
// 16-byte LDS read; the fragments shifted by one pixel along x come from the
// same read and its two neighbouring words by five byte alignments.  A halo
// row's three fragments serve up to three output rows, so a wavefront does 18
// products per channel tile for 2 + 4 fragment reads.  Wavefront w takes the
// pixel chunks 2w and 2w + 1 of every tile; a workgroup steps through every
// gridDim.x-th tile with the next one's loads in flight, keeps its 9 CT
// accumulators in registers, and the four wavefronts' sums are added in LDS in
// a fixed order at the end.  The bias gradient adds the same float32 values as
// they are staged.
//
// Bound by reading the gradient (fp32) and the input once: 16 x 16 channels at
// 256^2, batch 16, 21 us (96 MB, 4.6 TB/s).  Gathering the fragments from global
// memory one value at a time instead (wgrad_mfma) spends 38 load instructions per
// nine products; over the 18 layers 680 us of a training step, and 240 for the
// separate bias sums, against 250 here.
#include <hip/hip_runtime.h>

#include "nn.hpp"

namespace casclb {
namespace nn {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

__device__ __forceinline__ int wrap(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

__device__ __forceinline__ uint32_t pack2(float a, float b) {
    const __bf16 lo = (__bf16)a, hi = (__bf16)b;
    return (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
}

template <int TW>
struct Px {
    static constexpr int TH = 256 / TW, RP = 32 / TW;      // rows per tile, rows per 32-pixel chunk
    static constexpr int HH = TH + 2, PAIRS = TW / 2 + 2;  // halo rows; pixel pairs (-2, -1) .. (TW, TW + 1) of a row
    static constexpr int XR = TW == 32 ? 48 : 32;          // elements per halo row: pixel x at 8 + x
    static constexpr int XS = HH * XR + 8;                 // elements per input channel (reads of 8 lanes hit distinct banks)
    static constexpr int GS = 256 + 8;                     // elements per output channel
};

template <int TW, int CT>
__global__ void __launch_bounds__(256, 2) wgrad_lds(WgradArgs a) {
    using P = Px<TW>;
    constexpr int CH = 2 * CT;                               // 8-channel pieces of the input
    constexpr int XN = (P::HH * P::PAIRS * CH + 255) / 256;  // pixel pairs x pieces per thread
    extern __shared__ __align__(16) unsigned char lds_raw[];
    uint16_t* gt = reinterpret_cast<uint16_t*>(lds_raw);     // [16][GS]
    uint16_t* xt = gt + 16 * P::GS;                          // [16 CT][XS]
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6, grp = lane >> 4, col = lane & 15;
    const int ot_n = a.co_pad16 / 16, ot = (int)blockIdx.y % ot_n, cg = (int)blockIdx.y / ot_n;
    const uint32_t tiles_x = (uint32_t)(a.w / TW), tiles_y = (uint32_t)(a.h / P::TH);
    const uint32_t tiles = (uint32_t)a.n * tiles_x * tiles_y;
    const char* gbase = reinterpret_cast<const char*>(a.g.base);
    const char* xbase = reinterpret_cast<const char*>(a.x.base);
    const char* x2base = reinterpret_cast<const char*>(a.x2.base);
    const int ct_n = a.ci_pad16 / 16 - cg * CT < CT ? a.ci_pad16 / 16 - cg * CT : CT;   // channel tiles of this group

    f32x4 gl[2][2];    // [round][pixel of the pair]: 4 channels
    u32x4 xl[XN][2];   // [item][pixel of the pair]: 8 channels
    auto load = [&](uint32_t b) {
        const uint32_t trow = a.div_w.div(b), tx = b - trow * tiles_x;
        const uint32_t img = a.div_h.div(trow), ty = trow - img * tiles_y;
        const uint32_t img_row = img * (uint32_t)a.h;
        const int x0 = (int)tx * TW, y0 = (int)ty * P::TH;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const uint32_t pair = (uint32_t)(r * 64 + (tid >> 2)), q = 2 * pair;   // tile pixel q, q + 1
            const uint32_t row = q / TW, px = q % TW;
            const uint32_t pix = (img_row + (uint32_t)y0 + row) * (uint32_t)a.w + (uint32_t)x0 + px;
            const uint32_t off = (pix * (uint32_t)a.g.cs + (uint32_t)(a.g.co + ot * 16 + 4 * (tid & 3))) * 4u;
            gl[r][0] = *reinterpret_cast<const f32x4*>(gbase + off);
            gl[r][1] = *reinterpret_cast<const f32x4*>(gbase + (off + 4u * (uint32_t)a.g.cs));
        }
#pragma unroll
        for (int r = 0; r < XN; ++r) {
            const uint32_t e = (uint32_t)(r * 256 + tid);
            const uint32_t piece = e % CH, pair = e / CH, row = pair / P::PAIRS, k = pair - row * P::PAIRS;
            if (row < (uint32_t)P::HH && (int)(piece >> 1) < ct_n) {
                const uint32_t yy = (uint32_t)wrap(y0 - 1 + (int)row, a.h);
                const int xa = x0 - 2 + 2 * (int)k;   // the pair's pixels xa, xa + 1 (the outermost two are not used)
                const uint32_t pa = (img_row + yy) * (uint32_t)a.w + (uint32_t)wrap(xa, a.w);
                const uint32_t pb = (img_row + yy) * (uint32_t)a.w + (uint32_t)wrap(xa + 1, a.w);
                const uint32_t c = (uint32_t)(cg * CT * 16) + 8 * piece;
                if ((int)c < a.c_split) {
                    const uint32_t co = (uint32_t)a.x.co + c;
                    xl[r][0] = *reinterpret_cast<const u32x4*>(xbase + (pa * (uint32_t)a.x.cs + co) * 2u);
                    xl[r][1] = *reinterpret_cast<const u32x4*>(xbase + (pb * (uint32_t)a.x.cs + co) * 2u);
                } else {
                    const uint32_t half = ((img_row >> 1) + (yy >> 1)) * (uint32_t)(a.w >> 1), co = (uint32_t)a.x2.co + c - (uint32_t)a.c_split;
                    const uint32_t qa = half + ((uint32_t)wrap(xa, a.w) >> 1), qb = half + ((uint32_t)wrap(xa + 1, a.w) >> 1);
                    xl[r][0] = *reinterpret_cast<const u32x4*>(x2base + (qa * (uint32_t)a.x2.cs + co) * 2u);
                    xl[r][1] = *reinterpret_cast<const u32x4*>(x2base + (qb * (uint32_t)a.x2.cs + co) * 2u);
                }
            }
        }
    };
    f32x4 bias = {0.f, 0.f, 0.f, 0.f};
    auto store = [&]() {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int pair = r * 64 + (tid >> 2);
            bias += gl[r][0] + gl[r][1];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                *reinterpret_cast<uint32_t*>(gt + (4 * (tid & 3) + j) * P::GS + 2 * pair) = pack2(gl[r][0][j], gl[r][1][j]);
        }
#pragma unroll
        for (int r = 0; r < XN; ++r) {
            const uint32_t e = (uint32_t)(r * 256 + tid);
            const uint32_t piece = e % CH, pair = e / CH, row = pair / P::PAIRS, k = pair - row * P::PAIRS;
            if (row < (uint32_t)P::HH && (int)(piece >> 1) < ct_n) {
                uint16_t* to = xt + 8 * piece * P::XS + row * P::XR + 6 + 2 * k;
#pragma unroll
                for (int j = 0; j < 4; ++j) {   // channels 2j, 2j + 1: low and high halves of the two pixels
                    *reinterpret_cast<uint32_t*>(to + (2 * j) * P::XS) =
                        __builtin_amdgcn_perm(xl[r][1][j], xl[r][0][j], 0x05040100u);
                    *reinterpret_cast<uint32_t*>(to + (2 * j + 1) * P::XS) =
                        __builtin_amdgcn_perm(xl[r][1][j], xl[r][0][j], 0x07060302u);
                }
            }
        }
    };

    f32x4 acc[CT][9];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[c][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint16_t* gm = gt + col * P::GS + 64 * wave + 8 * grp;
    const uint16_t* xm = xt + col * P::XS + (2 * wave * P::RP + grp / (TW / 8)) * P::XR + 8 + 8 * (grp % (TW / 8));

    load(blockIdx.x);   // gridDim.x <= tiles
    for (uint32_t b = blockIdx.x; b < tiles; b += gridDim.x) {
        store();
        __syncthreads();
        if (b + gridDim.x < tiles) load(b + gridDim.x);
        bf16x8 av[2];
        av[0] = *reinterpret_cast<const bf16x8*>(gm);
        av[1] = *reinterpret_cast<const bf16x8*>(gm + 32);
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            if (c < ct_n) {
#pragma unroll
                for (int j = 0; j <= P::RP + 2; ++j) {   // halo rows: tap row dy of chunk i reads row i RP + dy
                    const uint16_t* at = xm + c * 16 * P::XS + j * P::XR;
                    const u32x4 v = *reinterpret_cast<const u32x4*>(at);
                    const uint32_t l = *reinterpret_cast<const uint32_t*>(at - 2), r = *reinterpret_cast<const uint32_t*>(at + 8);
                    const uint32_t s0 = __builtin_amdgcn_alignbit(v[0], l, 16), s1 = __builtin_amdgcn_alignbit(v[1], v[0], 16),
                                   s2 = __builtin_amdgcn_alignbit(v[2], v[1], 16), s3 = __builtin_amdgcn_alignbit(v[3], v[2], 16),
                                   s4 = __builtin_amdgcn_alignbit(r, v[3], 16);
                    const bf16x8 bv[3] = {__builtin_bit_cast(bf16x8, (u32x4{s0, s1, s2, s3})), __builtin_bit_cast(bf16x8, v),
                                          __builtin_bit_cast(bf16x8, (u32x4{s1, s2, s3, s4}))};
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const int dy = j - i * P::RP;
                        if (dy >= 0 && dy <= 2)
#pragma unroll
                            for (int dx = 0; dx < 3; ++dx)
                                acc[c][3 * dy + dx] =
                                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], bv[dx], acc[c][3 * dy + dx], 0, 0, 0);
                    }
                }
            }
        }
        __syncthreads();   // the fragments are read before the next tile overwrites them
    }

    // ---- the wavefronts' sums, three taps at a time: D row 4 grp + j = output, column col = input
    float* red = reinterpret_cast<float*>(lds_raw);   // [4][3][256]
    const int64_t record = (int64_t)a.co_pad16 * 9 * a.ci_pad16 + a.co_pad16;
    float* out = a.partials + (int64_t)blockIdx.x * record;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        if (c < ct_n) {
#pragma unroll
            for (int t0 = 0; t0 < 9; t0 += 3) {
                __syncthreads();
#pragma unroll
                for (int t = 0; t < 3; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j) red[(wave * 3 + t) * 256 + (4 * grp + j) * 16 + col] = acc[c][t0 + t][j];
                __syncthreads();
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    const float s = ((red[t * 256 + tid] + red[(3 + t) * 256 + tid]) + red[(6 + t) * 256 + tid]) +
                                    red[(9 + t) * 256 + tid];
                    const int o = ot * 16 + (tid >> 4), ci = (cg * CT + c) * 16 + (tid & 15);
                    out[((int64_t)o * 9 + t0 + t) * a.ci_pad16 + ci] = s;
                }
            }
        }
    }
    if (cg == 0) {
        // bias: the 16 threads of a wavefront with the same 4 channels, then the wavefronts in order
#pragma unroll
        for (int j = 0; j < 4; ++j)
            for (int off = 4; off < 64; off <<= 1) bias[j] += __shfl_xor(bias[j], off, 64);
        __syncthreads();
        if (lane < 4)
#pragma unroll
            for (int j = 0; j < 4; ++j) red[wave * 16 + 4 * lane + j] = bias[j];
        __syncthreads();
        if (tid < 16)
            out[(int64_t)a.co_pad16 * 9 * a.ci_pad16 + ot * 16 + tid] =
                ((red[tid] + red[16 + tid]) + red[32 + tid]) + red[48 + tid];
    }
}

template <int TW, int CT>
hipError_t launch_ct(const WgradArgs& a, hipStream_t s) {
    using P = Px<TW>;
    WgradArgs b = a;
    b.div_w = FastDiv((uint32_t)(a.w / TW));
    b.div_h = FastDiv((uint32_t)(a.h / P::TH));
    const size_t tile = (size_t)(16 * P::GS + 16 * CT * P::XS) * 2, sums = (size_t)4 * 3 * 256 * sizeof(float);
    const size_t lds = tile > sums ? tile : sums;
    if (lds > 65536) {
        const hipError_t e = hipFuncSetAttribute((const void*)wgrad_lds<TW, CT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    const int groups = (a.ci_pad16 / 16 + CT - 1) / CT;
    hipLaunchKernelGGL((wgrad_lds<TW, CT>), dim3((unsigned)a.splits, (unsigned)(groups * (a.co_pad16 / 16))), dim3(256), lds,
                       s, b);
    return hipGetLastError();
}

template <int TW>
hipError_t launch_tw(const WgradArgs& a, hipStream_t s) {
    const int ct = a.ci_pad16 / 16;
    if (ct == 1) return launch_ct<TW, 1>(a, s);
    if (ct == 2 || ct == 4) return launch_ct<TW, 2>(a, s);
    return launch_ct<TW, 3>(a, s);
}

}  // namespace

// Workgroups over the tiles: about two per CU with those of the channel groups.
int32_t wgrad_lds_splits(int32_t n, int32_t h, int32_t w, int32_t co_pad16, int32_t ci_pad16) {
    if (w % 16) return 0;
    const int tw = w % 32 ? 16 : 32, th = 256 / tw;
    if (h % th) return 0;
    const int ct = ci_pad16 / 16, per = ct == 1 ? 1 : (ct == 2 || ct == 4 ? 2 : 3);
    const int64_t tiles = (int64_t)n * (h / th) * (w / tw), groups = (int64_t)((ct + per - 1) / per) * (co_pad16 / 16);
    const int64_t want = (512 + groups - 1) / groups;
    return (int32_t)(tiles < want ? tiles : want);
}

hipError_t launch_wgrad_lds(const WgradArgs& a, hipStream_t s) {
    if (a.splits < 1 || a.splits > wgrad_lds_splits(a.n, a.h, a.w, a.co_pad16, a.ci_pad16)) return hipErrorInvalidValue;
    return a.w % 32 ? launch_tw<16>(a, s) : launch_tw<32>(a, s);
}

// The tensors' byte offsets fit 32 bits and every padded channel is there to read.
bool wgrad_lds_fits(const WgradArgs& a) {
    const int64_t px = (int64_t)a.n * a.h * a.w;
    return px * a.g.cs * 4 < ((int64_t)1 << 32) && px * a.x.cs * 2 < ((int64_t)1 << 32) &&
           a.g.co % 4 == 0 && a.g.cs % 4 == 0 && a.x.co % 8 == 0 && a.x.cs % 8 == 0 &&
           a.g.co + a.co_pad16 <= a.g.cs && a.c_split % 16 == 0 && a.x.co + a.c_split <= a.x.cs &&
           (a.c_split == a.ci_pad16 || (a.x2.co % 8 == 0 && a.x2.cs % 8 == 0 && px / 4 * a.x2.cs * 2 < ((int64_t)1 << 32) &&
                                        a.x2.co + a.ci_pad16 - a.c_split <= a.x2.cs));
}

}  // namespace nn
}  // namespace casclb
