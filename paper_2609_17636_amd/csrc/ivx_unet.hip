// Learned warm start: a U-Net (Ronneberger et al. 2015) on the dirty mosaic, trained on
// converged cold-start solutions of the Classic3D objective.  Every layer is a kernel
// here; the 3x3 convolutions are implicit GEMMs on the bf16 matrix cores.
//
// Implicit GEMM of a 3x3 convolution, NHWC: rows = output pixels p, columns = output
// channels o, reduction index k = (dy * 3 + dx) * Cin + c.  A[p][k] is the input pixel
// shifted by (dy - 1, dx - 1) (zero outside), B[k][o] = W[o][dy][dx][c].  The products run on
// gfx950's v_mfma_f32_16x16x32_bf16, one per 32-wide k step of a 16 x 16 output tile:
//   A operand : lane l holds A[l % 16][8 (l / 16) + v], v = 0..7 (8 consecutive k)
//   B operand : lane l holds B[8 (l / 16) + v][l % 16]  (the same 8 k of one column)
//   result    : lane l holds D[4 (l / 16) + v][l % 16], v = 0..3
// (A and B give each lane the same k indices, so the product does not depend on the order in
// which the instruction walks them.)
// The transposed correlation (gradient of the input) is the same kernel on flipped
// weights, and the weight gradient is a second implicit GEMM (rows o, columns k, reduction
// over pixels) split over pixel ranges with a fixed-order reduction of the partials.
#include "ivx_internal.hpp"
#include "ivx_unet.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <random>
#include <string>
#include <vector>

namespace ivx {
ivx_status set_error(ivx_status s, const std::string &msg); // defined with the objective ABI
}

using namespace ivx;

namespace {

constexpr int NT = 256;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// 8 bf16 values (as raw 16-bit patterns, element 0 in the low half of word 0) as an operand
__device__ __forceinline__ bf16x8 as_bf16x8(uint4 u) { return __builtin_bit_cast(bf16x8, u); }
__device__ __forceinline__ uint4 pack8(const uint16_t *e) {
    return uint4{e[0] | ((uint32_t)e[1] << 16), e[2] | ((uint32_t)e[3] << 16), e[4] | ((uint32_t)e[5] << 16),
                 e[6] | ((uint32_t)e[7] << 16)};
}
__device__ __forceinline__ f32x4 mma(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// ---------------------------------------------------------------- 3x3 convolution
template <int NTW>
__global__ __launch_bounds__(NT) void k_conv3x3(const float *__restrict__ x, int n, int h, int w, int cin,
                                                const uint16_t *__restrict__ wt, const float *__restrict__ bias,
                                                int cout, int relu, const float *__restrict__ mask, int accumulate,
                                                float *__restrict__ y, uint16_t *__restrict__ yb) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t P = (int64_t)n * h * w;
    const int64_t pbase = (int64_t)blockIdx.x * 64 + wave * 16;
    const int cobase = blockIdx.y * (16 * NTW);
    const int K = 9 * cin;
    const int row = lane & 15, kq = lane >> 4;
    const int64_t p = pbase + row;
    const bool pv = p < P;
    int pn = 0, py = 0, px = 0;
    if (pv) {
        pn = (int)(p / ((int64_t)h * w));
        const int r = (int)(p - (int64_t)pn * h * w);
        py = r / w;
        px = r - py * w;
    }
    f32x4 acc[NTW];
#pragma unroll
    for (int t = 0; t < NTW; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < K; k0 += 32) {
        // the lane's 8 k: two runs of 4 channels (cin % 4 == 0: each run stays in one tap)
        uint16_t ae[8];
#pragma unroll
        for (int hlf = 0; hlf < 2; ++hlf) {
            const int k = k0 + 8 * kq + 4 * hlf;
            float4 v = float4{0.f, 0.f, 0.f, 0.f};
            if (pv && k < K) {
                const int tap = k / cin, c = k - (k / cin) * cin;
                const int yy = py + tap / 3 - 1, xx = px + tap % 3 - 1;
                if (yy >= 0 && yy < h && xx >= 0 && xx < w)
                    v = *reinterpret_cast<const float4 *>(x + (((int64_t)pn * h + yy) * w + xx) * cin + c);
            }
            ae[4 * hlf + 0] = f2bf(v.x);
            ae[4 * hlf + 1] = f2bf(v.y);
            ae[4 * hlf + 2] = f2bf(v.z);
            ae[4 * hlf + 3] = f2bf(v.w);
        }
        const bf16x8 a = as_bf16x8(pack8(ae));
#pragma unroll
        for (int t = 0; t < NTW; ++t) {
            const int co = cobase + t * 16 + row;
            uint2 u[2] = {uint2{0u, 0u}, uint2{0u, 0u}};
#pragma unroll
            for (int hlf = 0; hlf < 2; ++hlf) {
                const int k = k0 + 8 * kq + 4 * hlf;
                if (co < cout && k < K) u[hlf] = *reinterpret_cast<const uint2 *>(wt + (int64_t)co * K + k);
            }
            acc[t] = mma(a, as_bf16x8(uint4{u[0].x, u[0].y, u[1].x, u[1].y}), acc[t]);
        }
    }
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
        const int co = cobase + t * 16 + row;
        if (co >= cout) continue;
        const float bb = bias ? bias[co] : 0.f;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t pp = pbase + 4 * kq + v;
            if (pp >= P) continue;
            const int64_t o = pp * cout + co;
            float val = acc[t][v] + bb;
            if (relu) val = fmaxf(val, 0.f);
            if (mask && !(mask[o] > 0.f)) val = 0.f;
            if (accumulate) val += y[o];
            if (y) y[o] = val;
            if (yb) yb[o] = f2bf(val);
        }
    }
}

// LDS-tiled implicit GEMM for the 3x3 convolution: block tile 64 pixels x BN channels
// (BN = 32 NJ), k chunks of 32 staged in LDS as bf16 (A: [pixel][k], B: [channel][k], rows
// padded to 40 elements), 4 waves in a 2 x 2 arrangement, each wave 2 x NJ tiles of
// v_mfma_f32_16x16x32_bf16 (one per chunk).  The next chunk's global loads are issued before
// the current chunk's matrix products.  (FP32 layers that the kernels below do not take or take slower: conv3x3_layer.)
constexpr int TBM = 64, TBK = 32, TLD = 40;
template <int NJ>
__global__ __launch_bounds__(NT) void k_conv3x3_tiled(const float *__restrict__ x, int n, int h, int w, int cin,
                                                      const uint16_t *__restrict__ wt, const float *__restrict__ bias,
                                                      int cout, int relu, const float *__restrict__ mask,
                                                      int accumulate, float *__restrict__ y) {
    constexpr int BN = 32 * NJ;
    __shared__ __align__(16) uint16_t As[TBM * TLD];
    __shared__ __align__(16) uint16_t Bs[BN * TLD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t P = (int64_t)n * h * w;
    const int K = 9 * cin;
    const int64_t m0 = (int64_t)blockIdx.x * TBM;
    const int n0 = blockIdx.y * BN;
    // ---- global -> register staging: A (pixel am, k quarter aq), B (channel rows)
    const int am = tid >> 2, aq = (tid & 3) * 8;
    const int64_t ap = m0 + am;
    int apn = 0, apy = 0, apx = 0;
    const bool apv = ap < P;
    if (apv) {
        apn = (int)(ap / ((int64_t)h * w));
        const int r = (int)(ap - (int64_t)apn * h * w);
        apy = r / w;
        apx = r - apy * w;
    }
    constexpr int BPIECES = BN * (TBK / 8);           // 8-element pieces of one B chunk
    constexpr int BROWS = (BPIECES + NT - 1) / NT;    // per thread (1 or 2)
    uint16_t ra[8];
    uint16_t rb[BROWS][8];
    auto gload = [&](int k0) {
#pragma unroll
        for (int hlf = 0; hlf < 2; ++hlf) {
            const int k = k0 + aq + 4 * hlf;
            float4 v = float4{0.f, 0.f, 0.f, 0.f};
            if (apv && k < K) {
                const int tap = k / cin, c = k - tap * cin;
                const int yy = apy + tap / 3 - 1, xx = apx + tap % 3 - 1;
                if (yy >= 0 && yy < h && xx >= 0 && xx < w)
                    v = *reinterpret_cast<const float4 *>(x + (((int64_t)apn * h + yy) * w + xx) * cin + c);
            }
            ra[4 * hlf + 0] = f2bf(v.x);
            ra[4 * hlf + 1] = f2bf(v.y);
            ra[4 * hlf + 2] = f2bf(v.z);
            ra[4 * hlf + 3] = f2bf(v.w);
        }
#pragma unroll
        for (int b = 0; b < BROWS; ++b) {
            const int e = tid + b * NT;
            const int o = e >> 2, bq = (e & 3) * 8;
#pragma unroll
            for (int hlf = 0; hlf < 2; ++hlf) {
                const int k = k0 + bq + 4 * hlf;
                uint2 u = uint2{0u, 0u};
                if (e < BPIECES && n0 + o < cout && k < K) u = *reinterpret_cast<const uint2 *>(wt + (int64_t)(n0 + o) * K + k);
                rb[b][4 * hlf + 0] = (uint16_t)(u.x & 0xFFFFu);
                rb[b][4 * hlf + 1] = (uint16_t)(u.x >> 16);
                rb[b][4 * hlf + 2] = (uint16_t)(u.y & 0xFFFFu);
                rb[b][4 * hlf + 3] = (uint16_t)(u.y >> 16);
            }
        }
    };
    auto sstore = [&]() {
        uint4 va;
        va.x = ra[0] | ((uint32_t)ra[1] << 16);
        va.y = ra[2] | ((uint32_t)ra[3] << 16);
        va.z = ra[4] | ((uint32_t)ra[5] << 16);
        va.w = ra[6] | ((uint32_t)ra[7] << 16);
        *reinterpret_cast<uint4 *>(&As[am * TLD + aq]) = va;
#pragma unroll
        for (int b = 0; b < BROWS; ++b) {
            const int e = tid + b * NT;
            if (e >= BPIECES) continue;
            const int o = e >> 2, bq = (e & 3) * 8;
            uint4 vb;
            vb.x = rb[b][0] | ((uint32_t)rb[b][1] << 16);
            vb.y = rb[b][2] | ((uint32_t)rb[b][3] << 16);
            vb.z = rb[b][4] | ((uint32_t)rb[b][5] << 16);
            vb.w = rb[b][6] | ((uint32_t)rb[b][7] << 16);
            *reinterpret_cast<uint4 *>(&Bs[o * TLD + bq]) = vb;
        }
    };
    // ---- matrix products: wave (wr, wc) owns rows 32 wr .. +32, columns 16 NJ wc .. +16 NJ
    const int wr = wave >> 1, wc = wave & 1;
    const int row = lane & 15, kq = lane >> 4;
    f32x4 acc[2][NJ];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nch = (K + TBK - 1) / TBK;
    gload(0);
    for (int kc = 0; kc < nch; ++kc) {
        __syncthreads();
        sstore();
        __syncthreads();
        if (kc + 1 < nch) gload((kc + 1) * TBK);
        static_assert(TBK == 32, "one 16x16x32 product per chunk");
        bf16x8 af[2], bfr[NJ];
#pragma unroll
        for (int i = 0; i < 2; ++i)
            af[i] = as_bf16x8(*reinterpret_cast<const uint4 *>(&As[(wr * 32 + i * 16 + row) * TLD + 8 * kq]));
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            bfr[j] = as_bf16x8(*reinterpret_cast<const uint4 *>(&Bs[(wc * 16 * NJ + j * 16 + row) * TLD + 8 * kq]));
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] = mma(af[i], bfr[j], acc[i][j]);
    }
    // ---- epilogue: D row (pixel) 4 kq + v, column (channel) = row index of the lane
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int co = n0 + wc * 16 * NJ + j * 16 + row;
            if (co >= cout) continue;
            const float bb = bias ? bias[co] : 0.f;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t pp = m0 + wr * 32 + i * 16 + 4 * kq + v;
                if (pp >= P) continue;
                const int64_t o = pp * cout + co;
                float val = acc[i][j][v] + bb;
                if (relu) val = fmaxf(val, 0.f);
                if (mask && !(mask[o] > 0.f)) val = 0.f;
                if (accumulate) val += y[o];
                y[o] = val;
            }
        }
}

// ------------------------------------------------- 3x3 convolution, one wave per output tile
// Input of a convolution as 8-channel pieces: bf16 activations (16 bytes a piece) or FP32 ones
// rounded to bf16 as they are loaded.  A second source continues the channels of the first, and the
// first may be at half resolution: the decoder's concatenation of an upsampled level and a skip is
// read in place instead of being written out.
template <typename T> struct ConvIn {
    const T *x0, *x1; // channels [0, ca) and [ca, cin)
    int ca;
    int half0;        // x0 is [n][h / 2][w / 2][ca]
};

// Output of a convolution: FP32 and / or bf16, [P][cout]; with `split` > 0 the FP32 output is two
// tensors, channels [0, split) in y and the rest in y1.
struct ConvOut {
    float *y, *y1;
    uint16_t *yb;
    int split;
    const float *bias;
    int relu, accumulate;
    const float *maskf;      // FP32 mask [P][cout] or NULL
    ConvIn<uint16_t> maskb;  // bf16 mask (x0 NULL: none)
};

// Buffer view of `bytes` from p: a load whose offset is not below the view's size returns 0, which is
// the padding of the image (a lane outside takes NO_PIECE), with no branch and no second address.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr unsigned NO_PIECE = 0x80000000u;
template <typename T> __device__ __forceinline__ __amdgpu_buffer_rsrc_t view(const T *p, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(p), 0, (int)(bytes < 0x7FFFFFFF ? bytes : 0x7FFFFFFF), 0x00020000);
}
// Eight channels at byte offset vo, as raw bf16 bits.  (No scalar offset: it is taken off the view's
// size in the range check, which wraps where the size is smaller.)
template <typename T> __device__ __forceinline__ uint4 load_raw(__amdgpu_buffer_rsrc_t r, unsigned vo) {
    const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(r, vo, 0, 0);
    if constexpr (sizeof(T) == 2) return uint4{a[0], a[1], a[2], a[3]};
    else {
        typedef float f32x4_ __attribute__((ext_vector_type(4)));
        const f32x4_ f = __builtin_bit_cast(f32x4_, a);
        const f32x4_ g = __builtin_bit_cast(f32x4_, __builtin_amdgcn_raw_buffer_load_b128(r, vo + 16, 0, 0));
        return __builtin_bit_cast(uint4, bf16x8{(__bf16)f[0], (__bf16)f[1], (__bf16)f[2], (__bf16)f[3], (__bf16)g[0],
                                                (__bf16)g[1], (__bf16)g[2], (__bf16)g[3]});
    }
}
template <typename T> __device__ __forceinline__ const T *uniform_ptr(const T *p) {
    const uint64_t u = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)u), hi = __builtin_amdgcn_readfirstlane((int)(u >> 32));
    return (const T *)((uint64_t)hi << 32 | lo);
}

// Four consecutive channels co .. co + 3 of pixel p = (img, py, px): bias, ReLU, mask, sum, store.
__device__ __forceinline__ void store_out(const ConvOut &out, f32x4 acc, int64_t p, int64_t img, int py, int px, int h,
                                          int w, int cout, int co) {
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = acc[e] + (out.bias ? out.bias[co + e] : 0.f);
        if (out.relu) v[e] = fmaxf(v[e], 0.f);
    }
    if (out.maskf) {
        const float4 q = *reinterpret_cast<const float4 *>(out.maskf + p * cout + co);
        v[0] = q.x > 0.f ? v[0] : 0.f;
        v[1] = q.y > 0.f ? v[1] : 0.f;
        v[2] = q.z > 0.f ? v[2] : 0.f;
        v[3] = q.w > 0.f ? v[3] : 0.f;
    }
    if (out.maskb.x0) { // activations after a ReLU: a positive bf16 is a positive 16-bit integer
        const bool first = co < out.maskb.ca;
        const int sh = first ? out.maskb.half0 : 0;
        const int64_t pix = (img * (h >> sh) + (py >> sh)) * (w >> sh) + (px >> sh);
        const uint16_t *at = first ? out.maskb.x0 + pix * out.maskb.ca + co
                                   : out.maskb.x1 + pix * (cout - out.maskb.ca) + (co - out.maskb.ca);
        const uint2 q = *reinterpret_cast<const uint2 *>(at);
        v[0] = (int16_t)(q.x & 0xFFFF) > 0 ? v[0] : 0.f;
        v[1] = (int16_t)(q.x >> 16) > 0 ? v[1] : 0.f;
        v[2] = (int16_t)(q.y & 0xFFFF) > 0 ? v[2] : 0.f;
        v[3] = (int16_t)(q.y >> 16) > 0 ? v[3] : 0.f;
    }
    if (out.y) {
        float4 *o = reinterpret_cast<float4 *>(out.split == 0     ? out.y + p * cout + co
                                               : co < out.split ? out.y + p * out.split + co
                                                                : out.y1 + p * (cout - out.split) + (co - out.split));
        if (out.accumulate) {
            const float4 q = *o;
            v[0] += q.x;
            v[1] += q.y;
            v[2] += q.z;
            v[3] += q.w;
        }
        *o = float4{v[0], v[1], v[2], v[3]};
    }
    if (out.yb) {
        typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
        *reinterpret_cast<uint2 *>(out.yb + p * cout + co) =
            __builtin_bit_cast(uint2, bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]});
    }
}

// Channel counts that the patch kernel below does not take (not both multiples of 32).  Output tile of one wave: 16 MI pixels x 16 NJ channels, K in 32-wide steps, operands
// straight from global memory (each lane's 8 consecutive k are 16 contiguous bytes of a pixel or of a weight
// row), DEPTH steps in flight; bound by those loads.
// The order of the steps fixes the bits of the sums: tap-major, or (chunks) channel-chunk-major.
// ANYC: cin is a multiple of 8 but not of 32 (a step spans taps).
template <typename T, int MI, int NJ, int DEPTH, bool ANYC>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 8))) void
k_conv3x3_wave(ConvIn<T> in, int n, int h, int w, int cin, const uint16_t *__restrict__ wt, int packed, int cout, int chunks,
               ConvOut out) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15, kq = lane >> 4;
    const int64_t P = (int64_t)n * h * w;
    const int64_t m0 = ((int64_t)blockIdx.x * 4 + wave) * (16 * MI);
    const int n0 = blockIdx.y * (16 * NJ);
    if (m0 >= P) return;
    const int K = 9 * cin, ca = in.ca, cb = cin - in.ca;
    constexpr int SZ = (int)sizeof(T);
    const int half0 = in.half0, w2 = w >> 1, h2 = h >> 1;
    // The wave's pixels start at (img0, py0): its views of the sources start above them, so offsets are
    // small and not negative whatever the size of the tensor.
    const int64_t img0 = m0 / ((int64_t)h * w);
    const int py0 = (int)(m0 - img0 * h * w) / w;
    const int64_t first1 = m0 - w - 1;                                             // tap (0, 0) of pixel m0
    const int row0 = py0 > 0 ? (py0 - 1) >> 1 : 0;                                 // its row at half resolution
    const int64_t first0 = half0 ? (img0 * h2 + row0) * w2 : first1;
    const __amdgpu_buffer_rsrc_t r0 =
        view(uniform_ptr(in.x0 + first0 * ca), ((half0 ? (int64_t)n * h2 * w2 : P) - first0) * ca * SZ);
    const __amdgpu_buffer_rsrc_t r1 = view(uniform_ptr(in.x1 + first1 * cb), (P - first1) * cb * SZ);
    const __amdgpu_buffer_rsrc_t rw = view(wt + (int64_t)n0 * K, (int64_t)(cout - n0) * K * 2);
    // pixel of operand row `row` of each tile and the taps that stay inside the image
    int py[MI], px[MI], ok[MI];
    int64_t img[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int64_t p = m0 + 16 * i + row, q = p < P ? p : P - 1;
        img[i] = q / ((int64_t)h * w);
        const int r = (int)(q - img[i] * h * w);
        py[i] = r / w;
        px[i] = r - py[i] * w;
        const int rows = (py[i] > 0 ? 7 : 0) | 7 << 3 | (py[i] + 1 < h ? 7 << 6 : 0);
        const int cols = (px[i] > 0 ? 0x49 : 0) | 0x92 | (px[i] + 1 < w ? 0x124 : 0);
        ok[i] = p < P ? rows & cols : 0;
    }
    // byte offset of pixel i's channel 0 at a tap, in the half-resolution source
    auto half_at = [&](int i, int dy, int dx) {
        return (unsigned)(((int)(img[i] - img0) * h2 - row0 + ((py[i] + dy) >> 1)) * w2 + ((px[i] + dx) >> 1)) *
               (unsigned)(ca * SZ);
    };
    const int wsh = !ANYC && packed ? 4 : 0; // (packed: a step is 1 KB per 16 channels)
    const unsigned wlane = wsh ? 16u * lane : (unsigned)(row * K + 8 * kq) * 2u; // (cout is a multiple of 16 NJ)
    const int nc = cin / 32, steps = ANYC ? (K + 31) / 32 : 9 * nc;
    int tap = 0, ch = 0, ks = 0; // the next step to load
    f32x4 acc[NJ][MI];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < MI; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    uint4 av[DEPTH][MI], wv[DEPTH][NJ];
    // One step of operands (steps past the last load zeros: the products after it add nothing)
#define IVX_CONV_LOAD(d)                                                                                        \
    do {                                                                                                        \
        if (ANYC) { /* a lane's eight k lie in one tap, the lanes' in several */                                \
            const int k = ks + 8 * kq, t = k / cin, c = k - t * cin, dy = t / 3 - 1, dx = t - 3 * (t / 3) - 1;  \
            _Pragma("unroll") for (int i = 0; i < MI; ++i) {                                                    \
                const bool in_k = k < K && ((ok[i] >> t) & 1);                                                  \
                unsigned o0 = half0 ? half_at(i, dy, dx) : (unsigned)(16 * i + row + (dy + 1) * w + dx + 1) * (unsigned)(ca * SZ); \
                unsigned o1 = (unsigned)(16 * i + row + (dy + 1) * w + dx + 1) * (unsigned)(cb * SZ);           \
                const uint4 a0 = load_raw<T>(r0, in_k && c < ca ? o0 + (unsigned)(c * SZ) : NO_PIECE);       \
                av[d][i] = a0;                                                                                  \
                if (cb) {                                                                                       \
                    const uint4 a1 = load_raw<T>(r1, in_k && c >= ca ? o1 + (unsigned)((c - ca) * SZ) : NO_PIECE); \
                    av[d][i] = uint4{a0.x | a1.x, a0.y | a1.y, a0.z | a1.z, a0.w | a1.w};                       \
                }                                                                                               \
            }                                                                                                   \
            _Pragma("unroll") for (int j = 0; j < NJ; ++j)                                                      \
                wv[d][j] = load_raw<uint16_t>(rw, k < K ? wlane + (unsigned)(32 * j * K + 2 * ks) : NO_PIECE); \
            ks += 32;                                                                                           \
        } else {                                                                                                \
            const int c = 32 * ch, dy = tap / 3 - 1, dx = tap - 3 * (tap / 3) - 1;                              \
            const int live = tap < 9 && ch < nc ? 1 : 0;                                                        \
            if (half0 && c < ca) {                                                                              \
                _Pragma("unroll") for (int i = 0; i < MI; ++i)                                                  \
                    av[d][i] = load_raw<T>(r0, (ok[i] >> tap) & live ? half_at(i, dy, dx) + (unsigned)((c + 8 * kq) * SZ) : NO_PIECE); \
            } else {                                                                                            \
                const bool a0 = c < ca || cb == 0;                                                              \
                const int cs = a0 ? ca : cb;                                                                    \
                const unsigned so = (unsigned)((((dy + 1) * w + dx + 1) * cs + (a0 ? c : c - ca)) * SZ);        \
                _Pragma("unroll") for (int i = 0; i < MI; ++i) {                                                \
                    const unsigned vo = (ok[i] >> tap) & live ? (unsigned)(((16 * i + row) * cs + 8 * kq) * SZ) + so : NO_PIECE; \
                    av[d][i] = a0 ? load_raw<T>(r0, vo) : load_raw<T>(r1, vo);                            \
                }                                                                                               \
            }                                                                                                   \
            _Pragma("unroll") for (int j = 0; j < NJ; ++j)                                                      \
                wv[d][j] = load_raw<uint16_t>(rw, live ? wlane + (unsigned)(32 * j * K + (2 * (tap * cin + c) << wsh)) : NO_PIECE);                                 \
            if (chunks) {                                                                                       \
                if (++tap == 9) tap = 0, ++ch;                                                                  \
            } else {                                                                                            \
                if (++ch == nc) ch = 0, ++tap;                                                                  \
            }                                                                                                   \
        }                                                                                                       \
    } while (0)
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) IVX_CONV_LOAD(d);
    for (int s0 = 0; s0 < steps; s0 += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int i = 0; i < MI; ++i) acc[j][i] = mma(as_bf16x8(wv[d][j]), as_bf16x8(av[d][i]), acc[j][i]);
            IVX_CONV_LOAD(d);
        }
    }
#undef IVX_CONV_LOAD
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int64_t p = m0 + 16 * i + row;
        if (p >= P) continue;
#pragma unroll
        for (int j = 0; j < NJ; ++j) store_out(out, acc[j][i], p, img[i], py[i], px[i], h, w, cout, n0 + 16 * j + 4 * kq);
    }
}

// Network layers on images whose rows are too long for 32-bit offsets into the three rows of a pixel (2^28 and more channels a row):
// 16 pixels x 16 channels a wave at 64-bit addresses.
__global__ __launch_bounds__(NT) void k_conv3x3_far(ConvIn<uint16_t> in, int n, int h, int w, int cin,
                                                    const uint16_t *__restrict__ wt, int packed, int cout, ConvOut out) {
    const int lane = threadIdx.x & 63, row = lane & 15, kq = lane >> 4;
    const int64_t P = (int64_t)n * h * w, p = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16 + row, q = p < P ? p : P - 1;
    const int64_t img = q / ((int64_t)h * w);
    const int py = (int)((q - img * h * w) / w), px = (int)(q - (img * h + py) * w);
    const int n0 = blockIdx.y * 16, K = 9 * cin, ca = in.ca, cb = cin - in.ca;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < K; k0 += 32) {
        const int k = k0 + 8 * kq, t = k / cin, c = k - t * cin, yy = py + t / 3 - 1, xx = px + t % 3 - 1;
        uint4 a = {0u, 0u, 0u, 0u}, b = {0u, 0u, 0u, 0u};
        if (k < K) {
            b = *reinterpret_cast<const uint4 *>(
                wt + (packed ? ((int64_t)(n0 >> 4) * (K >> 5) + (k >> 5)) * 512 + 8 * lane : (int64_t)(n0 + row) * K + k));
            if (p < P && yy >= 0 && yy < h && xx >= 0 && xx < w) {
                const int sh = c < ca ? in.half0 : 0;
                const int64_t pix = (img * (h >> sh) + (yy >> sh)) * (w >> sh) + (xx >> sh);
                a = *reinterpret_cast<const uint4 *>(c < ca ? in.x0 + pix * ca + c : in.x1 + pix * cb + (c - ca));
            }
        }
        acc = mma(as_bf16x8(b), as_bf16x8(a), acc);
    }
    if (p < P) store_out(out, acc, p, img, py, px, h, w, cout, n0 + 4 * kq);
}

// A block of WM x WN waves owns 2 WM rows x 32 columns of one image and 16 NJ WN output channels.  The
// patch with its one-pixel halo is staged in LDS once, all input channels of it (the order of the steps
// runs over channels inside the taps) or, where these do not fit, cp at a time, and serves the nine taps; the weights stay in the vector cache,
// DEPTH steps ahead (9 cin / 32 steps: DEPTH divides them).  A wave takes 64 pixels x 16 NJ channels: per 32-wide
// step 4 LDS reads, NJ weight loads, 4 NJ products.  Position rows are padded by 16 bytes, so that eight
// lanes' reads of consecutive positions cover all banks.
// Bound by the weight loads and the staging, which the block's own products do not hide (three blocks a CU
// do): 64 -> 64 channels at 16 x 128^2 in 44 us (440 TFLOP/s), 128 -> 128 at 16 x 64^2 in 31 us (620); staged per
// chunk and tap from FP32 activations these took 155 and 133 us.  One 256^2 image, whose deep levels
// are chains of 36 to 108 dependent steps on few blocks: 10 to 20 us a layer, from 47 to 110.
constexpr int PT_W = 32, PT_PW = PT_W + 2;
template <typename T, int WM, int WN, int NJ, int DEPTH, bool PARTS>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(2, 8))) void
k_conv3x3_patch(ConvIn<T> in, int n, int h, int w, int cin, int cp, const uint16_t *__restrict__ wt, int packed, int cout,
                int chunks, ConvOut out) {
    extern __shared__ __align__(16) uint16_t Ps[];
    constexpr int NTH = 64 * WM * WN, POS = (2 * WM + 2) * PT_PW, U = 8;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kq = lane >> 4, wm = wave % WM, wn = wave / WM;
    const int tx = (w + PT_W - 1) / PT_W, ty = (h + 2 * WM - 1) / (2 * WM);
    const int t = blockIdx.x, img = t / (tx * ty), r = t - img * tx * ty;
    const int y0 = (r / tx) * (2 * WM), x0 = (r % tx) * PT_W;
    const int n0 = (blockIdx.y * WN + wn) * (16 * NJ);
    const int K = 9 * cin, ca = in.ca, cb = cin - in.ca, ld = (PARTS ? cp : cin) + 8;
    auto stage_part = [&](int p0, int p1) { // channels [p0, p1) of the patch
        const int yt = y0 > 0 ? y0 - 1 : 0, sh = in.half0;
        const int64_t base = (int64_t)img * h * w + (int64_t)yt * w;
        const int64_t base0 = sh ? ((int64_t)img * (h >> 1) + (yt >> 1)) * (w >> 1) : base;
        const __amdgpu_buffer_rsrc_t v0 = view(in.x0 + base0 * ca, ((sh ? (int64_t)n * (h >> 1) * (w >> 1) : (int64_t)n * h * w) - base0) * ca * (int)sizeof(T));
        const __amdgpu_buffer_rsrc_t v1 = view(in.x1 + base * cb, ((int64_t)n * h * w - base) * cb * (int)sizeof(T));
        // channels [lo, hi) of a source of cs, from channel `at0` of the part on
        auto stage = [&](const __amdgpu_buffer_rsrc_t &v, int cs, int lo, int hi, int at0, int sh) {
            const int pieces = (hi - lo) / 8;
            const float inv = 1.f / (float)pieces; // ((e + 1/2) inv is further from an integer than its rounding)
            for (int e0 = tid; e0 < POS * pieces; e0 += U * NTH) {
                uint4 q[U];
                int at[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int e = e0 + u * NTH, pos = (int)(((float)e + 0.5f) * inv), c = 8 * (e - pos * pieces);
                    const int yy = y0 - 1 + pos / PT_PW, xx = x0 - 1 + pos % PT_PW;
                    const bool ok = e < POS * pieces && yy >= 0 && yy < h && xx >= 0 && xx < w;
                    const unsigned p = (unsigned)(((yy >> sh) - (yt >> sh)) * (w >> sh) + (xx >> sh));
                    at[u] = e < POS * pieces ? pos * ld + at0 + c : POS * ld; // (past the end: a spare piece)
                    q[u] = load_raw<T>(v, ok ? (p * cs + lo + c) * (unsigned)sizeof(T) : NO_PIECE);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) *reinterpret_cast<uint4 *>(&Ps[at[u]]) = q[u];
            }
        };
        if (p0 < ca) stage(v0, ca, p0, min(p1, ca), 0, sh);
        if (p1 > ca) stage(v1, cb, max(p0 - ca, 0), p1 - ca, max(ca - p0, 0), 0);
    };
    const __amdgpu_buffer_rsrc_t rw = view(wt + (int64_t)n0 * K, (int64_t)16 * NJ * K * 2);
    unsigned wv0[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) wv0[j] = packed ? (unsigned)(16 * j * K + 8 * lane) * 2u : (unsigned)((16 * j + row) * K + 8 * kq) * 2u;
    // The next step to load: inner and outer position (tap and chunk of the part, or chunk and tap), k in bytes.
    int s = 0, so = 0, k2 = 0, inner = 0, outer = 0, dk = 0, back = 0;
    u32x4 wv[DEPTH][NJ];
    int off[DEPTH]; // LDS element offset of the step
#define IVX_STEP_LOAD(d)                                                                                               \
    do {                                                                                                               \
        const bool live = so < outer; /* (steps past the last: the first one's operands, not used) */                  \
        const int tap = live ? (chunks ? s : so) : 0, ch = live ? (chunks ? so : s) : 0, ky = (tap * 11) >> 5;         \
        const int kk = __builtin_amdgcn_readfirstlane(live ? k2 << (packed ? 4 : 0) : 0);                              \
        _Pragma("unroll") for (int j = 0; j < NJ; ++j) wv[d][j] = __builtin_amdgcn_raw_buffer_load_b128(rw, wv0[j], kk, 0); \
        off[d] = __builtin_amdgcn_readfirstlane((ky * PT_PW + tap - 3 * ky) * ld + 32 * ch);                           \
        const bool wrap = ++s == inner;                                                                                \
        s = wrap ? 0 : s;                                                                                              \
        so += wrap;                                                                                                    \
        k2 += wrap ? back : dk;                                                                                        \
    } while (0)
    f32x4 acc[NJ][4];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint16_t *a0 = Ps + (2 * wm * PT_PW + row) * ld + 8 * kq;
    auto pixels = [&](int i, int at) {
        return as_bf16x8(*reinterpret_cast<const uint4 *>(a0 + at + ((i >> 1) * PT_PW + 16 * (i & 1)) * ld));
    };
    int p0 = 0;
    do { // (once unless PARTS)
        const int nc = (PARTS ? min(cp, cin - p0) : cin) / 32, steps = 9 * nc;
        inner = chunks ? 9 : nc;
        outer = chunks ? nc : 9;
        dk = chunks ? 2 * cin : 64;
        back = chunks ? 64 - 16 * cin : 2 * cin - 64 * (nc - 1);
        s = so = 0;
        k2 = 2 * p0;
        if (PARTS && p0 > 0) __syncthreads(); // the last part's operands are read
        stage_part(p0, p0 + 32 * nc);
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            IVX_STEP_LOAD(d);
            __builtin_amdgcn_sched_barrier(0); // (in this order: the loop's waits count them)
        }
        __syncthreads();
        bf16x8 a[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = pixels(i, 0);
        for (int s0 = 0; s0 < steps; s0 += DEPTH) { // (9 nc steps: a multiple of DEPTH)
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                const int next = off[(d + 1) % DEPTH]; // (the slot of step s0 + DEPTH holds it by now)
                bf16x8 an[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) an[i] = pixels(i, next);
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[j][i] = mma(__builtin_bit_cast(bf16x8, wv[d][j]), a[i], acc[j][i]);
                __builtin_amdgcn_sched_barrier(0); // (the loads of a step stay DEPTH steps ahead of their use)
                IVX_STEP_LOAD(d);
#pragma unroll
                for (int i = 0; i < 4; ++i) a[i] = an[i];
            }
        }
        p0 += cp;
    } while (PARTS && p0 < cin);
#undef IVX_STEP_LOAD
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int py = y0 + 2 * wm + (i >> 1), px = x0 + 16 * (i & 1) + row;
        if (py >= h || px >= w) continue;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            store_out(out, acc[j][i], ((int64_t)img * h + py) * w + px, img, py, px, h, w, cout, n0 + 16 * j + 4 * kq);
    }
}

// Weight-gradient partials: block (k tile of 64, o tile of 64, pixel range z).
constexpr int GW_PIX = 1024;
__global__ __launch_bounds__(NT) void k_conv3x3_gw(const float *__restrict__ x, const float *__restrict__ dy,
                                                   int n, int h, int w, int cin, int cout,
                                                   float *__restrict__ part) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t P = (int64_t)n * h * w;
    const int K = 9 * cin;
    const int row = lane & 15, q = lane >> 4;
    const int co = blockIdx.y * 64 + wave * 16 + row;   // A row
    const int kbase = blockIdx.x * 64;                   // 4 column tiles
    const int64_t p0 = (int64_t)blockIdx.z * GW_PIX;
    const int64_t p1 = p0 + GW_PIX < P ? p0 + GW_PIX : P;
    int tapy[4], tapx[4], tc[4];
    bool kv[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int k = kbase + t * 16 + row;
        kv[t] = k < K;
        const int tap = kv[t] ? k / cin : 0;
        tc[t] = kv[t] ? k - tap * cin : 0;
        tapy[t] = tap / 3 - 1;
        tapx[t] = tap % 3 - 1;
    }
    f32x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int64_t pb = p0; pb < p1; pb += 32) {
        uint16_t a[8], b[4][8];
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            a[v] = 0;
#pragma unroll
            for (int t = 0; t < 4; ++t) b[t][v] = 0;
            const int64_t p = pb + 8 * q + v;
            if (p >= p1) continue;
            if (co < cout) a[v] = f2bf(dy[p * cout + co]);
            const int pn = (int)(p / ((int64_t)h * w));
            const int r = (int)(p - (int64_t)pn * h * w);
            const int py = r / w, px = r - (r / w) * w;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int yy = py + tapy[t], xx = px + tapx[t];
                if (kv[t] && yy >= 0 && yy < h && xx >= 0 && xx < w)
                    b[t][v] = f2bf(x[(((int64_t)pn * h + yy) * w + xx) * cin + tc[t]]);
            }
        }
        const bf16x8 av = as_bf16x8(pack8(a));
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = mma(av, as_bf16x8(pack8(b[t])), acc[t]);
    }
    // D rows = output channels (4 q + v of this wave's 16), columns = k
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int k = kbase + t * 16 + row;
        if (k >= K) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int o = blockIdx.y * 64 + wave * 16 + 4 * q + v;
            if (o < cout) part[((int64_t)blockIdx.z * cout + o) * K + k] = acc[t][v];
        }
    }
}

// Weight and bias gradient partials, LDS-tiled: block (k tile of 64, o tile of 64, pixel
// range z of `ps` pixels).  The pixel range is walked in chunks of 32: dy (A, [o][pixel]) and
// the im2col view of x (B, [k][pixel]) are staged in LDS as bf16, transposed so that each
// lane's eight reduction elements are contiguous; 4 waves in a 2 x 2 arrangement each own
// 32 x 32 outputs (2 x 2 tiles of v_mfma_f32_16x16x32_bf16, one product per chunk).  Blocks of the first k tile also
// sum dy in FP32 for the bias.  part[z] = [dw partial (cout x K) | db partial (cout)].
// Requires cin % 4 == 0 and cout % 4 == 0.
constexpr int GW_PC = 32, GW_LD = 40, GW_TARGET_BLOCKS = 2048, GW_MIN_PIX = 256;
__global__ __launch_bounds__(NT) void k_conv3x3_gw_tiled(const float *__restrict__ x, const float *__restrict__ dy,
                                                         int n, int h, int w, int cin, int cout, int64_t ps,
                                                         float *__restrict__ part) {
    __shared__ __align__(16) uint16_t As[64 * GW_LD];
    __shared__ __align__(16) uint16_t Bs[64 * GW_LD];
    __shared__ float sb[16][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t P = (int64_t)n * h * w;
    const int64_t hw = (int64_t)h * w;
    const int K = 9 * cin;
    const int64_t len = (int64_t)cout * K + cout;
    const int o0 = blockIdx.y * 64, k0 = blockIdx.x * 64;
    const int64_t p0 = (int64_t)blockIdx.z * ps;
    const int64_t p1 = p0 + ps < P ? p0 + ps : P;
    // staging: pixel pair 2 sp (fastest within a wave), 4 rows g4 .. g4 + 3 of A and of B
    const int sp = tid & 15, g4 = (tid >> 4) * 4;
    const bool ov = o0 + g4 < cout;
    const int kk = k0 + g4;
    const bool kv = kk < K;
    const int tap = kv ? kk / cin : 0;
    const int tc = kk - tap * cin, tdy = tap / 3 - 1, tdx = tap % 3 - 1;
    const bool do_bias = blockIdx.x == 0;
    float4 ra[2], rb[2];
    float bs[4] = {0.f, 0.f, 0.f, 0.f};
    auto gload = [&](int64_t pc) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int64_t p = pc + 2 * sp + e;
            ra[e] = float4{0.f, 0.f, 0.f, 0.f};
            rb[e] = float4{0.f, 0.f, 0.f, 0.f};
            if (p < p1) {
                if (ov) ra[e] = *reinterpret_cast<const float4 *>(dy + p * cout + o0 + g4);
                const int pn = (int)(p / hw);
                const int r = (int)(p - pn * hw);
                const int yy = r / w + tdy, xx = r % w + tdx;
                if (kv && yy >= 0 && yy < h && xx >= 0 && xx < w)
                    rb[e] = *reinterpret_cast<const float4 *>(x + (((int64_t)pn * h + yy) * w + xx) * cin + tc);
            }
        }
    };
    auto sstore = [&]() {
        const float *a0 = reinterpret_cast<const float *>(&ra[0]), *a1 = reinterpret_cast<const float *>(&ra[1]);
        const float *b0 = reinterpret_cast<const float *>(&rb[0]), *b1 = reinterpret_cast<const float *>(&rb[1]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            *reinterpret_cast<uint32_t *>(&As[(g4 + i) * GW_LD + 2 * sp]) = f2bf(a0[i]) | ((uint32_t)f2bf(a1[i]) << 16);
            *reinterpret_cast<uint32_t *>(&Bs[(g4 + i) * GW_LD + 2 * sp]) = f2bf(b0[i]) | ((uint32_t)f2bf(b1[i]) << 16);
            bs[i] += a0[i] + a1[i];
        }
    };
    const int wr = wave >> 1, wc = wave & 1;
    const int row = lane & 15, kq = lane >> 4;
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    gload(p0);
    for (int64_t pc = p0; pc < p1; pc += GW_PC) {
        __syncthreads();
        sstore();
        __syncthreads();
        if (pc + GW_PC < p1) gload(pc + GW_PC);
        static_assert(GW_PC == 32, "one 16x16x32 product per chunk");
        bf16x8 af[2], bfr[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            af[i] = as_bf16x8(*reinterpret_cast<const uint4 *>(&As[(wr * 32 + i * 16 + row) * GW_LD + 8 * kq]));
            bfr[i] = as_bf16x8(*reinterpret_cast<const uint4 *>(&Bs[(wc * 32 + i * 16 + row) * GW_LD + 8 * kq]));
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = mma(af[i], bfr[j], acc[i][j]);
    }
    float *pz = part + (int64_t)blockIdx.z * len;
    // D row (o) 4 kq + v, column (k) = the lane's row index
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int k = k0 + wc * 32 + j * 16 + row;
            if (k >= K) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int o = o0 + wr * 32 + i * 16 + 4 * kq + v;
                if (o < cout) pz[(int64_t)o * K + k] = acc[i][j][v];
            }
        }
    if (do_bias) {
#pragma unroll
        for (int i = 0; i < 4; ++i) sb[sp][g4 + i] = bs[i];
        __syncthreads();
        if (tid < 64 && o0 + tid < cout) {
            float s = 0.f;
            for (int q = 0; q < 16; ++q) s += sb[q][tid];
            pz[(int64_t)cout * K + o0 + tid] = s;
        }
    }
}

// Weight and bias gradient partials over 4 x 16 pixel patches: block (c tile of CT channels, o tile of
// 32, patch range z).  Per patch the block stages dy (64 pixels x 32 o) and x with its one-pixel halo
// (6 x 18 positions x CT c) in LDS as bf16, once for all nine taps; the operands of a product, whose
// reduction runs over pixels, are columns of those rows and come through the transposing LDS load
// (two loads of four consecutive pixels: 32 pixels = two patch rows per product).  A wave owns 16 c x
// 32 o x 9 taps, 18 products for 22 operand halves.  CT = 64: four c tiles.  CT = 32: two, and waves
// 2, 3 take the patch's lower two rows (summed over LDS at the end).  Rows are padded by 16 elements, so
// that the four pixels a 16-lane group reads lie in different banks.
// Before, each of the nine taps restaged its own shifted view through registers with FP32 rounding:
// 268 -> 85 us on 32 channels at 256^2 x 16.  part[z] = [dw (cout x K) | db (cout)].
// Requires cin % 8 == 0 and cout % 8 == 0.
constexpr int GP_TH = 4, GP_TW = 16, GP_PW = GP_TW + 2, GP_POS = (GP_TH + 2) * GP_PW, GP_OL = 48;
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ s16x4 read_columns(const uint16_t *at) {
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)at);
}

// FAR: images whose rows are too long for 32-bit offsets into a patch's rows (plain loads at 64-bit addresses).
template <typename T, int CT, bool FAR = false>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_conv3x3_gw_patch(ConvIn<T> in, const T *__restrict__ dyb,
                                                         const float *__restrict__ dy, int n, int h, int w, int cin,
                                                         int cout, int tiles, int tps, float *__restrict__ part) {
    constexpr int XL = CT + 16, XPIECES = GP_POS * (CT / 8), XPER = (XPIECES + NT - 1) / NT;
    __shared__ __align__(16) uint16_t Xs[GP_POS * XL];
    __shared__ __align__(16) uint16_t Ds[GP_TH * GP_TW * GP_OL];
    __shared__ float red[CT == 32 ? 2 * 64 * 4 : 1];
    __shared__ float sb[8][32];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, g = lane >> 4;
    const int K = 9 * cin, ca = in.ca, cb = cin - in.ca;
    const int64_t len = (int64_t)cout * K + cout;
    const int c0 = blockIdx.x * CT, o0 = blockIdx.y * 32;
    const int t0 = blockIdx.z * tps, t1 = min(tiles, t0 + tps);
    const int tx = (w + GP_TW - 1) / GP_TW, ty = (h + GP_TH - 1) / GP_TH;
    uint4 rx[XPER], rd;
    float bs[8] = {};
    const bool do_bias = blockIdx.x == 0;
    // one 8-channel piece of dy per thread: pixel tid / 4, channels 8 (tid % 4)
    const int dp = tid >> 2, dc = o0 + 8 * (tid & 3);
    auto gload = [&](int t) {
        const int img = t / (tx * ty), r = t - img * tx * ty, y0 = (r / tx) * GP_TH, x0 = (r % tx) * GP_TW;
        // views of this image: offsets stay small whatever the batch
        const int64_t base = (int64_t)img * h * w, base0 = in.half0 ? (int64_t)img * (h >> 1) * (w >> 1) : base;
        if constexpr (FAR) {
            const int yy = y0 + (dp >> 4), xx = x0 + (dp & 15);
            const bool okp = yy < h && xx < w && dc < cout;
            const int64_t at = (base + (int64_t)yy * w + xx) * cout + dc;
            rd = uint4{0u, 0u, 0u, 0u};
            if (okp) rd = *reinterpret_cast<const uint4 *>(dyb + at);
            if (do_bias && okp)
#pragma unroll
                for (int e = 0; e < 8; ++e) bs[e] += dy[at + e];
#pragma unroll
            for (int u = 0; u < XPER; ++u) {
                const int e = tid + u * NT, pos = e / (CT / 8), c = c0 + 8 * (e % (CT / 8));
                const int yx = y0 - 1 + pos / GP_PW, xp = x0 - 1 + pos % GP_PW, sh = c < ca ? in.half0 : 0;
                const int64_t pix = (c < ca ? base0 : base) + (int64_t)(yx >> sh) * (w >> sh) + (xp >> sh);
                rx[u] = uint4{0u, 0u, 0u, 0u};
                if (e < XPIECES && c < cin && yx >= 0 && yx < h && xp >= 0 && xp < w)
                    rx[u] = *reinterpret_cast<const uint4 *>(c < ca ? in.x0 + pix * ca + c : in.x1 + pix * cb + (c - ca));
            }
            return;
        }
        {
            const int yy = y0 + (dp >> 4), xx = x0 + (dp & 15);
            const bool okp = yy < h && xx < w && dc < cout;
            const unsigned at = (unsigned)((yy - y0) * w + xx) * cout + dc;
            const int64_t at0 = (base + (int64_t)y0 * w) * cout, left = ((int64_t)n * h * w * cout - at0);
            rd = load_raw<T>(view(dyb + at0, left * (int)sizeof(T)), okp ? at * (unsigned)sizeof(T) : NO_PIECE);
            if (do_bias) {
                const __amdgpu_buffer_rsrc_t rf = view(dy + at0, left * 4);
                const f32x4 a = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rf, okp ? 4u * at : NO_PIECE, 0, 0));
                const f32x4 b = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rf, okp ? 4u * at + 16u : NO_PIECE, 0, 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    bs[e] += a[e];
                    bs[4 + e] += b[e];
                }
            }
        }
        const int yt = y0 > 0 ? y0 - 1 : 0, sh0 = in.half0;
        const int64_t s0 = base0 + (int64_t)(yt >> sh0) * (w >> sh0), s1 = base + (int64_t)yt * w;
        const __amdgpu_buffer_rsrc_t v0 = view(in.x0 + s0 * ca, ((sh0 ? (int64_t)n * (h >> 1) * (w >> 1) : (int64_t)n * h * w) - s0) * ca * (int)sizeof(T));
        const __amdgpu_buffer_rsrc_t v1 = view(in.x1 + s1 * cb, ((int64_t)n * h * w - s1) * cb * (int)sizeof(T));
#pragma unroll
        for (int u = 0; u < XPER; ++u) {
            const int e = tid + u * NT, pos = e / (CT / 8), c = c0 + 8 * (e % (CT / 8));
            const int yy = y0 - 1 + pos / GP_PW, xx = x0 - 1 + pos % GP_PW;
            const bool okx = e < XPIECES && c < cin && yy >= 0 && yy < h && xx >= 0 && xx < w;
            const unsigned p0 = (unsigned)(((yy >> sh0) - (yt >> sh0)) * (w >> sh0) + (xx >> sh0)), p1 = (unsigned)((yy - yt) * w + xx);
            if (c0 < ca) rx[u] = load_raw<T>(v0, okx && c < ca ? (p0 * ca + c) * (unsigned)sizeof(T) : NO_PIECE);
            else rx[u] = load_raw<T>(v1, okx ? (p1 * cb + (c - ca)) * (unsigned)sizeof(T) : NO_PIECE);
            if (c0 < ca && c0 + CT > ca && cb) { // (a tile that spans both sources)
                const uint4 q = load_raw<T>(v1, okx && c >= ca ? (p1 * cb + (c - ca)) * (unsigned)sizeof(T) : NO_PIECE);
                rx[u] = uint4{rx[u].x | q.x, rx[u].y | q.y, rx[u].z | q.z, rx[u].w | q.w};
            }
        }
    };
    auto sstore = [&]() {
        *reinterpret_cast<uint4 *>(&Ds[dp * GP_OL + 8 * (tid & 3)]) = rd;
#pragma unroll
        for (int u = 0; u < XPER; ++u) {
            const int e = tid + u * NT;
            if (e < XPIECES) *reinterpret_cast<uint4 *>(&Xs[(e / (CT / 8)) * XL + 8 * (e % (CT / 8))]) = rx[u];
        }
    };
    const int cw = CT == 64 ? wave : wave & 1;             // this wave's 16 channels
    const int r0 = CT == 64 ? 0 : 2 * (wave >> 1), r1 = CT == 64 ? GP_TH : r0 + 2; // and patch rows
    const bool live = c0 + 16 * cw < cin;
    f32x4 acc[2][9];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    union Op {
        s16x4 p[2];
        bf16x8 v;
    };
    // this lane's chunk: pixel 4 g + c16 / 4 of a row, channels 4 (c16 % 4)
    const int lp = 4 * g + (c16 >> 2), lc = 4 * (c16 & 3);
    if (t0 < t1) gload(t0);
    for (int t = t0; t < t1; ++t) {
        __syncthreads();
        sstore();
        __syncthreads();
        if (t + 1 < t1) gload(t + 1);
        if (live) {
            for (int r = r0; r < r1; r += 2) {
                Op a[2];
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int u = 0; u < 2; ++u) a[i].p[u] = read_columns(&Ds[((r + u) * GP_TW + lp) * GP_OL + 16 * i + lc]);
#pragma unroll
                for (int tap = 0; tap < 9; ++tap) {
                    Op b;
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        b.p[u] = read_columns(&Xs[((r + u + tap / 3) * GP_PW + lp + tap % 3) * XL + 16 * cw + lc]);
#pragma unroll
                    for (int i = 0; i < 2; ++i) acc[i][tap] = mma(a[i].v, b.v, acc[i][tap]);
                }
            }
        }
    }
    float *pz = part + (int64_t)blockIdx.z * len;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            if (CT == 32) { // the two halves of the patch
                __syncthreads();
                if (wave >= 2) *reinterpret_cast<f32x4 *>(&red[((wave & 1) * 64 + lane) * 4]) = acc[i][tap];
                __syncthreads();
                if (wave < 2) acc[i][tap] += *reinterpret_cast<const f32x4 *>(&red[(wave * 64 + lane) * 4]);
            }
            const int c = c0 + 16 * cw + c16;
            if ((CT == 32 && wave >= 2) || c >= cin) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int o = o0 + 16 * i + 4 * g + v;
                if (o < cout) pz[(int64_t)o * K + tap * cin + c] = acc[i][tap][v];
            }
        }
    if (do_bias) {
        // sum over the 16 lanes of a wave and the four waves that hold the same channels
#pragma unroll
        for (int e = 0; e < 8; ++e) {
#pragma unroll
            for (int q = 4; q < 64; q <<= 1) bs[e] += __shfl_xor(bs[e], q, 64);
        }
        __syncthreads();
        if (lane < 4) {
#pragma unroll
            for (int e = 0; e < 8; ++e) sb[wave][8 * lane + e] = bs[e];
        }
        __syncthreads();
        if (tid < 32 && o0 + tid < cout) pz[(int64_t)cout * K + o0 + tid] = (sb[0][tid] + sb[1][tid]) + (sb[2][tid] + sb[3][tid]);
    }
}

// out[i] = sum over splits of part[z][i] in a fixed order: block = 64 consecutive i x G
// interleaved split groups, combined in LDS.  i < nw goes to dw, the rest to db.  Sixteen groups for many
// splits of few weights (four left the 2,048 splits of the input layer to 19 blocks: 132 us), four for few splits of
// many, whose blocks twelve idle groups slowed down (four splits of 512 -> 512 channels: the gradient 109 -> 151 us).
template <int G>
__global__ __launch_bounds__(64 * G) void k_sum_splits(const float *__restrict__ part, int splits, int64_t len,
                                                       int64_t nw, float *__restrict__ dw, float *__restrict__ db) {
    __shared__ float sh[G][64];
    const int l = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + l;
    float s = 0.f;
    if (i < len) {
        int z = g;
        for (; z + 3 * G < splits; z += 4 * G) {
            float t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] = part[(int64_t)(z + G * u) * len + i];
#pragma unroll
            for (int u = 0; u < 4; ++u) s += t[u];
        }
        for (; z < splits; z += G) s += part[(int64_t)z * len + i];
    }
    sh[g][l] = s;
    __syncthreads();
    if (g == 0 && i < len) {
        float t = 0.f;
#pragma unroll
        for (int q = 0; q < G; q += 4) t += (sh[q][l] + sh[q + 1][l]) + (sh[q + 2][l] + sh[q + 3][l]);
        if (i < nw) dw[i] = t;
        else db[i - nw] = t;
    }
}

// dw[i] = sum over splits of part[s][i] (fixed order)
__global__ __launch_bounds__(NT) void k_sum_parts(const float *__restrict__ part, int splits, int64_t len,
                                                  float *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (i >= len) return;
    float s = 0.f;
    for (int z = 0; z < splits; ++z) s += part[(int64_t)z * len + i];
    out[i] = s;
}

// db[o] = sum over pixels of dy[p][o]; one block per channel, fixed-order tree
__global__ __launch_bounds__(NT) void k_colsum(const float *__restrict__ dy, int64_t P, int c, float *__restrict__ out) {
    __shared__ float sh[NT];
    const int o = blockIdx.x;
    float s = 0.f;
    for (int64_t p = threadIdx.x; p < P; p += NT) s += dy[p * c + o];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int m = NT / 2; m >= 1; m >>= 1) {
        if (threadIdx.x < m) sh[threadIdx.x] += sh[threadIdx.x + m];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[o] = sh[0];
}

// wt[c][a][b][o] = W[o][2-a][2-b][c]
__global__ __launch_bounds__(NT) void k_flip(const uint16_t *__restrict__ W, int cin, int cout, uint16_t *__restrict__ wt) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    const int64_t tot = (int64_t)9 * cin * cout;
    if (i >= tot) return;
    const int o = (int)(i % cout);
    const int ab = (int)((i / cout) % 9);
    const int c = (int)(i / ((int64_t)cout * 9));
    const int a = ab / 3, b = ab % 3;
    wt[i] = W[((int64_t)o * 9 + (2 - a) * 3 + (2 - b)) * cin + c];
}

// Place of weight (o, k) of a layer of K = 9 cin.  For cin a multiple of 32 and cout of 16 the network keeps its weights
// by steps: the 16 channels x 32 k that one product takes are 1 KB in lane order, so that a wave's load
// is one piece of memory.  From rows of K a load touches 16 rows of 64 bytes, and that
// bound the convolutions: 64 -> 44 us at 16 x 128^2 x 64 -> 64 channels, 52 -> 31 us at 16 x 64^2 x 128 -> 128.
// (A weight tensor that a caller passes stays in rows.)
__host__ __device__ inline int weights_packed(int cin, int cout) { return cin % 32 == 0 && cout % 16 == 0; }
__device__ __forceinline__ int64_t weight_at(int o, int k, int cin, int cout) {
    const int K = 9 * cin;
    if (!weights_packed(cin, cout)) return (int64_t)o * K + k;
    return ((int64_t)(o >> 4) * (K >> 5) + (k >> 5)) * 512 + (((k & 31) >> 3) * 16 + (o & 15)) * 8 + (k & 7);
}

// Both bf16 weight sets of a network layer from its master weights [cout][9][cin]: the layer's own and
// the flipped [cin][9][cout] of its input gradient (there cout is the input count).
__global__ __launch_bounds__(NT) void k_layer_weights(const float *__restrict__ W, int cin, int cout, uint16_t *__restrict__ wbf,
                                                      uint16_t *__restrict__ wflip) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (i >= (int64_t)9 * cin * cout) return;
    const int c = (int)(i % cin), tap = (int)(i / cin % 9), o = (int)(i / (9 * (int64_t)cin));
    const uint16_t b = f2bf(W[i]);
    wbf[weight_at(o, tap * cin + c, cin, cout)] = b;
    wflip[weight_at(c, (8 - tap) * cout + o, cout, cin)] = b;
}

__global__ __launch_bounds__(NT) void k_to_bf16(const float *__restrict__ x, int64_t n, uint16_t *__restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (i < n) y[i] = f2bf(x[i]);
}

// ---------------------------------------------------------------- other layers
__global__ __launch_bounds__(NT) void k_pool2(const float *__restrict__ x, int n, int h, int w, int c,
                                              float *__restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    const int ho = h / 2, wo = w / 2;
    const int64_t tot = (int64_t)n * ho * wo * c;
    if (i >= tot) return;
    const int ch = (int)(i % c);
    const int64_t pix = i / c;
    const int xo = (int)(pix % wo), yo = (int)((pix / wo) % ho), nn = (int)(pix / ((int64_t)wo * ho));
    const float *b = x + (((int64_t)nn * h + 2 * yo) * w + 2 * xo) * c + ch;
    y[i] = fmaxf(fmaxf(b[0], b[c]), fmaxf(b[(int64_t)w * c], b[(int64_t)w * c + c]));
}

// bf16 activations after a ReLU (non-negative: ordered as integers), eight channels per thread; the
// rounded maximum is the maximum of the rounded values
__global__ __launch_bounds__(NT) void k_pool2_bf16(const uint16_t *__restrict__ x, int n, int h, int w, int c,
                                                   uint16_t *__restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    const int ho = h / 2, wo = w / 2, c8 = c / 8;
    if (i >= (int64_t)n * ho * wo * c8) return;
    const int ch = 8 * (int)(i % c8);
    const int64_t pix = i / c8;
    const int xo = (int)(pix % wo), yo = (int)((pix / wo) % ho), nn = (int)(pix / ((int64_t)wo * ho));
    const uint16_t *b = x + (((int64_t)nn * h + 2 * yo) * w + 2 * xo) * c + ch;
    typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
    const u16x8 q0 = *reinterpret_cast<const u16x8 *>(b), q1 = *reinterpret_cast<const u16x8 *>(b + c);
    const u16x8 q2 = *reinterpret_cast<const u16x8 *>(b + (int64_t)w * c), q3 = *reinterpret_cast<const u16x8 *>(b + (int64_t)w * c + c);
    *reinterpret_cast<u16x8 *>(y + pix * c + ch) = __builtin_elementwise_max(__builtin_elementwise_max(q0, q1), __builtin_elementwise_max(q2, q3));
}

// dxb (may be NULL): the result rounded to bf16
__global__ __launch_bounds__(NT) void k_pool2_grad(const float *__restrict__ x, const float *__restrict__ dy, int n,
                                                   int h, int w, int c, int accumulate, float *__restrict__ dx,
                                                   uint16_t *__restrict__ dxb) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    const int ho = h / 2, wo = w / 2;
    const int64_t tot = (int64_t)n * ho * wo * c;
    if (i >= tot) return;
    const int ch = (int)(i % c);
    const int64_t pix = i / c;
    const int xo = (int)(pix % wo), yo = (int)((pix / wo) % ho), nn = (int)(pix / ((int64_t)wo * ho));
    const int64_t o00 = (((int64_t)nn * h + 2 * yo) * w + 2 * xo) * c + ch;
    const int64_t off[4] = {o00, o00 + c, o00 + (int64_t)w * c, o00 + (int64_t)w * c + c};
    float m = x[off[0]];
    for (int q = 1; q < 4; ++q) m = fmaxf(m, x[off[q]]);
    bool taken = false;
    for (int q = 0; q < 4; ++q) {
        float g = 0.f;
        if (!taken && x[off[q]] == m) {
            g = dy[i];
            taken = true;
        }
        const float v = accumulate ? dx[off[q]] + g : g;
        dx[off[q]] = v;
        if (dxb) dxb[off[q]] = f2bf(v);
    }
}

__global__ __launch_bounds__(NT) void k_up2(const float *__restrict__ x, int n, int h, int w, int c,
                                            float *__restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    const int64_t tot = (int64_t)n * (2 * h) * (2 * w) * c;
    if (i >= tot) return;
    const int ch = (int)(i % c);
    const int64_t pix = i / c;
    const int xo = (int)(pix % (2 * w)), yo = (int)((pix / (2 * w)) % (2 * h)), nn = (int)(pix / ((int64_t)4 * w * h));
    y[i] = x[(((int64_t)nn * h + yo / 2) * w + xo / 2) * c + ch];
}

__global__ __launch_bounds__(NT) void k_up2_grad(const float *__restrict__ dy, int n, int h, int w, int c,
                                                 float *__restrict__ dx, uint16_t *__restrict__ dxb) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    const int64_t tot = (int64_t)n * h * w * c;
    if (i >= tot) return;
    const int ch = (int)(i % c);
    const int64_t pix = i / c;
    const int xx = (int)(pix % w), yy = (int)((pix / w) % h), nn = (int)(pix / ((int64_t)w * h));
    const int W2 = 2 * w;
    const int64_t b = (((int64_t)nn * 2 * h + 2 * yy) * W2 + 2 * xx) * c + ch;
    const float v = dy[b] + dy[b + c] + dy[b + (int64_t)W2 * c] + dy[b + (int64_t)W2 * c + c];
    dx[i] = v;
    if (dxb) dxb[i] = f2bf(v);
}

// network input [n][h][w] -> [n][h][w][4] (channel 0)
__global__ __launch_bounds__(NT) void k_pad_input(const float *__restrict__ x, int64_t P, float *__restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (i >= P) return;
    reinterpret_cast<float4 *>(y)[i] = float4{x[i], 0.f, 0.f, 0.f};
}

// 1x1 head: y[p] = b + sum_c w[c] x[p][c]
// Head (1x1 convolution to one channel) on c-channel pixels, c % 4 == 0: G = c / 4 threads per
// pixel hold 4 channels each (float4 loads, contiguous across the threads of a block), NT / G
// pixels per block; the per-pixel and per-channel sums run over LDS in a fixed order.
__global__ __launch_bounds__(NT) void k_head(const float *__restrict__ x, int c, int64_t P, const float *__restrict__ wt,
                                             const float *__restrict__ b, float *__restrict__ y) {
    __shared__ float sh[NT];
    const int G = c >> 2, ppb = NT / G;
    const int t = threadIdx.x, g = t % G, lp = t / G;
    const int64_t p = (int64_t)blockIdx.x * ppb + lp;
    float s = 0.f;
    if (lp < ppb && p < P) {
        const float4 v = *reinterpret_cast<const float4 *>(x + p * c + 4 * g); // c % 4 == 0: aligned
        s = wt[4 * g] * v.x + wt[4 * g + 1] * v.y + wt[4 * g + 2] * v.z + wt[4 * g + 3] * v.w;
    }
    sh[t] = s;
    __syncthreads();
    const int64_t q = (int64_t)blockIdx.x * ppb + t;
    if (t < ppb && q < P) {
        float acc = b[0];
        for (int i = 0; i < G; ++i) acc += sh[t * G + i];
        y[q] = acc;
    }
}

// head backward: dx[p][k] = w[k] dy[p] [x > 0]; per-block partials of dw[k] = sum_p dy x[p][k]
// and db = sum_p dy (blocks walk the pixels grid-stride; part[block][0..c]).
constexpr int HEAD_BLOCKS = 512;
__global__ __launch_bounds__(NT) void k_head_grad(const float *__restrict__ x, int c, int64_t P,
                                                  const float *__restrict__ wt, const float *__restrict__ dy,
                                                  float *__restrict__ dx, uint16_t *__restrict__ dxb,
                                                  float *__restrict__ part) {
    __shared__ float4 sw[NT];
    __shared__ float sb[NT];
    const int G = c >> 2, ppb = NT / G;
    const int t = threadIdx.x, g = t % G, lp = t / G;
    const bool act = lp < ppb;
    const float4 w4 = act ? float4{wt[4 * g], wt[4 * g + 1], wt[4 * g + 2], wt[4 * g + 3]} : float4{0.f, 0.f, 0.f, 0.f};
    float4 a4 = float4{0.f, 0.f, 0.f, 0.f};
    float ab = 0.f;
    if (act) {
        for (int64_t p = (int64_t)blockIdx.x * ppb + lp; p < P; p += (int64_t)gridDim.x * ppb) {
            const float gy = dy[p];
            const float4 v = *reinterpret_cast<const float4 *>(x + p * c + 4 * g);
            const float4 d = float4{v.x > 0.f ? w4.x * gy : 0.f, v.y > 0.f ? w4.y * gy : 0.f, v.z > 0.f ? w4.z * gy : 0.f,
                                    v.w > 0.f ? w4.w * gy : 0.f};
            *reinterpret_cast<float4 *>(dx + p * c + 4 * g) = d;
            *reinterpret_cast<uint2 *>(dxb + p * c + 4 * g) =
                uint2{f2bf(d.x) | ((uint32_t)f2bf(d.y) << 16), f2bf(d.z) | ((uint32_t)f2bf(d.w) << 16)};
            a4.x += gy * v.x;
            a4.y += gy * v.y;
            a4.z += gy * v.z;
            a4.w += gy * v.w;
            ab += gy;
        }
    }
    sw[t] = a4;
    sb[t] = ab;
    __syncthreads();
    float *pz = part + (int64_t)blockIdx.x * (c + 1);
    for (int k = t; k <= c; k += NT) {
        float s = 0.f;
        if (k < c) {
            const int gg = k >> 2, e = k & 3;
            for (int i = 0; i < ppb; ++i) {
                const float4 v = sw[i * G + gg];
                s += e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w;
            }
        } else {
            for (int i = 0; i < ppb; ++i) s += sb[i * G];
        }
        pz[k] = s;
    }
}

// MSE: dy = 2 (y - t) / count; per-block partial sums of (y - t)^2
__global__ __launch_bounds__(NT) void k_mse(const float *__restrict__ y, const float *__restrict__ t, int64_t count,
                                            float *__restrict__ dy, double *__restrict__ part) {
    __shared__ double sh[NT];
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    double v = 0.0;
    if (i < count) {
        const float d = y[i] - t[i];
        dy[i] = 2.f * d / (float)count;
        v = (double)d * (double)d;
    }
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int m = NT / 2; m >= 1; m >>= 1) {
        if (threadIdx.x < m) sh[threadIdx.x] += sh[threadIdx.x + m];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(NT) void k_sum_double(const double *__restrict__ part, int n, double scale,
                                                   double *__restrict__ out) {
    __shared__ double sh[NT];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += NT) s += part[i];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int m = NT / 2; m >= 1; m >>= 1) {
        if (threadIdx.x < m) sh[threadIdx.x] += sh[threadIdx.x + m];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sh[0] * scale;
}

// head gradient partials -> grads (fixed order)
// One wave per output k: lane i sums partials i, i + 64, ... in order, then a fixed xor tree.
__global__ __launch_bounds__(NT) void k_head_reduce(const float *__restrict__ part, int nblk, int c,
                                                    float *__restrict__ dw, float *__restrict__ db) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int k = wave; k <= c; k += NT / 64) {
        float s = 0.f;
        for (int i = lane; i < nblk; i += 64) s += part[(int64_t)i * (c + 1) + k];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
        if (lane == 0) {
            if (k < c) dw[k] = s;
            else db[0] = s;
        }
    }
}

// Adam (Kingma & Ba 2015) with bias correction folded into lr_t and eps_t
__global__ __launch_bounds__(NT) void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                                             float *__restrict__ v, int64_t n, float lr_t, float eps_t) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = 0.9f * m[i] + 0.1f * gi;
    const float vi = 0.999f * v[i] + 0.001f * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr_t * mi / (sqrtf(vi) + eps_t);
}

unsigned nblocks(int64_t n) { return (unsigned)((n + NT - 1) / NT); }

// ------------------------------------------------------------------ launchers
// 32-bit offsets of a view that starts in the first of so many rows
bool rows_fit(int rows, int w, int c, size_t size) { return (int64_t)rows * (w + 64) * c * (int64_t)size < (int64_t)1 << 31; }

constexpr size_t LDS_MAX = 160 * 1024;
size_t patch_lds(int wm, int cp) { return ((size_t)(2 * wm + 2) * PT_PW * (cp + 8) + 8) * sizeof(uint16_t); }

// Channels of a patch that are staged together: all while they fit (in a launch of more than two blocks a CU, blocks
// of two waves: 64 KB, so that two of them still share a CU), else equal parts of at most 80 KB (two waves: 53).
// 768 -> 256 channels at 4 x 64^2 from FP32 activations: 123 us, 131 in parts of 53 KB, 472 from global memory;
// 640 -> 96 at 4 x 64^2: 53 (80 in parts of 80 KB); 288 -> 96 at 4 x 128^2: 79, 119 with the small tile;
// at 1 x 128^2 (768 blocks) 26, 38 unparted, and at 1 x 32^2 18 : 16.
int patch_channels(int waves, int wm, int cin, int64_t blocks) {
    if (patch_lds(wm, cin) <= (waves > 2 || blocks <= 512 ? LDS_MAX : 64 * 1024)) return cin;
    const int chunks = cin / 32;
    int parts = 2;
    while (patch_lds(wm, (chunks + parts - 1) / parts * 32) > (waves > 2 ? 80 * 1024 : 53 * 1024)) ++parts;
    return (chunks + parts - 1) / parts * 32;
}

template <typename T, int WM, int WN, int NJ, int DEPTH>
hipError_t conv3x3_patch(const ConvIn<T> &in, int n, int h, int w, int cin, const uint16_t *wt, int packed, int cout, int chunks,
                         const ConvOut &out, hipStream_t st) {
    const int64_t tiles = (int64_t)n * ((h + 2 * WM - 1) / (2 * WM)) * ((w + PT_W - 1) / PT_W);
    const int cp = patch_channels(WM * WN, WM, cin, tiles * (cout / (16 * NJ * WN)));
    const size_t lds = patch_lds(WM, cp);
    const auto kernel = cp < cin ? k_conv3x3_patch<T, WM, WN, NJ, DEPTH, true> : k_conv3x3_patch<T, WM, WN, NJ, DEPTH, false>;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_MAX);
        if (e != hipSuccess) return e;
    }
    kernel<<<dim3((unsigned)tiles, cout / (16 * NJ * WN)), 64 * WM * WN, lds, st>>>(in, n, h, w, cin, cp, wt, packed, cout, chunks, out);
    return hipGetLastError();
}

template <typename T, int MI, int NJ, int DEPTH>
void conv3x3_wave(const ConvIn<T> &in, int n, int h, int w, int cin, const uint16_t *wt, int packed, int cout, int chunks,
                  const ConvOut &out, hipStream_t st) {
    const int64_t P = (int64_t)n * h * w;
    const dim3 grid((unsigned)((P + 64 * MI - 1) / (64 * MI)), (unsigned)((cout + 16 * NJ - 1) / (16 * NJ)));
    if (cin % 32 == 0) k_conv3x3_wave<T, MI, NJ, DEPTH, false><<<grid, NT, 0, st>>>(in, n, h, w, cin, wt, packed, cout, chunks, out);
    else k_conv3x3_wave<T, MI, NJ, DEPTH, true><<<grid, NT, 0, st>>>(in, n, h, w, cin, wt, packed, cout, chunks, out);
}

// cin % 8 == 0, cout % 16 == 0.  The output tile of a wave: the largest whose launch still has two
// waves per SIMD (one for 32 x 32, 56 -> 64 at 128^2 17.6 : 13.4 us, and for 64 x 16 where no step spans taps, 64 -> 16
// at 256^2 33 : 24, but 40 -> 16 17 : 19; each halving of the tile doubles the operand loads per product), at smaller problems
// single 16 x 16 tiles with eight steps in flight.
template <typename T>
hipError_t conv3x3(const ConvIn<T> &in, int n, int h, int w, int cin, const uint16_t *wt, int packed, int cout,
                   const ConvOut &out, hipStream_t st) {
    // order of the 32-wide steps (fixes the bits of the sums): channel chunks outside the taps where
    // 32 but not 64 output channels divide, else taps outside
    const int chunks = cin % 32 == 0 && cout % 32 == 0 && cout % 64 != 0;
    const int64_t P = (int64_t)n * h * w;
    auto waves = [&](int mi, int nj) { return ((P + 16 * mi - 1) / (16 * mi)) * ((cout + 16 * nj - 1) / (16 * nj)); };
    if (cin % 32 == 0 && cout % 32 == 0) {
        // 64 pixels x 64 (32) channels a wave while that gives the chip's 1,024 SIMDs a wave each (limits of 512 and
        // 2,048 measure the same within 1%), else 16 channels a wave and nine steps in flight (of four waves'
        // blocks: one 32^2 image of 256 channels in 14 us, 29 with the large tile's three steps)
        const bool big = waves(4, cout % 64 == 0 ? 4 : 2) >= 1024;
#define IVX_PATCH(WM, WN, NJ, DEPTH)                                                                                    \
    if (rows_fit(2 * WM + 2, w, cin, sizeof(T)))                                                                        \
    return conv3x3_patch<T, WM, WN, NJ, DEPTH>(in, n, h, w, cin, wt, packed, cout, chunks, out, st)
        if (big && cout % 128 == 0) IVX_PATCH(2, 2, 4, 3);
        if (big && cout % 64 == 0) IVX_PATCH(4, 1, 4, 3);
        if (big && cout % 64 != 0) IVX_PATCH(4, 1, 2, 3);
        if (cout % 64 == 0) IVX_PATCH(1, 4, 1, 9);
        IVX_PATCH(1, 2, 1, 9);
#undef IVX_PATCH
    }
    if constexpr (sizeof(T) == 2)
        if (!rows_fit(4, w, cin, sizeof(T))) {
            k_conv3x3_far<<<dim3((unsigned)((P + 63) / 64), cout / 16), NT, 0, st>>>(in, n, h, w, cin, wt, packed, cout, out);
            return hipGetLastError();
        }
    constexpr int64_t FULL = 2048;
    if (cout % 64 == 0 && waves(4, 4) >= FULL) conv3x3_wave<T, 4, 4, 2>(in, n, h, w, cin, wt, packed, cout, chunks, out, st);
    else if (cout % 32 == 0 && waves(4, 2) >= FULL) conv3x3_wave<T, 4, 2, 2>(in, n, h, w, cin, wt, packed, cout, chunks, out, st);
    else if (cout % 32 == 0 && waves(2, 2) >= FULL / 2) conv3x3_wave<T, 2, 2, 4>(in, n, h, w, cin, wt, packed, cout, chunks, out, st);
    else if (waves(4, 1) >= (cin % 32 == 0 ? FULL / 2 : FULL)) conv3x3_wave<T, 4, 1, 2>(in, n, h, w, cin, wt, packed, cout, chunks, out, st);
    else conv3x3_wave<T, 1, 1, 8>(in, n, h, w, cin, wt, packed, cout, chunks, out, st);
    return hipGetLastError();
}

// FP32 input, any channel count that 4 divides
hipError_t conv3x3_rows(const float *x, int n, int h, int w, int cin, const uint16_t *wt, const float *bias, int cout,
                          int relu, const float *mask, int accumulate, float *y, uint16_t *yb, hipStream_t st) {
    const unsigned gx = (unsigned)(((int64_t)n * h * w + 63) / 64);
    if (cin >= 16 && cout % 32 == 0 && !yb) {
        if (cout % 64 == 0) k_conv3x3_tiled<2><<<dim3(gx, cout / 64), NT, 0, st>>>(x, n, h, w, cin, wt, bias, cout, relu, mask, accumulate, y);
        else k_conv3x3_tiled<1><<<dim3(gx, cout / 32), NT, 0, st>>>(x, n, h, w, cin, wt, bias, cout, relu, mask, accumulate, y);
    } else if (cout % 64 == 0) k_conv3x3<4><<<dim3(gx, cout / 64), NT, 0, st>>>(x, n, h, w, cin, wt, bias, cout, relu, mask, accumulate, y, yb);
    else if (cout % 32 == 0) k_conv3x3<2><<<dim3(gx, cout / 32), NT, 0, st>>>(x, n, h, w, cin, wt, bias, cout, relu, mask, accumulate, y, yb);
    else k_conv3x3<1><<<dim3(gx, (cout + 15) / 16), NT, 0, st>>>(x, n, h, w, cin, wt, bias, cout, relu, mask, accumulate, y, yb);
    return hipGetLastError();
}

// A layer on FP32 activations with weights in rows.  The wave kernel reads every tap of a pixel again, from L2
// while the pixels in flight fit there; the kernels above stage them in LDS or take few channels.  Where cin is no
// multiple of 32 these are the faster ones (us, wave kernel : they) at
//   32 or 64 output channels of at most 24: 16 -> 32 at 3 x 128^2 15.3 : 9.3, at 4 x 256^2 33 : 27, 24 -> 64 49 : 42
//   32 of more: 48 -> 32 at 3 x 128^2 27 : 18, at 4 x 256^2 90 : 64 (below 32,768 pixels 10.5 : 13.5; 248 -> 32 at 4 x 128^2 88 : 104)
//   multiples of 64 of more, 40,000 to 131,071 pixels: 208 -> 64 at 1 x 256^2 113 : 90 (2 x 256^2 156 : 183)
//   other counts of more than 16, more than 160,000 pixels, where the input leaves L2: 48 -> 48 at 4 x 256^2 284 : 205
//   (2 x 256^2 77 : 104), 144 -> 48 813 : 711 (238 : 357), 72 -> 96 492 : 324 (130 : 168)
hipError_t conv3x3_layer(const float *x, int n, int h, int w, int cin, const uint16_t *wt, const float *bias, int cout,
                         int relu, const float *mask, int accumulate, float *y, hipStream_t st) {
    const int64_t P = (int64_t)n * h * w;
    const bool few = cout % 32 == 0 && cin <= 24 && P >= 16384;
    const bool many = cout % 64 == 0 ? P >= 40000 && P < 131072 : (cout == 32 && cin < 128 && P >= 32768) || (cin > 16 && P > 160000);
    if (cin % 8 != 0 || (cin % 32 != 0 && (few || many)) || !rows_fit(4, w, cin, sizeof(float)))
        return conv3x3_rows(x, n, h, w, cin, wt, bias, cout, relu, mask, accumulate, y, nullptr, st);
    ConvOut o{};
    o.y = y;
    o.bias = bias;
    o.relu = relu;
    o.accumulate = accumulate;
    o.maskf = mask;
    return conv3x3<float>(ConvIn<float>{x, nullptr, cin, 0}, n, h, w, cin, wt, 0, cout, o, st);
}

int64_t gw_splits(int n, int h, int w) { return ((int64_t)n * h * w + GW_PIX - 1) / GW_PIX; }

bool gw_tiled(int cin, int cout) { return cin % 4 == 0 && cout % 4 == 0; }

// Split count asked for by the tiled weight gradient: about GW_TARGET_BLOCKS blocks in all
// and at least GW_MIN_PIX pixels per split; non-decreasing in P.
int64_t gw_want_splits(int64_t P, int cin, int cout) {
    const int64_t tiles = (int64_t)((9 * cin + 63) / 64) * ((cout + 63) / 64);
    const int64_t want = std::min((GW_TARGET_BLOCKS + tiles - 1) / tiles, (P + GW_MIN_PIX - 1) / GW_MIN_PIX);
    return std::max<int64_t>(want, 1);
}

// Pixels per split: a whole number of 32-pixel chunks, so at most gw_want_splits splits.
int64_t gw_split_pixels(int64_t P, int cin, int cout) {
    const int64_t want = gw_want_splits(P, cin, cout);
    const int64_t ps = (P + want - 1) / want;
    return (ps + GW_PC - 1) / GW_PC * GW_PC;
}

// Floats of split partials conv3x3_grad_weight needs for this shape; enough for any
// smaller n as well.
int64_t gw_part_len(int n, int h, int w, int cin, int cout) {
    const int64_t P = (int64_t)n * h * w;
    if (!gw_tiled(cin, cout)) return gw_splits(n, h, w) * cout * 9 * cin;
    return gw_want_splits(P, cin, cout) * ((int64_t)cout * 9 * cin + cout);
}

void sum_splits(const float *part, int64_t splits, int cin, int cout, float *dw, float *db, hipStream_t st) {
    const int64_t nw = (int64_t)cout * 9 * cin, len = nw + cout;
    const unsigned blocks = (unsigned)((len + 63) / 64);
    if (splits > 64) k_sum_splits<16><<<blocks, 64 * 16, 0, st>>>(part, (int)splits, len, nw, dw, db);
    else k_sum_splits<4><<<blocks, 64 * 4, 0, st>>>(part, (int)splits, len, nw, dw, db);
}

bool gw_patch(int cin, int cout) { return cin % 8 == 0 && cout % 8 == 0; }
int gw_patch_tile(int cin) { return cin > 32 ? 64 : 32; }
int gw_patch_columns(int cin) { return (cin + gw_patch_tile(cin) - 1) / gw_patch_tile(cin); }

// Weight and bias gradient over 4 x 16 patches (gw_patch(cin, cout)): dyb is dy as T.  About 1,024
// blocks (four per compute unit), within the splits the partial buffer is sized for.
template <typename T>
hipError_t grad_weight_patch(const ConvIn<T> &in, const T *dyb, const float *dy, int n, int h, int w, int cin, int cout,
                             float *part, float *dw, float *db, hipStream_t st) {
    const int tiles = n * ((h + GP_TH - 1) / GP_TH) * ((w + GP_TW - 1) / GP_TW);
    const int gx = gw_patch_columns(cin), gy = (cout + 31) / 32;
    const int64_t most = std::min<int64_t>(gw_want_splits((int64_t)n * h * w, cin, cout), (1024 + gx * gy - 1) / (gx * gy));
    const int tps = (int)((tiles + most - 1) / most), splits = (tiles + tps - 1) / tps;
    const dim3 grid(gx, gy, splits);
    const bool far = sizeof(T) == 2 && !rows_fit(GP_TH + 2, w, std::max(cin, cout), sizeof(float)); // (FP32 layers: the tiled kernel)
    auto kernel = gw_patch_tile(cin) == 64 ? k_conv3x3_gw_patch<T, 64> : k_conv3x3_gw_patch<T, 32>;
    if constexpr (sizeof(T) == 2)
        if (far) kernel = gw_patch_tile(cin) == 64 ? k_conv3x3_gw_patch<T, 64, true> : k_conv3x3_gw_patch<T, 32, true>;
    kernel<<<grid, NT, 0, st>>>(in, dyb, dy, n, h, w, cin, cout, tiles, tps, part);
    sum_splits(part, splits, cin, cout, dw, db, st);
    return hipGetLastError();
}

hipError_t conv3x3_grad_weight(const float *x, const float *dy, int n, int h, int w, int cin, int cout, float *part,
                               float *dw, float *db, hipStream_t st) {
    const int K = 9 * cin;
    const int64_t pixels = (int64_t)n * h * w, padded = (int64_t)n * ((h + GP_TH - 1) / GP_TH * GP_TH) * ((w + GP_TW - 1) / GP_TW * GP_TW);
    // Patches where images fill them at least by half and the launch has blocks enough for its longer per-patch work: the fewer
    // the channel tiles and the emptier the patches, the more pixels.  Kernel times, tiled : patches, us: 512 -> 512 channels on
    // 1 x 32^2 46 : 20, on 8 x 24^2 175 : 76, on 1 x 8^2 8.8 : 9.9, on 2048 x 4 278 : 343; 64 -> 64 on 1 x 32^2 11.3 : 13.5, on
    // 64 x 8^2 12.8 : 22, on 2048 x 8 20 : 26; 16 -> 16 on 16 x 40 x 24 11.8 : 15.5.
    const double ratio = (double)padded / pixels, blocks = (double)gw_patch_columns(cin) * ((cout + 31) / 32);
    const bool fill = ratio <= 2.0 && pixels * blocks >= 16384.0 * ratio * ratio;
    if (gw_patch(cin, cout) && fill && pixels <= INT32_MAX && rows_fit(GP_TH + 2, w, std::max(cin, cout), sizeof(float)))
        return grad_weight_patch<float>(ConvIn<float>{x, nullptr, cin, 0}, dy, dy, n, h, w, cin, cout, part, dw, db, st);
    if (gw_tiled(cin, cout)) {
        const int64_t ps = gw_split_pixels(pixels, cin, cout);
        const int64_t splits = (pixels + ps - 1) / ps;
        k_conv3x3_gw_tiled<<<dim3((K + 63) / 64, (cout + 63) / 64, (unsigned)splits), NT, 0, st>>>(
            x, dy, n, h, w, cin, cout, ps, part);
        sum_splits(part, splits, cin, cout, dw, db, st);
        return hipGetLastError();
    }
    const int64_t splits = gw_splits(n, h, w);
    k_conv3x3_gw<<<dim3((K + 63) / 64, (cout + 63) / 64, (unsigned)splits), NT, 0, st>>>(x, dy, n, h, w, cin, cout, part);
    const int64_t len = (int64_t)cout * K;
    k_sum_parts<<<nblocks(len), NT, 0, st>>>(part, (int)splits, len, dw);
    k_colsum<<<cout, NT, 0, st>>>(dy, (int64_t)n * h * w, cout, db);
    return hipGetLastError();
}

} // namespace

// ------------------------------------------------- allocation-free weight gradient
// Split partials of ivx_nn_conv3x3_grad_weight_noalloc live in this file-scope array: one
// copy on every device the library runs on, held until the process ends.  In host code the
// array's name is not a device address; its address on the current device comes from
// hipGetSymbolAddress, taken once per device and kept.  Every call on a device shares that
// device's copy (the partials are fully written before they are read, so nothing has to
// start at zero); calls that overlap on one device race.
constexpr int64_t NOALLOC_PART_FLOATS = int64_t(8) << 20; // 32 MiB
static __device__ __align__(256) float scratch[NOALLOC_PART_FLOATS];

constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
float *g_scratch_dev[NOALLOC_MAX_DEVICES] = {};

// Device address of `scratch` on the current device (looked up on the first call there).
hipError_t scratch_on_current_device(float **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_dev[dev] = static_cast<float *>(ptr);
    }
    *out = g_scratch_dev[dev];
    return hipSuccess;
}

// ======================================================================= network
struct ConvLayer {
    int cin, cout, h, w;       // input channels, output channels, spatial size
    int64_t w_off, b_off;      // offsets into the master parameter vector
    uint16_t *wbf = nullptr;   // bf16 weights [cout][3][3][cin], in weight_at's order
    uint16_t *wflip = nullptr; // bf16 flipped weights [cin][3][3][cout], in weight_at's order
};

struct ivx_unet {
    int L = 0, base = 0, maxb = 0, H = 0, W = 0;
    std::vector<int> ch;
    std::vector<ConvLayer> conv; // enc0a enc0b enc1a ... dec{L-2}a dec{L-2}b ... dec0a dec0b
    int64_t head_w = 0, head_b = 0, nparam = 0;
    int64_t step = 0;
    std::vector<void *> bufs;
    float *params = nullptr, *grads = nullptr, *mom = nullptr, *vel = nullptr;
    float *xin = nullptr;
    // Activations are bf16, as every convolution consumes them; FP32 only where a consumer is not a
    // convolution: the encoder outputs whose maximum the pooling gradient locates, and the head's input.
    // Gradients are FP32 (bias sums, pooling and upsampling transposes) with a bf16 copy for the products.
    std::vector<uint16_t *> ea, ebb, pool, da, dbb;
    std::vector<float *> eb;
    float *db0 = nullptr;
    std::vector<float *> g_ea, g_eb, g_pool, g_up, g_da, g_db;
    std::vector<uint16_t *> g_eab, g_ebb, g_dab, g_dbb;
    float *out = nullptr, *gout = nullptr;
    float *part = nullptr;
    int64_t part_len = 0;
    float *head_part = nullptr;
    double *loss_part = nullptr, *loss = nullptr;
};

namespace {

// Normal deviates by the polar method (Marsaglia and Bray 1964): the values that
// std::normal_distribution gives here for the same generator, without its extended-precision unit interval: creation
// of a network of 4 levels of base 32 76 -> 23 ms.
struct Normal {
    std::mt19937_64 &rng;
    double sd, spare = 0.0;
    bool have = false;
    Normal(std::mt19937_64 &r, double s) : rng(r), sd(s) {}
    double unit() { return std::min((double)rng() * 5.42101086242752217e-20, 1.0 - 1.11022302462515654e-16); } // 2^-64
    double operator()() {
        if (have) {
            have = false;
            return spare * sd;
        }
        double x, y, r2;
        do {
            x = 2.0 * unit() - 1.0;
            y = 2.0 * unit() - 1.0;
            r2 = x * x + y * y;
        } while (r2 > 1.0 || r2 == 0.0);
        const double m = std::sqrt(-2.0 * std::log(r2) / r2);
        spare = x * m;
        have = true;
        return y * m * sd;
    }
};

template <typename T> ivx_status ualloc(ivx_unet *u, T **p, int64_t count) {
    void *q = nullptr;
    if (hipMalloc(&q, (size_t)(count > 0 ? count : 1) * sizeof(T)) != hipSuccess) {
        (void)hipGetLastError();
        return set_error(IVX_ENOMEM, "hipMalloc failed in ivx_unet_create");
    }
    u->bufs.push_back(q);
    *p = (T *)q;
    return IVX_OK;
}

void ufree(ivx_unet *u) {
    for (void *p : u->bufs) (void)hipFree(p);
    u->bufs.clear();
}

int lvl_h(const ivx_unet *u, int l) { return u->H >> l; }
int lvl_w(const ivx_unet *u, int l) { return u->W >> l; }

// conv layer indices
int enc_a(int l) { return 2 * l; }
int enc_b(int l) { return 2 * l + 1; }
int dec_a(const ivx_unet *u, int l) { return 2 * u->L + 2 * (u->L - 2 - l); }
int dec_b(const ivx_unet *u, int l) { return dec_a(u, l) + 1; }

hipError_t refresh_bf16(ivx_unet *u, hipStream_t st) {
    for (ConvLayer &c : u->conv) {
        const int64_t nw = (int64_t)9 * c.cin * c.cout;
        k_layer_weights<<<nblocks(nw), NT, 0, st>>>(u->params + c.w_off, c.cin, c.cout, c.wbf, c.wflip);
    }
    return hipGetLastError();
}

ConvIn<uint16_t> single(const uint16_t *x, int c) { return ConvIn<uint16_t>{x, nullptr, c, 0}; }

// decoder input of level l: the level below upsampled (read at half resolution), then the skip
ConvIn<uint16_t> dec_in(const ivx_unet *u, int l) {
    return ConvIn<uint16_t>{l + 1 <= u->L - 2 ? u->dbb[l + 1] : u->ebb[u->L - 1], u->ebb[l], u->ch[l + 1], 1};
}

// ReLU convolution of the forward pass: bf16 output yb and / or FP32 output y
hipError_t conv_forward(ivx_unet *u, const ConvLayer &c, int B, const ConvIn<uint16_t> &in, float *y, uint16_t *yb,
                        hipStream_t st) {
    ConvOut o{};
    o.y = y;
    o.yb = yb;
    o.bias = u->params + c.b_off;
    o.relu = 1;
    return conv3x3<uint16_t>(in, B, c.h, c.w, c.cin, c.wbf, weights_packed(c.cin, c.cout), c.cout, o, st);
}

// keep: also store the FP32 encoder outputs that the backward pass reads
hipError_t forward(ivx_unet *u, const float *x, int B, bool keep, hipStream_t st) {
    const int64_t P0 = (int64_t)B * u->H * u->W;
    k_pad_input<<<nblocks(P0), NT, 0, st>>>(x, P0, u->xin);
    hipError_t e;
    for (int l = 0; l < u->L; ++l) {
        const int h = lvl_h(u, l), w = lvl_w(u, l);
        const ConvLayer &a = u->conv[enc_a(l)], &b = u->conv[enc_b(l)];
        if (l == 0) {
            e = conv3x3_rows(u->xin, B, h, w, a.cin, a.wbf, u->params + a.b_off, a.cout, 1, nullptr, 0, nullptr, u->ea[0], st);
        } else {
            k_pool2_bf16<<<nblocks((int64_t)B * h * w * (u->ch[l - 1] / 8)), NT, 0, st>>>(u->ebb[l - 1], B, 2 * h, 2 * w,
                                                                                          u->ch[l - 1], u->pool[l]);
            e = conv_forward(u, a, B, single(u->pool[l], a.cin), nullptr, u->ea[l], st);
        }
        if (e != hipSuccess) return e;
        const bool f32 = u->L == 1 || (keep && l < u->L - 1);
        if ((e = conv_forward(u, b, B, single(u->ea[l], b.cin), f32 ? u->eb[l] : nullptr, u->ebb[l], st)) != hipSuccess) return e;
    }
    for (int l = u->L - 2; l >= 0; --l) {
        const ConvLayer &a = u->conv[dec_a(u, l)], &b = u->conv[dec_b(u, l)];
        if ((e = conv_forward(u, a, B, dec_in(u, l), nullptr, u->da[l], st)) != hipSuccess) return e;
        if ((e = conv_forward(u, b, B, single(u->da[l], b.cin), l == 0 ? u->db0 : nullptr, l == 0 ? nullptr : u->dbb[l], st)) != hipSuccess) return e;
    }
    const float *top = u->L > 1 ? u->db0 : u->eb[0];
    const int hppb = NT / (u->ch[0] / 4);
    k_head<<<(unsigned)((P0 + hppb - 1) / hppb), NT, 0, st>>>(top, u->ch[0], P0, u->params + u->head_w,
                                                            u->params + u->head_b, u->out);
    return hipGetLastError();
}

// conv layer backward: weight/bias gradients into grads, then the input gradient into `o` (masked by
// the input activation > 0)
hipError_t conv_backward(ivx_unet *u, const ConvLayer &c, int B, const ConvIn<uint16_t> &in, const float *gout,
                         const uint16_t *goutb, ConvOut o, hipStream_t st) {
    hipError_t e;
    if ((e = grad_weight_patch<uint16_t>(in, goutb, gout, B, c.h, c.w, c.cin, c.cout, u->part, u->grads + c.w_off,
                                         u->grads + c.b_off, st)) != hipSuccess)
        return e;
    o.maskb = in;
    return conv3x3<uint16_t>(single(goutb, c.cout), B, c.h, c.w, c.cout, c.wflip, weights_packed(c.cout, c.cin), c.cin, o, st);
}

hipError_t backward(ivx_unet *u, int B, hipStream_t st) {
    hipError_t e;
    const int64_t P0 = (int64_t)B * u->H * u->W;
    const bool flat = u->L == 1;
    const int hppb = NT / (u->ch[0] / 4);
    const unsigned hb = (unsigned)std::min<int64_t>(HEAD_BLOCKS, (P0 + hppb - 1) / hppb);
    k_head_grad<<<hb, NT, 0, st>>>(flat ? u->eb[0] : u->db0, u->ch[0], P0, u->params + u->head_w, u->gout,
                                   flat ? u->g_eb[0] : u->g_db[0], flat ? u->g_ebb[0] : u->g_dbb[0], u->head_part);
    k_head_reduce<<<1, NT, 0, st>>>(u->head_part, (int)hb, u->ch[0], u->grads + u->head_w, u->grads + u->head_b);
    // decoder, top level first
    for (int l = 0; l <= u->L - 2; ++l) {
        const int h = lvl_h(u, l), w = lvl_w(u, l);
        const ConvLayer &a = u->conv[dec_a(u, l)], &b = u->conv[dec_b(u, l)];
        ConvOut o{};
        o.y = u->g_da[l];
        o.yb = u->g_dab[l];
        if ((e = conv_backward(u, b, B, single(u->da[l], b.cin), u->g_db[l], u->g_dbb[l], o, st)) != hipSuccess) return e;
        // skip half goes to the encoder output of this level, upsampled half to the level below
        o = ConvOut{};
        o.y = u->g_up[l];
        o.y1 = u->g_eb[l];
        o.split = u->ch[l + 1];
        if ((e = conv_backward(u, a, B, dec_in(u, l), u->g_da[l], u->g_dab[l], o, st)) != hipSuccess) return e;
        const bool mid = l + 1 <= u->L - 2;
        k_up2_grad<<<nblocks((int64_t)B * (h / 2) * (w / 2) * u->ch[l + 1]), NT, 0, st>>>(
            u->g_up[l], B, h / 2, w / 2, u->ch[l + 1], mid ? u->g_db[l + 1] : u->g_eb[u->L - 1],
            mid ? u->g_dbb[l + 1] : u->g_ebb[u->L - 1]);
    }
    // encoder, bottom level first; g_eb[l] for l < L-1 already holds the skip gradient
    for (int l = u->L - 1; l >= 0; --l) {
        const int h = lvl_h(u, l), w = lvl_w(u, l);
        const ConvLayer &a = u->conv[enc_a(l)], &b = u->conv[enc_b(l)];
        ConvOut o{};
        o.y = u->g_ea[l];
        o.yb = l > 0 ? u->g_eab[l] : nullptr;
        if ((e = conv_backward(u, b, B, single(u->ea[l], b.cin), u->g_eb[l], u->g_ebb[l], o, st)) != hipSuccess) return e;
        if (l == 0) {
            if ((e = conv3x3_grad_weight(u->xin, u->g_ea[0], B, h, w, a.cin, a.cout, u->part, u->grads + a.w_off,
                                         u->grads + a.b_off, st)) != hipSuccess)
                return e;
        } else {
            o = ConvOut{};
            o.y = u->g_pool[l];
            if ((e = conv_backward(u, a, B, single(u->pool[l], a.cin), u->g_ea[l], u->g_eab[l], o, st)) != hipSuccess) return e;
            const int64_t tot = (int64_t)B * h * w * u->ch[l - 1];
            k_pool2_grad<<<nblocks(tot), NT, 0, st>>>(u->eb[l - 1], u->g_pool[l], B, 2 * h, 2 * w, u->ch[l - 1], 1,
                                                      u->g_eb[l - 1], u->g_ebb[l - 1]);
        }
    }
    return hipGetLastError();
}

ivx_status check_net(const ivx_unet *u) {
    if (!u) return set_error(IVX_EINVAL, "network is NULL");
    return IVX_OK;
}

#define UHIP(call)                                                                            \
    do {                                                                                      \
        hipError_t e_ = (call);                                                               \
        if (e_ != hipSuccess) return set_error(IVX_EHIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

} // namespace

extern "C" {

ivx_status ivx_unet_create(int32_t levels, int32_t base, int32_t max_batch, int32_t height, int32_t width, uint64_t seed,
                           ivx_unet **out) {
    if (!out) return set_error(IVX_EINVAL, "out is NULL");
    *out = nullptr;
    if (levels < 1 || levels > 5 || base < 16 || base % 16 || max_batch < 1 || height < 1 || width < 1 ||
        height % (1 << (levels - 1)) || width % (1 << (levels - 1)))
        return set_error(IVX_EINVAL, "bad network geometry");
    ivx_unet *u = new ivx_unet();
    u->L = levels;
    u->base = base;
    u->maxb = max_batch;
    u->H = height;
    u->W = width;
    for (int l = 0; l < levels; ++l) u->ch.push_back(base << l);
    int64_t off = 0;
    auto add_conv = [&](int cin, int cout, int l) {
        ConvLayer c;
        c.cin = cin;
        c.cout = cout;
        c.h = height >> l;
        c.w = width >> l;
        c.w_off = off;
        off += (int64_t)9 * cin * cout;
        c.b_off = off;
        off += cout;
        u->conv.push_back(c);
    };
    int prev = 4;
    for (int l = 0; l < levels; ++l) {
        add_conv(prev, u->ch[l], l);
        add_conv(u->ch[l], u->ch[l], l);
        prev = u->ch[l];
    }
    for (int l = levels - 2; l >= 0; --l) {
        add_conv(u->ch[l + 1] + u->ch[l], u->ch[l], l);
        add_conv(u->ch[l], u->ch[l], l);
    }
    u->head_w = off;
    off += u->ch[0];
    u->head_b = off;
    off += 1;
    u->nparam = off;
    ivx_status s;
    const int64_t B = max_batch;
    auto fail = [&](ivx_status st) {
        ufree(u);
        delete u;
        return st;
    };
    if ((s = ualloc(u, &u->params, off)) || (s = ualloc(u, &u->grads, off)) || (s = ualloc(u, &u->mom, off)) ||
        (s = ualloc(u, &u->vel, off)))
        return fail(s);
    for (ConvLayer &c : u->conv) {
        if ((s = ualloc(u, &c.wbf, (int64_t)9 * c.cin * c.cout)) || (s = ualloc(u, &c.wflip, (int64_t)9 * c.cin * c.cout)))
            return fail(s);
    }
    const int64_t P0 = B * height * width;
    if ((s = ualloc(u, &u->xin, P0 * 4))) return fail(s);
    u->ea.resize(levels); u->ebb.resize(levels); u->eb.resize(levels); u->pool.resize(levels);
    u->da.resize(levels); u->dbb.resize(levels);
    u->g_ea.resize(levels); u->g_eb.resize(levels); u->g_pool.resize(levels); u->g_up.resize(levels);
    u->g_da.resize(levels); u->g_db.resize(levels);
    u->g_eab.resize(levels); u->g_ebb.resize(levels); u->g_dab.resize(levels); u->g_dbb.resize(levels);
    int64_t maxpart = 1;
    for (int l = 0; l < levels; ++l) {
        const int64_t P = B * (height >> l) * (width >> l);
        const int c = u->ch[l];
        if ((s = ualloc(u, &u->ea[l], P * c)) || (s = ualloc(u, &u->ebb[l], P * c)) || (s = ualloc(u, &u->eb[l], P * c)) ||
            (s = ualloc(u, &u->g_ea[l], P * c)) || (s = ualloc(u, &u->g_eb[l], P * c)) ||
            (s = ualloc(u, &u->g_eab[l], P * c)) || (s = ualloc(u, &u->g_ebb[l], P * c)))
            return fail(s);
        if (l > 0 && ((s = ualloc(u, &u->pool[l], P * u->ch[l - 1])) || (s = ualloc(u, &u->g_pool[l], P * u->ch[l - 1]))))
            return fail(s);
        if (l <= levels - 2) {
            if ((s = ualloc(u, &u->da[l], P * c)) || (s = ualloc(u, &u->dbb[l], P * c)) ||
                (s = ualloc(u, &u->g_up[l], P * u->ch[l + 1])) || (s = ualloc(u, &u->g_da[l], P * c)) ||
                (s = ualloc(u, &u->g_db[l], P * c)) || (s = ualloc(u, &u->g_dab[l], P * c)) ||
                (s = ualloc(u, &u->g_dbb[l], P * c)))
                return fail(s);
            if (l == 0 && (s = ualloc(u, &u->db0, P * c))) return fail(s);
        }
    }
    for (const ConvLayer &c : u->conv) maxpart = std::max<int64_t>(maxpart, gw_part_len((int)B, c.h, c.w, c.cin, c.cout));
    if ((s = ualloc(u, &u->part, maxpart)) || (s = ualloc(u, &u->out, P0)) || (s = ualloc(u, &u->gout, P0)) ||
        (s = ualloc(u, &u->head_part, (int64_t)HEAD_BLOCKS * (u->ch[0] + 1))) ||
        (s = ualloc(u, &u->loss_part, (int64_t)nblocks(P0))) || (s = ualloc(u, &u->loss, 1)))
        return fail(s);
    u->part_len = maxpart;
    // He-normal initialisation, zero biases
    std::vector<float> h(off, 0.f);
    std::mt19937_64 rng(seed);
    for (const ConvLayer &c : u->conv) {
        Normal nd(rng, std::sqrt(2.0 / (9.0 * c.cin)));
        for (int64_t i = 0; i < (int64_t)9 * c.cin * c.cout; ++i) h[c.w_off + i] = (float)nd();
    }
    {
        Normal nd(rng, std::sqrt(1.0 / u->ch[0]));
        for (int k = 0; k < u->ch[0]; ++k) h[u->head_w + k] = (float)nd();
    }
    if ((s = ivx_unet_set_params(u, h.data())) != IVX_OK) return fail(s);
    *out = u;
    return IVX_OK;
}

ivx_status ivx_unet_destroy(ivx_unet *u) {
    if (!u) return IVX_OK;
    ufree(u);
    delete u;
    return IVX_OK;
}

int64_t ivx_unet_param_count(const ivx_unet *u) { return u ? u->nparam : -1; }

ivx_status ivx_unet_get_params(const ivx_unet *u, float *params) {
    ivx_status s = check_net(u);
    if (s) return s;
    if (!params) return set_error(IVX_EINVAL, "params is NULL");
    UHIP(hipMemcpy(params, u->params, u->nparam * sizeof(float), hipMemcpyDefault));
    return IVX_OK;
}

ivx_status ivx_unet_set_params(ivx_unet *u, const float *params) {
    ivx_status s = check_net(u);
    if (s) return s;
    if (!params) return set_error(IVX_EINVAL, "params is NULL");
    UHIP(hipMemcpy(u->params, params, u->nparam * sizeof(float), hipMemcpyDefault));
    UHIP(hipMemset(u->mom, 0, u->nparam * sizeof(float)));
    UHIP(hipMemset(u->vel, 0, u->nparam * sizeof(float)));
    u->step = 0;
    UHIP(refresh_bf16(u, nullptr));
    UHIP(hipDeviceSynchronize());
    return IVX_OK;
}

ivx_status ivx_unet_forward(ivx_unet *u, const float *x, float *y, int32_t batch, void *stream) {
    ivx_status s = check_net(u);
    if (s) return s;
    if (!x || !y || batch < 1 || batch > u->maxb) return set_error(IVX_EINVAL, "bad forward arguments");
    hipStream_t st = (hipStream_t)stream;
    UHIP(forward(u, x, batch, false, st));
    UHIP(hipMemcpyAsync(y, u->out, (size_t)batch * u->H * u->W * sizeof(float), hipMemcpyDeviceToDevice, st));
    return IVX_OK;
}

ivx_status ivx_unet_train_step(ivx_unet *u, const float *x, const float *target, int32_t batch, float lr, double *loss,
                               void *stream) {
    ivx_status s = check_net(u);
    if (s) return s;
    if (!x || !target || batch < 1 || batch > u->maxb || !(lr > 0.f)) return set_error(IVX_EINVAL, "bad train arguments");
    hipStream_t st = (hipStream_t)stream;
    UHIP(forward(u, x, batch, true, st));
    const int64_t P0 = (int64_t)batch * u->H * u->W;
    k_mse<<<nblocks(P0), NT, 0, st>>>(u->out, target, P0, u->gout, u->loss_part);
    k_sum_double<<<1, NT, 0, st>>>(u->loss_part, (int)nblocks(P0), 1.0 / (double)P0, u->loss);
    UHIP(backward(u, batch, st));
    u->step += 1;
    const double b1t = 1.0 - std::pow(0.9, (double)u->step), b2t = 1.0 - std::pow(0.999, (double)u->step);
    // m_hat / (sqrt(v_hat) + eps) = (sqrt(b2t) / b1t) m / (sqrt(v) + eps sqrt(b2t))
    const float lr_t = (float)(lr * std::sqrt(b2t) / b1t), eps_t = (float)(1e-8 * std::sqrt(b2t));
    k_adam<<<nblocks(u->nparam), NT, 0, st>>>(u->params, u->grads, u->mom, u->vel, u->nparam, lr_t, eps_t);
    UHIP(refresh_bf16(u, st));
    if (loss) {
        UHIP(hipMemcpyAsync(loss, u->loss, sizeof(double), hipMemcpyDefault, st));
        hipPointerAttribute_t a;
        bool dev = false;
        if (hipPointerGetAttributes(&a, loss) == hipSuccess) dev = a.type == hipMemoryTypeDevice;
        else (void)hipGetLastError();
        if (!dev) UHIP(hipStreamSynchronize(st));
    }
    return IVX_OK;
}

ivx_status ivx_unet_loss_grad(ivx_unet *u, const float *x, const float *target, int32_t batch, float *grads, double *loss,
                              void *stream) {
    ivx_status s = check_net(u);
    if (s) return s;
    if (!x || !target || !grads || batch < 1 || batch > u->maxb) return set_error(IVX_EINVAL, "bad loss_grad arguments");
    hipStream_t st = (hipStream_t)stream;
    UHIP(forward(u, x, batch, true, st));
    const int64_t P0 = (int64_t)batch * u->H * u->W;
    k_mse<<<nblocks(P0), NT, 0, st>>>(u->out, target, P0, u->gout, u->loss_part);
    k_sum_double<<<1, NT, 0, st>>>(u->loss_part, (int)nblocks(P0), 1.0 / (double)P0, u->loss);
    UHIP(backward(u, batch, st));
    UHIP(hipMemcpyAsync(grads, u->grads, u->nparam * sizeof(float), hipMemcpyDefault, st));
    if (loss) UHIP(hipMemcpyAsync(loss, u->loss, sizeof(double), hipMemcpyDefault, st));
    UHIP(hipStreamSynchronize(st));
    return IVX_OK;
}

// ------------------------------------------------------------------ single layers
ivx_status ivx_nn_conv3x3(const float *x, int32_t n, int32_t h, int32_t w, int32_t cin, const uint16_t *weight,
                          const float *bias, int32_t cout, int32_t relu, const float *mask, int32_t accumulate, float *y,
                          void *stream) {
    if (!x || !weight || !y || n < 1 || h < 1 || w < 1 || cin < 4 || cin % 4 || cout < 16 || cout % 16)
        return set_error(IVX_EINVAL, "bad conv3x3 arguments");
    UHIP(conv3x3_layer(x, n, h, w, cin, weight, bias, cout, relu, mask, accumulate, y, (hipStream_t)stream));
    return IVX_OK;
}

ivx_status ivx_nn_conv3x3_grad_weight(const float *x, const float *dy, int32_t n, int32_t h, int32_t w, int32_t cin,
                                      int32_t cout, float *dw, float *db, void *stream) {
    if (!x || !dy || !dw || !db || n < 1 || h < 1 || w < 1 || cin < 1 || cout < 1)
        return set_error(IVX_EINVAL, "bad conv3x3_grad_weight arguments");
    hipStream_t st = (hipStream_t)stream;
    float *part = nullptr;
    UHIP(hipMalloc(&part, (size_t)gw_part_len(n, h, w, cin, cout) * sizeof(float)));
    hipError_t e = conv3x3_grad_weight(x, dy, n, h, w, cin, cout, part, dw, db, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(part);
    if (e != hipSuccess) return set_error(IVX_EHIP, std::string("conv3x3_grad_weight: ") + hipGetErrorString(e));
    return IVX_OK;
}

ivx_status ivx_nn_conv3x3_grad_weight_noalloc(const float *x, const float *dy, int32_t n, int32_t h, int32_t w,
                                              int32_t cin, int32_t cout, float *dw, float *db, void *stream) {
    if (!x || !dy || !dw || !db || n < 1 || h < 1 || w < 1 || cin < 1 || cout < 1)
        return set_error(IVX_EINVAL, "bad conv3x3_grad_weight_noalloc arguments");
    const int64_t need = gw_part_len(n, h, w, cin, cout);
    if (need > NOALLOC_PART_FLOATS)
        return set_error(IVX_EINVAL, "conv3x3_grad_weight_noalloc: this shape needs " + std::to_string(need) +
                                         " floats of split partials, more than the " +
                                         std::to_string(NOALLOC_PART_FLOATS) +
                                         " of the static scratch (use ivx_nn_conv3x3_grad_weight)");
    float *part = nullptr;
    hipError_t e = scratch_on_current_device(&part);
    if (e != hipSuccess)
        return set_error(IVX_EHIP, std::string("conv3x3_grad_weight_noalloc: hipGetSymbolAddress: ") +
                                       hipGetErrorString(e));
    e = conv3x3_grad_weight(x, dy, n, h, w, cin, cout, part, dw, db, (hipStream_t)stream);
    if (e != hipSuccess) return set_error(IVX_EHIP, std::string("conv3x3_grad_weight_noalloc: ") + hipGetErrorString(e));
    return IVX_OK;
}

int64_t ivx_nn_conv3x3_grad_weight_noalloc_capacity(void) { return NOALLOC_PART_FLOATS; }

int64_t ivx_nn_conv3x3_grad_weight_scratch_floats(int32_t n, int32_t h, int32_t w, int32_t cin, int32_t cout) {
    if (n < 1 || h < 1 || w < 1 || cin < 1 || cout < 1) return -1;
    return gw_part_len(n, h, w, cin, cout);
}

ivx_status ivx_nn_conv3x3_flip(const uint16_t *weight, int32_t cin, int32_t cout, uint16_t *flipped, void *stream) {
    if (!weight || !flipped || cin < 1 || cout < 1) return set_error(IVX_EINVAL, "bad flip arguments");
    const int64_t nw = (int64_t)9 * cin * cout;
    k_flip<<<nblocks(nw), NT, 0, (hipStream_t)stream>>>(weight, cin, cout, flipped);
    UHIP(hipGetLastError());
    return IVX_OK;
}

ivx_status ivx_nn_to_bf16(const float *x, int64_t count, uint16_t *out, void *stream) {
    if (!x || !out || count < 0) return set_error(IVX_EINVAL, "bad to_bf16 arguments");
    if (count) k_to_bf16<<<nblocks(count), NT, 0, (hipStream_t)stream>>>(x, count, out);
    UHIP(hipGetLastError());
    return IVX_OK;
}

ivx_status ivx_nn_pool2(const float *x, int32_t n, int32_t h, int32_t w, int32_t c, float *y, void *stream) {
    if (!x || !y || n < 1 || h < 2 || w < 2 || h % 2 || w % 2 || c < 1) return set_error(IVX_EINVAL, "bad pool2 arguments");
    k_pool2<<<nblocks((int64_t)n * (h / 2) * (w / 2) * c), NT, 0, (hipStream_t)stream>>>(x, n, h, w, c, y);
    UHIP(hipGetLastError());
    return IVX_OK;
}

ivx_status ivx_nn_pool2_grad(const float *x, const float *dy, int32_t n, int32_t h, int32_t w, int32_t c,
                             int32_t accumulate, float *dx, void *stream) {
    if (!x || !dy || !dx || n < 1 || h < 2 || w < 2 || h % 2 || w % 2 || c < 1)
        return set_error(IVX_EINVAL, "bad pool2_grad arguments");
    k_pool2_grad<<<nblocks((int64_t)n * (h / 2) * (w / 2) * c), NT, 0, (hipStream_t)stream>>>(x, dy, n, h, w, c,
                                                                                              accumulate, dx, nullptr);
    UHIP(hipGetLastError());
    return IVX_OK;
}

ivx_status ivx_nn_up2(const float *x, int32_t n, int32_t h, int32_t w, int32_t c, float *y, void *stream) {
    if (!x || !y || n < 1 || h < 1 || w < 1 || c < 1) return set_error(IVX_EINVAL, "bad up2 arguments");
    k_up2<<<nblocks((int64_t)n * 4 * h * w * c), NT, 0, (hipStream_t)stream>>>(x, n, h, w, c, y);
    UHIP(hipGetLastError());
    return IVX_OK;
}

ivx_status ivx_nn_up2_grad(const float *dy, int32_t n, int32_t h, int32_t w, int32_t c, float *dx, void *stream) {
    if (!dy || !dx || n < 1 || h < 1 || w < 1 || c < 1) return set_error(IVX_EINVAL, "bad up2_grad arguments");
    k_up2_grad<<<nblocks((int64_t)n * h * w * c), NT, 0, (hipStream_t)stream>>>(dy, n, h, w, c, dx, nullptr);
    UHIP(hipGetLastError());
    return IVX_OK;
}

} // extern "C"
