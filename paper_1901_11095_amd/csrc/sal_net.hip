// Learned surrogate of the saliency method: five 3x3x3 convolutions, channels
// 1 -> 24 -> 24 -> 24 -> 24 -> 3, GELU after the first four, predicting the three raw
// directional-comparison maps (S_t, S_x, S_y) of the plain method from the volume.  BF16
// weights and activations, FP32 accumulation on MFMA, FP32 master weights and Adam.
//
// Tensors are channel-last, act[b][t][u][w][c], over nb blocks of n0 x n1 x n2 voxels (a
// batch of training crops, or one whole volume).  Weights W[co][k][ci], tap k = (dt*3+du)*3+dw
// reading the input at (t+dt-1, u+du-1, w+dw-1), reflected inside the block (-1 -> 1).
//
// Training: the loss covers only voxels at least `margin` (>= 5) from every block face, so
// every nonzero gradient of a layer's output stays one voxel further inside than the
// previous one and the backward pass never meets the reflected taps: the input gradient is
// a zero-padded convolution with the flipped, transposed kernel, run by the same kernel.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <random>
#include <string>
#include <vector>

#include "sal_device.h"
#include "sal_internal.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int NL = 5;
constexpr int CH[NL + 1] = {1, 24, 24, 24, 24, 3};
constexpr int TT = 4, TU = 4, TW = 16;                  // output tile of a weight-gradient workgroup
constexpr int PT = TT + 2, PU = TU + 2, PW = TW + 2;    // input tile with the 1-voxel halo
constexpr int NPOS = PT * PU * PW;
// Output tile of a convolution workgroup: FT x FU x FW voxels, one wave per 4 rows of FW.
// Layers with 24 output channels take 4 x 8 x 16 (eight waves; the 6 x 10 x 18 input tile
// is 2.1 times the output instead of 2.5 times for 4 x 4 x 16), the 3-channel output layer
// keeps 4 x 4 x 16 (four waves), which measured faster there.
constexpr int FT = 4, FW = 16, FPT = FT + 2, FPW = FW + 2;
__host__ __device__ constexpr int conv_fu(int co) { return co >= 16 ? 8 : 4; }
__host__ __device__ constexpr int conv_threads(int co) { return 64 * FT * conv_fu(co) / 4; }
constexpr int WG_BLOCKS = 512;                          // workgroups of the weight-gradient pass
constexpr unsigned CONV_BLOCKS = 2048;                  // persistent workgroups of a convolution, at most

enum { MODE_REFLECT = 0, MODE_ZERO = 1 };
enum { EPI_GELU = 0, EPI_LINEAR = 1, EPI_DGELU = 2 };

__host__ __device__ constexpr int pad8(int c) { return (c + 7) / 8 * 8; }
// K of a conv with ci input channels: taps x channels padded to 8; a single channel packs
// 27 taps into one 32-wide step
__host__ __device__ constexpr int kgroups(int ci) { return ci == 1 ? 4 : 27 * pad8(ci) / 8; }
__host__ __device__ constexpr int ksteps(int ci) { return (kgroups(ci) + 3) / 4; }

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t f2bf(float f)
{
    const __bf16 h = (__bf16)f;
    return __builtin_bit_cast(uint16_t, h);
}

// erf by Abramowitz & Stegun 7.1.26 (|error| <= 1.5e-7), GELU(z) = z/2 (1 + erf(z/sqrt2)).
__device__ __forceinline__ void erf_as(float x, float &erfv, float &gauss)
{
    const float ax = fabsf(x);
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));
    const float poly = t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f),
                                         -0.284496736f), 0.254829592f);
    gauss = __expf(-ax * ax);
    erfv = copysignf(1.0f - poly * gauss, x);
}
__device__ __forceinline__ float gelu_f(float z)
{
    float e, gs;
    erf_as(z * 0.70710678118654752f, e, gs);
    return 0.5f * z * (1.0f + e);
}
__device__ __forceinline__ float gelu_grad_f(float z)
{
    float e, gs;
    erf_as(z * 0.70710678118654752f, e, gs);  // gs = exp(-z^2/2)
    return 0.5f * (1.0f + e) + z * gs * 0.39894228040143268f;
}

// Storage type of activations and gradients: BF16 (the network's arithmetic) or FP32 (the
// FP32-operand mode, which runs the same kernels with FP32 operands for element-wise checks)
template <bool F32>
struct ActT {
    using type = uint16_t;
};
template <>
struct ActT<true> {
    using type = float;
};
template <bool F32>
__device__ __forceinline__ typename ActT<F32>::type to_act(float f)
{
    if constexpr (F32)
        return f;
    else
        return f2bf(f);
}
template <bool F32>
__device__ __forceinline__ float from_act(typename ActT<F32>::type a)
{
    if constexpr (F32)
        return a;
    else
        return bf2f(a);
}

// 16 bytes from global memory straight into LDS at the row base `dst` + 16 * lane
__device__ __forceinline__ void load16_to_lds(const uint16_t *src, uint16_t *dst)
{
    __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

// four consecutive channels of one voxel (16-byte aligned in FP32, 8-byte in BF16)
template <bool F32>
__device__ __forceinline__ void store4(typename ActT<F32>::type *p, const typename ActT<F32>::type r[4])
{
    if constexpr (F32)
        *reinterpret_cast<float4 *>(p) = make_float4(r[0], r[1], r[2], r[3]);
    else
        *reinterpret_cast<uint2 *>(p) = make_uint2(r[0] | ((uint32_t)r[1] << 16), r[2] | ((uint32_t)r[3] << 16));
}
// two consecutive channels of one voxel (8-byte aligned in FP32, 4-byte in BF16)
template <bool F32>
__device__ __forceinline__ void store2(typename ActT<F32>::type *p, const typename ActT<F32>::type r[2])
{
    if constexpr (F32)
        *reinterpret_cast<float2 *>(p) = make_float2(r[0], r[1]);
    else
        *reinterpret_cast<uint32_t *>(p) = r[0] | ((uint32_t)r[1] << 16);
}
template <bool F32>
__device__ __forceinline__ void load4(const typename ActT<F32>::type *p, typename ActT<F32>::type r[4])
{
    if constexpr (F32) {
        const float4 v = *reinterpret_cast<const float4 *>(p);
        r[0] = v.x;
        r[1] = v.y;
        r[2] = v.z;
        r[3] = v.w;
    } else {
        const uint2 v = *reinterpret_cast<const uint2 *>(p);
        r[0] = (uint16_t)(v.x & 0xffff);
        r[1] = (uint16_t)(v.x >> 16);
        r[2] = (uint16_t)(v.y & 0xffff);
        r[3] = (uint16_t)(v.y >> 16);
    }
}

__device__ __forceinline__ int map_idx(int u, int n, int mode)
{
    if (mode == MODE_ZERO) return (u < 0 || u >= n) ? -1 : u;
    return refl_idx(u, n);
}

}  // namespace

// ------------------------------------------------------------------------------------
// 3x3x3 convolution as an implicit GEMM on 16x16x32 BF16 MFMA: D[co][voxel] =
// sum_K A[co][K] B[K][voxel], K = (tap, input channel).  A (the weights) stays in registers
// for the whole workgroup; B is read from the LDS input tile, 8 channels of one tap = 16
// bytes per lane.  Each wave computes 4 rows of 16 voxels.
//   in:   CI == 1: float [nb][n0][n1][n2]; else Act [nb][...][CI]
//   wtab: Act [MT*16][ksteps*32] (rows >= CO and K past the taps are zero)
//   EPI_GELU:   z = acc + bias -> out0 (Act, optional), GELU(z) -> out1 (Act)
//   EPI_LINEAR: (acc + bias) * oscale[c] -> out0 (float), element (v, c) at v*vstride + c*cstride
//   EPI_DGELU:  acc * GELU'(zprev) -> out0 (Act)
// Act is BF16, or FP32 with F32: the same tiles, K order and epilogues, each 16x16x32 step
// done as eight 16x16x4 FP32 MFMAs over the eight K elements a lane holds (a lane of group g
// holds K = 8g + e, e < 8, in both forms), the weights read from the table at each step,
// the tiles loaded synchronously (two FP32 buffers would not fit the LDS).
template <int CI, int CO, int MODE, int EPI, bool F32>
__global__ __launch_bounds__(conv_threads(CO)) void k_conv3(const void *__restrict__ in, int nb, int n0, int n1,
                                               int n2, const void *__restrict__ wtab,
                                               const float *__restrict__ bias,
                                               const void *__restrict__ zprev, void *out0,
                                               void *out1, int64_t vstride, int64_t cstride,
                                               float3 oscale)
{
    using Act = typename ActT<F32>::type;
    constexpr int CIP = CI == 1 ? 1 : pad8(CI);
    constexpr int KS = ksteps(CI), MT = (CO + 15) / 16;
    constexpr int FU = conv_fu(CO), FPU = FU + 2, FNPOS = FPT * FPU * FPW;
    constexpr int FWAVES = FT * FU / 4, FTHREADS = conv_threads(CO);
    // multi-channel BF16 layers with reflected borders (the forward pass) stream the next
    // tile into a second LDS buffer by direct global-to-LDS loads while the current one
    // computes
    constexpr bool ASYNC = !F32 && CI > 1 && CI % 8 == 0 && MODE == MODE_REFLECT;
    // forward BF16 layers with 24 input channels: two output rows share their input reads
    // (the weight table of these layers is laid out in the matching K order)
    constexpr bool PAIR = !F32 && CI == 24 && MODE == MODE_REFLECT;
    static_assert(!PAIR || ksteps(CI) == 21, "paired rows expect 27 taps x 3 chunks in 7 x 3 K steps");
    // two separate LDS objects, so the compiler can tell reads of one from the loads landing
    // in the other (a read of the same object would wait for them)
    __shared__ __attribute__((aligned(16))) Act tileA[FNPOS * CIP];
    __shared__ __attribute__((aligned(16))) Act tileB[ASYNC ? FNPOS * CIP : 8];
    // biases in LDS: a global load in the epilogue would wait for the tile in flight
    __shared__ float bias_s[MT * 16];

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, n = lane & 15;
    const int ntw = (n2 + FW - 1) / FW, ntu = (n1 + FU - 1) / FU, ntt = (n0 + FT - 1) / FT;
    const int ntiles = nb * ntt * ntu * ntw;
    const int64_t vol = (int64_t)n0 * n1 * n2;
    const Act *act_in = reinterpret_cast<const Act *>(in);

    // asynchronous load of tile `id` into buffer `bf`: each wave takes whole rows of FPW
    // positions; lane j < FPW * CIP / 8 brings 16 bytes (8 channels) and the hardware puts
    // them at row base + 16 j, which is the row's layout in LDS
    auto issue = [&](int id, Act *dst) {
        if constexpr (ASYNC) {
            constexpr int CHK = CIP / 8, ROWLEN = FPW * CHK;
            int bi = id;
            const int tw2 = bi % ntw;
            bi /= ntw;
            const int tu2 = bi % ntu;
            bi /= ntu;
            const int tt2 = bi % ntt;
            const int b2 = bi / ntt;
            const Act *src = act_in + b2 * vol * CI;
            const int pw = lane / CHK, ch = lane - (lane / CHK) * CHK;
            const int gw = refl_idx(tw2 * FW - 1 + pw, n2);
            const int wv = __builtin_amdgcn_readfirstlane(wave);
#pragma unroll
            for (int it = 0; it < (FPT * FPU + FWAVES - 1) / FWAVES; ++it) {
                const int row = FWAVES * it + wv;
                if (row < FPT * FPU) {
                    const int pt = row / FPU, pu = row - pt * FPU;
                    const int gt = refl_idx(tt2 * FT - 1 + pt, n0), gu = refl_idx(tu2 * FU - 1 + pu, n1);
                    if (lane < ROWLEN)
                        load16_to_lds(src + (((int64_t)gt * n1 + gu) * n2 + gw) * CI + 8 * ch, &dst[row * FPW * CIP]);
                }
            }
        }
    };
    for (int i = threadIdx.x; i < MT * 16; i += FTHREADS) bias_s[i] = (bias && i < CO) ? bias[i] : 0.f;
    __syncthreads();
    if (ASYNC && (int)blockIdx.x < ntiles) issue(blockIdx.x, tileA);

    // BF16: the weights stay in registers while the workgroup walks its tiles
    u32x4 A[MT][F32 ? 1 : KS];
    if constexpr (!F32) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int s = 0; s < KS; ++s)
                A[mt][s] = reinterpret_cast<const u32x4 *>(wtab)[((mt * 16 + n) * KS * 32 + s * 32 + 8 * g) / 8];
    }

    // one tile: wait for its input, start the next tile's loads into the other buffer,
    // convolve, write the epilogue
    auto process = [&](int tile_id, Act *tile, Act *other) __attribute__((always_inline)) {
    int bid = tile_id;
    const int tw_ = bid % ntw;
    bid /= ntw;
    const int tu_ = bid % ntu;
    bid /= ntu;
    const int tt_ = bid % ntt;
    const int b = bid / ntt;
    const int t0 = tt_ * FT, u0 = tu_ * FU, w0 = tw_ * FW;
    if (ASYNC) {
        // this tile's loads have landed (every wave waits for its own, then the barrier);
        // the other buffer is free again, so the next tile's loads can start
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tile_id + (int)gridDim.x < ntiles) issue(tile_id + gridDim.x, other);
    } else {
        __syncthreads();  // the previous tile is no longer read
    }

    // input tile with halo: one row of FPW positions per (pt, pu).  Each wave loads whole
    // rows, so the row's (t, u) source index is wave-uniform and a lane's position along
    // w is fixed for the tile.
    if (CI == 1) {
        // three rows of FPW floats per wave and step
        const float *src = reinterpret_cast<const float *>(in) + b * vol;
        const int r3 = lane / FPW, pw = lane - r3 * FPW;
        const bool act = r3 < 3;
        const int gw = map_idx(w0 - 1 + pw, n2, MODE);
#pragma unroll
        for (int it = 0; it < (FPT * FPU + 3 * FWAVES - 1) / (3 * FWAVES); ++it) {
            const int row = 3 * FWAVES * it + 3 * wave + r3;
            if (act && row < FPT * FPU) {
                const int pt = row / FPU, pu = row - pt * FPU;
                const int gt = map_idx(t0 - 1 + pt, n0, MODE), gu = map_idx(u0 - 1 + pu, n1, MODE);
                const float v = (gt < 0 || gu < 0 || gw < 0) ? 0.f : src[((int64_t)gt * n1 + gu) * n2 + gw];
                tile[row * FPW + pw] = to_act<F32>(v);
            }
        }
    } else if (ASYNC) {
        // loaded by issue()
    } else if (CI % 8 == 0) {
        // chunks of 8 channels (16 bytes in BF16, two 16-byte halves in FP32); a row of FPW
        // positions is ROWLEN <= 64 chunks
        constexpr int CHK = CIP / 8, ROWLEN = FPW * CHK, NQ = F32 ? 2 : 1;
        static_assert(ROWLEN <= 64, "one wave loads a whole row");
        const Act *src = act_in + b * vol * CI;
        const bool act = lane < ROWLEN;
        const int pw = lane / CHK, ch = lane - (lane / CHK) * CHK;
        const int gw = map_idx(w0 - 1 + pw, n2, MODE);
        const int wv = __builtin_amdgcn_readfirstlane(wave);
#pragma unroll
        for (int it = 0; it < (FPT * FPU + FWAVES - 1) / FWAVES; ++it) {
            const int row = FWAVES * it + wv;
            if (row < FPT * FPU) {
                const int pt = row / FPU, pu = row - pt * FPU;
                const int gt = map_idx(t0 - 1 + pt, n0, MODE), gu = map_idx(u0 - 1 + pu, n1, MODE);
                u32x4 val[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) val[q] = u32x4{0u, 0u, 0u, 0u};
                if (act && gt >= 0 && gu >= 0 && gw >= 0) {
                    const u32x4 *p = reinterpret_cast<const u32x4 *>(src + (((int64_t)gt * n1 + gu) * n2 + gw) * CI + 8 * ch);
#pragma unroll
                    for (int q = 0; q < NQ; ++q) val[q] = p[q];
                }
                if (act) {
                    u32x4 *d = reinterpret_cast<u32x4 *>(&tile[(row * FPW + pw) * CIP + 8 * ch]);
#pragma unroll
                    for (int q = 0; q < NQ; ++q) d[q] = val[q];
                }
            }
        }
    } else {
        const Act *src = act_in + b * vol * CI;
        for (int i = threadIdx.x; i < FNPOS * CIP; i += FTHREADS) {
            const int p = i / CIP, c = i - p * CIP;
            const int row = p / FPW, pw = p - row * FPW;
            const int pt = row / FPU, pu = row - pt * FPU;
            const int gt = map_idx(t0 - 1 + pt, n0, MODE), gu = map_idx(u0 - 1 + pu, n1, MODE),
                      gw = map_idx(w0 - 1 + pw, n2, MODE);
            tile[i] = (c >= CI || gt < 0 || gu < 0 || gw < 0) ? (Act)0 : src[(((int64_t)gt * n1 + gu) * n2 + gw) * CI + c];
        }
    }
    // (asynchronous tiles were complete at the barrier above; a barrier here would wait for
    // the next tile's loads)
    if (!ASYNC) __syncthreads();

    // epilogue of one row of 16 output voxels (lt, lu, n) of the tile
    auto epilogue = [&](f4(&acc)[MT], int lt, int lu) __attribute__((always_inline)) {
        // epilogue: lane (g, n) holds channels 16mt + 4g + j of voxel n.  With 24 output
        // channels the last M tile holds 8, all in lane groups 0 and 1: its channels +2 and +3
        // move to lane groups 2 and 3 (one lane swap per pair, done by every lane), so each lane
        // evaluates two GELUs there instead of half the lanes evaluating four.
        constexpr bool SPREAD = EPI == EPI_GELU && CO % 16 == 8;
        float sp[2] = {0.f, 0.f};
        if constexpr (SPREAD) {
            const auto s0 = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[MT - 1][0]),
                                                             __float_as_uint(acc[MT - 1][2]), false, false);
            const auto s1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[MT - 1][1]),
                                                             __float_as_uint(acc[MT - 1][3]), false, false);
            sp[0] = __uint_as_float(s0[0]);
            sp[1] = __uint_as_float(s1[0]);
        }
        const int gt = t0 + lt, gu = u0 + lu, gw = w0 + n;
        if (gt < n0 && gu < n1 && gw < n2) {
            const int64_t v = b * vol + ((int64_t)gt * n1 + gu) * n2 + gw;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int cb = 16 * mt + 4 * g;
                if (SPREAD && mt == MT - 1) {
                    // channels c2, c2 + 1 of this voxel
                    const int c2 = 16 * mt + 4 * (g & 1) + 2 * (g >> 1);
                    Act zz[2], r[2];
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        zz[j] = to_act<F32>(sp[j] + bias_s[c2 + j]);
                        r[j] = to_act<F32>(gelu_f(from_act<F32>(zz[j])));
                    }
                    if (out0) store2<F32>(reinterpret_cast<Act *>(out0) + v * CO + c2, zz);
                    store2<F32>(reinterpret_cast<Act *>(out1) + v * CO + c2, r);
                } else if (EPI == EPI_LINEAR) {
                    float *o = reinterpret_cast<float *>(out0);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (cb + j < CO) {
                            const float sc = cb + j == 0 ? oscale.x : (cb + j == 1 ? oscale.y : oscale.z);
                            o[v * vstride + (cb + j) * cstride] = (acc[mt][j] + bias_s[cb + j]) * sc;
                        }
                } else if (cb < CO) {  // CO is a multiple of 4 here
                    Act r[4];
                    if (EPI == EPI_GELU) {
                        Act zz[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float z = acc[mt][j] + bias_s[cb + j];
                            zz[j] = to_act<F32>(z);
                            r[j] = to_act<F32>(gelu_f(from_act<F32>(zz[j])));
                        }
                        if (out0) store4<F32>(reinterpret_cast<Act *>(out0) + v * CO + cb, zz);
                        store4<F32>(reinterpret_cast<Act *>(out1) + v * CO + cb, r);
                    } else {
                        Act zv[4];
                        load4<F32>(reinterpret_cast<const Act *>(zprev) + v * CO + cb, zv);
#pragma unroll
                        for (int j = 0; j < 4; ++j) r[j] = to_act<F32>(acc[mt][j] * gelu_grad_f(from_act<F32>(zv[j])));
                        store4<F32>(reinterpret_cast<Act *>(out0) + v * CO + cb, r);
                    }
                }
            }
        }
    };

    if constexpr (PAIR) {
        // Two rows (lu, lu + 1) at a time: for each (dt, dw, channel chunk) a lane reads the
        // four input rows lu .. lu + 3 once, and the three K steps du = 0, 1, 2 use rows du and
        // du + 1 for the two output rows (4 LDS reads for 12 MFMAs instead of 6; four
        // independent accumulator chains).  K slot (3 sg + du, g) of the weight table holds
        // tap (dt, du, dw) and chunk ch of tc = 4 sg + g = (dt * 3 + dw) * 3 + ch.
#pragma unroll 1
        for (int rp = 0; rp < 2; ++rp) {
            const int lt = wave % FT, lu = (wave / FT) * 4 + 2 * rp;
            f4 acc0[MT], acc1[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc0[mt] = acc1[mt] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int sg = 0; sg < KS / 3; ++sg) {
                const int tc = 4 * sg + g;
                u32x4 P[4];
                if (tc < 27) {
                    const int dt = tc / 9, dw = (tc / 3) % 3, ch = tc % 3;
                    const Act *src = &tile[(((lt + dt) * FPU + lu) * FPW + n + dw) * CIP + 8 * ch];
#pragma unroll
                    for (int i = 0; i < 4; ++i) P[i] = *reinterpret_cast<const u32x4 *>(src + i * FPW * CIP);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) P[i] = u32x4{0u, 0u, 0u, 0u};
                }
#pragma unroll
                for (int du = 0; du < 3; ++du) {
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        acc0[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A[mt][3 * sg + du]),
                                                                           __builtin_bit_cast(bf16x8, P[du]), acc0[mt], 0, 0, 0);
                        acc1[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A[mt][3 * sg + du]),
                                                                           __builtin_bit_cast(bf16x8, P[du + 1]), acc1[mt], 0, 0, 0);
                    }
                }
            }
            epilogue(acc0, lt, lu);
            epilogue(acc1, lt, lu + 1);
        }
    } else {
#pragma unroll 1
    for (int row = 0; row < 4; ++row) {
        const int lt = wave % FT, lu = (wave / FT) * 4 + row;  // output voxel (lt, lu, n) of the tile
        f4 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if constexpr (F32) {
                // the eight K elements of this lane, K = 32 s + 8 g + e, as FP32
                float bk[8];
                if (CI == 1) {
                    // K element e of group g is tap 8g + e
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int k = 8 * g + e;
                        bk[e] = 0.f;
                        if (k < 27) bk[e] = tile[((lt + k / 9) * FPU + (lu + (k / 3) % 3)) * FPW + n + k % 3];
                    }
                } else {
                    const int q = 4 * s + g;  // K group: tap q / (CIP/8), channels 8*(q % (CIP/8))
#pragma unroll
                    for (int e = 0; e < 8; ++e) bk[e] = 0.f;
                    if (q < kgroups(CI)) {
                        const int k = q / (CIP / 8), c0 = 8 * (q % (CIP / 8));
                        const int p = ((lt + k / 9) * FPU + (lu + (k / 3) % 3)) * FPW + n + k % 3;
                        const float4 *src4 = reinterpret_cast<const float4 *>(&tile[p * CIP + c0]);
                        const float4 lo = src4[0], hi = src4[1];
                        bk[0] = lo.x; bk[1] = lo.y; bk[2] = lo.z; bk[3] = lo.w;
                        bk[4] = hi.x; bk[5] = hi.y; bk[6] = hi.z; bk[7] = hi.w;
                    }
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const float *wr = reinterpret_cast<const float *>(wtab) + (mt * 16 + n) * KS * 32 + s * 32 + 8 * g;
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[mt] = mfma4(wr[e], bk[e], acc[mt]);
                }
            } else {
                u32x4 bv;
                if (CI == 1) {
                    // K element e of group g is tap 8g + e
#pragma unroll
                    for (int e2 = 0; e2 < 4; ++e2) {
                        uint32_t pr = 0;
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const int k = 8 * g + 2 * e2 + h;
                            uint32_t val = 0;
                            if (k < 27) {
                                const int p = ((lt + k / 9) * FPU + (lu + (k / 3) % 3)) * FPW + n + k % 3;
                                val = tile[p];
                            }
                            pr |= val << (16 * h);
                        }
                        bv[e2] = pr;
                    }
                } else {
                    const int q = 4 * s + g;  // K group: tap q / (CIP/8), channels 8*(q % (CIP/8))
                    if (q < kgroups(CI)) {
                        const int k = q / (CIP / 8), c0 = 8 * (q % (CIP / 8));
                        const int p = ((lt + k / 9) * FPU + (lu + (k / 3) % 3)) * FPW + n + k % 3;
                        bv = *reinterpret_cast<const u32x4 *>(&tile[p * CIP + c0]);
                    } else {
                        bv = u32x4{0u, 0u, 0u, 0u};
                    }
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A[mt][s]),
                                                                      __builtin_bit_cast(bf16x8, bv), acc[mt], 0,
                                                                      0, 0);
            }
        }
        epilogue(acc, lt, lu);
    }
    }
    };

    if constexpr (ASYNC) {
        // even steps read tileA and fill tileB, odd steps the other way round
        for (int tile_id = blockIdx.x; tile_id < ntiles;) {
            process(tile_id, tileA, tileB);
            tile_id += gridDim.x;
            if (tile_id >= ntiles) break;
            process(tile_id, tileB, tileA);
            tile_id += gridDim.x;
        }
    } else {
#pragma unroll 1
        for (int tile_id = blockIdx.x; tile_id < ntiles; tile_id += gridDim.x) process(tile_id, tileA, tileB);
    }

}

// Which walk a workgroup of the weight gradient takes: the tiles that carry a gradient recur with
// the blocks' period (16 tiles for 16^3), so consecutive walks go to one XCD (each then has whole
// blocks), shifted by half a period from one round over its CUs to the next.  Batch of 64 blocks of
// 16^3, walks in launch order -> this: layers 4, 3 and 2 24.2, 25.0 and 25.1 -> 20.7, 22.8 and 23.5 us, a
// training step 357 -> 347 us (of 128 593 -> 567).  Other grids have no such period or fewer
// workgroups than CUs, and keep the launch order.
__device__ __forceinline__ int wgrad_walk()
{
    int wg = blockIdx.x;
    if ((gridDim.x & 511) == 0) {
        const int i = wg >> 3, per = gridDim.x >> 3;
        wg = (wg & 7) * per + (i & ~31) + ((i + 8 * (i >> 5)) & 31);
    }
    return wg;
}

// ------------------------------------------------------------------------------------
// Weight and bias gradient of a layer with 24 BF16 input channels (the FP32-operand mode and the
// one-channel layer take k_conv3_wgrad below): dW[co][k][ci] = sum_v dz[v][co] in[refl(v+k-1)][ci],
// db[co] = sum_v dz[v][co].  BF16 16x16x32 MFMA, whose products of BF16 values are exact and
// whose sums are FP32, with M = co, N = ci, K = two rows of 16 voxels along w.  K runs over
// voxels, so both operands lie channel by channel in LDS ([ci][position], [co][voxel], two
// positions packed per write): a lane reads its eight voxels of a channel in one piece, and the
// ten positions that the taps dw = 0, 1, 2 of one (dt, du) need make three operands in registers.
// A unit is one (dt, du) with channels 0..15, or channels 16..23 of two (dt, du): 14 units, two
// per wave.  Each workgroup walks a fixed stride of tiles and writes its own partial sums
// (summed afterwards in a fixed order: deterministic).  A K step without a nonzero dz is passed
// over as in k_conv3_wgrad.  Batch of 64 16^3 blocks, 24 -> 24 channels, layers 4, 3 and 2: on FP32
// MFMA 53, 88 and 99 us, so 21, 23 and 24 us;
// gradients of layer 2 against FP64 from the same activations: RMS error 3.2e-7 either way (the FP32
// sums').
template <int CO>
__global__ __launch_bounds__(512) void k_conv3_wgrad16(const uint16_t *__restrict__ in, const uint16_t *__restrict__ dz,
                                                       int nb, int n0, int n1, int n2, float *__restrict__ part)
{
    constexpr int CI = 24, MT = (CO + 15) / 16, NV = TT * TU * TW, NPAR = CO * 27 * CI + CO;
    static_assert(TW == 16 && TU % 2 == 0 && NV % 32 == 0 && NV / 32 <= 32, "K steps of two rows of 16 voxels");
    constexpr int RW = 24;                            // positions' row stride: 16-byte reads
    constexpr int CS = ((TT + 2) * PU * RW / 2 + 63) / 64 * 128 + 8;  // channel stride: 4 banks apart
    constexpr int VS = NV + 8;                        // dz channel stride: 4 banks apart
    constexpr int UNITS = 14, NPP = PW / 2;
    static_assert(PW % 2 == 0 && PW <= RW, "pairs of positions");
    __shared__ __attribute__((aligned(16))) uint16_t tin[CI * CS];
    __shared__ __attribute__((aligned(16))) uint16_t tdz[16 * MT * VS];
    __shared__ uint32_t live_s;  // bit q: some dz of the voxels 32q .. 32q + 31 is not zero
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, n = lane & 15;
    const int ntw = (n2 + TW - 1) / TW, ntu = (n1 + TU - 1) / TU, ntt = (n0 + TT - 1) / TT;
    const int ntiles = nb * ntt * ntu * ntw;
    const int64_t vol = (int64_t)n0 * n1 * n2;

    // this lane's (dt, du) and channel in the wave's units, and where its operands start
    int uk[2], uc[2], ub[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const int u = wave + 8 * a;
        uk[a] = u < 9 ? u : 2 * (u - 9) + (n >> 3);
        uc[a] = u < 9 ? n : 16 + (n & 7);
        const int k = uk[a] < 9 ? uk[a] : 8;
        ub[a] = uc[a] * CS + ((k / 3) * PU + k % 3 + (g >> 1)) * RW + 8 * (g & 1);
    }
    f4 acc[2][3][MT];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int dw = 0; dw < 3; ++dw)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[a][dw][mt] = f4{0.f, 0.f, 0.f, 0.f};
    float dbias = 0.f;
    for (int i = threadIdx.x; i < (16 * MT - CO) * VS; i += 512) tdz[CO * VS + i] = 0;  // rows past CO
    auto inf_or_nan = [](uint32_t v) {  // two BF16 values
        return (((v & 0x7fff7fffu) + 0x00800080u) & 0x80008000u) != 0u;
    };

    const int wg = wgrad_walk();
    for (int tile = wg; tile < ntiles; tile += gridDim.x) {
        int bid = tile;
        const int tw_ = bid % ntw;
        bid /= ntw;
        const int tu_ = bid % ntu;
        bid /= ntu;
        const int tt_ = bid % ntt;
        const int b = bid / ntt;
        const int t0 = tt_ * TT, u0 = tu_ * TU, w0 = tw_ * TW;
        __syncthreads();
        if (threadIdx.x == 0) live_s = 0u;
        bool odd = false;  // an infinity or a NaN among this thread's inputs
        // channels 8 ch .. 8 ch + 7 of two positions or voxels next to each other, transposed
        auto put = [](uint16_t *d, int stride, const u32x4 &v0, const u32x4 &v1) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                *reinterpret_cast<uint32_t *>(d + 2 * e * stride) = (v0[e] & 0xffffu) | (v1[e] << 16);
                *reinterpret_cast<uint32_t *>(d + (2 * e + 1) * stride) = (v0[e] >> 16) | (v1[e] & 0xffff0000u);
            }
        };
        for (int i = threadIdx.x; i < (TT + 2) * PU * NPP * 3; i += 512) {
            const int pr = i / 3, ch = i - 3 * pr, row = pr / NPP, pw = 2 * (pr - row * NPP);
            const int64_t line =
                b * vol + ((int64_t)refl_idx(t0 - 1 + row / PU, n0) * n1 + refl_idx(u0 - 1 + row % PU, n1)) * n2;
            const u32x4 v0 = *reinterpret_cast<const u32x4 *>(in + (line + refl_idx(w0 - 1 + pw, n2)) * CI + 8 * ch);
            const u32x4 v1 = *reinterpret_cast<const u32x4 *>(in + (line + refl_idx(w0 + pw, n2)) * CI + 8 * ch);
#pragma unroll
            for (int e = 0; e < 4; ++e) odd |= inf_or_nan(v0[e]) | inf_or_nan(v1[e]);
            put(tin + 8 * ch * CS + row * RW + pw, CS, v0, v1);
        }
        __syncthreads();  // live_s is zero
        auto vox = [&](int vv, int64_t *gi) {
            const int gt = t0 + vv / (TU * TW), gu = u0 + (vv / TW) % TU, gw = w0 + vv % TW;
            *gi = b * vol + ((int64_t)gt * n1 + gu) * n2 + gw;
            return gt < n0 && gu < n1 && gw < n2;
        };
        if constexpr (CO == 24) {
            for (int i = threadIdx.x; i < NV / 2 * 3; i += 512) {
                const int vv = 2 * (i / 3), ch = i % 3;
                u32x4 v[2] = {u32x4{0u, 0u, 0u, 0u}, u32x4{0u, 0u, 0u, 0u}};
                uint32_t any = 0u;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    int64_t gi;
                    if (vox(vv + h, &gi)) v[h] = *reinterpret_cast<const u32x4 *>(dz + gi * CO + 8 * ch);
                    any |= v[h][0] | v[h][1] | v[h][2] | v[h][3];
                }
                put(tdz + 8 * ch * VS + vv, VS, v[0], v[1]);
                if (any & 0x7fff7fffu) atomicOr(&live_s, 1u << (vv >> 5));
            }
        } else {
            for (int i = threadIdx.x; i < NV * CO; i += 512) {
                const int vv = i / CO, c = i - vv * CO;
                int64_t gi;
                const uint16_t v = vox(vv, &gi) ? dz[gi * CO + c] : (uint16_t)0;
                tdz[c * VS + vv] = v;
                if (v & 0x7fffu) atomicOr(&live_s, 1u << (vv >> 5));
            }
        }
        const bool all = __syncthreads_or(odd);
        const uint32_t todo = __builtin_amdgcn_readfirstlane((int)(all ? ~0u : live_s));
        // the bias gradient: one lane per channel of the last wave, which has one unit
        if (threadIdx.x >= 448 && threadIdx.x < 448 + CO) {
#pragma unroll 16
            for (int vv = 0; vv < NV; ++vv) dbias += from_act<false>(tdz[(threadIdx.x - 448) * VS + vv]);
        }
        for (int ks = 0; ks < NV / 32; ++ks) {
            if (!(todo >> ks & 1)) continue;
            bf16x8 av[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                av[mt] = *reinterpret_cast<const bf16x8 *>(tdz + (16 * mt + n) * VS + 32 * ks + 8 * g);
            const int row = (2 * ks / TU * PU + 2 * ks % TU) * RW;
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                if (wave + 8 * a >= UNITS) continue;
                const u32x4 d = *reinterpret_cast<const u32x4 *>(tin + ub[a] + row);
                const uint32_t d4 = *reinterpret_cast<const uint32_t *>(tin + ub[a] + row + 8);
                const u32x4 bv[3] = {d,
                                     u32x4{__builtin_amdgcn_alignbit(d[1], d[0], 16), __builtin_amdgcn_alignbit(d[2], d[1], 16),
                                           __builtin_amdgcn_alignbit(d[3], d[2], 16), __builtin_amdgcn_alignbit(d4, d[3], 16)},
                                     u32x4{d[1], d[2], d[3], d4}};
#pragma unroll
                for (int dw = 0; dw < 3; ++dw)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[a][dw][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            av[mt], __builtin_bit_cast(bf16x8, bv[dw]), acc[a][dw][mt], 0, 0, 0);
            }
        }
    }
    float *pp = part + (int64_t)wg * NPAR;
    if (threadIdx.x >= 448 && threadIdx.x < 448 + CO) pp[CO * 27 * CI + threadIdx.x - 448] = dbias;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        if (wave + 8 * a >= UNITS || uk[a] >= 9) continue;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int co = 16 * mt + 4 * g + j;
                if (co >= CO) continue;
#pragma unroll
                for (int dw = 0; dw < 3; ++dw) pp[(co * 27 + 3 * uk[a] + dw) * CI + uc[a]] = acc[a][dw][mt][j];
            }
    }
}

// ------------------------------------------------------------------------------------
// Weight and bias gradient of one layer of the FP32-operand mode, or of the one-channel layer (its
// input is the FP32 volume): dW[co][k][ci] = sum_v dz[v][co] in[refl(v+k-1)][ci],
// db[co] = sum_v dz[v][co].  FP32 16x16x4 MFMA with M = co, N = ci, K = 4 voxels along w.  Each
// workgroup walks a fixed stride of tiles and writes its own partial sums (summed afterwards
// in a fixed order: deterministic).
//   24 input channels: wave w owns taps w, w+8, w+16, w+24; channels 16..23 of two taps share
//     an N tile (6 MFMAs for two taps at 24 output channels instead of 8);
//   one input channel: N = taps, waves 0..3 one (M, N) tile each.
// Bound by the FP32 matrix work of the voxels that carry a gradient: the loss margin keeps it
// inside the block, dz is zero on 3/4 (last layers) to 1/4 (first) of the voxels of 16^3 blocks,
// and a K step of four zero dz adds +-0 to every sum, so it is passed over (unless the tile's
// inputs hold an infinity or a NaN, whose product with zero counts).  The tiles stay in their
// storage type in LDS, loaded 16 bytes a lane.
template <int CI, int CO, bool F32>
__global__ __launch_bounds__(512) void k_conv3_wgrad(const void *__restrict__ in,
                                                     const void *__restrict__ dz_, int nb, int n0,
                                                     int n1, int n2, float *__restrict__ part)
{
    using Act = typename ActT<F32>::type;
    static_assert(CI == 1 || (CI == 24 && F32), "taps share N tiles in the two layouts above");
    const Act *dz = reinterpret_cast<const Act *>(dz_);
    constexpr int MT = (CO + 15) / 16, NKW = CI == 1 ? 1 : 4, NPR = NKW / 2;
    constexpr int NPAR = CO * 27 * CI + CO, NV = TT * TU * TW;
    __shared__ __attribute__((aligned(16))) float tin[NPOS * CI];
    __shared__ __attribute__((aligned(16))) Act tdz[NV * CO];
    __shared__ uint32_t live_s[2];  // bit q: some dz of the voxels 4q .. 4q + 3 is not zero
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, n = lane & 15;
    const int ntw = (n2 + TW - 1) / TW, ntu = (n1 + TU - 1) / TU, ntt = (n0 + TT - 1) / TT;
    const int ntiles = nb * ntt * ntu * ntw;
    const int64_t vol = (int64_t)n0 * n1 * n2;

    auto tapoff = [](int k) { return ((k / 9) * PU + (k / 3) % 3) * PW + k % 3; };
    // offsets of this lane's B operands from its voxel's position: channel n of the wave's taps,
    // and channels 16..23 of two taps (lanes 0..7 the first, 8..15 the second)
    int off[NKW], offp[NPR > 0 ? NPR : 1];
    if constexpr (CI == 1) {
        const int k = 16 * (wave >> 1) + n;
        off[0] = tapoff(k < 27 ? k : 0);
    } else {
#pragma unroll
        for (int a = 0; a < NKW; ++a) off[a] = tapoff(wave + 8 * a < 27 ? wave + 8 * a : 0) * CI + n;
#pragma unroll
        for (int q = 0; q < NPR; ++q) {
            const int k = wave + 8 * (2 * q + (n >> 3));
            offp[q] = tapoff(k < 27 ? k : 0) * CI + 16 + (n & 7);
        }
    }
    f4 acc[NKW][MT], accp[NPR > 0 ? NPR : 1][MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int a = 0; a < NKW; ++a) acc[a][mt] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < (NPR > 0 ? NPR : 1); ++q) accp[q][mt] = f4{0.f, 0.f, 0.f, 0.f};
    }
    float dbias = 0.f;
    const int wg = wgrad_walk();
    for (int tile = wg; tile < ntiles; tile += gridDim.x) {
        int bid = tile;
        const int tw_ = bid % ntw;
        bid /= ntw;
        const int tu_ = bid % ntu;
        bid /= ntu;
        const int tt_ = bid % ntt;
        const int b = bid / ntt;
        const int t0 = tt_ * TT, u0 = tu_ * TU, w0 = tw_ * TW;
        __syncthreads();
        if (threadIdx.x < 2) live_s[threadIdx.x] = 0u;
        bool odd = false;  // an infinity or a NaN among this thread's inputs
        auto src = [&](int p) {
            const int pt = p / (PU * PW), pu = (p / PW) % PU, pw = p % PW;
            return b * vol + ((int64_t)refl_idx(t0 - 1 + pt, n0) * n1 + refl_idx(u0 - 1 + pu, n1)) * n2 +
                   refl_idx(w0 - 1 + pw, n2);
        };
        if constexpr (CI == 1) {
            for (int p = threadIdx.x; p < NPOS; p += 512) {
                const float v = reinterpret_cast<const float *>(in)[src(p)];
                odd |= !(fabsf(v) < INFINITY);
                tin[p] = v;
            }
        } else {
            constexpr int CHK = CI / 4;  // chunks of 4 channels
            for (int i = threadIdx.x; i < NPOS * CHK; i += 512) {
                const int p = i / CHK, ch = i - p * CHK;
                const u32x4 v = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const float *>(in) + src(p) * CI + 4 * ch);
#pragma unroll
                for (int e = 0; e < 4; ++e) odd |= (v[e] & 0x7fffffffu) >= 0x7f800000u;
                *reinterpret_cast<u32x4 *>(&tin[p * CI + 4 * ch]) = v;
            }
        }
        __syncthreads();  // live_s is zero
        auto vox = [&](int vv, int64_t *gi) {
            const int gt = t0 + vv / (TU * TW), gu = u0 + (vv / TW) % TU, gw = w0 + vv % TW;
            *gi = b * vol + ((int64_t)gt * n1 + gu) * n2 + gw;
            return gt < n0 && gu < n1 && gw < n2;
        };
        if constexpr (CO % 8 == 0) {
            constexpr int CHK = CO / 8, NQ = F32 ? 2 : 1;
            for (int i = threadIdx.x; i < NV * CHK; i += 512) {
                const int vv = i / CHK, ch = i - vv * CHK;
                int64_t gi;
                u32x4 v[NQ];
#pragma unroll
                for (int k = 0; k < NQ; ++k) v[k] = u32x4{0u, 0u, 0u, 0u};
                if (vox(vv, &gi)) {
                    const u32x4 *q = reinterpret_cast<const u32x4 *>(dz + gi * CO + 8 * ch);
#pragma unroll
                    for (int k = 0; k < NQ; ++k) v[k] = q[k];
                }
                uint32_t any = 0u;
#pragma unroll
                for (int k = 0; k < NQ; ++k) {
                    any |= v[k][0] | v[k][1] | v[k][2] | v[k][3];
                    reinterpret_cast<u32x4 *>(&tdz[vv * CO + 8 * ch])[k] = v[k];
                }
                if (any & (F32 ? 0x7fffffffu : 0x7fff7fffu)) atomicOr(&live_s[vv >> 7], 1u << ((vv >> 2) & 31));
            }
        } else {
            for (int i = threadIdx.x; i < NV * CO; i += 512) {
                const int vv = i / CO, c = i - vv * CO;
                int64_t gi;
                const Act v = vox(vv, &gi) ? dz[gi * CO + c] : (Act)0;
                tdz[i] = v;
                if (from_act<F32>(v) != 0.f) atomicOr(&live_s[vv >> 7], 1u << ((vv >> 2) & 31));
            }
        }
        const bool all = __syncthreads_or(odd);
        uint64_t todo = all ? ~0ull : ((uint64_t)live_s[1] << 32 | live_s[0]);
        todo = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)todo) |
               (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(todo >> 32)) << 32;
        // the bias gradient: one lane per channel of the last wave, which has three taps
        if (threadIdx.x >= 448 && threadIdx.x < 448 + CO) {
#pragma unroll 16
            for (int vv = 0; vv < NV; ++vv) dbias += from_act<F32>(tdz[vv * CO + threadIdx.x - 448]);
        }
        if (CI == 1 && (wave >= 4 || (wave & 1) >= MT)) continue;
        // rows of 16 voxels, four K steps each: the operands' addresses are formed once per row
        for (int row = 0; row < TT * TU; ++row) {
            const uint32_t quads = (uint32_t)(todo >> (4 * row)) & 15u;
            if (!quads) continue;
            const int base = ((row / TU) * PU + row % TU) * PW + g;
            const float *bsrc[NKW], *bpsrc[NPR > 0 ? NPR : 1];
#pragma unroll
            for (int a = 0; a < NKW; ++a) bsrc[a] = tin + base * CI + off[a];
#pragma unroll
            for (int q = 0; q < NPR; ++q) bpsrc[q] = tin + base * CI + offp[q];
            const Act *asrc = tdz + (16 * row + g) * CO + n;
#pragma unroll
            for (int w4 = 0; w4 < 4; ++w4) {
                if (!(quads >> w4 & 1)) continue;
                const int ao = 4 * w4 * CO, bo = 4 * w4 * CI;
                if constexpr (CI == 1) {
                    const int mt = wave & 1;
                    const float av = 16 * mt + n < CO ? from_act<F32>(asrc[ao + 16 * mt]) : 0.f;
                    const float bv = 16 * (wave >> 1) + n < 27 ? bsrc[0][bo] : 0.f;
                    acc[0][0] = mfma4(av, bv, acc[0][0]);
                } else {
                    float av[MT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        av[mt] = (16 * mt + n < CO) ? from_act<F32>(asrc[ao + 16 * mt]) : 0.f;
#pragma unroll
                    for (int q = 0; q < NPR; ++q) {
                        const float b0 = bsrc[2 * q][bo], bp = bpsrc[q][bo];
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) acc[2 * q][mt] = mfma4(av[mt], b0, acc[2 * q][mt]);
                        if (wave + 8 * (2 * q + 1) < 27) {
                            const float b1 = bsrc[2 * q + 1][bo];
#pragma unroll
                            for (int mt = 0; mt < MT; ++mt) acc[2 * q + 1][mt] = mfma4(av[mt], b1, acc[2 * q + 1][mt]);
                        }
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) accp[q][mt] = mfma4(av[mt], bp, accp[q][mt]);
                    }
                }
            }
        }
    }
    float *pp = part + (int64_t)wg * NPAR;
    if (threadIdx.x >= 448 && threadIdx.x < 448 + CO) pp[CO * 27 * CI + threadIdx.x - 448] = dbias;
    if constexpr (CI == 1) {
        const int k = 16 * (wave >> 1) + n;
        if (wave < 4 && (wave & 1) < MT && k < 27)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int co = 16 * (wave & 1) + 4 * g + j;
                if (co < CO) pp[co * 27 + k] = acc[0][0][j];
            }
    } else {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int co = 16 * mt + 4 * g + j;
                if (co >= CO) continue;
#pragma unroll
                for (int a = 0; a < NKW; ++a)
                    if (wave + 8 * a < 27) pp[(co * 27 + wave + 8 * a) * CI + n] = acc[a][mt][j];
#pragma unroll
                for (int q = 0; q < NPR; ++q) {
                    const int k = wave + 8 * (2 * q + (n >> 3));
                    if (k < 27) pp[(co * 27 + k) * CI + 16 + (n & 7)] = accp[q][mt][j];
                }
            }
    }
}

// grad[j] += sum over partials (fixed order: one after the other).  Bound by the latency of the
// partials: a 24 -> 24 layer has 32 MB of them for its 15,576 sums, 244 waves' worth.  Four waves
// per 64 sums bring 4 SPB partials at a time into LDS, all their loads in flight, and the first
// adds them up.  Per layer: 61 workgroups of four waves with one load in flight at a time 122 us, one
// wave per 64 sums with 16 loads in flight 14.6 us, this 9.3 us.
constexpr int SPB = 32;
__global__ __launch_bounds__(256) void k_sum_partials(const float *__restrict__ part, int nparts,
                                                      int npar, float *__restrict__ grad)
{
    __shared__ float buf[2][4 * SPB][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = blockIdx.x * 64 + lane;
    const float *src = part + (j < npar ? j : npar - 1);
    float v[SPB], s = 0.f;
    auto load = [&](int p0) {
#pragma unroll
        for (int i = 0; i < SPB; ++i) {
            const int p = p0 + wave * SPB + i;
            v[i] = src[(int64_t)(p < nparts ? p : nparts - 1) * npar];
        }
    };
    load(0);
    for (int p0 = 0, b = 0; p0 < nparts; p0 += 4 * SPB, b ^= 1) {
#pragma unroll
        for (int i = 0; i < SPB; ++i) buf[b][wave * SPB + i][lane] = v[i];
        __syncthreads();
        if (p0 + 4 * SPB < nparts) load(p0 + 4 * SPB);
        if (wave == 0) {
            const int n = nparts - p0 < 4 * SPB ? nparts - p0 : 4 * SPB;
            int i = 0;
            for (; i + 16 <= n; i += 16)
#pragma unroll
                for (int q = 0; q < 16; ++q) s += buf[b][i + q][lane];
            for (; i < n; ++i) s += buf[b][i][lane];
        }
    }
    if (wave == 0 && j < npar) grad[j] += s;
}

// Masked mean squared error: dY = 2 (Y - T) / count on voxels at least `margin` from every
// face of their block (0 elsewhere), as bf16 [..][3]; loss partial sums per workgroup.
template <bool F32>
__global__ __launch_bounds__(256) void k_mse(const float *__restrict__ Y, const float *__restrict__ T,
                                             int nb, int S, int margin, float inv_count,
                                             typename ActT<F32>::type *__restrict__ dY, float *__restrict__ loss_part)
{
    const int64_t tot = (int64_t)nb * S * S * S;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    float l = 0.f;
    if (i < tot) {
        const int w = (int)(i % S), u = (int)((i / S) % S), t = (int)((i / ((int64_t)S * S)) % S);
        const bool in = t >= margin && t < S - margin && u >= margin && u < S - margin && w >= margin &&
                        w < S - margin;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float d = in ? Y[i * 3 + c] - T[i * 3 + c] : 0.f;
            l += d * d;
            dY[i * 3 + c] = to_act<F32>(2.f * d * inv_count);
        }
    }
    __shared__ float red[4];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) l += __shfl_xor(l, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = l;
    __syncthreads();
    if (threadIdx.x == 0) loss_part[blockIdx.x] = (red[0] + red[1] + red[2] + red[3]) * inv_count;
}

__global__ __launch_bounds__(256) void k_sum_loss(const float *__restrict__ part, int n, float *__restrict__ loss)
{
    __shared__ float red[256];
    float s = 0.f;
    for (int i = threadIdx.x; i < n; i += 256) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = red[0];
}

__global__ __launch_bounds__(256) void k_f32_to_bf16(const float *__restrict__ x, int64_t n, uint16_t *__restrict__ y)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) y[i] = f2bf(x[i]);
}

// Adam on the FP32 master parameters (bias-corrected), then clear the gradient.
__global__ __launch_bounds__(256) void k_adam(float *__restrict__ p, float *__restrict__ gr,
                                              float *__restrict__ m, float *__restrict__ v, int n,
                                              float lr, float b1, float b2, float eps, float c1,
                                              float c2)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float gg = gr[i];
    const float mm = b1 * m[i] + (1.f - b1) * gg;
    const float vv = b2 * v[i] + (1.f - b2) * gg * gg;
    m[i] = mm;
    v[i] = vv;
    p[i] -= lr * (mm * c1) / (sqrtf(vv * c2) + eps);
    gr[i] = 0.f;
}

struct prep_layer {
    const float *W;
    int ci, co, fwd_rows, fwd_k, bwd_rows, bwd_k;
    uint16_t *fwd, *bwd;
    float *fwd32, *bwd32;
};
struct prep_args {
    prep_layer l[NL];
};

// Operand tables of layer blockIdx.y from the FP32 master, in BF16 and in FP32 (the FP32-operand
// mode): forward [rows][ksteps*32] and the flipped/transposed kernel of the input-gradient
// conv.  Launch-bound: a launch per layer took 22 us of a training step, one for all 4.3 us.
__global__ __launch_bounds__(256) void k_prep_tables(prep_args args)
{
    const prep_layer &a = args.l[blockIdx.y];
    const float *__restrict__ W = a.W;
    const int ci = a.ci, co = a.co, fwd_rows = a.fwd_rows, fwd_k = a.fwd_k, bwd_rows = a.bwd_rows, bwd_k = a.bwd_k;
    uint16_t *__restrict__ fwd = a.fwd, *__restrict__ bwd = a.bwd;
    float *__restrict__ fwd32 = a.fwd32, *__restrict__ bwd32 = a.bwd32;
    const int i = blockIdx.x * 256 + threadIdx.x;
    // forward: row co, K index = tap * pad8(ci) + c (ci > 1) or tap (ci == 1).  The BF16 table
    // of the 24-channel layers is in the paired-row order of k_conv3: K index 32 s + 8 g + e
    // holds tap (dt, du, dw) and channel 8 ch + e, with s = 3 sg + du and 4 sg + g =
    // (dt * 3 + dw) * 3 + ch (zero past the 27 taps x 3 chunks).
    if (i < fwd_rows * fwd_k) {
        const int r = i / fwd_k, kk = i % fwd_k;
        float w = 0.f, wp = 0.f;
        if (r < co) {
            if (ci == 1) {
                if (kk < 27) w = W[(r * 27 + kk) * ci];
                wp = w;
            } else {
                const int cp = pad8(ci), k = kk / cp, c = kk % cp;
                if (k < 27 && c < ci) w = W[(r * 27 + k) * ci + c];
                wp = w;
                if (ci == 24) {
                    const int st = kk / 32, gg = (kk / 8) % 4, e = kk % 8;
                    const int tc = 4 * (st / 3) + gg, du = st % 3;
                    wp = 0.f;
                    if (tc < 27) {
                        const int dt = tc / 9, dw = (tc / 3) % 3, ch = tc % 3;
                        wp = W[(r * 27 + (dt * 3 + du) * 3 + dw) * ci + 8 * ch + e];
                    }
                }
            }
        }
        fwd[i] = f2bf(wp);
        fwd32[i] = w;
    }
    // backward (input gradient): row = input channel c, K = tap' * pad8(co) + o, weight
    // W[o][26 - tap'][c]
    if (bwd && i < bwd_rows * bwd_k) {
        const int r = i / bwd_k, kk = i % bwd_k;
        const int cp = pad8(co), k = kk / cp, o = kk % cp;
        float w = 0.f;
        if (r < ci && k < 27 && o < co) w = W[(o * 27 + (26 - k)) * ci + r];
        bwd[i] = f2bf(w);
        bwd32[i] = w;
    }
}

// ====================================================================== host side

struct sal_net {
    int device;
    std::vector<int64_t> woff, boff;  // offsets of W and bias of each layer in the flat vector
    int64_t npar;
    float *p, *gr, *m, *v;            // FP32 master, gradient, Adam moments
    uint16_t *fwd[NL], *bwd[NL];      // BF16 operand tables
    float *fwd32[NL], *bwd32[NL];     // FP32 operand tables (FP32-operand mode)
    bool f32 = false;                 // operands and activations in FP32 instead of BF16
    int64_t step;
    float out_scale[3];               // inference output = network output * out_scale
    std::string err;
};

namespace {

thread_local std::string g_net_err;

sal_status nfail(sal_net *n, sal_status s, const std::string &m)
{
    if (n)
        n->err = m;
    else
        g_net_err = m;
    return s;
}

int fwd_rows(int l) { return (CH[l + 1] + 15) / 16 * 16; }
int fwd_k(int l) { return ksteps(CH[l]) * 32; }
int bwd_rows(int l) { return (CH[l] + 15) / 16 * 16; }
int bwd_k(int l) { return ksteps(CH[l + 1]) * 32; }

hipError_t prep_tables(sal_net *n, hipStream_t s)
{
    prep_args a;
    int most = 0;
    for (int l = 0; l < NL; ++l) {
        a.l[l] = {n->p + n->woff[l], CH[l], CH[l + 1], fwd_rows(l), fwd_k(l), bwd_rows(l), l > 0 ? bwd_k(l) : 0,
                  n->fwd[l], l > 0 ? n->bwd[l] : nullptr, n->fwd32[l], l > 0 ? n->bwd32[l] : nullptr};
        most = std::max({most, fwd_rows(l) * fwd_k(l), l > 0 ? bwd_rows(l) * bwd_k(l) : 0});
    }
    hipLaunchKernelGGL(k_prep_tables, dim3((most + 255) / 256, NL), dim3(256), 0, s, a);
    return hipGetLastError();
}

int64_t nvox_of(int64_t nb, int64_t n0, int64_t n1, int64_t n2) { return nb * n0 * n1 * n2; }
unsigned conv_grid(int64_t nb, int64_t n0, int64_t n1, int64_t n2)
{
    return (unsigned)(nb * ((n0 + TT - 1) / TT) * ((n1 + TU - 1) / TU) * ((n2 + TW - 1) / TW));
}
unsigned conv_tiles_fwd(int co, int64_t nb, int64_t n0, int64_t n1, int64_t n2)
{
    const int fu = conv_fu(co);
    return (unsigned)(nb * ((n0 + FT - 1) / FT) * ((n1 + fu - 1) / fu) * ((n2 + FW - 1) / FW));
}

size_t al(size_t x) { return (x + 255) & ~(size_t)255; }

// Training workspace: z1..z4, a1..a4 (24 ch), Y (f32, 3 ch), dY (3 ch), two gradient buffers
// (24 ch), weight-gradient partials, loss partials; activations and gradients take `es`
// bytes per value (2: BF16, 4: the FP32-operand mode).
struct TrainWs {
    size_t z[4], a[4], y, dy, g0, g1, part, lossp, total;
};
TrainWs train_ws(int64_t nv, size_t es)
{
    TrainWs w;
    size_t o = 0;
    for (int l = 0; l < 4; ++l) {
        w.z[l] = o;
        o += al(nv * 24 * es);
        w.a[l] = o;
        o += al(nv * 24 * es);
    }
    w.y = o;
    o += al(nv * 3 * 4);
    w.dy = o;
    o += al(nv * 3 * es);
    w.g0 = o;
    o += al(nv * 24 * es);
    w.g1 = o;
    o += al(nv * 24 * es);
    w.part = o;
    o += al((size_t)WG_BLOCKS * (24 * 27 * 24 + 24) * 4);
    w.lossp = o;
    o += al(((nv + 255) / 256) * 4);
    w.total = o;
    return w;
}
size_t act_bytes(const sal_net *n) { return n->f32 ? 4 : 2; }
// inference workspace: two ping-pong activation buffers of 24 channels
size_t infer_ws(const sal_net *n, int64_t nv) { return 2 * al(nv * 24 * act_bytes(n)); }

template <int CI, int CO, int MODE, int EPI, bool F32>
void conv(const void *in, int64_t nb, int64_t n0, int64_t n1, int64_t n2, const void *w,
          const float *bias, const void *zprev, void *o0, void *o1, int64_t vs, int64_t cs,
          hipStream_t s, float3 oscale = make_float3(1.f, 1.f, 1.f))
{
    // Persistent workgroups, each walking tiles with its weights in registers.  With 24 BF16 input
    // channels as many as the chip holds at once, one or two per CU: more only load the weights
    // and wait for a first tile again (24 -> 24 on 64 blocks of 16^3 29.0 us with a workgroup per
    // tile, 23.6 with 256 for the 512 tiles; 130 x 150 x 170 222 and 183 us, 256^3 920 and 872;
    // 24 -> 3 16.6 and 13.8, 123 and 115, 579 and 570).  The others' weights are few and their
    // starts short: eight per CU balance better (1 -> 24 on 256^3 394 us, 647 with 256).
    constexpr unsigned most = CI == 24 && !F32 ? (CO == 24 ? 256 : 512) : CONV_BLOCKS;
    const unsigned tiles = conv_tiles_fwd(CO, nb, n0, n1, n2);
    const unsigned grid = tiles < most ? tiles : most;
    hipLaunchKernelGGL((k_conv3<CI, CO, MODE, EPI, F32>), dim3(grid), dim3(conv_threads(CO)), 0, s,
                       in, (int)nb, (int)n0, (int)n1, (int)n2, w, bias, zprev, o0, o1, vs, cs, oscale);
}

// forward through all layers; stores z/a (training) or ping-pongs (inference)
template <bool F32>
hipError_t net_forward_t(sal_net *n, const float *X, int64_t nb, int64_t n0, int64_t n1, int64_t n2,
                         char *ws, const TrainWs *tw, float *Y, int64_t vs, int64_t cs, float3 oscale,
                         hipStream_t s)
{
    using Act = typename ActT<F32>::type;
    const float *b[NL];
    const void *w[NL];
    for (int l = 0; l < NL; ++l) {
        b[l] = n->p + n->boff[l];
        w[l] = F32 ? (const void *)n->fwd32[l] : (const void *)n->fwd[l];
    }
    Act *z[4], *a[4];
    for (int l = 0; l < 4; ++l) {
        z[l] = tw ? (Act *)(ws + tw->z[l]) : nullptr;
        a[l] = (Act *)(ws + (tw ? tw->a[l] : (l % 2) * al(nvox_of(nb, n0, n1, n2) * 24 * sizeof(Act))));
    }
    conv<1, 24, MODE_REFLECT, EPI_GELU, F32>(X, nb, n0, n1, n2, w[0], b[0], nullptr, z[0], a[0], 0, 0, s);
    for (int l = 1; l < 4; ++l)
        conv<24, 24, MODE_REFLECT, EPI_GELU, F32>(a[l - 1], nb, n0, n1, n2, w[l], b[l], nullptr, z[l], a[l], 0, 0, s);
    conv<24, 3, MODE_REFLECT, EPI_LINEAR, F32>(a[3], nb, n0, n1, n2, w[4], b[4], nullptr, Y, nullptr, vs, cs, s,
                                               oscale);
    return hipGetLastError();
}
hipError_t net_forward(sal_net *n, const float *X, int64_t nb, int64_t n0, int64_t n1, int64_t n2, char *ws,
                       const TrainWs *tw, float *Y, int64_t vs, int64_t cs, float3 oscale, hipStream_t s)
{
    return n->f32 ? net_forward_t<true>(n, X, nb, n0, n1, n2, ws, tw, Y, vs, cs, oscale, s)
                  : net_forward_t<false>(n, X, nb, n0, n1, n2, ws, tw, Y, vs, cs, oscale, s);
}

template <int CI, int CO, bool F32>
void wgrad(sal_net *n, int l, const void *in, const void *dz, int64_t nb, int64_t n0, int64_t n1, int64_t n2,
           float *part, hipStream_t s)
{
    const int64_t tiles = conv_grid(nb, n0, n1, n2);
    const int grid = (int)(tiles < WG_BLOCKS ? tiles : WG_BLOCKS);
    if constexpr (CI == 24 && !F32)
        hipLaunchKernelGGL(k_conv3_wgrad16<CO>, dim3(grid), dim3(512), 0, s, (const uint16_t *)in, (const uint16_t *)dz,
                           (int)nb, (int)n0, (int)n1, (int)n2, part);
    else
        hipLaunchKernelGGL((k_conv3_wgrad<CI, CO, F32>), dim3(grid), dim3(512), 0, s, in, dz, (int)nb, (int)n0,
                           (int)n1, (int)n2, part);
    const int npar = CO * 27 * CI + CO;
    hipLaunchKernelGGL(k_sum_partials, dim3((npar + 63) / 64), dim3(256), 0, s, part, grid, npar,
                       n->gr + n->woff[l]);
}

// backward from dY ([..][3] in the activation type) through all layers, accumulating the
// gradient
template <bool F32>
hipError_t net_backward_t(sal_net *n, const float *X, const void *dY, int64_t nb, int64_t n0, int64_t n1,
                          int64_t n2, char *ws, const TrainWs &tw, hipStream_t s)
{
    using Act = typename ActT<F32>::type;
    Act *z[4], *a[4];
    for (int l = 0; l < 4; ++l) {
        z[l] = (Act *)(ws + tw.z[l]);
        a[l] = (Act *)(ws + tw.a[l]);
    }
    const void *wb[NL];
    for (int l = 1; l < NL; ++l) wb[l] = F32 ? (const void *)n->bwd32[l] : (const void *)n->bwd[l];
    Act *gbuf[2] = {(Act *)(ws + tw.g0), (Act *)(ws + tw.g1)};
    float *part = (float *)(ws + tw.part);
    // layer 5 (index 4): dW from a4 and dY; input gradient -> dz4 = (W5^T * dY) . GELU'(z4)
    wgrad<24, 3, F32>(n, 4, a[3], dY, nb, n0, n1, n2, part, s);
    conv<3, 24, MODE_ZERO, EPI_DGELU, F32>(dY, nb, n0, n1, n2, wb[4], nullptr, z[3], gbuf[0], nullptr, 0, 0, s);
    const Act *dz = gbuf[0];
    for (int l = 3; l >= 1; --l) {
        wgrad<24, 24, F32>(n, l, a[l - 1], dz, nb, n0, n1, n2, part, s);
        Act *dst = gbuf[(4 - l) % 2];
        conv<24, 24, MODE_ZERO, EPI_DGELU, F32>(dz, nb, n0, n1, n2, wb[l], nullptr, z[l - 1], dst, nullptr, 0, 0, s);
        dz = dst;
    }
    wgrad<1, 24, F32>(n, 0, X, dz, nb, n0, n1, n2, part, s);
    return hipGetLastError();
}
hipError_t net_backward(sal_net *n, const float *X, const void *dY, int64_t nb, int64_t n0, int64_t n1,
                        int64_t n2, char *ws, const TrainWs &tw, hipStream_t s)
{
    return n->f32 ? net_backward_t<true>(n, X, dY, nb, n0, n1, n2, ws, tw, s)
                  : net_backward_t<false>(n, X, dY, nb, n0, n1, n2, ws, tw, s);
}

// One Adam step on the accumulated gradient (which it clears), then the operand tables.
hipError_t adam_step(sal_net *n, float lr, hipStream_t s)
{
    n->step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.0f / (1.0f - std::pow(b1, (float)n->step)), c2 = 1.0f / (1.0f - std::pow(b2, (float)n->step));
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((n->npar + 255) / 256)), dim3(256), 0, s, n->p, n->gr, n->m, n->v,
                       (int)n->npar, lr, b1, b2, 1e-8f, c1, c2);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = prep_tables(n, s);
    return e;
}

struct NetDev {
    int prev = -1;
    explicit NetDev(int d)
    {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        (void)hipSetDevice(d);
    }
    ~NetDev()
    {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
};

}  // namespace

extern "C" {

int64_t sal_net_num_params(void)
{
    int64_t t = 0;
    for (int l = 0; l < NL; ++l) t += (int64_t)CH[l + 1] * 27 * CH[l] + CH[l + 1];
    return t;
}

const char *sal_net_last_error(const sal_net *n) { return n ? n->err.c_str() : g_net_err.c_str(); }

sal_status sal_net_create(int device, uint64_t seed, sal_net **out)
{
    if (!out) return nfail(nullptr, SAL_E_INVAL, "null output pointer");
    *out = nullptr;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev)
        return nfail(nullptr, SAL_E_DEVICE, "no such HIP device");
    NetDev nd(device);
    sal_net *n = new (std::nothrow) sal_net();
    if (!n) return nfail(nullptr, SAL_E_DEVICE, "out of host memory");
    n->device = device;
    n->step = 0;
    n->out_scale[0] = n->out_scale[1] = n->out_scale[2] = 1.f;
    n->p = n->gr = n->m = n->v = nullptr;
    for (int l = 0; l < NL; ++l) {
        n->fwd[l] = n->bwd[l] = nullptr;
        n->fwd32[l] = n->bwd32[l] = nullptr;
    }
    int64_t o = 0;
    for (int l = 0; l < NL; ++l) {
        n->woff.push_back(o);
        o += (int64_t)CH[l + 1] * 27 * CH[l];
        n->boff.push_back(o);
        o += CH[l + 1];
    }
    n->npar = o;
    // Kaiming-uniform weights (bound sqrt(6 / fan_in)), zero biases, from a seeded PCG-free
    // 64-bit Mersenne twister so the initial state depends only on the seed
    std::vector<float> h((size_t)o, 0.f);
    std::mt19937_64 rng(seed);
    std::uniform_real_distribution<double> uni(-1.0, 1.0);
    for (int l = 0; l < NL; ++l) {
        const double bound = std::sqrt(6.0 / (27.0 * CH[l])) * (l == NL - 1 ? 0.5 : 1.0);
        for (int64_t i = 0; i < (int64_t)CH[l + 1] * 27 * CH[l]; ++i) h[n->woff[l] + i] = (float)(bound * uni(rng));
    }
    hipError_t e = hipSuccess;
    float **bufs[4] = {&n->p, &n->gr, &n->m, &n->v};
    for (float **b : bufs) {
        if (e == hipSuccess) e = hipMalloc((void **)b, sizeof(float) * o);
        if (e == hipSuccess) e = hipMemset(*b, 0, sizeof(float) * o);
    }
    if (e == hipSuccess) e = hipMemcpy(n->p, h.data(), sizeof(float) * o, hipMemcpyHostToDevice);
    for (int l = 0; l < NL && e == hipSuccess; ++l) {
        e = hipMalloc((void **)&n->fwd[l], 2 * (size_t)fwd_rows(l) * fwd_k(l));
        if (e == hipSuccess) e = hipMalloc((void **)&n->fwd32[l], 4 * (size_t)fwd_rows(l) * fwd_k(l));
        if (e == hipSuccess && l > 0) e = hipMalloc((void **)&n->bwd[l], 2 * (size_t)bwd_rows(l) * bwd_k(l));
        if (e == hipSuccess && l > 0) e = hipMalloc((void **)&n->bwd32[l], 4 * (size_t)bwd_rows(l) * bwd_k(l));
    }
    if (e == hipSuccess) e = prep_tables(n, nullptr);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        sal_net_destroy(n);
        return nfail(nullptr, SAL_E_DEVICE, std::string("net create: ") + hipGetErrorString(e));
    }
    *out = n;
    return SAL_OK;
}

void sal_net_destroy(sal_net *n)
{
    if (!n) return;
    NetDev nd(n->device);
    float *fb[] = {n->p, n->gr, n->m, n->v};
    for (float *b : fb)
        if (b) (void)hipFree(b);
    for (int l = 0; l < NL; ++l) {
        if (n->fwd[l]) (void)hipFree(n->fwd[l]);
        if (n->bwd[l]) (void)hipFree(n->bwd[l]);
        if (n->fwd32[l]) (void)hipFree(n->fwd32[l]);
        if (n->bwd32[l]) (void)hipFree(n->bwd32[l]);
    }
    delete n;
}

sal_status sal_net_set_precision(sal_net *n, int32_t precision)
{
    if (!n) return nfail(n, SAL_E_INVAL, "null argument");
    if (precision != SAL_BF16 && precision != SAL_FP32)
        return nfail(n, SAL_E_INVAL, "the network runs in SAL_BF16 or SAL_FP32");
    n->f32 = precision == SAL_FP32;
    return SAL_OK;
}

sal_status sal_net_params(sal_net *n, float *host, int64_t count, int write)
{
    if (!n || !host) return nfail(n, SAL_E_INVAL, "null argument");
    if (count != n->npar) return nfail(n, SAL_E_INVAL, "parameter count mismatch");
    NetDev nd(n->device);
    hipError_t e;
    if (write) {
        e = hipMemcpy(n->p, host, sizeof(float) * count, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = prep_tables(n, nullptr);
        if (e == hipSuccess) e = hipDeviceSynchronize();
    } else {
        e = hipMemcpy(host, n->p, sizeof(float) * count, hipMemcpyDeviceToHost);
    }
    return e == hipSuccess ? SAL_OK : nfail(n, SAL_E_DEVICE, hipGetErrorString(e));
}

sal_status sal_net_grads(sal_net *n, float *host, int64_t count, int zero)
{
    if (!n || !host) return nfail(n, SAL_E_INVAL, "null argument");
    if (count != n->npar) return nfail(n, SAL_E_INVAL, "parameter count mismatch");
    NetDev nd(n->device);
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipMemcpy(host, n->gr, sizeof(float) * count, hipMemcpyDeviceToHost);
    if (e == hipSuccess && zero) e = hipMemset(n->gr, 0, sizeof(float) * count);
    return e == hipSuccess ? SAL_OK : nfail(n, SAL_E_DEVICE, hipGetErrorString(e));
}

sal_status sal_net_set_output_scale(sal_net *n, const float scale[3])
{
    if (!n || !scale) return nfail(n, SAL_E_INVAL, "null argument");
    for (int c = 0; c < 3; ++c) n->out_scale[c] = scale[c];
    return SAL_OK;
}

sal_status sal_net_workspace_size(sal_net *n, int64_t nb, int64_t n0, int64_t n1, int64_t n2, int train,
                                  size_t *bytes)
{
    if (!n || !bytes || nb < 1 || n0 < 2 || n1 < 2 || n2 < 2) return nfail(n, SAL_E_INVAL, "bad argument");
    const int64_t nv = nvox_of(nb, n0, n1, n2);
    *bytes = train ? train_ws(nv, act_bytes(n)).total : infer_ws(n, nv);
    return SAL_OK;
}

static sal_status check_blocks(sal_net *n, int64_t nb, int64_t n0, int64_t n1, int64_t n2)
{
    if (nb < 1 || n0 < 2 || n1 < 2 || n2 < 2) return nfail(n, SAL_E_INVAL, "every block dimension must be >= 2");
    if (nvox_of(nb, n0, n1, n2) * 24 > ((int64_t)1 << 40)) return nfail(n, SAL_E_INVAL, "too large");
    if (conv_grid(nb, n0, n1, n2) > 0x7fffffffu) return nfail(n, SAL_E_INVAL, "too many tiles");
    return SAL_OK;
}

sal_status sal_net_forward(sal_net *n, const float *X, int64_t nb, int64_t n0, int64_t n1, int64_t n2, float *Y,
                           void *ws, size_t ws_bytes, void *stream)
{
    if (!n || !X || !Y || !ws) return nfail(n, SAL_E_INVAL, "null argument");
    sal_status st = check_blocks(n, nb, n0, n1, n2);
    if (st != SAL_OK) return st;
    const TrainWs tw = train_ws(nvox_of(nb, n0, n1, n2), act_bytes(n));
    if (ws_bytes < tw.total) return nfail(n, SAL_E_WORKSPACE, "workspace too small");
    NetDev nd(n->device);
    hipError_t e = net_forward(n, X, nb, n0, n1, n2, (char *)ws, &tw, Y, 3, 1, make_float3(1.f, 1.f, 1.f),
                               (hipStream_t)stream);
    return e == hipSuccess ? SAL_OK : nfail(n, SAL_E_DEVICE, hipGetErrorString(e));
}

sal_status sal_net_backward(sal_net *n, const float *X, const float *dY, int64_t nb, int64_t n0, int64_t n1,
                            int64_t n2, void *ws, size_t ws_bytes, void *stream)
{
    if (!n || !X || !dY || !ws) return nfail(n, SAL_E_INVAL, "null argument");
    sal_status st = check_blocks(n, nb, n0, n1, n2);
    if (st != SAL_OK) return st;
    const int64_t nv = nvox_of(nb, n0, n1, n2);
    const TrainWs tw = train_ws(nv, act_bytes(n));
    if (ws_bytes < tw.total) return nfail(n, SAL_E_WORKSPACE, "workspace too small");
    NetDev nd(n->device);
    hipStream_t s = (hipStream_t)stream;
    char *w = (char *)ws;
    const void *dYa = dY;  // the FP32-operand mode reads the caller's FP32 gradient directly
    if (!n->f32) {
        hipLaunchKernelGGL(k_f32_to_bf16, dim3((unsigned)((nv * 3 + 255) / 256)), dim3(256), 0, s, dY, nv * 3,
                           (uint16_t *)(w + tw.dy));
        dYa = w + tw.dy;
    }
    hipError_t e = net_backward(n, X, dYa, nb, n0, n1, n2, w, tw, s);
    return e == hipSuccess ? SAL_OK : nfail(n, SAL_E_DEVICE, hipGetErrorString(e));
}

sal_status sal_net_adam(sal_net *n, float lr, void *stream)
{
    if (!n) return nfail(n, SAL_E_INVAL, "null argument");
    if (!(lr >= 0.f)) return nfail(n, SAL_E_INVAL, "lr must be >= 0");
    NetDev nd(n->device);
    hipError_t e = adam_step(n, lr, (hipStream_t)stream);
    return e == hipSuccess ? SAL_OK : nfail(n, SAL_E_DEVICE, hipGetErrorString(e));
}

sal_status sal_net_train_step(sal_net *n, const float *X, const float *T, int64_t nb, int64_t S, int32_t margin,
                              float lr, float *loss_out, void *ws, size_t ws_bytes, void *stream)
{
    if (!n || !X || !T || !ws) return nfail(n, SAL_E_INVAL, "null argument");
    if (margin < NL || 2 * margin >= S) return nfail(n, SAL_E_INVAL, "margin must be >= 5 and < S/2");
    if (!(lr >= 0.f)) return nfail(n, SAL_E_INVAL, "lr must be >= 0");
    sal_status st = check_blocks(n, nb, S, S, S);
    if (st != SAL_OK) return st;
    const int64_t nv = nvox_of(nb, S, S, S);
    const TrainWs tw = train_ws(nv, act_bytes(n));
    if (ws_bytes < tw.total) return nfail(n, SAL_E_WORKSPACE, "workspace too small");
    NetDev nd(n->device);
    hipStream_t s = (hipStream_t)stream;
    char *w = (char *)ws;
    float *Y = (float *)(w + tw.y);
    hipError_t e = net_forward(n, X, nb, S, S, S, w, &tw, Y, 3, 1, make_float3(1.f, 1.f, 1.f), s);
    const int64_t inner = S - 2 * margin;
    const float inv = 1.0f / (float)(nb * inner * inner * inner * 3);
    const unsigned nblk = (unsigned)((nv + 255) / 256);
    if (n->f32)
        hipLaunchKernelGGL(k_mse<true>, dim3(nblk), dim3(256), 0, s, Y, T, (int)nb, (int)S, margin, inv,
                           (float *)(w + tw.dy), (float *)(w + tw.lossp));
    else
        hipLaunchKernelGGL(k_mse<false>, dim3(nblk), dim3(256), 0, s, Y, T, (int)nb, (int)S, margin, inv,
                           (uint16_t *)(w + tw.dy), (float *)(w + tw.lossp));
    if (loss_out)
        hipLaunchKernelGGL(k_sum_loss, dim3(1), dim3(256), 0, s, (const float *)(w + tw.lossp), (int)nblk, loss_out);
    if (e == hipSuccess) e = net_backward(n, X, w + tw.dy, nb, S, S, S, w, tw, s);
    if (e == hipSuccess) e = adam_step(n, lr, s);
    if (e == hipSuccess) e = hipGetLastError();
    return e == hipSuccess ? SAL_OK : nfail(n, SAL_E_DEVICE, hipGetErrorString(e));
}

// Inference over a whole volume: raw maps [3][n0][n1][n2] in the units of the training
// targets times out_scale.
sal_status sal_net_infer(sal_net *n, const float *V, int64_t n0, int64_t n1, int64_t n2, float *S_raw, void *ws,
                         size_t ws_bytes, void *stream)
{
    if (!n || !V || !S_raw || !ws) return nfail(n, SAL_E_INVAL, "null argument");
    sal_status st = check_blocks(n, 1, n0, n1, n2);
    if (st != SAL_OK) return st;
    const int64_t nv = nvox_of(1, n0, n1, n2);
    if (ws_bytes < infer_ws(n, nv)) return nfail(n, SAL_E_WORKSPACE, "workspace too small");
    NetDev nd(n->device);
    hipError_t e = net_forward(n, V, 1, n0, n1, n2, (char *)ws, nullptr, S_raw, 1, nv,
                               make_float3(n->out_scale[0], n->out_scale[1], n->out_scale[2]), (hipStream_t)stream);
    return e == hipSuccess ? SAL_OK : nfail(n, SAL_E_DEVICE, hipGetErrorString(e));
}

}  // extern "C"
