// Steps 1-3 at cube L = 8 and 16 in FP32 with the window sliding along t (Sec. 2 steps 1-3),
// for windows at every voxel (stride S = 1) or on the lattice of a stride S below L/2.
//
// The L^3 DFT of the window centred on (t0, x0, y0) factors into a 2-D DFT of each of its
// L t-planes (x then y) followed by the DFT along t of those plane spectra.  With the
// t-phase taken from the absolute row index v (a unit-modulus factor per window and
// frequency, which the magnitudes of Eqs. (1)-(4) do not see),
//     D_t0[kt, kx, ky] = sum_{v = t0-L/2}^{t0+L/2-1} P_v[kx, ky] e^{-2 pi i kt v / L},
// and since e^{-2 pi i kt (v + L) / L} = e^{-2 pi i kt v / L}, the next window's spectrum
// is this one's plus (P_{v_in} - P_{v_out}) e^{-2 pi i kt v_in / L}, where the plane
// leaving (v_out = v_in - L) and the plane entering share the twiddle.  By linearity
// P_{v_in} - P_{v_out} is the 2-D DFT of the plane difference V[v_in] - V[v_out], so each
// window costs one 2-D plane DFT (matrix cores) and one complex multiply-add per bin (vector
// ALUs) instead of a full DFT along t.  Rows are reflected at the t faces exactly as the
// window's own rows are.
//
// Each product is rounded before it is added, so a plane that enters and later leaves
// cancels exactly (a unit spike leaves exact zeros behind).  The running sums restart from
// zero at fixed absolute rows (window t0 = 0, L/2, 512, 1024, ...; restarting at t0 = L/2
// keeps the rows reflected at the t = 0 face out of every later window's history), so a
// window's result does not depend on the box or batch it is computed in, and the rounding
// drift of the sums stays within 527 steps.
//
// Workgroup: one x0, 16 y0 S apart, one t segment; L/2 waves, wave c owning column c of
// the 2-D plane spectrum (c = 1..L/2-1: the x frequency kx = c; c = 0: kx = 0 and kx = L/2
// packed as one complex column Z = X_0 + i X_{L/2} of two real sequences).  Per t-step:
//   stage 1 (waves 1 .. L/2 - 1, 16 positions at a time): X[comp, y] =
//     sum_tau M1[comp, tau] dV[x0 - L/2 + tau, y] for the PY = 15 S + L positions y of the
//     tile, the real DFT along x packed into L real components;
//   stage 2 (wave c): P[ky, y0] = sum_tau W[ky, tau] X_c[y0 - L/2 + tau], complex, L ky on
//     L/8 M tiles whose lane groups hold ky and -ky, the 16 windows on N;
//   stage 3 (wave c): the lane's 4L bins (M tiles x two ky x L kt) of its window take their
//     update; at output steps (every S-th window along t) their magnitudes are weighted into
//     E_t, E_x, E_y.
// With S > 1 every row still enters and leaves (the sums slide one row per step), while the
// workgroups, the y positions and the magnitudes are those of the lattice windows only.  At cube
// 16 stage 2 is then a larger part of the step and takes ky and -ky together: the cosine and sine
// sums of both parts (16 rows for 16 ky, half the MFMAs) and eight additions.  Energies of stride 4
// on 512^3 4.38 -> 3.74 ms.  RMS error against FP64, of one sum per row of P: E 5.9e-8 to 8.8e-8, at
// strides 2 to 7 over 12 small volumes each 0.997 to 1.005 times that, on 200 x 256 x 190 to 512^3
// 0.995 to 0.997 times; S over 72 volumes 1.00 +- 0.02 times (of one volume 0.65 to 1.55: its scale
// hangs on the errors of six extreme voxels).  S = 1 keeps one sum per row and its bits.
// In wave 0 the bins (kt, ky) and (-kt, -ky) of the packed column sit in one lane; its
// update is applied to U = Z[k] + conj Z[-k] = 2 D_{kx=0}[k] and V = Z[k] - conj Z[-k] =
// 2i D_{kx=L/2}[k] instead (the plane spectra transformed the same way), so every slot is one
// bin's magnitude.  On the self-conjugate rows ky in {0, L/2} the slots kt and L - kt hold U
// and conj V, and kt in {0, L/2} hold Z itself, whose real and imaginary parts are two
// self-conjugate bins.
//
// The update's products.  The kernel is bound by vector issue, and a twiddle multiplication
// per bin was its largest part.  The t loop is unrolled by four, so the row index v = 4 q + r
// has a compile-time r, and e^{-2 pi i kt v / L} splits into quarter turns (swaps and signs)
// and a few constants.  Cube 16, kt = 4 a + b:
//     w^{kt v} = (-i)^{a r} * { 1, (-i)^q w^r, (-1)^q w^{2r}, (-1)^q (-i)^q w^{3r} }[b],
// so the 16 products of one plane bin are quarter turns of four, whose real and imaginary
// parts are x c +- y s over two multiplications for w and w^3 and one for w^2.  Cube 8,
// kt = 2 a + b: w^{kt v} = (-i)^{a r} { 1, (-1)^q w^r }[b].  The swap of (-i)^q selects
// between the two parts after the rounding, and its signs enter as the exact factors of the
// fused multiply-adds into the running sums, so every sum is bit for bit that of one rounded
// product per bin.  Per plane bin: 8 instructions (cube 16) and 2 (cube 8) beside the 2 L
// additions, 42 and 18 with a twiddle per bin.  Whole pass, twiddle per bin -> this: 106.4 ->
// 84.3 ms at cube 16 on 512^3 voxels, 7.33 -> 6.09 ms at cube 8 on 256 x 512 x 512, 6.9 ->
// 5.85 ms at cube 16 and stride 4 on 512^3.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "sal_device.h"
#include "sal_internal.h"

namespace {

constexpr int STY = 16;  // windows along y per workgroup

template <int L, int S>
struct SlideGeo {
    static constexpr int H = L / 2;            // window start = centre - H
    static constexpr int PY = S * (STY - 1) + L;  // stage-1 positions along y
    static constexpr int PLS = (PY + 15) / 32 * 32 + 16;  // plane row stride: tau rows 16 banks apart
    static constexpr int NW = L / 2;           // waves = packed columns of the x spectrum
    static constexpr int MT = L / 8;           // M tiles of the y contraction
    static constexpr int S1S = L + 2;          // stage-1 output row stride (floats)
    static constexpr int KS1 = L / 4;          // K steps of the x contraction
    static constexpr int KS2 = L / 2;          // K steps of the y contraction
    static constexpr int NP = L / 2 + 1;       // |kt| values
    static constexpr int SWP = slide_weights_per_group(L);
    static constexpr int NS1 = (PY + 15) / 16;  // stage-1 blocks of 16 positions
    static constexpr int NLD = (L * PY + 64 * NW - 1) / (64 * NW);  // plane samples per thread
    static constexpr int RW = NS1 + 1 < NW ? NS1 + 1 : NW - 1;       // the wave storing E
    static constexpr bool PAIR_Y = L == 16 && S > 1;                 // stage 2 in conjugate pairs
    static constexpr int NA2 = PAIR_Y ? 1 : MT * KS2 / 4;            // its operands, by four K steps
    static_assert(16 * NS1 <= PLS && 2 * S < L, "tile geometry");
};

__device__ __forceinline__ float mag(float re, float im) { return __builtin_amdgcn_sqrtf(fmaf(re, re, im * im)); }

// (x, y) as a complex number times (-i)^K
template <int K>
__device__ __forceinline__ float2 quarter(float2 p)
{
    if constexpr ((K & 3) == 0) return p;
    if constexpr ((K & 3) == 1) return make_float2(p.y, -p.x);
    if constexpr ((K & 3) == 2) return make_float2(-p.x, -p.y);
    return make_float2(-p.y, p.x);
}

// Quarter-turn state of the row v = 4 q + r: whether (-i)^q swaps the parts, the signs it
// gives them (sx, sy), (-1)^q = s1, and the signs of (-1)^q (-i)^q (tx, ty)
struct qturn {
    bool odd;
    float sx, sy, s1, tx, ty;
};
__device__ __forceinline__ qturn make_qturn(int q)
{
    const float m = -1.f, p = 1.f;
    return {(q & 1) != 0,           (q & 2) ? m : p,       ((q + 1) & 2) ? m : p,
            (q & 1) ? m : p,        ((q + 1) & 2) ? m : p, (q & 2) ? m : p};
}

// p w^{kt v} without the quarter turns (-i)^{a r} and the signs of take(): Q[b] of the header
// comment with the parts already swapped
template <int L, int R>
__device__ __forceinline__ void products(float2 p, const qturn &t, float2 (&Q)[L == 16 ? 4 : 2])
{
    constexpr float C8 = 0.92387953251128674f, S8 = 0.38268343236508977f, H = 0.70710678118654752f;
    Q[0] = p;
    const float a = p.y * H;
    const float2 p2 = make_float2(fmaf(p.x, H, a), fmaf(-p.x, H, a));  // p (1 - i) / sqrt 2
    if constexpr (L == 16) {
        auto swap = [&](float2 z) { return t.odd ? make_float2(z.y, z.x) : z; };
        if constexpr (R == 0) {
            Q[2] = p;
            Q[1] = Q[3] = swap(p);
        } else if constexpr (R == 2) {
            Q[1] = swap(p2);
            Q[2] = quarter<1>(p);             // w^4 = -i
            Q[3] = swap(quarter<1>(p2));      // w^6 = -i w^2
        } else {
            const float yc = p.y * C8, ys = p.y * S8;
            const float2 z1 = make_float2(fmaf(p.x, C8, ys), fmaf(-p.x, S8, yc));  // p w
            const float2 z3 = make_float2(fmaf(p.x, S8, yc), fmaf(-p.x, C8, ys));  // p w^3
            Q[1] = swap(R == 1 ? z1 : z3);
            Q[2] = R == 1 ? p2 : quarter<1>(p2);
            Q[3] = swap(R == 1 ? z3 : quarter<2>(z1));  // w^9 = -w
        }
    } else {
        if constexpr (R & 1)
            Q[1] = R == 1 ? p2 : quarter<1>(p2);  // w^3 = -i w
        else
            Q[1] = quarter<R / 2>(p);             // w^2 = -i
    }
}

// (x, y) in the order of a quarter turn by K, and the signs it gives them
template <int K>
struct turn {
    static constexpr bool SWAP = (K & 1) != 0;
    static constexpr float X = (K & 2) ? -1.f : 1.f, Y = ((K + 1) & 2) ? -1.f : 1.f;
};

// D += p w^{kt v} for the slot kt = KT, from products(); the factors are +-1, so the product
// rounded there is added exactly as it is
template <int L, int R, int KT>
__device__ __forceinline__ void take(float &dr, float &di, const float2 (&Q)[L == 16 ? 4 : 2], const qturn &t)
{
    constexpr int NB = L == 16 ? 4 : 2, A = KT / NB, B = KT % NB;
    using T = turn<(A * R) & 3>;
    const float2 q = Q[B];
    float gx = 1.f, gy = 1.f;
    if constexpr (L == 16 && B == 1) { gx = t.sx; gy = t.sy; }
    if constexpr (L == 16 && B == 3) { gx = t.tx; gy = t.ty; }
    if constexpr (L == 16 ? B == 2 : B == 1) gx = gy = t.s1;
    dr = fmaf(T::X * (T::SWAP ? gy : gx), T::SWAP ? q.y : q.x, dr);
    di = fmaf(T::Y * (T::SWAP ? gx : gy), T::SWAP ? q.x : q.y, di);
}
template <int L, int R, int LO, int HI>
__device__ __forceinline__ void take_range(float *dr, float *di, const float2 (&Q)[L == 16 ? 4 : 2], const qturn &t)
{
    if constexpr (LO < HI) {
        take<L, R, LO>(dr[LO], di[LO], Q, t);
        take_range<L, R, LO + 1, HI>(dr, di, Q, t);
    }
}

// Sums of e[0..2] over the four lane groups, (0 + 1) + (2 + 3): lane group m returns e[m]'s
// (three lane swaps and three adds; lane group 3 repeats e[2]'s).
__device__ __forceinline__ float group_sums(const float (&e)[3])
{
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(e[0]), __float_as_uint(e[1]), false, false);
    const auto c = __builtin_amdgcn_permlane16_swap(__float_as_uint(e[2]), __float_as_uint(e[2]), false, false);
    const float s01 = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const float s2 = __uint_as_float(c[0]) + __uint_as_float(c[1]);
    const auto d = __builtin_amdgcn_permlane32_swap(__float_as_uint(s01), __float_as_uint(s2), false, false);
    return __uint_as_float(d[0]) + __uint_as_float(d[1]);
}

}  // namespace

template <int L, int S>
__global__ __attribute__((amdgpu_waves_per_eu(2))) __launch_bounds__(64 * (L / 2)) void k_energy_slide(
    const float *__restrict__ V, int n0, int n1, int n2, ebox bx, int nseg, int np, int nbx, int nby,
    const float *__restrict__ w_s1, const float *__restrict__ w_s2, const float *__restrict__ w_sp,
    float *__restrict__ E, float *__restrict__ vmax_part)
{
    using G = SlideGeo<L, S>;
    constexpr int SL = L, SH = G::H, SPY = G::PY, SNW = G::NW, MT = G::MT, S1S = G::S1S;
    constexpr int KS1 = G::KS1, KS2 = G::KS2, NP = G::NP, SWP = G::SWP, NS1 = G::NS1, NLD = G::NLD;
    constexpr int RW = G::RW, PLS = G::PLS;
    __shared__ float plane_s[2][SL * PLS];
    __shared__ float s1_s[2][SPY * S1S + 2];
    __shared__ float wt_s[SNW * 4 * SWP];
    __shared__ float red_s[2][SNW][64];
    __shared__ float vred_s[SNW];
    // constant A operands, per lane: stage 1 [lane][K step], stage 2 [K step / 4][lane][4]
    __shared__ float4 a1_s[64];
    __shared__ float4 a2_s[G::NA2][64];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, n = lane & 15;

    // Column (x0, y tile) and t segment of this workgroup.  x0 fastest: the workgroups of
    // neighbouring x0 (L - 1 of their L plane rows shared) run together on one XCD and meet
    // the rows in its L2.  One box: every XCD takes a contiguous range of columns and walks it
    // once per segment, the first segment of the box (L/2 windows when it is the volume's)
    // last, so every XCD holds the same mix and the short walks fill the ends of the long
    // ones.  At cube 16 on 64^3 (256 columns, one workgroup per CU) the tiles in one range,
    // segment inside, put the long walks of a y tile on one XCD, two after each other on a CU:
    // 362 us for the pass, 240 us in this order.
    int box = 0, col, kr;
    const int ncol = nbx * nby;
    if (bx.table) {
        const int tile = box_tile(bx, &box);
        kr = (tile / nbx) % (nseg * np);
        col = tile / (nbx * nseg * np) * nbx + tile % nbx;
    } else {
        const int per = (ncol + 7) >> 3, i = blockIdx.x >> 3;
        kr = i / per;
        col = (blockIdx.x & 7) * per + (i - kr * per);
        if (col >= ncol) return;
        kr = kr + np < nseg * np ? kr + np : kr + np - nseg * np;
    }
    // part kp of the np parts of the segment's windows: the later ones repeat the updates of the
    // earlier ones without their magnitudes
    const int kp = kr % np;
    kr /= np;
    V += box * bx.vstride;
    E += box * bx.estride;
    const int xr = col % nbx, ty = col / nbx;
    const int y_base = bx.o2 + S * STY * ty, x0 = bx.o1 + S * xr;
    const int k = slide_seg_id(bx.o0, SH) + kr;
    const int s_start = slide_seg_start(k, SH);
    const int w_lo = max(s_start, bx.o0), w_hi = min(slide_seg_start(k + 1, SH), min(n0, bx.o0 + bx.d0));
    const int w_per = ((w_hi - w_lo + np - 1) / np + S - 1) / S * S;
    const int t_lo = w_lo + kp * w_per, t_hi = min(w_hi, t_lo + w_per);
    float *const vmax_out = vmax_part ? vmax_part + (kr * np + kp) * ncol + col : nullptr;
    if (kr >= nseg || t_lo >= t_hi || x0 >= bx.o1 + bx.d1 || y_base >= bx.o2 + bx.d2) {
        if (threadIdx.x == 0 && vmax_out) *vmax_out = 0.f;
        return;
    }
    const int K1 = bx.fk1, K2 = bx.fk2;
    const int64_t nbox = (int64_t)bx.fk0 * K1 * K2;
    const int y_end = bx.o2 + bx.d2;

    for (int i = threadIdx.x; i < SNW * 4 * SWP; i += 64 * SNW) wt_s[i] = w_sp[i];
    // (at cube 16 the 16 stage-2 operands would not fit the registers beside the 128 of the
    // spectra)
    if (threadIdx.x < 64) {
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
        a.x = w_s1[lane];
        a.y = w_s1[64 + lane];
        if (KS1 > 2) {
            a.z = w_s1[128 + lane];
            a.w = w_s1[192 + lane];
        }
        a1_s[lane] = a;
    }
    if constexpr (G::PAIR_Y) {
        // rows 4 q .. 4 q + 3: cos and sin of M tile 0's ky of lane group q (of ky = 0 and 8 the
        // cosines), then of M tile 1's; K step t has the taps 4 t .. 4 t + 3
        if (threadIdx.x < 64) {
            const int j = n & 3, row = n == 1 ? 2 : n & 12, mt = j >> 1, im = n == 1 ? 0 : j & 1;
            const float *w = w_s2 + (mt * KS2 + im) * 64 + (g << 4) + row;
            a2_s[0][lane] = make_float4(w[0], w[2 * 64], w[4 * 64], w[6 * 64]);
        }
    } else
    for (int i = threadIdx.x; i < MT * KS2 * 16; i += 64 * SNW) {
        const int r = i >> 6, ln = i & 63;  // operands 4 r .. 4 r + 3 in the order (mt, kk)
        float4 a;
        a.x = w_s2[(4 * r) * 64 + ln];
        a.y = w_s2[(4 * r + 1) * 64 + ln];
        a.z = w_s2[(4 * r + 2) * 64 + ln];
        a.w = w_s2[(4 * r + 3) * 64 + ln];
        a2_s[r][ln] = a;
    }

    // plane samples: sample i = threadIdx.x + 64 NW l < L PY (slot l of the thread) is
    // (tau, yy) = (i / PY, i % PY)
    const int n12 = n1 * n2;  // the volume holds at most 2^31 - 1 samples
    bool loader[NLD];
    int off[NLD], pidx[NLD];
#pragma unroll
    for (int l = 0; l < NLD; ++l) {
        const int i = threadIdx.x + 64 * SNW * l;
        loader[l] = i < SL * SPY;
        off[l] = pidx[l] = 0;
        if (loader[l]) {
            const int tau = i / SPY, yy = i - tau * SPY;
            off[l] = refl_idx(x0 - SH + tau, n1) * n2 + refl_idx(y_base - SH + yy, n2);
            pidx[l] = tau * PLS + yy;
        }
    }
    // step j brings row v_in = s_start - L/2 + j in and, from j = L on, takes v_in - L out;
    // the window t0 = s_start + j - (L - 1) is complete after step j
    const int nsteps = t_hi - s_start + SL - 1;
    float vmax = 0.f;
    // the samples of step j are loaded two steps ahead and only read when the plane is
    // written to LDS, so the loads' latency overlaps a whole step
    float ra[NLD], rb[NLD];
#pragma unroll
    for (int l = 0; l < NLD; ++l) ra[l] = rb[l] = 0.f;
    auto load_plane = [&](int j) {
        const int vin = s_start - SH + j;
        const int r_in = refl_idx(vin, n0) * n12, r_out = refl_idx(vin - SL, n0) * n12;
#pragma unroll
        for (int l = 0; l < NLD; ++l)
            if (loader[l]) {
                ra[l] = V[(uint32_t)(r_in + off[l])];
                rb[l] = V[(uint32_t)(r_out + off[l])];  // in the volume; unused before j = L
            }
    };
    // the plane difference of step j into LDS buffer buf
    auto store_plane = [&](int j, int buf) {
#pragma unroll
        for (int l = 0; l < NLD; ++l)
            if (loader[l]) {
                vmax = fmaxf(vmax, fmaxf(fabsf(ra[l]), fabsf(rb[l])));
                plane_s[buf][pidx[l]] = j >= SL ? ra[l] - rb[l] : ra[l];
            }
    };
    auto stage1 = [&](int buf) {
        // waves 1 .. L/2 - 1: positions 16 jt + n for jt = wave - 1, wave - 1 + L/2 - 1, ...
        const float4 a1 = a1_s[lane];
        for (int jt = wave - 1; jt < NS1; jt += SNW - 1) {
            f4 acc = f4{0.f, 0.f, 0.f, 0.f};
            const float *pl = plane_s[buf] + 16 * jt + n;
            acc = mfma4(a1.x, pl[g * PLS], acc);
            acc = mfma4(a1.y, pl[(4 + g) * PLS], acc);
            if (KS1 > 2) {
                acc = mfma4(a1.z, pl[(8 + g) * PLS], acc);
                acc = mfma4(a1.w, pl[(12 + g) * PLS], acc);
            }
            const int yy = 16 * jt + n;
            if (yy < SPY && 4 * g < SL) {
                float *o = s1_s[buf] + yy * S1S + 4 * g;
                *reinterpret_cast<float2 *>(o) = make_float2(acc[0], acc[1]);
                *reinterpret_cast<float2 *>(o + 2) = make_float2(acc[2], acc[3]);
            }
        }
    };

    // E of the window completed at step jo (red_s[buf]), summed over the waves in a fixed
    // order, at the lattice windows of the box
    const int ry = y_base + S * n;  // y of this lane's sums, their component is g
    float *const E_lane = E + g * nbox + (int64_t)((x0 - bx.fo1) / S) * K2 + (ry - bx.fo2) / S;
    const int64_t K12 = (int64_t)K1 * K2;
    auto store_energies = [&](int jo, int buf) __attribute__((always_inline)) {
        const int t0 = s_start + jo - (SL - 1);
        if (t0 < t_lo || (t0 - bx.o0) % S != 0) return;
        float e = red_s[buf][0][lane];
#pragma unroll
        for (int w = 1; w < SNW; ++w) e += red_s[buf][w][lane];
        if (g < 3 && ry < y_end) E_lane[(t0 - bx.fo0) / S * K12] = e;
    };

    load_plane(0);
    store_plane(0, 0);
    __syncthreads();
    if (wave >= 1) stage1(0);
    if (nsteps > 1) load_plane(1);

    // spectrum state: [M tile][ky slot][kt]
    float Dr[MT][2][SL], Di[MT][2][SL];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int kt = 0; kt < SL; ++kt) Dr[mt][q][kt] = Di[mt][q][kt] = 0.f;

    const float *wl = wt_s + (wave * 4 + g) * SWP;
    const bool sp_lane = g == 0;  // wave 0: lane group holding the self-conjugate rows 0, L/2

    // step j = 4 i + R
    auto step = [&](auto rc, int j) __attribute__((always_inline)) {
        constexpr int R = decltype(rc)::value, b = R & 1;
        if (j + 1 < nsteps) store_plane(j + 1, b ^ 1);
        __syncthreads();
        if (j + 2 < nsteps) load_plane(j + 2);
        // the previous step's energies: sum over the waves in a fixed order
        if (wave == RW && j >= SL) store_energies(j - 1, b ^ 1);

        // ---------------- stage 2: DFT along y of column c = wave -----------------------
        f4 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = f4{0.f, 0.f, 0.f, 0.f};
        if constexpr (G::PAIR_Y) {
            // cosine and sine sums of both parts, X of Re and Y of Im: P[+-ky] = (Cx +- Sy, Cy -+ Sx)
            const float *src = s1_s[b] + (S * n + g) * S1S + 2 * wave;
            const float4 w = a2_s[0][lane];
            f4 X = f4{0.f, 0.f, 0.f, 0.f}, Y = X;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float2 x = *reinterpret_cast<const float2 *>(src + 4 * t * S1S);
                const float wt = t == 0 ? w.x : (t == 1 ? w.y : (t == 2 ? w.z : w.w));
                X = mfma4(wt, x.x, X);
                Y = mfma4(wt, x.y, Y);
            }
            acc[0] = sp_lane ? f4{X[0], Y[0], X[1], Y[1]}
                             : f4{X[0] + Y[1], Y[0] - X[1], X[0] - Y[1], Y[0] + X[1]};
            acc[MT - 1] = f4{X[2] + Y[3], Y[2] - X[3], X[2] - Y[3], Y[2] + X[3]};
        } else {
            const float *src = s1_s[b] + (S * n + g) * S1S + 2 * wave;
#pragma unroll
            for (int kh = 0; kh < KS2 / 4; ++kh) {
                // operands (mt, kk) for kk = 4 kh .. 4 kh + 3
                float4 wm[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) wm[mt] = a2_s[mt * (KS2 / 4) + kh][lane];
                const float2 x0 = *reinterpret_cast<const float2 *>(src + 8 * kh * S1S);
                const float2 x1 = *reinterpret_cast<const float2 *>(src + (8 * kh + 4) * S1S);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[mt] = mfma4(wm[mt].x, x0.x, acc[mt]);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[mt] = mfma4(wm[mt].y, x0.y, acc[mt]);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[mt] = mfma4(wm[mt].z, x1.x, acc[mt]);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[mt] = mfma4(wm[mt].w, x1.y, acc[mt]);
            }
        }

        // stage 1 of the next step behind this step's stage 2: in front of it, the waves that take it
        // kept the others waiting (512^3 at cube 16 84.2 ms in front, 83.0 behind)
        if (wave >= 1 && j + 1 < nsteps) stage1(b ^ 1);
        // ---------------- stage 3: the t update -----------------------------------------
        // row v = s_start - L/2 + j = 4 q + R (segment starts and L/2 are multiples of four)
        const qturn qt = make_qturn((s_start - SH + j) >> 2);
        const int t0 = s_start + j - (SL - 1);
        const bool out = j >= SL - 1 && t0 >= t_lo && (t0 - bx.o0) % S == 0;
        using QA = float2[SL == 16 ? 4 : 2];
        // Slot inputs.  Columns 1..L/2-1: the plane spectrum itself.  Column 0: U = P_a +
        // conj P_b and V = P_a - conj P_b for the rows (a, b = -a); on the self-conjugate rows
        // (lane group 0 of M tile 0) Z itself at kt in {0, L/2}, 2 Re Z at kt = 1..L/2-1 (U)
        // and -2i Im Z at kt = L/2+1..L-1 (conj V).
        float2 p[MT][2];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const float2 pa = make_float2(acc[mt][0], acc[mt][1]), pb = make_float2(acc[mt][2], acc[mt][3]);
            p[mt][0] = pa;
            p[mt][1] = pb;
            if (wave == 0 && (mt > 0 || !sp_lane)) {
                p[mt][0] = make_float2(pa.x + pb.x, pa.y - pb.y);
                p[mt][1] = make_float2(pa.x - pb.x, pa.y + pb.y);
            }
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float *dr = Dr[mt][q], *di = Di[mt][q];
                const float2 z = p[mt][q];
                QA Q;
                products<SL, R>(z, qt, Q);
                if (mt == 0 && wave == 0) {
                    QA Ql, Qh;
                    products<SL, R>(sp_lane ? make_float2(2.f * z.x, 0.f) : z, qt, Ql);
                    products<SL, R>(sp_lane ? make_float2(0.f, -2.f * z.y) : z, qt, Qh);
                    take<SL, R, 0>(dr[0], di[0], Q, qt);
                    take_range<SL, R, 1, SH>(dr, di, Ql, qt);
                    take<SL, R, SH>(dr[SH], di[SH], Q, qt);
                    take_range<SL, R, SH + 1, SL>(dr, di, Qh, qt);
                } else {
                    take_range<SL, R, 0, SL>(dr, di, Q, qt);
                }
            }
        float e[3] = {0.f, 0.f, 0.f};
        if (out && wave != 0) {
            // M tile 0: the ky of the two slots differ in lane group 0 (0 and L/2): a weight
            // set per slot; M tile 1: ky and -ky, one set.  kt and L - kt share weights.
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                float m0[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    m0[q] = mag(Dr[0][q][p], Di[0][q][p]);
                    if (p > 0 && p < SH) m0[q] += mag(Dr[0][q][SL - p], Di[0][q][SL - p]);
                }
#pragma unroll
                for (int m = 0; m < 3; ++m)
                    e[m] = fmaf(wl[3 * NP + 3 * p + m], m0[1], fmaf(wl[3 * p + m], m0[0], e[m]));
#pragma unroll
                for (int mt = 1; mt < MT; ++mt) {
                    float m1 = mag(Dr[mt][0][p], Di[mt][0][p]) + mag(Dr[mt][1][p], Di[mt][1][p]);
                    if (p > 0 && p < SH)
                        m1 += mag(Dr[mt][0][SL - p], Di[mt][0][SL - p]) + mag(Dr[mt][1][SL - p], Di[mt][1][SL - p]);
#pragma unroll
                    for (int m = 0; m < 3; ++m) e[m] = fmaf(wl[6 * NP + 3 * p + m], m1, e[m]);
                }
            }
        } else if (out) {
            // M tile 0: weights A (slot kt) and B (slot L - kt) per ky slot; at kt in {0, L/2}
            // A weighs |Re Z| and B |Im Z| on the self-conjugate rows, A the magnitude
            // elsewhere.  M tile 1: one set per ky slot.
            const float sel = sp_lane ? 0.f : 1.f;
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    float ma, mb;
                    if (p == 0 || p == SH) {
                        const float re = Dr[0][q][p], im = Di[0][q][p];
                        ma = __builtin_amdgcn_sqrtf(fmaf(re, re, sel * im * im));
                        mb = fabsf(im);
                    } else {
                        ma = mag(Dr[0][q][p], Di[0][q][p]);
                        mb = mag(Dr[0][q][SL - p], Di[0][q][SL - p]);
                    }
                    const float *wa = wl + (q * NP + p) * 6;
#pragma unroll
                    for (int m = 0; m < 3; ++m) e[m] = fmaf(wa[3 + m], mb, fmaf(wa[m], ma, e[m]));
#pragma unroll
                    for (int mt = 1; mt < MT; ++mt) {
                        float m1 = mag(Dr[mt][q][p], Di[mt][q][p]);
                        if (p > 0 && p < SH) m1 += mag(Dr[mt][q][SL - p], Di[mt][q][SL - p]);
                        const float *wm = wl + 12 * NP + (q * NP + p) * 3;
#pragma unroll
                        for (int m = 0; m < 3; ++m) e[m] = fmaf(wm[m], m1, e[m]);
                    }
                }
        }
        // lanes n, n + 16, n + 32, n + 48 hold the same window
        if (out) red_s[b][wave][lane] = group_sums(e);
    };
#pragma unroll 1
    for (int j = 0; j < nsteps; j += 4) {
        step(std::integral_constant<int, 0>{}, j);
        if (j + 1 < nsteps) step(std::integral_constant<int, 1>{}, j + 1);
        if (j + 2 < nsteps) step(std::integral_constant<int, 2>{}, j + 2);
        if (j + 3 < nsteps) step(std::integral_constant<int, 3>{}, j + 3);
    }
    __syncthreads();
    if (wave == RW) store_energies(nsteps - 1, (nsteps - 1) & 1);
    // max |V| of everything this workgroup read (all of it lies in the volume)
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) vmax = fmaxf(vmax, __shfl_xor(vmax, o));
    if (lane == 0) vred_s[wave] = vmax;
    __syncthreads();
    if (threadIdx.x == 0 && vmax_out) {
        float m = vred_s[0];
        for (int w = 1; w < SNW; ++w) m = fmaxf(m, vred_s[w]);
        *vmax_out = m;
    }
}

// ====================================================================== launcher

// Segments of the t walk (window rows [slide_seg_start(k), slide_seg_start(k + 1)))
// touched by the box rows [o0, o0 + d0); the grid covers the most any box of the batch needs.
static int slide_nseg(int o0, int d0, int r) { return slide_seg_id(o0 + d0 - 1, r) - slide_seg_id(o0, r) + 1; }

// Parts a segment's windows are split into: one, doubled up to eight while the chip would not get
// two workgroups per CU at cube 8 (one at cube 16: eight waves of 256 registers) and the box has at
// least eight rows of t for each part.  The rows are the box's: a segment that holds fewer (the first
// has L/2 windows), or a stride S, leaves parts with fewer windows, down to none, which leave at once.
// Each part repeats the earlier ones' updates, without magnitudes (a third of
// a step's vector work, 0.7 of its time when one workgroup has a CU to itself), so splitting
// only pays in latency, on idle CUs: 32^3 at cube 8 31.4 us in one part, 27.1 in two, 25.6 in
// four; at cube 16 85 -> 73; 128 x 24 x 30 at cube 16 320 -> 244.  The sums are the same chain
// of additions, bit for bit.
static int slide_parts(int L, int64_t nseg, int64_t ncol, int64_t d0)
{
    const int64_t slots = L == 8 ? 512 : 256;
    int np = 1;
    while (np < 8 && 2 * np * nseg * ncol <= slots && d0 >= 16 * np) np *= 2;
    return np;
}

int64_t energy_slide_num_blocks(const sal_ctx *c, int64_t n0, int64_t n1, int64_t n2)
{
    const int64_t S = c->p.stride, k1 = (n1 + S - 1) / S, k2 = (n2 + S - 1) / S;
    const int64_t nseg = slide_nseg(0, (int)n0, c->L / 2), ncol = k1 * ((k2 + STY - 1) / STY);
    return nseg * slide_parts(c->L, nseg, ncol, n0) * ncol;
}

template <int L, int S>
static hipError_t launch_slide_L(const sal_ctx *c, const float *V, int64_t n0, int64_t n1, int64_t n2, ebox bx,
                                 float *E, float *vmax_part, int *nparts, hipStream_t s, int nbox)
{
    int nseg;
    if (bx.table)
        nseg = (bx.d0 + SLIDE_SEG - 1) / SLIDE_SEG + 2;  // any o0
    else
        nseg = slide_nseg(bx.o0, bx.d0, L / 2);
    // lattice windows of the box along x, groups of 16 along y
    const int nbx = (bx.d1 + S - 1) / S, nby = ((bx.d2 + S - 1) / S + STY - 1) / STY;
    const int np = slide_parts(L, nseg, (int64_t)nbx * nby * (bx.table ? nbox : 1), bx.d0);
    int64_t nb = (int64_t)nseg * np * nbx * nby;
    if (nparts) *nparts = (int)nb;  // (a batch takes no partials)
    if (bx.table) {
        bx.per_box = batch_per_box(nb);
        nb = (int64_t)bx.per_box * nbox;
    } else {
        nb = 8 * (((int64_t)nbx * nby + 7) / 8) * nseg * np;  // eight equal column ranges
    }
    hipLaunchKernelGGL((k_energy_slide<L, S>), dim3((unsigned)nb), dim3(64 * (L / 2)), 0, s, V, (int)n0, (int)n1,
                       (int)n2, bx, nseg, np, nbx, nby, c->t.w_s1, c->t.w_s2, c->t.w_sp, E, vmax_part);
    return hipGetLastError();
}

hipError_t launch_energy_slide(const sal_ctx *c, const float *V, int64_t n0, int64_t n1, int64_t n2, ebox bx,
                               float *E, float *vmax_part, int *nparts, hipStream_t s, int nbox)
{
#define SAL_SLIDE(LL, SS) \
    if (c->L == LL && c->p.stride == SS) return launch_slide_L<LL, SS>(c, V, n0, n1, n2, bx, E, vmax_part, nparts, s, nbox)
    SAL_SLIDE(8, 1);
    SAL_SLIDE(8, 2);
    SAL_SLIDE(8, 3);
    SAL_SLIDE(16, 1);
    SAL_SLIDE(16, 2);
    SAL_SLIDE(16, 3);
    SAL_SLIDE(16, 4);
    SAL_SLIDE(16, 5);
    SAL_SLIDE(16, 6);
    SAL_SLIDE(16, 7);
#undef SAL_SLIDE
    return hipErrorInvalidValue;
}
