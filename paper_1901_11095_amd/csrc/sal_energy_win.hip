// Steps 1-3 of the saliency method (Shafiq et al., ICIP 2017, Sec. 2) where the fused kernels'
// sharing of the first two axes between neighbouring windows does not apply or does not fit: the
// local 3D DFT of each window (DFT definition after Eq. (2)), its plane projections with DC
// excluded (Eqs. (1)-(4)) and the mean magnitudes E_t, E_x, E_y.
//   * Cubes 9..15 and 17..20, windows at every voxel or on a lattice of overlapping stride (Sec. 2
//     asks for more than 50 % overlap, s < L/2): runs of windows along y that share the first two
//     stages (k_energy_run), unless the stage outputs of a run of eight leave no room for two
//     workgroups on a CU (the widest strides of the largest cubes).
//   * Everything else window by window, nothing shared (k_energy_win, at cube 16 k_energy_win_mfma):
//     the non-overlapping stride s = L of the predecessor method (Sec. 1), overlapping strides of the
//     other cubes that neither the sliding kernel of cube 8 and 16 nor the vector-ALU kernel of
//     cubes 2..7 takes, and what does not fit a run.  The work falls by s^3 while unshared windows cost
//     2.5 times the shared contraction per window.
// FP32.  Window by window (cube 16 on the matrix cores, the other sides on the vector ALUs) a
// workgroup walks windows, grid-stride over the windows of its box; per window:
//   load    the L^3 samples, reflected at the volume faces, into LDS;
//   stage A per column (q, r): A[mu][q][r] = sum_p W[mu, p] win[p][q][r], mu <= L/2;
//   stage B per (mu, r): B[mu][nu][r] = sum_q W[nu, q] A[mu][q][r], every nu;
//   stage C per row (mu, nu): F[om] = sum_r W[om, r] B[mu][nu][r], |F| weighted by the
//           projections (times the conjugate multiplicity of mu and 1/(L^3 (L^3 - 1))),
//           summed over the workgroup into E_t, E_x, E_y.
// On the vector ALUs every stage takes its L-point DFTs with the terms and outputs in
// conjugate pairs (sal_dft.h).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "sal_device.h"
#include "sal_dft.h"
#include "sal_internal.h"

namespace {

template <int L>
struct WinCfg {
    static constexpr int h = L / 2 + 1;
    static constexpr int NT = 64 * ((h * L + 63) / 64);  // one thread per (mu, r) / (mu, nu)
    static constexpr int LP = L + 1;                      // padded row of B (LDS banks)
};

template <int L>
struct WinTw {
    float2 w[L];  // e^{-2 pi i k / L}, k = 0..L-1
};

}  // namespace

// bx: the windows of the volume positions o + S k, k < ceil(d / S), E stored in the frame
// (fo, fk) at index (p - fo) / S; with a table, workgroups [e * per_box, (e+1) * per_box)
// serve entry e.
template <int L>
__global__ __launch_bounds__(WinCfg<L>::NT) void k_energy_win(const float *__restrict__ V, int n0, int n1, int n2,
                                                              ebox bx, int S, WinTw<L> tw,
                                                              const float *__restrict__ wgen, float *__restrict__ E,
                                                              float *__restrict__ vmax_part)
{
    using C = WinCfg<L>;
    constexpr int H = L / 2, h = C::h, NT = C::NT, LP = C::LP, L2 = L * L, L3 = L * L * L;
    constexpr int NWV = NT / 64;
    __shared__ float win[L3];            // [p][q][r]
    __shared__ float2 A_s[h * L2];       // [mu][q][r]
    __shared__ float2 B_s[h * L * LP];   // [mu][nu][r], rows padded
    __shared__ float red_s[NWV][4];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int box;
    // (ranges: 150 tiles of 4^3 at cube 20, stride 8, 498 us in dispatch order, 487 so)
    const int blk = box_tile<true>(bx, &box);
    V += box * bx.vstride;
    E += box * bx.estride;
    const int nblk = bx.table ? bx.per_box : (int)gridDim.x;
    const int kd0 = (bx.d0 + S - 1) / S, kd1 = (bx.d1 + S - 1) / S, kd2 = (bx.d2 + S - 1) / S;
    const int nwin = kd0 * kd1 * kd2;
    const int K1 = bx.fk1, K2 = bx.fk2;
    const int64_t nfr = (int64_t)bx.fk0 * K1 * K2;
    const int64_t plane = (int64_t)n1 * n2;
    float vmax = 0.f;

    // The samples of the next window are loaded into registers while the current one
    // computes, so their latency is hidden; every thread holds NLD of them.
    constexpr int NLD = (L3 + NT - 1) / NT;
    float pre[NLD];
    auto load_win = [&](int w) {
        const int k2 = w % kd2, k1 = (w / kd2) % kd1, k0 = w / (kd2 * kd1);
        const int q0 = bx.o0 + S * k0 - H, q1 = bx.o1 + S * k1 - H, q2 = bx.o2 + S * k2 - H;
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            const int i = tid + NT * j;
            if (i < L3) {
                const int r = i % L, q = (i / L) % L, p = i / L2;
                pre[j] = V[(int64_t)refl_idx(q0 + p, n0) * plane + (int64_t)refl_idx(q1 + q, n1) * n2 +
                           refl_idx(q2 + r, n2)];
            }
        }
    };
    if (blk < nwin) load_win(blk);

    for (int w = blk; w < nwin; w += nblk) {
        const int k2 = w % kd2, k1 = (w / kd2) % kd1, k0 = w / (kd2 * kd1);
        const int p0 = bx.o0 + S * k0, p1 = bx.o1 + S * k1, p2 = bx.o2 + S * k2;
        __syncthreads();  // the previous window is done with win, A_s, B_s and red_s
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            const int i = tid + NT * j;
            if (i < L3) {
                vmax = fmaxf(vmax, fabsf(pre[j]));
                win[i] = pre[j];
            }
        }
        __syncthreads();
        if (w + nblk < nwin) load_win(w + nblk);
        // ---------------- stage A: real DFT along t, mu <= L/2 ---------------------------
        for (int c = tid; c < L2; c += NT) {
            float v[L];
            float2 x[h];
#pragma unroll
            for (int p = 0; p < L; ++p) v[p] = win[p * L2 + c];
            sal_dft::rdft_half<L>(v, tw.w, x);
#pragma unroll
            for (int mu = 0; mu < h; ++mu) A_s[mu * L2 + c] = x[mu];
        }
        __syncthreads();
        // ---------------- stage B: DFT along x per (mu, r), every nu ---------------------
        if (tid < h * L) {
            const int mu = tid / L, r = tid - (tid / L) * L;
            float2 a[L], f[L];
#pragma unroll
            for (int q = 0; q < L; ++q) a[q] = A_s[(mu * L + q) * L + r];
            sal_dft::cdft<L>(a, tw.w, f);
#pragma unroll
            for (int nu = 0; nu < L; ++nu) B_s[(mu * L + nu) * LP + r] = f[nu];
        }
        __syncthreads();
        // ---------------- stage C: DFT along y per row (mu, nu), projections -------------
        float e0 = 0.f, e1 = 0.f, e2 = 0.f;
        if (tid < h * L) {
            const int mu = tid / L, nu = tid - (tid / L) * L;
            float2 b[L], f[L];
#pragma unroll
            for (int r = 0; r < L; ++r) b[r] = B_s[(mu * L + nu) * LP + r];
            sal_dft::cdft<L>(b, tw.w, f);
            const float *wr = wgen + (int64_t)(mu * L + nu) * L * 3;
#pragma unroll
            for (int om = 0; om < L; ++om) {
                const float m = __builtin_amdgcn_sqrtf(fmaf(f[om].x, f[om].x, f[om].y * f[om].y));
                e0 = fmaf(wr[3 * om], m, e0);
                e1 = fmaf(wr[3 * om + 1], m, e1);
                e2 = fmaf(wr[3 * om + 2], m, e2);
            }
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            e0 += __shfl_xor(e0, o);
            e1 += __shfl_xor(e1, o);
            e2 += __shfl_xor(e2, o);
        }
        if (lane == 0) {
            red_s[wave][0] = e0;
            red_s[wave][1] = e1;
            red_s[wave][2] = e2;
        }
        __syncthreads();
        if (tid == 0) {
            float s0 = 0.f, s1 = 0.f, s2 = 0.f;
#pragma unroll
            for (int v = 0; v < NWV; ++v) {
                s0 += red_s[v][0];
                s1 += red_s[v][1];
                s2 += red_s[v][2];
            }
            const int64_t o = ((int64_t)((p0 - bx.fo0) / S) * K1 + (p1 - bx.fo1) / S) * K2 + (p2 - bx.fo2) / S;
            E[o] = s0;
            E[nfr + o] = s1;
            E[2 * nfr + o] = s2;
        }
    }
    // max |V| of everything this workgroup read (all of it lies in the volume)
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) vmax = fmaxf(vmax, __shfl_xor(vmax, o));
    __syncthreads();
    if (lane == 0) red_s[wave][3] = vmax;
    __syncthreads();
    if (tid == 0 && vmax_part) {
        float m = red_s[0][3];
        for (int v = 1; v < NWV; ++v) m = fmaxf(m, red_s[v][3]);
        vmax_part[blockIdx.x] = m;
    }
}

// ------------------------------------------------------------------------------------
// Cubes 9..15 and 17..20 with overlapping windows (stride S < L): a run of windows along y
// shares the first two stages.  Bound by vector issue, nearly all of it the L-point DFTs:
// k_energy_win spends 4 h L^3 + 8 h L^3 flops per window on stages A and B, which here are
// done once per y position of the run.  The run's samples and DFTs are the windows' own, so
// every value and every sum has the operands and the order of k_energy_win and the energies
// are the same bit for bit, whatever run, box or crop a window is computed in.
//   stage A  one thread per (x, y) column of the run: samples straight from global memory
//            (rows along y are contiguous), the real DFT along t into P[mu][x][y];
//   stage B  one thread per (mu, y): the DFT along x, in place (a thread reads and writes one
//            column of P);
//   stage C  one thread per row (mu, nu) of a window, as many windows at once as the threads
//            hold (the weights stay in registers; om and L - om share theirs): the DFT along y
//            of the row's L values, the magnitudes and weighted sums; then the tree of the
//            window's rows.  Where a window's rows fill whole waves the tree is lane swaps and
//            row rotations and no wave waits for another.  Elsewhere threads take rows across
//            waves, without gaps, and one wave at a time sums the tree from LDS.  Of the rows nu
//            and L - nu of a real t spectrum (mu = 0 and L/2), conjugates bin for bin, one
//            thread then transforms one and sums both, its magnitudes in either order.
// The row stride of P is odd (in complex values): the lanes of stage C, one row each, hit
// all banks.  Cube 12 on 131 x 187 x 253: 4.45 ms against 24.6 ms window by window (whole pass);
// with 64 rows of one window to a wave at every side, 96 lanes for its 84 rows, 5.4 ms.  Energies
// of 96 x 100 x 120, 64 rows to a wave -> this: cube 9 460 -> 387 us, 11 1,059 -> 743, 13 1,303 ->
// 1,069, 14 1,413 -> 1,251, 17 3,934 -> 2,696, 18 4,968 -> 2,967, 19 5,424 -> 4,207 and 20 6,480 ->
// 5,034 (the last two as whole waves in sets of four).
namespace {

template <int L>
struct RunCfg {
    static constexpr int h = L / 2 + 1, ROWS = h * L;
    static constexpr int NB = (ROWS + 63) / 64;  // blocks of rows in the sum's tree
    static constexpr int REAL = 2 - L % 2;       // mu with a real t spectrum: 0 (and L/2)
    static constexpr int M = (L - 1) / 2;        // conjugate rows (nu, L - nu) of each
    // Waves: whole sets of four, one per SIMD.  (With 3, 5, 6 or 7 the barriers wait for the
    // fullest SIMD: cube 12 5.2 to 6.4 ms with fewer idle lanes than four's 4.5 ms.)  More than
    // four meet more of the others at every barrier, so they have to need a fifth fewer lanes per
    // window (cube 10 546 us with four, 897 with twelve that need a seventh fewer).
    static constexpr int waves()
    {
        int best = 4, lanes = 64 * 4 / (64 * 4 / (ROWS - REAL * M));
        for (int n = 8; n <= 12; n += 4) {
            const int l = 64 * n / (64 * n / (ROWS - REAL * M));
            if (5 * l < 4 * lanes) {
                best = n;
                lanes = l;
            }
        }
        return best;
    }
    static constexpr int NWV = waves(), NT = 64 * NWV;
    // a window's rows in waves of their own where that takes no more waves
    static constexpr bool OWN = NT / (64 * NB) >= NT / (ROWS - REAL * M);
    static constexpr int PAIR = OWN ? 0 : REAL * M;  // conjugate pairs, a thread for both rows
    static constexpr int R = OWN ? 64 * NB : ROWS - PAIR;  // threads per window
    static constexpr int G = NT / R;             // windows transformed together
    static constexpr int ES = 64 * NB + 4;       // floats per window and component
    static constexpr int MAXRUN = 32;            // windows of a run, up to a multiple of G
    // floats of e_s: [run's window][component][block], or two of [window of G][component][row]
    static constexpr int NE = OWN ? MAXRUN * 3 * NB : 2 * G * 3 * ES;
    // registers for two workgroups of eight waves on a CU
    static constexpr int OCC = NWV == 8 ? 4 : 1;
    static_assert(G >= 1 && (!OWN || MAXRUN % G == 0), "threads for a window, e_s for a run");
};

constexpr int RUN_LDS_MAX = 80 * 1024;  // P of one workgroup: at least two fit a CU

__host__ __device__ constexpr int run_row_stride(int L, int S, int run) { return (S * (run - 1) + L) | 1; }

template <int CTL>
__device__ __forceinline__ float dpp(float v)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), CTL, 0xf, 0xf, true));
}
// x summed over the four lanes of a quad: pairs 2, then 1 lane apart
__device__ __forceinline__ float quad_sum(float x)
{
    x += dpp<0x4E>(x);  // quad_perm [2,3,0,1]
    x += dpp<0xB1>(x);  // quad_perm [1,0,3,2]
    return x;
}
// x summed over the 16 lanes of a row: rotations by 8 and 4, then the quad (the order of the xor
// butterfly from 8 down to 1)
__device__ __forceinline__ float row_sum(float x)
{
    x += dpp<0x128>(x);  // row_ror:8
    x += dpp<0x124>(x);  // row_ror:4
    return quad_sum(x);
}
// The two outputs of a swap of a and b, added: lanes of the lower half (or even rows) hold
// a's sum over the pair, the others b's.
__device__ __forceinline__ float pair32(float a, float b)
{
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ float pair16(float a, float b)
{
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

}  // namespace

template <int L>
__global__ __launch_bounds__(RunCfg<L>::NT, RunCfg<L>::OCC) void k_energy_run(const float *__restrict__ V, int n0, int n1, int n2,
                                                              ebox bx, int S, int run, WinTw<L> tw,
                                                              const float *__restrict__ wgen, float *__restrict__ E,
                                                              float *__restrict__ vmax_part)
{
    using C = RunCfg<L>;
    constexpr int H = L / 2, h = C::h, NT = C::NT;
    extern __shared__ float2 P[];  // [mu][x, then nu][RS]
    __shared__ float e_s[C::NE];
    __shared__ float vred_s[C::NWV];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int box;
    const int blk = box_tile(bx, &box);
    V += box * bx.vstride;
    E += box * bx.estride;
    const int nblk = bx.table ? bx.per_box : (int)gridDim.x;
    const int kd0 = (bx.d0 + S - 1) / S, kd1 = (bx.d1 + S - 1) / S, kd2 = (bx.d2 + S - 1) / S;
    const int nrun = (kd2 + run - 1) / run, ntile = kd0 * kd1 * nrun;
    const int PY = S * (run - 1) + L, RS = PY | 1;
    const int K1 = bx.fk1, K2 = bx.fk2;
    const int64_t nfr = (int64_t)bx.fk0 * K1 * K2;
    const int n12 = n1 * n2;  // the volume holds at most 2^31 - 1 samples
    float vmax = 0.f;

    // stage C: this thread's window of the G and its row; conjugate pairs in the first threads
    constexpr int NPR = C::G * C::PAIR, SINGLE = C::R - C::PAIR, SELF = C::REAL * C::REAL;
    const bool pair = tid < NPR;
    bool live = tid < C::G * C::R;
    int wsub = 0, mu = 0, nu = 0;
    if constexpr (C::OWN) {
        wsub = __builtin_amdgcn_readfirstlane(tid / C::R);
        live = tid % C::R < C::ROWS;
        mu = live ? tid % C::R / L : 0;
        nu = live ? tid % C::R % L : 0;
    } else if (pair) {
        const int i = tid % C::PAIR;
        wsub = tid / C::PAIR;
        mu = i / C::M * (L / 2);
        nu = 1 + i % C::M;
    } else if (live) {
        const int i = (tid - NPR) % SINGLE;
        wsub = (tid - NPR) / SINGLE;
        mu = i < SELF ? i / C::REAL * (L / 2) : 1 + (i - SELF) / L;
        nu = i < SELF ? i % C::REAL * (L / 2) : (i - SELF) % L;
    }
    const int row = mu * L + nu;
    float wt[L / 2 + 1][3];
#pragma unroll
    for (int om = 0; om <= L / 2; ++om)
#pragma unroll
        for (int m = 0; m < 3; ++m) wt[om][m] = wgen[(row * L + om) * 3 + m];
    if constexpr (!C::OWN)  // past the last row: zero
        for (int i = tid; i < 2 * C::G * 3 * (C::ES - C::ROWS); i += NT)
            e_s[i / (C::ES - C::ROWS) * C::ES + C::ROWS + i % (C::ES - C::ROWS)] = 0.f;

    // the row of this thread in window w of the run: the magnitudes' weighted sums
    auto row_sums = [&](int w, float (&m)[L], float (&e)[3]) __attribute__((always_inline)) {
        const float2 *src = P + row * RS + S * w;
        float2 b[L], f[L];
#pragma unroll
        for (int r = 0; r < L; ++r) b[r] = src[r];
        sal_dft::cdft<L>(b, tw.w, f);
        e[0] = e[1] = e[2] = 0.f;
#pragma unroll
        for (int om = 0; om < L; ++om) {
            m[om] = __builtin_amdgcn_sqrtf(fmaf(f[om].x, f[om].x, f[om].y * f[om].y));
#pragma unroll
            for (int c = 0; c < 3; ++c) e[c] = fmaf(wt[om <= L / 2 ? om : L - om][c], m[om], e[c]);
        }
    };

    for (int tile = blk; tile < ntile; tile += nblk) {
        const int kr = tile % nrun, k1 = (tile / nrun) % kd1, k0 = tile / (nrun * kd1);
        const int p0 = bx.o0 + S * k0, p1 = bx.o1 + S * k1, p2 = bx.o2 + S * run * kr;
        const int cnt = min(run, kd2 - run * kr);  // windows of this run
        // ---------------- stage A: real DFT along t of every column of the run -----------
        int rowo[L];
#pragma unroll
        for (int p = 0; p < L; ++p) rowo[p] = refl_idx(p0 - H + p, n0) * n12;
        for (int c = tid; c < L * PY; c += NT) {
            const int q = c / PY, r = c - q * PY;
            const int off = refl_idx(p1 - H + q, n1) * n2 + refl_idx(p2 - H + r, n2);
            float v[L];
            float2 x[h];
#pragma unroll
            for (int p = 0; p < L; ++p) v[p] = V[(uint32_t)(rowo[p] + off)];
#pragma unroll
            for (int p = 0; p < L; ++p) vmax = fmaxf(vmax, fabsf(v[p]));
            sal_dft::rdft_half<L>(v, tw.w, x);
#pragma unroll
            for (int mu = 0; mu < h; ++mu) P[(mu * L + q) * RS + r] = x[mu];
        }
        __syncthreads();
        // ---------------- stage B: DFT along x per (mu, y), in place ---------------------
        for (int c = tid; c < h * PY; c += NT) {
            const int mu = c / PY, r = c - mu * PY;
            float2 *col = P + mu * L * RS + r;
            float2 a[L], f[L];
#pragma unroll
            for (int q = 0; q < L; ++q) a[q] = col[q * RS];
            sal_dft::cdft<L>(a, tw.w, f);
#pragma unroll
            for (int nu = 0; nu < L; ++nu) col[nu * RS] = f[nu];
        }
        __syncthreads();
        // ---------------- stage C: DFT along y per row (mu, nu), projections -------------
        float *const E_run = E + ((int64_t)((p0 - bx.fo0) / S) * K1 + (p1 - bx.fo1) / S) * K2 + (p2 - bx.fo2) / S;
        if constexpr (C::OWN) {
            for (int w = wsub; w < cnt; w += C::G) {
                float m[L], e[3];
                row_sums(w, m, e);
#pragma unroll
                for (int c = 0; c < 3; ++c) e[c] = live ? e[c] : 0.f;
                // the block's tree: pairs 32, 16, 8, 4, 2, 1 lanes apart; rows of lanes: 0 holds
                // component 0, 2 component 1, 1 and 3 component 2
                const float a = row_sum(pair16(pair32(e[0], e[1]), pair32(e[2], e[2])));
                if ((lane & 15) == 0 && lane < 48)
                    e_s[(w * 3 + (lane == 0 ? 0 : (lane == 32 ? 1 : 2))) * C::NB + wave % C::NB] = a;
            }
            __syncthreads();
            for (int i = tid; i < 3 * cnt; i += NT) {
                float s = 0.f;
#pragma unroll
                for (int k = 0; k < C::NB; ++k) s += e_s[i * C::NB + k];
                E_run[i % 3 * nfr + i / 3] = s;
            }
            continue;
        }
        int ck = 0;
        for (int w0 = 0; w0 < cnt; w0 += C::G, ++ck) {
            float *const es = e_s + (ck & 1) * (C::G * 3 * C::ES);
            if (live && w0 + wsub < cnt) {
                float m[L], e[3];
                row_sums(w0 + wsub, m, e);
                float *o = es + wsub * 3 * C::ES + row;
#pragma unroll
                for (int c = 0; c < 3; ++c) o[c * C::ES] = e[c];
                if (pair) {  // the row L - nu: the magnitudes in the other order
                    o += L - 2 * nu;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        float s = 0.f;
#pragma unroll
                        for (int om = 0; om < L; ++om) s = fmaf(wt[om <= L / 2 ? om : L - om][c], m[om ? L - om : 0], s);
                        o[c * C::ES] = s;
                    }
                }
            }
            __syncthreads();
            // the rows' tree, 64 to a block, pairs 32, 16, 8, 4, 2, 1 apart: four lanes per window
            // and component, by one wave while the others go on (into the other half of e_s)
            if (wave == ck % C::NWV) {
                for (int it = lane >> 2; it < C::G * 3; it += 16) {
                    const float *src = es + it * C::ES + (lane & 3);
                    float s = 0.f;
#pragma unroll 1
                    for (int k = 0; k < C::NB; ++k, src += 64) {
                        float x[16];
#pragma unroll
                        for (int q = 0; q < 16; ++q) x[q] = src[4 * q];
#pragma unroll
                        for (int d = 8; d >= 1; d >>= 1)
#pragma unroll
                            for (int q = 0; q < d; ++q) x[q] += x[q + d];
                        s += quad_sum(x[0]);
                    }
                    const int w = w0 + it / 3;
                    if ((lane & 3) == 0 && w < cnt) E_run[it % 3 * nfr + w] = s;
                }
            }
        }
        // the next run's stage A may write P (every read of it lies before the last barrier), and
        // its stages' barriers separate the last two trees from the next writes of e_s
    }
    // max |V| of everything this workgroup read (all of it lies in the volume)
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) vmax = fmaxf(vmax, __shfl_xor(vmax, o));
    if (lane == 0) vred_s[wave] = vmax;
    __syncthreads();
    if (tid == 0 && vmax_part) {
        float m = vred_s[0];
        for (int v = 1; v < C::NWV; ++v) m = fmaxf(m, vred_s[v]);
        vmax_part[blockIdx.x] = m;
    }
}

// ------------------------------------------------------------------------------------
// Cube 16 on the matrix cores (FP32 16x16x4 MFMA), one window at a time per group of three
// waves (WM_GROUPS groups per workgroup would share the weight table; one group per workgroup,
// three workgroups per CU, measured fastest: 90 ms against 119 ms with two on a stride-4
// lattice of the 512 x 1024 x 1024 volume), the three contractions as small matrix products:
//   stage A (t, real -> half spectrum): rows (x, y) of the window, 16 per M tile (tile = x),
//           K = t, 16 columns (mu, re|im) for mu <= 8: the imaginary parts of mu = 0 and 8
//           are zero for a real input, so column 1 carries the real part of mu = 8; the
//           samples are the A operand straight from global memory (the next window's are
//           in flight during stages B and C);
//   stage B (x): rows y for one mu (tile = mu), K = (x, re|im), columns (re|im, nu);
//   stage C (y): rows nu for one mu (tile = mu), K = (y, re|im), columns (re|im, om): a lane
//           holds re and im of its bins in its two accumulators, so |F|, the projection
//           weights and the sums into E_t, E_x, E_y follow in registers.
// Stage outputs live in one LDS buffer per group [mu][row][re|im][17 columns] (B in place of
// A, plane by plane), the per-lane projection weights of stage C in another.  The wave that
// computes plane mu in stage B also reads it in stage C, so only stage A's output needs a
// barrier.  352 MFMAs per window (721 kflop; the separable transform counted with complex
// mu = 0 and 8 is 737 kflop).
namespace {
constexpr int WM_WAVES = 3, WM_GROUPS = 1;
constexpr int WM_L = 16, WM_H = 8, WM_h = 9, WM_RS = 17;  // row stride of the LDS planes
constexpr int WM_PLANE = WM_L * 2 * WM_RS;                // floats per mu plane
}  // namespace

__global__ __launch_bounds__(64 * WM_WAVES * WM_GROUPS) void k_energy_win_mfma(
    const float *__restrict__ V, int n0, int n1, int n2, ebox bx, int S, WinTw<16> tw,
    const float *__restrict__ wgen, float *__restrict__ E, float *__restrict__ vmax_part)
{
    constexpr int L = WM_L, H = WM_H, h = WM_h, RS = WM_RS, PL = WM_PLANE, G = WM_GROUPS;
    constexpr int NWV = WM_WAVES * G;
    constexpr int MTA = (L + WM_WAVES - 1) / WM_WAVES;  // stage-A M tiles per wave (at most)
    constexpr int MTB = (h + WM_WAVES - 1) / WM_WAVES;  // stage-B/C M tiles per wave
    __shared__ float P[G][h * PL];               // per group [mu][row][re|im][col], see above
    __shared__ float wl[h * 4 * 3 * 64];         // [mu][j][m][lane] projection weights
    __shared__ float red_s[NWV][4];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave / WM_WAVES, wv = wave - grp * WM_WAVES;  // group, wave in group
    const int g = lane >> 4, n = lane & 15;
    int box;
    // (ranges: 12 tiles of 8 x 30 x 40 at stride 16 90 us in dispatch order, 87 so)
    const int blk = box_tile<true>(bx, &box);
    V += box * bx.vstride;
    E += box * bx.estride;
    const int nblk = bx.table ? bx.per_box : (int)gridDim.x;
    const int kd0 = (bx.d0 + S - 1) / S, kd1 = (bx.d1 + S - 1) / S, kd2 = (bx.d2 + S - 1) / S;
    const int nwin = kd0 * kd1 * kd2;
    const int K1 = bx.fk1, K2 = bx.fk2;
    const int64_t nfr = (int64_t)bx.fk0 * K1 * K2;
    const int n12 = n1 * n2;  // the volume holds at most 2^31 - 1 samples
    float vmax = 0.f;
    float *Pg = P[grp];

    // weights of the bins (mu, nu = 4g + j, om = n) of this lane, with the conjugate
    // multiplicity of mu and 1/(L^3 (L^3 - 1)) (DC has weight 0)
    for (int i = tid; i < h * 4 * 3 * 64; i += 64 * NWV) {
        const int ln = i & 63, m = (i >> 6) % 3, j = (i / 192) & 3, mu = i / 768;
        wl[i] = wgen[((mu * L + 4 * (ln >> 4) + j) * L + (ln & 15)) * 3 + m];
    }
    // constant B operands: lane (g, n) at K step ks holds K = 4 ks + g, column n
    // stage A column n: (mu, re|im) = (n / 2, n % 2), except column 1 = (8, re)
    const int amu = n == 1 ? L / 2 : n >> 1, aim = n == 1 ? 0 : n & 1;
    float wa[4], wb[8][2];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const float2 w = tw.w[(amu * (4 * ks + g)) % L];
        wa[ks] = aim ? w.y : w.x;
    }
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            // K = (tap, re|im of the input), column (re|im of the output = nt, frequency n);
            // out = in * e^{-2 pi i tap f / L}, w = (cos, -sin)
            const int k = 4 * ks + g, tap = k >> 1, ci = k & 1;
            const float2 w = tw.w[(tap * n) % L];
            wb[ks][nt] = nt == 0 ? (ci == 0 ? w.x : -w.y) : (ci == 0 ? w.y : w.x);
        }

    // samples of this wave's stage-A tiles (x = wv + 3 i) for one window: lane (g, n)
    // holds V[t = 4 ks + g][x][y = n]
    float smp[MTA][4];
    auto load_win = [&](int w) {
        const int k2 = w % kd2, k1 = (w / kd2) % kd1, k0 = w / (kd2 * kd1);
        const int q0 = bx.o0 + S * k0 - H, q1 = bx.o1 + S * k1 - H, q2 = bx.o2 + S * k2 - H;
        const int yo = refl_idx(q2 + n, n2);
        int rowo[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) rowo[ks] = refl_idx(q0 + 4 * ks + g, n0) * n12 + yo;
#pragma unroll
        for (int i = 0; i < MTA; ++i) {
            const int x = wv + WM_WAVES * i;
            if (x < L) {
                const int xo = refl_idx(q1 + x, n1) * n2;
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) smp[i][ks] = V[(uint32_t)(rowo[ks] + xo)];
            }
        }
    };
    if (G * blk + grp < nwin) load_win(G * blk + grp);
    __syncthreads();  // wl complete

    // every wave of the workgroup takes the same number of steps (the barriers need it); a
    // group past the last window idles through its step
    for (int wb0 = G * blk; wb0 < nwin; wb0 += G * nblk) {
        const int w = wb0 + grp;
        const bool act = w < nwin;
        const int k2 = w % kd2, k1 = (w / kd2) % kd1, k0 = w / (kd2 * kd1);
        const int p0 = bx.o0 + S * k0, p1 = bx.o1 + S * k1, p2 = bx.o2 + S * k2;
        // ---------------- stage A: real DFT along t --------------------------------------
        if (act) {
#pragma unroll
            for (int i = 0; i < MTA; ++i) {
                const int x = wv + WM_WAVES * i;
                if (x < L) {
                    f4 acc = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) {
                        vmax = fmaxf(vmax, fabsf(smp[i][ks]));
                        acc = mfma4(smp[i][ks], wa[ks], acc);
                    }
                    // lane (g, n): rows y = 4g + j, column n = (amu, aim); lanes 0 and 1 also
                    // write the zero imaginary parts of mu = 0 and 8
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        Pg[amu * PL + (x * 2 + aim) * RS + 4 * g + j] = acc[j];
                        if (n < 2) Pg[amu * PL + (x * 2 + 1) * RS + 4 * g + j] = 0.f;
                    }
                }
            }
            if (w + G * nblk < nwin) load_win(w + G * nblk);
        }
        __syncthreads();
        float e0 = 0.f, e1 = 0.f, e2 = 0.f;
        if (act) {
#pragma unroll
            for (int i = 0; i < MTB; ++i) {
                const int mu = wv + WM_WAVES * i;
                if (mu < h) {
                    float *pl = Pg + mu * PL;
                    // ------------ stage B: DFT along x, plane mu in place ------------------
                    f4 acc[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                    for (int ks = 0; ks < 8; ++ks) {
                        const int k = 4 * ks + g;  // (x, re|im) = (k / 2, k % 2), row y = n
                        const float a = pl[k * RS + n];
#pragma unroll
                        for (int nt = 0; nt < 2; ++nt) acc[nt] = mfma4(a, wb[ks][nt], acc[nt]);
                    }
                    // rows y = 4g + j, column nu = n: (re, im) = (acc[0][j], acc[1][j]); every
                    // read of the plane is issued before these writes
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        pl[(n * 2) * RS + 4 * g + j] = acc[0][j];
                        pl[(n * 2 + 1) * RS + 4 * g + j] = acc[1][j];
                    }
                    // ------------ stage C: DFT along y, projections, energies -------------
#pragma unroll
                    for (int nt = 0; nt < 2; ++nt) acc[nt] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < 8; ++ks) {
                        const int k = 4 * ks + g;  // (y, re|im) = (k / 2, k % 2), row nu = n
                        const float a = pl[(n * 2 + (k & 1)) * RS + (k >> 1)];
#pragma unroll
                        for (int nt = 0; nt < 2; ++nt) acc[nt] = mfma4(a, wb[ks][nt], acc[nt]);
                    }
                    const float *wr = wl + mu * 768 + lane;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float m = __builtin_amdgcn_sqrtf(fmaf(acc[0][j], acc[0][j], acc[1][j] * acc[1][j]));
                        e0 = fmaf(wr[(j * 3 + 0) * 64], m, e0);
                        e1 = fmaf(wr[(j * 3 + 1) * 64], m, e1);
                        e2 = fmaf(wr[(j * 3 + 2) * 64], m, e2);
                    }
                }
            }
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            e0 += __shfl_xor(e0, o);
            e1 += __shfl_xor(e1, o);
            e2 += __shfl_xor(e2, o);
        }
        if (lane == 0) {
            red_s[wave][0] = e0;
            red_s[wave][1] = e1;
            red_s[wave][2] = e2;
        }
        __syncthreads();  // red_s complete; every wave is done with its group's P
        if (act && wv == 0 && lane == 0) {
            float s0 = 0.f, s1 = 0.f, s2 = 0.f;
#pragma unroll
            for (int v = 0; v < WM_WAVES; ++v) {
                s0 += red_s[wave + v][0];
                s1 += red_s[wave + v][1];
                s2 += red_s[wave + v][2];
            }
            const int64_t o = ((int64_t)((p0 - bx.fo0) / S) * K1 + (p1 - bx.fo1) / S) * K2 + (p2 - bx.fo2) / S;
            E[o] = s0;
            E[nfr + o] = s1;
            E[2 * nfr + o] = s2;
        }
        // (the next step's stage A may write P now; red_s is rewritten one barrier later)
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) vmax = fmaxf(vmax, __shfl_xor(vmax, o));
    __syncthreads();
    if (lane == 0) red_s[wave][3] = vmax;
    __syncthreads();
    if (tid == 0 && vmax_part) {
        float m = red_s[0][3];
        for (int v = 1; v < NWV; ++v) m = fmaxf(m, red_s[v][3]);
        vmax_part[blockIdx.x] = m;
    }
}

// ====================================================================== launchers

namespace {

constexpr int64_t WIN_BLOCKS = 4096;   // workgroups of a whole-volume launch
constexpr int64_t WIN_PER_BOX = 64;    // workgroups per box of a batch

int64_t win_blocks(int64_t nwin, int64_t nbox)
{
    if (nbox > 1) return (nwin < WIN_PER_BOX ? (nwin > 0 ? nwin : 1) : WIN_PER_BOX) * nbox;
    return nwin < WIN_BLOCKS ? (nwin > 0 ? nwin : 1) : WIN_BLOCKS;
}

// Windows per run of k_energy_run for a box of kd windows, or 0 where P would not leave room
// for two workgroups on a CU (wide strides of the largest cubes).  About 32, less where P is
// too large or the runs would not give every CU two workgroups, in multiples of the windows
// transformed together; then the runs of a row are made equal: at cube 18 on 61 x 87 x 101 rows
// of 3 x 32 + 5 windows took 3.27 ms, of 26 + 26 + 26 + 23 2.79 ms.
template <int L>
size_t run_lds(int S, int run)
{
    return (size_t)RunCfg<L>::ROWS * run_row_stride(L, S, run) * sizeof(float2);
}
template <int L>
constexpr size_t run_lds_static = (RunCfg<L>::NE + RunCfg<L>::NWV) * sizeof(float);

template <int L>
int run_length(int S, int64_t kd0, int64_t kd1, int64_t kd2, int64_t nbox)
{
    constexpr int G = RunCfg<L>::G;
    const size_t most = RUN_LDS_MAX - run_lds_static<L>;
    int run = (RunCfg<L>::MAXRUN + G - 1) / G * G;
    while (run - G >= 8 && (run_lds<L>(S, run) > most || kd0 * kd1 * ((kd2 + run - 1) / run) * nbox < 512)) run -= G;
    if (run_lds<L>(S, run) > most) return 0;
    const int64_t nrun = (kd2 + run - 1) / run, eq = (kd2 + nrun - 1) / nrun;
    return (int)((eq + G - 1) / G * G);
}

template <int L>
hipError_t launch_run_L(const sal_ctx *c, const float *V, int64_t n0, int64_t n1, int64_t n2, ebox bx, int S, int run,
                        float *E, float *vmax_part, int *nparts, hipStream_t s, int nbox)
{
    const int64_t ntile = (int64_t)((bx.d0 + S - 1) / S) * ((bx.d1 + S - 1) / S) * (((bx.d2 + S - 1) / S + run - 1) / run);
    const size_t lds = run_lds<L>(S, run), lds_all = lds + run_lds_static<L>;
    int64_t nb;
    if (bx.table) {
        // as window by window: a batch of one box has the chip to itself (a tile of 32^3 at cube 12
        // and stride 3 checked in 68 us window by window, 88 in runs on 64 workgroups, 56 so)
        bx.per_box = (int)(win_blocks(ntile, nbox) / nbox);
        nb = (int64_t)bx.per_box * nbox;
    } else {
        // at most WIN_BLOCKS workgroups (one partial each), in whole rounds of what 256 CUs hold
        const int64_t fit = 256 * (160 * 1024 / lds_all < 8 ? 160 * 1024 / lds_all : 8);
        nb = fit * (WIN_BLOCKS / fit);
        if (ntile < nb) nb = ntile;
    }
    if (nparts) *nparts = (int)nb;
    WinTw<L> tw;
    for (int k = 0; k < L; ++k) tw.w[k] = make_float2(c->tw_host[2 * k], c->tw_host[2 * k + 1]);
    if (lds_all > 65536)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_energy_run<L>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k_energy_run<L>, dim3((unsigned)nb), dim3(RunCfg<L>::NT), lds, s, V, (int)n0, (int)n1, (int)n2, bx,
                       S, run, tw, c->t.w_gen, E, vmax_part);
    return hipGetLastError();
}

template <int L>
hipError_t launch_win_L(const sal_ctx *c, const float *V, int64_t n0, int64_t n1, int64_t n2, ebox bx, int S,
                        float *E, float *vmax_part, int *nparts, hipStream_t s, int nbox)
{
    // overlapping windows of a cube without a fused kernel share their first stages in runs
    if constexpr (L > 8 && L != 16) {
        const int run = S < L ? run_length<L>(S, (bx.d0 + S - 1) / S, (bx.d1 + S - 1) / S, (bx.d2 + S - 1) / S,
                                              bx.table ? nbox : 1)
                              : 0;
        if (run) return launch_run_L<L>(c, V, n0, n1, n2, bx, S, run, E, vmax_part, nparts, s, nbox);
    }
    const int64_t nwin = ((bx.d0 + S - 1) / S) * ((bx.d1 + S - 1) / S) * ((bx.d2 + S - 1) / S);
    const int64_t nb = win_blocks(nwin, bx.table ? nbox : 1);
    if (bx.table) bx.per_box = (int)(nb / nbox);
    if (nparts) *nparts = (int)nb;
    WinTw<L> tw;
    for (int k = 0; k < L; ++k) tw.w[k] = make_float2(c->tw_host[2 * k], c->tw_host[2 * k + 1]);
    if constexpr (L == 16)
        hipLaunchKernelGGL(k_energy_win_mfma, dim3((unsigned)nb), dim3(64 * WM_WAVES * WM_GROUPS), 0, s, V, (int)n0, (int)n1,
                           (int)n2, bx, S, tw, c->t.w_gen, E, vmax_part);
    else
        hipLaunchKernelGGL(k_energy_win<L>, dim3((unsigned)nb), dim3(WinCfg<L>::NT), 0, s, V, (int)n0, (int)n1,
                           (int)n2, bx, S, tw, c->t.w_gen, E, vmax_part);
    return hipGetLastError();
}

}  // namespace

int64_t energy_win_num_blocks(const sal_ctx *c, int64_t k0, int64_t k1, int64_t k2)
{
    (void)c;
    return win_blocks(k0 * k1 * k2, 1);
}

hipError_t launch_energy_win(const sal_ctx *c, const float *V, int64_t n0, int64_t n1, int64_t n2, const ebox &bx,
                             float *E, float *vmax_part, int *nparts, hipStream_t s, int nbox)
{
    const int S = c->p.stride;
#define SAL_WIN(LL) \
    case LL: return launch_win_L<LL>(c, V, n0, n1, n2, bx, S, E, vmax_part, nparts, s, nbox)
    switch (c->L) {
        SAL_WIN(2); SAL_WIN(3); SAL_WIN(4); SAL_WIN(5); SAL_WIN(6); SAL_WIN(7); SAL_WIN(8);
        SAL_WIN(9); SAL_WIN(10); SAL_WIN(11); SAL_WIN(12); SAL_WIN(13); SAL_WIN(14); SAL_WIN(15);
        SAL_WIN(16); SAL_WIN(17); SAL_WIN(18); SAL_WIN(19); SAL_WIN(20);
    default: return hipErrorInvalidValue;
    }
#undef SAL_WIN
}
