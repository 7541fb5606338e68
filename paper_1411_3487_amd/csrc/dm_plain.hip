// dm_plain.hip -- FP64 kernels (gfx950): the dense transforms (positions and
// initial amplitudes of every path, and the mode step of chains beyond the
// persistent stepper, with its force stencil and mode update), the bead-space
// Euler baseline, observables, Monte Carlo and the inextensible limit.
//
// Data layout in HBM: a bucket of nch chains of M beads stores positions,
// forces and mode amplitudes as nch*3 columns of M doubles (SoA, column
// (chain, component) contiguous in the bead or mode index).  A transform is
// then one GEMM Y = A X^T with a square M x M table A and 3*nch columns:
//   inverse  r_n  = sum_{p>=1} phi_{n,p} R_p     (Eq. c1, internal coords)
//   forward  dH_p = sum_n phi_{n,p} F_n          (Eqs. c5, e11)
#include "dm_internal.h"
#include "dm_rng.h"

namespace dm {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// --------------------------------------------------------------------------
// GEMM on FP64 MFMA (v_mfma_f64_16x16x4f64).  MFMA operand layout per lane l:
// A[i = l%16][k = l/16], B[k = l/16][j = l%16]; result D[i = l/16 + 4r][j =
// l%16], r = 0..3 (the FP64 instruction interleaves its four result rows
// across the lane groups).
//
// Column c of the result goes to Y + c M, or, with off (one offset per chain of
// three columns), to Y + off[c / 3] + (c % 3) M: positions go straight to the
// caller's order.
//
// Any M: workgroup tile 32 rows x 32 columns, 4 waves of 16 x 16, K in chunks
// of 32, the next chunk in registers while the current one is multiplied from
// one of two LDS buffers.  Small tiles, because lengths that are no multiple
// of 16 come mostly in small launches: 140 chains of 257 beads make 126
// workgroups, where 64 x 64 tiles without a pipeline made 35 and took 32 us (7
// us now).  Full launches gain as well, by the pipeline: a call that reads the
// positions of 4000 chains of 257, 513 or 1025 beads takes 74, 196 and 691 us
// (102, 304 and 1038 with those tiles); of 16000 chains of 33 beads 31 (38).
// --------------------------------------------------------------------------
constexpr int kGemmBM = 64, kGemmBN = 64, kGemmBK = 16;

__device__ __forceinline__ double *gemm_column(double *Y, const int64_t *off, int M, int c)
{
    return off ? Y + off[c / 3] + (size_t)(c % 3) * M : Y + (size_t)c * M;
}

constexpr int kAnyB = 32, kAnyK = 32;
__global__ __launch_bounds__(256) void gemm_f64_any_kernel(const double *__restrict__ A,
                                                           const double *__restrict__ X,
                                                           double *__restrict__ Y,
                                                           const int64_t *__restrict__ off, int M,
                                                           int ncol)
{
    __shared__ double As[2][kAnyB][kAnyK + 1];
    __shared__ double Xs[2][kAnyB][kAnyK + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wi = 16 * (wave >> 1), wj = 16 * (wave & 1);
    // row tiles fastest, in one grid dimension: the second one ends at 65536
    // workgroups, which 699051 chains exceed
    const int nrow = (M + kAnyB - 1) / kAnyB;
    const int i0 = (int)(blockIdx.x % nrow) * kAnyB, c0 = (int)(blockIdx.x / nrow) * kAnyB;
    const int lk = tid & 31, lr = tid >> 5;  // rows lr, lr + 8, + 16, + 24
    double ra[4], rx[4];
    auto load = [&](int k0) {
        const int gk = k0 + lk;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int gi = i0 + lr + 8 * e, gc = c0 + lr + 8 * e;
            ra[e] = gi < M && gk < M ? A[(size_t)gi * M + gk] : 0.0;
            rx[e] = gc < ncol && gk < M ? X[(size_t)gc * M + gk] : 0.0;
        }
    };
    auto store = [&](int b) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            As[b][lr + 8 * e][lk] = ra[e];
            Xs[b][lr + 8 * e][lk] = rx[e];
        }
    };
    f64x4 acc = f64x4{0.0, 0.0, 0.0, 0.0};
    const int nk = (M + kAnyK - 1) / kAnyK;
    load(0);
    store(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int b = kt & 1;
        if (kt + 1 < nk) load((kt + 1) * kAnyK);
#pragma unroll
        for (int ks = 0; ks < kAnyK; ks += 4)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(As[b][wi + (lane & 15)][ks + (lane >> 4)],
                                                       Xs[b][wj + (lane & 15)][ks + (lane >> 4)],
                                                       acc, 0, 0, 0);
        if (kt + 1 < nk) store(b ^ 1);
        __syncthreads();
    }
    const int c = c0 + wj + (lane & 15), ib = i0 + wi + (lane >> 4);
    if (c >= ncol) return;
    double *y = gemm_column(Y, off, M, c);
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (ib + 4 * r < M) y[ib + 4 * r] = acc[r];
}

// The same product when M is a multiple of 16, workgroup tile 64 rows x BN
// columns, 4 waves of 32 x BN/2, K in chunks of 16: 16-byte loads of A and X, and a software
// pipeline over the K chunks -- the next chunk is loaded into registers while
// the current one is multiplied from the other of two LDS buffers, one
// barrier per chunk.  The MFMA sequence of every accumulator is the one of
// the kernel above, so both give the same bits.  BN = 64 or 32 columns per
// workgroup tile (each wavefront 32 rows x BN/2 columns): the narrower tile
// doubles the workgroups of small launches (1024 chains of 128 beads make 96
// tiles of 64 x 64 for 256 CUs) and leaves every accumulator's sequence as it
// is.
typedef double f64x2 __attribute__((ext_vector_type(2)));

// Workgroups of a launch are dispatched round-robin over the GPU's 8 XCDs
// (workgroup w to XCD w % 8), each with its own L2.  This maps the
// dispatch index w of n workgroups to a logical index such that every XCD
// takes one contiguous range of logical indices (a bijection on [0, n)).
__device__ __forceinline__ int xcd_local_index(int w, int n)
{
    constexpr int kXcd = 8;
    const int q = n / kXcd, r = n % kXcd, x = w % kXcd, s = w / kXcd;
    return x < r ? x * (q + 1) + s : r * (q + 1) + (x - r) * q + s;
}

template <int BN>
__global__ __launch_bounds__(256) void gemm_f64_pipe_kernel(const double *__restrict__ A,
                                                            const double *__restrict__ X,
                                                            double *__restrict__ Y,
                                                            const int64_t *__restrict__ off, int M,
                                                            int ncol)
{
    static_assert(BN == 64 || BN == 32, "column tile");
    constexpr int TJ = BN / 32;  // 16-column MFMA tiles per wavefront
    __shared__ double As[2][kGemmBM][kGemmBK + 1];
    __shared__ double Xs[2][BN][kGemmBK + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wi = wave >> 1, wj = wave & 1;
    // one-dimensional grid, row tiles fastest in the XCD-local order: the
    // row tiles that read the same column block of X run on one XCD and
    // share its L2, so each X block crosses HBM about once
    const int nrt = (M + kGemmBM - 1) / kGemmBM;
    const int L = xcd_local_index((int)blockIdx.x, (int)gridDim.x);
    const int i0 = (L % nrt) * kGemmBM;
    const int c0 = (L / nrt) * BN;
    // each thread moves 4 consecutive k of one row of A and (lr < BN) of one
    // column of X
    const int lr = tid >> 2, lk = (tid & 3) * 4;
    const bool xown = lr < BN;
    const bool arow = i0 + lr < M, xrow = xown && c0 + lr < ncol;
    const f64x2 *pa = reinterpret_cast<const f64x2 *>(A + (size_t)(arow ? i0 + lr : 0) * M + lk);
    const f64x2 *px = reinterpret_cast<const f64x2 *>(X + (size_t)(xrow ? c0 + lr : 0) * M + lk);
    f64x2 ra0, ra1, rx0, rx1;
    auto load = [&](int k0) {
        const f64x2 z = {0.0, 0.0};
        ra0 = arow ? pa[k0 / 2] : z;
        ra1 = arow ? pa[k0 / 2 + 1] : z;
        rx0 = xrow ? px[k0 / 2] : z;
        rx1 = xrow ? px[k0 / 2 + 1] : z;
    };
    auto store = [&](int b) {
        As[b][lr][lk] = ra0[0];
        As[b][lr][lk + 1] = ra0[1];
        As[b][lr][lk + 2] = ra1[0];
        As[b][lr][lk + 3] = ra1[1];
        if (xown) {
            Xs[b][lr][lk] = rx0[0];
            Xs[b][lr][lk + 1] = rx0[1];
            Xs[b][lr][lk + 2] = rx1[0];
            Xs[b][lr][lk + 3] = rx1[1];
        }
    };
    f64x4 acc[2][TJ];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < TJ; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};

    const int nk = M / kGemmBK;
    load(0);
    store(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int b = kt & 1;
        if (kt + 1 < nk) load((kt + 1) * kGemmBK);
#pragma unroll
        for (int ks = 0; ks < kGemmBK; ks += 4) {
            double a[2], x[TJ];
#pragma unroll
            for (int t = 0; t < 2; ++t)
                a[t] = As[b][32 * wi + 16 * t + (lane & 15)][ks + (lane >> 4)];
#pragma unroll
            for (int t = 0; t < TJ; ++t)
                x[t] = Xs[b][(BN / 2) * wj + 16 * t + (lane & 15)][ks + (lane >> 4)];
#pragma unroll
            for (int ti = 0; ti < 2; ++ti)
#pragma unroll
                for (int tj = 0; tj < TJ; ++tj)
                    acc[ti][tj] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ti], x[tj],
                                                                      acc[ti][tj], 0, 0, 0);
        }
        if (kt + 1 < nk) store(b ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj) {
            const int c = c0 + (BN / 2) * wj + 16 * tj + (lane & 15);
            const int ib = i0 + 32 * wi + 16 * ti + (lane >> 4);
            if (c >= ncol) continue;
            double *y = gemm_column(Y, off, M, c);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (ib + 4 * r < M) y[ib + 4 * r] = acc[ti][tj][r];
        }
}

// --------------------------------------------------------------------------
// Force stencil, one thread per (chain, bead).  Bonds u_n = r_n - r_{n-1}
// (n = 1..M-1), g_n = u_n (1/|u_n| - lin) with lin = 1 - 2 nu (Eq. e4),
// F_n = g_n - g_{n+1} with g_0 = g_M = 0.
// --------------------------------------------------------------------------
__device__ __forceinline__ void bond_g(const double *__restrict__ x, int M, int m,
                                       double lin, double g[3])
{
    const double ux = x[m] - x[m - 1];
    const double uy = x[M + m] - x[M + m - 1];
    const double uz = x[2 * M + m] - x[2 * M + m - 1];
    const double f = rsqrt64(ux * ux + uy * uy + uz * uz) - lin;
    g[0] = ux * f;
    g[1] = uy * f;
    g[2] = uz * f;
}

__global__ __launch_bounds__(256) void stencil_f64_kernel(const double *__restrict__ r,
                                                          double *__restrict__ F, int M,
                                                          int nch, double lin)
{
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)nch * M) return;
    const int c = (int)(idx / M), n = (int)(idx % M);
    const double *x = r + (size_t)c * 3 * M;
    double g0[3] = {0.0, 0.0, 0.0}, g1[3] = {0.0, 0.0, 0.0};
    if (n >= 1) bond_g(x, M, n, lin, g0);
    if (n + 1 <= M - 1) bond_g(x, M, n + 1, lin, g1);
    double *f = F + (size_t)c * 3 * M;
    f[n] = g0[0] - g1[0];
    f[M + n] = g0[1] - g1[1];
    f[2 * M + n] = g0[2] - g1[2];
}

// --------------------------------------------------------------------------
// Mode update (Eqs. d3, d6, f2, btum), one thread per (chain, 4 modes): its
// three Philox blocks (one per component) give all twelve normals, and for
// even M each row's quad moves as two 16-byte pieces, so the lanes of a
// wavefront read and write contiguous runs and the shear drift is folded
// into the one store.
// --------------------------------------------------------------------------
__global__ __launch_bounds__(256) void mode_update_f64_kernel(
    double *__restrict__ R, const double *__restrict__ dH, const double *__restrict__ E,
    const double *__restrict__ C, const double *__restrict__ W,
    const int32_t *__restrict__ ids, int M, int nch, uint64_t seed,
    const int64_t *__restrict__ step_dev, int64_t step_off, double gdt, int nonlinear)
{
    const int nq = (M + 3) / 4;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)nch * nq) return;
    const int c = (int)(idx / nq), q = (int)(idx % nq);
    const int64_t k = (step_dev ? *step_dev : 0) + step_off;
    const uint32_t chain = (uint32_t)ids[c];
    double z[3][4];
#pragma unroll
    for (int a = 0; a < 3; ++a)
        normals4_f64(noise_bits(seed, (uint32_t)q, chain, k, (uint32_t)a, kTagMode), z[a]);
    double *Rc = R + (size_t)c * 3 * M;
    const double *dHc = dH + (size_t)c * 3 * M;
    // a whole quad of an even-length chain moves as two 16-byte pieces per row
    const bool vec = (M % 2 == 0) && (4 * q + 3 < M);
    double r[3][4], d[3][4], e[4], w[4], cc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int p = min(4 * q + j, M - 1);
        e[j] = E[p];
        w[j] = W[p];
        cc[j] = C[p];
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (vec) {
            const f64x2 *src = reinterpret_cast<const f64x2 *>(Rc + a * M + 4 * q);
            const f64x2 lo = src[0], hi = src[1];
            r[a][0] = lo[0], r[a][1] = lo[1], r[a][2] = hi[0], r[a][3] = hi[1];
            if (nonlinear) {
                const f64x2 *hs = reinterpret_cast<const f64x2 *>(dHc + a * M + 4 * q);
                const f64x2 dl = hs[0], dh = hs[1];
                d[a][0] = dl[0], d[a][1] = dl[1], d[a][2] = dh[0], d[a][3] = dh[1];
            } else {
                d[a][0] = d[a][1] = d[a][2] = d[a][3] = 0.0;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int p = min(4 * q + j, M - 1);
                r[a][j] = Rc[a * M + p];
                d[a][j] = nonlinear ? dHc[a * M + p] : 0.0;
            }
        }
    }
    double v[3][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int p = 4 * q + j;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            v[a][j] = e[j] * r[a][j] + w[j] * z[a][j];
            if (nonlinear && p > 0) v[a][j] += cc[j] * d[a][j];
        }
        v[0][j] += gdt * e[j] * r[1][j];
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (vec) {
            f64x2 *dst = reinterpret_cast<f64x2 *>(Rc + a * M + 4 * q);
            dst[0] = f64x2{v[a][0], v[a][1]};
            dst[1] = f64x2{v[a][2], v[a][3]};
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (4 * q + j < M) Rc[a * M + 4 * q + j] = v[a][j];
        }
    }
}

// --------------------------------------------------------------------------
// Bead-space Euler (Eqs. b3-b5, btum).  One block per chain, positions held
// in LDS across all steps; thread t owns beads 4t..4t+3.
//   u_m = x_m - x_{m-1} for 1 <= m <= M-1, else 0;
//   h_m = (|u_m| - 1) u_m/|u_m| - nu (u_{m-1} + u_{m+1}) for 1 <= m <= M-1;
//   x_n += dtau (h_{n+1} - h_n) + sqrt(2 T* dtau) eta_n;  x_n += gdt y_n(old).
// --------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void euler_f64_kernel(double *__restrict__ pos,
                                                         const int32_t *__restrict__ ids,
                                                         int M, double nu, double dtau,
                                                         double amp, double gdt,
                                                         uint64_t seed, int64_t step0,
                                                         int n_steps)
{
    extern __shared__ double xs[];  // 3*M
    const int c = blockIdx.x, tid = threadIdx.x;
    double *P = pos + (size_t)c * 3 * M;
    for (int i = tid; i < 3 * M; i += blockDim.x) xs[i] = P[i];
    __syncthreads();
    const int nq = (M + 3) / 4;
    const bool active = tid < nq;
    const int n0 = 4 * tid;
    const uint32_t chain = (uint32_t)ids[c];
    for (int s = 0; s < n_steps; ++s) {
        double nx[3][4];
        if (active) {
            const int64_t k = step0 + s;
            double z[3][4];
#pragma unroll
            for (int a = 0; a < 3; ++a)
                normals4_f64(noise_bits(seed, (uint32_t)tid, chain, k, (uint32_t)a, kTagEuler),
                             z[a]);
            // bonds m = n0-1 .. n0+5  -> u[0..6]
            double u[3][7];
#pragma unroll
            for (int j = 0; j < 7; ++j) {
                const int m = n0 - 1 + j;
                const bool ok = (m >= 1) && (m <= M - 1);
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    u[a][j] = ok ? xs[a * M + m] - xs[a * M + m - 1] : 0.0;
            }
            // h_m for m = n0 .. n0+4 -> h[0..4] (u index j = m - n0 + 1)
            double h[3][5];
#pragma unroll
            for (int j = 0; j < 5; ++j) {
                const int m = n0 + j;
                const bool ok = (m >= 1) && (m <= M - 1);
                // (|u| - 1) / |u| = 1 - 1/|u|
                const double f = 1.0 - rsqrt64(u[0][j + 1] * u[0][j + 1] +
                                               u[1][j + 1] * u[1][j + 1] +
                                               u[2][j + 1] * u[2][j + 1]);
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    h[a][j] = ok ? f * u[a][j + 1] - nu * (u[a][j] + u[a][j + 2]) : 0.0;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = n0 + j;
                if (n >= M) break;
                const double y_old = xs[M + n];
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    nx[a][j] = xs[a * M + n] + (dtau * (h[a][j + 1] - h[a][j]) + amp * z[a][j]);
                nx[0][j] += gdt * y_old;
            }
        }
        __syncthreads();
        if (active) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = n0 + j;
                if (n >= M) break;
#pragma unroll
                for (int a = 0; a < 3; ++a) xs[a * M + n] = nx[a][j];
            }
        }
        __syncthreads();
    }
    for (int i = tid; i < 3 * M; i += blockDim.x) P[i] = xs[i];
}

// --------------------------------------------------------------------------
// Observables (Sec. V.B): one wave per chain, FP64 wavefront reductions.
// --------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ double wave_min(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

__global__ __launch_bounds__(64) void chain_obs_kernel(const double *__restrict__ pos,
                                                       const double *__restrict__ R,
                                                       double *__restrict__ obs,
                                                       double *__restrict__ m2,
                                                       double *__restrict__ acc,
                                                       const double *__restrict__ cm0,
                                                       double *__restrict__ tstate,
                                                       double *__restrict__ tlast,
                                                       const int64_t *__restrict__ step_dev,
                                                       double *__restrict__ ring,
                                                       double *__restrict__ ccount, int K,
                                                       int M, int accumulate)
{
    const int c = blockIdx.x, lane = threadIdx.x;
    const double *x = pos + (size_t)c * 3 * M;
    double ls = 0.0, l2s = 0.0, sx = 0.0, sy = 0.0, sz = 0.0;
    double xmin = x[0], xmax = x[0];
    for (int n = lane; n < M; n += 64) {
        sx += x[n];
        sy += x[M + n];
        sz += x[2 * M + n];
        xmin = fmin(xmin, x[n]);
        xmax = fmax(xmax, x[n]);
        if (n >= 1) {
            const double ux = x[n] - x[n - 1], uy = x[M + n] - x[M + n - 1],
                         uz = x[2 * M + n] - x[2 * M + n - 1];
            const double q = ux * ux + uy * uy + uz * uz;
            ls += sqrt(q);
            l2s += q;
        }
    }
    ls = wave_sum(ls);
    l2s = wave_sum(l2s);
    sx = wave_sum(sx);
    sy = wave_sum(sy);
    sz = wave_sum(sz);
    xmin = wave_min(xmin);
    xmax = wave_max(xmax);
    const double *Rc = R + (size_t)c * 3 * M;
    double *accc = acc + (size_t)c * acc_width(M);
    for (int p = lane; p < M; p += 64) {
        const double v = Rc[p] * Rc[p] + Rc[M + p] * Rc[M + p] + Rc[2 * M + p] * Rc[2 * M + p];
        m2[(size_t)c * M + p] = v;
        if (accumulate) accc[DM_NACC_HEAD + p] += v;
    }
    if (lane == 0) {
        double o[16];
        o[0] = ls / (M - 1);
        const double Lx = x[M - 1] - x[0], Ly = x[2 * M - 1] - x[M],
                     Lz = x[3 * M - 1] - x[2 * M];
        o[1] = Lx * Lx + Ly * Ly + Lz * Lz;
        o[2] = Lx;
        o[3] = Ly;
        o[4] = Lz;
        o[5] = sx / M;
        o[6] = sy / M;
        o[7] = sz / M;
        const int m = M / 2, mid = (M - 1) / 2;
        for (int a = 0; a < 3; ++a) {
            o[8 + a] = x[a * M + m] - x[a * M + m - 1];
            o[11 + a] = x[a * M + mid] - o[5 + a];
        }
        o[14] = xmax - xmin;
        o[15] = l2s / (M - 1);
        for (int j = 0; j < 16; ++j) obs[(size_t)c * 16 + j] = o[j];
        if (accumulate) {
            const double dx = o[5] - cm0[3 * c], dy = o[6] - cm0[3 * c + 1],
                         dz = o[7] - cm0[3 * c + 2];
            accc[DM_ACC_NSAMPLES] += 1.0;
            accc[DM_ACC_BOND] += o[0];
            accc[DM_ACC_BOND2] += o[15];
            accc[DM_ACC_L2] += o[1];
            accc[DM_ACC_MSDCM] += dx * dx + dy * dy + dz * dz;
            accc[DM_ACC_DMID2] += o[11] * o[11] + o[12] * o[12] + o[13] * o[13];
            accc[DM_ACC_XSPAN] += o[14];
            // tumbling in the flow plane, with hysteresis (see dnamodes.h)
            const double rho = sqrt(Lx * Lx + Ly * Ly);
            const double s0 = tstate[c];
            const double s1 = Lx > 0.5 * rho ? 1.0 : (Lx < -0.5 * rho ? -1.0 : s0);
            if (s0 != 0.0 && s1 != s0) {
                const double k = (double)*step_dev;
                accc[DM_ACC_TUMBLES] += 1.0;
                if (tlast[c] > 0.0) {
                    const double tau = k - (tlast[c] - 1.0);
                    accc[DM_ACC_TAU] += tau;
                    accc[DM_ACC_TAU2] += tau * tau;
                    accc[DM_ACC_NTAU] += 1.0;
                    const int bin = min(DM_NTUMBLE_BINS - 1, max(0, ilogb(tau)));
                    accc[DM_NACC_HEAD + M + bin] += 1.0;
                }
                tlast[c] = k + 1.0;
            }
            tstate[c] = s1;
            if (K > 0) {
                const double v[9] = {Lx, Ly, Lz, o[8], o[9], o[10], o[11], o[12], o[13]};
                corr_update(ring + (size_t)c * ((size_t)9 << (K - 1)), ccount + c,
                            accc + DM_NACC_HEAD + M + DM_NTUMBLE_BINS, v, K);
            }
        }
    }
}

// Sum over the wavefront, in every lane: DPP row shifts and row broadcasts
// (two 32-bit moves and an add each, no LDS crossbar), then lane 63's value
// through a scalar register.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo =
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xF, true);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xF, true);
    return v + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double read_lane(double v, int lane)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double wave_total(double v)
{
    v = dpp_add<0x111, 0xF>(v);  // row_shr:1, 2, 4, 8: lane 15 of a row holds its sum
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
    return read_lane(v, 63);
}

// Metropolis Monte Carlo in the mode representation, one wavefront per
// chain (the paper's equilibrium benchmark, Sec. V.B).  A sweep proposes, for
// p = 1..M-1 and component a = x, y, z in order, R_p^a += delta with delta
// uniform on (-s_p, s_p), and accepts with probability
// min(1, exp(-dH'/T*)) for the reduced Hamiltonian of Eq. (b3).  Random
// numbers: Philox block (p, chain, sweep, a, tag 2), word 0 for delta, word 1
// for the acceptance test u < exp(-dH'/T*), i.e. dH' < -T* ln u.
//
// The quadratic part of H' is diagonal in the modes (Eqs. c6, c9), so
//   dH' = zeta^l_p (R_p^a delta + delta^2 / 2) - sum_n (|u'_n| - |u_n|):
// a move costs one square root and about five operations per bond.  It is
// accepted when sum_n (|u'_n| - |u_n|) > thr with
//   thr = zeta^l_p (R_p^a delta + delta^2 / 2) + T* ln u,
// which needs nothing of the bonds: lane i draws delta and thr of proposal i
// of a batch of 63 (21 modes) and the proposals read them from that lane.
// The bonds u_n, their squares and lengths stay in registers, BPL bonds
// n = lane + 64 b per lane; squares and lengths are formed from the bonds
// anew at every sweep.
//
// Bound by the chain of dependent proposals: 0.22 us each at 128 beads, most
// of it the latency of the square root and of the sum over the wavefront
// (1.2 us with the bonds in LDS, every lane drawing the same random numbers,
// two square roots per bond and the sum over the LDS crossbar); 0.98 us at
// 1025 beads, 2.8 beyond (BPL = 22: 86 of its registers are spilled), where it
// was 7 to 9.
constexpr int kMcBatch = 21;  // modes of a batch
template <int BPL>
__global__ __launch_bounds__(64) void mc_kernel(double *__restrict__ R,
                                                const double *__restrict__ chiT,
                                                const double *__restrict__ sstep,
                                                const double *__restrict__ zeta_l,
                                                const int32_t *__restrict__ ids, int M,
                                                double T_star, uint64_t seed, int64_t step0,
                                                int n_sweeps, int64_t *__restrict__ accepted)
{
    extern __shared__ double Rl[];  // the amplitudes R[3][M], for the first bonds only
    const int c = blockIdx.x, lane = threadIdx.x, NB = M - 1;
    double *Rc = R + (size_t)c * 3 * M;
    const uint32_t chain = (uint32_t)ids[c];
    for (int i = lane; i < 3 * M; i += 64) Rl[i] = Rc[i];
    __syncthreads();
    double u[3][BPL], l2[BPL], l[BPL], ch[BPL], nx[BPL];
    // chi of mode p at the own bonds, 0 where there is no bond
    auto load_chi = [&](int p, double (&d)[BPL]) {
#pragma unroll
        for (int b = 0; b < BPL; ++b) {
            const int n = lane + 64 * b;
            const double v = chiT[(size_t)p * NB + min(n, NB - 1)];
            d[b] = n < NB ? v : 0.0;
        }
    };
    // u_n = sum_{p >= 1} chi_{n,p} R_p
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < BPL; ++b) u[a][b] = 0.0;
    for (int p = 1; p < M; ++p) {
        load_chi(p, ch);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double r = Rl[a * M + p];
#pragma unroll
            for (int b = 0; b < BPL; ++b) u[a][b] = fma64(ch[b], r, u[a][b]);
        }
    }
    int64_t acc = 0;
    const double two_m32 = 2.3283064365386962890625e-10;
    // sqrt64 takes no 0: the offset is below the last bit of any bond
    constexpr double kTiny = 1e-300;
    load_chi(1, nx);
    for (int s = 0; s < n_sweeps; ++s) {
        const int64_t k = step0 + s;
#pragma unroll
        for (int b = 0; b < BPL; ++b) {
            l2[b] = fma64(u[0][b], u[0][b], fma64(u[1][b], u[1][b], u[2][b] * u[2][b]));
            l[b] = sqrt64(l2[b] + kTiny);
        }
        for (int pb = 1; pb < M; pb += kMcBatch) {
            const int np = min(kMcBatch, M - pb);
            const int a0 = lane % 3, p0 = pb + lane / 3;
            const bool mine = lane < 3 * np;
            const int pr = mine ? p0 : 1;
            double *slot = Rc + (size_t)a0 * M + pr;
            const double r = *slot;
            const Block4 x = noise_bits(seed, (uint32_t)pr, chain, k, (uint32_t)a0, kTagMC);
            const double u0 = ((double)x.v[0] + 0.5) * two_m32;
            const double delta = sstep[pr] * (2.0 * u0 - 1.0);
            const double thr =
                zeta_l[pr] * delta * (r + 0.5 * delta) - 0.5 * T_star * neg2log_u32(x.v[1]);
            uint64_t taken = 0;
            for (int i = 0; i < np; ++i) {
                const int p = pb + i;
#pragma unroll
                for (int b = 0; b < BPL; ++b) ch[b] = nx[b];
                load_chi(p + 1 < M ? p + 1 : 1, nx);
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const double d = read_lane(delta, 3 * i + a);
                    double sh[BPL], l2n[BPL], ln[BPL], sum = 0.0;
#pragma unroll
                    for (int b = 0; b < BPL; ++b) {
                        sh[b] = ch[b] * d;
                        l2n[b] = fma64(sh[b], fma64(2.0, u[a][b], sh[b]), l2[b]);
                        ln[b] = sqrt64(l2n[b] + kTiny);
                        sum += ln[b] - l[b];
                    }
                    if (wave_total(sum) > read_lane(thr, 3 * i + a)) {
                        taken |= 1ull << (3 * i + a);
#pragma unroll
                        for (int b = 0; b < BPL; ++b) {
                            u[a][b] += sh[b];
                            l2[b] = l2n[b];
                            l[b] = ln[b];
                        }
                    }
                }
            }
            if (mine && ((taken >> lane) & 1)) *slot = r + delta;
            acc += __popcll(taken);
        }
    }
    if (lane == 0) accepted[c] = acc;
}

// The nu -> 0 limit (Sec. VI.A, Eqs. y2-y14), one thread per chain, FP64: the
// inextensible chain in bending units (tau-bar, T-bar), bonds of unit
// length held by tensions.  A step moves bead n by
//   dr_n = (-f_n u^m_n + f_{n+1} u^m_{n+1} + h_{n+1} - h_n) dt + sqrt(2 T-bar dt) eta_n,
// h_n = -(u^m_{n-1} + u^m_{n+1}) the bending gradient, u^m_n = (u_n + u'_n) /
// |u_n + u'_n| the midpoint bonds (Eq. y14); the tensions f_n solve the
// tridiagonal system (u_n + u'_n) . du_n = 0 (Eqs. y11-y13) by the Thomas
// algorithm, and the cycle (midpoint, tensions, u') is repeated from u' = u
// until it converges: at most `iters` times, fewer when tol > 0 and a cycle
// moves no component of u' by more than tol.  Scratch, chain-fastest ([index][chain], coalesced):
// u, u', u^m (3 (N+2) each, bonds 0 and N+1 zero), noise (3 (N+1)), the
// Thomas coefficients c', d' (N each) and f (N+2).  Noise: the bead index
// with tag 3.  The bonds are scaled to unit length on entry.
__global__ __launch_bounds__(64) void wlc_kernel(double *__restrict__ pos,
                                                 double *__restrict__ scr,
                                                 const int32_t *__restrict__ ids, int M, int nch,
                                                 double T_bar, double dt, int iters, double tol,
                                                 int midpoint, uint64_t seed, int64_t step0,
                                                 int n_steps)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nch) return;
    const int N = M - 1;
    const size_t S = (size_t)nch;
    double *U = scr, *UN = U + 3 * (size_t)(N + 2) * S, *UM = UN + 3 * (size_t)(N + 2) * S;
    double *NZ = UM + 3 * (size_t)(N + 2) * S, *CP = NZ + 3 * (size_t)(N + 1) * S;
    double *DP = CP + (size_t)N * S, *F = DP + (size_t)N * S;
#define V3(A, n, a) A[((size_t)3 * (n) + (a)) * S + c]
    double *x = pos + (size_t)c * 3 * M;
    const uint32_t chain = (uint32_t)ids[c];
    const double amp = sqrt(2.0 * T_bar * dt);
    for (int a = 0; a < 3; ++a) {
        V3(U, 0, a) = V3(U, N + 1, a) = 0.0;
        V3(UN, 0, a) = V3(UN, N + 1, a) = 0.0;
        V3(UM, 0, a) = V3(UM, N + 1, a) = 0.0;
    }
    for (int n = 1; n <= N; ++n) {  // bonds, scaled to unit length
        double u[3], s2 = 0.0;
        for (int a = 0; a < 3; ++a) {
            u[a] = x[a * M + n] - x[a * M + n - 1];
            s2 += u[a] * u[a];
        }
        const double inv = s2 > 0.0 ? 1.0 / sqrt(s2) : 0.0;
        for (int a = 0; a < 3; ++a) V3(U, n, a) = u[a] * inv;
    }
    F[0 * S + c] = 0.0;
    F[(size_t)(N + 1) * S + c] = 0.0;
    double r0[3] = {x[0], x[M], x[2 * M]};
    // regular displacement of bead n (bending at the midpoint bonds + noise)
    auto drr = [&](int n, int a) {
        const double hn = n >= 1 ? -(V3(UM, n - 1, a) + V3(UM, n + 1, a)) : 0.0;
        const double hn1 = n + 1 <= N ? -(V3(UM, n, a) + V3(UM, n + 2 <= N + 1 ? n + 2 : N + 1, a))
                                      : 0.0;
        return (hn1 - hn) * dt + V3(NZ, n, a);
    };
    for (int s = 0; s < n_steps; ++s) {
        const int64_t k = step0 + s;
        for (int a = 0; a < 3; ++a)
            for (int q = 0; q <= N / 4; ++q) {
                double z[4];
                normals4_f64(noise_bits(seed, (uint32_t)q, chain, k, (uint32_t)a, kTagWLC), z);
                for (int e = 0; e < 4 && 4 * q + e <= N; ++e) V3(NZ, 4 * q + e, a) = amp * z[e];
            }
        for (int n = 1; n <= N; ++n)
            for (int a = 0; a < 3; ++a) V3(UN, n, a) = V3(U, n, a);
        for (int it = 0; it < iters; ++it) {
            for (int n = 1; n <= N; ++n) {
                double w[3], s2 = 0.0;
                for (int a = 0; a < 3; ++a) {
                    w[a] = V3(U, n, a) + V3(UN, n, a);
                    s2 += w[a] * w[a];
                }
                const double inv = 1.0 / sqrt(s2);
                for (int a = 0; a < 3; ++a) V3(UM, n, a) = midpoint ? w[a] * inv : V3(U, n, a);
            }
            // Thomas forward sweep: a f_{n-1} + b f_n + c f_{n+1} = r
            double cp = 0.0, dp = 0.0;
            for (int n = 1; n <= N; ++n) {
                double wl = 0.0, wm = 0.0, wr = 0.0, wd = 0.0;
                for (int a = 0; a < 3; ++a) {
                    const double w = V3(U, n, a) + V3(UN, n, a);
                    wl += w * V3(UM, n - 1, a);
                    wm += w * V3(UM, n, a);
                    wr += w * V3(UM, n + 1, a);
                    wd += w * (drr(n, a) - drr(n - 1, a));
                }
                const double ca = wl * dt, cb = -2.0 * wm * dt, cc = wr * dt, rr = -wd;
                const double m = n == 1 ? cb : cb - ca * cp;
                cp = cc / m;
                dp = (n == 1 ? rr : rr - ca * dp) / m;
                CP[(size_t)(n - 1) * S + c] = cp;
                DP[(size_t)(n - 1) * S + c] = dp;
            }
            double fn = DP[(size_t)(N - 1) * S + c];
            F[(size_t)N * S + c] = fn;
            for (int n = N - 1; n >= 1; --n) {
                fn = DP[(size_t)(n - 1) * S + c] - CP[(size_t)(n - 1) * S + c] * fn;
                F[(size_t)n * S + c] = fn;
            }
            double change = 0.0;
            for (int n = 1; n <= N; ++n) {
                const double fl = F[(size_t)(n - 1) * S + c], fm = F[(size_t)n * S + c],
                             fr = F[(size_t)(n + 1) * S + c];
                for (int a = 0; a < 3; ++a) {
                    const double v = V3(U, n, a) + (drr(n, a) - drr(n - 1, a)) +
                                     (fl * V3(UM, n - 1, a) - 2.0 * fm * V3(UM, n, a) +
                                      fr * V3(UM, n + 1, a)) * dt;
                    change = fmax(change, fabs(v - V3(UN, n, a)));
                    V3(UN, n, a) = v;
                }
            }
            if (tol > 0.0 && change <= tol) break;
        }
        for (int a = 0; a < 3; ++a) r0[a] += drr(0, a) + F[(size_t)1 * S + c] * V3(UM, 1, a) * dt;
        for (int n = 1; n <= N; ++n)
            for (int a = 0; a < 3; ++a) V3(U, n, a) = V3(UN, n, a);
    }
    for (int a = 0; a < 3; ++a) {
        x[a * M] = r0[a];
        for (int n = 1; n <= N; ++n) x[a * M + n] = x[a * M + n - 1] + V3(U, n, a);
    }
#undef V3
}

// The same step with one wavefront per chain and the chain in LDS: bonds and
// beads are spread over the lanes, and the tension system is solved by
// parallel cyclic reduction (each of ceil(log2 N) rounds eliminates the
// couplings to the rows s apart, s = 1, 2, 4, ...) instead of the serial
// Thomas sweep.  LDS, doubles ([axis][index]): u, u', u^m (3 (N+2) each),
// noise and the regular displacements (3 (N+1) each), two sets of the
// tridiagonal rows a, b, c, r (4 N each) and f (N+2): wlc_lds_doubles(M).
constexpr size_t kWlcMaxLds = 64 * 1024;  // the wave kernel's LDS limit

__host__ __device__ inline size_t wlc_lds_doubles(int M)
{
    const size_t N = (size_t)M - 1;
    return 9 * (N + 2) + 6 * (N + 1) + 8 * N + (N + 2);
}

// Registers for at most 4 wavefronts a SIMD: the LDS (49 KB at 257 beads, the
// shortest) lets no more than 3 chains onto a compute unit, and with the
// compiler's own choice of 5 (93 registers for 113) fewer LDS reads are in
// flight: 1024 chains of 257 beads 1198 us for 4 steps of 8 cycles, 1084 so; of
// 341 beads 1797 and 1621.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 4)))
void wlc_wave_kernel(double *__restrict__ pos, const int32_t *__restrict__ ids, int M,
                     double T_bar, double dt, int iters, double tol, int midpoint, uint64_t seed,
                     int64_t step0, int n_steps)
{
    extern __shared__ double lds[];
    const int c = blockIdx.x, t = threadIdx.x;
    const int N = M - 1, P = N + 2, Q = N + 1;
    double *U = lds, *UN = U + 3 * P, *UM = UN + 3 * P;
    double *NZ = UM + 3 * P, *D = NZ + 3 * Q;
    double *const rows = D + 3 * Q;  // set h: a, b, c, r at rows + (4 h + 0..3) N
    double *F = rows + 8 * (size_t)N;
    double *x = pos + (size_t)c * 3 * M;
    const uint32_t chain = (uint32_t)ids[c];
    const double amp = sqrt(2.0 * T_bar * dt);
    for (int i = t; i < 3 * P; i += 64) U[i] = UN[i] = UM[i] = 0.0;
    for (int i = t; i < P; i += 64) F[i] = 0.0;
    __syncthreads();
    for (int n = 1 + t; n <= N; n += 64) {  // bonds, scaled to unit length
        double u[3], s2 = 0.0;
        for (int a = 0; a < 3; ++a) {
            u[a] = x[a * M + n] - x[a * M + n - 1];
            s2 += u[a] * u[a];
        }
        const double inv = s2 > 0.0 ? 1.0 / sqrt(s2) : 0.0;
        for (int a = 0; a < 3; ++a) U[a * P + n] = u[a] * inv;
    }
    double r0 = t < 3 ? x[t * M] : 0.0;
    const int nq = N / 4 + 1;
    __syncthreads();
    for (int s = 0; s < n_steps; ++s) {
        const int64_t k = step0 + s;
        for (int i = t; i < 3 * nq; i += 64) {
            const int a = i / nq, q = i - a * nq;
            double z[4];
            normals4_f64(noise_bits(seed, (uint32_t)q, chain, k, (uint32_t)a, kTagWLC), z);
            for (int e = 0; e < 4 && 4 * q + e <= N; ++e) NZ[a * Q + 4 * q + e] = amp * z[e];
        }
        for (int n = 1 + t; n <= N; n += 64)
            for (int a = 0; a < 3; ++a) UN[a * P + n] = U[a * P + n];
        __syncthreads();
        for (int it = 0; it < iters; ++it) {
            for (int n = 1 + t; n <= N; n += 64) {  // midpoint bonds
                double w[3], s2 = 0.0;
                for (int a = 0; a < 3; ++a) {
                    w[a] = U[a * P + n] + UN[a * P + n];
                    s2 += w[a] * w[a];
                }
                const double inv = 1.0 / sqrt(s2);
                for (int a = 0; a < 3; ++a) UM[a * P + n] = midpoint ? w[a] * inv : U[a * P + n];
            }
            __syncthreads();
            for (int n = t; n <= N; n += 64)  // regular displacements of the beads
                for (int a = 0; a < 3; ++a) {
                    const double *um = UM + a * P;
                    const double hn = n >= 1 ? -(um[n - 1] + um[n + 1]) : 0.0;
                    const double hn1 = n + 1 <= N ? -(um[n] + um[n + 2]) : 0.0;
                    D[a * Q + n] = (hn1 - hn) * dt + NZ[a * Q + n];
                }
            __syncthreads();
            for (int n = 1 + t; n <= N; n += 64) {  // row n: a f_{n-1} + b f_n + c f_{n+1} = r
                double wl = 0.0, wm = 0.0, wr = 0.0, wd = 0.0;
                for (int a = 0; a < 3; ++a) {
                    const double w = U[a * P + n] + UN[a * P + n];
                    wl += w * UM[a * P + n - 1];
                    wm += w * UM[a * P + n];
                    wr += w * UM[a * P + n + 1];
                    wd += w * (D[a * Q + n] - D[a * Q + n - 1]);
                }
                rows[n - 1] = wl * dt;
                rows[N + n - 1] = -2.0 * wm * dt;
                rows[2 * N + n - 1] = wr * dt;
                rows[3 * N + n - 1] = -wd;
            }
            __syncthreads();
            int h = 0;
            for (int sd = 1; sd < N; sd *= 2, h ^= 1) {
                const double *ra = rows + (size_t)(4 * h) * N, *rb = ra + N, *rc = rb + N,
                             *rr = rc + N;
                double *oa = rows + (size_t)(4 * (h ^ 1)) * N, *ob = oa + N, *oc = ob + N,
                       *od = oc + N;
                for (int j = t; j < N; j += 64) {
                    double an = 0.0, cn = 0.0, bn = rb[j], dn = rr[j];
                    if (j - sd >= 0) {
                        const double al = -ra[j] / rb[j - sd];
                        an = al * ra[j - sd];
                        bn += al * rc[j - sd];
                        dn += al * rr[j - sd];
                    }
                    if (j + sd < N) {
                        const double ga = -rc[j] / rb[j + sd];
                        cn = ga * rc[j + sd];
                        bn += ga * ra[j + sd];
                        dn += ga * rr[j + sd];
                    }
                    oa[j] = an;
                    ob[j] = bn;
                    oc[j] = cn;
                    od[j] = dn;
                }
                __syncthreads();
            }
            for (int j = t; j < N; j += 64)
                F[j + 1] = rows[(size_t)(4 * h + 3) * N + j] / rows[(size_t)(4 * h + 1) * N + j];
            __syncthreads();
            double change = 0.0;
            for (int n = 1 + t; n <= N; n += 64) {  // bond update
                const double fl = F[n - 1], fm = F[n], fr = F[n + 1];
                for (int a = 0; a < 3; ++a) {
                    const double v = U[a * P + n] + (D[a * Q + n] - D[a * Q + n - 1]) +
                                     (fl * UM[a * P + n - 1] - 2.0 * fm * UM[a * P + n] +
                                      fr * UM[a * P + n + 1]) * dt;
                    change = fmax(change, fabs(v - UN[a * P + n]));
                    UN[a * P + n] = v;
                }
            }
            __syncthreads();
            if (tol > 0.0) {  // the same maximum in every lane: a uniform exit
                for (int o = 32; o >= 1; o >>= 1) change = fmax(change, __shfl_xor(change, o));
                if (change <= tol) break;
            }
        }
        if (t < 3) r0 += D[t * Q] + F[1] * UM[t * P + 1] * dt;
        for (int n = 1 + t; n <= N; n += 64)
            for (int a = 0; a < 3; ++a) U[a * P + n] = UN[a * P + n];
        __syncthreads();
    }
    if (t < 3) {
        double v = r0;
        x[t * M] = v;
        for (int n = 1; n <= N; ++n) {
            v += U[t * P + n];
            x[t * M + n] = v;
        }
    }
}

// Chains of up to 256 beads in registers: G = 16, 32 or 64 lanes per chain, four
// consecutive bonds per lane (lane q of the group holds bonds 4q+1 .. 4q+4 and
// draws the noise of beads 4q .. 4q+3, one Philox block per component), so
// most neighbours are in the lane and the others one lane away, by DPP.
//
// The tension rows are scaled to the diagonal -2 (by 1/|w|, w = u + u', in the
// midpoint form, where the couplings become the cosines between midpoint
// bonds, the same for both rows they join; by 1/(w.u) otherwise).  A lane
// eliminates its first three tensions by hand (the first and the third
// without a division), which leaves one tridiagonal row per lane in its
// fourth; those are solved by parallel cyclic reduction over the lanes of
// the group, rows kept at unit diagonal (one reciprocal a round), by DPP row
// shifts where a group is a row of 16 lanes.
//
// Bound by FP64 issue: about 350 vector instructions a lane and cycle, two
// wavefronts a SIMD at 8192 chains of 64 beads, where a step of 8 cycles
// takes 18 us (86 us with one bond per lane: six rounds of reduction over
// the LDS crossbar with two divisions each).
constexpr int kWlcRegMaxM = 256;

// The value of v `S` lanes before (after) this one in its group, else 0;
// gl = lane % G.
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF,
                                                              true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL,
                                                              0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int G, int S = 1>
__device__ __forceinline__ double from_prev(double v, int gl)
{
    if constexpr (G == 16) {
        return lane_shift<0x110 + S>(v);  // row_shr
    } else {
        const double x = S == 1 ? lane_shift<0x138>(v)  // wave_shr:1
                                : __shfl(v, (int)(threadIdx.x & 63) - S, 64);
        return gl >= S ? x : 0.0;
    }
}
template <int G, int S = 1>
__device__ __forceinline__ double from_next(double v, int gl)
{
    if constexpr (G == 16) {
        return lane_shift<0x100 + S>(v);  // row_shl
    } else {
        const double x = S == 1 ? lane_shift<0x130>(v)  // wave_shl:1
                                : __shfl(v, (int)(threadIdx.x & 63) + S, 64);
        return gl + S < G ? x : 0.0;
    }
}

// 1 / x for normal x: one third-order step from the hardware's reciprocal.
__device__ __forceinline__ double rcp64(double x)
{
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma64(-x, y, 1.0);
    return fma64(y, fma64(e, e, e), y);
}

// One round of cyclic reduction at distance S of the rows
// A f_(lane-S) + f_lane + C f_(lane+S) = R.
template <int G, int S>
__device__ __forceinline__ void reduce_rows(double &A, double &C, double &R, int gl)
{
    const double Al = from_prev<G, S>(A, gl), Cl = from_prev<G, S>(C, gl),
                 Rl = from_prev<G, S>(R, gl);
    const double Ar = from_next<G, S>(A, gl), Cr = from_next<G, S>(C, gl),
                 Rr = from_next<G, S>(R, gl);
    const double i = rcp64(fma64(-C, Ar, fma64(-A, Cl, 1.0)));
    R = fma64(-C, Rr, fma64(-A, Rl, R)) * i;
    A = -A * Al * i;
    C = -C * Cr * i;
}

// PAIR: chains of 2 beads, whose one tension has no neighbour: without the
// elimination and the bonds that are not there 1024 of them take 28 us for 4
// steps of 8 cycles, 54 with them (48 with one bond per lane).
template <int G, bool MID, bool PAIR = false>
__global__ __launch_bounds__(256) void wlc_reg_kernel(double *__restrict__ pos,
                                                      const int32_t *__restrict__ ids, int M,
                                                      int nch, double T_bar, double dt, int iters,
                                                      double tol, uint64_t seed, int64_t step0,
                                                      int n_steps)
{
    const int lane = threadIdx.x & 63, gl = lane % G;
    const int c0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * (64 / G);
    if (c0 >= nch) return;  // a whole wavefront
    const int c = c0 + lane / G;
    const bool live = c < nch;
    const int N = PAIR ? 1 : M - 1, nl = (N + 3) / 4;  // lanes that hold bonds
    double *x = pos + (size_t)(live ? c : 0) * 3 * M;
    const uint32_t chain = live ? (uint32_t)ids[c] : 0u;
    const double amp = sqrt(2.0 * T_bar * dt);
    bool bond[4];
    double U[3][4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {  // bonds, scaled to unit length
        const int n = 4 * gl + 1 + m;
        bond[m] = live && n <= N;
        double s2 = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            U[a][m] = bond[m] ? x[a * M + n] - x[a * M + n - 1] : 0.0;
            s2 += U[a][m] * U[a][m];
        }
        const double inv = s2 > 0.0 ? 1.0 / sqrt(s2) : 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) U[a][m] *= inv;
    }
    double r0[3];  // bead 0, in lane 0 of the group
#pragma unroll
    for (int a = 0; a < 3; ++a) r0[a] = live ? x[a * M] : 0.0;
    for (int s = 0; s < n_steps; ++s) {
        const int64_t k = step0 + s;
        // noise of bead 0 and noise differences over the own bonds
        double dz[3][4], z0[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double z[4];
            normals4_f64(noise_bits(seed, (uint32_t)gl, chain, k, (uint32_t)a, kTagWLC), z);
            const double zn = from_next<G>(z[0], gl);
            z0[a] = amp * z[0];
            dz[a][0] = amp * (z[1] - z[0]);
            dz[a][1] = amp * (z[2] - z[1]);
            dz[a][2] = amp * (z[3] - z[2]);
            dz[a][3] = amp * (zn - z[3]);
        }
        double UN[3][4], d0[3] = {0.0, 0.0, 0.0};  // d0: displacement of bead 0
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int m = 0; m < 4; ++m) UN[a][m] = U[a][m];
        bool active = live;  // this chain's cycle has not converged
        for (int it = 0; it < iters; ++it) {
            // midpoint bonds; sc scales the tension rows
            double um[3][4], w[3][4], sc[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                double s2 = 0.0;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    w[a][m] = U[a][m] + UN[a][m];
                    s2 = fma64(w[a][m], MID ? w[a][m] : U[a][m], s2);
                }
                if constexpr (MID) {
                    const double inv = bond[m] ? rsqrt64(s2) : 0.0;
#pragma unroll
                    for (int a = 0; a < 3; ++a) um[a][m] = w[a][m] * inv;
                } else {
                    sc[m] = bond[m] ? rcp64(s2) : 0.0;
#pragma unroll
                    for (int a = 0; a < 3; ++a) um[a][m] = U[a][m];
                }
            }
            // bending gradients h_n = -(u^m_(n-1) + u^m_(n+1)) of the bonds and
            // the differences dd of the regular bead displacements over them
            double ul[3], ur[3], dd[3][4], h1[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                ul[a] = from_prev<G>(um[a][3], gl);
                ur[a] = from_next<G>(um[a][0], gl);
                double h[4];
                h[0] = -(ul[a] + um[a][1]);
                h[1] = -(um[a][0] + um[a][2]);
                h[2] = -(um[a][1] + um[a][3]);
                h[3] = -(um[a][2] + ur[a]);
#pragma unroll
                for (int m = 0; m < 4; ++m) h[m] = bond[m] ? h[m] : 0.0;
                const double hl = from_prev<G>(h[3], gl), hr = from_next<G>(h[0], gl);
                dd[a][0] = fma64(fma64(-2.0, h[0], hl + h[1]), dt, dz[a][0]);
                dd[a][1] = fma64(fma64(-2.0, h[1], h[0] + h[2]), dt, dz[a][1]);
                dd[a][2] = fma64(fma64(-2.0, h[2], h[1] + h[3]), dt, dz[a][2]);
                dd[a][3] = fma64(fma64(-2.0, h[3], h[2] + hr), dt, dz[a][3]);
                h1[a] = h[0];
            }
            // rows av f_(n-1) - 2 f_n + cv f_(n+1) = rv of the tensions times dt
            double av[4], cv[4], rv[4];
            auto dot = [](const double(&p)[3][4], int i, const double(&q)[3][4], int j) {
                return fma64(p[0][i], q[0][j], fma64(p[1][i], q[1][j], p[2][i] * q[2][j]));
            };
            auto dot1 = [](const double(&p)[3][4], int i, const double(&q)[3]) {
                return fma64(p[0][i], q[0], fma64(p[1][i], q[1], p[2][i] * q[2]));
            };
            if constexpr (MID) {
                cv[0] = dot(um, 0, um, 1);
                cv[1] = dot(um, 1, um, 2);
                cv[2] = dot(um, 2, um, 3);
                cv[3] = dot1(um, 3, ur);
                av[0] = from_prev<G>(cv[3], gl);
                av[1] = cv[0];
                av[2] = cv[1];
                av[3] = cv[2];
#pragma unroll
                for (int m = 0; m < 4; ++m) rv[m] = -dot(um, m, dd, m);
            } else {
                av[0] = dot1(w, 0, ul) * sc[0];
                cv[3] = dot1(w, 3, ur) * sc[3];
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    if (m > 0) av[m] = dot(w, m, um, m - 1) * sc[m];
                    if (m < 3) cv[m] = dot(w, m, um, m + 1) * sc[m];
                    rv[m] = -dot(w, m, dd, m) * sc[m];
                }
            }
            double F0, F1 = 0.0, F2 = 0.0, F3 = 0.0, Fl = 0.0, Fr = 0.0;
            if constexpr (PAIR) {
                F0 = -0.5 * rv[0];
            } else {
                // f_m = al + be f_(previous lane's fourth) + ga f_3 for m = 0, 1, 2
                const double i2 = rcp64(fma64(-av[1], cv[0], fma64(-cv[1], av[2], 4.0)));
                const double al1 = -fma64(2.0, rv[1], fma64(av[1], rv[0], cv[1] * rv[2])) * i2;
                const double be1 = av[1] * av[0] * i2, ga1 = cv[1] * cv[2] * i2;
                const double al0 = 0.5 * fma64(cv[0], al1, -rv[0]);
                const double be0 = 0.5 * fma64(cv[0], be1, av[0]), ga0 = 0.5 * (cv[0] * ga1);
                const double al2 = 0.5 * fma64(av[2], al1, -rv[2]);
                const double be2 = 0.5 * (av[2] * be1), ga2 = 0.5 * fma64(av[2], ga1, cv[2]);
                // the fourth row, the next lane's first tension replaced likewise
                const double aln = from_next<G>(al0, gl), ben = from_next<G>(be0, gl),
                             gan = from_next<G>(ga0, gl);
                const double ib = rcp64(fma64(av[3], ga2, fma64(cv[3], ben, -2.0)));
                double A = av[3] * be2 * ib, C = cv[3] * gan * ib;
                F3 = fma64(-av[3], al2, fma64(-cv[3], aln, rv[3])) * ib;
                if (1 < nl) reduce_rows<G, 1>(A, C, F3, gl);
                if (2 < nl) reduce_rows<G, 2>(A, C, F3, gl);
                if (4 < nl) reduce_rows<G, 4>(A, C, F3, gl);
                if (8 < nl) reduce_rows<G, 8>(A, C, F3, gl);
                if constexpr (G > 16) {
                    if (16 < nl) reduce_rows<G, 16>(A, C, F3, gl);
                    if (G > 32 && 32 < nl) reduce_rows<G, 32>(A, C, F3, gl);
                }
                Fl = from_prev<G>(F3, gl);
                F0 = fma64(ga0, F3, fma64(be0, Fl, al0));
                F1 = fma64(ga1, F3, fma64(be1, Fl, al1));
                F2 = fma64(ga2, F3, fma64(be2, Fl, al2));
                Fr = from_next<G>(F0, gl);
            }
            // new bonds
            double change = 0.0;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const double p0 = F0 * um[a][0], p1 = F1 * um[a][1], p2 = F2 * um[a][2],
                             p3 = F3 * um[a][3];
                double v[4];
                v[0] = U[a][0] + dd[a][0] + fma64(-2.0, p0, fma64(Fl, ul[a], p1));
                v[1] = U[a][1] + dd[a][1] + fma64(-2.0, p1, p0 + p2);
                v[2] = U[a][2] + dd[a][2] + fma64(-2.0, p2, p1 + p3);
                v[3] = U[a][3] + dd[a][3] + fma64(-2.0, p3, fma64(Fr, ur[a], p2));
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const double nv = bond[m] && active ? v[m] : UN[a][m];
                    change = fmax(change, fabs(nv - UN[a][m]));
                    UN[a][m] = nv;
                }
                if (active) d0[a] = fma64(h1[a], dt, z0[a]) + p0;
            }
            if (tol > 0.0) {  // the chain's largest change, in every lane of its group
#pragma unroll
                for (int o = G / 2; o >= 1; o >>= 1)
                    change = fmax(change, __shfl_xor(change, o, 64));
                active = active && !(change <= tol);
                if (!__any(active)) break;
            }
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            r0[a] += d0[a];
#pragma unroll
            for (int m = 0; m < 4; ++m) U[a][m] = UN[a][m];
        }
    }
    // positions: the running sums of the bonds, in the lane and then over the
    // lanes of the group
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double p[4];
        p[0] = U[a][0];
        p[1] = p[0] + U[a][1];
        p[2] = p[1] + U[a][2];
        p[3] = p[2] + U[a][3];
        double run = p[3];  // inclusive sum over the lanes
        for (int o = 1; o < G; o *= 2) {
            const double q = __shfl(run, lane - o, 64);
            if (gl >= o) run += q;
        }
        const double before = from_prev<G>(run, gl);
        const double base = __shfl(r0[a], lane - gl, 64);
        if (live) {
            if (gl == 0) x[a * M] = base;
#pragma unroll
            for (int m = 0; m < 4; ++m)
                if (bond[m]) x[a * M + 4 * gl + 1 + m] = base + (before + p[m]);
        }
    }
}

// out[j] = sum_c acc[c][j]: kRedCols columns per workgroup (one 64-byte run of
// every chain's row) and kRedRows chains in flight, each thread with four
// loads outstanding, then a tree over the chain slices in LDS (a fixed order,
// the same sum at every call).  Bound by memory: 12 MB at 4096 chains of 256
// beads.  With one thread per column walking the chains one after the other
// that sum took 985 us there and 369 us on average over the seven lengths of
// an uneven ensemble of 8192 chains, all latency; this form takes 15 us and
// 6 us.
constexpr int kRedCols = 8, kRedRows = 128;
__global__ __launch_bounds__(kRedCols *kRedRows) void reduce_chains_kernel(
    const double *__restrict__ acc, double *__restrict__ out, int width, int nch)
{
    __shared__ double part[kRedRows][kRedCols];
    const int col = threadIdx.x % kRedCols, row = threadIdx.x / kRedCols;
    const int j = blockIdx.x * kRedCols + col;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (j < width) {
        const double *p = acc + j;
        int c = row;
        for (; c + 3 * kRedRows < nch; c += 4 * kRedRows)
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += p[(size_t)(c + e * kRedRows) * width];
        for (; c < nch; c += kRedRows) s[0] += p[(size_t)c * width];
    }
    part[row][col] = (s[0] + s[1]) + (s[2] + s[3]);
    __syncthreads();
#pragma unroll
    for (int h = kRedRows / 2; h >= 1; h /= 2) {
        if (row < h) part[row][col] += part[row + h][col];
        __syncthreads();
    }
    if (row == 0 && j < width) out[j] = part[0][col];
}

template <typename T>
__global__ void check_finite_kernel(const T *__restrict__ x, size_t n, int *flag)
{
    int bad = 0;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        bad |= !isfinite(x[i]);
    if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

inline unsigned blocks_for(size_t n, unsigned t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

hipError_t launch_gemm_f64(const double *A, const double *X, double *Y, int M, int ncol,
                           hipStream_t st, const int64_t *off)
{
    if (M <= 0 || ncol <= 0) return hipSuccess;
    dim3 grid((M + kGemmBM - 1) / kGemmBM, (ncol + kGemmBN - 1) / kGemmBN);
    if (M % kGemmBK == 0) {
        // narrower column tiles while 64 x 64 tiles would not give every CU
        // of the GPU two workgroups
        if (grid.x * grid.y < 512) {
            const dim3 g1(grid.x * ((ncol + 31) / 32));
            hipLaunchKernelGGL(gemm_f64_pipe_kernel<32>, g1, dim3(256), 0, st, A, X, Y, off,
                               M, ncol);
        } else {
            const dim3 g1(grid.x * grid.y);
            hipLaunchKernelGGL(gemm_f64_pipe_kernel<64>, g1, dim3(256), 0, st, A, X, Y, off,
                               M, ncol);
        }
    } else {
        const dim3 g((unsigned)((M + kAnyB - 1) / kAnyB) * ((ncol + kAnyB - 1) / kAnyB));
        hipLaunchKernelGGL(gemm_f64_any_kernel, g, dim3(256), 0, st, A, X, Y, off, M, ncol);
    }
    return hipGetLastError();
}

hipError_t launch_stencil_f64(const double *r, double *F, int M, int nch, double lin,
                              hipStream_t st)
{
    const size_t n = (size_t)nch * M;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(stencil_f64_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, r, F, M,
                       nch, lin);
    return hipGetLastError();
}

hipError_t launch_mode_update_f64(double *R, const double *dH, const double *E, const double *C,
                                  const double *W, const int32_t *ids, int M, int nch,
                                  uint64_t seed, const int64_t *step_dev, int64_t step_off,
                                  double gdt, int nonlinear, hipStream_t st)
{
    const size_t n = (size_t)nch * ((M + 3) / 4);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(mode_update_f64_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, R,
                       dH, E, C, W, ids, M, nch, seed, step_dev, step_off, gdt, nonlinear);
    return hipGetLastError();
}

hipError_t launch_euler_f64(double *pos, const int32_t *ids, int M, int nch, double nu,
                            double dtau, double T_star, double gdt, uint64_t seed, int64_t step0,
                            int n_steps, hipStream_t st)
{
    if (nch == 0 || n_steps == 0) return hipSuccess;
    const int nq = (M + 3) / 4;
    if (nq > 1024) return hipErrorInvalidValue;
    const int threads = ((nq + 63) / 64) * 64;
    const size_t lds = sizeof(double) * 3 * (size_t)M;
    if (lds > 64 * 1024) return hipErrorInvalidValue;  // positions must fit the LDS
    hipLaunchKernelGGL(euler_f64_kernel, dim3(nch), dim3(threads), lds, st, pos, ids, M, nu,
                       dtau, sqrt(2.0 * T_star * dtau), gdt, seed, step0, n_steps);
    return hipGetLastError();
}

size_t wlc_scratch_doubles(int M, int nch)
{
    if (sizeof(double) * wlc_lds_doubles(M) <= kWlcMaxLds) return 0;  // chain held in LDS
    const size_t N = (size_t)M - 1;
    return (9 * (N + 2) + 3 * (N + 1) + 2 * N + (N + 2)) * (size_t)nch;
}

hipError_t launch_wlc(double *pos, double *scr, const int32_t *ids, int M, int nch, double T_bar,
                      double dt, int iters, double tol, int midpoint, uint64_t seed,
                      int64_t step0, int n_steps, hipStream_t st)
{
    if (nch == 0 || n_steps == 0) return hipSuccess;
    if (M < 2 || iters < 1) return hipErrorInvalidValue;
    if (M <= kWlcRegMaxM) {
        const int G = M <= 64 ? 16 : M <= 128 ? 32 : 64, per_wg = 4 * (64 / G);
#define DM_WLC(...)                                                                             \
    hipLaunchKernelGGL((wlc_reg_kernel<__VA_ARGS__>), dim3((nch + per_wg - 1) / per_wg), dim3(256), 0, \
                       st, pos, ids, M, nch, T_bar, dt, iters, tol, seed, step0, n_steps)
        if (M == 2) {
            if (midpoint) DM_WLC(16, true, true);
            else DM_WLC(16, false, true);
        } else if (midpoint) {
            if (G == 16) DM_WLC(16, true);
            else if (G == 32) DM_WLC(32, true);
            else DM_WLC(64, true);
        } else {
            if (G == 16) DM_WLC(16, false);
            else if (G == 32) DM_WLC(32, false);
            else DM_WLC(64, false);
        }
#undef DM_WLC
        return hipGetLastError();
    }
    const size_t lds = sizeof(double) * wlc_lds_doubles(M);
    if (lds <= kWlcMaxLds) {
        hipLaunchKernelGGL(wlc_wave_kernel, dim3(nch), dim3(64), lds, st, pos, ids, M, T_bar, dt,
                           iters, tol, midpoint, seed, step0, n_steps);
        return hipGetLastError();
    }
    if (!scr) return hipErrorInvalidValue;
    hipLaunchKernelGGL(wlc_kernel, dim3((nch + 63) / 64), dim3(64), 0, st, pos, scr, ids, M, nch,
                       T_bar, dt, iters, tol, midpoint, seed, step0, n_steps);
    return hipGetLastError();
}

hipError_t launch_mc(double *R, const double *chiT, const double *sstep, const double *zeta_l,
                     const int32_t *ids, int M, int nch, double T_star, uint64_t seed,
                     int64_t step0, int n_sweeps, int64_t *accepted, hipStream_t st)
{
    if (nch == 0 || n_sweeps == 0) return hipSuccess;
    const size_t lds = sizeof(double) * 3 * (size_t)M;
    if (M < 2 || M > kMcMaxM) return hipErrorInvalidValue;
    const int per_lane = (M - 1 + 63) / 64;
#define DM_MC(B)                                                                               \
    hipLaunchKernelGGL(mc_kernel<B>, dim3(nch), dim3(64), lds, st, R, chiT, sstep, zeta_l, ids, \
                       M, T_star, seed, step0, n_sweeps, accepted)
    if (per_lane <= 1) DM_MC(1);
    else if (per_lane <= 2) DM_MC(2);
    else if (per_lane <= 3) DM_MC(3);
    else if (per_lane <= 4) DM_MC(4);
    else if (per_lane <= 6) DM_MC(6);
    else if (per_lane <= 8) DM_MC(8);
    else if (per_lane <= 12) DM_MC(12);
    else if (per_lane <= 16) DM_MC(16);
    else DM_MC(22);
#undef DM_MC
    return hipGetLastError();
}

hipError_t launch_chain_obs(const double *pos, const double *R, double *obs, double *m2,
                            double *acc, const double *cm0, double *tstate, double *tlast,
                            const int64_t *step_dev, double *ring, double *ccount, int K, int M,
                            int nch, int accumulate, hipStream_t st)
{
    if (nch == 0) return hipSuccess;
    hipLaunchKernelGGL(chain_obs_kernel, dim3(nch), dim3(64), 0, st, pos, R, obs, m2, acc, cm0,
                       tstate, tlast, step_dev, ring, ccount, K, M, accumulate);
    return hipGetLastError();
}

hipError_t launch_reduce_chains(const double *acc, double *out, int width, int nch,
                                hipStream_t st)
{
    hipLaunchKernelGGL(reduce_chains_kernel, dim3(blocks_for(width, kRedCols)),
                       dim3(kRedCols * kRedRows), 0, st, acc, out, width, nch);
    return hipGetLastError();
}

hipError_t launch_check_finite_f64(const double *x, size_t n, int *flag, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    unsigned b = blocks_for(n, 256);
    if (b > 2048) b = 2048;
    hipLaunchKernelGGL(check_finite_kernel<double>, dim3(b), dim3(256), 0, st, x, n, flag);
    return hipGetLastError();
}

hipError_t launch_check_finite_f32(const float *x, size_t n, int *flag, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    unsigned b = blocks_for(n, 256);
    if (b > 2048) b = 2048;
    hipLaunchKernelGGL(check_finite_kernel<float>, dim3(b), dim3(256), 0, st, x, n, flag);
    return hipGetLastError();
}

}  // namespace dm
