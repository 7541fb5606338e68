// dm_modes64.hip -- FP64 mode stepper: a workgroup keeps a tile of chains in
// its LDS and registers and runs all steps of a launch (gfx950).
//
// Each step is the one of the reduced-precision stepper, in FP64 throughout:
//   u = chi R, g_n = u_n (1/|u_n| - (1-2nu)), Delta H = chi^T g,
//   R <- E R + C Delta H + W eta (+ shear)          (Eqs. e5, e4, e11, d3, d6, f2, btum)
// with chi_{n,p} = phi_{n,p} - phi_{n-1,p} = sigma_p sin(p n pi/M),
// sigma_p = -2 sqrt(2/M) sin(p pi/2M), and its mirror symmetry
// chi_{M-n,p} = (-1)^{p+1} chi_{n,p}: for half-bond rows b = n - 1 < H = M/2
//   S_b = sum_{p odd} chi R_p, A_b = sum_{p even} chi R_p,
//   u_{b+1} = S + A, u_{M-1-b} = S - A,
//   Delta H_{p odd} = sum_b chi (g + g'), Delta H_{p even} = sum_b chi (g - g')
// (the middle bond of an even chain, its own mirror, enters g + g' twice: its
// column of the coupling table is halved).  Half the matrix products of the
// dense form, no pass over HBM inside a launch, one launch for all steps.
//
// What bounds it: FP64 matrix products and vector work share the FP64 units
// of a SIMD (78.6 TFLOP/s either way), so a step costs the products of u =
// chi R (3 M^2 flops per chain), those of the coupled mode tiles and the
// noise in series.  At 4096 chains of 256 beads and dtau = 100 (4 of 8 mode
// tiles coupled) a step takes 23.6 us: noise and update 5.1, measured alone,
// the products 10.2 + 5.1 at that rate, and 3.2 for bond forces, operand reads
// and barriers.
//
// Tiles.  The columns of every product are (chain, component) pairs, 16 to a
// v_mfma_f64_16x16x4_f64.
//   NT = 3: 16 chains, one column tile per component (up to 256 beads).  A lane holds x, y, z
//     of a bond, so bond lengths are lane-local, and each table fragment
//     serves 48 columns.  The amplitudes and the forces share one LDS buffer
//     (98 KB at M = 256).
//   NT = 1: 5 chains, column 3 chain + component (the last is unused); bond
//     lengths are summed over three lanes by DPP.  For launches that would
//     leave compute units idle at 16 chains per workgroup, and for chains of
//     258..513 beads, whose 16-chain state does not fit the LDS.
// Wavefront w owns mode tile T = w, w + P, ... (32 modes: 16 odd, 16 even)
// and half-bond row tile I = w, w + P, ....
//
// Orders.  A result tile has row l/16 + 4 r, column l%16 in lane l, element r.
// Row i of a table tile stands for index 16 T + 4 (i % 4) + i / 4, so lane
// group g = l/16 holds the four consecutive indices 4 g + r.  Slot j stands
// for the odd mode 2 j + 1 and the even mode 2 j + 2 (the centre of mass, p =
// 0, takes no part in the products and is kept apart), so a lane holds the
// modes 32 T + 8 g + 1 .. + 8: two Philox blocks per component but for the
// last mode, whose normal is the first one of the next lane group or, for the
// last group, of the next mode tile (exchanged through LDS; where an odd chain
// fills its tiles, the last tile draws that block too).  The products run over K slab pairs q of 8 indices; lane group g
// supplies 8 q + 2 g + e for the product e = 0, 1, so both operands are read
// as 16-byte pairs, and the LDS buffers [parity][t][index/2][column][2] give
// every wavefront read one contiguous kilobyte.
#include "dm_modes64.h"

#include <algorithm>
#include <cmath>

#include "dm_internal.h"
#include "dm_rng.h"

namespace dm {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

constexpr int kSmallTile = 5, kLargeTile = 16;  // chains of NT = 1 and NT = 3

struct Item64 {
    int bucket, tile;
};

struct Launch64 {
    const Modes64Args *buckets;  // null: `one` for every item
    const Item64 *items;         // null: item i is tile i of `one`
    Modes64Args one;
    const int64_t *step;         // added to step0 when non-null
    int64_t step0;
    uint64_t seed;
    int n_steps, nonlinear;
};

inline __host__ __device__ int half_tiles(int M) { return modes64_half_tiles(M); }

// Lane moves inside a 16-lane row, out-of-row sources read 0 (row_shl:n gives
// lane i the value of lane i + n).
template <int CTRL>
__device__ __forceinline__ double dpp64(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo =
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, true);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// The same, 0 in lanes whose mask is 0 (otherwise ~0), whatever the source holds.
template <int CTRL>
__device__ __forceinline__ double dpp64_masked(double v, uint32_t mask)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo =
        mask & (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, true);
    const uint32_t hi = mask & (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32),
                                                                    CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
constexpr int kShl1 = 0x101, kShl2 = 0x102, kShr1 = 0x111, kShr2 = 0x112;

// Sum over the three component lanes of this lane's chain, in one order for
// all three (alpha = column % 3).
__device__ __forceinline__ double chain_sum(double v, int alpha)
{
    const double s = v + dpp64<kShl1>(v) + dpp64<kShl2>(v);  // complete at alpha == 0
    const double s1 = dpp64<kShr1>(s), s2 = dpp64<kShr2>(s);
    return alpha == 0 ? s : (alpha == 1 ? s1 : s2);
}

// One mirror pair of 16-row products: odd and even accumulators of NT column
// tiles over Q slab pairs.  X: fragments [q][parity][lane]; B: LDS operands,
// [parity][t] at stride bs, [q][lane] inside.  The fragments, from L2, are
// loaded two slab pairs ahead; the LDS operands two ahead for one column tile,
// and for three each as soon as its products have issued, the other tiles'
// products (512 cycles) covering the read (two buffers spill).
// x holds the first two fragments pairs of each parity on entry (first_pairs).
__device__ __forceinline__ void first_pairs(const f64x2 *__restrict__ X, f64x2 (&x)[2][2])
{
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int par = 0; par < 2; ++par) x[k][par] = X[(size_t)(2 * k + par) * 64];
}
template <int NT>
__device__ __forceinline__ void mirror_product(const f64x2 *__restrict__ X, f64x2 (&x)[2][2],
                                               const f64x2 *B, int bs, int Q, f64x4 (&so)[NT],
                                               f64x4 (&se)[NT])
{
    constexpr int KB = NT == 1 ? 2 : 1;
    f64x2 b[KB][2][NT];
    auto load_x = [&](int k, int q) {
#pragma unroll
        for (int par = 0; par < 2; ++par) x[k][par] = X[(size_t)(2 * q + par) * 64];
    };
    auto load_b = [&](int k, int t, int q) {
#pragma unroll
        for (int par = 0; par < 2; ++par) b[k][par][t] = B[(par * NT + t) * bs + q * 64];
    };
#pragma unroll
    for (int t = 0; t < NT; ++t) so[t] = se[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < KB; ++k)
#pragma unroll
        for (int t = 0; t < NT; ++t) load_b(k, t, k);
    for (int q = 0; q < Q; q += 2) {  // Q is even
#pragma unroll
        for (int k = 0; k < 2; ++k) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    so[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[k][0][e], b[k % KB][0][t][e],
                                                                 so[t], 0, 0, 0);
                    se[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[k][1][e], b[k % KB][1][t][e],
                                                                 se[t], 0, 0, 0);
                }
                load_b(k % KB, t, min(q + k + KB, Q - 1));
            }
            load_x(k, min(q + k + 2, Q - 1));
        }
    }
}

// The same for one column tile with all fragments in registers (QH >= Q).
template <int QH>
__device__ __forceinline__ void held_product(const f64x2 (&x)[QH][2], const f64x2 *B, int bs, int Q,
                                             f64x4 &so, f64x4 &se)
{
    constexpr int D = QH > 4 ? 2 : QH;  // operands read ahead
    f64x2 b[D][2];
#pragma unroll
    for (int q = 0; q < D; ++q)
#pragma unroll
        for (int par = 0; par < 2; ++par) b[q][par] = B[par * bs + min(q, Q - 1) * 64];
    so = se = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < QH; ++q)
        if (q < Q) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                so = __builtin_amdgcn_mfma_f64_16x16x4f64(x[q][0][e], b[q % D][0][e], so, 0, 0, 0);
                se = __builtin_amdgcn_mfma_f64_16x16x4f64(x[q][1][e], b[q % D][1][e], se, 0, 0, 0);
            }
            if (q + D < QH)
#pragma unroll
                for (int par = 0; par < 2; ++par)
                    b[q % D][par] = B[par * bs + min(q + D, Q - 1) * 64];
        }
}

// Workgroup barrier for the LDS exchanges that leaves the fragment loads in
// flight (__syncthreads() waits for every outstanding vector memory load).
__device__ __forceinline__ void lds_barrier()
{
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0) alone
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// NOISE: wavefronts RT .. P - 1 draw the normals, one step ahead, for the
// others (RT <= 4): in a launch with a tile or less per compute unit the step is
// a chain of latencies, and the FP64 noise of a wavefront's own modes is a
// third of it (3.2 -> 2.6 us per step of one chain of 64 beads).
// There the fragments of both products stay in registers too (QH slab pairs;
// 0: streamed, the first two pairs of a product in flight across the barrier
// before it).
// ODD: some chain's last mode needs the block beyond its tiles.
// LEAN: 128 registers, for two workgroups of 8 wavefronts on a compute unit.
template <int NT, int P, int NU, bool NOISE, bool ODD, int QH, bool LEAN = false>
__global__ __launch_bounds__(64 * P, LEAN ? 4 : 1) void modes64_kernel(Launch64 la)
{
    static_assert(!NOISE || (NT == 1 && NU == 1), "noise wavefronts: one small tile");
    extern __shared__ double lds[];
    const Item64 it = la.items ? la.items[blockIdx.x] : Item64{0, (int)blockIdx.x};
    const Modes64Args a = la.buckets ? la.buckets[it.bucket] : la.one;
    const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int M = a.M, H = M / 2, RT = half_tiles(M), Hp = 16 * RT, Q = 2 * RT;
    const int bs = Hp * 8;  // f64x2 of one (parity, column tile) buffer
    double *cf = lds;                                  // [E, C, W][parity][Hp]
    const bool beyond = ODD && 32 * RT < M;  // the last mode's normal is one block further
    double *r0 = cf + 6 * Hp;         // centre of mass: [t][column]
    double *cz = r0 + 16 * NT;        // normal 0 of every lane: [t][T][lane]
    f64x2 *Rb = reinterpret_cast<f64x2 *>(cz + NT * 64 * (RT + 1));  // [parity][t][index/2][column]
    f64x2 *Gb = NT == 1 ? Rb + 2 * bs : Rb;            // [sum, difference][t][index/2][column]
    double *zb = reinterpret_cast<double *>(Gb + 2 * bs);  // NOISE: [step parity][T][8][lane]
    const int zs = (RT + 1) * 512;                         // of one step parity
    for (int i = threadIdx.x; i < 6 * Hp; i += 64 * P) {
        const int kind = i / (2 * Hp), par = (i / Hp) % 2, p = 2 * (i % Hp) + 1 + par;
        const double *src = kind == 0 ? a.E : kind == 1 ? a.C : a.W;
        cf[i] = p < M ? src[p] : 0.0;
    }
    const double W0 = a.W[0];
    // chain and component of this lane's column(s)
    const int alpha = NT == 1 ? col % 3 : 0;
    const int j = NT == 1 ? kSmallTile * it.tile + col / 3 : kLargeTile * it.tile + col;
    const bool valid = j < a.n && (NT == 3 || col < 15);
    const uint32_t chain = valid ? (uint32_t)a.ids[j] : 0u;
    double *Rj = a.R + (size_t)3 * M * (valid ? j : 0);
    const f64x2 *X1 = reinterpret_cast<const f64x2 *>(a.X) + lane;
    const f64x2 *X2 = X1 + (size_t)RT * Q * 128;

    // amplitudes of the own mode tiles: [parity odd, even][component][r]
    double R[NU][2][NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const size_t row = (size_t)(NT == 1 ? alpha : t) * M;
        if (wave == 0 && g == 0) r0[16 * t + col] = valid ? Rj[row] : 0.0;
#pragma unroll
        for (int ii = 0; ii < NU; ++ii)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int par = 0; par < 2; ++par) {
                    const int p = 32 * (wave + P * ii) + 8 * g + 2 * r + 1 + par;
                    R[ii][par][t][r] = valid && p < M ? Rj[row + p] : 0.0;
                }
    }
    // values v[r] of index tile T into a buffer
    auto put = [&](f64x2 *buf, int par, int t, int T, const double (&v)[4]) {
        f64x2 *d = buf + (par * NT + t) * bs + (8 * T + 2 * g) * 16 + col;
        d[0] = f64x2{v[0], v[1]};
        d[16] = f64x2{v[2], v[3]};
    };
    auto put_state = [&]() {
#pragma unroll
        for (int ii = 0; ii < NU; ++ii) {
            const int T = wave + P * ii;
            if (T < RT)
#pragma unroll
                for (int par = 0; par < 2; ++par)
#pragma unroll
                    for (int t = 0; t < NT; ++t) put(Rb, par, t, T, R[ii][par][t]);
        }
    };
    // noise wavefronts: half h of the normals of mode tile T at step k
    auto draw_ahead = [&](int64_t k, int buf) {
        for (int u = wave - RT; u < 2 * RT + (beyond ? 1 : 0); u += P - RT) {
            const int T = u >> 1, h = u & 1;
            double z[4];
            normals4_f64(noise_bits(la.seed, (uint32_t)(8 * T + 2 * g + h), chain, k,
                                    (uint32_t)alpha, kTagMode),
                         z);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                zb[buf * zs + (T * 8 + 4 * h + e) * 64 + lane] = z[e];
        }
    };
    const int64_t k0 = la.step0 + (la.step ? *la.step : 0);
    if (la.nonlinear) put_state();
    if constexpr (NOISE) {
        if (wave >= RT && la.n_steps > 0) draw_ahead(k0, 0);
    }
    [[maybe_unused]] f64x2 x1[2][2], x2[2][2], h1[QH > 0 ? QH : 1][2], h2[QH > 0 ? QH : 1][2];
    if (wave < RT && la.nonlinear) {
        if constexpr (QH > 0) {
#pragma unroll
            for (int q = 0; q < QH; ++q)
#pragma unroll
                for (int par = 0; par < 2; ++par) {
                    const size_t i = ((size_t)wave * Q + min(q, Q - 1)) * 128 + 64 * par;
                    h1[q][par] = X1[i];
                    h2[q][par] = X2[i];
                }
        } else {
            first_pairs(X1 + (size_t)wave * Q * 128, x1);
        }
    }
    __syncthreads();

    for (int s = 0; s < la.n_steps; ++s) {
        const int64_t k = k0 + s;
        // ---- bonds of the own half-bond rows and their forces
        double Gs[NT][4], Gd[NT][4];
        if (la.nonlinear) {
#pragma unroll
            for (int ii = 0; ii < NU; ++ii) {
                const int I = wave + P * ii;
                if (I >= RT) continue;
                f64x4 so[NT], se[NT];
                if constexpr (QH > 0) {
                    held_product(h1, Rb + lane, bs, Q, so[0], se[0]);
                } else {
                    if (ii > 0) first_pairs(X1 + (size_t)I * Q * 128, x1);
                    mirror_product<NT>(X1 + (size_t)I * Q * 128, x1, Rb + lane, bs, Q, so, se);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    // rows and columns of padding have u = 0: a small number
                    // under their root (a true bond of length 0 gives NaN)
                    const double pad = valid && 16 * I + 4 * g + r < H ? 0.0 : 1e-300;
                    // |u|^2 = (x^2 + y^2) + z^2 with rounded squares in either
                    // tile: a chain's bits do not depend on its tile
                    double up[NT], um[NT], vp[NT], vm[NT], qp, qm;
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        up[t] = so[t][r] + se[t][r];
                        um[t] = so[t][r] - se[t][r];
                        vp[t] = fma64(up[t], up[t], pad);
                        vm[t] = fma64(um[t], um[t], pad);
                    }
                    if constexpr (NT == 1) {
                        qp = chain_sum(vp[0], alpha);
                        qm = chain_sum(vm[0], alpha);
                        if (!valid) qp = qm = 1.0;
                    } else {
                        qp = (vp[0] + vp[1]) + vp[2];
                        qm = (vm[0] + vm[1]) + vm[2];
                    }
                    const double fp = rsqrt64(qp) - a.lin, fm = rsqrt64(qm) - a.lin;
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const double gm = um[t] * fm;
                        Gs[t][r] = fma64(up[t], fp, gm);
                        Gd[t][r] = fma64(up[t], fp, -gm);
                    }
                }
                if constexpr (NT == 1) {
                    put(Gb, 0, 0, I, Gs[0]);
                    put(Gb, 1, 0, I, Gd[0]);
                }
            }
        }
        if constexpr (NT == 3) {
            static_assert(NT == 1 || NU == 1, "the forces of one row tile stay in registers");
            if (la.nonlinear) {
                lds_barrier();  // every wavefront has read the amplitudes
                if (wave < RT)
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        put(Gb, 0, t, wave, Gs[t]);
                        put(Gb, 1, t, wave, Gd[t]);
                    }
            }
        }
        // ---- E R + W eta (+ shear) of the own modes: the normals of a Philox
        // block as they come (z of block h; normal 0 of the first belongs to
        // the lane group before, the last even mode takes its own below)
        if (a.gdt != 0.0) {  // the x amplitudes drift with R^y before its update
            // (opaque: a select of 0 costs two moves more at every use, and a
            // mask held through the step a register that spills)
            [[maybe_unused]] uint32_t xmask = alpha == 0 ? ~0u : 0u;
            if constexpr (NT == 1) asm("" : "+v"(xmask) : "s"(s));
#pragma unroll
            for (int ii = 0; ii < NU; ++ii)
#pragma unroll
                for (int par = 0; par < 2; ++par)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if constexpr (NT == 1) {
                            // (masked, not scaled by 0: the lane after a
                            // chain's z is the next chain's x, which may be NaN)
                            const double y =
                                dpp64_masked<kShl1>(R[ii][par][0][r], xmask);
                            R[ii][par][0][r] = fma64(a.gdt, y, R[ii][par][0][r]);
                        } else {
                            R[ii][par][0][r] = fma64(a.gdt, R[ii][par][1][r], R[ii][par][0][r]);
                        }
                    }
        }
        auto update = [&](int ii, int T, int t, int h, const double (&z)[4]) {
            const double *Eo = cf + 16 * T + 4 * g, *Ee = Eo + Hp;
            const double *Wo = Eo + 4 * Hp, *We = Eo + 5 * Hp;
            double(&o)[4] = R[ii][0][t];
            double(&e)[4] = R[ii][1][t];
            if (h == 0) {
                o[0] = fma64(Eo[0], o[0], Wo[0] * z[1]);
                e[0] = fma64(Ee[0], e[0], We[0] * z[2]);
                o[1] = fma64(Eo[1], o[1], Wo[1] * z[3]);
            } else {
                e[1] = fma64(Ee[1], e[1], We[1] * z[0]);
                o[2] = fma64(Eo[2], o[2], Wo[2] * z[1]);
                e[2] = fma64(Ee[2], e[2], We[2] * z[2]);
                o[3] = fma64(Eo[3], o[3], Wo[3] * z[3]);
                e[3] *= Ee[3];
            }
        };
        if constexpr (!NOISE) {
#pragma unroll
            for (int ii = 0; ii < NU; ++ii) {
                const int T = wave + P * ii;
                if (T >= RT) continue;
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const uint32_t comp = (uint32_t)(NT == 1 ? alpha : t);
                    double first = 0.0;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        double z[4];
                        normals4_f64(noise_bits(la.seed, (uint32_t)(8 * T + 2 * g + h), chain, k,
                                                comp, kTagMode),
                                     z);
                        if (h == 0) first = z[0];
                        update(ii, T, t, h, z);
                    }
                    // (written after the updates: an LDS write between them
                    // keeps every coefficient read above it in registers)
                    cz[(t * (RT + 1) + T) * 64 + lane] = first;
                }
            }
            if (ODD && beyond && wave == (RT - 1) % P) {
#pragma unroll 1
                for (int t = 0; t < NT; ++t) {
                    double z[2];
                    normal_pair_f64(noise_bits(la.seed, (uint32_t)(8 * RT), chain, k,
                                               (uint32_t)(NT == 1 ? alpha : t), kTagMode),
                                    0, z);
                    cz[(t * (RT + 1) + RT) * 64 + lane] = z[0];
                }
            }
        } else {
            if (wave >= RT && s + 1 < la.n_steps) draw_ahead(k + 1, (s + 1) & 1);
        }
        if constexpr (QH == 0) {
            if (la.nonlinear && wave < a.jc) first_pairs(X2 + (size_t)wave * Q * 128, x2);
        }
        lds_barrier();  // forces and normals 0 written (NT = 1: and the amplitudes read)
        if (wave == P - 1 && lane < 16) {  // centre of mass: a free walk, drift from R_0^y
            double v[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const double z0 = NOISE ? zb[(s & 1) * zs + lane] : cz[t * (RT + 1) * 64 + lane];
                v[t] = fma64(W0, z0, r0[16 * t + lane]);
            }
            if constexpr (NT == 1) {
                // (0 times its own coordinate for y and z, not the next lane's,
                // which may be another chain's)
                v[0] = fma64(alpha == 0 ? a.gdt : 0.0, r0[alpha == 0 && lane < 15 ? lane + 1 : lane],
                             v[0]);
            } else {
                v[0] = fma64(a.gdt, r0[16 + lane], v[0]);
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) r0[16 * t + lane] = v[t];
        }
        // ---- the last even mode's normal, and the coupling of the own modes
#pragma unroll
        for (int ii = 0; ii < NU; ++ii) {
            const int T = wave + P * ii;
            if (T >= RT) continue;
            if constexpr (NOISE) {
                const double *zp = zb + (s & 1) * zs + T * 512 + lane;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    double z[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) z[e] = zp[64 * (4 * h + e)];
                    update(ii, T, 0, h, z);
                }
            }
            // normal 0 of lane group g + 1, or of the next tile's group 0
            const double w3 = cf[5 * Hp + 16 * T + 4 * g + 3];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                double zl;
                if constexpr (NOISE) {
                    const int l = T * 512 + (g < 3 ? lane + 16 : 512 + col);
                    zl = T + 1 < RT || beyond || g < 3 ? zb[(s & 1) * zs + l] : 0.0;
                } else {
                    const int l = T * 64 + lane + 16;
                    zl = T + 1 < RT || beyond || g < 3 ? cz[t * (RT + 1) * 64 + l] : 0.0;
                }
                R[ii][1][t][3] = fma64(w3, zl, R[ii][1][t][3]);
            }
            if (la.nonlinear && T < a.jc) {
                f64x4 so[NT], se[NT];
                if constexpr (QH > 0) {
                    held_product(h2, Gb + lane, bs, Q, so[0], se[0]);
                } else {
                    if (ii > 0) first_pairs(X2 + (size_t)T * Q * 128, x2);
                    mirror_product<NT>(X2 + (size_t)T * Q * 128, x2, Gb + lane, bs, Q, so, se);
                }
                const double *Co = cf + 2 * Hp + 16 * T + 4 * g, *Ce = Co + Hp;
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        R[ii][0][t][r] = fma64(Co[r], so[t][r], R[ii][0][t][r]);
                        R[ii][1][t][r] = fma64(Ce[r], se[t][r], R[ii][1][t][r]);
                    }
            }
        }
        if (la.nonlinear) {
            if constexpr (QH == 0) {
                if (wave < RT) first_pairs(X1 + (size_t)wave * Q * 128, x1);
            }
            if constexpr (NT == 3) lds_barrier();  // every wavefront has read the forces
            put_state();
        }
        lds_barrier();  // amplitudes written, normals 0 read
    }
    if (!valid) return;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const size_t row = (size_t)(NT == 1 ? alpha : t) * M;
        if (wave == 0 && g == 0) Rj[row] = r0[16 * t + col];
#pragma unroll
        for (int ii = 0; ii < NU; ++ii)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int par = 0; par < 2; ++par) {
                    const int p = 32 * (wave + P * ii) + 8 * g + 2 * r + 1 + par;
                    if (p < M) Rj[row + p] = R[ii][par][t][r];
                }
    }
}

__global__ __launch_bounds__(256) void modes64_table_kernel(double *__restrict__ X, int M)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < modes64_table_bytes(M) / sizeof(double)) X[i] = modes64_table_value(i, M);
}

// Kernel shapes, and the smallest that holds a chain length at NT = 1 (with
// noise wavefronts where the launch leaves compute units to spare).
enum { kS1n2, kS1n4, kS1x2, kS1x4, kS1x8, kS1x8b, kS1x8l, kS3x2, kS3x4, kS3x8, kShapes };
int small_shape(int M, bool noise)
{
    const int RT = half_tiles(M);
    if (noise && RT <= 4) return RT <= 2 ? kS1n2 : kS1n4;
    return RT <= 2 ? kS1x2 : RT <= 4 ? kS1x4 : RT <= 8 ? kS1x8 : kS1x8b;
}
// 5-chain tiles of 130 to 256 beads (of odd lengths with their last mode inside
// the tiles) share a compute unit in pairs where a launch has more tiles than
// units: 1285 to 2560 chains of 160 beads 11.2 to 12.0 us a step against 14.0 to
// 14.6, of 256 beads 21.4 to 22.8 against 23.1 to 24.0.  A tile with a unit to
// itself is 3 to 4 % faster with the registers it likes (7.1 against 7.4).
int paired_shape(int shape, bool odd, int nitems, int ncu)
{
    return shape == kS1x8 && !odd && nitems > ncu ? kS1x8l : shape;
}
constexpr int kLargeMaxM = 256;  // RT <= 8: one row tile per wavefront

// Whether the normal of the chain's last mode lies in the block beyond its
// mode tiles.
bool beyond_tiles(int M) { return 32 * half_tiles(M) < M; }

size_t lds_bytes(int shape, int M)
{
    const size_t Hp = 16 * (size_t)half_tiles(M);
    const size_t nt = shape >= kS3x2 ? 3 : 1, bufs = shape >= kS3x2 ? 6 : 4;
    return sizeof(double) *
           (6 * Hp + nt * 16 + nt * 4 * (Hp + 16) + bufs * Hp * 16 + (shape <= kS1n4 ? 64 * (Hp + 16) : 0));
}
int tile_chains(int shape) { return shape >= kS3x2 ? kLargeTile : kSmallTile; }
int large_shape(int M)
{
    const int RT = half_tiles(M);
    return RT <= 2 ? kS3x2 : RT <= 4 ? kS3x4 : kS3x8;
}

// 16-chain tiles where their rounds over the compute units take less time.
// Above 4 row tiles a 16-chain workgroup fills a compute unit and takes the
// time of about 2.6 5-chain ones one after another (it reads each table
// fragment once for 48 columns).  Up to 4, several 5-chain workgroups share a
// compute unit, so their time grows with the chains (microseconds per step
// and 1000 chains), and a 16-chain workgroup's is its own (two share one at
// RT <= 2), both measured on 256 compute units: at 4096 x 128 16.1 against 12.8
// us, at 8192 x 64 11.5 against 8.9, but at 3000 x 128 12.2 against 12.6.
bool large_tiles_pay(int M, int n, int ncu)
{
    const int RT = half_tiles(M);
    if (M > kLargeMaxM || beyond_tiles(M)) return false;
    const int w3 = (n + kLargeTile - 1) / kLargeTile, w1 = (n + kSmallTile - 1) / kSmallTile;
    const int r3 = (w3 + ncu - 1) / ncu, r1 = (w1 + ncu - 1) / ncu;
    if (RT > 4) return 2.6 * r3 < (double)r1;
    static const double small_us[4] = {0.7, 1.4, 2.9, 4.0}, large_us[4] = {5.7, 8.8, 10.3, 12.7};
    return large_us[RT - 1] * (RT <= 2 ? (r3 + 1) / 2 : r3) <
           small_us[RT - 1] * 1e-3 * n * 256.0 / ncu;
}

hipError_t launch_shape(int shape, bool odd, size_t lds, int nitems, const Launch64 &la,
                        hipStream_t st)
{
    if (nitems <= 0 || la.n_steps <= 0) return hipSuccess;
    switch (shape + (odd ? kShapes : 0)) {
#define DM_M64(SHAPE, NT, P, NU, ...)                                                      \
    case SHAPE:                                                                            \
        hipLaunchKernelGGL((modes64_kernel<NT, P, NU, __VA_ARGS__>), dim3(nitems),         \
                           dim3(64 * P), lds, st, la);                                     \
        break
        DM_M64(kS1n2, 1, 8, 1, true, false, 4);
        DM_M64(kS1n4, 1, 8, 1, true, false, 8);
        DM_M64(kS1x2, 1, 2, 1, false, false, 0);
        DM_M64(kS1x4, 1, 4, 1, false, false, 0);
        DM_M64(kS1x8, 1, 8, 1, false, false, 0);
        DM_M64(kS1x8b, 1, 8, 2, false, false, 0);
        DM_M64(kS1x8l, 1, 8, 1, false, false, 0, true);
        DM_M64(kS3x2, 3, 2, 1, false, false, 0);
        DM_M64(kS3x4, 3, 4, 1, false, false, 0);
        DM_M64(kS3x8, 3, 8, 1, false, false, 0);
        DM_M64(kShapes + kS1n2, 1, 8, 1, true, true, 4);
        DM_M64(kShapes + kS1n4, 1, 8, 1, true, true, 8);
        DM_M64(kShapes + kS1x2, 1, 2, 1, false, true, 0);
        DM_M64(kShapes + kS1x4, 1, 4, 1, false, true, 0);
        DM_M64(kShapes + kS1x8, 1, 8, 1, false, true, 0);
        DM_M64(kShapes + kS1x8b, 1, 8, 2, false, true, 0);
#undef DM_M64
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

Launch64 launch_args(uint64_t seed, int64_t step0, const int64_t *d_step, int n_steps,
                     int nonlinear)
{
    Launch64 la{};
    la.step = d_step;
    la.step0 = step0;
    la.seed = seed;
    la.n_steps = n_steps;
    la.nonlinear = nonlinear;
    return la;
}

}  // namespace

hipError_t modes64_build_tables(double *X, int M, hipStream_t st)
{
    const size_t n = modes64_table_bytes(M) / sizeof(double);
    hipLaunchKernelGGL(modes64_table_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, X,
                       M);
    return hipGetLastError();
}

// Mode tiles whose coupling can change the update: for modes that
// equilibrate within a step C_p falls off as exp(-16 nu s^4 dtau) (Eq. f4).
// |Delta H_p| <= 2 s_p * |g| sqrt(M) (column norm 2 s_p from Eq. e6).  Tiles are
// kept up to the first whose lowest mode has C_p 2 s_p sqrt(M) < 2^-100 W_p
// (beyond it the exponential falls further), which leaves out what is below
// the last bit of the noise term for |g| up to 2^47.  Logarithms, because C_p
// underflows.
int modes64_coupled_tiles(int M, double nu, double T_star, double dtau)
{
    const int RT = half_tiles(M);
    for (int T = 1; T < RT; ++T) {
        const double s = std::sin(3.141592653589793 * 32 * T / (2.0 * M)), s2 = s * s;
        const double z = 16.0 * nu * s2 * s2, dz = (1.0 - 2.0 * nu) * 4.0 * s2;
        const double w2 = z > 0.0 ? -T_star * std::expm1(-2.0 * z * dtau) / z
                                  : 2.0 * T_star * dtau;
        const double lc = -z * dtau + std::log(-std::expm1(-dz * dtau) / dz);
        if (lc + std::log(2.0 * s * std::sqrt((double)M)) <
            -100.0 * 0.6931471805599453 + 0.5 * std::log(w2))
            return T;
    }
    return RT;
}

void modes64_plan_free(Modes64Plan &p)
{
    for (Modes64Group &g : p.groups) {
        if (g.d_buckets) (void)hipFree(g.d_buckets);
        if (g.d_items) (void)hipFree(g.d_items);
    }
    p.groups.clear();
}

// Buckets on 16-chain tiles get a launch each.  Those on 5-chain tiles share
// one launch in the widest of their shapes while it is small (all lengths in
// flight at once; the spare wavefronts of the shorter chains only wait), and
// get one launch per shape beyond that, where each fills the GPU by itself.
// Up to a tile per compute unit the shorter chains have noise wavefronts.
hipError_t modes64_plan(Modes64Plan &p, const std::vector<Modes64Args> &bs, int ncu,
                        hipStream_t st)
{
    modes64_plan_free(p);
    std::vector<int> shape(bs.size());
    size_t small_tiles = 0;
    for (const Modes64Args &a : bs)
        if (!large_tiles_pay(a.M, a.n, ncu))
            small_tiles += (size_t)(a.n + kSmallTile - 1) / kSmallTile;
    int widest = 0;
    for (size_t b = 0; b < bs.size(); ++b) {
        if (large_tiles_pay(bs[b].M, bs[b].n, ncu)) {
            shape[b] = large_shape(bs[b].M);
            continue;
        }
        shape[b] = small_shape(bs[b].M, small_tiles <= (size_t)ncu);
        widest = std::max(widest, shape[b]);
    }
    if (small_tiles <= 2 * (size_t)ncu)
        for (int &s : shape)
            if (s < kS3x2) s = widest;
    for (int s = 0; s < kShapes; ++s) {
        std::vector<size_t> in;
        for (size_t b = 0; b < bs.size(); ++b)
            if (shape[b] == s) in.push_back(b);
        if (in.empty()) continue;
        // longest chains first: an in-order dispatch is then a longest-first
        // schedule
        std::stable_sort(in.begin(), in.end(), [&](size_t x, size_t y) { return bs[x].M > bs[y].M; });
        Modes64Group g;
        g.shape = s;
        std::vector<Modes64Args> ba;
        std::vector<Item64> items;
        for (size_t b : in) {
            const int nt = (bs[b].n + tile_chains(s) - 1) / tile_chains(s);
            for (int t = 0; t < nt; ++t) items.push_back({(int)ba.size(), t});
            ba.push_back(bs[b]);
            g.lds = std::max(g.lds, lds_bytes(s, bs[b].M));
            g.odd = g.odd || beyond_tiles(bs[b].M);
        }
        g.nitems = (int)items.size();
        g.shape = paired_shape(s, g.odd, g.nitems, ncu);
        g.single = ba.size() == 1;
        g.one = ba[0];
        hipError_t e = hipSuccess;
        if (!g.single) {
            if ((e = hipMalloc(&g.d_buckets, sizeof(Modes64Args) * ba.size())) == hipSuccess &&
                (e = hipMalloc(&g.d_items, sizeof(Item64) * items.size())) == hipSuccess &&
                (e = hipMemcpyAsync(g.d_buckets, ba.data(), sizeof(Modes64Args) * ba.size(),
                                    hipMemcpyHostToDevice, st)) == hipSuccess &&
                (e = hipMemcpyAsync(g.d_items, items.data(), sizeof(Item64) * items.size(),
                                    hipMemcpyHostToDevice, st)) == hipSuccess)
                e = hipStreamSynchronize(st);  // the host vectors die here
        }
        p.groups.push_back(g);
        if (e != hipSuccess) {  // no launch of a part of the buckets
            modes64_plan_free(p);
            return e;
        }
    }
    return hipSuccess;
}

hipError_t modes64_launch(const Modes64Plan &p, uint64_t seed, int64_t step0,
                          const int64_t *d_step, int n_steps, int nonlinear, hipStream_t st)
{
    for (const Modes64Group &g : p.groups) {
        Launch64 la = launch_args(seed, step0, d_step, n_steps, nonlinear);
        la.one = g.one;
        la.buckets = static_cast<const Modes64Args *>(g.d_buckets);
        la.items = static_cast<const Item64 *>(g.d_items);
        const hipError_t e = launch_shape(g.shape, g.odd, g.lds, g.nitems, la, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t modes64_launch_one(const Modes64Args &a, int ncu, uint64_t seed, int64_t step0,
                              int n_steps, int nonlinear, hipStream_t st)
{
    int shape = large_tiles_pay(a.M, a.n, ncu) ? large_shape(a.M)
                                               : small_shape(a.M, a.n <= kSmallTile * ncu);
    const int nitems = (a.n + tile_chains(shape) - 1) / tile_chains(shape);
    shape = paired_shape(shape, beyond_tiles(a.M), nitems, ncu);
    Launch64 la = launch_args(seed, step0, nullptr, n_steps, nonlinear);
    la.one = a;
    return launch_shape(shape, beyond_tiles(a.M), lds_bytes(shape, a.M), nitems, la, st);
}

}  // namespace dm
