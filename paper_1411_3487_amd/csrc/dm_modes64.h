// dm_modes64.h -- persistent FP64 mode stepper (dm_modes64.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

namespace dm {

// One length bucket as the kernel sees it.
struct Modes64Args {
    const double *X;        // transform fragments (modes64_table_bytes(M))
    const double *E, *C, *W;  // update coefficients by mode, M each
    double *R;              // n chains of 3 M amplitudes (SoA, p = 0..M-1)
    const int32_t *ids;     // global chain index per local chain
    int n, M;
    int jc;                 // coupled mode tiles of 32 modes
    double lin, gdt;        // 1 - 2 nu, gamma_dot dtau
};

constexpr int kModes64MaxM = 513;
inline bool modes64_supports(int M) { return M >= 2 && M <= kModes64MaxM; }

// 16-row tiles of half the bonds (and of half the modes p >= 1).
__host__ __device__ inline int modes64_half_tiles(int M) { return (M / 2 + 15) / 16; }

// Transform tables of chains of M beads: bytes, value i, and their
// construction on the device (they depend on M alone).  Fragments of both
// products: [product][tile][q][parity][lane][2]; product 0 (u = chi R): row =
// half-bond, K = mode; product 1 (coupling): row = mode, K = half-bond.
// chi_{n,p} = sigma_p sin(pi (p n mod 2M) / M), exact zeros at multiples of M.
__host__ __device__ inline size_t modes64_table_bytes(int M)
{
    const size_t RT = modes64_half_tiles(M);
    return sizeof(double) * 2 * RT * 2 * RT * 256;
}
__device__ inline double modes64_table_value(size_t i, int M)
{
    const int RT = modes64_half_tiles(M), Q = 2 * RT, H = M / 2;
    const int e = (int)(i % 2), lane = (int)(i / 2 % 64), par = (int)(i / 128 % 2);
    const int q = (int)(i / 256 % Q), T = (int)(i / 256 / Q % RT), prod = (int)(i / 256 / Q / RT);
    const int row = lane % 16, ri = 16 * T + 4 * (row % 4) + row / 4;
    const int ki = 8 * q + 2 * (lane / 16) + e;
    const int b = prod == 0 ? ri : ki, jm = prod == 0 ? ki : ri;
    const int n = b + 1, p = 2 * jm + 1 + par;
    if (b >= H || p >= M) return 0.0;
    const int m = (int)((long)p * n % (2L * M));
    if (m == 0 || m == M) return 0.0;
    const double v = -2.0 * sqrt(2.0 / M) * sinpi((double)p / (2.0 * M)) * sinpi((double)m / M);
    return prod == 1 && 2 * n == M ? 0.5 * v : v;  // the middle bond enters twice
}
hipError_t modes64_build_tables(double *X, int M, hipStream_t st);
// Coupled mode tiles of 32 modes for these parameters.
int modes64_coupled_tiles(int M, double nu, double T_star, double dtau);

// The launches that advance a set of buckets: groups of one kernel shape.
struct Modes64Group {
    int shape = 0, nitems = 0;
    bool odd = false;         // a length whose last mode lies beyond its tiles
    size_t lds = 0;
    bool single = false;      // one bucket, passed by value; item = tile index
    Modes64Args one{};
    void *d_buckets = nullptr, *d_items = nullptr;
};
struct Modes64Plan {
    std::vector<Modes64Group> groups;
};
hipError_t modes64_plan(Modes64Plan &p, const std::vector<Modes64Args> &bs, int ncu,
                        hipStream_t st);
void modes64_plan_free(Modes64Plan &p);
// n_steps mode steps of every bucket of the plan, first Philox step
// (*d_step or 0) + step0.  Only enqueues.
hipError_t modes64_launch(const Modes64Plan &p, uint64_t seed, int64_t step0,
                          const int64_t *d_step, int n_steps, int nonlinear, hipStream_t st);
// The same for one bucket without a plan (no allocation).
hipError_t modes64_launch_one(const Modes64Args &a, int ncu, uint64_t seed, int64_t step0,
                              int n_steps, int nonlinear, hipStream_t st);

}  // namespace dm
