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

// Transform tables of chains of M beads: bytes, and their construction on
// the device (they depend on M alone).
size_t modes64_table_bytes(int M);
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
