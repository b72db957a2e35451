// Internal types shared by the HIP kernels and the host runtime of libarlbm.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace arlbm {

// Cells produced per wave along x.  With one column per lane a wave of 64
// lanes covers x0-3 .. x0+60: the 3-cell halo on each side feeds the
// radius-2 indicator stencil and the radius-1 pull (omega is needed one cell
// beyond the outputs).  With V columns per lane the halo is rounded up to
// whole lanes, so that every lane's V columns start V-aligned.
constexpr int kWave = 64;
constexpr int kHalo = 3;
constexpr int kOutW = kWave - 2 * kHalo;  // 58
__host__ __device__ constexpr int strip_halo(int v) { return (kHalo + v - 1) / v * v; }
__host__ __device__ constexpr int strip_out_w(int v) { return kWave * v - 2 * strip_halo(v); }
static_assert(strip_out_w(1) == kOutW && strip_out_w(2) == 120, "strip geometry");
// The march of 1D lattices in registers (k_march1d).  One workgroup of at most
// kMarchWaves waves, of one cell per lane where 58 cells a wave hold the
// lattice (Euler FP32 400 cells 1.67 against 1.70 us per step of two, 100 cells
// 1.08 against 1.51), else, for advection, of two (1920 cells FP32 1.13 us,
// FP64 1.72, against 1.92 and 2.07 for 1921 over several workgroups).  Larger lattices
// march over several workgroups: for Euler and shallow water beyond 928 cells
// (928 in one against 929 in several: Euler FP32 2.46 against 2.58 us, FP64 3.78
// against 3.22, shallow water 1.98 against 2.22 and 3.16 against 2.90; two cells
// per lane at 1500 cells 3.89), for the reactive system, bound by one CU's
// kinetics, earlier (FP64 406 cells 4.90 against 5.11 for 407, 928 9.2 against
// 5.8; FP32 696 3.51 against 3.56, 928 4.5 against 3.6).
constexpr int kMarchWaves = 16;
__host__ __device__ constexpr int march_width(int64_t nx) { return nx <= kMarchWaves * strip_out_w(1) ? 1 : 2; }
constexpr int march_cells(int system, bool f64)
{
    return system == 0 ? kMarchWaves * strip_out_w(2) : (system == 3 ? (f64 ? 7 : 12) : kMarchWaves) * kOutW;
}
// Several workgroups: four waves each (one per SIMD), and at most a quarter of
// what the device holds at once (kGridShare), so that the lattices of several
// streams, of which a process runs four at a time by default, find room beside
// each other; the reactive system's registers set the sizes.  us per step and
// lattice, one launch per step against the march, for one lattice: Euler FP32
// 4096 cells 4.54 / 2.58, 29000 4.60 / 2.92, 59392 4.75 / 3.36, FP64 4096 5.11 /
// 3.48, 29696 5.36 / 3.99; for two, each on a stream and host thread of its
// own: FP32 29000 2.48 / 1.89, 58000 2.64 / 2.41, FP64 29000 3.03 / 2.44; for
// four, whose workgroups share the CUs and wait for one another's slowest: FP32
// 14800 1.32 / 1.00, 29000 1.41 / 1.31, 37000 1.46 / 1.54, 45000 1.51 / 1.68,
// FP64 9500 1.51 / 1.33, 19000 1.62 / 1.62, 29000 1.71 / 2.06.  So one or two
// lattices gain over the whole range, three up to three quarters of it and four
// up to about two thirds, and the largest sizes are drawn for one or two.
constexpr int kGridWaves = 4, kGridShare = 4;
constexpr int64_t grid_march_cells(bool f64) { return (int64_t)(f64 ? 128 : 256) * kGridWaves * kOutW; }
// Steps from which the several workgroups pay for their three launches (us per
// step in calls of 32, against one launch per step: Euler FP32 4096 cells 2.85
// against 4.38, 58000 3.70 against 4.61, FP64 4096 3.76 against 4.93).
constexpr int kGridMinSteps = 32;
// Looks of about 1 us at the words of other workgroups before one calls a march
// off (60 ms, in which other work on the device lets the rest come to run) or,
// in the march, gives it up.
constexpr int kGatherLooks = 1 << 16, kHearLooks = 1 << 24;
constexpr int kStripWaves = 16;           // waves of k_strips1d
constexpr int kMaxTileRows = 16;          // rows (waves) of a tile of the tiled 2D step
// The tiled 3D step of small lattices (tile3d.hpp): tiles of kTile3X x kTile3Y
// x tile3_z cells, or, where those fit one round of the CUs, of 4 cells in z.
constexpr int kTile3X = 8, kTile3Y = 8;
__host__ __device__ constexpr int tile3_z(int system, bool f64) { return system == 3 && f64 ? 4 : 8; }
constexpr int64_t tiles3(int64_t nx, int64_t ny, int64_t nz, int64_t tz)
{
    return ((nx + kTile3X - 1) / kTile3X) * ((ny + kTile3Y - 1) / kTile3Y) * ((nz + tz - 1) / tz);
}
// Tiles per CU up to which the tiles beat the march, whose workgroups take as
// long for a small lattice as for one of their own size: Euler FP32 64^3 (2
// tiles per CU) 32 against 81 us, 96^3 (6.75) 107 against 91, FP64 61 / 162
// and 246 / 193; advection 96^3 25 / 31 and 128^3 (16) 50 / 51, FP64 39 / 46
// and 78 / 80.
constexpr int kTiles3PerCu = 5, kTiles3PerCuAdv = 16;
// Cells in z of a lattice's tiles, 0 where it marches through planes.
constexpr int choose_tile_z(int system, bool f64, int64_t nx, int64_t ny, int64_t nz, int64_t cus)
{
    if (tiles3(nx, ny, nz, 4) <= cus) return 4;
    const int tz = tile3_z(system, f64);
    return tiles3(nx, ny, nz, tz) <= cus * (system == 0 ? kTiles3PerCuAdv : kTiles3PerCu) ? tz : 0;
}
constexpr int kBlock = 256;               // 4 independent waves per block
constexpr int kWavesPerBlock = kBlock / kWave;

enum Variant : int32_t {
    V_ADV1 = 0, V_EUL1 = 1, V_SWE1 = 2, V_REU1 = 3,
    V_ADV2 = 4, V_EUL2 = 5, V_SWE2 = 6, V_REU2 = 7,
    V_ADV3 = 8, V_EUL3 = 9, V_REU3 = 11
};

__host__ __device__ constexpr int variant_of(int system, int dim) { return (dim - 1) * 4 + system; }
__host__ __device__ constexpr int num_fields(int system, int dim) {
    return system == 0 ? 1 : (system == 1 ? dim + 2 : (system == 2 ? dim + 1 : dim + 3));
}

// Per-lattice device scalars (FP64), kept resident between launches.
// One copy of a wave-speed slot: one 128-byte line, v[0..2] the directions.
struct AbarCopy {
    unsigned long long v[16];
};
// Copies per slot.  A wave maxes its bounds into copy (wave index mod
// kAbarCopies) and readers take the max over the copies: with a single copy
// the waves of a launch queued on one line at about 11 ns per atomic, about
// 9 us of a 2048^2 2D step.  Atomics on one line serialize even at different
// addresses: copies packed 16 to a line measured 0.1586 against 0.1574 ms per
// 2048^2 Euler step and 17.2 against 7.9 us per 262144-cell 1D step.
constexpr int kAbarCopies = 64;
struct DevScalars {
    // alpha_bar bit patterns (non-negative doubles order like unsigned
    // integers, so the grid-wide max is an integer atomic max).  Three slots:
    // step n reads slot n%3, maxes into (n+1)%3 and clears (n+2)%3.
    AbarCopy abar[3][kAbarCopies];
    double last_dt;
    unsigned long long first_bad_step;  // min over flagged steps (~0 = none)
    unsigned int flags;
    unsigned int pad;
    // time of the state step n reads (slot n%3; the step writes slot (n+1)%3,
    // so every wave of a launch sees the same value)
    double t[3];
    unsigned long long null_launches;   // launches that found t >= t_stop (left the state as it was)
};
static_assert(sizeof(DevScalars) == 3 * kAbarCopies * sizeof(AbarCopy) + 56, "DevScalars layout");

// Everything a kernel needs to know about one lattice.  Uploaded once at
// creation (and at admission in the server); the step index is derived from
// the launch's iteration counter: n = iter - iter0.
struct LatticeDesc {
    void *f[2];
    void *u[2];
    const void *bed;
    void *omega;
    DevScalars *sc;
    int32_t variant, nx, ny, nz, bc[6];
    int32_t omega_fixed_on;
    int32_t band_h;       // rows per strip (2D)
    int32_t ncols;        // strips along x
    int32_t tile_rows;    // 2D: rows per tile of the tiled step, 0: the marching step
    int64_t iter0;
    double t_stop;        // a launch whose state time is >= t_stop copies f unchanged (null step)
    int64_t plane;        // nx * ny * nz
    int64_t pstride;      // elements between planes: plane rounded up to 64, plus a pad
    int32_t omega_on;     // omega export plane present (else omega is null and never written)
    int32_t cpl;          // 2D: columns per lane of the step's strips (1, or 2 when nx is even)
    int32_t buf;          // 2D: population buffers below 4 GiB, addressed by buffer resources
    int32_t abar_n;       // copies of each wave-speed slot in use: a power of two <= kAbarCopies, fixed per lattice
    double dx, cfl, eps, gamma, g, adv[3], h_dry, rho_floor, p_floor, omega_fixed;
    double q_heat, k_rate, t_act;  // reactive Euler: heat release, rate constant, activation temperature
    int32_t gather_looks, hear_looks;  // 1D march over several workgroups: the limits of its waits
};

// One work item of a batched launch.  2D: rows y0 .. y1-1 of strip col.
// 1D: strips col .. y1-1 (y0 unused).  The item that holds the lattice's
// first cell (col 0, row 0) also updates its scalars.
struct Segment {
    int32_t lattice;
    int32_t col;
    int32_t y0;
    int32_t y1;
};

// Conservation sums: per-block compensated partial sums of each field, over
// kConsBlocks blocks, for at most kConsMaxFields fields (3D reactive Euler).
constexpr int kConsBlocks = 256;
constexpr int kConsMaxFields = 6;

// Work queues of a batched launch: one per XCD, counters 128 bytes apart.
constexpr int kQueues = 8;
constexpr int kQueueStride = 32;

}  // namespace arlbm

// Host-side launchers, implemented once per precision (kernels.hip is
// compiled twice, FP32 and FP64, both without contraction).
#define ARLBM_DECLARE_LAUNCHERS(NS)                                                                    \
    namespace arlbm {                                                                                  \
    namespace NS {                                                                                     \
    hipError_t reduce_abar(const LatticeDesc &h, const double *U0, int slot, hipStream_t s);          \
    hipError_t init(const LatticeDesc &h, const double *U0, const double *bed64, int slot_in,         \
                    hipStream_t s);                                                                    \
    hipError_t step_single(const LatticeDesc &h, int64_t iter, hipStream_t s);                        \
    hipError_t steps1d(const LatticeDesc &h, int64_t iter0, int32_t nsteps, hipStream_t s);           \
    hipError_t steps1d_grid(const LatticeDesc &h, int64_t iter0, int32_t nsteps, hipStream_t s);      \
    hipError_t step_batched(const LatticeDesc *d_descs, const Segment *d_segs, const int32_t *d_qstart, \
                            unsigned *d_counters, int32_t parity, int32_t nwaves, int64_t iter,        \
                            hipStream_t s);                                                            \
    hipError_t conservation(const void *u, int64_t plane, int64_t pstride, int m, double *partial,    \
                            int nblocks, hipStream_t s);                                               \
    hipError_t moments(const void *f, void *u, int64_t plane, int64_t pstride, int m, int q,          \
                       hipStream_t s);                                                                 \
    hipError_t to_double(const void *src, double *dst, int64_t plane, int64_t pstride, int m,         \
                         hipStream_t s);                                                               \
    int step_kernel_vgprs(int variant, int cpl);                                                       \
    int step_waves_per_cu(int variant, int cpl);                                                       \
    }                                                                                                  \
    }

ARLBM_DECLARE_LAUNCHERS(f32)
ARLBM_DECLARE_LAUNCHERS(f64)

namespace arlbm {
// out[i] = descs[i].sc->flags for i < n (either precision: the scalars are FP64).
hipError_t gather_flags_launch(const LatticeDesc *descs, int32_t n, unsigned *out, hipStream_t s);
// Device address of this GPU's copy of the conservation scratch (a
// file-scope device array of kConsBlocks * kConsMaxFields doubles), looked up
// once per device with that device current.
hipError_t conservation_scratch(double **out);
}  // namespace arlbm
