// The 2D step of small and middling lattices: one workgroup per tile, one wave
// per row of the tile, so that a step is one round of memory latency and three
// barriers however small the lattice is.  The marching kernel (step.hpp) gives
// a wave a band of at least 8 rows, 13 dependent row steps with its warm-up;
// that is the better deal where the lattice fills the SIMDs with tall bands,
// but below it every lattice takes the same 11-60 us.  What bounds this one:
// the launch and one memory latency (about 5 us) up to 128^2, then the
// instruction issue of the tiles' rows, halo rows included.  us per step, march
// -> tiles: 64^2 Euler FP32 19.4 -> 5.8, FP64 32.1 -> 7.7, shallow water FP64
// 52.8 -> 7.2; 256^2 Euler FP32 20.1 -> 8.6, FP64 34.4 -> 11.6; 400^2 reactive
// FP32 34.1 -> 15.3.
//
// A tile of `rows` waves writes rows - 6 rows of 58 columns; the outer three
// rows and lanes on each side are its halo.  Row w of the tile:
//   all rows              populations (with the ghost map) -> U into LDS
//   rows 1 .. rows-2      U of rows w-1, w, w+1 -> nu into LDS (2.13-2.14)
//   rows 2 .. rows-3      3x3 box sum, omega (2.15-2.16), collision (2.2);
//                         f*_{+y} and f*_{-y} into LDS, +-x by lane shifts
//   rows 3 .. rows-4      pull, moment update (2.8), second half source, store
// Waves outside a stage's rows leave its issue slots to the others.  Every
// expression is the marching kernel's, so both give the same bits.
// f* takes the LDS space of U, which nothing reads after the indicator.
// BUF: plane addresses through buffer resources take about 73 scalar registers
// instead of 90, and a CU then holds two tiles of 16 rows (512^2 Euler FP32
// 19.8 -> 15.9 us, shallow water 16.4 -> 13.5, reactive FP64 45.6 -> 44.5; the
// same vector registers); with at most one tile per CU 64-bit addresses are
// the faster (64^2 Euler FP32 6.4 against 6.6 us).
#pragma once

#include "step.hpp"

namespace arlbm {

template <int SYS, bool BED, typename T>
__host__ __device__ constexpr size_t tile2d_row_elems()
{
    return (size_t)kWave * (2 * SysInfo<SYS, 2>::M + 1 + (BED ? 1 : 0));
}
// LDS bytes of a tile of `rows` rows: f* (over U), nu, bed, and the
// coefficients shared by the waves.
template <typename T>
struct TileShared {
    Coefs<T> cf;
    int state;  // 0: step, 1: degenerate bounds, 2: at the stop time
};
template <int SYS, bool BED, typename T>
constexpr size_t tile2d_lds(int rows)
{
    return (size_t)rows * tile2d_row_elems<SYS, BED, T>() * sizeof(T) + sizeof(TileShared<T>);
}

template <int SYS, bool BED, typename T, bool BUF>
__global__ __launch_bounds__(kMaxTileRows * kWave) void k_tile2d(LatticeDesc L, int64_t iter, int32_t ntiles_y, int32_t nwork)
{
    constexpr int D = 2, M = SysInfo<SYS, 2>::M, Q = 5;
    extern __shared__ __align__(16) char smem[];
    TileShared<T> &sh = *(TileShared<T> *)smem;
    const int rows = (int)(blockDim.x >> 6);
    T *lF = (T *)(smem + sizeof(TileShared<T>));  // [row][2 M][lane]; U as [row][M][lane] first
    T *lnu = lF + (size_t)rows * 2 * M * kWave;    // [row][lane]
    T *lbed = lnu + (size_t)rows * kWave;          // [row][lane]
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int w = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // consecutive tiles (down a strip, then across) on one XCD
    const int nb = (int)gridDim.x;
    const int item = ((int)blockIdx.x & 7) * (nb >> 3) + ((int)blockIdx.x >> 3);
    if (item >= nwork) return;
    const int col = item / ntiles_y, tile = item - col * ntiles_y;
    const int out_rows = rows - 2 * kHalo;
    const int nx = L.nx, ny = L.ny;
    const int x = col * kOutW - kHalo + lane, y = tile * out_rows - kHalo + w;
    const int64_t n = iter - L.iter0;
    const bool xout = lane >= kHalo && lane < kWave - kHalo && x < nx;
    const bool yout = w >= kHalo && w < rows - kHalo && y < ny;
    const int bxl = L.bc[0], bxh = L.bc[1], byl = L.bc[2], byh = L.bc[3];
    bool rx, ry;
    const int xm = bc_map(x, nx, bxl, bxh, rx), ym = bc_map(y, ny, byl, byh, ry);
    const unsigned off = (unsigned)ym * (unsigned)nx + (unsigned)xm;

    const PlaneIO<T, 1, BUF> io(L, n);
    T f[Q][M];
#pragma unroll
    for (int k = 0; k < Q; ++k)
#pragma unroll
        for (int c = 0; c < M; ++c) {
            T v[1];
            io.ld(k * M + c, off, v);
            f[k][c] = v[0];
        }
    T b = T(0);
    if constexpr (BED) b = ((const T *)L.bed)[off];
    // The coefficients, once per tile, by the last wave, which has no indicator
    // to form: beside the others' (kBeside) or, before the first barrier, while
    // they wait for their rows.  There everybody waits for its chain of
    // quotients too (us per step, before -> beside: 64^2 Euler FP32 6.4 -> 5.9,
    // FP64 8.3 -> 7.7; 256^2 9.2 -> 8.7, 12.2 -> 11.6; 512^2 shallow water FP64
    // 27.6 -> 26.3); but advection's indicator is too short to cover it, and the
    // reactive kernels lack the registers (FP32 80 -> 83, one tile per CU: 400^2
    // 15.3 -> 16.8; FP64 spills: 256^2 18.2 -> 18.6).
    constexpr bool kBeside = SYS == 1 || SYS == 2;
    if constexpr (kBeside) {
        if (stopped(L, n)) {  // the state carries over (a step that is not defined is flagged here too)
            Coefs<T> cf;
            if (step_coefs<D, T>(L, n, cf)) null_copy<T>(L, n, Q * M, x, xout && yout, y, y + 1, item == 0 && w == 0);
            else if (item == 0 && w == 0 && lane == 0) flag_degenerate(L, n);
            return;
        }
    } else if (w == rows - 1) {
        Coefs<T> cf;
        const bool ok = step_coefs<D, T>(L, n, cf);
        if (lane == 0) {
            if (ok) sh.cf = cf;
            sh.state = !ok ? 1 : (stopped(L, n) ? 2 : 0);
        }
    }
    const Phys<T> P = make_phys<T>(L);
    T U[M];
#pragma unroll
    for (int c = 0; c < M; ++c) {
        T sum = f[0][c];
#pragma unroll
        for (int k = 1; k < Q; ++k) sum = sum + f[k][c];
        U[c] = sum;
    }
    if constexpr (SYS != 0) {
        if (rx) U[1] = -U[1];
        if (ry) U[2] = -U[2];
    }
    {
        T *u = lF + (size_t)w * M * kWave + lane;
#pragma unroll
        for (int c = 0; c < M; ++c) u[c * kWave] = U[c];
        if constexpr (BED) lbed[w * kWave + lane] = b;
    }
    Prim<T> q;
    primitives<SYS, D, T>(U, P, q);
    __syncthreads();
    if constexpr (kBeside) {
        if (w == rows - 1) {
            Coefs<T> cf;
            const bool ok = step_coefs<D, T>(L, n, cf);
            if (lane == 0) {
                if (ok) sh.cf = cf;
                sh.state = !ok;
            }
        }
    } else {
        const int state = __builtin_amdgcn_readfirstlane(sh.state);
        if (state != 0) {
            if (state == 1) {
                if (item == 0 && w == 0 && lane == 0) flag_degenerate(L, n);
            } else {
                null_copy<T>(L, n, Q * M, x, xout && yout, y, y + 1, item == 0 && w == 0);
            }
            return;
        }
    }
    if (w >= 1 && w < rows - 1) {
        T nu = T(0);
        if (!L.omega_fixed_on) {
            {
                T UL[M], UR[M];
#pragma unroll
                for (int c = 0; c < M; ++c) {
                    UL[c] = from_left(U[c]);
                    UR[c] = from_right(U[c]);
                }
                add_theta<SYS, D, T>(0, q, U, UL, UR, P, nu);
            }
            T Um[M], Up[M];
            const T *um = lF + (size_t)(w - 1) * M * kWave + lane, *up = lF + (size_t)(w + 1) * M * kWave + lane;
#pragma unroll
            for (int c = 0; c < M; ++c) {
                Um[c] = um[c * kWave];
                Up[c] = up[c * kWave];
            }
            add_theta<SYS, D, T>(1, q, U, Um, Up, P, nu);
        }
        lnu[w * kWave + lane] = nu;
    }
    __syncthreads();
    if constexpr (kBeside) {
        if (__builtin_amdgcn_readfirstlane(sh.state)) {
            if (item == 0 && w == 0 && lane == 0) flag_degenerate(L, n);
            return;
        }
    }
    const Coefs<T> cf = sh.cf;
    T fs[Q][M], dbx = T(0), dby = T(0);
    if (w >= 2 && w < rows - 2) {
        // 3x3 box sum (2.15) in row-major order, relaxation parameter (2.16)
        const T N0 = lnu[(w - 1) * kWave + lane], N1 = lnu[w * kWave + lane], N2 = lnu[(w + 1) * kWave + lane];
        const T N0l = from_left(N0), N0r = from_right(N0), N1l = from_left(N1), N1r = from_right(N1);
        const T N2l = from_left(N2), N2r = from_right(N2);
        const T nt = N0l + N0 + N0r + N1l + N1 + N1r + N2l + N2 + N2r;
        const T om = L.omega_fixed_on ? cf.omega_fixed : omega_of<T>(nt);
        if (L.omega_on && xout && yout) ((T *)L.omega)[(unsigned)y * (unsigned)nx + (unsigned)x] = om;
        if constexpr (BED) {
            const T two_dx = T(2) * P.dx;
            dbx = ddiv<T>(from_right(b) - from_left(b), two_dx);
            dby = ddiv<T>(lbed[(w + 1) * kWave + lane] - lbed[(w - 1) * kWave + lane], two_dx);
        }
        // equilibrium (2.20) and collision at the source nodes
        T Fx[M], Fy[M];
        flux<SYS, D, T>(0, U, q, P, Fx);
        flux<SYS, D, T>(1, U, q, P, Fy);
#pragma unroll
        for (int c = 0; c < M; ++c) {
            const T u = U[c];
            const T feq[Q] = {cf.a0 * u, cf.ap[0] * u + cf.bp * Fx[c], cf.ap[1] * u + cf.bp * Fy[c],
                              cf.ap[0] * u + cf.bm * Fx[c], cf.ap[1] * u + cf.bm * Fy[c]};
#pragma unroll
            for (int k = 0; k < Q; ++k) fs[k][c] = f[k][c] - om * (f[k][c] - feq[k]);
        }
        const T ak[Q] = {cf.a0, cf.ap[0], cf.ap[1], cf.ap[0], cf.ap[1]};
        if constexpr (BED) {
            const T S1 = -P.g * U[0] * dbx, S2 = -P.g * U[0] * dby;
#pragma unroll
            for (int k = 0; k < Q; ++k) {
                fs[k][1] = fs[k][1] + cf.hdt * (ak[k] * S1);
                fs[k][2] = fs[k][2] + cf.hdt * (ak[k] * S2);
            }
        }
        if constexpr (SYS == 3) {  // Arrhenius sink of rho Y, first half (2.6)
            const T SY = -arrhenius_rate<T>(P, U[0], reactive_eint<D, T>(U), U[M - 1], nullptr);
#pragma unroll
            for (int k = 0; k < Q; ++k) fs[k][M - 1] = fs[k][M - 1] + cf.hdt * (ak[k] * SY);
        }
        T *o = lF + (size_t)w * 2 * M * kWave + lane;
#pragma unroll
        for (int c = 0; c < M; ++c) {
            o[c * kWave] = fs[2][c];
            o[(M + c) * kWave] = fs[4][c];
        }
    }
    __syncthreads();
    if (yout) {
        // F_0, F_{+x}, F_{+y}, F_{-x}, F_{-y} with the ghost map at the walls
        T Fk[Q][M];
        const T *below = lF + (size_t)(w - 1) * 2 * M * kWave + lane;
        const T *above = lF + (size_t)(w + 1) * 2 * M * kWave + M * kWave + lane;
#pragma unroll
        for (int c = 0; c < M; ++c) {
            Fk[0][c] = fs[0][c];
            Fk[1][c] = from_left(fs[1][c]);
            Fk[2][c] = below[c * kWave];
            Fk[3][c] = from_right(fs[3][c]);
            Fk[4][c] = above[c * kWave];
        }
        if (x == 0 && bxl != 0) {
#pragma unroll
            for (int c = 0; c < M; ++c) Fk[1][c] = bxl == 1 ? fs[1][c] : (c == 1 ? -fs[3][c] : fs[3][c]);
        }
        if (x == nx - 1 && bxh != 0) {
#pragma unroll
            for (int c = 0; c < M; ++c) Fk[3][c] = bxh == 1 ? fs[3][c] : (c == 1 ? -fs[1][c] : fs[1][c]);
        }
        if (y == 0 && byl != 0) {
#pragma unroll
            for (int c = 0; c < M; ++c) Fk[2][c] = byl == 1 ? fs[2][c] : (c == 2 ? -fs[4][c] : fs[4][c]);
        }
        if (y == ny - 1 && byh != 0) {
#pragma unroll
            for (int c = 0; c < M; ++c) Fk[4][c] = byh == 1 ? fs[4][c] : (c == 2 ? -fs[2][c] : fs[2][c]);
        }
        const T ak[Q] = {cf.a0, cf.ap[0], cf.ap[1], cf.ap[0], cf.ap[1]};
        T sumF[M];
#pragma unroll
        for (int c = 0; c < M; ++c) sumF[c] = Fk[0][c] + Fk[1][c] + Fk[2][c] + Fk[3][c] + Fk[4][c];
        if constexpr (BED) {
            const T S1 = -P.g * sumF[0] * dbx, S2 = -P.g * sumF[0] * dby;
#pragma unroll
            for (int k = 0; k < Q; ++k) {
                Fk[k][1] = Fk[k][1] + cf.hdt * (ak[k] * S1);
                Fk[k][2] = Fk[k][2] + cf.hdt * (ak[k] * S2);
            }
        }
        if constexpr (SYS == 3) {  // (2.8) for rho Y, then the second half source
            const T eint = reactive_eint<D, T>(sumF);
            const T z = reactive_solve<T>(P, sumF[0], eint, sumF[M - 1], cf.hdt);
            const T SY = -arrhenius_rate<T>(P, sumF[0], eint, z, nullptr);
#pragma unroll
            for (int k = 0; k < Q; ++k) Fk[k][M - 1] = Fk[k][M - 1] + cf.hdt * (ak[k] * SY);
        }
        T Un[M];
#pragma unroll
        for (int c = 0; c < M; ++c) Un[c] = Fk[0][c] + Fk[1][c] + Fk[2][c] + Fk[3][c] + Fk[4][c];
        T s0 = T(0), s1 = T(0);
        unsigned flags = 0;
        if (xout) {
            const unsigned o = (unsigned)y * (unsigned)nx + (unsigned)x;
#pragma unroll
            for (int k = 0; k < Q; ++k)
#pragma unroll
                for (int c = 0; c < M; ++c) {
                    const T v[1] = {Fk[k][c]};
                    io.st(k * M + c, o, v);
                }
            Prim<T> qn;
            primitives<SYS, D, T>(Un, P, qn);
            const T v0 = max_speed<SYS, T>(0, qn, P), v1 = max_speed<SYS, T>(1, qn, P);
            bool fin_ok = true;
#pragma unroll
            for (int c = 0; c < M; ++c) fin_ok = fin_ok && finite_val<T>(Un[c]);
            flags = qn.flags | (fin_ok ? 0u : 1u);
            if (finite_val<T>(v0) && v0 > s0) s0 = v0;
            if (finite_val<T>(v1) && v1 > s1) s1 = v1;
        }
        commit<T>(L, n, s0, s1, flags, 2);
    }
    if (item == 0 && w == 0) scalar_update(L, n, cf.dt);
}

}  // namespace arlbm
