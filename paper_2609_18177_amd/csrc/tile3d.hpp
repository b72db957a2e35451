// The 3D step of small lattices: one workgroup per x-y-z tile.  The marching step (step3d.hpp) gives a workgroup a column of at
// least 8 planes, whose plane iterations (5 more for its prologue) follow one
// another behind two barriers each; here every plane of a tile is worked on at
// once and a step has three barriers in all, for more halo work per cell.
//
// LDS holds the moments of the tile and a three-cell halo, the indicator over
// the tile and two cells, omega (and, for the reactive system, the source
// rate) over the tile and one cell, each formed by all threads in turn.  Then
// one thread per cell collides its rest population and the six it pulls, at
// their source nodes (moments and omega from LDS, the population requested
// before the first barrier), completes the cell (2.8) and stores it.  Every
// expression is the marching step's, so both give the same bits.
//
// What bounds it: the indicator over the halo (3.4 evaluations per cell; FP64
// divisions) and, for a lattice of one round of tiles, the chain of its
// stages.  us per step, march -> tiles: 24^3 Euler FP32 77 -> 13, FP64 143 ->
// 18, 48^3 FP64 174 -> 28, 64^3 FP32 81 -> 31, FP64 179 -> 59, reactive FP64
// 161 -> 94, advection FP32 28 -> 12.
#pragma once

#include "step3d.hpp"

namespace arlbm {

// Tiles of 8 x 8 x 8 cells and one thread per cell; of 8 x 8 x 4 with two
// threads per cell to form the halo where those fit one round of the CUs
// (kLow: 32^3 Euler FP32 16.4 -> 13.1 us, FP64 25.7 -> 18.8; 64^3 32 -> 47),
// and for FP64 reactive Euler, six fields of whose larger tile exceed the LDS.
// (16 x 8 x 4: FP32 Euler 64^3 29.0 against 31.9, reactive 45 against 38,
// FP64 Euler 63 against 61; 1024 threads for 8 x 8 x 8: 64^3 39 against 32.)
template <int SYS, typename T, bool kLow>
struct Block3 {
    static constexpr int TX = kTile3X, TY = kTile3Y, TZ = kLow ? 4 : tile3_z(SYS, sizeof(T) == 8);
    static constexpr int kCells = TX * TY * TZ, kThreads = 512;
    static constexpr int W3 = TX + 6, H3 = TY + 6, N3 = W3 * H3 * (TZ + 6);
    static constexpr int W2 = TX + 4, H2 = TY + 4, N2 = W2 * H2 * (TZ + 4);
    static constexpr int W1 = TX + 2, H1 = TY + 2, N1 = W1 * H1 * (TZ + 2);
};
template <int SYS, typename T, bool kLow>
__global__ __launch_bounds__((Block3<SYS, T, kLow>::kThreads)) void k_tile3d(LatticeDesc L, int64_t iter, int32_t ntx,
                                                                        int32_t nty, int32_t nwork)
{
    using G = Block3<SYS, T, kLow>;
    constexpr int D = 3, M = SysInfo<SYS, 3>::M, Q = 7, TX = G::TX, TY = G::TY, TZ = G::TZ, NT = G::kThreads;
    constexpr int W3 = G::W3, P3 = G::W3 * G::H3, W2 = G::W2, P2 = G::W2 * G::H2, W1 = G::W1, P1 = G::W1 * G::H1;
    __shared__ T lu[M][G::N3];
    __shared__ T lnu[G::N2];
    __shared__ T lw[G::N1];
    __shared__ T lrate[SYS == 3 ? G::N1 : 1];
    __shared__ Coefs<T> scf;
    __shared__ int sstate;

    // consecutive tiles (x fastest) on one XCD
    const int nb = (int)gridDim.x;
    const int item = ((int)blockIdx.x & 7) * (nb >> 3) + ((int)blockIdx.x >> 3);
    if (item >= nwork) return;
    const int64_t n = iter - L.iter0;
    const int tid = (int)threadIdx.x;
    const int nx = L.nx, ny = L.ny, nz = L.nz;
    const int x0 = (item % ntx) * TX, y0 = (item / ntx % nty) * TY, z0 = (item / ntx / nty) * TZ;
    const int64_t ps = L.pstride;
    const T *fin = (const T *)L.f[n & 1];
    const T *u = (const T *)L.u[n & 1];
    T *fout = (T *)L.f[(n + 1) & 1];
    T *uout = (T *)L.u[(n + 1) & 1];

    // this thread's cell and the populations its collision takes: its own
    // k = 0 and the six pulled from k's source, or at a wall this cell's own
    // (reflective: the mirrored velocity, its normal momentum negated)
    const int tx = tid % TX, ty = tid / TX % TY, tz = tid / (TX * TY);
    const int gx = x0 + tx, gy = y0 + ty, gz = z0 + tz;
    const bool live = tid < G::kCells && gx < nx && gy < ny && gz < nz;
    const unsigned cell = live ? ((unsigned)gz * (unsigned)ny + (unsigned)gy) * (unsigned)nx + (unsigned)gx : 0u;
    // moments of the tile + 3 requested first (cells outside the diamond of the
    // indicator's reach too: cheaper than telling them apart)
    constexpr int UP = (G::N3 + NT - 1) / NT;
    T Ul[UP][M];
#pragma unroll
    for (int j = 0; j < UP; ++j) {
        const int i = tid + j * NT;
        if (i < G::N3)
            load_U3<M, T>(L, u, x0 - 3 + i % W3, y0 - 3 + i / W3 % G::H3, z0 - 3 + i / P3, SYS != 0, Ul[j]);
    }
    unsigned own_m = 0, refl_m = 0;
    T fk[Q][M];
    if (live) {
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            unsigned src = cell;
            int ks = k;
            if (k > 0) {
                const int dir = (k - 1) % 3, sgn = k <= 3 ? 1 : -1;
                int s[3] = {gx, gy, gz};
                const int nn = dir == 0 ? nx : (dir == 1 ? ny : nz);
                s[dir] -= sgn;
                if (s[dir] < 0 || s[dir] >= nn) {
                    const int b = L.bc[2 * dir + (s[dir] < 0 ? 0 : 1)];
                    if (b == 0) {
                        s[dir] = s[dir] < 0 ? nn - 1 : 0;
                    } else {
                        s[dir] += sgn;
                        own_m |= 1u << k;
                        if (b == 2) {
                            refl_m |= 1u << k;
                            ks = mirror3(k);
                        }
                    }
                }
                src = ((unsigned)s[2] * (unsigned)ny + (unsigned)s[1]) * (unsigned)nx + (unsigned)s[0];
            }
#pragma unroll
            for (int c = 0; c < M; ++c) fk[k][c] = ldo(fin + (int64_t)(ks * M + c) * ps, src);
        }
    }
#pragma unroll
    for (int j = 0; j < UP; ++j) {
        const int i = tid + j * NT;
        if (i < G::N3)
#pragma unroll
            for (int c = 0; c < M; ++c) lu[c][i] = Ul[j][c];
    }
    // The coefficients, once per tile, by the last wave: after its indicator
    // cells, of which it has the fewest, or, where tiles are low and it has as
    // many as the others, while they wait for their moments (us per step, before
    // -> after the indicator: 64^3 Euler FP32 32.2 -> 30.6, FP64 60.3 -> 58.5;
    // low tiles 24^3 advection FP64 8.5 -> 8.9).
    auto form_coefs = [&] {
        if (tid >= NT - kWave) {
            Coefs<T> cf;
            const bool ok = step_coefs<D, T>(L, n, cf);
            if (tid == NT - 1) {
                if (ok) scf = cf;
                sstate = !ok ? 1 : (stopped(L, n) ? 2 : 0);
            }
        }
    };
    if constexpr (kLow) form_coefs();
    const Phys<T> P = make_phys<T>(L);
    __syncthreads();
    const bool fixed = L.omega_fixed_on != 0;
    if (!fixed) {
        for (int i = tid; i < G::N2; i += NT) {
            const int r = (i / P2 + 1) * P3 + (i / W2 % G::H2 + 1) * W3 + i % W2 + 1;
            T Uc[M], Um[M], Up[M];
#pragma unroll
            for (int c = 0; c < M; ++c) Uc[c] = lu[c][r];
            Prim<T> q;
            primitives<SYS, D, T>(Uc, P, q);
            T nu = T(0);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const int st = d == 0 ? 1 : (d == 1 ? W3 : P3);
#pragma unroll
                for (int c = 0; c < M; ++c) {
                    Um[c] = lu[c][r - st];
                    Up[c] = lu[c][r + st];
                }
                add_theta<SYS, D, T>(d, q, Uc, Um, Up, P, nu);
            }
            lnu[i] = nu;
        }
    }
    if constexpr (!kLow) form_coefs();
    __syncthreads();
    const int state = __builtin_amdgcn_readfirstlane(sstate);
    if (state != 0) {
        if (state == 1) {
            if (item == 0 && tid == 0) flag_degenerate(L, n);
            return;
        }
        if (live) {  // at the stop time: the state carries over
            for (int p = 0; p < Q * M; ++p) fout[(int64_t)p * ps + cell] = fin[(int64_t)p * ps + cell];
            for (int p = 0; p < M; ++p) uout[(int64_t)p * ps + cell] = u[(int64_t)p * ps + cell];
        }
        if (item == 0 && tid < kWave) null_scalars(L, n);
        return;
    }
    for (int i = tid; i < G::N1; i += NT) {
        const int wx = i % W1, wy = i / W1 % G::H1, wz = i / P1;
        T w = T(L.omega_fixed);
        if (!fixed) {
            const int r = (wz + 1) * P2 + (wy + 1) * W2 + wx + 1;
            T nt = T(0);
#pragma unroll
            for (int kl = -1; kl <= 1; ++kl)
#pragma unroll
                for (int kj = -1; kj <= 1; ++kj)
#pragma unroll
                    for (int ki = -1; ki <= 1; ++ki) nt = nt + lnu[r + kl * P2 + kj * W2 + ki];
            w = omega_of<T>(nt);
        }
        lw[i] = w;
        if constexpr (SYS == 3) {
            const int r = (wz + 2) * P3 + (wy + 2) * W3 + wx + 2;
            T Uc[M];
#pragma unroll
            for (int c = 0; c < M; ++c) Uc[c] = lu[c][r];
            lrate[i] = -arrhenius_rate<T>(P, Uc[0], reactive_eint<D, T>(Uc), Uc[M - 1], nullptr);
        }
        if (L.omega_on && wx >= 1 && wx <= TX && wy >= 1 && wy <= TY && wz >= 1 && wz <= TZ) {
            const int ox = x0 - 1 + wx, oy = y0 - 1 + wy, oz = z0 - 1 + wz;
            if (ox < nx && oy < ny && oz < nz) ((T *)L.omega)[cell3(L, ox, oy, oz)] = w;
        }
    }
    __syncthreads();
    const Coefs<T> cf = scf;
    T smax[3] = {T(0), T(0), T(0)};
    unsigned flags = 0;
    if (live) {
        const int r3 = (tz + 3) * P3 + (ty + 3) * W3 + tx + 3, r1 = (tz + 1) * P1 + (ty + 1) * W1 + tx + 1;
        const T ak[Q] = {cf.a0, cf.ap[0], cf.ap[1], cf.ap[2], cf.ap[0], cf.ap[1], cf.ap[2]};
        T S[M], last[Q];
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const int dir = k == 0 ? 0 : (k - 1) % 3, sgn = k <= 3 ? 1 : -1;
            const bool own = k == 0 || ((own_m >> k) & 1u), refl = k > 0 && ((refl_m >> k) & 1u);
            const int s3 = own ? r3 : r3 - sgn * (dir == 0 ? 1 : (dir == 1 ? W3 : P3));
            const int s1 = own ? r1 : r1 - sgn * (dir == 0 ? 1 : (dir == 1 ? W1 : P1));
            T Us[M], Fs[M], F[M];
#pragma unroll
            for (int c = 0; c < M; ++c) Us[c] = lu[c][s3];
            if (k > 0) {
                Prim<T> q;
                primitives<SYS, D, T, false>(Us, P, q);
                flux<SYS, D, T>(dir, Us, q, P, Fs);
            }
            const T w = lw[s1], a = ak[k];
            const T bk = (k <= 3) != refl ? cf.bp : cf.bm;
#pragma unroll
            for (int c = 0; c < M; ++c) {
                const T feq = k == 0 ? a * Us[c] : a * Us[c] + bk * Fs[c];
                F[c] = fk[k][c] - w * (fk[k][c] - feq);
                if constexpr (SYS == 3)
                    if (c == M - 1) F[c] = F[c] + cf.hdt * (a * lrate[s1]);
            }
            if (SYS != 0 && refl) F[1 + dir] = -F[1 + dir];
#pragma unroll
            for (int c = 0; c < M; ++c) S[c] = k == 0 ? F[c] : S[c] + F[c];
#pragma unroll
            for (int c = 0; c < (SYS == 3 ? M - 1 : M); ++c) sto(fout + (int64_t)(k * M + c) * ps, cell, F[c]);
            last[k] = F[M - 1];
        }
        if constexpr (SYS == 3) {
            const T eint = reactive_eint<D, T>(S);
            const T z = reactive_solve<T>(P, S[0], eint, S[M - 1], cf.hdt);
            const T SY = -arrhenius_rate<T>(P, S[0], eint, z, nullptr);
#pragma unroll
            for (int k = 0; k < Q; ++k) last[k] = last[k] + cf.hdt * (ak[k] * SY);
            T sn = last[0];
#pragma unroll
            for (int k = 1; k < Q; ++k) sn = sn + last[k];
            S[M - 1] = sn;
#pragma unroll
            for (int k = 0; k < Q; ++k) sto(fout + (int64_t)(k * M + M - 1) * ps, cell, last[k]);
        }
#pragma unroll
        for (int c = 0; c < M; ++c) sto(uout + (int64_t)c * ps, cell, S[c]);
        Prim<T> qn;
        primitives<SYS, D, T>(S, P, qn);
        bool ok = true;
#pragma unroll
        for (int c = 0; c < M; ++c) ok = ok && finite_val<T>(S[c]);
        flags = qn.flags | (ok ? 0u : 1u);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const T v = max_speed<SYS, T>(d, qn, P);
            if (finite_val<T>(v)) smax[d] = v;
        }
    }
    if (item == 0 && tid < kWave) scalar_update(L, n, cf.dt);
    commit<T>(L, n, smax[0], smax[1], flags, 3, smax[2]);
}

}  // namespace arlbm
