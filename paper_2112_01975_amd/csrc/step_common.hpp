// step_common.hpp -- device code shared by the two-pass and the fused step kernels:
// pull gather with halfway or interpolated bounce-back, moments, and the deviation-form
// collision.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>

#include "kernels.hpp"
#include "lattice.hpp"

namespace lbm {

__device__ __forceinline__ int wrapi(int v, int n) {
    if ((unsigned)v < (unsigned)n) return v;
    v %= n;
    return v < 0 ? v + n : v;
}

// virtual density of solid node n (Sec. 4.5): per node when a wall field is given
template <class C> __device__ __forceinline__ C wall_density(const Params<C> &p, int n) {
    return p.rho_wf ? p.rho_wf[n] : p.rho_w;
}

template <class C> __device__ __forceinline__ C omega_of(const Params<C> &p, C rho) {
    if (!p.var_visc) return p.omega_l;
    C s = (rho - p.rho_v) / (p.rho_l - p.rho_v);
    s = s < C(0) ? C(0) : (s > C(1) ? C(1) : s);
    C nu = p.nu_v + (p.nu_l - p.nu_v) * s;
    return rcp(C(3) * nu + C(0.5));
}

// wrapped neighbour coordinates of (x, y, z): xs[k] = x + k - 1, ro[j][l] = row offset of (y + j - 1, z + l - 1)
template <int D> struct Nbr {
    int xs[3];
    int ro[3][3];
    __device__ __forceinline__ Nbr(const Geom &g, int x, int y, int z) {
        xs[0] = wrapi(x - 1, g.nx); xs[1] = x; xs[2] = wrapi(x + 1, g.nx);
        int ys[3] = {wrapi(y - 1, g.ny), y, wrapi(y + 1, g.ny)};
        if constexpr (D == 3) {
            int zs[3] = {wrapi(z - 1, g.nz), z, wrapi(z + 1, g.nz)};
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int l = 0; l < 3; ++l) ro[j][l] = g.px * (ys[j] + g.ny * zs[l]);
        } else {
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int l = 0; l < 3; ++l) ro[j][l] = g.px * ys[j];
        }
    }
    // from per-axis wrapped coordinates already multiplied out: xs = x-1, x, x+1;
    // ry = nx * (y-1, y, y+1); pz = nx * ny * (z-1, z, z+1)
    __device__ __forceinline__ Nbr(const int (&xs_)[3], const int (&ry)[3], const int (&pz)[3]) {
#pragma unroll
        for (int k = 0; k < 3; ++k) xs[k] = xs_[k];
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int l = 0; l < 3; ++l) ro[j][l] = ry[j] + pz[l];
    }
    // node index of r + k*c for k = +-1
    __device__ __forceinline__ int at(int dx, int dy, int dz) const { return xs[1 + dx] + ro[1 + dy][1 + dz]; }
};

// Element idx of the array that starts at `base`, addressed as a uniform 64-bit base plus
// a 32-bit byte offset: the compiler then issues global loads/stores with an SGPR base
// and one VGPR offset (saddr form) instead of a 64-bit address per lane. Arrays of more than
// 4 GiB (far_arrays) take Ix = size_t, with 64-bit offsets.
template <class Ix = unsigned, class T> __device__ __forceinline__ T ld_at(const T *__restrict__ base, Ix idx) {
    return *(const T *)((const char *)base + idx * (Ix)sizeof(T));
}
template <class Ix = unsigned, class T> __device__ __forceinline__ void st_at(T *__restrict__ base, Ix idx, T v) {
    *(T *)((char *)base + idx * (Ix)sizeof(T)) = v;
}
// The same store with the non-temporal cache policy, for a lattice that the step writing it
// does not read again (its lines then do not displace the ones being read from L2).
template <class Ix = unsigned, class T> __device__ __forceinline__ void st_nt_at(T *__restrict__ base, Ix idx, T v) {
    __builtin_nontemporal_store(v, (T *)((char *)base + idx * (Ix)sizeof(T)));
}

// Solid-neighbour bits of a node (one word per node, built once per geometry): bit i is set
// when the source node n - c_i of population i is solid, bit LINK_SELF when n is.
constexpr int LINK_SELF = 27;
__device__ __forceinline__ bool link_solid(uint32_t lm) { return (lm >> LINK_SELF) & 1u; }

// Interpolated bounce-back: population i arriving at fluid node n whose source n - c_i is solid.
// Halfway bounce-back returns the opposite post-collision population of n itself, back =
// A_opp(n). With the wall at fraction q of the link, the linearly interpolated bounce-back of
// Bouzidi et al. that the paper uses for curved walls (Sec. 4.5, 5.3):
//   q <  1/2: 2q A_opp(n) + (1 - 2q) A_opp(n + c_i)   (A_opp(n) when n + c_i is solid)
//   q >= 1/2: A_opp(n) / (2q) + (1 - 1/(2q)) A_i(n)
// Both weight pairs sum to one and w_i = w_opp(i), so FP32 deviations interpolate as is.
template <class C>
__device__ __forceinline__ C wall_mix(C q, C back, bool ahead_solid, C ahead, C same) {
    if (q < C(0.5)) return C(2) * q * back + (C(1) - C(2) * q) * (ahead_solid ? back : ahead);
    const C h2q = C(2) * q;
    return back / h2q + (C(1) - C(1) / h2q) * same;
}

// Pull gather of the Q populations arriving at fluid node n with links lm at this time step; lq:
// wall fractions for interpolated bounce-back, or nullptr (halfway). The word of links makes
// every pull one load at a selected address: a mask byte per source node cost as many loads
// again, each before a branch (512x256x256 with pillars, FP32: moment pass 1.30 ms so, 0.83
// with the links).
template <int D, class S, class C, bool MASK, class Ix = unsigned>
__device__ __forceinline__ void gather_links(const S *__restrict__ A, long long qs, uint32_t lm, const Nbr<D> &nb, int n,
                                             C (&h)[Lat<D>::Q], const C *__restrict__ lq) {
    static_for<0, Lat<D>::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr int cx = Lat<D>::c(i, 0), cy = Lat<D>::c(i, 1), cz = Lat<D>::c(i, 2);
        if constexpr (i == 0) {
            h[0] = C(ld_at(A, (Ix)n));
        } else if constexpr (!MASK) {
            h[i] = C(ld_at(A + i * qs, (Ix)nb.at(-cx, -cy, -cz)));
        } else {
            const bool w = (lm >> i) & 1u;
            const S *a = A + (w ? opp<D>(i) * qs : i * qs) + (w ? n : nb.at(-cx, -cy, -cz));
            h[i] = C(*a);
        }
    });
    if (MASK && lq && (lm & ((1u << LINK_SELF) - 1u)))
        static_for<1, Lat<D>::Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            constexpr int o = opp<D>(i);   // the fraction of the link n -> n - c_i is stored under opp(i)
            if ((lm >> i) & 1u)
                h[i] = wall_mix<C>(ld_at(lq + o * qs, (Ix)n), h[i], (lm >> o) & 1u,
                                   C(ld_at(A + o * qs, (Ix)nb.at(Lat<D>::c(i, 0), Lat<D>::c(i, 1), Lat<D>::c(i, 2)))),
                                   C(ld_at(A + i * qs, (Ix)n)));
        });
}

// The same pull with the solid flags of a mask and halfway walls (the batched sweep). Both candidates
// are loaded beside the flag instead of after it (4 cases of 512^2 FP32 41.7 -> 39.8 us a step, 8 of
// 40^3 FP32 90 -> 86), but for FP64 D3Q27, whose registers do not hold them (8 of 40^3 139, 118 so).
template <int D, class S, class C, bool MASK, class Ix = unsigned>
__device__ __forceinline__ void gather(const S *__restrict__ A, long long qs, const uint8_t *__restrict__ mask,
                                       const Nbr<D> &nb, int n, C (&h)[Lat<D>::Q]) {
    static_for<0, Lat<D>::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr int cx = Lat<D>::c(i, 0), cy = Lat<D>::c(i, 1), cz = Lat<D>::c(i, 2);
        if constexpr (i == 0) {
            h[0] = C(ld_at(A, (Ix)n));
        } else {
            const Ix s = (Ix)nb.at(-cx, -cy, -cz);
            if constexpr (MASK) {
                if constexpr (D == 3 && sizeof(C) == 8) {
                    h[i] = ld_at(mask, s) ? C(ld_at(A + opp<D>(i) * qs, (Ix)n)) : C(ld_at(A + i * qs, s));
                } else {
                    const C back = C(ld_at(A + opp<D>(i) * qs, (Ix)n)), from = C(ld_at(A + i * qs, s));
                    h[i] = ld_at(mask, s) ? back : from;
                }
            } else {
                h[i] = C(ld_at(A + i * qs, s));
            }
        }
    });
}

// sum h and j = sum c h in a fixed order (pass 1 and pass 2 must agree bit for bit)
template <int D, class C>
__device__ __forceinline__ void moments_of(const C (&h)[Lat<D>::Q], C &sum, C (&j)[3]) {
    sum = C(0);
    j[0] = j[1] = j[2] = C(0);
    static_for<0, Lat<D>::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        sum += h[i];
        static_for<0, D>([&](auto A) {
            constexpr int a = decltype(A)::value;
            constexpr int ca = Lat<D>::c(i, a);
            if constexpr (ca == 1) j[a] += h[i];
            if constexpr (ca == -1) j[a] -= h[i];
        });
    });
}

// Product-form equilibrium and extended equilibrium in deviation form, then LBGK.
// drho = sum of the pre-collision deviations (the node's mass minus rho_ref).
// Per axis the triplet Psi_c(xi, zeta) = W_c + d_c with W = (1/6, 2/3, 1/6) for
// c = (-1, 0, 1); products are differenced by telescoping so no O(1) terms cancel:
//   f_eq - w rho_ref = drho w + rho [prod(W + d) - prod W]
//   f*   - f_eq      = rho [prod(W + d + D) - prod(W + d)]
// with the x-y parts of both telescoped sums formed once per (c_x, c_y) pair.
// The update f + omega (f_eq - f) + (f* - f_eq) is evaluated as
//   (1 - omega) h + (omega drho) w + rho (omega eqd + fsd).
template <int D, class C>
__device__ __forceinline__ void collide(C (&h)[Lat<D>::Q], C rho, C drho, const C (&u)[3], const C (&S)[3],
                                        const C (&Phi)[3], C omega) {
    constexpr C W0 = C(1.0 / 6.0), W1 = C(2.0 / 3.0);
    C dv[3][3], Av[3][3], Dv[3][3], Bv[3][3];
    const C rinv = rcp(rho);
#pragma unroll
    for (int a = 0; a < D; ++a) {
        const C ua = u[a], u2 = ua * ua;
        dv[a][0] = C(0.5) * (u2 - ua);
        dv[a][1] = -u2;
        dv[a][2] = C(0.5) * (u2 + ua);
        const C s = S[a] * rinv;                           // xi* - u
        const C de = s * (C(2) * ua + s) + Phi[a] * rinv;  // zeta* - zeta_eq
        Dv[a][0] = C(0.5) * (de - s);
        Dv[a][1] = -de;
        Dv[a][2] = C(0.5) * (de + s);
        Av[a][0] = W0 + dv[a][0]; Av[a][1] = W1 + dv[a][1]; Av[a][2] = W0 + dv[a][2];
#pragma unroll
        for (int k = 0; k < 3; ++k) Bv[a][k] = Av[a][k] + Dv[a][k];
    }
    // x-y factors: E = d_x A_y + W_x d_y, F = D_x B_y + A_x D_y, AA = A_x A_y
    C E[3][3], F[3][3], AA[3][3];
#pragma unroll
    for (int kx = 0; kx < 3; ++kx)
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) {
            const C Wx = kx == 1 ? W1 : W0;
            E[kx][ky] = dv[0][kx] * Av[1][ky] + Wx * dv[1][ky];
            F[kx][ky] = Dv[0][kx] * Bv[1][ky] + Av[0][kx] * Dv[1][ky];
            AA[kx][ky] = Av[0][kx] * Av[1][ky];
        }
    const C om1 = C(1) - omega, omd = omega * drho;
    static_for<1, Lat<D>::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr int kx = Lat<D>::c(i, 0) + 1, ky = Lat<D>::c(i, 1) + 1, kz = Lat<D>::c(i, 2) + 1;
        constexpr C WW = (kx == 1 ? W1 : W0) * (ky == 1 ? W1 : W0);
        constexpr C wi = C(weight<D>(i));
        C eqd, fsd;
        if constexpr (D == 2) {
            eqd = E[kx][ky];
            fsd = F[kx][ky];
        } else {
            eqd = Av[2][kz] * E[kx][ky] + WW * dv[2][kz];
            fsd = Bv[2][kz] * F[kx][ky] + AA[kx][ky] * Dv[2][kz];
        }
        h[i] = om1 * h[i] + omd * wi + rho * (omega * eqd + fsd);
    });
    // The update conserves mass exactly (sum heq = drho, sum of the source term = 0), but
    // the rounded weights of the storage precision do not sum to one; taking the rest
    // population as the remainder keeps the per-node mass error an unbiased rounding.
    C rest = drho;
    static_for<1, Lat<D>::Q>([&](auto I) { rest -= h[decltype(I)::value]; });
    h[0] = rest;
}

// D2Q9 force and FP64 update with every multiply-add written out: compiled into several kernels, they
// round alike in each. The rest of a step (moments, psi, the FP32 update of collide()) does too, so
// that steps in tiles of any shape, with a thread per node and in two passes agree bit for bit.

// Momentum source S = -F + rho g (eq Kforce_final) of one node. at(k, x, y) gives the density and
// signed pseudo-potential at r + k (x, y); gw the ring factors of psi (axis, diagonal) and rho of the
// first ring, then of the second. FP32 adds one direction after the other, in the library's
// order. FP64 takes differences first, ten operations per ring and field instead of fourteen
// (summed so, FP32 leaves the sums of earlier states by more than the bounds on its results allow).
template <class C, class At>
__device__ __forceinline__ void source_plane(const C (&gw)[8], C rho, C spsi, const C (&accel)[2], At &&at, C (&S)[2]) {
#pragma clang fp contract(off)
    C Fp[2] = {C(0), C(0)}, Fc[2] = {C(0), C(0)};
    if constexpr (sizeof(C) == 4) {
        static_for<1, 9>([&](auto I) {
            constexpr int i = decltype(I)::value, cx = Lat<2>::c(i, 0), cy = Lat<2>::c(i, 1), o = cx * cy != 0;
            const auto n1 = at(1, cx, cy), n2 = at(2, cx, cy);
            const C tp = fma_c(gw[o], fabs(n1.psi), gw[4 + o] * fabs(n2.psi));
            const C tc = fma_c(gw[2 + o], n1.rho, gw[6 + o] * n2.rho);
            if constexpr (cx == 1) { Fp[0] += tp; Fc[0] += tc; }
            if constexpr (cx == -1) { Fp[0] -= tp; Fc[0] -= tc; }
            if constexpr (cy == 1) { Fp[1] += tp; Fc[1] += tc; }
            if constexpr (cy == -1) { Fp[1] -= tp; Fc[1] -= tc; }
        });
    } else {
#pragma unroll
        for (int k = 1; k <= 2; ++k) {
            const int o = 4 * (k - 1);
            const auto E = at(k, 1, 0), W = at(k, -1, 0), N = at(k, 0, 1), So = at(k, 0, -1);
            const auto NE = at(k, 1, 1), SW = at(k, -1, -1), SE = at(k, 1, -1), NW = at(k, -1, 1);
            auto ring = [&](C (&F)[2], C a, C b, C e, C w, C n, C s, C ne, C sw, C se, C nw) __attribute__((always_inline)) {
#pragma clang fp contract(off)
                const C d1 = ne - sw, d2 = se - nw;
                F[0] = fma_c(a, e - w, fma_c(b, d1 + d2, F[0]));
                F[1] = fma_c(a, n - s, fma_c(b, d1 - d2, F[1]));
            };
            ring(Fp, gw[o], gw[o + 1], fabs(E.psi), fabs(W.psi), fabs(N.psi), fabs(So.psi), fabs(NE.psi), fabs(SW.psi), fabs(SE.psi),
                 fabs(NW.psi));
            ring(Fc, gw[o + 2], gw[o + 3], E.rho, W.rho, N.rho, So.rho, NE.rho, SW.rho, SE.rho, NW.rho);
        }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a) S[a] = fma_c(rho, accel[a], -fma_c(C(2) * spsi, Fp[a], rho * Fc[a]));
}

// The D2Q9 update of collide() with the terms of each direction gathered by axis. With d = Psi - W
// and D = Psi* - Psi per axis, A = W + d:
//   omega (f_eq - w rho_ref) + (f* - f_eq)
//     = A_y rho (omega d_x + D_x) + D_y rho (A_x + D_x) + W_x (omega rho d_y + omega drho W_y),
// again without O(1) terms that cancel: three multiply-adds per direction, where the general form
// takes eight operations. rinv = 1 / rho. FP64 only (update_plane): FP32 keeps the general form, whose
// density error is a third of this one's after 300 steps of a drop (2e-6 against 6e-6).
template <class C>
__device__ __forceinline__ void collide_plane(C (&h)[9], C rho, C drho, C rinv, const C (&j)[2], const C (&S)[2],
                                              const C (&Phi)[2], C omega) {
#pragma clang fp contract(off)
    constexpr C W[3] = {C(1.0 / 6.0), C(2.0 / 3.0), C(1.0 / 6.0)};
    C d[2][3], D[2][3];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const C ua = j[a] * rinv, u2 = ua * ua;
        d[a][0] = C(0.5) * (u2 - ua);
        d[a][1] = -u2;
        d[a][2] = C(0.5) * (u2 + ua);
        const C s = S[a] * rinv;                                        // xi* - u
        const C de = fma_c(s, fma_c(C(2), ua, s), Phi[a] * rinv);       // zeta* - zeta_eq
        D[a][0] = C(0.5) * (de - s);
        D[a][1] = -de;
        D[a][2] = C(0.5) * (de + s);
    }
    C P[3], R[3], Ay[3], V[3][2];
    const C om1 = C(1) - omega, orho = omega * rho, omd = omega * drho;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        P[k] = rho * fma_c(omega, d[0][k], D[0][k]);
        R[k] = rho * ((W[k] + d[0][k]) + D[0][k]);
        Ay[k] = W[k] + d[1][k];
        const C v = fma_c(orho, d[1][k], omd * W[k]);
        V[k][0] = W[0] * v;
        V[k][1] = W[1] * v;
    }
    C rest = drho;
    static_for<1, 9>([&](auto I) {
        constexpr int i = decltype(I)::value, kx = Lat<2>::c(i, 0) + 1, ky = Lat<2>::c(i, 1) + 1;
        h[i] = fma_c(om1, h[i], fma_c(Ay[ky], P[kx], fma_c(D[1][ky], R[kx], V[ky][kx == 1])));
        rest -= h[i];
    });
    h[0] = rest;   // the remainder, as in collide()
}

template <class C>
__device__ __forceinline__ void update_plane(C (&h)[9], C rho, C drho, C rinv, const C (&j)[2], const C (&S)[2],
                                             const C (&Phi)[2], C omega) {
    if constexpr (sizeof(C) == 8) {
        collide_plane<C>(h, rho, drho, rinv, j, S, Phi, omega);
    } else {
        const C u[3] = {j[0] * rinv, j[1] * rinv, C(0)}, S3[3] = {S[0], S[1], C(0)}, P3[3] = {Phi[0], Phi[1], C(0)};
        collide<2, C>(h, rho, drho, u, S3, P3, omega);
    }
}

}  // namespace lbm
