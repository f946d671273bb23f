// step_kernels.hip -- the two-pass step (D3Q27 grids the fused z-march does not take) of the
// two-phase LBGK model (Sec. 2.3), the initial state, output fields and pressure tensor, for gfx950.
//
// Storage: structure of arrays A[i*qs + n], n = x + nx*(y + ny*z). The array holds
// post-collision populations at the node that produced them; every pass pulls
// f_i(r) = A_i(r - c_i), or A_opp(i)(r) when r - c_i is solid (halfway bounce-back),
// or with per-link wall fractions an interpolation of A_opp(i) at r and r + c_i or of
// A_opp(i) and A_i at r (interpolated bounce-back).
//
// Pass 1 (moments): rho = rho_ref + sum h_i, j = sum c_i h_i, g_a = rho u_a^3; FP64
//   per-workgroup partial sums of mass and momentum for the watchdog.
// Pass 2 (collide): stages rho and the signed pseudo-potential of a 64x4xZB tile
//   plus a two-node halo in LDS, evaluates the two-ring Korteweg force (eq Kforce_final, or
//   the stencil coefficients of another force model), the diagonal correction Phi (eq
//   correction), the product-form equilibrium and extended equilibrium (eqs LBMeq, LBMstar)
//   in cancellation-free deviation form, and the LBGK update (eq LBGK).
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "kernels.hpp"
#include "lattice.hpp"
#include "step_common.hpp"

namespace lbm {

namespace {

constexpr int TX = 64;   // tile width in x: one wave64 row, coalesced 256 B (FP32) loads
constexpr int TY = 4;    // tile height in y: 4 waves per workgroup
constexpr int HALO = 2;  // two neighbour rings

// ------------------------------------------------------------------ reductions
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// block of 256 threads: sums 5 values in a fixed order, thread 0 writes them
__device__ __forceinline__ void block_sum5(double (&v)[kPartialSlots], double *__restrict__ dst) {
    __shared__ double red[4][kPartialSlots];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < kPartialSlots; ++k) v[k] = wave_sum(v[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < kPartialSlots; ++k) red[wv][k] = v[k];
    __syncthreads();
    if (threadIdx.x < kPartialSlots) {
        const int k = threadIdx.x;
        dst[k] = (red[0][k] + red[1][k]) + (red[2][k] + red[3][k]);
    }
}

// ------------------------------------------------------------------ pass 1
// Moment pass. Only what the caller uses is written: the two-pass step and the pressure tensor
// take rho (and g) in the pitched layout, the output of fields rho and the bare velocity in
// the user layout, a watchdog check the partials alone.
template <int D, class S, class C, bool MASK, class Ix>
__global__ __launch_bounds__(256) void k_moments(const S *__restrict__ A, Geom g, const uint32_t *__restrict__ links,
                                                 Params<C> p, C *__restrict__ rho_out, C *__restrict__ gf,
                                                 double *__restrict__ out_rho, double *__restrict__ out_U,
                                                 double *__restrict__ partials) {
    const int tx = threadIdx.x & (TX - 1), ty = threadIdx.x / TX;
    const int x = blockIdx.x * TX + tx, y = blockIdx.y * TY + ty, z = blockIdx.z;
    double v[kPartialSlots] = {0, 0, 0, 0, 0};
    if (x < g.nx && y < g.ny) {
        const int n = x + g.px * (y + g.ny * z);
        const uint32_t lm = MASK ? links[n] : 0u;
        C rho, u[3] = {C(0), C(0), C(0)};
        if (MASK && link_solid(lm)) {
            rho = wall_density(p, n);
        } else {
            Nbr<D> nb(g, x, y, z);
            C h[Lat<D>::Q];
            gather_links<D, S, C, MASK, Ix>(A, g.qs, lm, nb, n, h, p.link_q);
            C sum, j[3];
            moments_of<D, C>(h, sum, j);
            rho = p.rho_ref + sum;
            const C rinv = rcp(rho);
#pragma unroll
            for (int a = 0; a < D; ++a) u[a] = j[a] * rinv;
            v[0] = double(rho);
            v[1] = double(j[0]);
            v[2] = double(j[1]);
            v[3] = D == 3 ? double(j[2]) : 0.0;
            v[4] = p.eos.in_domain(rho) ? 0.0 : 1.0;
        }
        if (rho_out) rho_out[n] = rho;
        if (gf)
#pragma unroll
            for (int a = 0; a < D; ++a) gf[(long long)a * g.N + n] = rho * u[a] * u[a] * u[a];
        const int un = x + g.nx * (y + g.ny * z);
        if (out_rho) out_rho[un] = double(rho);
        if (out_U)
#pragma unroll
            for (int a = 0; a < D; ++a) out_U[(long long)a * g.nx * g.ny * g.nz + un] = double(u[a]);
    }
    const int blk = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    block_sum5(v, partials + (long long)blk * kPartialSlots);
}

// Solid-neighbour bits, one word per node (bit i: the source node n - c_i is solid; bit LINK_SELF: n is)
template <int D>
__global__ __launch_bounds__(256) void k_links(const uint8_t *__restrict__ mask, uint32_t *__restrict__ links, Geom g) {
    const int n = blockIdx.x * 256 + threadIdx.x;
    if (n >= g.N) return;
    const int x = n % g.px, y = (n / g.px) % g.ny, z = n / (g.px * g.ny);
    if (x >= g.nx) {   // row padding
        links[n] = 0u;
        return;
    }
    const Nbr<D> nb(g, x, y, z);
    uint32_t b = mask[n] ? (1u << LINK_SELF) : 0u;
    static_for<1, Lat<D>::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if (mask[nb.at(-Lat<D>::c(i, 0), -Lat<D>::c(i, 1), -Lat<D>::c(i, 2))]) b |= 1u << i;
    });
    links[n] = b;
}

// ------------------------------------------------------------------ pass 2
template <int D> struct Tile {
    static constexpr int ZB = D == 3 ? 2 : 1;                  // z-planes per workgroup
    static constexpr int LX = TX + 2 * HALO, LY = TY + 2 * HALO;
    static constexpr int LZ = D == 3 ? ZB + 2 * HALO : 1;
    static constexpr int LS = LX * LY * LZ;
};

enum { MODE_STEP = 0, MODE_VEL = 1, MODE_INIT = 2, MODE_PT = 3 };

// MODE_STEP: one collide-stream step A -> B.
// MODE_VEL:  U = u + S/(2 rho) in FP64 (user layout), in place of the bare u in out_U (D2Q9).
// MODE_INIT: equilibrium of the density in rho_f and the flow velocity U0 (= out_U, may be
//            NULL): bare u = U0 - S/(2 rho), written into B in pull layout.
// MODE_PT:   discrete pressure tensor of the state in A (Appendix E) into out_U, FP64
//            [D(D+1)/2][N]: xx, yy, [zz,] xy[, xz, yz]; zero at solid nodes. The lattice
//            momentum flux of the pulled (pre-collision) populations minus the one- and
//            two-ring pseudo-potential and capillary tensors, which enter with the sign of
//            the momentum source S = -F.
template <int D, class S, class C, bool MASK, int MODE, class Ix = unsigned>
__global__ __launch_bounds__(TX *TY) void k_collide(
    const S *__restrict__ A, S *__restrict__ B, Geom g, const uint8_t *__restrict__ mask,
    const uint32_t *__restrict__ links, Params<C> p, const C *__restrict__ rho_f, const C *__restrict__ gf,
    double *__restrict__ out_U) {
    // MODE_INIT has the mask, the others the solid-neighbour bits
    constexpr int NTH = TX * TY;
    using T = Tile<D>;
    __shared__ C s_rho[T::LS];
    __shared__ C s_psi[T::LS];
    const int x0 = blockIdx.x * TX, y0 = blockIdx.y * TY, z0 = D == 3 ? blockIdx.z * T::ZB : 0;
    for (int e = threadIdx.x; e < T::LS; e += NTH) {
        const int lx = e % T::LX, t = e / T::LX, ly = t % T::LY, lz = t / T::LY;
        const int gx = wrapi(x0 - HALO + lx, g.nx), gy = wrapi(y0 - HALO + ly, g.ny);
        const int gz = D == 3 ? wrapi(z0 - HALO + lz, g.nz) : 0;
        const C r = rho_f[gx + g.px * (gy + g.ny * gz)];
        s_rho[e] = r;
        s_psi[e] = signed_psi(p.eos, r);
    }
    __syncthreads();
    const int tx = threadIdx.x & (TX - 1), ty = threadIdx.x / TX;
    const int x = x0 + tx, y = y0 + ty;
    if (x >= g.nx || y >= g.ny) return;
#pragma unroll 1
    for (int zz = 0; zz < T::ZB; ++zz) {
        const int z = z0 + zz;
        if (z >= g.nz) break;
        const int n = x + g.px * (y + g.ny * z);
        const uint32_t lm = MASK && MODE != MODE_INIT ? links[n] : 0u;
        if (MASK && (MODE == MODE_INIT ? mask[n] != 0 : link_solid(lm))) {
            if constexpr (MODE == MODE_PT)
                for (int k = 0; k < D * (D + 1) / 2; ++k) out_U[(long long)k * g.N + n] = 0.0;
            continue;
        }
        const int lc0 = ((D == 3 ? zz + HALO : 0) * T::LY + ty + HALO) * T::LX + tx + HALO;
        if constexpr (MODE == MODE_PT) {
            Nbr<D> nb(g, x, y, z);
            C h[Lat<D>::Q];
            gather_links<D, S, C, MASK, Ix>(A, g.qs, lm, nb, n, h, p.link_q);
            constexpr int NC = D * (D + 1) / 2;
            constexpr int ca[6] = {0, 1, D == 3 ? 2 : 0, 0, 0, 1}, cb[6] = {0, 1, D == 3 ? 2 : 1, 1, 2, 2};
            C flux[NC], ringA[NC], ringB[NC], across[NC], cap1[NC], cap2[NC], capx[NC];
            for (int k = 0; k < NC; ++k) flux[k] = ringA[k] = ringB[k] = across[k] = cap1[k] = cap2[k] = capx[k] = C(0);
            static_for<0, Lat<D>::Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                constexpr int cx = Lat<D>::c(i, 0), cy = Lat<D>::c(i, 1), cz = Lat<D>::c(i, 2);
                constexpr int off = (cz * T::LY + cy) * T::LX + cx;
                constexpr C w3 = C(3.0 * weight<D>(i));
                const C p1 = fabs(s_psi[lc0 + off]), p2 = fabs(s_psi[lc0 + 2 * off]), m1 = fabs(s_psi[lc0 - off]);
                const C r1 = s_rho[lc0 + off], r2 = s_rho[lc0 + 2 * off], rm = s_rho[lc0 - off];
                static_for<0, NC>([&](auto K) {
                    constexpr int k = decltype(K)::value;
                    constexpr int cc = Lat<D>::c(i, ca[k]) * Lat<D>::c(i, cb[k]);
                    if constexpr (cc != 0) {
                        flux[k] += C(cc) * h[i];
                        constexpr C wc = w3 * C(cc);
                        ringA[k] += wc * p1;
                        ringB[k] += wc * p2;
                        across[k] += wc * m1 * p1;
                        cap1[k] += wc * r1;
                        cap2[k] += wc * r2;
                        capx[k] += wc * rm * r1;
                    }
                });
            });
            const C rho = s_rho[lc0], sp = s_psi[lc0];
            const C psi = fabs(sp), sg = sp > C(0) ? C(1) : C(-1);
            for (int k = 0; k < NC; ++k) {
                // Appendix E's parts for the stencil pairs (G1, G2), (G3, G4): each part is
                // linear in its coefficient (printed for 4/3, -1/6, 2 kappa, -kappa)
                const C PA = -sg * p.G[0] * psi * ringA[k];
                const C PB = -sg * p.G[1] * (psi * ringB[k] + across[k]);
                const C PC = C(-0.5) * p.G[2] * rho * cap1[k];
                const C PD = C(-0.5) * p.G[3] * (rho * cap2[k] + capx[k]);
                // FP32 deviation storage: the reference part w_i rho_ref adds rho_ref/3 on the diagonal
                const C kin = flux[k] + (k < D ? p.rho_ref * C(1.0 / 3.0) : C(0));
                out_U[(long long)k * g.N + n] = double(kin) - (double(PA) + double(PB) + double(PC) + double(PD));
            }
            continue;
        }
        const int lc = ((D == 3 ? zz + HALO : 0) * T::LY + ty + HALO) * T::LX + tx + HALO;
        const C rho = s_rho[lc], spc = s_psi[lc];
        C Sf[3] = {C(0), C(0), C(0)};   // S = -F + rho g
        if constexpr (D == 2) {         // as the D2Q9 tiles
            const C gw[8] = {p.gw[0][0], p.gw[1][0], p.gw[0][2], p.gw[1][2], p.gw[0][1], p.gw[1][1], p.gw[0][3], p.gw[1][3]};
            const C accel[2] = {p.accel[0], p.accel[1]};
            C S2[2];
            struct Node { C rho, psi; };
            source_plane<C>(gw, rho, spc, accel, [&](int k, int cx, int cy) __attribute__((always_inline)) {
                const int e = lc + k * (cx + cy * T::LX);
                return Node{s_rho[e], s_psi[e]};
            }, S2);
            Sf[0] = S2[0];
            Sf[1] = S2[1];
        } else {
            C Fp[3] = {C(0), C(0), C(0)}, Fc[3] = {C(0), C(0), C(0)};
            static_for<1, Lat<D>::Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                constexpr int cx = Lat<D>::c(i, 0), cy = Lat<D>::c(i, 1), cz = Lat<D>::c(i, 2);
                constexpr int off = (cz * T::LY + cy) * T::LX + cx;
                constexpr int cls = cx * cx + cy * cy + cz * cz - 1;   // weight class of c_i
                const C p1 = fabs(s_psi[lc + off]), p2 = fabs(s_psi[lc + 2 * off]);
                const C r1 = s_rho[lc + off], r2 = s_rho[lc + 2 * off];
                const C tp = p.gw[cls][0] * p1 + p.gw[cls][1] * p2;   // 3w (G1 psi1 + G2 psi2)
                const C tc = p.gw[cls][2] * r1 + p.gw[cls][3] * r2;   // 3w (G3 rho1 + G4 rho2)
                static_for<0, D>([&](auto A_) {
                    constexpr int a = decltype(A_)::value;
                    constexpr int ca = Lat<D>::c(i, a);
                    if constexpr (ca == 1) { Fp[a] += tp; Fc[a] += tc; }
                    if constexpr (ca == -1) { Fp[a] -= tp; Fc[a] -= tc; }
                });
            });
#pragma unroll
            for (int a = 0; a < D; ++a) Sf[a] = rho * p.accel[a] - (C(2) * spc * Fp[a] + rho * Fc[a]);
        }

        if constexpr (MODE == MODE_VEL) {
            const int un = x + g.nx * (y + g.ny * z);
            const C half = C(0.5) * rcp(rho);
#pragma unroll
            for (int a = 0; a < D; ++a) {
                double *U = out_U + (long long)a * g.nx * g.ny * g.nz + un;
                *U = double(C(*U) + Sf[a] * half);
            }
            continue;
        }
        Nbr<D> nb(g, x, y, z);
        C h[Lat<D>::Q];
        if constexpr (MODE == MODE_INIT) {
            C u[3] = {C(0), C(0), C(0)};
#pragma unroll
            for (int a = 0; a < D; ++a)
                u[a] = (out_U ? C(out_U[(long long)a * g.N + n]) : C(0)) - Sf[a] * (C(0.5) * rcp(rho));
#pragma unroll
            for (int i = 0; i < Lat<D>::Q; ++i) h[i] = C(0);
            // omega = 1 with no source and no correction returns the equilibrium deviation
            const C zero3[3] = {C(0), C(0), C(0)};
            collide<D, C>(h, rho, rho - p.rho_ref, u, zero3, zero3, C(1));
            static_for<0, Lat<D>::Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                constexpr int cx = Lat<D>::c(i, 0), cy = Lat<D>::c(i, 1), cz = Lat<D>::c(i, 2);
                if constexpr (i == 0) {
                    B[n] = S(h[0]);
                } else {
                    // pulled at n from n - c_i, or from opp(i) at n when n - c_i is solid
                    const int src = nb.at(-cx, -cy, -cz);
                    if (MASK && mask[src])
                        B[(long long)opp<D>(i) * g.qs + n] = S(h[i]);
                    else
                        B[(long long)i * g.qs + src] = S(h[i]);
                }
            });
            continue;
        } else {
        gather_links<D, S, C, MASK, Ix>(A, g.qs, lm, nb, n, h, p.link_q);
        C drho, j[3];
        moments_of<D, C>(h, drho, j);
        C u[3] = {C(0), C(0), C(0)};
        const C rinv = rcp(rho);
#pragma unroll
        for (int a = 0; a < D; ++a) u[a] = j[a] * rinv;
        const C omega = omega_of(p, rho);
        C Phi[3] = {C(0), C(0), C(0)};
        const C cf = (C(1) - C(0.5) * omega) * C(0.5);
        Phi[0] = cf * (gf[nb.at(1, 0, 0)] - gf[nb.at(-1, 0, 0)]);
        Phi[1] = cf * (gf[(long long)g.N + nb.at(0, 1, 0)] - gf[(long long)g.N + nb.at(0, -1, 0)]);
        if constexpr (D == 3)
            Phi[2] = cf * (gf[2LL * g.N + nb.at(0, 0, 1)] - gf[2LL * g.N + nb.at(0, 0, -1)]);
        if constexpr (D == 2) {
            const C j2[2] = {j[0], j[1]}, S2[2] = {Sf[0], Sf[1]}, P2[2] = {Phi[0], Phi[1]};
            update_plane<C>(h, rho, drho, rinv, j2, S2, P2, omega);
        } else {
            collide<D, C>(h, rho, drho, u, Sf, Phi, omega);
        }
        static_for<0, Lat<D>::Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            st_nt_at(B + i * g.qs, (Ix)n, S(h[i]));
        });
        }
    }
}

// ------------------------------------------------------------------ velocity (D3Q27)
// U = u + S/(2 rho) in place of the bare u in U (FP64, user layout), from the density field. One
// workgroup marches a TX x TY column of nodes through tz planes with rho and s psi of the last
// planes in an LDS ring: each plane's 68 x 8 densities are read and turned into s psi once
// (2.1 per node; the 64 x 4 x 2 tile of k_collide takes 6.4, whose square roots and divisions
// bound it). Plane z + 3 is loaded before plane z's stencil and stored behind it; with six slots
// one barrier per plane is enough. Bound by the 104 LDS reads per node, then by HBM (56 bytes
// per node): 256^3 FP32 0.215 ms, FP64 0.39 ms, 512x256x256 FP32 with pillars 0.48 ms, against
// 0.59, 1.21 and 4.69 ms for an output pass that gathered the populations once more.
template <class C, bool MASK>
__global__ __launch_bounds__(TX *TY) void k_velocity3(Geom g, const uint32_t *__restrict__ links, Params<C> p,
                                                      const C *__restrict__ rho_f, double *__restrict__ U, int tz) {
    constexpr int LX = TX + 2 * HALO, LY = TY + 2 * HALO, LP = LX * LY, RING = 6, NTH = TX * TY;
    constexpr int PER = (LP + NTH - 1) / NTH;   // staged entries per thread and plane
    __shared__ C s_rho[RING * LP];
    __shared__ C s_psi[RING * LP];
    const int t = threadIdx.x, tx = t & (TX - 1), ty = t / TX;
    const int x0 = blockIdx.x * TX, y0 = blockIdx.y * TY, z0 = blockIdx.z * tz, nzi = min(tz, g.nz - z0);
    const int x = x0 + tx, y = y0 + ty, nxy = g.px * g.ny;
    const bool own = x < g.nx && y < g.ny;
    int at[PER];
#pragma unroll
    for (int m = 0; m < PER; ++m) {
        const int e = t + m * NTH;
        at[m] = e < LP ? wrapi(x0 - HALO + e % LX, g.nx) + g.px * wrapi(y0 - HALO + e / LX, g.ny) : 0;
    }
    auto load = [&](int j, C (&r)[PER]) __attribute__((always_inline)) {   // plane z0 + j
        const C *plane = rho_f + (long long)nxy * wrapi(z0 + j, g.nz);
#pragma unroll
        for (int m = 0; m < PER; ++m) r[m] = plane[at[m]];
    };
    auto stage = [&](int j, const C (&r)[PER]) __attribute__((always_inline)) {
        const int slot = (j + 2) % RING * LP;
#pragma unroll
        for (int m = 0; m < PER; ++m) {
            const int e = t + m * NTH;
            if (e >= LP) break;
            s_rho[slot + e] = r[m];
            s_psi[slot + e] = signed_psi(p.eos, r[m]);
        }
    };
    // the first five planes' loads together, one latency instead of five
    C first[5][PER], r[PER];
#pragma unroll
    for (int j = 0; j < 5; ++j) load(j - 2, first[j]);
#pragma unroll
    for (int j = 0; j < 5; ++j) stage(j - 2, first[j]);
    __syncthreads();
    const int e0 = (ty + HALO) * LX + tx + HALO;
    const long long Nu = (long long)g.nx * g.ny * g.nz;
#pragma unroll 1
    for (int k = 0; k < nzi; ++k) {
        const int z = z0 + k;
        if (k + 1 < nzi) load(k + 3, r);
        const bool act = own && !(MASK && link_solid(links[x + g.px * (y + g.ny * z)]));
        if (act) {
            double *u = U + (x + (long long)g.nx * (y + (long long)g.ny * z));
            const double ub[3] = {u[0], u[Nu], u[2 * Nu]};
            int base[5];
#pragma unroll
            for (int d = 0; d < 5; ++d) base[d] = (k + d) % RING * LP + e0;
            const C rho = s_rho[base[2]], spc = s_psi[base[2]];
            C Fp[3] = {C(0), C(0), C(0)}, Fc[3] = {C(0), C(0), C(0)};
            static_for<1, 27>([&](auto I) {
                constexpr int i = decltype(I)::value;
                constexpr int cx = Lat<3>::c(i, 0), cy = Lat<3>::c(i, 1), cz = Lat<3>::c(i, 2);
                constexpr int o1 = cy * LX + cx, cls = cx * cx + cy * cy + cz * cz - 1;
                const int r1 = base[2 + cz] + o1, r2 = base[2 + 2 * cz] + 2 * o1;
                const C tp = p.gw[cls][0] * fabs(s_psi[r1]) + p.gw[cls][1] * fabs(s_psi[r2]);
                const C tc = p.gw[cls][2] * s_rho[r1] + p.gw[cls][3] * s_rho[r2];
                static_for<0, 3>([&](auto A_) {
                    constexpr int a = decltype(A_)::value;
                    constexpr int ca = Lat<3>::c(i, a);
                    if constexpr (ca == 1) { Fp[a] += tp; Fc[a] += tc; }
                    if constexpr (ca == -1) { Fp[a] -= tp; Fc[a] -= tc; }
                });
            });
            const C half = C(0.5) * rcp(rho);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const C S = rho * p.accel[a] - (C(2) * spc * Fp[a] + rho * Fc[a]);
                u[a * Nu] = double(C(ub[a]) + S * half);
            }
        }
        if (k + 1 < nzi) stage(k + 3, r);
        __syncthreads();
    }
}

// ------------------------------------------------------------------ init
// density field of the initial state in compute precision; solid nodes carry rho_w
template <class C, bool MASK>
__global__ __launch_bounds__(256) void k_prep_rho(C *__restrict__ rho_f, const double *__restrict__ rho0,
                                                  const uint8_t *__restrict__ mask, Params<C> p, int N) {
    const int n = blockIdx.x * 256 + threadIdx.x;
    if (n >= N) return;
    rho_f[n] = (MASK && mask[n]) ? wall_density(p, n) : C(rho0[n]);
}

// Interpolated bounce-back at init. The init kernel folds the equilibrium population i
// of a fluid node n whose source n - c_i is solid into slot opp(i) at n, which only that
// wall link reads. The interpolated pull mixes this slot X with a second entry:
//   q <  1/2: 2q X + (1 - 2q) Y, Y = slot opp(i) at n + c_i (fluid: already f_eq_opp(i)(n);
//             solid: the pull uses X alone)
//   q >= 1/2: a X + (1 - a) Z,  a = 1/(2q), Z = slot i at n (n + c_i fluid: already the
//             equilibrium pulled there; solid: the slot X' of the opposite wall link)
// so X is re-solved for the pull to return the folded value P; the opposite-pair case is a
// 2x2 system with determinant a + a' - 1 (bounded away from 0 by host validation). Only
// the node's own wall slots change, and every entry read is either one of them, read
// before any write, or a regular entry, so nodes are independent.
template <int D, class S, class C>
__global__ __launch_bounds__(256) void k_wall_init(S *__restrict__ A, Geom g, const uint8_t *__restrict__ mask,
                                                   const C *__restrict__ lq) {
    const int n = blockIdx.x * 256 + threadIdx.x;
    if (n >= g.N) return;
    const int x = n % g.px, t = n / g.px, y = t % g.ny, z = t / g.ny;
    if (x >= g.nx || mask[n]) return;   // row padding, or solid
    Nbr<D> nb(g, x, y, z);
    constexpr int Q = Lat<D>::Q;
    C P[Q], X[Q];
    bool wall[Q];
    static_for<1, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr int cx = Lat<D>::c(i, 0), cy = Lat<D>::c(i, 1), cz = Lat<D>::c(i, 2);
        wall[i] = mask[nb.at(-cx, -cy, -cz)] != 0;
        P[i] = wall[i] ? C(A[(long long)opp<D>(i) * g.qs + n]) : C(0);
    });
    static_for<1, Q>([&](auto I) {
        constexpr int i = decltype(I)::value, o = opp<D>(i);
        constexpr int cx = Lat<D>::c(i, 0), cy = Lat<D>::c(i, 1), cz = Lat<D>::c(i, 2);
        X[i] = P[i];
        if (!wall[i]) return;
        const C q = lq[(long long)o * g.qs + n];
        const int b = nb.at(cx, cy, cz);
        const bool bsolid = mask[b] != 0;   // n + c_i solid <=> (n, opp(i)) is a wall link too
        if (q < C(0.5)) {
            if (!bsolid) X[i] = (P[i] - (C(1) - C(2) * q) * C(A[(long long)o * g.qs + b])) / (C(2) * q);
            return;
        }
        const C a = C(1) / (C(2) * q);
        if (!bsolid) {
            X[i] = (P[i] - (C(1) - a) * C(A[(long long)i * g.qs + n])) / a;
            return;
        }
        const C q2 = lq[(long long)i * g.qs + n];
        if (q2 < C(0.5)) {                   // the opposite link keeps its folded value
            X[i] = (P[i] - (C(1) - a) * P[o]) / a;
            return;
        }
        const C a2 = C(1) / (C(2) * q2);
        X[i] = (a2 * P[i] - (C(1) - a) * P[o]) / (a + a2 - C(1));
    });
    static_for<1, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if (wall[i]) A[(long long)opp<D>(i) * g.qs + n] = S(X[i]);
    });
}

template <class S> __global__ __launch_bounds__(256) void k_fill_zero(S *__restrict__ A, long long count) {
    for (long long k = (long long)blockIdx.x * 256 + threadIdx.x; k < count; k += (long long)gridDim.x * 256)
        A[k] = S(0);
}

// One level of the deterministic FP64 tree over partial rows of kPartialSlots values: block b
// sums rows [b R, (b + 1) R) (R = 2048) into out[b]. Each thread adds its eight rows
// t, t + 256, ... in order, then the block halves in LDS; the order depends only on n.
constexpr int kReduceRows = 2048;
__global__ __launch_bounds__(256) void k_reduce(const double *__restrict__ in, int n, double *__restrict__ out) {
    __shared__ double red[256][kPartialSlots];
    double acc[kPartialSlots] = {0, 0, 0, 0, 0};
    const long long r0 = (long long)blockIdx.x * kReduceRows;
    for (int k = 0; k < kReduceRows / 256; ++k) {
        const long long r = r0 + threadIdx.x + 256LL * k;
        if (r < n)
#pragma unroll
            for (int q = 0; q < kPartialSlots; ++q) acc[q] += in[r * kPartialSlots + q];
    }
#pragma unroll
    for (int q = 0; q < kPartialSlots; ++q) red[threadIdx.x][q] = acc[q];
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h)
#pragma unroll
            for (int q = 0; q < kPartialSlots; ++q) red[threadIdx.x][q] += red[threadIdx.x + h][q];
        __syncthreads();
    }
    if (threadIdx.x < kPartialSlots) out[(long long)blockIdx.x * kPartialSlots + threadIdx.x] = red[0][threadIdx.x];
}

// ------------------------------------------------------------------ launchers
dim3 moment_grid(int D, const Geom &g) {
    return dim3((g.nx + TX - 1) / TX, (g.ny + TY - 1) / TY, D == 3 ? g.nz : 1);
}

// Ix: index type of the population arrays (size_t: far_arrays)
template <int D, class S, class C, bool MASK, class Ix> struct Launch {
    static dim3 collide_grid(const Geom &g) {
        return dim3((g.nx + TX - 1) / TX, (g.ny + TY - 1) / TY, D == 3 ? (g.nz + Tile<D>::ZB - 1) / Tile<D>::ZB : 1);
    }
    static void fill_zero(hipStream_t s, void *A, long long count) {
        long long blocks = (count + 255) / 256;
        if (blocks > 65536) blocks = 65536;
        hipLaunchKernelGGL(k_fill_zero<S>, dim3((unsigned)blocks), dim3(256), 0, s, (S *)A, count);
    }
    static void init(hipStream_t s, void *A, const Geom &g, const uint8_t *mask, const void *prm, void *rho,
                     const double *rho0, const double *U0) {
        const Params<C> &p = *(const Params<C> *)prm;
        hipLaunchKernelGGL((k_prep_rho<C, MASK>), dim3((g.N + 255) / 256), dim3(256), 0, s, (C *)rho, rho0, mask,
                           p, g.N);
        hipLaunchKernelGGL((k_collide<D, S, C, MASK, MODE_INIT>), collide_grid(g), dim3(256), 0, s,
                           (const S *)nullptr, (S *)A, g, mask, nullptr, p, (const C *)rho, (const C *)nullptr,
                           (double *)U0);
        if constexpr (MASK)
            if (p.link_q)
                hipLaunchKernelGGL((k_wall_init<D, S, C>), dim3((g.N + 255) / 256), dim3(256), 0, s, (S *)A, g, mask,
                                   p.link_q);
    }
    static void make_links(hipStream_t s, const uint8_t *mask, uint32_t *links, const Geom &g) {
        hipLaunchKernelGGL(k_links<D>, dim3((g.N + 255) / 256), dim3(256), 0, s, mask, links, g);
    }
    static void moments(hipStream_t s, const void *A, const Geom &g, const uint32_t *links, const void *prm, void *rho,
                        void *gfl, double *orho, double *oU, double *partials) {
        hipLaunchKernelGGL((k_moments<D, S, C, MASK, Ix>), moment_grid(D, g), dim3(256), 0, s, (const S *)A, g, links,
                           *(const Params<C> *)prm, (C *)rho, (C *)gfl, orho, oU, partials);
    }
    static void collide(hipStream_t s, const void *A, void *B, const Geom &g, const uint32_t *links, const void *prm,
                        const void *rho, const void *gfl) {
        hipLaunchKernelGGL((k_collide<D, S, C, MASK, MODE_STEP, Ix>), collide_grid(g), dim3(256), 0, s, (const S *)A, (S *)B, g,
                           nullptr, links, *(const Params<C> *)prm, (const C *)rho, (const C *)gfl, nullptr);
    }
    static void pressure(hipStream_t s, const void *A, const Geom &g, const uint32_t *links, const void *prm,
                         const void *rho, double *out) {
        hipLaunchKernelGGL((k_collide<D, S, C, MASK, MODE_PT, Ix>), collide_grid(g), dim3(256), 0, s, (const S *)A,
                           (S *)nullptr, g, nullptr, links, *(const Params<C> *)prm, (const C *)rho, (const C *)nullptr,
                           out);
    }
    static void velocity(hipStream_t s, const Geom &g, const uint32_t *links, const void *prm, const void *rho,
                         double *oU) {
        if constexpr (D == 3) {
            // planes per workgroup: long marches (each re-stages four planes), but about four
            // workgroups per CU while chunks of four planes or more give them; small grids take
            // shorter ones as long as they get by with two per CU (fields in us, chunks of four
            // planes | these: 32^3 FP64 17.6 | 12.5, 64^3 FP32 20.3 | 16.1, FP64 26.2 | 23.1; two
            // planes at 128x128x32 FP64 47.4, four 43.9)
            const long long cols = (long long)((g.nx + TX - 1) / TX) * ((g.ny + TY - 1) / TY), planes = cols * g.nz;
            const int tz = (int)std::min<long long>(32, std::max<long long>(std::min<long long>(4, (planes + 511) / 512), planes / 1024));
            hipLaunchKernelGGL((k_velocity3<C, MASK>),
                               dim3((g.nx + TX - 1) / TX, (g.ny + TY - 1) / TY, (g.nz + tz - 1) / tz), dim3(TX * TY), 0, s, g,
                               links, *(const Params<C> *)prm, (const C *)rho, oU, tz);
        } else {
            hipLaunchKernelGGL((k_collide<D, S, C, MASK, MODE_VEL>), collide_grid(g), dim3(256), 0, s, (const S *)nullptr,
                               (S *)nullptr, g, nullptr, links, *(const Params<C> *)prm, (const C *)rho,
                               (const C *)nullptr, oU);
        }
    }
    static KernelSet set() {
        KernelSet k;
        k.fill_zero = fill_zero;
        k.init = init;
        k.moments = moments;
        k.collide = collide;
        k.links = make_links;
        k.velocity = velocity;
        k.pressure = pressure;
        k.moment_blocks = 0;
        return k;
    }
};

}  // namespace

int moment_block_count(int D, const Geom &g) {
    dim3 gr = moment_grid(D, g);
    return (int)(gr.x * gr.y * gr.z);
}

bool far_arrays(const Geom &g, bool fp64) { return (unsigned long long)g.N * (fp64 ? 8 : 4) > (1ull << 32); }

namespace {
template <int D, class Ix> KernelSet set_of(bool fp64, bool masked) {
    if (fp64) return masked ? Launch<D, double, double, true, Ix>::set() : Launch<D, double, double, false, Ix>::set();
    return masked ? Launch<D, float, float, true, Ix>::set() : Launch<D, float, float, false, Ix>::set();
}
}  // namespace

KernelSet kernel_set(int D, bool fp64, bool masked, bool far) {
    if (D == 2) return far ? set_of<2, size_t>(fp64, masked) : set_of<2, unsigned>(fp64, masked);
    return far ? set_of<3, size_t>(fp64, masked) : set_of<3, unsigned>(fp64, masked);
}

long long reduce_scratch_rows(int n) {
    long long rows = 0;
    for (long long m = n; m > 1;) {
        m = (m + kReduceRows - 1) / kReduceRows;
        rows += m;
    }
    return rows + 1;
}

void launch_reduce(hipStream_t s, const double *partials, int n, double *scratch, double *totals) {
    // levels of k_reduce until one row is left; the intermediate rows go to consecutive
    // regions of scratch, the last level writes totals
    const double *src = partials;
    double *dst = scratch;
    long long m = n;
    do {
        const long long nb = (m + kReduceRows - 1) / kReduceRows;
        double *out = nb == 1 ? totals : dst;
        hipLaunchKernelGGL(k_reduce, dim3((unsigned)(nb > 0 ? nb : 1)), dim3(256), 0, s, src, (int)m, out);
        src = out;
        dst += nb * kPartialSlots;
        m = nb;
    } while (m > 1);
}

}  // namespace lbm
