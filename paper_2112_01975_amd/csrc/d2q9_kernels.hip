// d2q9_kernels.hip -- the D2Q9 stream-collide step, one to kMaxTileSteps steps per launch (gfx950).
//
// A workgroup advances a tile of tx x ty nodes by nsteps steps in LDS. Step s (of nsteps, r =
// nsteps - 1 - s steps still to come) needs the densities of the tile widened by m = 2 + 3 r
// nodes on every side (one node for the pull of the next step, two for the ring stencils of the
// nodes it pulls from) and collides the tile widened by m - 2:
//   fields:  every node of the widened tile pulls its populations, from the lattice in step 0 and
//            from LDS afterwards (halfway or interpolated bounce-back at solid links), and leaves
//            rho, s psi and g = rho u^3 in LDS; the populations stay in registers;
//   collide: two-ring force (eq Kforce_final) and correction (eq correction) from LDS, LBGK
//            update (eqs LBMeq, LBMstar, LBGK) in registers, post-collision populations back to
//            LDS, or in the last step to the other lattice.
// Nodes outside the tile are recomputed by the neighbouring workgroups. One loop body serves
// every step of a tile, and the arithmetic rounds alike in every instance and in the other D2Q9
// kernels, so the state does not depend on the tile or on how a run is cut into launches, bit for bit.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "d2q9.hpp"
#include "lattice.hpp"
#include "step_common.hpp"

namespace lbm {

namespace {

constexpr int kXcds = 8;         // MI355X: workgroups are dealt to 8 XCDs in turn
constexpr int kXcdChunk = 128;   // consecutive tiles per XCD chunk, at most

// node e of a region of width w: row e / w by a multiplication, exact while e w < 2^20 with
// inv = 2^20 / w + 1
__device__ __forceinline__ int row_of(int e, unsigned inv) { return (int)(((unsigned)e * inv) >> 20); }

// A uniform value kept in a vector register. The step's constants take more scalar registers
// than there are beside the addresses; spilled, each use costs two lane reads.
__device__ __forceinline__ float in_vgpr(float v) { asm volatile("" : "+v"(v)); return v; }
__device__ __forceinline__ double in_vgpr(double v) { asm volatile("" : "+v"(v)); return v; }
// An opaque zero: an address with it added is computed where it is used, and not held in scalar
// registers over the step loop.
__device__ __forceinline__ long long here() {
    long long z = 0;
    asm volatile("" : "+s"(z));
    return z;
}

// wrapi with one addition for all but the smallest grids
__device__ __forceinline__ int wrap1(int v, int n) {
    v = v < 0 ? v + n : (v >= n ? v - n : v);
    return wrapi(v, n);
}

template <class C> struct alignas(2 * sizeof(C)) Pair { C rho, psi; };   // psi signed

// quotient of n by a uniform d with inv = min(ceil(2^32 / d), 2^32 - 1): the estimate is off by one at most
__device__ __forceinline__ int quotient(int n, int d, unsigned inv, int &rem) {
    int q = (int)__umulhi((unsigned)n, inv);
    rem = n - q * d;
    if (rem < 0) { --q; rem += d; }
    if (rem >= d) { ++q; rem -= d; }
    return q;
}

// tile of this workgroup (false: padding). The hardware deals workgroups to the XCDs in turn; the
// tiles, in row-major order, go to them in chunks of equal numbers of consecutive tiles, so that
// neighbouring tiles mostly share an XCD and read each other's halo from its L2, and each XCD gets
// as many (chunks of 128 with a remainder left some XCDs twice the work: 1000x900 FP32 22.8
// us a step, in equal shares 16.8).
__device__ __forceinline__ bool tile_of_block(const D2Tiles &tl, int &ix, int &iy) {
    int k;
    const int c = quotient((int)(blockIdx.x / kXcds), tl.chunk, tl.inv_chunk, k);
    const int tile = (c * kXcds + (int)(blockIdx.x % kXcds)) * tl.chunk + k;
    if (tile >= tl.ntx * tl.nty) return false;
    iy = quotient(tile, tl.ntx, tl.inv_ntx, ix);
    return true;
}

// Collides one node: force and correction from the LDS fields around it (rp, gx, gy point at the
// node's entries, rows of W), the populations in h updated in place. gw: ring factors of psi
// (axis, diagonal) and rho of the first ring, then of the second.
template <class C>
__device__ __forceinline__ void update_node(const Params<C> &p, const C (&gw)[8], const Pair<C> *rp, const C *gx, const C *gy,
                                            int W, C rho_ref, C accx, C accy, C drho, C rinv, C spsi, const C (&j)[2],
                                            C (&h)[9]) {
    const C rho = rho_ref + drho;
    const C accel[2] = {accx, accy};
    C S2[2];
    source_plane<C>(gw, rho, spsi, accel, [&](int k, int x, int y) __attribute__((always_inline)) { return rp[k * (x + y * W)]; }, S2);
    const C omega = omega_of(p, rho), cf = (C(1) - C(0.5) * omega) * C(0.5);
    const C Phi[2] = {cf * (gx[1] - gx[-1]), cf * (gy[W] - gy[-W])};
    update_plane<C>(h, rho, drho, rinv, j, S2, Phi, omega);
}

// Bound by the vector instructions of the nodes and their halo, with the launch itself on small
// grids: per launch of two steps of 32 x 32 tiles (512^2 FP32, 10 us) 1 us prologue, 2.5 us pulls,
// 2.5 us first step, 2.5 us second step, 2 us gap to the next launch. What a step costs is its
// instruction count, so constants sit in vector registers, and in FP64 the force takes differences
// before factors and the update gathers its terms by axis (collide_plane). Holding a frame of
// populations in LDS, loaded with 16-byte copies, was slower (5.5 against 5.1 us a step).
template <class S, class C, bool MASK, int NT, int NPT>
__global__ __launch_bounds__(NT) void k_d2q9(const S *__restrict__ A, S *__restrict__ B, Geom g,
                                             const uint32_t *__restrict__ links, Params<C> p, D2Tiles tl) {
    constexpr int Q = 9, F0 = d2_fields(NT, NPT), P0 = d2_pops(NT, NPT);
    extern __shared__ __align__(16) char lds[];
    int ix, iy;
    if (!tile_of_block(tl, ix, iy)) return;   // the padding of the last XCD's share (whole workgroup)
    const int x0 = ix * tl.tx, y0 = iy * tl.ty;

    const int t = threadIdx.x;
    Pair<C> *const s_rp = (Pair<C> *)lds;
    C *const s_gx = (C *)(s_rp + F0), *const s_gy = s_gx + F0;
    S *const s_pop = (S *)(s_gy + F0);
    int *const s_col = (int *)(s_pop + (tl.nsteps > 1 ? Q * P0 : 0));
    // wrapped columns and row offsets of the first step's region and one node around it
    const int m0 = 3 * tl.nsteps, W0 = tl.tx + 2 * m0, H0 = tl.ty + 2 * m0;
    int *const s_row = s_col + W0;
    for (int k = t; k < W0 + H0; k += NT) s_col[k] = k < W0 ? wrap1(x0 - m0 + k, g.nx) : g.px * wrap1(y0 - m0 + k - W0, g.ny);

    const C gw[8] = {in_vgpr(p.gw[0][0]), in_vgpr(p.gw[1][0]), in_vgpr(p.gw[0][2]), in_vgpr(p.gw[1][2]),
                     in_vgpr(p.gw[0][1]), in_vgpr(p.gw[1][1]), in_vgpr(p.gw[0][3]), in_vgpr(p.gw[1][3])};
    const C rho_ref = in_vgpr(p.rho_ref), accx = in_vgpr(p.accel[0]), accy = in_vgpr(p.accel[1]);
    // waves past a region's end skip (a scalar branch); the lanes of its last wave that are past
    // it repeat its last node, so that little here is conditional per lane
    const int w0 = __builtin_amdgcn_readfirstlane(t & ~63);
    __syncthreads();

    for (int st = 0; st < tl.nsteps; ++st) {
        const int rem = tl.nsteps - 1 - st, m = 2 + 3 * rem;
        const int W = tl.tx + 2 * m, H = tl.ty + 2 * m, F = W * H;
        const unsigned inv = tl.inv[rem];
        C h[NPT][Q];
        C drho[NPT], jx[NPT], jy[NPT], rinv[NPT], spsi[NPT];
        uint32_t lm[NPT];
        // pulls of every node of this thread (a run-time first step, so that the compiler peels no
        // copy of the body for it)
        if (st == tl.first) {
            const S *const Ah = A + here();
#pragma unroll
            for (int k = 0; k < NPT; ++k) {
                if (w0 + k * NT >= F) break;
                const int e = min(t + k * NT, F - 1), ry = row_of(e, inv), rx = e - ry * W;
                const int xs[3] = {s_col[rx], s_col[rx + 1], s_col[rx + 2]};
                const int ro[3] = {s_row[ry], s_row[ry + 1], s_row[ry + 2]};
                const int pz[3] = {0, 0, 0};
                const Nbr<2> nb(xs, ro, pz);
                const int n = xs[1] + ro[1];
                lm[k] = MASK ? links[n] : 0u;
                gather_links<2, S, C, MASK>(Ah, g.qs, lm[k], nb, n, h[k], p.link_q);
            }
        } else {
            const int Wp = W + 2;   // the region the previous step collided: one node wider on each side
#pragma unroll
            for (int k = 0; k < NPT; ++k) {
                if (w0 + k * NT >= F) break;
                const int e = min(t + k * NT, F - 1), ry = row_of(e, inv), rx = e - ry * W;
                const int o = rx + 1 + (ry + 1) * Wp;
                const int n = MASK ? s_col[rx + 1 + 3 * st] + s_row[ry + 1 + 3 * st] : 0;
                lm[k] = MASK ? links[n] : 0u;
                static_for<0, Q>([&](auto I) {
                    constexpr int i = decltype(I)::value, cx = Lat<2>::c(i, 0), cy = Lat<2>::c(i, 1);
                    const bool w = MASK && ((lm[k] >> i) & 1u);
                    h[k][i] = C(s_pop[w ? opp<2>(i) * P0 + o : i * P0 + o - cx - cy * Wp]);
                });
                if (MASK && p.link_q && (lm[k] & ((1u << LINK_SELF) - 1u)))
                    static_for<1, Q>([&](auto I) {   // interpolated bounce-back, as in gather_links
                        constexpr int i = decltype(I)::value, q_ = opp<2>(i);
                        constexpr int cx = Lat<2>::c(i, 0), cy = Lat<2>::c(i, 1);
                        if ((lm[k] >> i) & 1u)
                            h[k][i] = wall_mix<C>(ld_at(p.link_q + q_ * g.qs, (unsigned)n), h[k][i], (lm[k] >> q_) & 1u,
                                                  C(s_pop[q_ * P0 + o + cx + cy * Wp]), C(s_pop[i * P0 + o]));
                    });
            }
        }
        // rho, s psi and g of every node
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            if (w0 + k * NT >= F) break;
            const int e = min(t + k * NT, F - 1);
            C j[3];
            moments_of<2, C>(h[k], drho[k], j);
            C rho = rho_ref + drho[k];
            jx[k] = j[0];
            jy[k] = j[1];
            rinv[k] = rcp(rho);
            C ga[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const C ua = j[a] * rinv[k];
                ga[a] = rho * ua * ua * ua;
            }
            if (MASK && link_solid(lm[k])) {
                rho = p.rho_w;
                if (p.rho_wf) {
                    const int ry = row_of(e, inv), rx = e - ry * W;
                    rho = p.rho_wf[s_col[rx + 1 + 3 * st] + s_row[ry + 1 + 3 * st]];
                }
                ga[0] = ga[1] = C(0);
            }
            spsi[k] = signed_psi(p.eos, rho);
            s_rp[e] = Pair<C>{rho, spsi[k]};
            s_gx[e] = ga[0];
            s_gy[e] = ga[1];
        }
        __syncthreads();
        // force, correction, collision
        const int Wc = W - 4;
        S *const Bh = B + here();
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            if (w0 + k * NT >= F) break;
            const int e = min(t + k * NT, F - 1), ry = row_of(e, inv), rx = e - ry * W;
            if ((unsigned)(rx - 2) < (unsigned)Wc && (unsigned)(ry - 2) < (unsigned)(H - 4) &&
                !(MASK && link_solid(lm[k]))) {
                const C j[2] = {jx[k], jy[k]};
                update_node<C>(p, gw, s_rp + e, s_gx + e, s_gy + e, W, rho_ref, accx, accy, drho[k], rinv[k], spsi[k], j, h[k]);
                if (rem) {
                    const int o = rx - 2 + (ry - 2) * Wc;
                    static_for<0, Q>([&](auto I) {
                        constexpr int i = decltype(I)::value;
                        s_pop[i * P0 + o] = S(h[k][i]);
                    });
                } else {
                    const int x = x0 + rx - 2, y = y0 + ry - 2;
                    if (x < g.nx && y < g.ny)
                        static_for<0, Q>([&](auto I) {
                            constexpr int i = decltype(I)::value;
                            st_nt_at(Bh + i * g.qs, (unsigned)(x + g.px * y), S(h[k][i]));
                        });
                }
            }
        }
        if (rem) __syncthreads();   // the next step pulls these populations and overwrites the fields
    }
}

// One step per launch on a 64 x 8 tile, one thread per tile node, 304 of which also pull one node of
// the two-node halo. Only the tile's own nodes are collided and kept in registers, and two
// workgroups share a CU, so this moves a large FP64 grid faster than the tiles above, whose
// recomputed halo costs more there than the launches and traffic they save: 2040x1900 FP64 115 to
// 121 us a step (by placement in memory), 4.6 to 4.9 TB/s of populations against 5.4 for a copy, and
// 126 in tiles. NT: see d2_stream.
constexpr int SX = 64, SY = 8, SHALO = 2;
template <class S, class C, bool MASK, class Ix, bool NT>
__global__ __launch_bounds__(SX *SY) void k_d2q9_single(const S *__restrict__ A, S *__restrict__ B, Geom g,
                                                        const uint32_t *__restrict__ links, Params<C> p, D2Tiles tl) {
    constexpr int LX = SX + 2 * SHALO, LY = SY + 2 * SHALO, LS = LX * LY, NTH = SX * SY, NH = LS - NTH;
    static_assert(NH <= NTH, "one halo node per thread at most");
    __shared__ Pair<C> s_rp[LS];
    __shared__ C s_gx[LS], s_gy[LS];
    int ix, iy;
    if (!tile_of_block(tl, ix, iy)) return;   // the padding of the last XCD's share (whole workgroup)
    const int x0 = ix * SX, y0 = iy * SY;
    // every thread its own tile node (wrapped past the grid's edge: those feed the stencils of the
    // last columns and rows), and at most one halo node: rows 0, 1, LY-2, LY-1 of the staged
    // tile, then columns 0, 1, LX-2, LX-1 of the rows between. Both nodes' pulls are issued
    // before either is reduced.
    const int t = threadIdx.x, tx = t & (SX - 1), ty = t / SX;
    const bool has_halo = t < NH;
    int lx = 0, ly = 0;
    if (t < 4 * LX) {
        const int r = t / LX;
        lx = t % LX;
        ly = r < 2 ? r : SY + r;
    } else if (has_halo) {
        const int q = t - 4 * LX, c4 = q % 4;
        ly = 2 + q / 4;
        lx = c4 < 2 ? c4 : SX + c4;
    }
    const int e = (ty + SHALO) * LX + tx + SHALO, e_halo = ly * LX + lx;
    const int ox = wrap1(x0 + tx, g.nx), oy = wrap1(y0 + ty, g.ny);
    const int hx = wrap1(x0 - SHALO + lx, g.nx), hy = wrap1(y0 - SHALO + ly, g.ny);
    const int on = ox + g.px * oy, hn = hx + g.px * hy;
    const uint32_t olm = MASK ? links[on] : 0u, hlm = MASK && has_halo ? links[hn] : 0u;
    C h[9], hh[9];
    if (!link_solid(olm)) gather_links<2, S, C, MASK, Ix>(A, g.qs, olm, Nbr<2>(g, ox, oy, 0), on, h, p.link_q);
    if (has_halo && !link_solid(hlm)) gather_links<2, S, C, MASK, Ix>(A, g.qs, hlm, Nbr<2>(g, hx, hy, 0), hn, hh, p.link_q);
    C drho = C(0), rinv = C(0), spsi = C(0), jj[2] = {C(0), C(0)};
    auto stage = [&](int at, int n, uint32_t lm, const C (&hs)[9], bool own) __attribute__((always_inline)) {
        C rho, ga[2] = {C(0), C(0)};
        if (MASK && link_solid(lm)) {
            rho = wall_density(p, n);
        } else {
            C sum, j[3];
            moments_of<2, C>(hs, sum, j);
            rho = p.rho_ref + sum;
            const C ri = rcp(rho);
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const C ua = j[a] * ri;
                ga[a] = rho * ua * ua * ua;
            }
            if (own) { drho = sum; rinv = ri; jj[0] = j[0]; jj[1] = j[1]; }
        }
        const C sp = signed_psi(p.eos, rho);
        if (own) spsi = sp;
        s_rp[at] = Pair<C>{rho, sp};
        s_gx[at] = ga[0];
        s_gy[at] = ga[1];
    };
    stage(e, on, olm, h, true);
    if (has_halo) stage(e_halo, hn, hlm, hh, false);
    __syncthreads();
    const int x = x0 + tx, y = y0 + ty;
    if (x >= g.nx || y >= g.ny || link_solid(olm)) return;
    const C gw[8] = {p.gw[0][0], p.gw[1][0], p.gw[0][2], p.gw[1][2], p.gw[0][1], p.gw[1][1], p.gw[0][3], p.gw[1][3]};
    update_node<C>(p, gw, s_rp + e, s_gx + e, s_gy + e, LX, p.rho_ref, p.accel[0], p.accel[1], drho, rinv, spsi, jj, h);
    const Ix n = (Ix)(x + g.px * y);
    static_for<0, 9>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if constexpr (NT) st_nt_at(B + i * g.qs, n, S(h[i]));
        else st_at(B + i * g.qs, n, S(h[i]));
    });
}

// workgroups of a launch: its tiles, padded to a whole number of chunks per XCD
unsigned blocks(const D2Tiles &t) {
    const int nt = t.ntx * t.nty, per = kXcds * t.chunk;
    return (unsigned)((nt + per - 1) / per) * (unsigned)per;
}

// workgroup shapes: threads x nodes per thread (0: the single step)
template <class S, class C, bool MASK, int NT, int NPT>
void launch(hipStream_t s, const void *A, void *B, const Geom &g, const uint32_t *links, const void *prm,
            const D2Tiles &t) {
    hipLaunchKernelGGL((k_d2q9<S, C, MASK, NT, NPT>), dim3(blocks(t)), dim3(NT), t.lds, s,
                       (const S *)A, (S *)B, g, links, *(const Params<C> *)prm, t);
}

template <class S, class C, bool MASK, class Ix>
void launch_single(hipStream_t s, const void *A, void *B, const Geom &g, const uint32_t *links, const void *prm,
                   const D2Tiles &t) {
    auto *kernel = t.stream ? k_d2q9_single<S, C, MASK, Ix, true> : k_d2q9_single<S, C, MASK, Ix, false>;
    hipLaunchKernelGGL(kernel, dim3(blocks(t)), dim3(SX * SY), 0, s, (const S *)A, (S *)B, g, links, *(const Params<C> *)prm, t);
}

template <class S, class C, bool MASK>
D2Launch pick(int threads, int per) {
    if (threads == SX * SY && per == 0) return launch_single<S, C, MASK, unsigned>;
    if (threads == 256 && per == 1) return launch<S, C, MASK, 256, 1>;
    if (threads == 512 && per == 2) return launch<S, C, MASK, 512, 2>;
    if (threads == 512 && per == 3) return launch<S, C, MASK, 512, 3>;
    if constexpr (sizeof(C) == 4)   // FP64 does not fit the 128 registers of 1024 threads
        if (threads == 1024 && per == 2) return launch<S, C, MASK, 1024, 2>;
    return nullptr;
}

}  // namespace

D2Tiles d2_tiles(const Geom &g, bool fp64, const D2Shape &sh, int nsteps) {
    D2Tiles t;
    t.tx = sh.tx;
    t.ty = sh.ty;
    t.ntx = (g.nx + t.tx - 1) / t.tx;
    t.nty = (g.ny + t.ty - 1) / t.ty;
    t.nsteps = nsteps;
    t.first = 0;
    t.stream = d2_stream(g, fp64);
    const int nt = t.ntx * t.nty, full = kXcds * kXcdChunk, rounds = (nt + full - 1) / full;
    t.chunk = (nt + kXcds * rounds - 1) / (kXcds * rounds);
    auto inverse = [](int d) { return (unsigned)std::min<unsigned long long>(((1ull << 32) + d - 1) / d, 0xFFFFFFFFull); };
    t.inv_chunk = inverse(t.chunk);
    t.inv_ntx = inverse(t.ntx);
    const int m0 = 3 * nsteps;
    t.lds = (size_t)(fp64 ? 8 : 4) * (4 * (size_t)d2_fields(sh.threads, sh.per) +
                                      (nsteps > 1 ? 9 * (size_t)d2_pops(sh.threads, sh.per) : 0)) +
            sizeof(int) * (size_t)(t.tx + t.ty + 4 * m0);
    for (int r = 0; r < kMaxTileSteps; ++r) t.inv[r] = (1u << 20) / (unsigned)(t.tx + 2 * (2 + 3 * r)) + 1u;
    return t;
}

// Non-temporal stores keep the lattice being read in the L2s while both fit there (32 MB), and
// make no difference to a lattice that has to come from HBM again. Between the two the next
// step finds an ordinarily stored lattice in the 256 MB memory-side cache. us per step,
// non-temporal | ordinary, by the two lattices' size:
//   FP32  22 MB 6.1 | 6.9    32 MB 10.3 | 8.5   141 MB 35.4 | 26.1   264 MB 61.2 | 55.6   302 MB 68.9 | 73.7
//   FP64  32 MB 8.5 | 8.7    38 MB  9.9 | 9.4   151 MB 35.9 | 30.4   274 MB 60.6 | 60.1   560 MB 115 | 124
bool d2_stream(const Geom &g, bool fp64) {
    const double mb = 18e-6 * (fp64 ? 8 : 4) * (double)g.qs;
    return mb < (fp64 ? 33.5 : 30.0) || mb > 268.0;
}

bool d2_fits(bool fp64, const D2Shape &sh) {
    if (sh.per == 0) return sh.threads == SX * SY && sh.tx == SX && sh.ty == SY && sh.steps == 1;
    if (sh.steps < 1 || sh.steps > kMaxTileSteps || sh.tx < 1 || sh.ty < 1 || sh.tx > 192 || sh.ty > 192) return false;
    const int m = 2 + 3 * (sh.steps - 1), w = sh.tx + 2 * m, h = sh.ty + 2 * m;
    return w * h <= d2_fields(sh.threads, sh.per) && (sh.steps == 1 || (w - 4) * (h - 4) <= d2_pops(sh.threads, sh.per)) &&
           d2_tiles(Geom{1, 1, 1, 1, 1, 1}, fp64, sh, sh.steps).lds <= 160 * 1024;
}

D2Launch d2_far_launcher(bool fp64, bool masked) {
    if (fp64) return masked ? launch_single<double, double, true, size_t> : launch_single<double, double, false, size_t>;
    return masked ? launch_single<float, float, true, size_t> : launch_single<float, float, false, size_t>;
}

D2Launch d2_launcher(bool fp64, bool masked, const D2Shape &sh) {
    if (fp64) return masked ? pick<double, double, true>(sh.threads, sh.per) : pick<double, double, false>(sh.threads, sh.per);
    return masked ? pick<float, float, true>(sh.threads, sh.per) : pick<float, float, false>(sh.threads, sh.per);
}

// The choice of the tiles: the least estimated time per step.
// A launch costs about 4 us whatever it does (the gap to the next one, the prologue, the first
// loads' latency). A workgroup then takes the vector instructions of its nodes, step by step with
// their halo (0.133 us per 64 nodes and step in FP32, 0.25 in FP64), and its share of the memory
// traffic (21 GB/s per CU); the two overlap in part. So small grids take several steps of tiny
// tiles per launch, larger ones two steps of larger tiles.
// One step per launch with a thread per node is faster, and taken, on FP64 grids past 190,000 nodes
// (bound by memory and by the halo's FP64 arithmetic), and on FP32 grids from 275,000 nodes (the
// tiles' second round on the CUs) to lattices of 268 MB (d2_stream), but for flat or narrow ones,
// whose rows of tiles are spread over several XCDs or whose lanes are idle. Measured us per
// step: best tiles | one thread per node of 64 x 8 tiles:
//   FP64  64^2 2.6 | 5.0    256^2 3.9 | 5.5     400x380 5.7 | 7.0   448x440 9.3 | 8.1   2040x1900 126 | 115
//   FP32  64^2 2.2 | 4.0    256^2 3.0 | 4.2     512^2 5.1 | 5.7     353x852 7.1 | 6.1   641x482 7.3 | 6.2
//         640^2 8.3 | 8.0   922x488 10.1 | 8.5  800^2 13.1 | 11.7   1500x1300 31 | 26   2048^2 60 | 69
//         20000x16 6.6 | 8.4
D2Shape d2_plan(const Geom &g, bool fp64, bool masked, int cus) {
    static constexpr int shapes[][2] = {{256, 1}, {512, 2}, {512, 3}, {1024, 2}};
    const int size = fp64 ? 8 : 4;
    D2Shape best{SX * SY, 0, SX, SY, 1};
    const double nodes = (double)g.nx * g.ny;
    const bool square = g.ny >= 32 * SY && (g.nx + SX - 1) / SX * SX <= 1.2 * g.nx;
    if (far_arrays(g, fp64) || (fp64 ? nodes > 190e3 : nodes > 275e3 && 72e-6 * (double)g.qs < 268.0 && square)) return best;
    double least = -1.0;
    for (const auto &wg : shapes)
        for (int tx = 8; tx <= 64; tx += 8)
            for (int ty = 4; ty <= 32; ty += 4)
                for (int steps = 1; steps <= 3; ++steps) {
                    const D2Shape sh{wg[0], wg[1], tx, ty, steps};
                    if (!d2_fits(fp64, sh) || !d2_launcher(fp64, masked, sh)) continue;
                    double waves = 0.0, first = 0.0;
                    for (int r = 0; r < steps; ++r) {
                        first = (double)(tx + 4 + 6 * r) * (ty + 4 + 6 * r);
                        waves += ceil(first / 64.0);
                    }
                    const double rounds = ceil(ceil((double)g.nx / tx) * ceil((double)g.ny / ty) / cus);
                    if (rounds > 3 && wg[0] == 1024) continue;   // one workgroup per CU: nothing overlaps its barriers
                    const double compute = (fp64 ? 0.25 : 0.133) * waves;
                    // rows of whole cache lines, unless every CU has a tile of its own (2048^2
                    // FP32: 24 x 32 tiles 71 us a step, 32 x 24 ones 68)
                    const double lines = rounds > 1 && tx * size % 128 ? 1.5 : 1.0;
                    const double memory = lines * (first + tx * ty) * 9.0 * size / 21e3;
                    const double overlap = fp64 && wg[1] == 3 ? 0.79 : 0.72;   // 139 KB of LDS
                    const double us = (4.0 + overlap * rounds * (compute + memory)) / steps;
                    if (least < 0.0 || us < least) { least = us; best = sh; }
                }
    return best;
}

// A launch of one step has the tiles' halo to recompute and nothing to save by it: from 64,000 nodes on a
// thread per node is faster. us per step of one-step calls, tile of the plan | thread per node:
//   FP32  256^2 4.8 | 4.8   300^2 5.8 | 5.1   640^2 10.2 | 7.6   1000x900 23.5 | 18.9   2048^2 94 | 70
//   FP64  256^2 5.6 | 5.8   300^2 6.8 | 6.3   360^2 7.1 | 7.3    420^2 8.9 | 7.8
D2Shape d2_plan_one(const Geom &g, const D2Shape &plan) {
    return (double)g.nx * g.ny < 64e3 ? plan : D2Shape{SX * SY, 0, SX, SY, 1};
}

}  // namespace lbm
