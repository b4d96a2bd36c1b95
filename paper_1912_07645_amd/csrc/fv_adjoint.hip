// fv_adjoint.hip -- discrete adjoint of the finite-volume scheme: the transpose of the
// linearised Runge--Kutta stage (reconstruction -> Rusanov flux -> divergence) for the
// Euler equations, the kinetic-energy quantity of interest, and the contraction of the
// initial-state adjoint with the derivative of line-wise initial data.
//
// The reverse stage is in gather form. With L_i = -sum_k (F_{i+1/2} - F_{i-1/2}) / dx_k,
// sum_i lam_i . L_i = sum_faces F_f . w_f, w_f = (lam_right - lam_left) / dx. Every face
// therefore contributes (dF_f / dU_c)^T w_f to the four cells c of its stencil, through
// g_L = (dF/dU_L)^T w and g_R = (dF/dU_R)^T w and the reconstruction's partial derivatives.
// The faces of a tile store (g_L, g_R, minmod branch codes) in LDS, one axis at a time; each
// cell then adds that axis's four faces in a fixed order, with no atomics, so results are
// reproducible.
// Branches follow the forward pass: the larger Rusanov speed (ties to the right state), the
// minmod argument selected (ties as the forward comparison), sign(0) = 0 for |u|.
#include "fv_adjoint.h"
#include "fv_stage.h"

namespace fvk {

// (A^T w) for the Euler flux along nd at state U: A = dF/dU.
template <int DIM>
__device__ __forceinline__ void euler_flux_jt(const double* U, const EulerPrim<DIM>& pr, int nd,
                                              const double* w, const Phys& ph, double* out)
{
    constexpr int NF = DIM + 2;
    const double un = pick<DIM>(pr.u, nd);
    const double H = (U[NF - 1] + pr.p) * pr.ir;           // (E + p) / rho
    double usq = 0.0, S = 0.0;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        usq = usq + pr.u[k] * pr.u[k];
        S = S + w[1 + k] * pr.u[k];
    }
    const double p_rho = ph.gm1 * (0.5 * usq);
    const double p_E = ph.gm1;
    const double wn = pick<DIM>(w + 1, nd);
    const double wE = w[NF - 1];
    const double Wp = wn + wE * un;
    out[0] = -un * (S + wE * H) + Wp * p_rho;
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
        const double pm = -ph.gm1 * pr.u[j];
        double v = w[1 + j] * un + Wp * pm;
        if (j == nd) v = v + (w[0] + S + wE * H);
        out[1 + j] = v;
    }
    out[NF - 1] = wE * un + Wp * p_E;
}

// One side of a face, as speed_grad needs it.
template <int DIM>
struct SpeedSide {
    double rho, ir, c, u[DIM];
};

// Gradient of |u_n| + c with respect to U; TAME: the quotients of fv_fast.h.
template <int DIM, bool TAME>
__device__ __forceinline__ void speed_grad(const SpeedSide<DIM>& k, int nd, const Phys& ph, double* g)
{
    constexpr int NF = DIM + 2;
    const double un = pick<DIM>(k.u, nd);
    const double sg = (un > 0.0) ? 1.0 : ((un < 0.0) ? -1.0 : 0.0);
    double usq = 0.0;
#pragma unroll
    for (int j = 0; j < DIM; ++j) usq = usq + k.u[j] * k.u[j];
    const double d[2] = {2.0 * k.c * k.rho, 2.0 * k.rho};
    double a, cr;                                          // dc/dp, c / (2 rho)
    if constexpr (TAME) {
        double y[2];
        recips<2, true>(d, y);
        a = quotient(ph.gamma, d[0], y[0]);
        cr = quotient(k.c, d[1], y[1]);
    } else {
        a = ph.gamma / d[0];
        cr = k.c / d[1];
    }
    const double p_rho = ph.gm1 * (0.5 * usq);
    g[0] = sg * (-un * k.ir) + (a * p_rho - cr);
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
        double v = a * (-ph.gm1 * k.u[j]);
        if (j == nd) v = v + sg * k.ir;
        g[1 + j] = v;
    }
    g[NF - 1] = a * ph.gm1;
}

// Face terms from the two states and the jump of lambda (over dx): g_L, g_R, the side whose
// speed is the larger and its normal velocity. False where the windows of fv_fast.h do not hold.
template <int DIM, bool TAME>
__device__ __forceinline__ bool adjoint_face(const double* UL, const double* UR, const double* w,
                                             int nd, const Phys& ph, double* gL, double* gR,
                                             bool& selL, double& un)
{
    constexpr int NF = DIM + 2;
    EulerPrim<DIM> pl, pr;
    bool ok = true;
    if constexpr (TAME) {
        ok = euler_prims<DIM>(UL, UR, ph, pl, pr);
    } else {
        pl = euler_prim<DIM>(UL, ph);
        pr = euler_prim<DIM>(UR, ph);
    }
    const double sL = fabs(pick<DIM>(pl.u, nd)) + pl.c;
    const double sR = fabs(pick<DIM>(pr.u, nd)) + pr.c;
    selL = sL > sR;
    const double s = selL ? sL : sR;
    SpeedSide<DIM> k;   // the faster side
    k.rho = selL ? UL[0] : UR[0];
    k.ir = selL ? pl.ir : pr.ir;
    k.c = selL ? pl.c : pr.c;
#pragma unroll
    for (int j = 0; j < DIM; ++j) k.u[j] = selL ? pl.u[j] : pr.u[j];
    un = pick<DIM>(k.u, nd);
    double gs[NF];
    speed_grad<DIM, TAME>(k, nd, ph, gs);
    double wd = 0.0;
#pragma unroll
    for (int q = 0; q < NF; ++q) wd = wd + w[q] * (UR[q] - UL[q]);
    euler_flux_jt<DIM>(UL, pl, nd, w, ph, gL);
    euler_flux_jt<DIM>(UR, pr, nd, w, ph, gR);
#pragma unroll
    for (int q = 0; q < NF; ++q) {
        const double ds = 0.5 * wd * gs[q];
        gL[q] = 0.5 * (gL[q] + s * w[q]) - (selL ? ds : 0.0);
        gR[q] = 0.5 * (gR[q] - s * w[q]) - (selL ? 0.0 : ds);
    }
    return ok;
}

// minmod branch: 0 -> 0, 1 -> first argument, 2 -> second (as the forward comparisons).
__device__ __forceinline__ int minmod_code(double a, double b)
{
    if (a > 0.0 && b > 0.0) return (a < b) ? 1 : 2;
    if (a < 0.0 && b < 0.0) return (a > b) ? 1 : 2;
    return 0;
}

// SplitMix64's finaliser (Steele, Lea and Flood 2014): hashes the branch-signature terms.
__device__ __forceinline__ unsigned long long sig_mix(unsigned long long z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

template <int DIM, int RECON, int BX, int BY, int NT>
struct AdjTile {
    static constexpr int NF = DIM + 2;
    static constexpr int R = (RECON == REC_MUSCL) ? 1 : 0;  // extra faces per side
    static constexpr int HU = (RECON == REC_MUSCL) ? 3 : 1;  // halo of U
    static constexpr int HL = (RECON == REC_MUSCL) ? 2 : 1;  // halo of lambda
    static constexpr int UX = BX + 2 * HU, UY = (DIM >= 2) ? BY + 2 * HU : 1;
    static constexpr int LX = BX + 2 * HL, LY = (DIM >= 2) ? BY + 2 * HL : 1;
    // x faces: right-cell index k in [x0 - R, x0 + BX + R], all rows of the tile
    static constexpr int EXN = BX + 1 + 2 * R;
    static constexpr int NFX = EXN * BY;
    static constexpr int EYN = (DIM >= 2) ? BY + 1 + 2 * R : 0;
    static constexpr int NFY = (DIM >= 2) ? BX * EYN : 0;
    static constexpr int NFACES = NFX + NFY;
    static constexpr int CELLS = BX * BY;
};

// What bounds it is FP64 issue (about 1.2 faces' work of the forward stage, twice over) and, before,
// how few workgroups fitted a CU: tiles and face terms side by side took 41.7 KB, three
// workgroups. A tile has at most one x face and one y face per thread, so both faces' terms wait
// in registers until every thread has read the tiles, and then take the tiles' place, an axis at
// a time: 25.3 KB; its 106 registers leave four wavefronts per SIMD. With the short face
// arithmetic and uniform tile addresses, 16 samples of 256^2: 73.8 -> 61.5 us.
template <int DIM, int RECON, int BX, int BY, int NT>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 8)))
adjoint_stage_kernel(const AdjArgs a)
{
    using T = AdjTile<DIM, RECON, BX, BY, NT>;
    constexpr int NF = T::NF, R = T::R, HU = T::HU, HL = T::HL;
    constexpr int UX = T::UX, UY = T::UY, LX = T::LX, LY = T::LY;
    constexpr int NFX = T::NFX, EXN = T::EXN, NFY = T::NFY;
    constexpr int UC = UX * UY, LC = LX * LY;
    constexpr int HUY = (DIM >= 2) ? HU : 0, HLY = (DIM >= 2) ? HL : 0;
    constexpr int MAXF = NFX > NFY ? NFX : NFY;   // faces of one axis
    static_assert(MAXF <= NT && T::CELLS <= NT, "one face of an axis and one cell per thread");
    constexpr int TILES = NF * (UC + LC), TERMS = 2 * NF * MAXF;
    __shared__ double lds[TILES > TERMS ? TILES : TERMS];
    __shared__ int scode[MAXF];            // minmod codes, 2 bits per component and side
    __shared__ unsigned long long ssig;    // the workgroup's branch-signature sum
    __shared__ int wild[NT / 64];          // per wavefront: it loaded a cell that is not tame
    double* su = lds;
    double* sl = lds + NF * UC;
    double* sg = lds;                      // g_L, g_R per face of the axis in hand

    const uint32_t blk = xcd_remap(blockIdx.x, (uint32_t)a.nblocks);
    const int32_t sample = (int32_t)a.by_ntiles.quotient(blk);
    const int32_t tile = (int32_t)blk - sample * a.ntiles;
    const int32_t ty = (int32_t)a.by_t0.quotient((uint32_t)tile);
    const int32_t tx = tile - ty * a.tiles[0];
    const int32_t x0 = tx * BX, y0 = ty * BY;
    const int32_t nx = a.n[0], ny = a.n[1];
    const int64_t sbase = (int64_t)sample * NF * a.cells;
    const double* U = a.U + sbase;
    const double* lam = a.lam + sbase;

    // the haloed tiles of U and lambda into LDS, every load issued before the first store; a tile
    // away from the grid's edges at 32-bit offsets from one address per field
    const bool inner = x0 >= HU && x0 + BX + HU <= nx && (DIM < 2 || (y0 >= HU && y0 + BY + HU <= ny)) &&
                       (int64_t)UY * nx < (1 << 29);
    {
        constexpr int UPT = (UC + NT - 1) / NT, LPT = (LC + NT - 1) / NT;
        double vu[UPT][NF], vl[LPT][NF];
        if (inner) {
            const double* bu = U + ((int64_t)(y0 - HUY) * nx + (x0 - HU));
            const double* bl = lam + ((int64_t)(y0 - HLY) * nx + (x0 - HL));
#pragma unroll
            for (int k = 0; k < UPT; ++k) {
                const uint32_t e = threadIdx.x + k * NT;
                if ((k + 1) * NT <= UC || e < UC) {
                    const uint32_t off = (uint32_t)sizeof(double) * ((e / UX) * (uint32_t)nx + e % UX);
#pragma unroll
                    for (int q = 0; q < NF; ++q) vu[k][q] = *at_byte(bu + q * a.cells, off);
                }
            }
#pragma unroll
            for (int k = 0; k < LPT; ++k) {
                const uint32_t e = threadIdx.x + k * NT;
                if ((k + 1) * NT <= LC || e < LC) {
                    const uint32_t off = (uint32_t)sizeof(double) * ((e / LX) * (uint32_t)nx + e % LX);
#pragma unroll
                    for (int q = 0; q < NF; ++q) vl[k][q] = *at_byte(bl + q * a.cells, off);
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < UPT; ++k) {
                const int e = threadIdx.x + k * NT;
                if ((k + 1) * NT <= UC || e < UC) {
                    const int px = e % UX, py = e / UX;
                    const int32_t gx = wrap_index(x0 + px - HU, nx, a.bc[0]);
                    const int32_t gy = (DIM >= 2) ? wrap_index(y0 + py - HU, ny, a.bc[1]) : 0;
                    const int32_t gi = gy * nx + gx;   // cells < 2^31
#pragma unroll
                    for (int q = 0; q < NF; ++q) vu[k][q] = U[q * a.cells + gi];
                }
            }
#pragma unroll
            for (int k = 0; k < LPT; ++k) {
                const int e = threadIdx.x + k * NT;
                if ((k + 1) * NT <= LC || e < LC) {
                    const int px = e % LX, py = e / LX;
                    const int32_t gx = wrap_index(x0 + px - HL, nx, a.bc[0]);
                    const int32_t gy = (DIM >= 2) ? wrap_index(y0 + py - HL, ny, a.bc[1]) : 0;
                    const int32_t gi = gy * nx + gx;
#pragma unroll
                    for (int q = 0; q < NF; ++q) vl[k][q] = lam[q * a.cells + gi];
                }
            }
        }
        CellRange range;
#pragma unroll
        for (int k = 0; k < UPT; ++k) {
            const int e = threadIdx.x + k * NT;
            if ((k + 1) * NT <= UC || e < UC) {
#pragma unroll
                for (int q = 0; q < NF; ++q) {
                    range.add<true>(vu[k][q]);
                    su[q * UC + e] = vu[k][q];
                }
            }
        }
#pragma unroll
        for (int k = 0; k < LPT; ++k) {
            const int e = threadIdx.x + k * NT;
            if ((k + 1) * NT <= LC || e < LC) {
#pragma unroll
                for (int q = 0; q < NF; ++q) sl[q * LC + e] = vl[k][q];
            }
        }
        const bool any = any_lane(!range.tame());
        if ((threadIdx.x & 63) == 0) wild[threadIdx.x >> 6] = any;
        if (threadIdx.x == 0) ssig = 0ull;
    }
    __syncthreads();
    int anywild = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) anywild |= wild[i];
    const bool tame = __builtin_amdgcn_readfirstlane(anywild) == 0;

    // the thread's face of each axis: g_L, g_R and codes in registers
    const int f = threadIdx.x;
    double g[DIM][2][NF];
    int code[DIM];
    unsigned long long hsig = 0ull;   // this thread's signature terms (faces it owns)
#pragma unroll
    for (int nd = 0; nd < DIM; ++nd) {
        const int nfaces = (nd == 0) ? NFX : NFY;
        code[nd] = 0;
        if (f < nfaces) {
            int fx, fy;   // face between (right cell) and (right cell - e_nd), tile-local
            if (nd == 0) {
                fx = f % EXN - R;          // right-cell x offset from x0, in [-R, BX + R]
                fy = f / EXN;
            } else {
                fx = f % BX;
                fy = f / BX - R;
            }
            const int cu = ((DIM >= 2 ? fy + HU : 0)) * UX + (fx + HU);
            const int cl = ((DIM >= 2 ? fy + HL : 0)) * LX + (fx + HL);
            const double inv = (nd == 0) ? a.ph.inv_dx[0] : a.ph.inv_dx[1];
            constexpr int SX = 1;
            const int us = (nd == 0) ? SX : UX, ls = (nd == 0) ? SX : LX;
            double w[NF];
#pragma unroll
            for (int q = 0; q < NF; ++q) w[q] = inv * (sl[q * LC + cl] - sl[q * LC + cl - ls]);
            bool selL = false, done = false;
            double un = 0.0;
            if (tame) {
                double UL[NF], UR[NF];
                int codes = 0;
#pragma unroll
                for (int q = 0; q < NF; ++q) {
                    const double* sp = su + q * UC + cu;
                    const double ua = sp[-us], ub = sp[0];
                    if (RECON == REC_MUSCL) {
                        const double dl = ua - sp[-2 * us], dm = ub - ua, dr = sp[us] - ub;
                        codes |= (minmod_code(dl, dm) | (minmod_code(dm, dr) << 2)) << (4 * q);
                        UL[q] = __builtin_fma(0.5, minmod_finite(dl, dm), ua);
                        UR[q] = __builtin_fma(-0.5, minmod_finite(dm, dr), ub);
                    } else {
                        UL[q] = ua;
                        UR[q] = ub;
                    }
                }
                code[nd] = codes;
                done = !any_lane(!adjoint_face<DIM, true>(UL, UR, w, nd, a.ph, g[nd][0], g[nd][1], selL, un));
            }
            if (!done) {
                int c = cu;
                asm volatile("" : "+v"(c));   // read again: nothing is kept for this path
                double UL[NF], UR[NF];
                int codes = 0;
#pragma unroll
                for (int q = 0; q < NF; ++q) {
                    const double* sp = su + q * UC + c;
                    const double ua = sp[-us], ub = sp[0];
                    if (RECON == REC_MUSCL) {
                        const double dl = ua - sp[-2 * us], dm = ub - ua, dr = sp[us] - ub;
                        codes |= (minmod_code(dl, dm) | (minmod_code(dm, dr) << 2)) << (4 * q);
                        UL[q] = ua + (0.5 * minmod(dl, dm));
                        UR[q] = ub - (0.5 * minmod(dm, dr));
                    } else {
                        UL[q] = ua;
                        UR[q] = ub;
                    }
                }
                code[nd] = codes;
                adjoint_face<DIM, false>(UL, UR, w, nd, a.ph, g[nd][0], g[nd][1], selL, un);
            }
            if (a.sig) {
                // each face once: by the tile of its right cell, inside the grid
                const int32_t gx = x0 + fx, gy = (DIM >= 2) ? y0 + fy : 0;
                const bool own = (nd == 0) ? (fx >= 0 && fx < BX) : (fy >= 0 && fy < BY);
                if (own && gx < nx && gy < ny) {
                    const unsigned long long sgn = (un > 0.0) ? 2ull : ((un < 0.0) ? 0ull : 1ull);
                    const unsigned long long cd = (unsigned long long)(unsigned)code[nd] |
                                                  ((selL ? 1ull : 0ull) << 32) | (sgn << 33);
                    const unsigned long long key = ((unsigned long long)(gy * nx + gx) << 2) | nd;
                    hsig += sig_mix(a.salt ^ sig_mix(key * 0x9E3779B97F4A7C15ull + cd));
                }
            }
        }
    }

    // this thread's cell: its lambda, then the contributions of its faces, axis 0 before axis 1 as
    // in eq. 2.1, each axis's four (MUSCL) or two faces in a fixed order
    const int c = threadIdx.x;
    const int cx = c % BX, cy = c / BX;
    double lq[NF], jt[NF];
#pragma unroll
    for (int q = 0; q < NF; ++q) {
        lq[q] = (c < T::CELLS) ? sl[q * LC + (cy + HLY) * LX + (cx + HL)] : 0.0;
        jt[q] = 0.0;
    }
#pragma unroll
    for (int nd = 0; nd < DIM; ++nd) {
        __syncthreads();   // the tiles, or the axis before, are read
        const int nfaces = (nd == 0) ? NFX : NFY;
        if (f < nfaces) {
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                sg[(2 * q) * MAXF + f] = g[nd][0][q];
                sg[(2 * q + 1) * MAXF + f] = g[nd][1][q];
            }
            scode[f] = code[nd];
        }
        __syncthreads();
        if (c < T::CELLS) {
            // face index (within this axis) with right cell at tile offset o + shift along nd
            auto face = [&](int shift) -> int {
                if (nd == 0) return cy * EXN + (cx + shift + R);
                return (cy + shift + R) * BX + cx;
            };
            if constexpr (RECON == REC_MUSCL) {
                const int f0 = face(-1), f1 = face(0), f2 = face(1), f3 = face(2);
                const int c0 = scode[f0], c1 = scode[f1], c2 = scode[f2], c3 = scode[f3];
#pragma unroll
                for (int q = 0; q < NF; ++q) {
                    const int b = 4 * q;
                    const int r0 = (c0 >> (b + 2)) & 3, l1 = (c1 >> b) & 3, r1 = (c1 >> (b + 2)) & 3;
                    const int l2 = (c2 >> b) & 3, r2 = (c2 >> (b + 2)) & 3, l3 = (c3 >> b) & 3;
                    const double* gl = sg + (2 * q) * MAXF;
                    const double* gr = gl + MAXF;
                    double v = jt[q];
                    v = v + gr[f0] * ((r0 == 2) ? -0.5 : 0.0);   // face c - 3/2: this cell is b + 1
                    v = v + gl[f1] * ((l1 == 2) ? 0.5 : 0.0);    // face c - 1/2: this cell is b
                    v = v + gr[f1] * ((r1 == 1) ? 0.5 : ((r1 == 2) ? 1.5 : 1.0));
                    v = v + gl[f2] * ((l2 == 1) ? 1.5 : ((l2 == 2) ? 0.5 : 1.0));   // c + 1/2: a
                    v = v + gr[f2] * ((r2 == 1) ? 0.5 : 0.0);
                    v = v + gl[f3] * ((l3 == 1) ? -0.5 : 0.0);   // face c + 3/2: this cell is a - 1
                    jt[q] = v;
                }
            } else {
                const int f1 = face(0), f2 = face(1);
#pragma unroll
                for (int q = 0; q < NF; ++q) {
                    jt[q] = jt[q] + sg[(2 * q + 1) * MAXF + f1];   // face c - 1/2: g_R
                    jt[q] = jt[q] + sg[(2 * q) * MAXF + f2];       // face c + 1/2: g_L
                }
            }
        }
    }
    if (a.sig) {   // uniform over the launch
        atomicAdd(&ssig, hsig);
        __syncthreads();
        if (threadIdx.x == 0) atomicAdd(a.sig + sample, ssig);
    }

    // the reverse stage combination
    const int32_t gx = x0 + cx, gy = y0 + cy;
    if (c >= T::CELLS || gx >= nx || gy >= ny) return;
    double* prev = a.prev + sbase;
    double* acc = a.acc + sbase;
    const int32_t gi = gy * nx + gx;
#pragma unroll
    for (int q = 0; q < NF; ++q) {
        const double contrib = a.beta * (lq[q] + a.dt * jt[q]);
        const int64_t o = q * a.cells + gi;
        if (a.mode == 2) {
            prev[o] = acc[o] + contrib;
        } else {
            prev[o] = contrib;
            const double keep = (1.0 - a.beta) * lq[q];
            acc[o] = (a.mode == 0) ? keep : (acc[o] + keep);
        }
    }
}

template <int DIM, int RECON, int BX, int BY, int NT>
void launch_adjoint(const AdjArgs& a, hipStream_t s)
{
    hipLaunchKernelGGL((adjoint_stage_kernel<DIM, RECON, BX, BY, NT>), dim3((unsigned)a.nblocks),
                       dim3(NT), 0, s, a);
}

struct AdjEntry {
    int dim, recon;
    AdjKernel k;
};

static const AdjEntry kAdj[] = {
    {1, REC_FIRST, {&launch_adjoint<1, REC_FIRST, 255, 1, 256>, 255, 1, 1}},
    {1, REC_MUSCL, {&launch_adjoint<1, REC_MUSCL, 253, 1, 256>, 253, 1, 1}},
    {2, REC_FIRST, {&launch_adjoint<2, REC_FIRST, 16, 15, 256>, 16, 15, 1}},
    {2, REC_MUSCL, {&launch_adjoint<2, REC_MUSCL, 16, 13, 256>, 16, 13, 1}},
};

const AdjKernel* find_adjoint_kernel(int dim, int eq, int recon, int flux)
{
    if (eq != EQ_EULER || flux != FLUX_RUSANOV) return nullptr;
    for (const AdjEntry& e : kAdj)
        if (e.dim == dim && e.recon == recon) return &e.k;
    return nullptr;
}

// ------------------------------------------------------------------ quantity of interest

constexpr int kQoiCells = 4096;

int qoi_blocks(int64_t cells) { return (int)((cells + kQoiCells - 1) / kQoiCells); }

template <int DIM>
__global__ void __launch_bounds__(256)
qoi_ke_kernel(const double* __restrict__ state, int32_t nx, int32_t ny, int32_t nz, int32_t j0,
              int32_t j1, double volume, const double* __restrict__ seed, double* __restrict__ grad,
              double* __restrict__ partial, int32_t nblk)
{
    constexpr int NF = DIM + 2;
    __shared__ double red[256];
    const int64_t cells = (int64_t)nx * ny * nz;
    const int blk = blockIdx.x;
    const int32_t b = blockIdx.y;
    const double* U = state + (int64_t)b * NF * cells;
    const double g = seed ? seed[b] : 0.0;
    double acc = 0.0;
    const int64_t c0 = (int64_t)blk * kQoiCells;
    for (int64_t c = c0 + threadIdx.x; c < c0 + kQoiCells && c < cells; c += 256) {
        const int32_t j = (int32_t)((c / nx) % ny);
        const bool in = (j >= j0 && j < j1);
        double V[NF];
#pragma unroll
        for (int q = 0; q < NF; ++q) V[q] = U[q * cells + c];
        const double ir = 1.0 / V[0];
        double mm = V[1] * V[1];
#pragma unroll
        for (int k = 1; k < DIM; ++k) mm = mm + (V[1 + k] * V[1 + k]);
        if (in) acc = acc + (0.5 * (mm * ir));
        if (grad) {
            double* G = grad + (int64_t)b * NF * cells + c;
            const double s = in ? g * volume : 0.0;
            G[0] = s * (-0.5 * (mm * ir) * ir);
#pragma unroll
            for (int k = 0; k < DIM; ++k) G[(1 + k) * cells] = s * (V[1 + k] * ir);
            G[(NF - 1) * cells] = 0.0;
        }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] = red[threadIdx.x] + red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[(int64_t)b * nblk + blk] = red[0];
}

__global__ void qoi_finish_kernel(const double* __restrict__ partial, int32_t nblk, int32_t batch,
                                  double volume, double* __restrict__ Q)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= batch) return;
    double s = partial[(int64_t)b * nblk];
    for (int k = 1; k < nblk; ++k) s = s + partial[(int64_t)b * nblk + k];
    Q[b] = s * volume;
}

void launch_qoi_ke(const double* state, int32_t dim, const int32_t n[3], int32_t batch,
                   int32_t j0, int32_t j1, double volume, const double* seed, double* Q,
                   double* grad, double* partial, int32_t nblk, hipStream_t s)
{
    const dim3 grid((unsigned)nblk, (unsigned)batch);
    if (dim == 1)
        hipLaunchKernelGGL(qoi_ke_kernel<1>, grid, dim3(256), 0, s, state, n[0], n[1], n[2], j0, j1,
                           volume, seed, grad, partial, nblk);
    else if (dim == 2)
        hipLaunchKernelGGL(qoi_ke_kernel<2>, grid, dim3(256), 0, s, state, n[0], n[1], n[2], j0, j1,
                           volume, seed, grad, partial, nblk);
    else
        hipLaunchKernelGGL(qoi_ke_kernel<3>, grid, dim3(256), 0, s, state, n[0], n[1], n[2], j0, j1,
                           volume, seed, grad, partial, nblk);
    if (Q)
        hipLaunchKernelGGL(qoi_finish_kernel, dim3((batch + 63) / 64), dim3(64), 0, s, partial, nblk,
                           batch, volume, Q);
}

// ------------------------------------------------------------------ line contraction

// One thread per (sample, line): sum over the line's cells (y order) and the fields.
__global__ void line_sum_kernel(const double* __restrict__ lam, const double* __restrict__ D,
                                int32_t nf, int32_t nx, int32_t ny, int32_t nz, int32_t batch,
                                double* __restrict__ sums)
{
    const int64_t lines = (int64_t)nx * nz;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= lines * batch) return;
    const int64_t b = t / lines, line = t % lines;
    const int64_t i = line % nx, k = line / nx;
    const int64_t cells = (int64_t)nx * ny * nz;
    const double* L = lam + b * nf * cells;
    const double* Dm = D + b * nf * cells;
    double s = 0.0;
    for (int32_t j = 0; j < ny; ++j) {
        const int64_t c = (k * ny + j) * nx + i;
        for (int q = 0; q < nf; ++q) s = s + L[q * cells + c] * Dm[q * cells + c];
    }
    sums[t] = s;
}

// One thread per (sample, parameter): sum over lines in order.
__global__ void line_theta_kernel(const double* __restrict__ sums, const double* __restrict__ E,
                                  int64_t lines, int32_t ntheta, int32_t batch,
                                  double* __restrict__ out)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ntheta * batch) return;
    const int b = t / ntheta, k = t % ntheta;
    const double* S = sums + (int64_t)b * lines;
    const double* Eb = E + (int64_t)b * lines * ntheta;
    double acc = 0.0;
    for (int64_t l = 0; l < lines; ++l) acc = acc + S[l] * Eb[l * ntheta + k];
    out[t] = acc;
}

void launch_line_vjp(const double* lam, const double* D, const double* E, int32_t nf,
                     const int32_t n[3], int32_t batch, int32_t ntheta, double* line_sums,
                     double* out, hipStream_t s)
{
    const int64_t lines = (int64_t)n[0] * n[2];
    const int64_t t = lines * batch;
    hipLaunchKernelGGL(line_sum_kernel, dim3((unsigned)((t + 255) / 256)), dim3(256), 0, s, lam, D,
                       nf, n[0], n[1], n[2], batch, line_sums);
    const int t2 = ntheta * batch;
    hipLaunchKernelGGL(line_theta_kernel, dim3((t2 + 63) / 64), dim3(64), 0, s, line_sums, E, lines,
                       ntheta, batch, out);
}

}  // namespace fvk
