// fv_small.hip -- the whole time loop of a small 1D problem in one workgroup per sample.
//
// A 1D grid of up to a few thousand cells is latency-bound on the tiled path: each step is a
// handful of tiny launches (stages and the step decision) of a few microseconds each. Here one
// workgroup of up to 1024 threads (512 for the heaviest faces) keeps its sample's state on the
// chip and runs every step there: the step decision, the stages and the wave-speed reduction,
// until the sample stops or has taken `chunk` steps in this launch (the host launches again while
// samples run, so no launch runs unboundedly). The arithmetic of each face, update and speed
// is the tiled kernels' own (the same operations in the same order), and the decision repeats
// the control kernel's rules, so the results equal the tiled path's bit for bit.
//
// What bounds a step is the chain of its phases: the instructions of one CU's few wavefronts
// between barriers. Two kernels:
//   * small1d_kernel, any scheme: state with ghost layers and face fluxes in LDS, two barriers per
//     stage (fluxes complete; state complete, with the ghosts, which the owners of the mirrored
//     cells write, and with the wavefronts' wave speeds, kept twice so that none is overwritten
//     while it is read).
//   * small1d_cells_kernel, first-order Rusanov of the Euler and shallow-water equations: a face
//     combines what its two cells have by themselves (flux and signal speed), so a cell's
//     primitives are formed once per stage, where the faces and the wave speed formed them five
//     times; cells stay in registers, neighbours' terms come from the neighbouring lanes and, at
//     the ends of a wavefront, through LDS; one barrier per stage.
// Sod's tube on 1024 cells, forward Euler: 2.1 us per step, before (six barriers) 4.5.
#include "fv_small.h"
#include "fv_fast.h"
#include "fv_stage.h"

namespace fvk {

// Threads per workgroup: 1024, or 512 where a face needs more registers than 1024 threads
// leave (128 each): ideal MHD's eight fields and the Euler Godunov flux's Newton iteration.
template <int EQ, int FLUX>
constexpr int small_threads() { return (EQ == EQ_MHD || (EQ == EQ_EULER && FLUX == FLUX_GODUNOV)) ? 512 : 1024; }

// Cells per thread: 4 for a scalar equation, 2 for small systems (3 with 512 threads), 1 for
// MHD (LDS caps its grids below the thread count).
template <int EQ, int FLUX>
constexpr int small_cpt()
{
    constexpr int NF = NumFields<1, EQ>::value;
    return NF >= 5 ? 1 : (NF >= 2 ? (small_threads<EQ, FLUX>() == 512 ? 3 : 2) : 4);
}

// The step decision from the largest wave speed and whether a state is non-physical: every thread
// takes it alike from uniform values. False: the sample stops here.
struct SmallClock {
    double t, dt;
    int64_t steps;
    int32_t err;

    __device__ __forceinline__ bool decide(const SmallArgs& a, double M, bool bad)
    {
        if (bad) {
            err = ST_ENONPHYS;
            return false;
        }
        if (a.fixed) {
            if (steps >= a.max_steps) return false;
            if (a.fixed_dt * M > a.cfl_bound) {
                err = ST_ECFL;
                return false;
            }
            dt = a.fixed_dt;
        } else {
            if (!(t < a.t_end)) return false;
            if (steps >= a.max_steps) {
                if (a.limit_is_error) err = ST_EMAXSTEPS;
                return false;
            }
            dt = (M == 0.0) ? (a.t_end - t) : (a.cfl / M);
            bool last = false;
            if (t + dt >= a.t_end) {
                dt = a.t_end - t;
                last = true;
            }
            t = last ? a.t_end : (t + dt);
        }
        steps = steps + 1;
        return true;
    }
    __device__ __forceinline__ void store(const SmallArgs& a, int64_t b, bool running) const
    {
        if (!a.fixed) a.t[b] = t;
        a.steps[b] = steps;
        a.err[b] = err;
        a.running[b] = running ? 1 : 0;
        if (running) atomicAdd(a.n_running, 1);
    }
};

// The value of another lane (lanes that have none to read: 0).
template <int CTRL>
__device__ __forceinline__ double dpp(double x)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// Largest of a speed over the 16 lanes of a row, in each of them. (The instruction itself: a NaN
// here belongs to a bad state, whose speed is not used.)
__device__ __forceinline__ double speed_max(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double row_max(double v)
{
    constexpr int ROW_ROR = 0x120;
    v = speed_max(v, dpp<ROW_ROR + 8>(v));
    v = speed_max(v, dpp<ROW_ROR + 4>(v));
    v = speed_max(v, dpp<ROW_ROR + 2>(v));
    return speed_max(v, dpp<ROW_ROR + 1>(v));
}
__device__ __forceinline__ double lane_value(double x, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                            __builtin_amdgcn_readlane(__double2loint(x), l));
}

// Wave speeds of a workgroup's cells by rows of 16 lanes and physicality by wavefront: put before a
// barrier, got after it. Two sets by turns, so that one barrier between uses is enough.
struct SmallSpeeds {
    double m[2][64];
    int32_t bad[2][16];

    __device__ __forceinline__ void put(int set, double v, bool b)
    {
        v = row_max(v);
        const bool any = __ballot(b) != 0ull;
        if ((threadIdx.x & 15) == 0) m[set][threadIdx.x >> 4] = v;
        if ((threadIdx.x & 63) == 0) bad[set][threadIdx.x >> 6] = any;
    }
    __device__ __forceinline__ void get(int set, double& v, bool& b) const
    {
        const int l = threadIdx.x & 63, rows = blockDim.x >> 4;
        const double x = row_max(l < rows ? m[set][l] : 0.0);
        b = __ballot(l < rows / 4 && bad[set][l & 15]) != 0ull;
        v = speed_max(speed_max(lane_value(x, 0), lane_value(x, 16)),
                      speed_max(lane_value(x, 32), lane_value(x, 48)));
    }
};

template <int EQ, int RECON, int FLUX>
__global__ void __launch_bounds__((small_threads<EQ, FLUX>())) small1d_kernel(const SmallArgs a)
{
    constexpr int NF = NumFields<1, EQ>::value;
    constexpr int G = Ghost<RECON>::value;
    constexpr int CPT = small_cpt<EQ, FLUX>();
    extern __shared__ double lds[];
    const int n = a.n, nt = blockDim.x;
    const int PX = n + 2 * G;
    const int nf = a.bc == BC_PERIODIC ? n : n + 1;   // faces: the last is the first on a ring
    double* su = lds;                    // [NF][PX] state with ghost layers
    double* sf = lds + NF * PX;          // [NF][n + 1] face fluxes
    __shared__ SmallSpeeds speeds;

    const int64_t b = blockIdx.x;
    if (!a.first && !a.running[b]) return;   // uniform across the workgroup
    double* U = a.state + b * NF * (int64_t)n;
    const Phys& ph = a.ph;

    // a cell's new state, also to the ghosts that mirror it
    auto put_cell = [&](int c, const double (&v)[NF]) {
#pragma unroll
        for (int q = 0; q < NF; ++q) su[q * PX + G + c] = v[q];
        if (c < G || c >= n - G) {
#pragma unroll
            for (int j = 0; j < 2 * G; ++j) {
                const int i = (j < G) ? (j - G) : (n + j - G);     // -G..-1, n..n+G-1
                if (wrap_index(i, n, a.bc) == c) {
#pragma unroll
                    for (int q = 0; q < NF; ++q) su[q * PX + G + i] = v[q];
                }
            }
        }
    };

    double un[CPT][NF];   // U^n of the thread's cells
    int set = 0;
    double m = 0.0;
    bool bad = false;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
        const int c = threadIdx.x + k * nt;
        if (c < n) {
#pragma unroll
            for (int q = 0; q < NF; ++q) un[k][q] = U[q * n + c];
            put_cell(c, un[k]);
            bool bk;
            m = vmax(m, cell_speed<1, EQ>(un[k], ph, bk));
            bad = bad || bk;
        }
    }
    speeds.put(set, m, bad);
    __syncthreads();

    SmallClock clk{a.fixed ? 0.0 : a.t[b], 0.0, a.first ? 0 : a.steps[b], ST_OK};
    bool running = true;
    for (int64_t it = 0; it < a.chunk; ++it) {
        speeds.get(set, m, bad);
        running = clk.decide(a, m, bad);
        if (!running) break;
        set ^= 1;
        for (int st = 0; st < a.nst; ++st) {
            // faces f between cells f - 1 and f
            for (int f = threadIdx.x; f < nf; f += nt) {
                double UL[NF], UR[NF], F[NF];
#pragma unroll
                for (int q = 0; q < NF; ++q) {
                    const double* s = su + q * PX + G + f;
                    if (RECON == REC_FIRST) {
                        reconstruct<RECON>(0.0, s[-1], s[0], 0.0, UL[q], UR[q]);
                    } else {
                        reconstruct<RECON>(s[-2], s[-1], s[0], s[1], UL[q], UR[q]);
                    }
                }
                numflux<1, EQ, FLUX>(UL, UR, 0, F, ph);
#pragma unroll
                for (int q = 0; q < NF; ++q) sf[q * (n + 1) + f] = F[q];
            }
            __syncthreads();
            // divergence and stage combination of the thread's cells
            const double beta = a.beta[st];
            const bool use_un = st > 0, last = st + 1 == a.nst;
            m = 0.0;
            bad = false;
#pragma unroll
            for (int k = 0; k < CPT; ++k) {
                const int c = threadIdx.x + k * nt;
                if (c < n) {
                    const int fr = c + 1 < nf ? c + 1 : 0;
                    double out[NF];
#pragma unroll
                    for (int q = 0; q < NF; ++q) {
                        const double acc = (sf[q * (n + 1) + fr] - sf[q * (n + 1) + c]) * ph.inv_dx[0];
                        const double rhs = -acc;
                        const double up = su[q * PX + G + c];
                        const double u0 = use_un ? un[k][q] : up;
                        out[q] = u0 + (beta * ((up - u0) + (clk.dt * rhs)));
                    }
                    // in this phase a thread reads only its own cells' state, so the new value
                    // can replace it at once
                    put_cell(c, out);
                    if (last) {
#pragma unroll
                        for (int q = 0; q < NF; ++q) un[k][q] = out[q];
                        bool bk;
                        m = vmax(m, cell_speed<1, EQ>(out, ph, bk));
                        bad = bad || bk;
                    }
                }
            }
            if (last) speeds.put(set, m, bad);
            __syncthreads();
        }
    }

#pragma unroll
    for (int k = 0; k < CPT; ++k) {
        const int c = threadIdx.x + k * nt;
        if (c < n) {
#pragma unroll
            for (int q = 0; q < NF; ++q) U[q * n + c] = un[k][q];
        }
    }
    if (threadIdx.x == 0) clk.store(a, b, running);
}

// ---------------------------------------------------------------- first order, Rusanov

// Whether a face's flux is a combination of terms of its two cells (SmallCell).
template <int EQ, int RECON, int FLUX>
constexpr bool small_cellwise()
{
    return RECON == REC_FIRST && FLUX == FLUX_RUSANOV && (EQ == EQ_EULER || EQ == EQ_SWE);
}

// A cell's state, physical flux and signal speed |u| + c. F[0] is U[1].
template <int EQ>
struct SmallCell {
    static constexpr int NF = NumFields<1, EQ>::value;
    static constexpr int NV = 2 * NF;
    double v[NV];   // U, then F[1..], then the speed

    __device__ __forceinline__ double U(int q) const { return v[q]; }
    __device__ __forceinline__ double F(int q) const { return q == 0 ? v[1] : v[NF + q - 1]; }
    __device__ __forceinline__ double speed() const { return v[NV - 1]; }

    template <class Prim>
    __device__ __forceinline__ void set(const double (&u)[NF], const Prim& w, const Phys& ph)
    {
        double F[NF];
        if constexpr (EQ == EQ_EULER) euler_flux<1>(u, w, 0, F);
        else swe_flux<1>(u, w, 0, F, ph);
#pragma unroll
        for (int q = 0; q < NF; ++q) v[q] = u[q];
#pragma unroll
        for (int q = 1; q < NF; ++q) v[NF + q - 1] = F[q];
        v[NV - 1] = fabs(w.u[0]) + w.c;
    }

    // The terms of state U with the short reciprocal and root: false where they do not hold. Where
    // they do the state is physical: what is positive and finite implies it for every field.
    __device__ __forceinline__ bool form(const double (&u)[NF], const Phys& ph)
    {
        HighRange r;
        r.add(u[0]);
        double x;
        if constexpr (EQ == EQ_EULER) {
            EulerPrim<1> w;
            w.ir = inverse(u[0]);
            w.u[0] = u[1] * w.ir;
            double ke = u[1] * w.u[0];
            ke = 0.5 * ke;
            w.p = ph.gm1 * (u[2] - ke);
            x = (ph.gamma * w.p) * w.ir;
            w.c = root(x);
            r.add(x);
            set(u, w, ph);
            return r.within<-100, 100>();
        } else {
            SwePrim<1> w;
            w.ih = inverse(u[0]);
            w.u[0] = u[1] * w.ih;
            x = ph.grav * u[0];
            w.c = root(x);
            r.add(x);
            set(u, w, ph);
            return r.within<-100, 100>() && isfinite(u[1]);
        }
    }

    // The same in general; whether the state is physical.
    __device__ __forceinline__ bool form_any(const double (&u)[NF], const Phys& ph)
    {
        bool ok = u[0] > 0.0;
#pragma unroll
        for (int q = 0; q < NF; ++q) ok = ok && isfinite(u[q]);
        if constexpr (EQ == EQ_EULER) {
            const EulerPrim<1> w = euler_prim<1>(u, ph);
            ok = ok && w.p > 0.0;
            set(u, w, ph);
        } else {
            set(u, swe_prim<1>(u, ph), ph);
        }
        return ok;
    }
};

// The Rusanov flux between two cells.
template <int EQ>
__device__ __forceinline__ void small_face(const SmallCell<EQ>& l, const SmallCell<EQ>& r, double* F)
{
    const double s = vmax(l.speed(), r.speed());
#pragma unroll
    for (int q = 0; q < SmallCell<EQ>::NF; ++q)
        F[q] = 0.5 * ((l.F(q) + r.F(q)) - (s * (r.U(q) - l.U(q))));
}

// CPT cells per thread, c = tid + k nt: a wavefront's k-th 64 of them are cells 64 slot .. 64 slot
// + 63. Threads past the last cell carry a copy of it along, which nothing reads.
constexpr int kCellThreads = 1024, kCellSlots = 32;

template <int EQ, int CPT>
__global__ void __launch_bounds__(kCellThreads) small1d_cells_kernel(const SmallArgs a)
{
    using Cell = SmallCell<EQ>;
    constexpr int NF = Cell::NF, NV = Cell::NV;
    constexpr int FROM_LEFT = 0x138, FROM_RIGHT = 0x130;   // wave_shr:1, wave_shl:1
    // first and last cell of every 64, of two stages by turns
    __shared__ double ends[2][kCellSlots][2][NV];
    __shared__ SmallSpeeds speeds;
    const int n = a.n, nw = blockDim.x >> 6;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    const int64_t b = blockIdx.x;
    if (!a.first && !a.running[b]) return;   // uniform across the workgroup
    double* U = a.state + b * NF * (int64_t)n;
    const Phys& ph = a.ph;
    const bool ring = a.bc == BC_PERIODIC;

    int set = 0;
    double m = 0.0;
    bool bad = false;
    Cell cell[CPT];
    auto publish = [&](const double (&u)[CPT][NF]) {
        bool tame = true;
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            const int c = (wave + k * nw) * 64 + lane;
            const bool ok = cell[k].form(u[k], ph);
            tame = tame && (ok || c >= n);
        }
        m = 0.0;
        bad = false;
        if (any_lane(!tame)) {
#pragma unroll
            for (int k = 0; k < CPT; ++k) {
                const int c = (wave + k * nw) * 64 + lane;
                const bool ok = cell[k].form_any(u[k], ph);
                bad = bad || (!ok && c < n);
            }
        }
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            const int slot = wave + k * nw, c = slot * 64 + lane;
            if (lane == 0) {
#pragma unroll
                for (int i = 0; i < NV; ++i) ends[set][slot][0][i] = cell[k].v[i];
            }
            if (c == n - 1 || (lane == 63 && c < n)) {
#pragma unroll
                for (int i = 0; i < NV; ++i) ends[set][slot][1][i] = cell[k].v[i];
            }
            const double s = cell[k].speed() * ph.inv_dx[0];
            m = c < n ? vmax(m, s) : m;
        }
    };
    {
        double u[CPT][NF];
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            const int c = (wave + k * nw) * 64 + lane, i = c < n ? c : n - 1;
#pragma unroll
            for (int q = 0; q < NF; ++q) u[k][q] = U[q * n + i];
        }
        publish(u);
    }
    speeds.put(set, m, bad);
    __syncthreads();

    SmallClock clk{a.fixed ? 0.0 : a.t[b], 0.0, a.first ? 0 : a.steps[b], ST_OK};
    bool running = true;
    for (int64_t it = 0; it < a.chunk; ++it) {
        speeds.get(set, m, bad);
        running = clk.decide(a, m, bad);
        if (!running) break;
        double un[CPT][NF];   // U^n
#pragma unroll
        for (int k = 0; k < CPT; ++k)
#pragma unroll
            for (int q = 0; q < NF; ++q) un[k][q] = cell[k].U(q);
#pragma unroll 1
        for (int st = 0; st < a.nst; ++st) {
            const double beta = a.beta[st];
            double out[CPT][NF];
#pragma unroll
            for (int k = 0; k < CPT; ++k) {
                const int slot = wave + k * nw, c = slot * 64 + lane;
                const Cell& me = cell[k];
                Cell l, r;
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    l.v[i] = dpp<FROM_LEFT>(me.v[i]);
                    r.v[i] = dpp<FROM_RIGHT>(me.v[i]);
                }
                if (lane == 0) {
                    if (c > 0 || ring) {
                        const int s = c > 0 ? slot - 1 : (n - 1) >> 6;
#pragma unroll
                        for (int i = 0; i < NV; ++i) l.v[i] = ends[set][s][1][i];
                    } else l = me;
                }
                if (lane == 63 || c == n - 1) {
                    if (c < n - 1 || (c == n - 1 && ring)) {
                        const int s = c < n - 1 ? slot + 1 : 0;
#pragma unroll
                        for (int i = 0; i < NV; ++i) r.v[i] = ends[set][s][0][i];
                    } else r = me;
                }
                double FL[NF], FR[NF];
                small_face(l, me, FL);
                small_face(me, r, FR);
#pragma unroll
                for (int q = 0; q < NF; ++q) {
                    const double acc = (FR[q] - FL[q]) * ph.inv_dx[0];
                    const double rhs = -acc;
                    const double up = me.U(q), u0 = un[k][q];
                    out[k][q] = u0 + (beta * ((up - u0) + (clk.dt * rhs)));
                }
            }
            set ^= 1;
            publish(out);
            if (st + 1 == a.nst) speeds.put(set, m, bad);
            __syncthreads();
        }
    }

#pragma unroll
    for (int k = 0; k < CPT; ++k) {
        const int c = (wave + k * nw) * 64 + lane;
        if (c < n) {
#pragma unroll
            for (int q = 0; q < NF; ++q) U[q * n + c] = cell[k].U(q);
        }
    }
    if (threadIdx.x == 0) clk.store(a, b, running);
}

template <int EQ, int RECON, int FLUX>
static void launch_small(const SmallArgs& a, hipStream_t s)
{
    constexpr int NF = NumFields<1, EQ>::value;
    constexpr int G = Ghost<RECON>::value;
    const dim3 grid((unsigned)a.batch);
    // no more wavefronts than the cells fill: a barrier waits for each
    if constexpr (small_cellwise<EQ, RECON, FLUX>()) {
        // one cell per thread (two with half the threads, though a step's reduction and decision
        // cost a wavefront the same for one or two: 550 against 509 us for Sod's 200 steps)
        const int cpt = a.n <= kCellThreads ? 1 : 2;
        const dim3 block((unsigned)((a.n + 64 * cpt - 1) / (64 * cpt) * 64));
        if (cpt == 1) hipLaunchKernelGGL((small1d_cells_kernel<EQ, 1>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((small1d_cells_kernel<EQ, 2>), grid, block, 0, s, a);
    } else {
        const int need = (a.n + 1 + 63) / 64 * 64, most = small_threads<EQ, FLUX>();   // and the last face
        const size_t lds = sizeof(double) * (size_t)NF * ((a.n + 2 * G) + (a.n + 1));
        hipLaunchKernelGGL((small1d_kernel<EQ, RECON, FLUX>), grid, dim3((unsigned)(need < most ? need : most)),
                           lds, s, a);
    }
}

template <int EQ, int RECON, int FLUX>
constexpr SmallKernel make_small()
{
    constexpr int NF = NumFields<1, EQ>::value;
    constexpr int G = Ghost<RECON>::value;
    // LDS of the state with ghosts and the faces within 60 KiB, and the cells per thread
    static_assert(!small_cellwise<EQ, RECON, FLUX>() || NF >= 2, "at most 64 kCellSlots cells");
    constexpr int by_lds = (60 * 1024 / (8 * NF) - 2 * G - 1) / 2;
    constexpr int cap = small_threads<EQ, FLUX>() * small_cpt<EQ, FLUX>();
    return SmallKernel{EQ, RECON, FLUX, &launch_small<EQ, RECON, FLUX>, by_lds < cap ? by_lds : cap};
}

#define SMALL4(E, F) make_small<E, REC_FIRST, F>(), make_small<E, REC_MUSCL, F>(), \
                     make_small<E, REC_WENO3, F>(), make_small<E, REC_ENO2, F>()
static const SmallKernel kSmall[] = {
    SMALL4(EQ_EULER, FLUX_RUSANOV), SMALL4(EQ_EULER, FLUX_HLL), SMALL4(EQ_EULER, FLUX_HLLC),
    SMALL4(EQ_EULER, FLUX_ROE), SMALL4(EQ_EULER, FLUX_GODUNOV), SMALL4(EQ_EULER, FLUX_EC),
    SMALL4(EQ_BURGERS, FLUX_RUSANOV), SMALL4(EQ_BURGERS, FLUX_HLL), SMALL4(EQ_BURGERS, FLUX_ROE),
    SMALL4(EQ_BURGERS, FLUX_GODUNOV), SMALL4(EQ_BURGERS, FLUX_EC),
    SMALL4(EQ_ADVECTION, FLUX_RUSANOV), SMALL4(EQ_ADVECTION, FLUX_HLL), SMALL4(EQ_ADVECTION, FLUX_ROE),
    SMALL4(EQ_ADVECTION, FLUX_GODUNOV),
    SMALL4(EQ_SWE, FLUX_RUSANOV), SMALL4(EQ_SWE, FLUX_HLL), SMALL4(EQ_SWE, FLUX_ROE),
    SMALL4(EQ_MHD, FLUX_RUSANOV), SMALL4(EQ_MHD, FLUX_HLL),
};
#undef SMALL4

const SmallKernel* find_small_kernel(int eq, int recon, int flux)
{
    for (const SmallKernel& k : kSmall)
        if (k.eq == eq && k.recon == recon && k.flux == flux) return &k;
    return nullptr;
}

}  // namespace fvk
