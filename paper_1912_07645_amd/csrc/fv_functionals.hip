// fv_functionals.hip -- point PDFs, joint PDFs and shell structure functions of a batch of
// samples: the statistics that Section 2.2 lists after Fjordholm, Lye and Mishra, beside the
// mean, variance and axis structure functions of fv_stats.hip.
//
// Quantities are those of the statistics: Euler (rho, u_1..u_dim, E) with u_k = m_k * (1/rho),
// shallow water (h, u_1..u_dim) with u_k = hu_k * (1/h), scalar equations the field itself.
//
// PDFs. One thread per (sample, point or pair) finds the bin of the quantity's value in FP64:
// t = ((v - lo) / (hi - lo)) * nbins, bin floor(t), the last bin also taking a value that
// rounds onto its upper edge; values below lo and values not below hi (NaN included) have a
// counter each (point PDFs), and pairs with either value outside its range share one
// (joint PDFs). Counts are added with 64-bit atomics, so they are exact in any order.
//
// Shell structure functions. S_p(h) = 1/(N |A_h|) sum_{o in A_h} sum_x |q(x + o) - q(x)|^p on
// the periodic grid, p in {1, 2}, over the cube shell A_h = {o : max_k |o_k| = h} or the ball
// shell {o : (h - 1)^2 < |o|^2 <= h^2}. One workgroup takes one tile of one quantity of one
// sample: the quantity over the tile and a periodic halo of max_h cells on every active axis
// goes into LDS, then every thread walks the shells h = 1..max_h of its cells (all threads take
// the same offsets, so the shell tests are uniform; one offset of every pair o, -o, whose sums
// over the periodic grid are equal) and the workgroup sums its cells per h
// (wavefront shuffles, then the wavefronts in order). A second pass adds the tiles in order
// and divides. Sums run in another order than the definition's, so results agree with it to
// rounding (relative 1e-12 and better in the tests), not bit for bit.
#include <algorithm>
#include <vector>

#include "fv_host.h"
#include "fv_stage.h"

namespace fvk {

constexpr int kFnThreads = 256;
constexpr int kShellMaxH = 64;
constexpr int kShellTile2 = 64;    // side of the register-tiled 2D shell kernel's tile
constexpr int kShellBlocks2 = 16;  // blocks of 16 x 16 cells in it
constexpr int kShellMaxH2 = 16;    // and its largest radius (61 KB of LDS; beyond, one cell per thread)

// kind: 0 the field itself; 1 Euler (momenta over rho); 2 shallow water (momenta over h);
// 3 ideal MHD (the three momenta over rho).
__device__ __forceinline__ bool quantity_divides(int kind, int nf, int qi)
{
    return !(kind == 0 || qi == 0 || (kind == 1 && qi == nf - 1) || (kind == 3 && qi > 3));
}

__device__ __forceinline__ double quantity_at(const double* U, int64_t cells, int nf, int kind,
                                              int64_t c, int qi)
{
    if (!quantity_divides(kind, nf, qi)) return U[(int64_t)qi * cells + c];
    const double ir = 1.0 / U[c];
    return U[(int64_t)qi * cells + c] * ir;
}

// Bin 0..nbins-1; -1 below lo; nbins not below hi (NaN included).
__device__ __forceinline__ int bin_of(double v, double lo, double hi, int nbins)
{
    if (v < lo) return -1;
    if (!(v < hi)) return nbins;
    const int64_t k = (int64_t)floor(((v - lo) / (hi - lo)) * (double)nbins);
    return k < nbins ? (int)k : nbins - 1;
}

struct PdfArgs {
    const double* state;         // [batch][nf][cells]
    int64_t cells;
    int32_t nf, kind;
    int64_t batch, n;            // samples; points (or pairs)
    const int64_t* cell;         // [n] points, or [n][2] pairs
    int32_t qa, qb, nbins, joint;
    double lo_a, hi_a, lo_b, hi_b;
    unsigned long long* counts;  // [n][nbins + 2] or [n][nbins * nbins + 1]
};

__global__ void __launch_bounds__(kFnThreads) pdf_kernel(const PdfArgs a)
{
    const int64_t t = (int64_t)blockIdx.x * kFnThreads + threadIdx.x;
    if (t >= a.batch * a.n) return;
    const int64_t b = t / a.n, i = t % a.n;
    const double* U = a.state + b * a.nf * a.cells;
    if (!a.joint) {
        const int k = bin_of(quantity_at(U, a.cells, a.nf, a.kind, a.cell[i], a.qa), a.lo_a, a.hi_a, a.nbins);
        const int slot = (k < 0) ? a.nbins : (k >= a.nbins ? a.nbins + 1 : k);
        atomicAdd(&a.counts[i * (a.nbins + 2) + slot], 1ull);
    } else {
        const int ka = bin_of(quantity_at(U, a.cells, a.nf, a.kind, a.cell[2 * i], a.qa), a.lo_a, a.hi_a, a.nbins);
        const int kb = bin_of(quantity_at(U, a.cells, a.nf, a.kind, a.cell[2 * i + 1], a.qb), a.lo_b, a.hi_b, a.nbins);
        const int64_t per = (int64_t)a.nbins * a.nbins + 1;
        const bool in = ka >= 0 && ka < a.nbins && kb >= 0 && kb < a.nbins;
        atomicAdd(&a.counts[i * per + (in ? (int64_t)ka * a.nbins + kb : per - 1)], 1ull);
    }
}

// Tile of the shell kernel: 256 cells.
template <int DIM>
struct ShellTile {
    static constexpr int TX = (DIM == 1) ? 256 : (DIM == 2 ? 16 : 8);
    static constexpr int TY = (DIM == 1) ? 1 : (DIM == 2 ? 16 : 8);
    static constexpr int TZ = (DIM == 3) ? 4 : 1;
};

struct ShellArgs {
    const double* state;   // first sample of the chunk: [samples][nf][cells]
    int64_t cells;
    int32_t n[3];
    int32_t tiles[3];
    int32_t ntiles;
    int32_t nf, kind, nq, H, ball;
    double* partial;       // [sample][q][H][ntiles]
};

__device__ __forceinline__ int32_t wrap_mod(int32_t i, int32_t n)
{
    i %= n;
    return i < 0 ? i + n : i;
}

__device__ __forceinline__ bool in_ball_shell(int ox, int oy, int oz, int h)
{
    const int r2 = ox * ox + oy * oy + oz * oz;
    return (h - 1) * (h - 1) < r2 && r2 <= h * h;
}

// acc + |d|^P
template <int P>
__device__ __forceinline__ double shell_add(double acc, double d)
{
    return (P == 1) ? acc + fabs(d) : __builtin_fma(d, d, acc);
}

// Sums over half a shell. On the periodic grid sum_x |q(x + o) - q(x)|^p is the same for o and -o,
// so of every such pair one offset is taken (the first nonzero of oz, oy, ox positive), and the
// sum over the shell is twice that over its half: half the terms.

// One cell per thread (1D, 3D, and 2D where the kernels below do not apply).
template <int DIM, int P>
__global__ void __launch_bounds__(kFnThreads) shell_kernel(const ShellArgs a)
{
    using T = ShellTile<DIM>;
    constexpr int TX = T::TX, TY = T::TY, TZ = T::TZ;
    extern __shared__ double lds[];
    const int H = a.H;
    const int HY = (DIM >= 2) ? H : 0, HZ = (DIM >= 3) ? H : 0;
    const int PX = TX + 2 * H, PY = TY + 2 * HY, PZ = TZ + 2 * HZ;
    double* lq = lds;                       // quantity over tile + halo
    double* wsum = lds + PX * PY * PZ;      // [waves][H]

    const int64_t blk = blockIdx.x;
    const int32_t tile = (int32_t)(blk % a.ntiles);
    const int64_t sq = blk / a.ntiles;      // sample * nq + quantity
    const int qi = (int)(sq % a.nq);
    const int64_t b = sq / a.nq;
    const int32_t x0 = (tile % a.tiles[0]) * TX;
    const int32_t y0 = ((tile / a.tiles[0]) % a.tiles[1]) * TY;
    const int32_t z0 = (tile / (a.tiles[0] * a.tiles[1])) * TZ;
    const double* U = a.state + b * a.nf * a.cells;

    for (int e = threadIdx.x; e < PX * PY * PZ; e += kFnThreads) {
        const int px = e % PX, py = (e / PX) % PY, pz = e / (PX * PY);
        const int32_t gx = wrap_mod(x0 + px - H, a.n[0]);
        const int32_t gy = (DIM >= 2) ? wrap_mod(y0 + py - HY, a.n[1]) : 0;
        const int32_t gz = (DIM >= 3) ? wrap_mod(z0 + pz - HZ, a.n[2]) : 0;
        lq[e] = quantity_at(U, a.cells, a.nf, a.kind, ((int64_t)gz * a.n[1] + gy) * a.n[0] + gx, qi);
    }
    __syncthreads();

    const int cx = threadIdx.x % TX, cy = (threadIdx.x / TX) % TY, cz = threadIdx.x / (TX * TY);
    const bool inside = x0 + cx < a.n[0] && y0 + cy < a.n[1] && z0 + cz < a.n[2];
    const int lc = ((cz + HZ) * PY + (cy + HY)) * PX + (cx + H);
    const double q0 = lq[lc];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int h = 1; h <= H; ++h) {
        const int hy = (DIM >= 2) ? h : 0, hz = (DIM >= 3) ? h : 0;
        double acc = 0.0;
        for (int oz = 0; oz <= hz; ++oz)
            for (int oy = (oz == 0) ? 0 : -hy; oy <= hy; ++oy) {
                const double* row = lq + lc + (oz * PY + oy) * PX;
                const bool own = oz == 0 && oy == 0;   // the cell's own row: to the right only
                if (a.ball) {
                    for (int ox = own ? 1 : -h; ox <= h; ++ox)
                        if (in_ball_shell(ox, oy, oz, h)) acc = shell_add<P>(acc, row[ox] - q0);
                } else if ((DIM >= 2 && (oy == -h || oy == h)) || (DIM >= 3 && oz == h)) {
                    // a row on a face of the cube (only active axes have faces)
                    for (int ox = -h; ox <= h; ++ox) acc = shell_add<P>(acc, row[ox] - q0);
                } else {
                    // an inner row of the cube: only its two ends are on the shell
                    if (!own) acc = shell_add<P>(acc, row[-h] - q0);
                    acc = shell_add<P>(acc, row[h] - q0);
                }
            }
        acc = inside ? acc : 0.0;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) acc = acc + __shfl_xor(acc, off, 64);
        if (lane == 0) wsum[wave * H + (h - 1)] = acc;
    }
    __syncthreads();
    for (int h = threadIdx.x; h < H; h += kFnThreads) {
        double s = wsum[h];
        for (int w = 1; w < kFnThreads / 64; ++w) s = s + wsum[w * H + h];
        a.partial[(sq * H + h) * a.ntiles + tile] = s;
    }
}

// The offsets of half a 2D shell in the order that both 2D kernels below take them for a cell:
// row(oy, lo, hi) takes (lo, oy) .. (hi, oy), column(ox, hi) takes (ox, 1) .. (ox, hi).
template <bool BALL, class Row, class Column>
__device__ __forceinline__ void shell2d_half(int h, const Row& row, const Column& column)
{
    if constexpr (BALL) {
        // (h - 1)^2 < ox^2 + oy^2 <= h^2: of row oy the columns lo..hi and -hi..-lo
        int hi = h, lo = h;
#pragma unroll 1
        for (int oy = 0; oy <= h; ++oy) {
            while (hi * hi > h * h - oy * oy) --hi;
            const int inner = (h - 1) * (h - 1) - oy * oy;
            if (inner < 0) {
                row(oy, -hi, hi);
            } else {
                while (lo > 1 && (lo - 1) * (lo - 1) > inner) --lo;
                if (lo <= hi) {
                    row(oy, lo, hi);
                    if (oy > 0) row(oy, -hi, -lo);
                }
            }
        }
    } else {
        row(h, -h, h);
        column(h, h - 1);
        column(-h, h - 1);
        row(0, h, h);
    }
}

// The sum over a 64 x 64 tile, in the order that both 2D kernels take: 4 x 4 cells pairwise, by
// columns, then rows; four such squares along x pairwise, then four along y (a block of 16 x 16);
// four blocks along x pairwise; the four rows of blocks in order. Cells and blocks outside the
// grid add +0 to sums of terms >= +0. The tiles are added in order by the second pass.
__device__ __forceinline__ double pairwise4(double a, double b, double c, double d)
{
    return (a + b) + (c + d);
}

// 2D, radii up to HM: 64 x 64 cells to a workgroup, 4 x 4 to a thread. What bounded one cell per
// thread was LDS, a read for every term. Here a thread slides a window of four values along a row
// of offsets (or, for the cube's two side columns, along a column): one read serves the terms of
// four cells, 0.3 reads per term for a cube of radius 8, and the FP64 pipe (a subtraction and a
// fused multiply-add per term) is the bound. Rows are stored by column modulo 4, so that the
// lanes of a row, four columns apart, read neighbouring slots. The halo is 16 rows less (offsets
// point up), and 1.4 cells are staged per cell instead of 4. 64 samples of 256^2, cube shells to
// radius 8: 1030 -> 282 us
// (18 T operations/s; the FP64 pipe sustains about 30 under its power limit).
template <int P, bool BALL, int HM>
__global__ void __launch_bounds__(kFnThreads) __attribute__((amdgpu_waves_per_eu(3, 8)))
shell2d_kernel(const ShellArgs a)
{
    constexpr int T = kShellTile2, PX = T + 2 * HM, Q = PX / 4;
    static_assert(HM % 4 == 0 && T == 64 && kFnThreads == 256, "4 x 4 cells per thread");
    extern __shared__ double lds[];
    const int H = a.H, rows = T + H;
    double* wsum = lds + rows * PX;         // [waves][H]

    const int64_t blk = blockIdx.x;
    const int32_t tile = (int32_t)(blk % a.ntiles);
    const int64_t sq = blk / a.ntiles;      // sample * nq + quantity
    const int qi = (int)(sq % a.nq);
    const double* U = a.state + (sq / a.nq) * a.nf * a.cells;
    const int32_t x0 = (tile % a.tiles[0]) * T, y0 = (tile / a.tiles[0]) * T;

    // the quantity over the tile and its halo: eight values at a time are requested before the
    // first is used
    const bool divide = quantity_divides(a.kind, a.nf, qi);   // uniform
    const double* F = U + (int64_t)qi * a.cells;
    constexpr int D = 8;
    for (int e0 = threadIdx.x; e0 < rows * PX; e0 += D * kFnThreads) {
        double v[D], d[D];
#pragma unroll
        for (int i = 0; i < D; ++i) {
            const int e = e0 + i * kFnThreads;
            const int px = e % PX, py = e / PX;
            const int32_t gx = wrap_index(x0 + px - HM, a.n[0], BC_PERIODIC);
            const int32_t gy = wrap_index(y0 + py, a.n[1], BC_PERIODIC);
            const int32_t c = gy * a.n[0] + gx;   // cells < 2^31
            v[i] = F[c];
            d[i] = divide ? U[c] : 1.0;
        }
#pragma unroll
        for (int i = 0; i < D; ++i) {
            const int e = e0 + i * kFnThreads;
            const int px = e % PX, py = e / PX;
            if (e < rows * PX)
                lds[py * PX + (px & 3) * Q + (px >> 2)] = divide ? v[i] * (1.0 / d[i]) : v[i];
        }
    }
    __syncthreads();

    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const double* own = lds + 4 * ty * PX + tx;
    // slot of the value `col` columns right of the thread's first cell
    auto slot = [&](int col) {
        const int k = HM + col;
        return (k & 3) * Q + (k >> 2);
    };
    double q[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) q[r][j] = own[r * PX + slot(j)];
    bool in_x[4], in_y[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        in_x[i] = x0 + 4 * tx + i < a.n[0];
        in_y[i] = y0 + 4 * ty + i < a.n[1];
    }
    double acc[4][4];
    // the offsets (ox, oy), ox = lo..hi, of every cell: a window w[row] of four columns that
    // slides to the right, all four rows at a time
    auto along_row = [&](int oy, int lo, int hi) {
        const double* base = own + oy * PX;
        double w[4][4];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const double* p = base + slot(lo + j);
#pragma unroll
            for (int r = 0; r < 4; ++r) w[r][j] = p[r * PX];
        }
        int ox = lo;
#pragma unroll 1
        for (; ox + 3 <= hi; ox += 4) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const double* p = base + slot(ox + s + 3);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    w[r][(s + 3) & 3] = p[r * PX];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc[r][j] = shell_add<P>(acc[r][j], w[r][(s + j) & 3] - q[r][j]);
                }
            }
        }
#pragma unroll 1
        for (; ox <= hi; ++ox) {
            const double* p = base + slot(ox + 3);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                w[r][3] = p[r * PX];
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[r][j] = shell_add<P>(acc[r][j], w[r][j] - q[r][j]);
#pragma unroll
                for (int j = 0; j < 3; ++j) w[r][j] = w[r][j + 1];
            }
        }
    };
    // the offsets (ox, oy), oy = 1..hi, of every cell: a window w[column] of four rows that slides up
    auto along_column = [&](int ox, int hi) {
        const double* p[4];
        double w[4][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            p[j] = own + PX + slot(ox + j);
#pragma unroll
            for (int r = 0; r < 3; ++r) w[j][r] = p[j][r * PX];
        }
        int oy = 1;
#pragma unroll 1
        for (; oy + 3 <= hi; oy += 4) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    w[j][(s + 3) & 3] = p[j][(s + 3) * PX];
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        acc[r][j] = shell_add<P>(acc[r][j], w[j][(s + r) & 3] - q[r][j]);
                }
                p[j] += 4 * PX;
            }
        }
#pragma unroll 1
        for (; oy <= hi; ++oy) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                w[j][3] = p[j][3 * PX];
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r][j] = shell_add<P>(acc[r][j], w[j][r] - q[r][j]);
#pragma unroll
                for (int r = 0; r < 3; ++r) w[j][r] = w[j][r + 1];
                p[j] += PX;
            }
        }
    };
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll 1
    for (int h = 1; h <= H; ++h) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[r][j] = 0.0;
        shell2d_half<BALL>(h, along_row, along_column);
        double row[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[r][j] = (in_x[j] && in_y[r]) ? acc[r][j] : 0.0;
            row[r] = pairwise4(acc[r][0], acc[r][1], acc[r][2], acc[r][3]);
        }
        double sum = pairwise4(row[0], row[1], row[2], row[3]);
        constexpr int order[6] = {1, 2, 16, 32, 4, 8};   // 4 threads along x, 4 along y, 4 blocks
#pragma unroll
        for (int i = 0; i < 6; ++i) sum = sum + __shfl_xor(sum, order[i], 64);
        if (lane == 0) wsum[wave * H + (h - 1)] = sum;
    }
    __syncthreads();
    for (int h = threadIdx.x; h < H; h += kFnThreads) {
        double s = wsum[h];
        for (int w = 1; w < kFnThreads / 64; ++w) s = s + wsum[w * H + h];
        a.partial[(sq * H + h) * a.ntiles + tile] = s;
    }
}

// The same for too few tiles to keep the chip busy, bit for bit: one cell per thread, one of a
// tile's sixteen 16 x 16 blocks to a workgroup (ntiles counts blocks); a call of a few tiles is
// bound by the longest workgroup, and this one's is a sixteenth (figures at the choice, in
// fv_structure_shell). Lane bits 0 and 1 are the
// column and 2 and 3 the row in a square of 4 x 4 cells, bits 4 and 5 the square along x, the
// wavefront is the square along y.
template <int P, bool BALL>
__global__ void __launch_bounds__(kFnThreads) shell2d_cell_kernel(const ShellArgs a)
{
    constexpr int T = 16;
    extern __shared__ double lds[];
    const int H = a.H, PX = T + 2 * H, rows = T + H;
    double* wsum = lds + rows * PX;         // [waves][H]

    const int64_t blk = blockIdx.x;
    const int32_t block = (int32_t)(blk % a.ntiles), tile = block / kShellBlocks2;
    const int64_t sq = blk / a.ntiles;      // sample * nq + quantity
    const int qi = (int)(sq % a.nq);
    const double* U = a.state + (sq / a.nq) * a.nf * a.cells;
    const int32_t x0 = (tile % a.tiles[0]) * kShellTile2 + (block & 3) * T;
    const int32_t y0 = (tile / a.tiles[0]) * kShellTile2 + ((block >> 2) & 3) * T;
    double* out = a.partial + sq * H * a.ntiles + block;   // one per radius, ntiles apart
    if (x0 >= a.n[0] || y0 >= a.n[1]) {   // uniform
        for (int h = threadIdx.x; h < H; h += kFnThreads) out[(int64_t)h * a.ntiles] = 0.0;
        return;
    }

    for (int e = threadIdx.x; e < rows * PX; e += kFnThreads) {
        const int px = e % PX, py = e / PX;
        const int32_t gx = wrap_index(x0 + px - H, a.n[0], BC_PERIODIC);
        const int32_t gy = wrap_index(y0 + py, a.n[1], BC_PERIODIC);
        lds[e] = quantity_at(U, a.cells, a.nf, a.kind, (int64_t)gy * a.n[0] + gx, qi);
    }
    __syncthreads();

    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int cx = 4 * (lane >> 4) + (lane & 3), cy = 4 * wave + ((lane >> 2) & 3);
    const bool inside = x0 + cx < a.n[0] && y0 + cy < a.n[1];
    const double* own = lds + cy * PX + (cx + H);
    const double q0 = own[0];
#pragma unroll 1
    for (int h = 1; h <= H; ++h) {
        double acc = 0.0;
        shell2d_half<BALL>(
            h,
            [&](int oy, int lo, int hi) {
                const double* p = own + oy * PX;
                for (int ox = lo; ox <= hi; ++ox) acc = shell_add<P>(acc, p[ox] - q0);
            },
            [&](int ox, int hi) {
                const double* p = own + ox;
                for (int oy = 1; oy <= hi; ++oy) acc = shell_add<P>(acc, p[oy * PX] - q0);
            });
        double sum = inside ? acc : 0.0;
#pragma unroll
        for (int off = 1; off <= 32; off *= 2) sum = sum + __shfl_xor(sum, off, 64);
        if (lane == 0) wsum[wave * H + (h - 1)] = sum;
    }
    __syncthreads();
    for (int h = threadIdx.x; h < H; h += kFnThreads)
        out[(int64_t)h * a.ntiles] = pairwise4(wsum[h], wsum[H + h], wsum[2 * H + h], wsum[3 * H + h]);
}

struct ShellFinishArgs {
    const double* partial;   // [rows][ntiles], row = (sample * nq + q) * H + h - 1
    int64_t rows;
    int32_t ntiles, H, blocks; // blocks: partials are the 16 blocks of every tile
    double cells;
    double shell[kShellMaxH];  // |A_h| / 2
    double* out;             // [rows]
};

__global__ void __launch_bounds__(kFnThreads) shell_finish_kernel(const ShellFinishArgs a)
{
    const int64_t r = (int64_t)blockIdx.x * kFnThreads + threadIdx.x;
    if (r >= a.rows) return;
    const double* p = a.partial + r * a.ntiles;
    double s = 0.0;   // sums of terms >= +0
    if (a.blocks) {
        for (int t = 0; t < a.ntiles; t += kShellBlocks2) {
            double tile = 0.0;
            for (int k = t; k < t + kShellBlocks2; k += 4)
                tile = tile + pairwise4(p[k], p[k + 1], p[k + 2], p[k + 3]);
            s = s + tile;
        }
    } else {
        for (int t = 0; t < a.ntiles; ++t) s = s + p[t];
    }
    a.out[r] = s / (a.cells * a.shell[r % a.H]);
}

template <int DIM, int P>
static void launch_shell(const ShellArgs& a, int64_t blocks, size_t lds, hipStream_t s)
{
    hipLaunchKernelGGL((shell_kernel<DIM, P>), dim3((unsigned)blocks), dim3(kFnThreads), lds, s, a);
}

static void launch_shell2d_cells(const ShellArgs& a, int order, int64_t blocks, hipStream_t s)
{
    const size_t lds = sizeof(double) * (size_t)((16 + a.H) * (16 + 2 * a.H) + (kFnThreads / 64) * a.H);
    const dim3 grid((unsigned)blocks), block(kFnThreads);
    if (order == 1 && a.ball) hipLaunchKernelGGL((shell2d_cell_kernel<1, true>), grid, block, lds, s, a);
    else if (order == 1) hipLaunchKernelGGL((shell2d_cell_kernel<1, false>), grid, block, lds, s, a);
    else if (a.ball) hipLaunchKernelGGL((shell2d_cell_kernel<2, true>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((shell2d_cell_kernel<2, false>), grid, block, lds, s, a);
}

template <int HM>
static void launch_shell2d(const ShellArgs& a, int order, int64_t blocks, hipStream_t s)
{
    const size_t lds = sizeof(double) * (size_t)((kShellTile2 + a.H) * (kShellTile2 + 2 * HM) + (kFnThreads / 64) * a.H);
    const dim3 grid((unsigned)blocks), block(kFnThreads);
    if (order == 1 && a.ball) hipLaunchKernelGGL((shell2d_kernel<1, true, HM>), grid, block, lds, s, a);
    else if (order == 1) hipLaunchKernelGGL((shell2d_kernel<1, false, HM>), grid, block, lds, s, a);
    else if (a.ball) hipLaunchKernelGGL((shell2d_kernel<2, true, HM>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((shell2d_kernel<2, false, HM>), grid, block, lds, s, a);
}

// Number of offsets in the shell of radius h (same membership rule as the kernel).
static int64_t shell_size(int dim, int h, int ball)
{
    int64_t c = 0;
    const int hy = dim >= 2 ? h : 0, hz = dim >= 3 ? h : 0;
    for (int oz = -hz; oz <= hz; ++oz)
        for (int oy = -hy; oy <= hy; ++oy)
            for (int ox = -h; ox <= h; ++ox) {
                if (ball) {
                    const int r2 = ox * ox + oy * oy + oz * oz;
                    c += (h - 1) * (h - 1) < r2 && r2 <= h * h;
                } else {
                    c += std::max({std::abs(ox), std::abs(oy), std::abs(oz)}) == h;
                }
            }
    return c;
}

}  // namespace fvk

using namespace fvk;

static int32_t num_quantities(const fv_solver* s) { return quantity_kind(s) ? s->nf : 1; }

static fv_status pdf_common(const fv_solver* s, const double* state, int64_t batch, int32_t qa,
                            int32_t qb, int64_t n, const int64_t* cells_host, int per, double lo_a,
                            double hi_a, double lo_b, double hi_b, int32_t nbins, int64_t* counts,
                            bool joint)
{
    if (!s || !state || !counts || (n > 0 && !cells_host)) return fail(FV_EINVAL, "NULL argument");
    if (batch < 1) return fail(FV_EINVAL, "batch must be >= 1");
    if (n < 0) return fail(FV_EINVAL, "negative number of points");
    const int32_t nq = num_quantities(s);
    if (qa < 0 || qa >= nq || qb < 0 || qb >= nq) return fail(FV_EINVAL, "no such quantity");
    if (nbins < 1 || nbins > 65536) return fail(FV_EINVAL, "nbins must be in 1..65536");
    if (!(lo_a < hi_a) || !(lo_b < hi_b)) return fail(FV_EINVAL, "empty bin range (lo < hi required)");
    for (int64_t i = 0; i < n * per; ++i)
        if (cells_host[i] < 0 || cells_host[i] >= s->cells) return fail(FV_EINVAL, "cell index out of range");
    if (n == 0) return FV_OK;
    fv_solver* sm = const_cast<fv_solver*>(s);
    HIP_TRY(hipSetDevice(s->device));
    fv_status e = ensure_scratch(sm, sizeof(int64_t) * (size_t)(n * per));
    if (e) return e;
    e = stream_enter(sm);
    if (e) return e;
    HIP_TRY(hipMemcpyAsync(sm->scratch, cells_host, sizeof(int64_t) * (size_t)(n * per),
                           hipMemcpyHostToDevice, sm->stream));
    PdfArgs a{};
    a.state = state;
    a.cells = s->cells;
    a.nf = s->nf;
    a.kind = quantity_kind(s);
    a.batch = batch;
    a.n = n;
    a.cell = (const int64_t*)sm->scratch;
    a.qa = qa;
    a.qb = qb;
    a.nbins = nbins;
    a.joint = joint;
    a.lo_a = lo_a;
    a.hi_a = hi_a;
    a.lo_b = lo_b;
    a.hi_b = hi_b;
    a.counts = (unsigned long long*)counts;
    const int64_t threads = batch * n;
    hipLaunchKernelGGL(pdf_kernel, dim3((unsigned)((threads + kFnThreads - 1) / kFnThreads)),
                       dim3(kFnThreads), 0, sm->stream, a);
    HIP_TRY(hipGetLastError());
    return stream_leave(sm);
}

extern "C" fv_status fv_point_pdf(const fv_solver* solver, const double* state, int64_t batch,
                                  int32_t quantity, int64_t npoints, const int64_t* points,
                                  double lo, double hi, int32_t nbins, int64_t* counts)
{
    return pdf_common(solver, state, batch, quantity, quantity, npoints, points, 1, lo, hi, lo, hi,
                      nbins, counts, false);
}

extern "C" fv_status fv_joint_pdf(const fv_solver* solver, const double* state, int64_t batch,
                                  int32_t quantity_a, int32_t quantity_b, int64_t npairs,
                                  const int64_t* pairs, double lo_a, double hi_a, double lo_b,
                                  double hi_b, int32_t nbins, int64_t* counts)
{
    return pdf_common(solver, state, batch, quantity_a, quantity_b, npairs, pairs, 2, lo_a, hi_a,
                      lo_b, hi_b, nbins, counts, true);
}

extern "C" fv_status fv_structure_shell(const fv_solver* s, const double* state, int64_t batch,
                                        int32_t max_h, int32_t order, int32_t ball, double* out)
{
    if (!s || !state || !out) return fail(FV_EINVAL, "NULL argument");
    if (batch < 1) return fail(FV_EINVAL, "batch must be >= 1");
    if (max_h < 1 || max_h > kShellMaxH) return fail(FV_EINVAL, "max_h must be in 1..64");
    if (order != 1 && order != 2) return fail(FV_EINVAL, "order must be 1 or 2");
    if (ball != 0 && ball != 1) return fail(FV_EINVAL, "ball must be 0 or 1");
    const int dim = s->grid.dim;
    for (int k = 0; k < dim; ++k) {
        if (s->grid.bc[k] != FV_BC_PERIODIC) return fail(FV_ENOTSUP, "shell structure functions need periodic axes");
        if (max_h >= s->grid.n[k]) return fail(FV_ENOTSUP, "max_h must be below the cells of every axis");
    }
    const int T[3] = {dim == 1 ? 256 : (dim == 2 ? 16 : 8), dim == 1 ? 1 : (dim == 2 ? 16 : 8), dim == 3 ? 4 : 1};
    const int64_t P[3] = {T[0] + 2 * max_h, dim >= 2 ? T[1] + 2 * max_h : 1, dim >= 3 ? T[2] + 2 * max_h : 1};
    const size_t lds = sizeof(double) * (size_t)(P[0] * P[1] * P[2] + (kFnThreads / 64) * max_h);
    if (lds > 65536) return fail(FV_ENOTSUP, "max_h too large for this dimension (tile and halo exceed 64 KB of LDS)");
    // 2D, radii up to kShellMaxH2, tiles of 64 x 64 at least a quarter full: 4 x 4 cells per thread
    // where that makes enough workgroups to keep the chip busy, else one cell per thread with the
    // same sums, so results do not depend on the batch. us, one cell per thread -> 4 x 4 (4
    // quantities, radius 8, cube / ball shells): one sample of 64^2 (4 workgroups of tiles) 69 -> 88
    // / 69 -> 101, 256^2 (64) 70 -> 78 / 76 -> 90, 7 of 128^2 (112) 80 -> 79 / 91 -> 91, two of
    // 256^2 (128) 86 -> 78 / 92 -> 86, 64 of 40^2 (256, 39% full) 109 -> 78 / 117 -> 91, 64 of
    // 256^2 (4096) 998 -> 328 / 1112 -> 364; radius 16, two of 128^2 (32) 80 -> 130 / 107 -> 182.
    // Below a quarter, 64 of 20^2 (256, 10% full) took 53 us in tiles of 16 x 16 and 67 in tiles of
    // 64 x 64 (cube).
    const int64_t tiles64 = ((s->grid.n[0] + kShellTile2 - 1) / kShellTile2) * ((s->grid.n[1] + kShellTile2 - 1) / kShellTile2);
    const bool tiled = dim == 2 && max_h <= kShellMaxH2 &&
                       4 * s->cells >= tiles64 * kShellTile2 * kShellTile2;
    const bool wide = tiled && batch * num_quantities(s) * tiles64 >= 128;
    ShellArgs a{};
    a.cells = s->cells;
    a.ntiles = 1;
    for (int k = 0; k < 3; ++k) {
        const int tk = (tiled && k < 2) ? kShellTile2 : T[k];
        a.n[k] = (int32_t)s->grid.n[k];
        a.tiles[k] = (int32_t)((s->grid.n[k] + tk - 1) / tk);
        a.ntiles *= a.tiles[k];
    }
    if (tiled && !wide) a.ntiles *= kShellBlocks2;
    a.nf = s->nf;
    a.kind = quantity_kind(s);
    a.nq = num_quantities(s);
    a.H = max_h;
    a.ball = ball;
    ShellFinishArgs f{};
    f.ntiles = a.ntiles;
    f.H = max_h;
    f.blocks = tiled && !wide;
    f.cells = (double)s->cells;
    for (int h = 1; h <= max_h; ++h) f.shell[h - 1] = 0.5 * (double)shell_size(dim, h, ball);
    // samples per pass: partial sums of at most 2^22 doubles (32 MiB)
    const int64_t per_sample = (int64_t)a.nq * max_h * a.ntiles;
    const int64_t chunk = std::max<int64_t>(1, std::min<int64_t>(batch, (int64_t(1) << 22) / per_sample));
    fv_solver* sm = const_cast<fv_solver*>(s);
    HIP_TRY(hipSetDevice(s->device));
    fv_status e = ensure_scratch(sm, sizeof(double) * (size_t)(chunk * per_sample));
    if (e) return e;
    e = stream_enter(sm);
    if (e) return e;
    a.partial = (double*)sm->scratch;
    f.partial = a.partial;
    for (int64_t b0 = 0; b0 < batch; b0 += chunk) {
        const int64_t nb = std::min<int64_t>(chunk, batch - b0);
        a.state = state + b0 * s->nf * s->cells;
        const int64_t blocks = nb * a.nq * a.ntiles;
        if (wide) {
            if (max_h <= 8) launch_shell2d<8>(a, order, blocks, sm->stream);
            else launch_shell2d<kShellMaxH2>(a, order, blocks, sm->stream);
        } else if (tiled) {
            launch_shell2d_cells(a, order, blocks, sm->stream);
        } else switch (dim * 10 + order) {
            case 11: launch_shell<1, 1>(a, blocks, lds, sm->stream); break;
            case 12: launch_shell<1, 2>(a, blocks, lds, sm->stream); break;
            case 21: launch_shell<2, 1>(a, blocks, lds, sm->stream); break;
            case 22: launch_shell<2, 2>(a, blocks, lds, sm->stream); break;
            case 31: launch_shell<3, 1>(a, blocks, lds, sm->stream); break;
            default: launch_shell<3, 2>(a, blocks, lds, sm->stream); break;
        }
        f.rows = nb * a.nq * max_h;
        f.out = out + b0 * a.nq * max_h;
        hipLaunchKernelGGL(shell_finish_kernel, dim3((unsigned)((f.rows + kFnThreads - 1) / kFnThreads)),
                           dim3(kFnThreads), 0, sm->stream, f);
        HIP_TRY(hipGetLastError());
    }
    return stream_leave(sm);
}
