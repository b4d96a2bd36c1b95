// fv_stage_y.h -- the 2D Runge--Kutta stage kernel in its row-marching form: one wavefront, no
// barrier.
//
// It computes exactly what the tiled stage kernel computes (same faces, same arithmetic, same
// order of the divergence terms). A wavefront owns a strip of 64 columns, one lane each, and
// walks a segment of rows along y:
//   * each lane keeps the 2G cells of its column that the next y face reads in registers; the y
//     flux on the lower face of a cell is the one the lane computed a row before;
//   * the current row goes through LDS for the x faces: a lane computes the face on the left of
//     its cell and takes the flux on the right from its neighbour. LDS operations of one
//     wavefront complete in order, so the exchange needs no barrier, and nothing couples the
//     wavefronts of a CU;
//   * the columns beside the strip, and the x faces on the strip's right end (64 cells have 65),
//     are taken care of before the march, one lane per row: a single load and face pass for the
//     whole segment. In the march the end lanes read those from LDS, through addresses that
//     advance a row at a time where the other lanes' stay;
//   * the cell two rows up is requested at the top of a row and used after its x face, U^n is
//     requested then and used after the y face.
// What bounds it is the issue of FP64 instructions, and this form issues fewer per cell than a
// tile does: no index arithmetic per cell (a tile spends about 150 instructions per thread on
// it), 2 + 2/R faces per cell instead of 2.13, every lane a cell (a tile of 16 x 15 leaves 16 of
// 256 threads idle, and part of its last row of tiles). The price is parallelism: it needs
// many segments of 64 R cells each to fill the chip (the rule is march_pays in fv_api.hip).
#pragma once

#include "fv_stage.h"

namespace fvk {

constexpr int kStrip = 64;       // columns of a strip: one lane each
constexpr int kStripWaves = 4;   // wavefronts of a workgroup, each with a strip segment of its own

template <int EQ, int RECON, int R>
struct Strip {
    static constexpr int NF = NumFields<2, EQ>::value;
    static constexpr int G = Ghost<RECON>::value;
    // LDS of one field, in doubles: the row with its G cells on the left and one on the right;
    // the x fluxes of the row, 65 for a full strip; the y fluxes below the row; and for every
    // row of the segment what the end lanes need (SIDE columns: the G cells on the left, the one
    // on the right, the x flux at the right end)
    static constexpr int SIDE = G + 2;
    static constexpr int FX = kStrip + G + 1;
    static constexpr int FY = FX + kStrip + 1;
    static constexpr int END = FY + kStrip;
    static constexpr int QS = END + SIDE * R;
    static_assert(R <= kStrip, "one lane per row before the march");
};

// Cells around the x face on the left of a lane's own cell (from registers), the others from
// the row in LDS; s is the lane's.
template <int NF, int G, int QS>
struct StripCells {
    const double* row;
    const double (&own)[NF];
    int lane;
    __device__ __forceinline__ double operator()(int q, int j) const
    {
        return j == 2 ? own[q] : row[q * QS + lane + (j - 2 + G)];
    }
    __device__ __forceinline__ Reread<StripCells> reread() const { return Reread<StripCells>{*this}; }
};

// Orders LDS accesses of the wavefront's lanes: what was written before is read after.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int EQ, int RECON, int FLUX, int R, int WPE>
__global__ void __launch_bounds__(64 * kStripWaves) __attribute__((amdgpu_waves_per_eu(WPE, 8)))
stage_kernel_y(const StageArgs args)
{
    using T = Strip<EQ, RECON, R>;
    constexpr int NF = T::NF, G = T::G, QS = T::QS;
    constexpr bool TAME = has_tame_face<EQ, RECON, FLUX>();
    constexpr bool FIN = cells_need_finite<EQ, RECON, FLUX>();
    __shared__ double lds[kStripWaves * NF * QS];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double* s = lds + wave * (NF * QS);

    // nblocks counts strip segments, kStripWaves of them to a workgroup
    const uint32_t blk = (uint32_t)xcd_remap(blockIdx.x, gridDim.x) * kStripWaves + wave;
    if (blk >= (uint32_t)args.nblocks) return;
    const int gi = find_group(args.g, args.ngroups, blk);
    const Group& g = args.g[gi];
    const uint32_t local = blk - (uint32_t)g.block0;
    const uint32_t sample = g.by_ntiles.quotient(local);
    const uint32_t tile = local - sample * (uint32_t)g.ntiles;
    if (!g.active[sample]) return;   // uniform
    const uint32_t ty = g.by_t0.quotient(tile);
    const uint32_t tx = tile - ty * (uint32_t)g.tiles[0];
    const int32_t nx = g.n[0], ny = g.n[1];
    const int32_t x0 = (int32_t)tx * kStrip, y0 = (int32_t)ty * R;
    const int32_t W = (nx - x0 < kStrip) ? nx - x0 : kStrip;
    const int32_t y1 = (ny - y0 < R) ? ny : y0 + R;
    const int64_t cells = g.cells;
    const int64_t sbase = (int64_t)sample * NF * cells;
    const double* src = g.src + sbase;
    const double* un = g.un + sbase + x0;
    double* dst = g.dst + sbase + x0;
    const int lane = threadIdx.x & 63;
    const bool own = lane < W;
    const int pos = own ? lane : W - 1;   // lanes past the strip shadow its last column
    const uint32_t col = sizeof(double) * pos;

    // before the march: lane r loads the columns beside the strip in row y0 + r and computes the
    // x face at the strip's right end there
    bool tame = true;   // every cell loaded so far is, uniform
    const int rows = y1 - y0;
    if (lane < rows) {
        const int32_t row = (y0 + lane) * nx;   // cells < 2^31
        double e[2 * G][NF];   // around the right end
#pragma unroll
        for (int j = 0; j < 2 * G; ++j) {
            const int32_t c = row + wrap_index(x0 + W - G + j, nx, args.bc[0]);
#pragma unroll
            for (int q = 0; q < NF; ++q) e[j][q] = src[q * cells + c];
        }
        double l[G][NF];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const int32_t c = row + wrap_index(x0 - G + j, nx, args.bc[0]);
#pragma unroll
            for (int q = 0; q < NF; ++q) l[j][q] = src[q * cells + c];
        }
#pragma unroll
        for (int q = 0; q < NF; ++q) {
#pragma unroll
            for (int j = 0; j < G; ++j) s[q * QS + T::END + j * R + lane] = l[j][q];
            s[q * QS + T::END + G * R + lane] = e[G][q];
        }
        if constexpr (TAME) {
            CellRange range;
#pragma unroll
            for (int q = 0; q < NF; ++q) {
#pragma unroll
                for (int j = 0; j < G; ++j) range.add<FIN>(l[j][q]);
#pragma unroll
                for (int j = 0; j < 2 * G; ++j) range.add<FIN>(e[j][q]);
            }
            tame = !any_lane(!range.tame());
        }
        double F[NF];
        face_flux<2, EQ, RECON, FLUX, 0>(RowCells<NF, G>{e}, g.ph, TAME && tame, F);
#pragma unroll
        for (int q = 0; q < NF; ++q) s[q * QS + T::END + (G + 1) * R + lane] = F[q];
    }
    tame = TAME && !any_lane(!tame);

    // column window: w[j] = row k - G + 1 + j of the column at the face above row k
    src += x0;
    double w[2 * G][NF];
#pragma unroll
    for (int j = 0; j < 2 * G; ++j) {
        const double* p = row_ptr(src, wrap_index(y0 - G + j, ny, args.bc[1]), nx);
#pragma unroll
        for (int q = 0; q < NF; ++q) w[j][q] = *at_byte(p + q * cells, col);
    }
    if constexpr (TAME) {
        CellRange range;
#pragma unroll
        for (int j = 0; j < 2 * G; ++j)
#pragma unroll
            for (int q = 0; q < NF; ++q) range.add<FIN>(w[j][q]);
        tame = tame && !any_lane(!range.tame());
    }
    MarchReconstruct<RECON, NF> rec;
    rec.start(RowCells<NF, G>{w});
    {
        double F[NF];
        face_flux<2, EQ, RECON, FLUX, 1>(RowCells<NF, G>{w}, g.ph, tame, F, rec);
#pragma unroll
        for (int q = 0; q < NF; ++q) s[q * QS + T::FY + lane] = F[q];
    }
#pragma unroll
    for (int j = 0; j + 1 < 2 * G; ++j)
#pragma unroll
        for (int q = 0; q < NF; ++q) w[j][q] = w[j + 1][q];

    const double dt = g.dt[sample];
    const double beta = args.beta;
    double m = 0.0;
    bool bad = false;

    wave_fence();   // the ends of every row are in LDS
#pragma unroll 1
    for (int32_t k = y0; k < y1; ++k) {
        // 1. the row into LDS, its ends by the first lanes; request the cell G rows up
        if (own) {
#pragma unroll
            for (int q = 0; q < NF; ++q) s[q * QS + G + lane] = w[G - 1][q];
        }
        if (lane < T::SIDE) {
            const int to = lane < G ? lane : (lane == G ? G + W : T::FX + W);
#pragma unroll
            for (int q = 0; q < NF; ++q) s[q * QS + to] = s[q * QS + T::END + lane * R + (k - y0)];
        }
        {
            const double* p = row_ptr(src, wrap_index(k + G, ny, args.bc[1]), nx);
#pragma unroll
            for (int q = 0; q < NF; ++q) w[2 * G - 1][q] = *at_byte(p + q * cells, col);
        }
        wave_fence();
        // 2. the x face on the left of the cell
        {
            double F[NF];
            face_flux<2, EQ, RECON, FLUX, 0>(StripCells<NF, G, QS>{s, w[G - 1], pos}, g.ph, tame, F);
            if (own) {
#pragma unroll
                for (int q = 0; q < NF; ++q) s[q * QS + T::FX + lane] = F[q];
            }
        }
        // 3. the y face above it
        if constexpr (TAME) {
            CellRange range;
#pragma unroll
            for (int q = 0; q < NF; ++q) range.add<FIN>(w[2 * G - 1][q]);
            tame = tame && !any_lane(!range.tame());
        }
        double fyp[NF];
        face_flux<2, EQ, RECON, FLUX, 1>(RowCells<NF, G>{w}, g.ph, tame, fyp, rec);
        wave_fence();
        double unr[NF];
        if (args.use_un) {
            const double* p = row_ptr(un, k, nx);
#pragma unroll
            for (int q = 0; q < NF; ++q) unr[q] = *at_byte(p + q * cells, col);
        }
        // 4. divergence (x, y) and the Runge--Kutta stage combination
        double out[NF];
#pragma unroll
        for (int q = 0; q < NF; ++q) {
            double acc = (s[q * QS + T::FX + pos + 1] - s[q * QS + T::FX + pos]) * g.ph.inv_dx[0];
            acc = acc + ((fyp[q] - s[q * QS + T::FY + lane]) * g.ph.inv_dx[1]);
            const double rhs = -acc;
            const double up = w[G - 1][q];
            const double u0 = args.use_un ? unr[q] : up;
            out[q] = u0 + (beta * ((up - u0) + (dt * rhs)));
            s[q * QS + T::FY + lane] = fyp[q];
        }
        if (own) {
            double* p = row_ptr(dst, k, nx);
#pragma unroll
            for (int q = 0; q < NF; ++q) *at_byte(p + q * cells, col) = out[q];
        }
        if (args.last) {
            bool b;
            const double v = cell_speed<2, EQ>(out, g.ph, b);
            m = vmax(m, v);
            bad = bad || b;   // a shadow lane repeats a cell of the strip
        }
        // 5. the next row
#pragma unroll
        for (int j = 0; j + 1 < 2 * G; ++j)
#pragma unroll
            for (int q = 0; q < NF; ++q) w[j][q] = w[j + 1][q];
        wave_fence();
    }
    if (args.last) {
        m = wave_max(m);
        const bool anybad = any_lane(bad);
        if (lane == 0) {
            atomicMax(&g.mbits[(tile % kSpeedSlots) * speed_pitch(g.batch) + sample],
                      (unsigned long long)__double_as_longlong(m));
            if (anybad) atomicOr(&g.bad[sample], 1);
        }
    }
}

template <int EQ, int RECON, int FLUX, int R, int WPE>
void launch_stage_y(const StageArgs& a, hipStream_t s)
{
    hipLaunchKernelGGL((stage_kernel_y<EQ, RECON, FLUX, R, WPE>), dim3((unsigned)((a.nblocks + kStripWaves - 1) / kStripWaves)), dim3(64 * kStripWaves), 0, s,
                       a);
}

// Rows of a segment: each costs a face pass of its rows' lanes for the right end and a first y
// face besides its rows, and long segments leave the last round of wavefronts thin. 256 samples
// of 256^2, us per step: WENO3 + HLLC 1478 with 8 rows, 1452 with 12, 1439 with 16; MUSCL + HLL
// 740, 749, 766.
template <int EQ, int RECON, int FLUX, int WPE = 4>
constexpr StageKernel make_stage_kernel_y()
{
    constexpr int R = (RECON == REC_WENO3) ? 16 : 8;
    return StageKernel{&launch_stage_y<EQ, RECON, FLUX, R, WPE>, &launch_speed<2, EQ>,
                       kStrip, R, 1, kSpeedCellsPerBlock, kMarchRows};
}

}  // namespace fvk
