// fv_stats.h -- statistics kernels (internal).
#pragma once

#include "fv_common.h"

namespace fvk {

// Fine grid, coarse grid and their integer refinement ratio per axis.
struct DiffGeom {
    int32_t nf[3];
    int32_t nc[3];
    int32_t r[3];
};

constexpr int kMaxLevels = 8;

struct CombineArgs {
    const double* mean[kMaxLevels];  // [quantity][cells of level l]
    int32_t n[kMaxLevels][3];        // grid of level l
    int32_t r[kMaxLevels][3];        // finest / level l, per axis
    int32_t nfine[3];
    int32_t nlevels;
    int32_t nq;
};

void launch_welford_diff(int nf, int kind, const double* fine, const double* coarse,
                         const DiffGeom& geo, int32_t batch, int64_t count0, double* mean,
                         double* m2, hipStream_t s);
void launch_mlmc_combine(const CombineArgs& a, double* out, hipStream_t s);

// Partial sums per (sample, quantity, lag) of the structure-function pass.
int64_t sf_units(int32_t dim, const int32_t n[3], int32_t max_h);
// Samples whose partial sums (and S_q(h)) are held at a time.
int32_t sf_chunk(int32_t dim, const int32_t n[3], int32_t nq, int32_t max_h);
void launch_welford(int nf, int kind, const double* state, int64_t cells, int32_t batch,
                    int64_t count0, double* mean, double* m2, hipStream_t s);
// The quantities are formed from the state as launch_welford forms them.
void launch_sf_partial(const double* state, int32_t dim, const int32_t n[3], int32_t nq,
                       int32_t max_h, int32_t batch, int kind, double* partial, hipStream_t s);
// x: scratch of batch * nq * max_h doubles (S_q(h) of each sample of the chunk).
void launch_sf_welford(const double* partial, int32_t nq, int32_t max_h, int64_t nblk,
                       int32_t batch, int64_t count0, double denom, double* x, double* s2mean,
                       double* s2m2, hipStream_t s);
void launch_variance(const double* m2, int64_t n, double count, double* var, hipStream_t s);
void launch_fill_zero(double* p, int64_t n, hipStream_t s);

}  // namespace fvk
