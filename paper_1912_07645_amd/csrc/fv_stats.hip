// fv_stats.hip -- on-device Monte Carlo statistics (Section 2.2): per-cell mean and
// variance of the quantities over samples (Welford, samples in index order) and the
// second-order two-point structure function S_q(h) of every sample, averaged over samples.
//
// Quantities: Euler (rho, u_1..u_dim, E) with u_k = m_k * (1 / rho); scalar: the field.
#include "fv_stats.h"
#include "fv_stage_y.h"

#include <algorithm>

namespace fvk {

// Per-cell Welford update over the samples of one batch, in sample order. A workgroup covers
// 64 cells with one wavefront per quantity (64 NF threads): each thread keeps the running
// moments of one (cell, quantity) in registers, so a batch has NF times as many wavefronts as
// cells / 64. The loads of the next kWelfordDepth samples are issued before the current ones
// are processed, so each thread has that many samples' loads in flight.
// KIND: 0 the field itself; 1 Euler (the momenta divided by rho); 2 shallow water (the
// momenta divided by h); 3 ideal MHD (the three momenta divided by rho). The divisor is field
// 0. SHARE: its own wavefront, which loads it anyway, passes each group of samples' values to
// the other wavefronts through LDS (two buffers, one barrier per group), so every field of a
// sample is read from memory once (400 us against 472 us with field 0 loaded by every dividing
// wavefront, for 1024 samples of 256^2 Euler).
constexpr int kWelfordDepth = 8;

template <int NF, int KIND>
__global__ void __launch_bounds__(512)
welford_kernel(const double* __restrict__ state, int64_t cells, int32_t batch, int64_t count0,
               double* __restrict__ mean, double* __restrict__ m2)
{
    constexpr bool SHARE = KIND != 0;
    constexpr int D = kWelfordDepth;
    __shared__ double f0[SHARE ? 2 * D * 64 : 1];   // [group parity][sample][cell]
    const int q = threadIdx.x >> 6;   // the wavefront's quantity
    const int lane = threadIdx.x & 63;
    const int64_t c = (int64_t)blockIdx.x * 64 + lane;
    const bool live = c < cells;      // lanes past the last cell only take part in barriers
    if (!SHARE && !live) return;      // no barrier without SHARE: such lanes leave at once
    constexpr int DIV_END = (KIND == 1) ? NF - 1 : ((KIND == 3) ? 4 : NF);
    const bool div = SHARE && q >= 1 && q < DIV_END;   // uniform across the wavefront
    const int64_t per = (int64_t)NF * cells;
    const double* F = state + q * cells + (live ? c : 0);
    double mu = live ? mean[q * cells + c] : 0.0, s2 = live ? m2[q * cells + c] : 0.0;
    double xc[D];
#pragma unroll
    for (int i = 0; i < D; ++i) xc[i] = (live && i < batch) ? F[i * per] : 0.0;
    for (int32_t b0 = 0, g = 0; b0 < batch; b0 += D, ++g) {
        double xn[D];
#pragma unroll
        for (int i = 0; i < D; ++i) {   // the next group's loads, before this group's work
            const int32_t b = b0 + D + i;
            xn[i] = (live && b < batch) ? F[b * per] : 0.0;
        }
        double* sh = f0 + (SHARE ? (g & 1) * D * 64 : 0);
        if constexpr (SHARE) {
            // the buffer written here was last read before the previous group's barrier
            if (q == 0) {
#pragma unroll
                for (int i = 0; i < D; ++i) sh[i * 64 + lane] = xc[i];
            }
            __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < D; ++i) {
            const int32_t b = b0 + i;
            if (live && b < batch) {
                double x = xc[i];
                if constexpr (SHARE) {
                    if (div) x = xc[i] * (1.0 / sh[i * 64 + lane]);
                }
                const double n = (double)(count0 + b + 1);
                const double delta = x - mu;
                mu = mu + (delta / n);
                s2 = s2 + (delta * (x - mu));
            }
        }
#pragma unroll
        for (int i = 0; i < D; ++i) xc[i] = xn[i];
    }
    if (live) {
        mean[q * cells + c] = mu;
        m2[q * cells + c] = s2;
    }
}

// Structure-function partial sums: for every lag h, sum (q(y) - q(y - h))^2 over the cells y of a
// segment of a line (with the line's periodic continuation, sum over its cells of
// (q(y + h) - q(y))^2 in another order).
//
// A lane takes a segment of a line and marches along it with the last W values in a ring of
// registers (its indices are compile-time: the march is unrolled by W), so a value is read once
// and serves W terms, a subtraction and a fused multiply-add each, into W accumulators. With more
// than 48 lags, `split` neighbouring lanes share a segment (MULTI): each takes W lags, and a value
// that leaves a lane's ring enters the next lane's. Neighbouring segments are the same part of
// neighbouring lines, then the next part, so wavefronts are full also where lines are few. The sums
// meet once, at the end. A workgroup is one wavefront (3 to a SIMD at W = 32; with four to a group,
// whose place is free only when the last ends, 556 us against 512).
//
// Lines along y and z: loads four or eight steps ahead. Lines along x: chunks of 8 columns of the
// wavefront's segments go through LDS (8 lanes a row of 64 bytes), half a chunk or one ahead.
//
// The bound is partly memory (read once per axis, 537 MB for 256 samples of 256^2 Euler, 4.6 TB/s
// with 8 lags) and partly FP64 issue (64 instructions per value and lane at W = 32, 120 us). The
// kernels before this staged lines in LDS, read 47 values from there for 256 terms and summed every
// 16 lags over the workgroup after 256 terms per thread: 322 and 296 us for the rows and the columns
// of those samples with 32 lags, now 253 and 236.
//
// Beyond 64 x 32 lags a pass is repeated with the rings delayed by h0 - 1 cells, which takes a
// second stream of the line's values (DELAY).
constexpr int kSfChunk = 8;    // columns staged at a time (lines along x)
constexpr int kSfPitch = kSfChunk + 1;
constexpr int kSfAlone = 48;   // lags of a lane that has a segment to itself

struct SfPlan {
    int32_t width, split;         // lags of a lane, lanes of a segment
    int32_t seg[3];               // per axis: cells of a segment
    int64_t segs[3];              // segments of all lines
    int64_t first[4];             // first unit (wavefront) of each axis; first[dim..3]: their number
};

// Widths 8 to 48 in one lane (37 lags of 64 samples of 256^2: 158 us per pass with one lane of 40, 2
// wavefronts to a SIMD, 225 with two lanes of 24; 64 lags of 16 samples of 512^2: 295 with one lane
// of 64, 275 with two of 32), else 2 to 64 lanes of 24 or 32. Segments of up to 128 cells (497 us
// per pass of 256 samples of 256^2 with 32 lags, against 508 with 64: every segment reads W cells
// ahead of it, and waits for them), longer ones with many lanes, which keeps the number of partial
// sums within a small multiple of the field (256 with two lanes: 64 lags of 64 samples of 256^2 340
// -> 332 us, of 16 samples 172 -> 228); shorter ones, down to 16, on grids that would have fewer than
// 16 units. A choice by grid and lags alone: sums do not depend on the batch.
static SfPlan sf_plan(int32_t dim, const int32_t n[3], int32_t max_h)
{
    SfPlan p{};
    p.split = 1;
    if (max_h > kSfAlone)
        while (p.split < 64 && 32 * p.split < max_h) p.split *= 2;
    const int32_t w = (max_h + 8 * p.split - 1) / (8 * p.split) * 8, most = p.split > 1 ? 32 : kSfAlone;
    p.width = w < most ? w : most;
    const int64_t cells = (int64_t)n[0] * n[1] * n[2];
    // twice as long where max_h sums per unit come to more than the field
    for (int32_t len = 64 * std::max(2, p.split) * ((int64_t)max_h * dim > 8192 ? 2 : 1);; len /= 2) {
        int64_t at = 0;
        for (int d = 0; d < 3; ++d) {
            const int32_t per = (n[d] + len - 1) / len;
            p.seg[d] = (n[d] + per - 1) / per;
            p.segs[d] = cells / n[d] * ((n[d] + p.seg[d] - 1) / p.seg[d]);
            p.first[d] = at;
            if (d < dim) at += (p.segs[d] * p.split + 63) / 64;
        }
        p.first[3] = at;
        if (at >= 16 || len == 16) return p;
    }
}

struct SfArgs {
    const double* state;   // [batch][nq][cells]
    int32_t n[3];
    int64_t cells;
    int32_t axis, nq, max_h, h0;
    int32_t seg, lsplit;   // log2 of the lanes of a segment
    int64_t segs;          // segments of the axis
    int64_t first, nblk;   // the axis's first unit; units of a field
    int32_t div_lo, div_hi;
    double* partial;       // [batch][nq][max_h][nblk]
};

// A line along y or z: a stream of its values from some position on, four steps ahead.
template <int B>
struct SfColumn {
    const double* q;       // the field
    const double* rho;     // field 0
    int32_t stride, span;  // of a line, in cells (cells < 2^31)
    uint32_t at, end;      // the lane's next cell to request; the cell past its line
    bool div;
    double v[B], r[B], cur[B];

    template <int G>
    __device__ __forceinline__ void load(double (&x)[G], double (&y)[G])
    {
        uint32_t p[G];
#pragma unroll
        for (int i = 0; i < G; ++i) {
            p[i] = at;
            x[i] = q[at];
            at += stride;
            at = (at == end) ? at - span : at;
        }
        if (div) {
#pragma unroll
            for (int i = 0; i < G; ++i) y[i] = rho[p[i]];
        }
    }
    template <int G>
    __device__ __forceinline__ void finish(double (&out)[G], const double (&x)[G], const double (&y)[G])
    {
        if (div) {
#pragma unroll
            for (int i = 0; i < G; ++i) out[i] = x[i] * (1.0 / y[i]);
        } else {
#pragma unroll
            for (int i = 0; i < G; ++i) out[i] = x[i];
        }
    }
    template <int G>
    __device__ __forceinline__ void fetch(double* out, double*)   // G values at once
    {
        double x[G], y[G], z[G];
        load<G>(x, y);
        finish<G>(z, x, y);
#pragma unroll
        for (int i = 0; i < G; ++i) out[i] = z[i];
    }
    __device__ __forceinline__ void begin(double*) { fetch<B>(cur, nullptr); }
    __device__ __forceinline__ void request() { load<B>(v, r); }
    __device__ __forceinline__ void take(double (&out)[B], double*)
    {
#pragma unroll
        for (int i = 0; i < B; ++i) out[i] = cur[i];
    }
    __device__ __forceinline__ void commit(double*) { finish<B>(cur, v, r); }
};

// The same for lines along x, through LDS (buf: two chunks of 64 segments x kSfPitch).
template <int B>
struct SfRow {
    const double* q;       // the field
    const double* rho;
    const int2* seg;       // per segment of the wavefront: first cell of its line, first column
    int32_t n, y;          // cells of a line; next chunk's distance from the segment's first, mod n
    bool div;
    int32_t half, side;    // B cells of the chunk at hand; buffer it is in
    double v[B], r[B];

    static __device__ __forceinline__ int32_t slot(int k) { return k * 8 + ((threadIdx.x & 63) >> 3); }

    // The values of segments slot(k0), slot(k0 + 1), ... of the next chunk.
    template <int G>
    __device__ __forceinline__ void load(double* x, double* y, int k0)
    {
        const int j = threadIdx.x & (kSfChunk - 1);
        int32_t c[G];
#pragma unroll
        for (int t = 0; t < G; ++t) {
            const int2 g = seg[slot(k0 + t)];
            uint32_t p = (uint32_t)g.y + (uint32_t)(this->y + j);   // below 2 n + 6
            p = p < (uint32_t)n ? p : p - n;
            p = p < (uint32_t)n ? p : p - n;
            if (n < kSfChunk) p %= (uint32_t)n;   // uniform
            c[t] = g.x + (int32_t)p;              // cells < 2^31
            x[t] = q[c[t]];
        }
        if (div) {
#pragma unroll
            for (int t = 0; t < G; ++t) y[t] = rho[c[t]];
        }
    }
    template <int G>
    __device__ __forceinline__ void store(const double* x, const double* y, double* buf, int k0)
    {
        double* p = buf + slot(k0) * kSfPitch + (threadIdx.x & (kSfChunk - 1));
        if (div) {
#pragma unroll
            for (int t = 0; t < G; ++t) p[t * 8 * kSfPitch] = x[t] * (1.0 / y[t]);
        } else {
#pragma unroll
            for (int t = 0; t < G; ++t) p[t * 8 * kSfPitch] = x[t];
        }
    }
    __device__ __forceinline__ void advance()
    {
        y += kSfChunk;
        if (y >= n) y = (y - n) % n;
    }
    template <int G>
    __device__ __forceinline__ void fetch(double* out, double* buf)   // G = 8 or 16 values at once
    {
        constexpr int C = G / kSfChunk;   // chunks
        double x[C][8], z[C][8];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            load<8>(x[c], z[c], 0);
            advance();
        }
#pragma unroll
        for (int c = 0; c < C; ++c) store<8>(x[c], z[c], buf + c * 64 * kSfPitch, 0);
        wave_fence();
#pragma unroll
        for (int i = 0; i < G; ++i)
            out[i] = buf[((i / kSfChunk) * 64 + (threadIdx.x & 63)) * kSfPitch + i % kSfChunk];
        wave_fence();
    }
    __device__ __forceinline__ void begin(double* buf)
    {
        double x[8], z[8];
        load<8>(x, z, 0);
        advance();
        store<8>(x, z, buf, 0);
        wave_fence();
        half = side = 0;
    }
    __device__ __forceinline__ void request() { load<B>(v, r, half * B); }
    __device__ __forceinline__ void take(double (&out)[B], double* buf)
    {
        const double* p = buf + (side * 64 + (threadIdx.x & 63)) * kSfPitch + half * B;
#pragma unroll
        for (int i = 0; i < B; ++i) out[i] = p[i];
    }
    __device__ __forceinline__ void commit(double* buf)
    {
        store<B>(v, r, buf + (side ^ 1) * 64 * kSfPitch, half * B);
        half = half + 1 < kSfChunk / B ? half + 1 : 0;
        if (half == 0) {
            side ^= 1;
            advance();
            wave_fence();
        }
    }
};

// The W cells ahead of a segment.
template <int W, class Line>
__device__ __forceinline__ void sf_fill(Line& line, double (&ring)[W], double* buf)
{
#pragma unroll
    for (int s0 = 0; s0 + 16 <= W; s0 += 16) line.template fetch<16>(ring + s0, buf);
    if constexpr (W % 16 != 0) line.template fetch<8>(ring + W / 16 * 16, buf);
}

// Sums over the wavefront of W accumulators per lane, in a fixed order (neighbouring lanes first): a
// transposing butterfly halves the lags that a lane holds at each step (the lane keeps the half
// that its bit selects and adds the partner's copy of it); the remaining steps finish the sums.
// The sum of lag h0 + l ends in the lane whose low bits, reversed, are l.
template <int H, int M, int W>
__device__ __forceinline__ void sf_wave_sum(double (&v)[W])
{
    if constexpr (H >= 1) {
        const bool up = threadIdx.x & M;
#pragma unroll
        for (int k = 0; k < H; ++k) {
            const double keep = up ? v[H + k] : v[k];
            const double give = up ? v[k] : v[H + k];
            v[k] = keep + __shfl_xor(give, M);
        }
        sf_wave_sum<H / 2, 2 * M>(v);
    } else if constexpr (M <= 32) {
        v[0] = v[0] + __shfl_xor(v[0], M);
        sf_wave_sum<0, 2 * M>(v);
    }
}

// The preceding lane's value (lane 0: unspecified).
__device__ __forceinline__ double sf_from_left(double x)
{
    constexpr int WAVE_SHR1 = 0x138;
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), WAVE_SHR1, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), WAVE_SHR1, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// a: the stream from the segment's first cell; d (DELAY): the same, delayed. ring: the W cells
// ahead of them; head: first lane of a segment; len: cells of the lane's segment, most: of any.
template <int W, int B, bool MULTI, bool DELAY, class Line>
__device__ __forceinline__ void sf_march(Line& a, Line& d, double* abuf, double* dbuf, bool head,
                                         int32_t len, int32_t most, double (&ring)[W],
                                         double (&acc)[W])
{
    a.begin(abuf);
    if (DELAY) d.begin(dbuf);
#pragma unroll 1
    for (int32_t y = 0; y < most; y += W) {
#pragma unroll
        for (int s0 = 0; s0 < W; s0 += B) {
            if (y + s0 < most) {   // uniform
                double v[B], r[B];
                a.request();
                if (DELAY) d.request();
                a.take(v, abuf);
                if (DELAY) d.take(r, dbuf);
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    const int s = s0 + i;
                    if (y + s < len) {
#pragma unroll
                        for (int l = 0; l < W; l += 4) {
                            double d0 = v[i] - ring[(s - l - 1 + W) % W];
                            double d1 = v[i] - ring[(s - l - 2 + W) % W];
                            double d2 = v[i] - ring[(s - l - 3 + W) % W];
                            double d3 = v[i] - ring[(s - l - 4 + W) % W];
                            // four at a time, since a result takes two issues (beyond 32 lags the
                            // unroller would give up)
                            if constexpr (W <= 32)
                                asm volatile("" : "+v"(d0), "+v"(d1), "+v"(d2), "+v"(d3));
                            acc[l] = __builtin_fma(d0, d0, acc[l]);
                            acc[l + 1] = __builtin_fma(d1, d1, acc[l + 1]);
                            acc[l + 2] = __builtin_fma(d2, d2, acc[l + 2]);
                            acc[l + 3] = __builtin_fma(d3, d3, acc[l + 3]);
                        }
                    }
                    const double in = DELAY ? r[i] : v[i];
                    if constexpr (MULTI) {
                        const double left = sf_from_left(ring[s]);
                        ring[s] = head ? in : left;
                    } else ring[s] = in;
                }
                a.commit(abuf);
                if (DELAY) d.commit(dbuf);
            }
        }
    }
}

// B: march steps between requests. With 8 lags a step is short against a load: 8 at a time (256
// samples of 256^2: 524 us with 4, 500 with 8); with 16 where there are few wavefronts to hide it
// (24 samples: 131 and 124; 256 samples: 549 and 565); else 4.
template <int W, int B, bool MULTI, bool DELAY, bool ROWS>
__global__ void __launch_bounds__(64)
__attribute__((amdgpu_waves_per_eu(W > 32 || DELAY ? 2 : (W >= 24 ? 3 : 4), 8)))
sf_kernel(const SfArgs a)
{
    constexpr int BUF = 2 * 64 * kSfPitch;
    __shared__ double lds[ROWS ? BUF * (DELAY ? 2 : 1) : 1];
    __shared__ int2 seg[ROWS ? 64 : 1];
    const int lane = threadIdx.x;
    const int64_t unit = blockIdx.x;
    const int lsplit = MULTI ? a.lsplit : 0, part = lane & ((1 << lsplit) - 1);
    const int64_t want = (unit * 64 + lane) >> lsplit;
    const bool live = want < a.segs;
    const uint32_t at = (uint32_t)(live ? want : a.segs - 1);   // segs <= cells < 2^31
    const int32_t n = a.n[a.axis];
    const uint32_t lines = (uint32_t)(a.cells / n);
    const int32_t line = (int32_t)(at % lines), y0 = (int32_t)(at / lines) * a.seg;
    const int32_t len = !live ? 0 : (n - y0 < a.seg ? n - y0 : a.seg);
    const int qi = blockIdx.y, b = blockIdx.z;
    const double* F = a.state + ((int64_t)b * a.nq + qi) * a.cells;
    const double* R = a.state + (int64_t)b * a.nq * a.cells;
    const bool div = qi >= a.div_lo && qi < a.div_hi;
    const int32_t shift = a.h0 - 1;
    // first cells of the lane's ring and of the delayed stream
    const int32_t yr = wrap_index(y0 - shift - (part + 1) * W, n, BC_PERIODIC);
    const int32_t yd = DELAY ? wrap_index(y0 - shift, n, BC_PERIODIC) : 0;
    double ring[W], acc[W];
#pragma unroll
    for (int l = 0; l < W; ++l) acc[l] = 0.0;
    if constexpr (ROWS) {
        double* dbuf = lds + (DELAY ? BUF : 0);
        seg[lane] = make_int2(line * n, yr);
        wave_fence();
        using Row = SfRow<B>;
        Row d{F, R, seg, n, 0, div};
        sf_fill<W>(d, ring, lds);
        seg[lane] = make_int2(line * n, y0);
        wave_fence();
        Row v{F, R, seg, n, 0, div};
        if (DELAY) d = Row{F, R, seg, n, n - shift % n, div};
        if (DELAY && d.y == n) d.y = 0;
        sf_march<W, B, MULTI, DELAY>(v, d, lds, dbuf, part == 0, len, a.seg, ring, acc);
    } else {
        const int32_t stride = (a.axis == 1) ? a.n[0] : a.n[0] * a.n[1];
        const uint32_t base = (uint32_t)(line / stride) * stride * n + line % stride;
        const uint32_t end = base + n * stride;   // < 2^32: base and span are below 2^31
        using Column = SfColumn<B>;
        Column v{F, R, stride, n * stride, base + yr * stride, end, div};
        sf_fill<W>(v, ring, nullptr);
        v.at = base + y0 * stride;
        Column d{F, R, stride, n * stride, base + yd * stride, end, div};
        sf_march<W, B, MULTI, DELAY>(v, d, nullptr, nullptr, part == 0, len, a.seg, ring, acc);
    }
    double* out = a.partial + ((int64_t)b * a.nq + qi) * a.max_h * a.nblk + a.first + unit;
    if constexpr (MULTI) {   // lanes of one part of the lags are 1 << lsplit apart
#pragma unroll
        for (int l = 0; l < W; ++l) {
            for (int m = 1 << lsplit; m <= 32; m *= 2) acc[l] = acc[l] + __shfl_xor(acc[l], m);
            const int h = a.h0 + part * W + l;
            if (lane == part && h <= a.max_h) out[(int64_t)(h - 1) * a.nblk] = acc[l];
        }
    } else {
        constexpr int P = W <= 8 ? 8 : (W <= 16 ? 16 : (W <= 32 ? 32 : 64));   // lags, padded
        double sum[P];
#pragma unroll
        for (int l = 0; l < P; ++l) sum[l] = l < W ? acc[l] : 0.0;
        sf_wave_sum<P / 2, 1>(sum);
        const int l = (int)(__brev((unsigned)lane) / (0x80000000u / (P / 2))), h = a.h0 + l;
        if (lane < P && l < W && h <= a.max_h) out[(int64_t)(h - 1) * a.nblk] = sum[0];
    }
}

// The same partial sums, bit for bit, for launches of few units. A wavefront of the kernel above is
// alone on its SIMD there, and takes the segment's cells one after the other for all its lags
// (256^2, one sample, 37 lags: two launches of 32 wavefronts and 128 steps, 130 us the call). Here a
// workgroup stages a unit's segments and the cells behind them in LDS, each value formed once, and
// a thread takes four lags of a segment: the same terms in the same order, and the same tree over
// the segments. One launch for all axes. 73 us the call; the bound is the chain of loads, steps
// and sums of one workgroup, and with more of them the two LDS reads for eight operations.
// LDS: val[cell][segment], cell 0 the one max_h behind the segment's first.
constexpr int kSfSmallLags = 4;
constexpr int kSfSmallThreads = 1024;

struct SfSmallArgs {
    const double* state;   // [batch][nq][cells]
    int32_t n[3];
    int64_t cells;
    int32_t nq, max_h, parts, staged;   // a unit's segments: `parts` times `staged` of them
    SfPlan p;
    int32_t div_lo, div_hi;
    double* partial;       // [batch][nq][max_h][units]
};

__global__ void __launch_bounds__(kSfSmallThreads) sf_small_kernel(const SfSmallArgs a)
{
    constexpr int L = kSfSmallLags, D = 4;
    extern __shared__ double val[];
    __shared__ int2 from[64];   // of a segment's line, the first cell; the column of cell 0
    const int64_t unit = blockIdx.x;
    const int axis = unit >= a.p.first[2] ? 2 : (unit >= a.p.first[1] ? 1 : 0);
    const int S = a.staged, parts = a.parts, H = a.max_h;
    const int pitch = S | 1;   // odd: cells of a line in different banks
    const int32_t n = a.n[axis], seg = a.p.seg[axis];
    const int64_t segs = a.p.segs[axis];
    const uint32_t lines = (uint32_t)(a.cells / n);
    const uint32_t stride = axis == 0 ? 1u : (axis == 1 ? (uint32_t)a.n[0] : (uint32_t)a.n[0] * (uint32_t)a.n[1]);
    const int qi = blockIdx.y, b = blockIdx.z;
    const double* F = a.state + ((int64_t)b * a.nq + qi) * a.cells;
    const double* R = a.state + (int64_t)b * a.nq * a.cells;
    const bool div = qi >= a.div_lo && qi < a.div_hi;   // uniform
    const int s = threadIdx.x & (S - 1), h0 = 1 + (int)(threadIdx.x / S) * L;
    double sum[L];
#pragma unroll
    for (int l = 0; l < L; ++l) sum[l] = 0.0;

#pragma unroll 1
    for (int part = 0; part < parts; ++part) {
        const int64_t at0 = ((unit - a.p.first[axis]) * parts + part) * S;
        if (at0 >= segs) break;   // uniform
        if (threadIdx.x < (unsigned)S) {
            const uint32_t at = (uint32_t)(at0 + threadIdx.x < segs ? at0 + threadIdx.x : segs - 1);   // segs < 2^31
            const uint32_t line = at % lines;
            from[threadIdx.x] = make_int2((int32_t)(line / stride * stride * n + line % stride),
                                          wrap_index((int32_t)(at / lines) * seg - H, n, BC_PERIODIC));
        }
        __syncthreads();   // and the part before is read
        // the segments' values: D cells of a segment at a time, `apart` cells from each other, by
        // lanes along the line for x, across the lines for y and z
        const int span = seg + H, waves = blockDim.x >> 6, lane = threadIdx.x & 63;
        const int apart = axis == 0 ? 64 : (int)blockDim.x / S;
        for (int k = axis == 0 ? (int)threadIdx.x >> 6 : s; k < S; k += axis == 0 ? waves : S) {
            const int2 f = from[k];
            for (int c0 = axis == 0 ? lane : (int)threadIdx.x / S; c0 < span; c0 += D * apart) {
                double v[D], r[D];
#pragma unroll
                for (int i = 0; i < D; ++i) {
                    const int c = c0 + i * apart;
                    v[i] = r[i] = 1.0;
                    if (c < span) {
                        const uint32_t cell = (uint32_t)f.x + (uint32_t)wrap_index(f.y + c, n, BC_PERIODIC) * stride;
                        v[i] = F[cell];   // cells < 2^31
                        if (div) r[i] = R[cell];
                    }
                }
#pragma unroll
                for (int i = 0; i < D; ++i) {
                    const int c = c0 + i * apart;
                    if (c < span) val[c * pitch + k] = div ? v[i] * (1.0 / r[i]) : v[i];
                }
            }
        }
        __syncthreads();

        const int64_t want = at0 + s;
        const int32_t y0 = (int32_t)(want / lines) * seg;
        const int32_t len = (want >= segs || h0 > H) ? 0 : (n - y0 < seg ? n - y0 : seg);
        const double* now = val + H * pitch + s;
        // w[l]: the value h0 + l cells behind (lags beyond max_h: any, and not stored)
        double w[L], acc[L];
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const int c = H - h0 - l;
            w[l] = val[(c < 0 ? 0 : c) * pitch + s];
            acc[l] = 0.0;
        }
        for (int y = 0; y < len; y += D) {   // D cells of padding past the last segment's end
            double v[D], in[D];
#pragma unroll
            for (int i = 0; i < D; ++i) {
                v[i] = now[(y + i) * pitch];
                in[i] = now[(y + i + 1 - h0) * pitch];
            }
#pragma unroll
            for (int i = 0; i < D; ++i) {
                if (y + i < len) {
#pragma unroll
                    for (int l = 0; l < L; ++l) {
                        const double d = v[i] - w[l];
                        acc[l] = __builtin_fma(d, d, acc[l]);
                    }
                }
#pragma unroll
                for (int l = L - 1; l > 0; --l) w[l] = w[l - 1];
                w[0] = in[i];
            }
        }
#pragma unroll
        for (int l = 0; l < L; ++l) {
            for (int m = 1; m < S; m *= 2) acc[l] = acc[l] + __shfl_xor(acc[l], m);
            sum[l] = sum[l] + acc[l];   // 0 + the first half + the second
        }
    }
    double* out = a.partial + ((int64_t)b * a.nq + qi) * H * a.p.first[3] + unit;
#pragma unroll
    for (int l = 0; l < L; ++l)
        if (s == 0 && h0 + l <= H) out[(int64_t)(h0 + l - 1) * a.p.first[3]] = sum[l];
}

// S_q(h) of every sample of the chunk: the unit partials of (sample, quantity, lag) summed and
// normalised. kSumLanes lanes per (sample, quantity, lag), each over every kSumLanes-th unit, for
// loads in flight and in whole lines (512 x 512, 64 lags, 128 units: 5.9 us, with one lane 18.8).
constexpr int kSumLanes = 8;
__global__ void sf_sum_kernel(const double* __restrict__ partial, int32_t n_out, int64_t nblk,
                              double denom, double* __restrict__ x)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t t = i / kSumLanes;
    const int lane = (int)(i % kSumLanes);
    double s = 0.0;   // sums of squares: +0 is neutral
    if (t < n_out)
        for (int64_t k = lane; k < nblk; k += kSumLanes) s = s + partial[t * nblk + k];
#pragma unroll
    for (int m = kSumLanes / 2; m >= 1; m /= 2) s = s + __shfl_xor(s, m);
    if (t < n_out && lane == 0) x[t] = s / denom;
}

// Moments over samples of S_q(h), in sample order. One thread per (quantity, lag).
__global__ void sf_welford_kernel(const double* __restrict__ x, int32_t nq, int32_t max_h,
                                  int32_t batch, int64_t count0, double* __restrict__ s2mean,
                                  double* __restrict__ s2m2)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int nt = nq * max_h;
    if (t >= nt) return;
    constexpr int D = kWelfordDepth;
    double mu = s2mean[t], s2 = s2m2[t];
    double xc[D];
#pragma unroll
    for (int i = 0; i < D; ++i) xc[i] = (i < batch) ? x[(int64_t)i * nt + t] : 0.0;
    for (int32_t b0 = 0; b0 < batch; b0 += D) {
        double xn[D];
#pragma unroll
        for (int i = 0; i < D; ++i)   // the next group's loads, before this group's work
            xn[i] = (b0 + D + i < batch) ? x[(int64_t)(b0 + D + i) * nt + t] : 0.0;
#pragma unroll
        for (int i = 0; i < D; ++i) {
            const int32_t b = b0 + i;
            if (b < batch) {
                const double v = xc[i];
                const double n = (double)(count0 + b + 1);
                const double delta = v - mu;
                mu = mu + (delta / n);
                s2 = s2 + (delta * (v - mu));
            }
        }
#pragma unroll
        for (int i = 0; i < D; ++i) xc[i] = xn[i];
    }
    s2mean[t] = mu;
    s2m2[t] = s2;
}

// Multilevel Monte Carlo level differences: per fine cell, Welford over coupled samples of
// x = q(u_fine) - q(u_coarse at the parent cell) (piecewise-constant prolongation).
template <int NF, int KIND>
__global__ void __launch_bounds__(256)
welford_diff_kernel(const double* __restrict__ fine, const double* __restrict__ coarse,
                    DiffGeom geo, int32_t batch, int64_t count0, double* __restrict__ mean,
                    double* __restrict__ m2)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t cells = (int64_t)geo.nf[0] * geo.nf[1] * geo.nf[2];
    const int64_t ccells = (int64_t)geo.nc[0] * geo.nc[1] * geo.nc[2];
    if (c >= cells) return;
    const int32_t i = (int32_t)(c % geo.nf[0]);
    const int32_t j = (int32_t)((c / geo.nf[0]) % geo.nf[1]);
    const int32_t k = (int32_t)(c / ((int64_t)geo.nf[0] * geo.nf[1]));
    const int64_t pc = ((int64_t)(k / geo.r[2]) * geo.nc[1] + (j / geo.r[1])) * geo.nc[0] + (i / geo.r[0]);
    double mu[NF], s2[NF];
#pragma unroll
    for (int q = 0; q < NF; ++q) {
        mu[q] = mean[q * cells + c];
        s2[q] = m2[q * cells + c];
    }
    for (int32_t b = 0; b < batch; ++b) {
        const double* Uf = fine + (int64_t)b * NF * cells + c;
        const double* Uc = coarse + (int64_t)b * NF * ccells + pc;
        double xf[NF], xc[NF];
#pragma unroll
        for (int q = 0; q < NF; ++q) {
            xf[q] = Uf[q * cells];
            xc[q] = Uc[q * ccells];
        }
        if (KIND != 0) {
            const double irf = 1.0 / xf[0];
            const double irc = 1.0 / xc[0];
#pragma unroll
            for (int q = 1; q < ((KIND == 1) ? NF - 1 : ((KIND == 3) ? 4 : NF)); ++q) {
                xf[q] = xf[q] * irf;
                xc[q] = xc[q] * irc;
            }
        }
        const double n = (double)(count0 + b + 1);
#pragma unroll
        for (int q = 0; q < NF; ++q) {
            const double x = xf[q] - xc[q];
            const double delta = x - mu[q];
            mu[q] = mu[q] + (delta / n);
            s2[q] = s2[q] + (delta * (x - mu[q]));
        }
    }
#pragma unroll
    for (int q = 0; q < NF; ++q) {
        mean[q * cells + c] = mu[q];
        m2[q * cells + c] = s2[q];
    }
}

// Multilevel estimate on the finest grid: out = sum_l P_{l->L} mean_l, levels in order.
__global__ void mlmc_combine_kernel(const CombineArgs a, double* __restrict__ out)
{
    const int64_t cells = (int64_t)a.nfine[0] * a.nfine[1] * a.nfine[2];
    const int64_t total = cells * a.nq;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t q = t / cells, c = t % cells;
        const int32_t i = (int32_t)(c % a.nfine[0]);
        const int32_t j = (int32_t)((c / a.nfine[0]) % a.nfine[1]);
        const int32_t k = (int32_t)(c / ((int64_t)a.nfine[0] * a.nfine[1]));
        double acc = 0.0;
        for (int l = 0; l < a.nlevels; ++l) {
            const int32_t* n = a.n[l];
            const int32_t* r = a.r[l];
            const int64_t lc = (int64_t)n[0] * n[1] * n[2];
            const int64_t pc = ((int64_t)(k / r[2]) * n[1] + (j / r[1])) * n[0] + (i / r[0]);
            const double v = a.mean[l][q * lc + pc];
            acc = (l == 0) ? v : (acc + v);
        }
        out[t] = acc;
    }
}

void launch_welford_diff(int nf, int kind, const double* fine, const double* coarse,
                         const DiffGeom& geo, int32_t batch, int64_t count0, double* mean,
                         double* m2, hipStream_t s)
{
    const int64_t cells = (int64_t)geo.nf[0] * geo.nf[1] * geo.nf[2];
    const unsigned nb = (unsigned)((cells + 255) / 256);
#define FV_DIFF(NFV, K) hipLaunchKernelGGL((welford_diff_kernel<NFV, K>), dim3(nb), dim3(256), 0, s, \
                                           fine, coarse, geo, batch, count0, mean, m2)
    if (kind == 0) FV_DIFF(1, 0);
    else if (kind == 3) FV_DIFF(8, 3);
    else if (kind == 2 && nf == 2) FV_DIFF(2, 2);
    else if (kind == 2) FV_DIFF(3, 2);
    else if (nf == 3) FV_DIFF(3, 1);
    else if (nf == 4) FV_DIFF(4, 1);
    else FV_DIFF(5, 1);
#undef FV_DIFF
}

void launch_mlmc_combine(const CombineArgs& a, double* out, hipStream_t s)
{
    hipLaunchKernelGGL(mlmc_combine_kernel, dim3(1024), dim3(256), 0, s, a, out);
}

__global__ void variance_kernel(const double* __restrict__ m2, int64_t n, double count,
                                double* __restrict__ var)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        var[i] = m2[i] / count;
}

__global__ void fill_zero_kernel(double* __restrict__ p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

int64_t sf_units(int32_t dim, const int32_t n[3], int32_t max_h)
{
    return sf_plan(dim, n, max_h).first[3];
}

// At most 256 samples, 512 MB of states and 1 GB of partial sums (or those of one sample).
int32_t sf_chunk(int32_t dim, const int32_t n[3], int32_t nq, int32_t max_h)
{
    const int64_t state = (int64_t)sizeof(double) * nq * n[0] * n[1] * n[2];
    const int64_t sums = (int64_t)sizeof(double) * nq * max_h * (sf_units(dim, n, max_h) + 1);
    const int64_t most = std::min((int64_t(512) << 20) / state, (int64_t(1) << 30) / sums);
    return (int32_t)std::max<int64_t>(1, std::min<int64_t>(256, most));
}

template <int NF, int KIND>
static void welford_launch(const double* state, int64_t cells, int32_t batch, int64_t count0,
                           double* mean, double* m2, hipStream_t s)
{
    static_assert(NF * 64 <= 512, "one wavefront per quantity");
    const unsigned nb = (unsigned)((cells + 63) / 64);
    hipLaunchKernelGGL((welford_kernel<NF, KIND>), dim3(nb), dim3(64 * NF), 0, s, state, cells, batch,
                       count0, mean, m2);
}

void launch_welford(int nf, int kind, const double* state, int64_t cells, int32_t batch,
                    int64_t count0, double* mean, double* m2, hipStream_t s)
{
    if (kind == 0) welford_launch<1, 0>(state, cells, batch, count0, mean, m2, s);
    else if (kind == 3) welford_launch<8, 3>(state, cells, batch, count0, mean, m2, s);
    else if (kind == 2 && nf == 2) welford_launch<2, 2>(state, cells, batch, count0, mean, m2, s);
    else if (kind == 2) welford_launch<3, 2>(state, cells, batch, count0, mean, m2, s);
    else if (nf == 3) welford_launch<3, 1>(state, cells, batch, count0, mean, m2, s);
    else if (nf == 4) welford_launch<4, 1>(state, cells, batch, count0, mean, m2, s);
    else welford_launch<5, 1>(state, cells, batch, count0, mean, m2, s);
}

template <int W, int B, bool MULTI, bool DELAY>
static void sf_launch(const SfArgs& a, int32_t batch, hipStream_t s)
{
    const dim3 grid((unsigned)(((a.segs << a.lsplit) + 63) / 64), a.nq, batch), block(64);
    if (a.axis == 0) hipLaunchKernelGGL((sf_kernel<W, B, MULTI, DELAY, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((sf_kernel<W, B, MULTI, DELAY, false>), grid, block, 0, s, a);
}

// Passes of few units go by sf_small_kernel. us per call, marching -> small (Euler, 2D):
// one lane per segment, to 1024 units: 256^2, one sample (64 units) 8 lags 95 -> 68, 37 lags
// 130 -> 73; 8 samples (512) 101 -> 79, 138 -> 96; 16 samples (1024) 110 -> 107, 151 -> 133; 24 samples
// (1536) 108 -> 130, 154 -> 164;
// several lanes, to 4096: 64 lags, 256^2, one sample (128) 144 -> 68, 24 samples (3072) 217 -> 181,
// 32 samples (4096) 226 -> 216, 48 samples (6144) 282 -> 293; 512^2 x 8 (4096) 244 -> 210, x 16 (8192)
// 335 -> 347; 250 lags, 512^2 x 8 (4096) 612 -> 522, x 16 (8192) 898 -> 975.
// A unit of 64 segments is staged at once where few units are about or two fit a CU's LDS, else in
// halves, for three workgroups per CU: 256^2, 37 lags, one sample 73 at once and 84 in halves, 16
// samples 147 and 133.
static bool sf_small(const SfPlan& p, int32_t nq, int32_t max_h, int32_t batch, SfSmallArgs& a, size_t& lds)
{
    const int64_t units = p.first[3] * nq * batch;
    if (units > (p.split > 1 ? 4096 : 1024)) return false;
    const int32_t seg = std::max(p.seg[0], std::max(p.seg[1], p.seg[2]));
    auto bytes = [&](int staged) { return sizeof(double) * (size_t)(seg + max_h + 4) * (staged | 1); };
    a.parts = p.split == 1 && units > 512 && bytes(64) > 80 * 1024 ? 2 : 1;
    a.staged = 64 / p.split / a.parts;
    lds = bytes(a.staged);
    return (max_h + kSfSmallLags - 1) / kSfSmallLags * a.staged <= kSfSmallThreads && lds <= 160 * 1024;
}

void launch_sf_partial(const double* state, int32_t dim, const int32_t n[3], int32_t nq,
                       int32_t max_h, int32_t batch, int kind, double* partial, hipStream_t s)
{
    const SfPlan p = sf_plan(dim, n, max_h);
    SfArgs a{};
    a.state = state;
    for (int d = 0; d < 3; ++d) a.n[d] = n[d];
    a.cells = (int64_t)n[0] * n[1] * n[2];
    a.nq = nq;
    a.max_h = max_h;
    a.nblk = p.first[3];
    a.partial = partial;
    while (1 << a.lsplit < p.split) ++a.lsplit;
    // quantities formed from the state as the Welford pass forms them: fields div_lo..div_hi-1
    // divided by field 0
    a.div_lo = kind > 0 ? 1 : 0;
    a.div_hi = kind == 1 ? nq - 1 : (kind == 3 ? 4 : (kind == 2 ? nq : 0));
    SfSmallArgs b{};
    size_t lds;
    if (sf_small(p, nq, max_h, batch, b, lds)) {
        b.state = state;
        for (int d = 0; d < 3; ++d) b.n[d] = n[d];
        b.cells = a.cells;
        b.nq = nq;
        b.max_h = max_h;
        b.p = p;
        b.div_lo = a.div_lo;
        b.div_hi = a.div_hi;
        b.partial = partial;
        const int tasks = b.staged * ((max_h + kSfSmallLags - 1) / kSfSmallLags);
        hipLaunchKernelGGL(sf_small_kernel, dim3((unsigned)p.first[3], nq, batch),
                           dim3(tasks > 512 ? kSfSmallThreads : 512), lds, s, b);
        return;
    }
    const bool few = p.first[3] * nq * batch <= 2048;
    for (a.h0 = 1; a.h0 <= max_h; a.h0 += p.width * p.split) {
        for (a.axis = 0; a.axis < dim; ++a.axis) {
            a.seg = p.seg[a.axis];
            a.segs = p.segs[a.axis];
            a.first = p.first[a.axis];
            if (a.h0 > 1) sf_launch<32, 4, true, true>(a, batch, s);   // width 32: max_h > 64 * 32
            else if (p.split > 1 && p.width == 24) sf_launch<24, 4, true, false>(a, batch, s);
            else if (p.split > 1) sf_launch<32, 4, true, false>(a, batch, s);
            else if (p.width == 48) sf_launch<48, 4, false, false>(a, batch, s);
            else if (p.width == 40) sf_launch<40, 4, false, false>(a, batch, s);
            else if (p.width == 32) sf_launch<32, 4, false, false>(a, batch, s);
            else if (p.width == 24) sf_launch<24, 4, false, false>(a, batch, s);
            else if (p.width == 16 && few) sf_launch<16, 8, false, false>(a, batch, s);
            else if (p.width == 16) sf_launch<16, 4, false, false>(a, batch, s);
            else sf_launch<8, 8, false, false>(a, batch, s);
        }
    }
}

void launch_sf_welford(const double* partial, int32_t nq, int32_t max_h, int64_t nblk,
                       int32_t batch, int64_t count0, double denom, double* x, double* s2mean,
                       double* s2m2, hipStream_t s)
{
    const int n_out = batch * nq * max_h;
    const int64_t threads = (int64_t)n_out * kSumLanes;
    hipLaunchKernelGGL(sf_sum_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, partial,
                       n_out, nblk, denom, x);
    const int t = nq * max_h;
    hipLaunchKernelGGL(sf_welford_kernel, dim3((t + 63) / 64), dim3(64), 0, s, x, nq, max_h, batch,
                       count0, s2mean, s2m2);
}

void launch_variance(const double* m2, int64_t n, double count, double* var, hipStream_t s)
{
    hipLaunchKernelGGL(variance_kernel, dim3(1024), dim3(256), 0, s, m2, n, count, var);
}

void launch_fill_zero(double* p, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(fill_zero_kernel, dim3(1024), dim3(256), 0, s, p, n);
}

}  // namespace fvk
