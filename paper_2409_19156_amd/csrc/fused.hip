// FP64 Zernike series without a stored basis: the recurrence runs inside the
// contraction, and its values go from the lane that forms them straight into
// an FP64 MFMA operand (forward and forward-mode derivative) or weigh what an
// MFMA returns to it (column dots of the backward); the coefficient gradient
// passes them through a wave's own piece of LDS.
//
// MFMA 16x16x4 (FP64): lane l = x + 16 y (x < 16, y < 4) supplies A[x][y] and
// B[y][x] and receives D[y + 4 t][x], t = 0..3.
//
// Forward (fwd_kernel): D = points x sets.  Lane (x, y) walks chain y of a
// quad at point x, so at every degree its value is A[x][y] with the
// contraction index running over the quad's four chains; the cos and the sin
// columns of a degree are two contraction steps over one recurrence value
// times two angular factors.  B is the four coefficient rows.
// Column dots (dot_kernel): D = modes x points, H = c g^T for two degrees at a
// time: D[y + 4 t][x] is the cos (t even) or sin column of degree t / 2 on
// chain y at point x, so lane (x, y) receives exactly the modes of the chain
// that it walks itself, and weighs them with its own recurrence values.  Over
// a chain only the sums of H v^(i) are kept; the powers, angles and chain-rule
// factors are applied once per chain.
// Coefficient gradient (grad_kernel): D = modes x sets, contracted over
// points.  A lane walks whole chains at its own point and a wave collects 16
// modes x 64 points in LDS, read back as A[mode][point].
//
// Arithmetic of the walk: as the basis kernel (chain_kernel.hip).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "angle.hpp"
#include "series.hpp"

namespace zp {
namespace {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256; // kSlices waves
static_assert(kThreads == 64 * kSlices, "one wave per slice");

// x^e for e >= 0 by binary powering (about 2 log2(e) roundings).
__device__ __forceinline__ double ipow(double x, int e)
{
    double acc = 1.0;
    while (e) {
        if (e & 1) acc *= x;
        x *= x;
        e >>= 1;
    }
    return acc;
}

// Anchor, s(r) and ds/dr of a point (zp_internal.hpp).
struct Anchor {
    double s, s1;
    bool high;
    __device__ __forceinline__ explicit Anchor(double r)
    {
        const double r2 = r * r;
        high = !(r2 < 0.5);
        s = high ? __builtin_fma(-2.0 * r, r, 2.0) : 2.0 * r2;
        s1 = high ? -4.0 * r : 4.0 * r;
    }
    __device__ __forceinline__ Anchor() {}
};

// The recurrence of one (chain, point): v^(i) and d^(i), i <= J, and the
// factor a (QuadStep) of the current degree times v.
template <int J> struct Walk {
    double v[J + 1], d[J + 1], a;
    __device__ __forceinline__ void start()
    {
#pragma unroll
        for (int i = 0; i <= J; ++i) {
            v[i] = i == 0 ? 1.0 : 0.0;
            d[i] = 0.0;
        }
        a = 1.0;
    }
    __device__ __forceinline__ void step(double cc, double bs, double s)
    {
#pragma unroll
        for (int i = J; i >= 1; --i)
            d[i] = __builtin_fma(cc, d[i], -bs * __builtin_fma(s, v[i], (double)i * v[i - 1]));
        d[0] = __builtin_fma(cc, d[0], -bs * (s * v[0]));
#pragma unroll
        for (int i = 0; i <= J; ++i) v[i] += d[i];
    }
};

typedef int i2 __attribute__((ext_vector_type(2)));

// Orders a wave's own LDS writes before its reads (and the other way round);
// the hardware does, this keeps the compiler to it.
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wave's window of kWindow rows of its quad's recurrence steps in LDS.  The
// steps come from LDS so that a step is never waited for behind the
// coefficient loads in flight (loads from memory return in order); the next
// step's record is read a step ahead, each point's lane reading its own
// anchor's half (no selects).
constexpr int kWindow = kStepTail;
template <int N> struct StepWindow {
    QuadStep *lds; // [kWindow][4][2]
    const QuadStep *rows;
    int lane, off[N]; // off: place of (chain, anchor) of each point within a row
    int K;
    double cc[N], bs[N], fa[N]; // step K + 1
    d2 pre[kWindow * 16 / 64];
    // Rows 0 .. kWindow - 1 on their way (fetch), then in place (start).
    __device__ __forceinline__ void fetch(const QuadStep *from)
    {
#pragma unroll
        for (int k = 0; k < kWindow * 16 / 64; ++k) pre[k] = ((const d2 *)from + lane)[64 * k];
    }
    __device__ __forceinline__ void place()
    {
        wave_lds_order();
#pragma unroll
        for (int k = 0; k < kWindow * 16 / 64; ++k) ((d2 *)lds + lane)[64 * k] = pre[k];
        wave_lds_order();
    }
    __device__ __forceinline__ void read()
    {
        const QuadStep *row = lds + 8 * ((K + 1) & (kWindow - 1));
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const d2 c = *(const d2 *)&row[off[i]];
            cc[i] = c[0];
            bs[i] = c[1];
            fa[i] = row[off[i]].a;
        }
    }
    __device__ __forceinline__ void start()
    {
        place();
        K = 0;
        read();
    }
    template <int J> __device__ __forceinline__ void advance(Walk<J> (&w)[N], const Anchor (&an)[N])
    {
        ++K;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            w[i].step(cc[i], bs[i], an[i].s);
            w[i].a = fa[i];
        }
        if (((K + 1) & (kWindow - 1)) == 0) { // the window moves on
            fetch(rows + 8 * (K + 1));
            place();
        }
        read();
    }
};

// r^e for the four chains of a quad: the power of the smallest alpha is the
// same for every lane, and where the others are within three of it the rest
// is a product of r and r^2 chosen by the lane.
__device__ __forceinline__ double quad_pow(double r, double r2, int e, int e_min, int spread)
{
    if (spread > 3) return ipow(r, e);
    const int k = e - e_min;
    double w = ipow(r, __builtin_amdgcn_readfirstlane(e_min));
    w = k & 1 ? w * r : w;
    return k & 2 ? w * r2 : w;
}

// Logical workgroup number: consecutive ones run on one XCD (workgroups are
// dealt round-robin to the 8 XCDs, each with its own L2).
__device__ __forceinline__ int64_t xcd_order(int64_t id, int64_t total)
{
    const int64_t t8 = total / 8 * 8;
    return id < t8 ? (id % 8) * (t8 / 8) + id / 8 : id;
}

// ---------------------------------------------------------------- forward --

struct FwdArgs {
    const Quad *quads;
    const QuadStep *steps;
    const int32_t *hdr, *cols, *slice;
    const double *r, *th;
    int64_t P;
    const double *c;  // Z's coefficients (DIR: may be null)
    const double *c2; // DIR: the directional derivative's coefficients
    const double *tr, *tt;
    uint32_t B;
    double *f;
    int64_t npb; // point blocks
};

// FM x FN output tiles of 16 points x 16 sets per wave; a workgroup's four
// waves take the plan's four slices of the modes for the same tiles and add
// their sums through LDS.
//
// What bounds it: on gfx950 FP64 MFMAs and vector instructions do not overlap
// (counters of the n <= 64 forward add up to MFMA cycles + 4 cycles per vector
// instruction within 7% of the elapsed cycles), so the split takes vector
// instructions out: the recurrence runs once per point and chain for both
// angular factors and all sets of the tile, table values come from LDS in the
// lane that needs them, angles by Turn.  Two waves per SIMD (at most 256
// registers, accumulators in vector registers: a build that kept them in
// accumulation registers moved them at every step).  Measured, n <= 64, 65536
// points: 1 set 130 us where the basis + GEMM took 745 (the basis alone writes
// 1.1 GB), 64 sets 382 us (47.1 TFLOP/s) from 755; n <= 20, 5000 points, 8
// sets 54 -> under 15 us a call.
template <int FM, int FN, bool DIR>
__global__ __launch_bounds__(kThreads, 2) void fwd_kernel(FwdArgs g)
{
    constexpr int J = DIR ? 1 : 0;
    __shared__ double red[kSlices][FN * 256];
    __shared__ QuadStep windows[kSlices][8 * kWindow];
    const int lane = threadIdx.x & 63, x = lane & 15, y = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t lid = xcd_order(blockIdx.x, gridDim.x);
    const int64_t pb = lid % g.npb;
    const uint32_t b0 = (uint32_t)(lid / g.npb) * (16 * FN);
    const int64_t p0 = pb * (16 * FM);

    d4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int n = 0; n < FN; ++n) acc[i][n] = d4{0, 0, 0, 0};

    const int q0 = g.slice[wave], q1 = g.slice[wave + 1];
    if (q0 < q1) {
        double rr[FM], r2[FM], tr[DIR ? FM : 1], tt[DIR ? FM : 1];
        Turn th[FM];
        Anchor an[FM];
        StepWindow<FM> win;
        win.lds = windows[wave];
        win.lane = lane;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int64_t p = p0 + 16 * i + x;
            const int64_t pl = p < g.P ? p : g.P - 1; // lanes past the end repeat the last point
            rr[i] = g.r[pl];
            r2[i] = rr[i] * rr[i];
            th[i] = Turn(g.th[pl]);
            an[i] = Anchor(rr[i]);
            win.off[i] = 2 * y + an[i].high;
            if constexpr (DIR) {
                tr[i] = g.tr ? g.tr[pl] : 0.0;
                tt[i] = g.tt ? g.tt[pl] : 0.0;
            }
        }
        const bool with_c = !DIR || g.c != nullptr;
        // byte offsets of this lane's sets in a row; sets past the end repeat
        // the last one (their sums are not stored)
        uint32_t bo[FN];
#pragma unroll
        for (int n = 0; n < FN; ++n) bo[n] = 8 * (b0 + 16 * n + x < g.B ? b0 + 16 * n + x : g.B - 1);
        // Groups of two entries, four contraction steps: coefficients are
        // fetched a group ahead of their use, their row numbers two.  The
        // fetched values are first touched by take(), a group later, so that
        // nothing waits for them in between.
        uint32_t col[4];
        auto load_cols = [&](int e) {
            const int32_t *c = g.cols + 8 * (int64_t)e + y;
#pragma unroll
            for (int j = 0; j < 4; ++j) col[j] = (uint32_t)c[4 * j];
        };
        auto load_c = [&](const double *c, double (&dst)[4][FN]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t row = __umul24(col[j], 8 * g.B);
#pragma unroll
                for (int n = 0; n < FN; ++n) dst[j][n] = *(const double *)((const char *)c + (row + bo[n]));
            }
        };
        // zero where a degree has no such column on this lane's chain
        auto take = [&](const i2 h, const double (&src)[4][FN], double (&dst)[4][FN]) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int n = 0; n < FN; ++n) dst[j][n] = src[j][n];
            if (((h[0] >> 16) & (h[1] >> 16)) != 255) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool has = (h[j >> 1] >> (16 + 4 * (j & 1) + y)) & 1;
#pragma unroll
                    for (int n = 0; n < FN; ++n) dst[j][n] = has ? dst[j][n] : 0.0;
                }
            }
        };
        int e = g.quads[q0].entry_off;
        double cur[4][FN], nxt[4][FN], cur2[DIR ? 4 : 1][FN], nxt2[DIR ? 4 : 1][FN];
        i2 hn = *(const i2 *)(g.hdr + e);
        load_cols(e);
        if (with_c) load_c(g.c, nxt);
        if constexpr (DIR) load_c(g.c2, nxt2);
        load_cols(e + 2);
        if (with_c) take(hn, nxt, cur);
        if constexpr (DIR) take(hn, nxt2, cur2);
        for (int q = q0; q < q1; ++q) {
            const Quad *Q = g.quads + q;
            const int alpha = Q->alpha[y];
            const int e_end = Q->entry_end;
            win.rows = g.steps + (int64_t)Q->step_off * 8;
            win.fetch(win.rows);
            // angular factors times r^alpha; DIR: the directional derivative
            // as kc0 R + kc1 dv/ds terms of a cos column, ks* of a sin column
            double wc[FM], ws[FM], kc0[DIR ? FM : 1], kc1[DIR ? FM : 1], ks0[DIR ? FM : 1], ks1[DIR ? FM : 1], av[FM];
            Walk<J> w[FM];
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                const double fa = (double)alpha;
                double cs, sn;
                th[i].angle(fa, cs, sn);
                const double w0 = quad_pow(rr[i], r2[i], alpha, Q->alpha_min, Q->spread);
                wc[i] = w0 * cs;
                ws[i] = w0 * sn;
                if constexpr (DIR) {
                    const double w1 = alpha ? fa * ipow(rr[i], alpha - 1) : 0.0;
                    kc0[i] = __builtin_fma(tr[i], w1 * cs, -(tt[i] * fa) * ws[i]);
                    ks0[i] = __builtin_fma(tr[i], w1 * sn, (tt[i] * fa) * wc[i]);
                    kc1[i] = tr[i] * an[i].s1 * wc[i];
                    ks1[i] = tr[i] * an[i].s1 * ws[i];
                }
                w[i].start();
                av[i] = 1.0;
            }
            win.start();
            for (e = Q->entry_off; e < e_end; e += 2) {
                const i2 hg = hn;
                hn = *(const i2 *)(g.hdr + e + 2);
                if (with_c) load_c(g.c, nxt);
                if constexpr (DIR) load_c(g.c2, nxt2);
                load_cols(e + 4);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int h = hg[j];
                    if (h < 0x10000) continue; // the padding of an odd number of entries
                    while (win.K < (h & 0xffff)) {
                        win.advance(w, an);
#pragma unroll
                        for (int i = 0; i < FM; ++i) av[i] = w[i].a * w[i].v[0];
                    }
#pragma unroll
                    for (int f = 0; f < 2; ++f) {
                        const int mask = (h >> (16 + 4 * f)) & 15;
                        if (mask == 0) continue;
                        double a[FM], a2[DIR ? FM : 1];
#pragma unroll
                        for (int i = 0; i < FM; ++i) {
                            a[i] = (f ? ws[i] : wc[i]) * av[i];
                            if constexpr (DIR)
                                a2[i] = __builtin_fma(f ? ks0[i] : kc0[i], av[i], (f ? ks1[i] : kc1[i]) * (w[i].a * w[i].v[J]));
                        }
                        if (mask != 15) { // a chain without this column: its lanes contribute nothing
                            asm volatile(""); // (kept as a branch: most degrees have all four)
                            const bool has = (mask >> y) & 1;
#pragma unroll
                            for (int i = 0; i < FM; ++i) {
                                a[i] = has ? a[i] : 0.0;
                                if constexpr (DIR) a2[i] = has ? a2[i] : 0.0;
                            }
                        }
                        if (with_c) {
#pragma unroll
                            for (int n = 0; n < FN; ++n)
#pragma unroll
                                for (int i = 0; i < FM; ++i)
                                    acc[i][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], cur[2 * j + f][n], acc[i][n], 0, 0, 0);
                        }
                        if constexpr (DIR) {
#pragma unroll
                            for (int n = 0; n < FN; ++n)
#pragma unroll
                                for (int i = 0; i < FM; ++i)
                                    acc[i][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a2[i], cur2[2 * j + f][n], acc[i][n], 0, 0, 0);
                        }
                    }
                }
                if (with_c) take(hn, nxt, cur);
                if constexpr (DIR) take(hn, nxt2, cur2);
            }
        }
    }
    // the four slices' sums, always as (0 + 1) + (2 + 3)
    constexpr int C = 16 * FN;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        if (i) __syncthreads();
#pragma unroll
        for (int n = 0; n < FN; ++n)
#pragma unroll
            for (int t = 0; t < 4; ++t) red[wave][(y + 4 * t) * C + 16 * n + x] = acc[i][n][t];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < FN; ++k) {
            const int e = k * kThreads + (int)threadIdx.x;
            const int64_t p = p0 + 16 * i + e / C;
            const uint32_t b = b0 + e % C;
            if (p < g.P && b < g.B) g.f[p * g.B + b] = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
        }
    }
}

template <int FM, int FN, bool DIR> void launch_fwd_t(FwdArgs g, hipStream_t s)
{
    g.npb = (g.P + 16 * FM - 1) / (16 * FM);
    const int64_t nsb = (g.B + 16 * FN - 1) / (16 * FN);
    hipLaunchKernelGGL((fwd_kernel<FM, FN, DIR>), dim3((unsigned)(g.npb * nsb)), dim3(kThreads), 0, s, g);
}

template <int FN, bool DIR> void launch_fwd_n(const FwdArgs &g, int fm, hipStream_t s)
{
    if (fm == 4 && FN == 1 && !DIR)
        launch_fwd_t<FN == 1 && !DIR ? 4 : 2, FN, DIR>(g, s);
    else if (fm >= 2)
        launch_fwd_t<2, FN, DIR>(g, s);
    else
        launch_fwd_t<1, FN, DIR>(g, s);
}

// ------------------------------------------------------------ column dots --

struct DotArgs {
    const Quad *quads;
    const QuadStep *steps;
    const int32_t *hdr, *cols, *slice;
    const double *r, *th;
    int64_t P;
    const double *c;      // first order: coefficients; second order: those of the Er, Et term
    const double *u;      // second order: coefficients of the dZ/dr, dZ/dtheta term
    const double *ur, *ut; // second order
    uint32_t B;
    const double *g;
    double *part; // [set chunk][2][P]
    double *out_r, *out_t; // with one set chunk: the outputs (nullable) instead of part
    int64_t npb;
    bool vec; // c, u and g are 16-byte aligned
};

// FP blocks of 16 points per wave, KB contraction steps of four sets (one
// chunk of 4 KB sets, on the grid).  SEC: the second-order sums; HU / HC:
// with the u and / or the c term (first order: HC alone).
//
// Bound as the forward, by MFMA and vector cycles together; the gradient's
// fragments stay in registers for the whole walk and H is weighed in the
// registers that the MFMA leaves it in, so no derivative plane is written or
// read.  n <= 64, 65536 points: 1 set 1096 -> 115 us, 64 sets 1104 -> 581 us.
template <int FP, int KB, bool SEC, bool HU, bool HC>
__global__ __launch_bounds__(kThreads, 2) void dot_kernel(DotArgs g)
{
    constexpr int J = SEC && HC ? 2 : 1;
    // sums of H v^(i): first-order term (i <= 1) and, SEC, the c term (i <= 2)
    constexpr bool FIRST = !SEC || HU;
    __shared__ double red[kSlices][2][FP * 16];
    __shared__ QuadStep windows[kSlices][8 * kWindow];
    const int lane = threadIdx.x & 63, x = lane & 15, y = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t lid = xcd_order(blockIdx.x, gridDim.x);
    const int64_t pb = lid % g.npb, chunk = lid / g.npb;
    const int64_t p0 = pb * (16 * FP);
    const uint32_t b0 = (uint32_t)chunk * (4 * KB);

    double gr[FP], gt[FP];
#pragma unroll
    for (int i = 0; i < FP; ++i) gr[i] = gt[i] = 0.0;
    const int q0 = g.slice[wave], q1 = g.slice[wave + 1];
    if (q0 < q1) {
        double rr[FP], r2[FP], ur[SEC ? FP : 1], ut[SEC ? FP : 1];
        Turn th[FP];
        Anchor an[FP];
        StepWindow<FP> win;
        win.lds = windows[wave];
        win.lane = lane;
        // Set of contraction step k: pairs of steps take neighbouring sets, so
        // that a lane's two coefficients are one 16-byte load where rows
        // allow it.  Sets past the end count as zero.
        auto set_of = [&](int k) -> uint32_t { return KB == 1 ? b0 + y : b0 + 8 * (k >> 1) + 2 * y + (k & 1); };
        const bool pairs = KB > 1 && (g.B & 1) == 0 && g.vec;
        const bool whole = b0 + 4 * KB <= g.B;
        double gv[FP][KB]; // B[y][x]: set of k at point x
        auto load_row = [&](const char *base, uint32_t off, double (&dst)[KB]) {
            if (pairs) {
#pragma unroll
                for (int k = 0; k + 1 < KB; k += 2) {
                    const uint32_t b = set_of(k);
                    const d2 v = *(const d2 *)(base + (off + 8 * (whole || b < g.B ? b : 0)));
                    dst[k] = v[0];
                    dst[k + 1] = v[1];
                }
            } else {
#pragma unroll
                for (int k = 0; k < KB; ++k) {
                    const uint32_t b = set_of(k);
                    dst[k] = *(const double *)(base + (off + 8 * (whole || b < g.B ? b : 0)));
                }
            }
        };
        // zero for sets past the end, and for a row without a column (as in
        // the forward: values are first touched here, a group after the load)
        auto take = [&](const double (&src)[KB], bool some, bool valid, double (&dst)[KB]) {
#pragma unroll
            for (int k = 0; k < KB; ++k) dst[k] = src[k];
            if (some || !whole) {
#pragma unroll
                for (int k = 0; k < KB; ++k) dst[k] = valid && (whole || set_of(k) < g.B) ? dst[k] : 0.0;
            }
        };
#pragma unroll
        for (int i = 0; i < FP; ++i) {
            const int64_t p = p0 + 16 * i + x;
            const int64_t pl = p < g.P ? p : g.P - 1;
            rr[i] = g.r[pl];
            r2[i] = rr[i] * rr[i];
            th[i] = Turn(g.th[pl]);
            an[i] = Anchor(rr[i]);
            win.off[i] = 2 * y + an[i].high;
            load_row((const char *)(g.g + pl * g.B), 0, gv[i]);
            take(gv[i], false, true, gv[i]);
            if constexpr (SEC) {
                ur[i] = g.ur ? g.ur[pl] : 0.0;
                ut[i] = g.ut ? g.ut[pl] : 0.0;
            }
        }
        // A[x][y]: row x of the group of two entries is entry x / 8, cos or
        // sin (x / 4) % 2, chain x % 4
        uint32_t col;
        auto has_row = [&](const i2 h) -> bool { return ((x & 8 ? h[1] : h[0]) >> (16 + (x & 7))) & 1; };
        auto some_absent = [&](const i2 h) -> bool { return ((h[0] >> 16) & (h[1] >> 16)) != 255; };
        double cur[KB], nxt[KB], curu[HU ? KB : 1], nxtu[HU ? KB : 1];
        int e = g.quads[q0].entry_off;
        auto load_next = [&]() {
            if constexpr (HC) load_row((const char *)g.c, __umul24(col, 8 * g.B), nxt);
            if constexpr (HU) load_row((const char *)g.u, __umul24(col, 8 * g.B), nxtu);
        };
        auto take_next = [&](const i2 h) {
            const bool some = some_absent(h), valid = has_row(h);
            if constexpr (HC) take(nxt, some, valid, cur);
            if constexpr (HU) take(nxtu, some, valid, curu);
        };
        i2 hn = *(const i2 *)(g.hdr + e);
        col = (uint32_t)g.cols[8 * (int64_t)e + x];
        load_next();
        col = (uint32_t)g.cols[8 * (int64_t)(e + 2) + x];
        take_next(hn);
        for (int q = q0; q < q1; ++q) {
            const Quad *Q = g.quads + q;
            const int alpha = Q->alpha[y];
            const int e_end = Q->entry_end;
            win.rows = g.steps + (int64_t)Q->step_off * 8;
            win.fetch(win.rows);
            Walk<J> w[FP];
            double F[FP][2][FIRST ? 2 : 1], S[FP][2][SEC && HC ? 3 : 1]; // [point][cos | sin][i]
#pragma unroll
            for (int i = 0; i < FP; ++i) {
                w[i].start();
#pragma unroll
                for (int f = 0; f < 2; ++f) {
#pragma unroll
                    for (int k = 0; k < (FIRST ? 2 : 1); ++k) F[i][f][k] = 0.0;
#pragma unroll
                    for (int k = 0; k < (SEC && HC ? 3 : 1); ++k) S[i][f][k] = 0.0;
                }
            }
            win.start();
            for (e = Q->entry_off; e < e_end; e += 2) {
                const i2 hg = hn;
                hn = *(const i2 *)(g.hdr + e + 2);
                load_next();
                col = (uint32_t)g.cols[8 * (int64_t)(e + 4) + x];
                d4 H[FP], U[HU ? FP : 1];
#pragma unroll
                for (int i = 0; i < FP; ++i) {
                    H[i] = d4{0, 0, 0, 0};
                    if constexpr (HU) U[i] = d4{0, 0, 0, 0};
                }
#pragma unroll
                for (int k = 0; k < KB; ++k)
#pragma unroll
                    for (int i = 0; i < FP; ++i) {
                        if constexpr (HC) H[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[k], gv[i][k], H[i], 0, 0, 0);
                        if constexpr (HU) U[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(curu[k], gv[i][k], U[i], 0, 0, 0);
                    }
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int h = hg[j];
                    if (h < 0x10000) continue;
                    while (win.K < (h & 0xffff)) win.advance(w, an);
                    const bool all = (h >> 16) == 255;
#pragma unroll
                    for (int f = 0; f < 2; ++f) {
                        const bool has = (h >> (16 + 4 * f + y)) & 1;
#pragma unroll
                        for (int i = 0; i < FP; ++i) {
                            if constexpr (FIRST) {
                                double hv = (HU ? U[HU ? i : 0][2 * j + f] : H[i][2 * j + f]) * w[i].a;
                                if (!all) {
                                    asm volatile("");
                                    hv = has ? hv : 0.0;
                                }
#pragma unroll
                                for (int k = 0; k < 2; ++k)
                                    F[i][f][FIRST ? k : 0] = __builtin_fma(hv, w[i].v[k], F[i][f][FIRST ? k : 0]);
                            }
                            if constexpr (SEC && HC) {
                                double hv = H[i][2 * j + f] * w[i].a;
                                if (!all) {
                                    asm volatile("");
                                    hv = has ? hv : 0.0;
                                }
#pragma unroll
                                for (int k = 0; k < 3; ++k) S[i][f][k] = __builtin_fma(hv, w[i].v[k < J ? k : J], S[i][f][k]);
                            }
                        }
                    }
                }
                take_next(hn);
            }
            // the chain's factors: w_i = d^i/dr^i r^alpha, angles, and the
            // chain rule through s(r)
#pragma unroll
            for (int i = 0; i < FP; ++i) {
                const double fa = (double)alpha;
                double cs, sn;
                th[i].angle(fa, cs, sn);
                const double w0 = quad_pow(rr[i], r2[i], alpha, Q->alpha_min, Q->spread);
                const double w1 = alpha ? fa * ipow(rr[i], alpha - 1) : 0.0;
                const double s1 = an[i].s1;
                // R and dR/dr summed with the cos and the sin columns' weights
                if constexpr (FIRST) {
                    const double zc = w0 * F[i][0][0], zs = w0 * F[i][1][0];
                    const double rc = __builtin_fma(w0 * s1, F[i][0][FIRST ? 1 : 0], w1 * F[i][0][0]);
                    const double rs = __builtin_fma(w0 * s1, F[i][1][FIRST ? 1 : 0], w1 * F[i][1][0]);
                    gr[i] += __builtin_fma(rc, cs, rs * sn);
                    gt[i] += fa * __builtin_fma(zs, cs, -(zc * sn));
                }
                if constexpr (SEC && HC) {
                    const double s2 = an[i].high ? -4.0 : 4.0;
                    const double w2 = alpha > 1 ? fa * (fa - 1.0) * ipow(rr[i], alpha - 2) : 0.0;
                    double z[2], r1[2], r2[2];
#pragma unroll
                    for (int f = 0; f < 2; ++f) {
                        z[f] = w0 * S[i][f][0];
                        r1[f] = __builtin_fma(w0 * s1, S[i][f][1], w1 * S[i][f][0]);
                        r2[f] = __builtin_fma(w0 * s1 * s1, S[i][f][2],
                                              __builtin_fma(__builtin_fma(w0, s2, 2.0 * w1 * s1), S[i][f][1], w2 * S[i][f][0]));
                    }
                    const double zrr = __builtin_fma(r2[0], cs, r2[1] * sn);
                    const double zrt = fa * __builtin_fma(r1[1], cs, -(r1[0] * sn));
                    const double ztt = -fa * fa * __builtin_fma(z[0], cs, z[1] * sn);
                    gr[i] += __builtin_fma(ur[SEC ? i : 0], zrr, ut[SEC ? i : 0] * zrt);
                    gt[i] += __builtin_fma(ur[SEC ? i : 0], zrt, ut[SEC ? i : 0] * ztt);
                }
            }
        }
    }
    // over the four chains of each lane column, then over the four slices
#pragma unroll
    for (int i = 0; i < FP; ++i) {
        gr[i] += __shfl_xor(gr[i], 16);
        gt[i] += __shfl_xor(gt[i], 16);
        gr[i] += __shfl_xor(gr[i], 32);
        gt[i] += __shfl_xor(gt[i], 32);
        if (y == 0) {
            red[wave][0][16 * i + x] = gr[i];
            red[wave][1][16 * i + x] = gt[i];
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 2 * FP * 16; e += kThreads) {
        const int o = e / (FP * 16), pl = e % (FP * 16);
        const int64_t p = p0 + pl;
        if (p >= g.P) continue;
        const double v = (red[0][o][pl] + red[1][o][pl]) + (red[2][o][pl] + red[3][o][pl]);
        if (g.part)
            g.part[(chunk * 2 + o) * g.P + p] = v;
        else if (double *out = o ? g.out_t : g.out_r)
            out[p] = v;
    }
}

template <int FP, int KB, bool SEC, bool HU, bool HC> void launch_dot_t(DotArgs g, hipStream_t s)
{
    g.npb = (g.P + 16 * FP - 1) / (16 * FP);
    const int64_t chunks = (g.B + 4 * KB - 1) / (4 * KB);
    hipLaunchKernelGGL((dot_kernel<FP, KB, SEC, HU, HC>), dim3((unsigned)(g.npb * chunks)), dim3(kThreads), 0, s, g);
}

template <int FP, bool SEC, bool HU, bool HC> void launch_dot_k(const DotArgs &g, int kb, hipStream_t s)
{
    switch (kb) {
    case 1: launch_dot_t<FP, 1, SEC, HU, HC>(g, s); break;
    case 2: launch_dot_t<FP, 2, SEC, HU, HC>(g, s); break;
    case 4: launch_dot_t<FP, 4, SEC, HU, HC>(g, s); break;
    default: launch_dot_t<SEC && HU && HC ? 1 : FP, 8, SEC, HU, HC>(g, s); break; // (two blocks would spill)
    }
}

template <bool SEC, bool HU, bool HC> void launch_dot_p(const DotArgs &g, int fp, int kb, hipStream_t s)
{
    if (fp == 2)
        launch_dot_k<2, SEC, HU, HC>(g, kb, s);
    else
        launch_dot_k<1, SEC, HU, HC>(g, kb, s);
}

// --------------------------------------------------- coefficient gradient --

struct GradArgs {
    const Chain *chains; // whole chains in emission order
    const int32_t *row_chain;
    const Coef *coefs;
    const Emit *emits;
    const double *r, *th;
    int64_t P, M;
    const double *wq;      // nullable: per-point weight of g
    const double *tr, *tt; // DIR
    const double *g;
    uint32_t B;
    int splits;
    int64_t tiles, batches; // row tiles; 64-point batches per split (a multiple of four)
    double *out;            // [split][M][B]
    int norm;               // divide by the modes' norms (one split only)
};

// (2 (n + 1)) / (eps_m pi): one over the integral of Z^2 over the disc.
__device__ __forceinline__ double inv_norm(int K, int alpha)
{
    const double inv_pi = 0.318309886183790671537767526745028724;
    return (alpha == 0 ? 1.0 : 2.0) * (double)(2 * K + alpha + 1) * inv_pi;
}

constexpr int kLd = 66;         // LDS row stride: rows 4 banks apart, the fragment read is conflict-free
constexpr int kStageSteps = 160; // recurrence steps of a tile kept in LDS

// One row of a tile's program: steps to take on its chain before the row,
// flags, and the low-anchor factor.
struct Row {
    int32_t hdr; // steps | sin << 10 | first of its chain << 11 | alpha << 12 | valid << 22
    int32_t pad;
    double a_lo;
};

// R row tiles of 16 modes (consecutive emissions) x FN tiles of 16 sets per
// workgroup; its four waves take every fourth batch of 64 points of its split
// and add their sums through LDS at the end.  A lane walks whole chains at its
// own point: the rows of a tile then need not belong to chains of one length.  The rows' program and the
// recurrence coefficients in the order the walk takes them are staged in LDS
// once per workgroup (a tile whose chains need more than kStageSteps reads
// the coefficients from memory).
//
// Bound by vector and MFMA cycles in turn and by the LDS round trip between
// them, at two or three waves per SIMD; R = 2 is the tile that fits there
// (one row tile: 388 against 347 us on n <= 64, 65536 points, 1 set; four:
// 338).  Six workgroups per CU are launched, so that the uneven tiles even
// out.  That case took 830 us with the basis stored.
template <int R, int FN, bool DIR>
__global__ __launch_bounds__(kThreads, DIR || FN > 1 ? 2 : 3) void grad_kernel(GradArgs g)
{
    constexpr int J = DIR ? 1 : 0;
    __shared__ double buf[kSlices * 16 * (16 * FN > kLd ? 16 * FN : kLd)];
    __shared__ Row prog[16 * R];
    __shared__ Coef stage[kStageSteps + 2];
    __shared__ int row_coef[16 * R]; // coefficient index of a row's first step
    __shared__ int total_steps;
    const int lane = threadIdx.x & 63, x = lane & 15, y = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t lid = xcd_order(blockIdx.x, gridDim.x);
    const int64_t tile = lid % g.tiles, rest = lid / g.tiles;
    const int64_t split = rest % g.splits;
    const uint32_t b0 = (uint32_t)(rest / g.splits) * (16 * FN);
    const int e0 = (int)tile * (16 * R);
    double *zl = buf + wave * (16 * kLd);

    // the tile's program: row t is emission e0 + t
    if ((int)threadIdx.x < 16 * R) {
        const int e = e0 + (int)threadIdx.x;
        Row rw{0, 0, 0.0};
        int first = 0;
        if (e < g.M) {
            int ci = g.row_chain[e >> 4];
            while (e >= g.chains[ci].emit_off + g.chains[ci].emit_cnt) ++ci;
            const Chain ch = g.chains[ci];
            const Emit em = g.emits[e];
            const bool fresh = e == e0 || e == ch.emit_off;
            const int before = fresh ? 0 : g.emits[e - 1].K; // degree reached by the row before
            rw.hdr = (em.K - before) | (em.flags & 1) << 10 | (fresh ? 1 << 11 : 0) | ch.alpha << 12 | 1 << 22;
            rw.a_lo = em.a_lo;
            first = ch.coef_off + before;
        }
        prog[threadIdx.x] = rw;
        row_coef[threadIdx.x] = first;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int n = 0;
        for (int t = 0; t < 16 * R; ++t) n += prog[t].hdr & 1023;
        total_steps = n;
    }
    __syncthreads();
    const bool staged = total_steps <= kStageSteps;
    if (staged && (int)threadIdx.x < 16 * R) { // each row's steps to its place in the stream
        int at = 0;
        for (int t = 0; t < (int)threadIdx.x; ++t) at += prog[t].hdr & 1023;
        const int n = prog[threadIdx.x].hdr & 1023;
        for (int k = 0; k < n; ++k) stage[at + k] = g.coefs[row_coef[threadIdx.x] + k];
    }
    __syncthreads();
    // lane t keeps row t of the program; the walk reads it lane by lane
    const Row mine = prog[lane < 16 * R ? lane : 0];
    const int a_lo_lo = (int)__builtin_bit_cast(int64_t, mine.a_lo), a_lo_hi = (int)(__builtin_bit_cast(int64_t, mine.a_lo) >> 32);

    d4 acc[R][FN];
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int n = 0; n < FN; ++n) acc[i][n] = d4{0, 0, 0, 0};

    uint32_t bo[FN]; // this lane's sets in a row, in bytes; those past the end are not stored
#pragma unroll
    for (int n = 0; n < FN; ++n) bo[n] = 8 * (b0 + 16 * n + x < g.B ? b0 + 16 * n + x : g.B - 1);
    const int64_t nb = (g.P + 63) / 64;
    const int64_t bt1 = std::min(nb, (split + 1) * g.batches);
    // the batch's own point, loaded a batch ahead
    double xr = 0, xt = 0, tr = 0, tt = 0;
    auto load_point = [&](int64_t bt) {
        const int64_t p = bt * 64 + lane, pl = p < g.P ? p : g.P - 1;
        xr = g.r[pl];
        xt = g.th[pl];
        if constexpr (DIR) {
            tr = g.tr ? g.tr[pl] : 0.0;
            tt = g.tt ? g.tt[pl] : 0.0;
        }
    };
    int64_t bt = split * g.batches + wave;
    if (bt < bt1) load_point(bt);
    for (; bt < bt1; bt += kSlices) {
        const int64_t pb = bt * 64;
        const double r = xr, tgr = tr, tgt = tt;
        const Turn th(xt);
        // B[y][x]: point pb + 4 k + y, set b0 + 16 n + x; rows past the last
        // point repeat it and count as zero below
        const uint32_t last = g.P - pb < 64 ? (uint32_t)(g.P - pb) - 1 : 63;
        const char *gb = (const char *)(g.g + pb * g.B);
        double gv[16][FN];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const uint32_t row = __umul24(std::min<uint32_t>(4 * k + y, last), 8 * g.B);
#pragma unroll
            for (int n = 0; n < FN; ++n) gv[k][n] = *(const double *)(gb + (row + bo[n]));
        }
        if (bt + kSlices < bt1) load_point(bt + kSlices);
        const Anchor an(r);
        int at = 0; // next step of the stream
        Coef q = stage[0];
        double wc = 0, wsn = 0, kc0 = 0, kc1 = 0, ks0 = 0, ks1 = 0;
        Walk<J> w;
        w.start();
#pragma unroll
        for (int i = 0; i < R; ++i) {
#pragma unroll 2
            for (int row = 0; row < 16; ++row) {
                const int h = __builtin_amdgcn_readlane(mine.hdr, 16 * i + row);
                double val = 0.0; // rows past the last mode
                if (h) {
                    if (h & 2048) { // a chain's first mode of this tile
                        const int alpha = (h >> 12) & 1023;
                        const double fa = (double)alpha;
                        double cs, sn;
                        th.angle(fa, cs, sn);
                        const double w0 = ipow(r, alpha);
                        wc = w0 * cs;
                        wsn = w0 * sn;
                        if constexpr (DIR) {
                            const double w1 = alpha ? fa * ipow(r, alpha - 1) : 0.0;
                            kc0 = __builtin_fma(tgr, w1 * cs, -(tgt * fa) * wsn);
                            ks0 = __builtin_fma(tgr, w1 * sn, (tgt * fa) * wc);
                            kc1 = tgr * an.s1 * wc;
                            ks1 = tgr * an.s1 * wsn;
                        }
                        w.start();
                    }
                    const int n = h & 1023;
                    if (staged) {
                        for (int k = 0; k < n; ++k) {
                            const Coef now_q = q;
                            q = stage[++at];
                            w.step(an.high ? now_q.cc_hi : now_q.cc_lo, an.high ? now_q.bs_hi : now_q.bs_lo, an.s);
                        }
                    } else {
                        const Coef *cf = g.coefs + __builtin_amdgcn_readfirstlane(row_coef[16 * i + row]);
                        for (int k = 0; k < n; ++k)
                            w.step(an.high ? cf[k].cc_hi : cf[k].cc_lo, an.high ? cf[k].bs_hi : cf[k].bs_lo, an.s);
                    }
                    const int64_t bits = (int64_t)(uint32_t)__builtin_amdgcn_readlane(a_lo_lo, 16 * i + row) |
                                         (int64_t)__builtin_amdgcn_readlane(a_lo_hi, 16 * i + row) << 32;
                    const double a = an.high ? 1.0 : __builtin_bit_cast(double, bits);
                    const double av = a * w.v[0];
                    const bool is_sin = h & 1024;
                    if constexpr (DIR) {
                        const double av1 = a * w.v[J];
                        val = is_sin ? __builtin_fma(ks0, av, ks1 * av1) : __builtin_fma(kc0, av, kc1 * av1);
                    } else {
                        val = (is_sin ? wsn : wc) * av;
                    }
                }
                zl[row * kLd + lane] = val;
            }
            if (i == 0) { // the gradient's weights, and zeros past the last point
                if (g.wq) {
#pragma unroll
                    for (int k = 0; k < 16; ++k) {
                        const double wgt = g.wq[pb + std::min<uint32_t>(4 * k + y, last)];
#pragma unroll
                        for (int n = 0; n < FN; ++n) gv[k][n] *= wgt;
                    }
                }
                if (last < 63) {
#pragma unroll
                    for (int k = 0; k < 16; ++k)
#pragma unroll
                        for (int n = 0; n < FN; ++n) gv[k][n] = 4 * k + y <= (int)last ? gv[k][n] : 0.0;
                }
            }
            wave_lds_order();
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const double a = zl[x * kLd + 4 * k + y];
#pragma unroll
                for (int n = 0; n < FN; ++n)
                    acc[i][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, gv[k][n], acc[i][n], 0, 0, 0);
            }
            wave_lds_order();
        }
    }
    constexpr int C = 16 * FN;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        __syncthreads();
#pragma unroll
        for (int n = 0; n < FN; ++n)
#pragma unroll
            for (int t = 0; t < 4; ++t) buf[wave * 16 * C + (y + 4 * t) * C + 16 * n + x] = acc[i][n][t];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < FN; ++k) {
            const int el = k * kThreads + (int)threadIdx.x;
            const int64_t e = e0 + 16 * i + el / C;
            const uint32_t b = b0 + el % C;
            if (e >= g.M || b >= g.B) continue;
            double v = (buf[el] + buf[16 * C + el]) + (buf[32 * C + el] + buf[48 * C + el]);
            const Emit em = g.emits[e];
            if (g.norm) {
                int lo = g.row_chain[e >> 4]; // the chain of emission e: at or after that of its row's first
                while (e >= g.chains[lo].emit_off + g.chains[lo].emit_cnt) ++lo;
                v *= inv_norm(em.K, g.chains[lo].alpha);
            }
            g.out[(split * g.M + em.col) * g.B + b] = v;
        }
    }
}

template <int R, int FN, bool DIR> void launch_grad_t(const GradArgs &g, int64_t nsb, hipStream_t s)
{
    hipLaunchKernelGGL((grad_kernel<R, FN, DIR>), dim3((unsigned)(g.tiles * g.splits * nsb)), dim3(kThreads), 0, s, g);
}

template <int R, bool DIR> void launch_grad_n(const GradArgs &g, int fn, int64_t nsb, hipStream_t s)
{
    if (fn == 2)
        launch_grad_t<R, 2, DIR>(g, nsb, s);
    else
        launch_grad_t<R, 1, DIR>(g, nsb, s);
}

// out[m][b] = (out +) sum over splits, in order; norm: times the inverse mode
// norms.  One coefficient per thread, from i0 on.
__global__ __launch_bounds__(kThreads) void grad_reduce_kernel(const double *__restrict__ part, int S, int64_t M,
                                                               int64_t B, const Chain *chains,
                                                               const int32_t *row_chain, const Emit *emits, int norm,
                                                               int accumulate, int64_t i0, double *__restrict__ out)
{
    const int64_t b = i0 + (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t e = b / B; // emission, set b - e B
    if (e >= M) return;
    const Emit em = emits[e];
    const int64_t o = em.col * B + (b - e * B);
    double v = 0.0;
#pragma unroll 8
    for (int k = 0; k < S; ++k) v += part[k * M * B + o];
    if (accumulate) v += out[o];
    if (norm) {
        int lo = row_chain[e >> 4];
        while (e >= chains[lo].emit_off + chains[lo].emit_cnt) ++lo;
        v *= inv_norm(em.K, chains[lo].alpha);
    }
    out[o] = v;
}

// Two workgroups of four waves per CU is what the larger tiles' registers
// allow; a smaller point tile is taken where that would leave CUs idle.
int64_t wanted_workgroups() { return 2 * (int64_t)std::max(1, device_cus()); }

// 24-bit products and 32-bit byte offsets into the coefficients.
bool small_rows(int64_t M, int64_t B) { return M < (1 << 24) && B < (1 << 20) && 8 * M * B < ((int64_t)1 << 32); }

} // namespace

// Chosen by the sets and the modes alone (and the 32-bit offsets), so that a
// point's row does not depend on how many points a call has or on whether it
// fills a cache.  Forward, basis + GEMM -> fused, us: (n <= 64, 65536 points)
// 565 -> 382 with 64 sets, 771 -> 598 with 96, 785 -> 745 with 128; (n <= 40,
// 2048 points) 57 -> 24 and (16384 points) 99 -> 98 with 128.  A call that fills a
// cache writes the planes as well, which the GEMM then reads, while the fused
// kernel forms the basis again: (n <= 64, 65536 points) 1145 -> 1247 with 96 sets,
// 1150 -> 1404 with 128; (n <= 40, 16384 points) 138 -> 142, 139 -> 161.  Autograd
// keeps a basis from 97 sets on (the column dot's limit), so there the line is
// 96: forward and backward of 97 to 128 sets, fused -> GEMM, 2757 -> 2520 (n <=
// 64, 65536 points), 329 -> 311 (n <= 40, 16384), 127 -> 115 (n <= 20, 16384).  The
// contraction pads the modes to 128 or 256: up to 192 modes it loses with a
// cache too, 340 -> 356 (n <= 16, 65536 points), 193 -> 202 (n <= 14, 16384).
// With the directional derivative (n <= 64, 65536 points) 1502 -> 1288 with 96
// sets, 1521 -> 1712 with 128.
bool fused_fwd_ok(int64_t M, int64_t B, bool dir) { return B <= (dir || M > 192 ? 96 : 128) && small_rows(M, B); }

zp_status launch_fused_fwd(const Plan &p, const double *r, const double *th, int64_t P, const double *c,
                           const double *c2, const double *tr, const double *tt, int64_t B, double *f, hipStream_t s)
{
    FwdArgs g{p.d_quads, p.d_qsteps, p.d_entry_hdr, p.d_entry_cols, p.d_slice_off, r, th, P, c, c2, tr, tt,
              (uint32_t)B, f, 0};
    // as few blocks of sets as 256 registers hold, of equal width
    const int64_t tiles = (B + 15) / 16, widest = c2 ? 2 : 4, nsb = (tiles + widest - 1) / widest;
    const int fn = (int)((tiles + nsb - 1) / nsb);
    int fm = 4;
    while (fm > 1 && (P + 16 * fm - 1) / (16 * fm) * nsb < wanted_workgroups()) fm /= 2;
    const int64_t most = max_workgroups(kThreads) / nsb * 16; // points of one launch, 16 or more to a workgroup
    for (int64_t p0 = 0; p0 < P; p0 += most) {
        g.r = r + p0;
        g.th = th + p0;
        g.P = std::min(most, P - p0);
        g.tr = tr ? tr + p0 : nullptr;
        g.tt = tt ? tt + p0 : nullptr;
        g.f = f + p0 * B;
        if (c2) {
            fn == 2 ? launch_fwd_n<2, true>(g, fm, s) : launch_fwd_n<1, true>(g, fm, s);
        } else {
            switch (fn) {
            case 1: launch_fwd_n<1, false>(g, fm, s); break;
            case 2: launch_fwd_n<2, false>(g, fm, s); break;
            case 3: launch_fwd_n<3, false>(g, fm, s); break;
            default: launch_fwd_n<4, false>(g, fm, s); break;
            }
        }
        const zp_status st = hip_check(hipGetLastError(), "fused forward launch");
        if (st != ZP_OK) return st;
    }
    return ZP_OK;
}

// As the forward, by the sets alone.  Column-dot GEMM (basis kept) -> fused:
// (n <= 64, 65536 points) 1104 -> 586 us with 64 sets, 1113 -> 876 with 96,
// 1097 -> 1164 with 128; (n <= 40, 16384 points) 114 -> 78, 115 -> 113, 104 ->
// 148 us; the derivative planes then need not be written either.
bool fused_dot_ok(int64_t M, int64_t B) { return B <= kFusedDotSets && small_rows(M, B); }

namespace {
// Contraction steps of four sets per chunk: 32 sets at most (with 64 the
// gradient's fragments alone take 64 registers and one wave fits a SIMD:
// 155 us on n <= 64, 4257 points, 64 sets, where two chunks of 32 took 94).
int dot_steps(int64_t B) { return B <= 4 ? 1 : B <= 8 ? 2 : B <= 16 ? 4 : 8; }
} // namespace

int64_t fused_dot_chunks(int64_t B) { return (B + 4 * dot_steps(B) - 1) / (4 * dot_steps(B)); }

int64_t fused_dot_points(int64_t B) { return max_workgroups(kThreads) / fused_dot_chunks(B) * 16; }

zp_status launch_fused_dot(const Plan &p, const double *r, const double *th, int64_t P, const double *c,
                           const double *u, const double *ur, const double *ut, bool second, int64_t B,
                           const double *g_up, double *part, double *out_r, double *out_t, hipStream_t s)
{
    const int kb = dot_steps(B);
    const int64_t chunks = fused_dot_chunks(B);
    DotArgs g{p.d_quads, p.d_qsteps, p.d_entry_hdr, p.d_entry_cols, p.d_slice_off, r, th, P, c, u, ur, ut, (uint32_t)B, g_up,
              chunks > 1 ? part : nullptr, out_r, out_t, 0,
              (((uintptr_t)c | (uintptr_t)u | (uintptr_t)g_up) & 15) == 0};
    const int fp = (P + 31) / 32 * chunks >= wanted_workgroups() ? 2 : 1;
    if (!second)
        launch_dot_p<false, false, true>(g, fp, kb, s);
    else if (u && c)
        launch_dot_p<true, true, true>(g, fp, kb, s);
    else if (u)
        launch_dot_p<true, true, false>(g, fp, kb, s);
    else
        launch_dot_p<true, false, true>(g, fp, kb, s);
    zp_status st = hip_check(hipGetLastError(), "fused column-dot launch");
    if (st != ZP_OK || chunks == 1) return st;
    return launch_coldot_reduce(part, (int)chunks, P, out_r, out_t, s);
}

// Up to 32 sets the recurrence is repeated for no second block of sets; with
// more, the basis stored once and the split-K GEMM win.  Basis + GEMM -> fused
// (dL/dc alone): (n <= 64, 65536 points) 830 -> 335 us with 1 to 16 sets, 549
// -> 459 with 32, 568 -> 857 with 64; (n <= 40, 16384 points) 87 -> 50 and 88
// -> 65 us with 16 and 32 sets, 85 -> 106 with 64; (n <= 24, 65536 points, 32
// sets) 153 -> 100 us.
bool fused_grad_ok(int64_t M, int64_t P, int64_t B) { return B <= 32 && small_rows(M, B) && P < ((int64_t)1 << 40); }

namespace {
constexpr int kGradRows = 2; // row tiles of 16 modes per workgroup
int64_t grad_set_blocks(int64_t B) { return B <= 16 ? 1 : (B + 31) / 32; }

// Point ranges of the gradient: six workgroups per CU (grad_kernel).
int64_t grad_splits(int64_t M, int64_t P, int64_t B)
{
    const int64_t tiles = (M + 16 * kGradRows - 1) / (16 * kGradRows), nb = (P + 63) / 64;
    const int64_t wanted = 6 * (int64_t)device_cus() / (tiles * grad_set_blocks(B));
    return std::min((nb + kSlices - 1) / kSlices, std::max<int64_t>(1, wanted));
}
} // namespace

size_t fused_grad_bytes(int64_t M, int64_t P, int64_t B)
{
    if (M <= 0 || P <= 0 || B <= 0) return 0;
    return 8 * (size_t)grad_splits(M, P, B) * (size_t)M * (size_t)B;
}

zp_status launch_fused_grad(const Plan &p, const double *r, const double *th, int64_t P, const double *wq,
                            const double *tr, const double *tt, const double *g_up, int64_t B, bool norm,
                            double *part, size_t part_bytes, double *out, hipStream_t s)
{
    const int64_t M = (int64_t)p.n.size();
    constexpr int R = kGradRows;
    const int fn = B <= 16 ? 1 : 2;
    const int64_t nsb = grad_set_blocks(B);
    const int64_t tiles = (M + 16 * R - 1) / (16 * R);
    const int64_t nb = (P + 63) / 64;
    int64_t S = std::min(grad_splits(M, P, B), std::max<int64_t>(1, (int64_t)(part_bytes / (8 * (size_t)M * (size_t)B))));
    const int64_t batches = ((nb + S - 1) / S + kSlices - 1) / kSlices * kSlices;
    S = (nb + batches - 1) / batches;
    if (tiles * S * nsb > max_workgroups(kThreads)) return set_error(ZP_ERR_ARG, "too many modes for one launch");
    GradArgs g{p.d_achains, p.d_row_chain, p.d_coefs, p.d_emits, r, th, P, M, wq, tr, tt, g_up, (uint32_t)B, (int)S, tiles,
               batches, S > 1 ? part : out, norm && S == 1};
    if (tr || tt)
        launch_grad_n<R, true>(g, fn, nsb, s);
    else
        launch_grad_n<R, false>(g, fn, nsb, s);
    zp_status st = hip_check(hipGetLastError(), "fused gradient launch");
    if (st != ZP_OK || S == 1) return st;
    return launch_grad_reduce(p, part, (int)S, M, B, norm, false, out, s);
}

zp_status launch_grad_reduce(const Plan &p, const double *part, int S, int64_t M, int64_t B, bool norm,
                             bool accumulate, double *C, hipStream_t s)
{
    constexpr int64_t kMost = max_workgroups(kThreads) * kThreads;
    for (int64_t i0 = 0; i0 < M * B; i0 += kMost) {
        const int64_t blocks = (std::min(kMost, M * B - i0) + kThreads - 1) / kThreads;
        hipLaunchKernelGGL(grad_reduce_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, s, part, S, M, B, p.d_achains,
                           p.d_row_chain, p.d_emits, norm ? 1 : 0, accumulate ? 1 : 0, i0, C);
        const zp_status st = hip_check(hipGetLastError(), "gradient reduce launch");
        if (st != ZP_OK) return st;
    }
    return ZP_OK;
}

} // namespace zp
