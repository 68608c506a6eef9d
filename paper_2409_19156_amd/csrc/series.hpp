// Internal declarations for the Zernike series (contraction of the basis with
// coefficient sets) and its adjoint.
#pragma once

#include "zp_internal.hpp"

namespace zp {

// Contraction element types.  BF3 is a value split into three bf16 planes
// (hi, mid, lo) stored `sub` elements apart.
enum CType : int { CT_F64 = 0, CT_F32 = 1, CT_BF3 = 2 };

inline size_t ct_bytes(int ct) { return ct == CT_F64 ? 8 : ct == CT_F32 ? 4 : 6; }

// All GEMM operands live in zero-padded buffers whose dimensions are
// multiples of kPad, so tile loads never need bounds checks.
constexpr int64_t kPad = 128;
inline int64_t pad_up(int64_t x) { return (x + kPad - 1) / kPad * kPad; }

// Memory layout of a GEMM operand, element (x, k) where x is the operand's
// output index (i for A, j for B):
//   LAY_KC  : base[x*ld + k]                      (contiguous along k)
//   LAY_XC  : base[k*ld + x]                      (contiguous along x)
//   LAY_KB8 : base[((k/8)*ld + x)*8 + k%8]        (k in blocks of eight)
//   LAY_KC32: as LAY_KC, but FP32 values of a BF3 operand; the GEMM splits
//             them into the three bf16 planes on the way into LDS
enum Layout : int { LAY_KC = 0, LAY_XC = 1, LAY_KB8 = 2, LAY_KC32 = 3, LAY_FRAG = 4 };

// Operand of C(i,j) = sum_k A(i,k) B(k,j); `sub` separates the BF3 planes.
struct Operand {
    const void *base;
    int64_t ld;
    int64_t sub;
    int lay;
};

enum Epi : int {
    EPI_STORE = 0,   // C[i*ldc + j] = acc (FP64)
    EPI_PARTIAL = 1, // split-K: C + split*M*ldc, reduced later
    EPI_COLDOT = 2   // part[itile][0|1][j] = sum_i acc(i,j) D1|D2[i*ldd + j]
};

struct GemmDesc {
    int ct;
    Operand a, b;
    int64_t M, N, K; // output M x N (unpadded); K a multiple of kPad
    int splits;      // split-K count (EPI_PARTIAL); the last split may be shorter
    int64_t kchunk;  // k per split (set by launch_gemm)
    int epi;
    double *C;
    int64_t ldc;
    const void *D1, *D2; // EPI_COLDOT: derivative planes, FP64 or FP32
    int64_t ldd;
    bool d_f32;
    double *part; // EPI_COLDOT output partials [ceil(M/BM)][2][N]
    // Order of the output tiles over the launch: 0 = along a row of tiles
    // first (workgroups in flight share an A panel), 1 = down a column of
    // tiles first (they share a B panel).
    int order;
    bool beside; // another kernel runs beside this contraction (pipelined chunks)
};

// Row-tile height of the column-dot epilogue for a compute type (its
// partials buffer has ceil(M / coldot_bm(ct)) tiles).
int coldot_bm(int ct);

zp_status launch_gemm(const GemmDesc &g, hipStream_t s);

// Compute units of the current device (cached per device; 0 if unknown).
int device_cus();

// Largest number of sets for which the FP64 backward forms the derivative
// planes of dL/dr and dL/dtheta inside the contraction (fused.hip).  The
// autograd functions keep no basis up to here.
constexpr int64_t kFusedDotSets = 96;

// Series forward pieces shared by zp_series_fwd and its allocation-free
// variant: argument checks (ZP_OK also for the M, P or B == 0 no-op), the
// smallest workspace without a cache, and the work itself for a plan whose
// device tables are in place.  allow_pipe lets the forward overlap chunks on
// the library's helper stream (which it creates on first use).
zp_status series_fwd_checks(const int32_t *h_n, const int32_t *h_m, int64_t M, const double *d_r,
                            const double *d_theta, int64_t P, const double *d_c, int64_t B, int32_t prec,
                            const double *d_f);
size_t series_fwd_min_ws(int64_t M, int64_t P, int64_t B, int32_t prec);
zp_status series_fwd_run(const Plan &plan, int64_t M, const double *d_r, const double *d_theta, int64_t P,
                         const double *d_c, int64_t B, int32_t prec, double *d_f, void *d_cache, void *d_ws,
                         size_t ws_bytes, bool allow_pipe, hipStream_t s);
// Whether series_fwd_run takes the fused kernel, which needs no workspace but
// the fused tables of the plan (plan.d_quads not null).
bool series_fwd_fused(int64_t M, int64_t B, int32_t prec);

// ---- FP64 without a stored basis (fused.hip) ----

// f[p][b] = sum_k Z_k(p) c[k][b] + sum_k (tr[p] dZ_k/dr + tt[p] dZ_k/dtheta) c2[k][b]
// (c or c2 nullable, one of them given; tr, tt nullable), where
// fused_fwd_ok(.., dir = c2 given) says that the kernel takes the sizes and
// is the faster one.
bool fused_fwd_ok(int64_t M, int64_t B, bool dir);
zp_status launch_fused_fwd(const Plan &p, const double *r, const double *th, int64_t P, const double *c,
                           const double *c2, const double *tr, const double *tt, int64_t B, double *f, hipStream_t s);

// First order (second = false): out_r[p] = sum_b g[p][b] sum_k dZ_k/dr c[k][b], out_t with dZ_k/dtheta.
// Second order: the same with u in place of c (if u), plus the sums of the
// second-order planes Er, Et along (ur, ut) with c (if c).  out_r, out_t
// nullable.  part: 16 fused_dot_chunks(B) P bytes, needed when there is more
// than one chunk.  P: at most fused_dot_points(B).
bool fused_dot_ok(int64_t M, int64_t B);
int64_t fused_dot_chunks(int64_t B);
int64_t fused_dot_points(int64_t B);
zp_status launch_fused_dot(const Plan &p, const double *r, const double *th, int64_t P, const double *c,
                           const double *u, const double *ur, const double *ut, bool second, int64_t B,
                           const double *g, double *part, double *out_r, double *out_t, hipStream_t s);

// out[k][b] = sum_p Z_k(p) w[p] g[p][b] (w nullable: 1), or with the
// directional derivative along (tr, tt) in place of Z if either is given;
// norm: divided by the integral of Z_k^2.  part: workspace of part_bytes for
// the partial sums of point ranges (any size; fused_grad_bytes for as many
// ranges as are wanted).
bool fused_grad_ok(int64_t M, int64_t P, int64_t B);
size_t fused_grad_bytes(int64_t M, int64_t P, int64_t B);
zp_status launch_fused_grad(const Plan &p, const double *r, const double *th, int64_t P, const double *w,
                            const double *tr, const double *tt, const double *g, int64_t B, bool norm, double *part,
                            size_t part_bytes, double *out, hipStream_t s);

// dst (compute type, [rows_pad][ldd]) from a row-major FP64 src [R][C]
// (leading dimension lds), row r times roww[r] (roww nullable); zero padding.
zp_status launch_convert(const double *src, int64_t R, int64_t C, int64_t lds, int ct, void *dst, int64_t ldd,
                         int64_t rows_pad, int64_t sub, const double *roww, hipStream_t s);

// bf16 x 3 operand in MFMA fragment order for B(k = e, j = x) = src[perm[e]][x]:
// per k step of 32 and block of 16 columns, 64 lanes x 8 bf16 contiguous (lane
// = 16 (k % 32 / 8) + x % 16), blocks along x fastest (xblocks = xpad / 16);
// three planes sub apart; zero outside R x C.
zp_status launch_convert_gather_frag(const double *src, const int32_t *perm, int64_t R, int64_t C, int64_t lds,
                                     void *dst, int64_t xpad, int64_t kpad, int64_t sub, hipStream_t s);

// The upstream gradient g [R][C] (rows = points) as the backward's bf16 x 3
// operands from one read: [xpad_r][xpad_c] k-contiguous into dst_c (the
// column-dot's B(k = set, j = point)) and, if dst_s is set, MFMA fragment
// order into dst_s (the split-K's B(k = point, j = set)); xpad_r, xpad_c are
// the padded point and set counts (multiples of 32 and 64).  roww as above.
zp_status launch_convert_g_bwd(const double *src, int64_t R, int64_t C, int64_t lds, void *dst_c, int64_t subc,
                               void *dst_s, int64_t subs, int64_t xpad_r, int64_t xpad_c, const double *roww,
                               hipStream_t s);
// Zero the pad (modes >= M, points >= P) of a k-blocked bf16 operand.
zp_status launch_zero_kb8(void *dst, int64_t M, int64_t Mp, int64_t P, int64_t ld, int64_t sub, hipStream_t s);

// Zero the pad region of a [rows_pad][ld] plane (FP64 or FP32) whose valid
// block is [rows][cols].
zp_status launch_zero_pad(void *dst, int ct, int64_t rows, int64_t cols, int64_t rows_pad, int64_t ld, hipStream_t s);

// C[i][j] (=|+=) sum_s part[s][i][j] for s = 0..S-1, fixed order.
zp_status launch_splitk_reduce(const double *part, int S, int64_t M, int64_t N, double *C, bool accumulate,
                               hipStream_t s);
// The same for coefficients C [M][B], divided by the integrals of Z_k^2 (after
// the addition) if norm is set.
zp_status launch_grad_reduce(const Plan &p, const double *part, int S, int64_t M, int64_t B, bool norm,
                             bool accumulate, double *C, hipStream_t s);

// Whether an FP64 split-K or column-dot of these sizes takes the narrow tiles
// (64 columns): its B operand then needs 64, not 128, columns of padding.
bool gemm_narrow(int64_t M, int64_t N, int splits);
// The largest split count for which it does.
int64_t gemm_narrow_splits(int64_t M, int64_t N);

// zp_series_bwd for checked arguments; w: nullable weights of the rows of g
// (dL/dc only), norm: dL/dc divided by the integrals of Z_k^2.
zp_status series_bwd_run(const Plan &plan, int64_t M, const double *d_r, const double *d_theta, int64_t P,
                         const double *d_c, int64_t B, int32_t prec, const double *d_g, const double *d_w, bool norm,
                         const void *d_cache, double *d_grad_c, double *d_grad_r, double *d_grad_theta, void *d_ws,
                         size_t ws_bytes, hipStream_t s);

// out1[p] = sum_t part[t][0][p], out2[p] = sum_t part[t][1][p] (either nullable).
zp_status launch_coldot_reduce(const double *part, int T, int64_t P, double *out1, double *out2, hipStream_t s);

} // namespace zp
