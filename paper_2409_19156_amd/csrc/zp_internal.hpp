// Internal declarations shared by the host API (zp_api.cpp), the plan builder
// (plan.cpp) and the HIP kernels.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/zp.h"

namespace zp {

// ---------------------------------------------------------------- plan --
//
// A plan is everything about a mode list that does not depend on the points:
// the modes grouped by alpha = |m| into recurrence chains (one chain per
// alpha, shared by every n of that alpha, as in Algorithm 1), the per-step
// recurrence coefficients of each chain, and the list of (K, column) pairs
// each chain must emit.
//
// Recurrence (endpoint-anchored difference form of the beta = 0 Jacobi
// recurrence of Sec. 2).  With x = 1 - 2r^2 and v_k the Jacobi polynomial
// P_k^{(alpha,0)}(x) normalised to 1 at one end of [-1, 1]:
//   low anchor (x = +1):  s = 2r^2,      v_k = P_k / C(k+alpha, k)
//   high anchor (x = -1): s = 2(1-r^2),  v_k = (-1)^k P_k
// the three-term recurrence becomes, with d_k = v_k - v_{k-1},
//   d_k = cc_k d_{k-1} - bs_k s v_{k-1},   v_k = v_{k-1} + d_k,
//   v_0 = 1, d_0 = 0, cc_1 = 0,
// low:  cc_k = (k-1)^2 (2k+alpha) / ((k+alpha)^2 (2k+alpha-2)),
//       bs_k = (2k+alpha-1)(2k+alpha) / (2 (k+alpha)^2)
// high: cc_k = (k+alpha-1)(k-1)(2k+alpha) / (k (k+alpha)(2k+alpha-2)),
//       bs_k = (2k+alpha-1)(2k+alpha) / (2k (k+alpha)).
// It is an exact algebraic rewrite of the paper's recurrence (the sum rule
// of its coefficients makes v = 1 at s = 0 a fixed point), so the end point
// is reproduced exactly and rounding errors vanish with s.
constexpr int kSegEmits = 32; // emissions per chain piece

struct Chain {
    int32_t alpha;    // |m| of every mode on this chain
    int32_t kmax;     // largest K requested on this chain
    int32_t coef_off; // first Coef of this chain (entry k-1 holds step k)
    int32_t emit_off; // first Emit of this chain
    int32_t emit_cnt; // number of Emits
    int32_t pad;
};

struct Coef {
    double cc_lo, bs_lo, cc_hi, bs_hi;
};

struct Emit {
    int32_t K;     // Jacobi degree (n - alpha)/2
    int32_t col;   // output column (position in the caller's mode list)
    int32_t flags; // bit 0: m < 0 (sin column of the basis)
    int32_t pad;
    double a_lo; // (-1)^K C(K+alpha, K): low-anchor factor from v_K to R / r^alpha
};

// ---- tables of the fused FP64 series kernels (fused.hip) ----
//
// A wave of those kernels evaluates four chains at once: lane l works on
// chain l / 16 of a quad, which is the layout of an FP64 MFMA operand whose
// contraction index runs over the four chains.  The chains of a plan are
// taken four at a time, longest first, and walk their steps together.
//
// QuadStep: recurrence step k of one chain (k = 0: no step) for one anchor,
// and the factor a from v_k to R / r^alpha: (-1)^k C(k+alpha, k) for the low
// anchor, 1 for the high one.  Rows of eight: [chain y][low, high].  Every
// chain of a quad has steps up to the quad's kmax; past its own last degree
// they change nothing (cc = bs = 0).
struct QuadStep {
    double cc, bs, a, pad;
};

// Entries: one per degree of a quad (more where columns repeat).  Entry e
// has, for each of the quad's four chains y, at most one cos and one sin
// column of degree K: hdr[e] = K | cos mask << 16 | sin mask << 20 (bit y:
// chain y has one), cols[8 e + y] and cols[8 e + 4 + y] (0 where none).
// A quad's entries are in ascending K, padded to an even count with one that
// has no column; the whole list ends with kEntryTail such entries.
constexpr int kEntryTail = 8;
constexpr int kStepTail = 32; // empty rows of steps at the end: whole windows of rows are loaded
struct Quad {
    int32_t alpha[4];
    int32_t step_off; // row of this quad's step 0
    int32_t kmax;
    int32_t entry_off, entry_end; // even; the end without the padding
    int32_t alpha_min, spread; // smallest alpha, largest alpha - alpha_min
};

// The quads are dealt to kSlices slices of about equal work, one per wave of
// a workgroup; the slices' partial sums are always combined in the same
// order, so a point's sums do not depend on the launch.
constexpr int kSlices = 4;

struct Plan {
    int device = -1;
    std::vector<int32_t> n, m; // the key
    std::vector<Chain> chains; // in launch order (most work first)
    // The same chains cut into pieces of at most kSegEmits emissions (piece
    // boundaries on multiples of 8 of the emission index).  A piece walks its
    // chain from k = 0 to its own last K and emits only its range, so it costs
    // a short recurrence prefix again; the launcher uses pieces when there
    // are too few point tiles to fill the chip with whole chains.
    std::vector<Chain> pieces;
    std::vector<Coef> coefs;
    std::vector<Emit> emits;
    std::vector<Chain> achains;      // whole chains, ascending emission index
    std::vector<int32_t> row_chain;  // row_chain[t]: index into achains of the chain of emission 16 t
    std::vector<Quad> quads;         // slice by slice: quads slice_off[w] .. slice_off[w+1] - 1 are slice w's
    std::vector<int32_t> slice_off;  // [kSlices + 1]
    std::vector<QuadStep> qsteps;    // [step_off + k][chain][anchor]
    std::vector<int32_t> entry_hdr, entry_cols;
    int32_t nmax = 0;
    // device copies (one allocation)
    void *dmem = nullptr;
    const Chain *d_chains = nullptr;
    const Chain *d_pieces = nullptr;
    const Coef *d_coefs = nullptr;
    const Emit *d_emits = nullptr;
    const int32_t *d_perm = nullptr; // d_perm[e] = emits[e].col: chain-major order -> column
    const Chain *d_achains = nullptr;
    const int32_t *d_row_chain = nullptr;
    const Quad *d_quads = nullptr;
    const int32_t *d_slice_off = nullptr;
    const QuadStep *d_qsteps = nullptr;
    const int32_t *d_entry_hdr = nullptr, *d_entry_cols = nullptr;
    // Coefficient table of the direct (closed-form) evaluation, built on first
    // use: per mode, for j = 0..3, the K+1 values c_s (n-2s)!/(n-2s-j)! of
    // d^j/dr^j of Eq. (radial-part-eq), rounded to double.
    std::once_flag direct_once;
    zp_status direct_status = ZP_OK;
    void *d_direct = nullptr;
    const int64_t *d_direct_off = nullptr; // per mode: offset of its 4 (K+1) coefficients
    const int32_t *d_direct_n = nullptr, *d_direct_m = nullptr;
    const double *d_direct_coef = nullptr;
    // Column table of the Zernike-recursion comparator, built on first use:
    // for every (n, alpha) of the triangle n <= nmax in row order (alpha =
    // n%2, n%2+2, ..., n), the output columns of the requested modes with
    // that (n, |m|): zrec_off [entries+1] into zrec_cols [M].
    std::once_flag zrec_once;
    zp_status zrec_status = ZP_OK;
    void *d_zrec = nullptr;
    const int32_t *d_zrec_off = nullptr, *d_zrec_cols = nullptr;
    ~Plan();
};

// Device table for zp_radial_zernike_recursion (uploaded once per plan).
zp_status get_zrec_table(Plan &plan);

// Zernike-recursion evaluation (Eq. zernike-recursion): out[j][i][p], j <= J.
constexpr int kZrecNmax = 60;
zp_status launch_zrec_kernel(const Plan &plan, const double *d_r, int64_t P, int J, double *out, hipStream_t s);

// Device table for zp_radial_direct (uploaded once per plan).
zp_status get_direct_table(Plan &plan);

// Direct evaluation of the closed form: out[j][i][p] for j <= J.
zp_status launch_direct_kernel(const Plan &plan, const double *d_r, int64_t P, int J, double *out, hipStream_t s);

// Validates the modes; returns ZP_OK or ZP_ERR_MODE (with the offending index
// in *bad).
zp_status validate_modes(const int32_t *n, const int32_t *m, int64_t M, int64_t *bad);

// Host-side construction of a plan (no device work).
std::shared_ptr<Plan> build_plan_host(const int32_t *n, const int32_t *m, int64_t M);

// Byte offsets of a plan's device tables within one contiguous image (the
// chains and pieces start at offset 0).
// The fused series kernels' tables come last: an image of base bytes leaves
// them out.
struct PlanOffsets {
    size_t coefs, emits, perm, base, achains, row_chain, quads, slice_off, qsteps, entry_hdr, entry_cols, total;
};
// Size of the image (and, if host is not null, the image itself).
size_t plan_image(const Plan &p, std::vector<unsigned char> *host, PlanOffsets *o);
// Point the plan's device table pointers into an image at base; the fused
// kernels' tables (the image from achains on) lie at `fused`, null: nowhere.
void plan_bind(Plan &p, const void *base, const PlanOffsets &o, const void *fused);

// Cached plan for the current device, uploaded on first use.
zp_status get_plan(const int32_t *n, const int32_t *m, int64_t M, std::shared_ptr<Plan> *out);
void clear_plans();
void clear_plans3(); // three-dimensional series tables (series3d.cpp)

// ------------------------------------------------------------- outputs --

enum PlaneFmt : int32_t { F64 = 0, F32 = 1 };

// Where the chain kernel writes.  plane[q] for q = 0..4 is R (or Z), d/dr,
// d2/dr2, d3/dr3, d/dtheta; null planes are not written.  Column i of a plane
// starts ld elements after column i-1.
// kb, if not null, receives Z once more as three bf16 planes (kb_sub apart) in
// the k-blocked layout the series forward contracts over: the mode index is
// the emission index e (chain-major order, see Plan::d_perm) and element
// (e, p) sits at ((e/8)*kb_ld + p)*8 + e%8.
// dir, if not null, receives the directional derivative
//   dZ = dr[p] dZ/dr + dtheta[p] dZ/dtheta
// of the basis along per-point tangents (dr, dtheta; either may be null),
// in format dir_fmt with the planes' ld; kb_dir, if not null, gets its
// k-blocked bf16 copy (like kb).
// sec_r / sec_t, if not null (with J = 2 and the basis), receive the
// derivatives of that directional derivative along r and theta:
//   sec_r = dr[p] d2Z/dr2 + dtheta[p] d2Z/(dr dtheta)
//   sec_t = dr[p] d2Z/(dr dtheta) + dtheta[p] d2Z/dtheta2
// in format sec_fmt with the planes' ld.
struct Planes {
    void *plane[5];
    int64_t ld;
    int32_t fmt[5];
    void *kb;
    int64_t kb_ld;
    int64_t kb_sub;
    void *dir;
    int32_t dir_fmt;
    const double *dir_r;
    const double *dir_th;
    void *kb_dir;
    void *sec_r;
    void *sec_t;
    int32_t sec_fmt;
};

// Launch the chain kernel: radial only (angular = false) or basis.  J is the
// highest radial derivative needed (0..3).
zp_status launch_chain_kernel(const Plan &plan, const double *d_r, const double *d_theta, int64_t P,
                              int J, bool angular, const Planes &out, hipStream_t s);

// The basis on a tensor grid: point p = i * nt + j at radius r[i], angle
// theta[j] (i < nr, j < nt), into plain planes with ld = nr * nt.
zp_status launch_chain_kernel_polar(const Plan &plan, const double *d_r, int64_t nr, const double *d_theta, int64_t nt,
                                    int J, const Planes &out, hipStream_t s);

// Error plumbing.
zp_status set_error(zp_status s, const std::string &msg);
zp_status hip_check(hipError_t e, const char *what);

// Workgroups that one dimension of a launch can hold: fewer than 2^32 work
// items.  (More is no error: the count wraps, and work is left out.)
constexpr int64_t max_workgroups(int64_t threads) { return (((int64_t)1 << 32) - 1) / threads; }

} // namespace zp
