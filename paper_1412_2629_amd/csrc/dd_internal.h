// Host-side interface between the C-ABI layer and the kernel launchers.
#pragma once
#include <hip/hip_runtime.h>

#include <vector>

#include "dd_device.h"
#include "dd_form.h"

namespace dd {

// Canonical FP64 spinor [V][12] complex <-> internal layout in precision prec.
hipError_t import_spinor(const Geo &g, const double *canon, void *internal, int prec, hipStream_t s);
hipError_t export_spinor(const Geo &g, const void *internal, int prec, double *canon, hipStream_t s);

// Canonical FP64 links -> internal FP64 full links [d][mu][9][Vd].
hipError_t import_gauge(const Geo &g, const double *canon, double2 *U64, hipStream_t s);
// Internal FP64 full links -> first two rows in FP32 or FP16 [d][mu][6][Vd].
hipError_t compress_links(const Geo &g, const double2 *U64, void *out, int prec, hipStream_t s);
// Clover term C(x) = 1/(2 kappa) + D_cl(x), packed [d][36][Vd] FP64.
hipError_t clover_build(const Geo &g, const double2 *U64, double kappa, double csw, double2 *C64, hipStream_t s);
// Site matrices used by the block solves: C on even sites, C^-1 on odd sites.
// *bad (device int) is set to 1 if a block is singular.
hipError_t clover_schur(const Geo &g, const double2 *C64, double2 *Cs64, int *bad, hipStream_t s);
// Elementwise FP64 pairs -> FP32 / FP16 pairs.
hipError_t convert_pairs(const double2 *in, void *out, long n, int prec, hipStream_t s);
// Number of non-finite values in n FP64 pairs (device counter *cnt, accumulated).
hipError_t count_nonfinite(const double2 *v, long n, int *cnt, hipStream_t s);

// out = A in (internal layouts; links/clover in the given precision).
hipError_t apply_A(const Geo &g, const void *in, void *out, const void *links, const void *clov, int prec,
                   hipStream_t s);
// out[k] = A in[k], k < n, on one lattice: the right-hand sides share each link
// and clover load; the bits of n apply_A calls.
hipError_t apply_A_multi(const Geo &g, const void *const *in, void *const *out, int n, const void *links, const void *clov,
                         int prec, hipStream_t s);
// Right-hand sides in one launch.
enum { A_MAX_RHS = 16 };
// out = A in for nrhs fields in the canonical FP64 layout, one after the other
// in memory, rounded to prec on the way in and out: the values that
// import_spinor, apply_A and export_spinor give, in one pass.  Where
// apply_A_canonical_fits(g, prec); hipErrorInvalidValue otherwise.
bool apply_A_canonical_fits(const Geo &g, int prec);
hipError_t apply_A_canonical(const Geo &g, const double *in, double *out, int nrhs, const void *links, const void *clov,
                             int prec, hipStream_t s);

// What one visit of a domain reads and writes.
struct Visit {
    int first;      // first visit in this preconditioner call: residual is eta
    int faces_in;   // add the neighbours' boundary terms
    int last;       // last visit: write psi to the FP64 output
    int faces_out;  // write this domain's boundary terms
    int res_out;    // store the block residual
    int flip;       // additive schedule: which of the two boundary buffers is written
};

// Arguments of the block solves of one system (one lattice, one right-hand side).
struct SapArgs {
    Geo g;
    int n_mr;
    const double2 *eta; // FP64 input of the preconditioner
    double2 *out;       // FP64 output
    void *psi;          // solution accumulator (FP64, or FP32 for FP32/FP16 storage)
    void *res;          // block residual on even sites [d][12][Vd/2]
    float *res_scale;   // per-domain scale of res (FP16 storage)
    void *face;         // boundary half-spinors [d][8 faces][6][face sites]
    float *face_scale;  // per-domain scale of face (FP16 storage)
    void *face_alt;     // second boundary buffer (additive schedule), else null
    float *face_scale_alt;
    const void *face_in;          // set in the kernel: the buffer this visit reads
    const float *face_in_scale;
    const void *links;  // [d][mu][9 or 6][Vd]
    const void *cs;     // C_e on even / C_o^-1 on odd sites [d][36][Vd]
    void *rho_tmp;      // odd-site right-hand sides [d][12][Vd/2] when not kept in LDS
    int active;         // 0: skip this system (already converged)
    int io32;           // eta and out are FP32 (float2) vectors (FP32/FP16/BF16 block solves only)
};
bool sap_shape_supported(const int b[4]);
bool sap_prec_supported(const int b[4], int prec);
long sap_face_sites(const int b[4]);
int sap_shape_id(const int b[4]);
// The form (dd_form.h) of this lattice's block solves, given the caller's product;
// the functions below take it, or the launch's form, as their product.
int sap_lattice_form(const Geo &g, int prec, int product);
bool sap_product_supported(const int b[4], int prec, int product);
// Right-hand sides one workgroup takes (1, or 2 or 4 for the tile forms): the items
// of a tile launch are (first system | systems in the tile << 24, domain).
int sap_rhs_per_workgroup(int product);
// Domains one block-solve workgroup takes for (shape, precision, product): the
// items of a launch come in runs of this many domains of one system, and a run
// is never split or padded.
int sap_domains_per_workgroup(int shape, int prec, int product);
// The compiled domain shapes: ids 0 .. sap_shape_count() - 1 and their extents.
int sap_shape_count();
void sap_shape_extents(int shape, int b[4]);
// Work items of one system on the device: [0, nd/2) its black domains, then
// its white domains, each in increasing domain number (the order a plan of
// one system uses), with item.x = x.  items holds nd entries.
hipError_t sap_schedule_items(const Geo &g, int x, int2 *items, hipStream_t s);
// *dst = a on the device, in stream order (no host copy).
hipError_t sap_put_args(const SapArgs &a, SapArgs *dst, hipStream_t s);
// One colour of one half-sweep for a list of (system, domain) items; args and
// items are device arrays.  All systems share one domain shape (shape id).
hipError_t sap_sweep_batch(const SapArgs *args, const int2 *items, int nitems, int shape, int prec, int product,
                           Visit v, hipStream_t s);

// ---- FP64 linear algebra on flat complex vectors (double2) ---------------
struct Blas {
    double2 *partial = nullptr;   // [NBLK][32]
    double2 *result = nullptr;    // [32] pinned host memory, set while a solve runs
    double2 *coef = nullptr;      // [32] device: coefficients and scalars between kernels
};
enum { BLAS_NBLK = 1024, BLAS_MAXK = 16, BLAS_LIST = 16 };
// One system's operands of a launch over several: columns W (W_j = W + j*n),
// vectors w and r
struct BlasOp {
    const double2 *W;
    double2 *w, *r, *partial, *result, *coef;
    long n;
    int nblk;
};
struct BlasList {
    BlasOp op[BLAS_LIST];
};
BlasOp blas_op(const Blas &B, long n);   // W, w, r left empty
// result[j] = <W_j, v>, j < k (1 <= k <= 16); W_j = W + j*n
hipError_t multidot(Blas &B, const double2 *W, int k, double2 *v, long n, hipStream_t s);
// w -= sum_j coef[j] W_j (coef on device, k <= 16); result[0] = (|w|^2, 0), result[1] = <w, r>
hipError_t cgs_update(Blas &B, double2 *w, const double2 *W, int k, double2 *r, long n, hipStream_t s);
// A Gram-Schmidt pass of FGCR step k for each system (w: the new vector, W: the
// k before it, unnormalised, the norms of which earlier steps left in coef):
// result[STEP_DOTS + j] = <W_j, w>, j < nd (nd = k, or k + 1 with w itself last);
// w -= sum_j <W_j, w> / |W_j|^2 W_j; result[STEP_W] = (|w|^2, 0), result[STEP_W + 1]
// = <w, r>; then r -= <w, r> / |w|^2 w, result[STEP_R] = (|r|^2, 0), left out where
// may_repeat and |w|^2 is not more than a quarter of what it was, or w vanished.
enum { STEP_DOTS = 0, STEP_W = 16, STEP_R = 18 };
// end: takes the device's clock afterwards.
hipError_t fgcr_step(const std::vector<BlasOp> &ops, int k, int nd, bool may_repeat, unsigned long long *end, hipStream_t s);
hipError_t stamp(unsigned long long *t, hipStream_t s);   // *t (pinned host memory) = the device's clock
// x += sum_j coef[j] Z_j (coef on the host, 1 <= k <= 16)
hipError_t axpy_multi(double2 *x, const double2 *Z, const double2 *coef, int k, long n, hipStream_t s);
// r = b - r; result[0] = (|r|^2, 0); in a list, b is the operand w
hipError_t residual(Blas &B, double2 *b, double2 *r, long n, hipStream_t s);
hipError_t residual(const std::vector<BlasOp> &ops, hipStream_t s);
// result[0] = (|v|^2, 0); in a list, v is the operand w
hipError_t norm2(Blas &B, double2 *v, long n, hipStream_t s);
hipError_t norm2(const std::vector<BlasOp> &ops, hipStream_t s);
hipError_t zero(double2 *v, long n, hipStream_t s);
// FP32 vectors, FP64 accumulation: result[j] = <W_j, v> (k <= 16);
// w -= sum_j coef[j] W_j with result[0] = |w|^2; w *= inv_b with result[0] =
// <w, r>; r -= c w with result[0] = |r|^2; x (FP64) += scale sum_j coef[j] Z_j;
// out = sc * in rounded to FP32
hipError_t multidot32(Blas &B, const float2 *W, long ldw, int k, const float2 *v, long n, hipStream_t s);
hipError_t cgs_update32(Blas &B, float2 *w, const float2 *W, long ldw, int k, long n, hipStream_t s);
hipError_t scale_dot32(Blas &B, float2 *w, double inv_b, const float2 *r, long n, hipStream_t s);
hipError_t axpy32(Blas &B, float2 *r, double2 c, const float2 *w, long n, hipStream_t s);
hipError_t axpy_mixed(Blas &B, double2 *x, const float2 *Z, long ldz, int k, double scale, long n, hipStream_t s);
hipError_t to_f32(const double2 *in, double sc, float2 *out, long n, hipStream_t s);
// out_q = sum_i W_i P[i][q], q < nq, i < nin (<= 24 each; P row-major on the
// device; out must not overlap W)
hipError_t recombine(const double2 *W, long ldw, int nin, const double2 *P, int nq, double2 *out, long ldo, long n,
                     hipStream_t s);
// BiCGstab on the device's own scalars: rho = <r0, r> at a (re)start, where p and
// v are zero (result[BICG_RHO]); p = r + beta (p - omega v); with v = A p, alpha =
// rho / <r0, v> (result[BICG_STOP].x not 0: not finite) and s = r - alpha v; with t
// = A s, omega (result[BICG_OMEGA]), x += alpha p + omega s and r = s - omega t
// unless stopped, |r|^2 (result[BICG_RR]) and the next rho
struct BicgVectors {
    double2 *x, *r, *r0, *p, *v, *s, *t;
};
enum { BICG_R0V = 0, BICG_STOP = 1, BICG_TS = 2, BICG_OMEGA = 4, BICG_RR = 5, BICG_RHO = 6 };
hipError_t bicg_start(Blas &B, const BicgVectors &V, long n, hipStream_t s);
hipError_t bicg_direction(Blas &B, const BicgVectors &V, long n, hipStream_t s);
hipError_t bicg_half(Blas &B, const BicgVectors &V, long n, hipStream_t s);
hipError_t bicg_update(Blas &B, const BicgVectors &V, long n, hipStream_t s);
// out = ca a + cb b + cc c; c may be null; out may alias an input
hipError_t lincomb(double2 *out, const double2 *a, double2 ca, const double2 *b, double2 cb, const double2 *c,
                   double2 cc, long n, hipStream_t s);

}  // namespace dd
