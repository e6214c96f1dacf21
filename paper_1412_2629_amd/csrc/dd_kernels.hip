// Layout conversion, clover set-up, the global operator A and the FP64
// linear algebra of the outer solver.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "dd_device.h"
#include "dd_internal.h"

namespace dd {

static inline unsigned nblocks(long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// ===========================================================================
// layout conversion
// ===========================================================================

__device__ __forceinline__ long canon_index(const Geo &g, const int x[4])
{
    return x[0] + (long)g.L[0] * (x[1] + (long)g.L[1] * (x[2] + (long)g.L[2] * x[3]));
}

template <typename S> __global__ void k_import_spinor(Geo g, const double2 *canon, v2<S> *out)
{
    long I = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (I >= g.V) return;
    int x[4], d, loc;
    decode(g, I, x, d, loc);
    long c = canon_index(g, x) * 12;
#pragma unroll
    for (int k = 0; k < 12; k++) st<double, S>(out, ((long)d * 12 + k) * g.Vd + loc, ld<double, double>(canon, c + k));
}

template <typename S> __global__ void k_export_spinor(Geo g, const v2<S> *in, double2 *canon)
{
    long I = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (I >= g.V) return;
    int x[4], d, loc;
    decode(g, I, x, d, loc);
    long c = canon_index(g, x) * 12;
#pragma unroll
    for (int k = 0; k < 12; k++) st<double, double>(canon, c + k, ld<double, S>(in, ((long)d * 12 + k) * g.Vd + loc));
}

// The same conversions through LDS, one workgroup per domain of VD sites
// (VD threads): the canonical side is moved as the domain's x-runs (b0 sites
// x 12 components, contiguous in memory), consecutive threads on consecutive
// 16-byte entries; the internal side one component at a time, consecutive
// threads on consecutive sites.  buf holds the domain as [local lexicographic
// site][12].
__device__ __forceinline__ long dom_run_base(const Geo &g, int d, int j)
{
    // canonical index of the first site of x-run j (= (ly, lz, lt)) of domain d
    int r = d, x[4];
    x[0] = (r % g.n[0]) * g.b[0]; r /= g.n[0];
    x[1] = (r % g.n[1]) * g.b[1]; r /= g.n[1];
    x[2] = (r % g.n[2]) * g.b[2];
    x[3] = (r / g.n[2]) * g.b[3];
    x[1] += j % g.b[1]; j /= g.b[1];
    x[2] += j % g.b[2];
    x[3] += j / g.b[2];
    return canon_index(g, x);
}

__device__ __forceinline__ int local_lex(const Geo &g, const int x[4])
{
    return x[0] % g.b[0] + g.b[0] * (x[1] % g.b[1] + g.b[1] * (x[2] % g.b[2] + g.b[2] * (x[3] % g.b[3])));
}

template <int VD, typename S> __global__ __launch_bounds__(VD) void k_import_dom(Geo g, const double2 *canon, v2<S> *out)
{
    __shared__ double2 buf[12 * VD];
    const int d = blockIdx.x, t = threadIdx.x;
    const int runlen = g.b[0] * 12;
    for (int e = t; e < 12 * VD; e += VD) {
        const int j = e / runlen, o = e - j * runlen;
        buf[e] = canon[dom_run_base(g, d, j) * 12 + o];
    }
    __syncthreads();
    int x[4], dd, loc;
    decode(g, (long)d * VD + t, x, dd, loc);
    const int ll = local_lex(g, x);
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const double2 v = buf[ll * 12 + k];
        st<double, S>(out, ((long)d * 12 + k) * VD + t, cx<double>{v.x, v.y});
    }
}

template <int VD, typename S> __global__ __launch_bounds__(VD) void k_export_dom(Geo g, const v2<S> *in, double2 *canon)
{
    __shared__ double2 buf[12 * VD];
    const int d = blockIdx.x, t = threadIdx.x;
    int x[4], dd, loc;
    decode(g, (long)d * VD + t, x, dd, loc);
    const int ll = local_lex(g, x);
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const cx<double> v = ld<double, S>(in, ((long)d * 12 + k) * VD + t);
        buf[ll * 12 + k] = make_double2(v.r, v.i);
    }
    __syncthreads();
    const int runlen = g.b[0] * 12;
    for (int e = t; e < 12 * VD; e += VD) {
        const int j = e / runlen, o = e - j * runlen;
        canon[dom_run_base(g, d, j) * 12 + o] = buf[e];
    }
}

template <int VD>
static void launch_convert_dom(const Geo &g, const double *canon, void *internal, int prec, bool import,
                               hipStream_t s)
{
    const unsigned nb = (unsigned)g.nd;
    if (import) {
        const double2 *c = (const double2 *)canon;
        if (prec == P64) hipLaunchKernelGGL((k_import_dom<VD, double>), nb, VD, 0, s, g, c, (double2 *)internal);
        else if (prec == P32) hipLaunchKernelGGL((k_import_dom<VD, float>), nb, VD, 0, s, g, c, (float2 *)internal);
        else if (prec == P16) hipLaunchKernelGGL((k_import_dom<VD, half_t>), nb, VD, 0, s, g, c, (half2_t *)internal);
        else hipLaunchKernelGGL((k_import_dom<VD, bf16_t>), nb, VD, 0, s, g, c, (bf162_t *)internal);
    } else {
        double2 *c = (double2 *)canon;
        if (prec == P64) hipLaunchKernelGGL((k_export_dom<VD, double>), nb, VD, 0, s, g, (const double2 *)internal, c);
        else if (prec == P32) hipLaunchKernelGGL((k_export_dom<VD, float>), nb, VD, 0, s, g, (const float2 *)internal, c);
        else if (prec == P16) hipLaunchKernelGGL((k_export_dom<VD, half_t>), nb, VD, 0, s, g, (const half2_t *)internal, c);
        else hipLaunchKernelGGL((k_export_dom<VD, bf16_t>), nb, VD, 0, s, g, (const bf162_t *)internal, c);
    }
}

// domains of 256 or 512 sites through LDS, others one thread per site
static bool convert_dom(const Geo &g, const double *canon, void *internal, int prec, bool import, hipStream_t s)
{
    if (g.Vd == 256) launch_convert_dom<256>(g, canon, internal, prec, import, s);
    else if (g.Vd == 512) launch_convert_dom<512>(g, canon, internal, prec, import, s);
    else return false;
    return true;
}

hipError_t import_spinor(const Geo &g, const double *canon, void *internal, int prec, hipStream_t s)
{
    if (convert_dom(g, canon, internal, prec, true, s)) return hipGetLastError();
    unsigned nb = nblocks(g.V, 256);
    if (prec == P64) hipLaunchKernelGGL(k_import_spinor<double>, nb, 256, 0, s, g, (const double2 *)canon, (double2 *)internal);
    else if (prec == P32) hipLaunchKernelGGL(k_import_spinor<float>, nb, 256, 0, s, g, (const double2 *)canon, (float2 *)internal);
    else if (prec == P16) hipLaunchKernelGGL(k_import_spinor<half_t>, nb, 256, 0, s, g, (const double2 *)canon, (half2_t *)internal);
    else hipLaunchKernelGGL(k_import_spinor<bf16_t>, nb, 256, 0, s, g, (const double2 *)canon, (bf162_t *)internal);
    return hipGetLastError();
}

hipError_t export_spinor(const Geo &g, const void *internal, int prec, double *canon, hipStream_t s)
{
    if (convert_dom(g, canon, const_cast<void *>(internal), prec, false, s)) return hipGetLastError();
    unsigned nb = nblocks(g.V, 256);
    if (prec == P64) hipLaunchKernelGGL(k_export_spinor<double>, nb, 256, 0, s, g, (const double2 *)internal, (double2 *)canon);
    else if (prec == P32) hipLaunchKernelGGL(k_export_spinor<float>, nb, 256, 0, s, g, (const float2 *)internal, (double2 *)canon);
    else if (prec == P16) hipLaunchKernelGGL(k_export_spinor<half_t>, nb, 256, 0, s, g, (const half2_t *)internal, (double2 *)canon);
    else hipLaunchKernelGGL(k_export_spinor<bf16_t>, nb, 256, 0, s, g, (const bf162_t *)internal, (double2 *)canon);
    return hipGetLastError();
}

__global__ void k_import_gauge(Geo g, const double2 *canon, double2 *U)
{
    long I = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (I >= g.V) return;
    int x[4], d, loc;
    decode(g, I, x, d, loc);
    long c = canon_index(g, x) * 36;
    for (int mu = 0; mu < 4; mu++)
#pragma unroll
        for (int e = 0; e < 9; e++) U[(((long)d * 4 + mu) * 9 + e) * g.Vd + loc] = canon[c + mu * 9 + e];
}

hipError_t import_gauge(const Geo &g, const double *canon, double2 *U64, hipStream_t s)
{
    hipLaunchKernelGGL(k_import_gauge, nblocks(g.V, 256), 256, 0, s, g, (const double2 *)canon, U64);
    return hipGetLastError();
}

template <typename S> __global__ void k_compress_links(Geo g, const double2 *U, v2<S> *out)
{
    long I = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (I >= g.V) return;
    int d = (int)(I / g.Vd), loc = (int)(I - (long)d * g.Vd);
    for (int mu = 0; mu < 4; mu++)
#pragma unroll
        for (int e = 0; e < 6; e++)
            st<double, S>(out, (((long)d * 4 + mu) * 6 + e) * g.Vd + loc,
                          ld<double, double>(U, (((long)d * 4 + mu) * 9 + e) * g.Vd + loc));
}

hipError_t compress_links(const Geo &g, const double2 *U64, void *out, int prec, hipStream_t s)
{
    unsigned nb = nblocks(g.V, 256);
    if (prec == P32) hipLaunchKernelGGL(k_compress_links<float>, nb, 256, 0, s, g, U64, (float2 *)out);
    else if (prec == P16) hipLaunchKernelGGL(k_compress_links<half_t>, nb, 256, 0, s, g, U64, (half2_t *)out);
    else hipLaunchKernelGGL(k_compress_links<bf16_t>, nb, 256, 0, s, g, U64, (bf162_t *)out);
    return hipGetLastError();
}

template <typename S> __global__ void k_convert_pairs(const double2 *in, v2<S> *out, long n)
{
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) st<double, S>(out, i, ld<double, double>(in, i));
}

hipError_t convert_pairs(const double2 *in, void *out, long n, int prec, hipStream_t s)
{
    unsigned nb = nblocks(n, 256);
    if (prec == P32) hipLaunchKernelGGL(k_convert_pairs<float>, nb, 256, 0, s, in, (float2 *)out, n);
    else if (prec == P16) hipLaunchKernelGGL(k_convert_pairs<half_t>, nb, 256, 0, s, in, (half2_t *)out, n);
    else hipLaunchKernelGGL(k_convert_pairs<bf16_t>, nb, 256, 0, s, in, (bf162_t *)out, n);
    return hipGetLastError();
}

__global__ void k_count_nonfinite(const double2 *v, long n, int *cnt)
{
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    int bad = 0;
    for (; i < n; i += (long)gridDim.x * blockDim.x) bad |= !isfinite(v[i].x) || !isfinite(v[i].y);
    if (bad) atomicOr(cnt, 1);
}

hipError_t count_nonfinite(const double2 *v, long n, int *cnt, hipStream_t s)
{
    hipLaunchKernelGGL(k_count_nonfinite, 1024, 256, 0, s, v, n, cnt);
    return hipGetLastError();
}

// ===========================================================================
// clover term (Sec. II-B, Eq. 3) and its odd-site inverse (Sec. II-D, Eq. 5)
// ===========================================================================

struct m3 {
    cx<double> e[9];
};

// the links of site x begin here in U
__device__ __forceinline__ long links_at(const Geo &g, const int x[4])
{
    const long J = encode(g, x);
    const int d = (int)(J / g.Vd);
    return (long)d * 36 * g.Vd + (J - (long)d * g.Vd);
}

__device__ __forceinline__ m3 m3_load(const Geo &g, const double2 *U, long site, int mu)
{
    m3 r;
#pragma unroll
    for (int e = 0; e < 9; e++) r.e[e] = ld<double, double>(U, site + (long)(mu * 9 + e) * g.Vd);
    return r;
}

// a * b with optional daggers
__device__ __forceinline__ m3 m3_mul(const m3 &a, bool da, const m3 &b, bool db)
{
    m3 r;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            cx<double> s = czero<double>();
#pragma unroll
            for (int k = 0; k < 3; k++) {
                cx<double> av = da ? cx<double>{a.e[k * 3 + i].r, -a.e[k * 3 + i].i} : a.e[i * 3 + k];
                cx<double> bv = db ? cx<double>{b.e[j * 3 + k].r, -b.e[j * 3 + k].i} : b.e[k * 3 + j];
                s = s + av * bv;
            }
            r.e[i * 3 + j] = s;
        }
    return r;
}

__device__ __forceinline__ void shift(const Geo &g, const int x[4], int mu, int step, int y[4])
{
#pragma unroll
    for (int m = 0; m < 4; m++) {   // (mu is uniform in a wave, the arrays stay in registers)
        y[m] = m == mu ? x[m] + step : x[m];
        if (y[m] >= g.L[m]) y[m] -= g.L[m];
        if (y[m] < 0) y[m] += g.L[m];
    }
}

// A link (site, direction) that enters a leaf as itself or as its adjoint.
struct LeafLink {
    long site;
    int mu;
    bool dag;
};
// Product of four links.  U is made to depend on what has been formed, so that
// no more than two links' matrices are in registers ahead of their product.
__device__ __forceinline__ m3 leaf(const Geo &g, const double2 *&U, LeafLink a, LeafLink b, LeafLink c, LeafLink d)
{
    m3 t = m3_mul(m3_load(g, U, a.site, a.mu), a.dag, m3_load(g, U, b.site, b.mu), b.dag);
    asm volatile("" : "+s"(U) : "v"(t.e[0].r), "v"(t.e[4].r), "v"(t.e[8].i));
    t = m3_mul(t, false, m3_load(g, U, c.site, c.mu), c.dag);
    t = m3_mul(t, false, m3_load(g, U, d.site, d.mu), d.dag);
    asm volatile("" : "+s"(U) : "v"(t.e[0].r), "v"(t.e[4].r), "v"(t.e[8].i));
    return t;
}

// Q_munu = sum of the four leaves at x oriented mu -> nu
__device__ __forceinline__ m3 clover_leaves(const Geo &g, const double2 *U, const int x[4], int mu, int nu)
{
    auto at = [&](int m, int step_m, int n, int step_n) {   // links of x + step_m m + step_n n
        int y[4], z[4];
        shift(g, x, m, step_m, y);
        shift(g, y, n, step_n, z);
        return links_at(g, z);
    };
    const long o = links_at(g, x), xpm = at(mu, +1, nu, 0), xmm = at(mu, -1, nu, 0), xpn = at(mu, 0, nu, +1),
               xmn = at(mu, 0, nu, -1), a = at(mu, -1, nu, +1), b = at(mu, -1, nu, -1), c = at(mu, +1, nu, -1);
    // U_mu(x) U_nu(x+mu) U_mu(x+nu)^+ U_nu(x)^+
    m3 Q = leaf(g, U, {o, mu, false}, {xpm, nu, false}, {xpn, mu, true}, {o, nu, true}), t;
    auto add = [&] {
#pragma unroll
        for (int e = 0; e < 9; e++) Q.e[e] = Q.e[e] + t.e[e];
    };
    // U_nu(x) U_mu(x+nu-mu)^+ U_nu(x-mu)^+ U_mu(x-mu)
    t = leaf(g, U, {o, nu, false}, {a, mu, true}, {xmm, nu, true}, {xmm, mu, false});
    add();
    // U_mu(x-mu)^+ U_nu(x-mu-nu)^+ U_mu(x-mu-nu) U_nu(x-nu)
    t = leaf(g, U, {xmm, mu, true}, {b, nu, true}, {b, mu, false}, {xmn, nu, false});
    add();
    // U_nu(x-nu)^+ U_mu(x-nu) U_nu(x-nu+mu) U_mu(x)^+
    t = leaf(g, U, {xmn, nu, true}, {xmn, mu, false}, {c, nu, false}, {o, mu, true});
    add();
    return Q;
}

// In the chiral basis sigma_jk = -eps_jkl diag(s_l, s_l) (j,k spatial) and
// sigma_kt = diag(-s_k, s_k), so with E_l the colour matrices multiplying
// s_l, each chiral block of D_cl is [[E3, E1 - i E2], [E1 + i E2, -E3]] with
//   upper: E1 = -(i c/2)(F_yz + F_xt), E2 = (i c/2)(F_xz - F_yt), E3 = -(i c/2)(F_xy + F_zt)
//   lower: E1 = -(i c/2)(F_yz - F_xt), E2 = (i c/2)(F_xz + F_yt), E3 = -(i c/2)(F_xy - F_zt)
//
// A workgroup takes 64 consecutive sites: wave p forms F_munu = (Q - Q^dag) / 8
// of plane p for all of them in registers and leaves it in LDS; then wave w
// forms and stores entries 6w .. 6w + 5 of the 36 packed pairs.  With all six F of
// a site in one thread the matrices went to scratch (7.7 kB a thread): 16^3x32
// 0.78 ms, 32^3x64 11.1 ms; now 0.18 and 2.96 ms.  Bound by the links' way through the
// caches: each is read some hundred times.
constexpr int CLOVER_SITES = 64;
__global__ __launch_bounds__(6 * CLOVER_SITES) void k_clover_build(Geo g, const double2 *U, double kappa, double csw, double2 *C)
{
    __shared__ cx<double> F[6][9][CLOVER_SITES];   // planes xy, xz, xt, yz, yt, zt
    const int lane = threadIdx.x % CLOVER_SITES, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / CLOVER_SITES);
    const long I = (long)blockIdx.x * CLOVER_SITES + lane;   // V is a multiple of 64
    int x[4], d, loc;
    decode(g, I, x, d, loc);
    {
        const m3 Q = clover_leaves(g, U, x, w < 3 ? 0 : w < 5 ? 1 : 2, w < 3 ? w + 1 : w < 5 ? w - 1 : 3);
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++)
                F[w][i * 3 + j][lane] = scal(0.125, Q.e[i * 3 + j] - cx<double>{Q.e[j * 3 + i].r, -Q.e[j * 3 + i].i});
    }
    __syncthreads();
    // entry (I, J), I >= J, of block blk: colour e, spins I / 3 and J / 3
    auto entry = [&](int blk, int row, int col) {
        const double sg = blk == 0 ? 1.0 : -1.0;
        const int e = row % 3 * 3 + col % 3;
        // -(i c/2) X = (c/2) (X.i, -X.r)
        if (row / 3 == col / 3) {
            const cx<double> s3 = F[0][e][lane] + scal(sg, F[5][e][lane]);
            const cx<double> E3 = scal(0.5 * csw, cx<double>{s3.i, -s3.r});
            return row < 3 ? E3 : neg(E3);
        }
        const cx<double> s1 = F[3][e][lane] + scal(sg, F[2][e][lane]), s2 = F[1][e][lane] - scal(sg, F[4][e][lane]);
        const cx<double> E1 = scal(0.5 * csw, cx<double>{s1.i, -s1.r}), E2 = scal(0.5 * csw, cx<double>{-s2.i, s2.r});
        return E1 + times_i(E2);
    };
    const double diag = 1.0 / (2.0 * kappa);
    const long base = (long)d * 36 * g.Vd + loc;
    for (int k = 0; k < 6; k++) {
        const int n = 6 * w + k, blk = n / 18, q = n % 18;
        double2 v;
        if (q < 3) {
            v = make_double2(entry(blk, 2 * q, 2 * q).r + diag, entry(blk, 2 * q + 1, 2 * q + 1).r + diag);
        } else {
            int row = 1;
            while (tri_index(row + 1, 0) <= q - 3) row++;
            const cx<double> m = entry(blk, row, q - 3 - tri_index(row, 0));
            v = make_double2(m.r, m.i);
        }
        C[base + (long)n * g.Vd] = v;
    }
}

hipError_t clover_build(const Geo &g, const double2 *U64, double kappa, double csw, double2 *C64, hipStream_t s)
{
    if (g.V % CLOVER_SITES) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_clover_build, (unsigned)(g.V / CLOVER_SITES), 6 * CLOVER_SITES, 0, s, g, U64, kappa, csw, C64);
    return hipGetLastError();
}

// one thread per (site, chiral block): copy on even sites, inverse on odd sites
// by Gauss-Jordan elimination in place with partial pivoting.  Every index is
// known at compile time (rows are exchanged by selection), so the matrix stays in
// registers; with 6 x 12 augmented rows in scratch 16^3x32 took 0.70 ms, 32^3x64
// 11.0 ms; now 0.039 and 0.48 ms, bound by memory (1152 bytes a site).
__global__ __launch_bounds__(128) void k_clover_schur(Geo g, const double2 *C, double2 *Cs, int *bad)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2 * g.V) return;
    const int blk = t >= g.V;
    const long I = t - blk * g.V;
    const int d = (int)(I / g.Vd), loc = (int)(I - (long)d * g.Vd);
    const long base = ((long)d * 36 + blk * 18) * g.Vd + loc;
    double2 in[18];
#pragma unroll
    for (int q = 0; q < 18; q++) in[q] = C[base + q * g.Vd];
    if (loc < g.Vh) {
#pragma unroll
        for (int q = 0; q < 18; q++) Cs[base + q * g.Vd] = in[q];
        return;
    }
    cx<double> M[6][6];
#pragma unroll
    for (int q = 0; q < 3; q++) {
        M[2 * q][2 * q] = {in[q].x, 0};
        M[2 * q + 1][2 * q + 1] = {in[q].y, 0};
    }
#pragma unroll
    for (int i = 1; i < 6; i++)
#pragma unroll
        for (int j = 0; j < i; j++) {
            const double2 v = in[3 + tri_index(i, j)];
            M[i][j] = {v.x, v.y};
            M[j][i] = {v.x, -v.y};
        }
    int piv[6];   // the row exchanged with row c
#pragma unroll
    for (int c = 0; c < 6; c++) {
        int p = c;
        double best = M[c][c].r * M[c][c].r + M[c][c].i * M[c][c].i;
#pragma unroll
        for (int r = c + 1; r < 6; r++) {
            const double v = M[r][c].r * M[r][c].r + M[r][c].i * M[r][c].i;
            if (v > best) { best = v; p = r; }
        }
        if (!(best > 0)) { atomicOr(bad, 1); return; }
        piv[c] = p;
#pragma unroll
        for (int r = c + 1; r < 6; r++) {
            if (p != r) continue;
#pragma unroll
            for (int j = 0; j < 6; j++) { const cx<double> tmp = M[c][j]; M[c][j] = M[r][j]; M[r][j] = tmp; }
        }
        const double inv = 1.0 / best;
        const cx<double> ip = {M[c][c].r * inv, -M[c][c].i * inv};
#pragma unroll
        for (int j = 0; j < 6; j++) M[c][j] = j == c ? ip : M[c][j] * ip;
#pragma unroll
        for (int r = 0; r < 6; r++) {
            if (r == c) continue;
            const cx<double> f = M[r][c];
#pragma unroll
            for (int j = 0; j < 6; j++) M[r][j] = j == c ? neg(f * ip) : M[r][j] - f * M[c][j];
        }
    }
    // (P A)^-1 = A^-1 P^-1: the row exchanges, last first, on the columns
#pragma unroll
    for (int c = 5; c >= 0; c--)
#pragma unroll
        for (int r = c + 1; r < 6; r++) {
            if (piv[c] != r) continue;
#pragma unroll
            for (int i = 0; i < 6; i++) { const cx<double> tmp = M[i][c]; M[i][c] = M[i][r]; M[i][r] = tmp; }
        }
#pragma unroll
    for (int q = 0; q < 3; q++) Cs[base + q * g.Vd] = make_double2(M[2 * q][2 * q].r, M[2 * q + 1][2 * q + 1].r);
#pragma unroll
    for (int i = 1; i < 6; i++)
#pragma unroll
        for (int j = 0; j < i; j++)
            // Hermitian inverse: average the two triangles to remove rounding asymmetry
            Cs[base + (3 + tri_index(i, j)) * g.Vd] =
                make_double2(0.5 * (M[i][j].r + M[j][i].r), 0.5 * (M[i][j].i - M[j][i].i));
}

hipError_t clover_schur(const Geo &g, const double2 *C64, double2 *Cs64, int *bad, hipStream_t s)
{
    hipLaunchKernelGGL(k_clover_schur, nblocks(2 * g.V, 128), 128, 0, s, g, C64, Cs64, bad);
    return hipGetLastError();
}

// ===========================================================================
// global operator A (Sec. II-B, Eqs. 1-2): one thread per site
// ===========================================================================

// The spinor of site y (internal position (dj, lj)) from the input field
template <typename T, typename SI, bool CANON>
__device__ __forceinline__ void a_load(const Geo &g, const v2<std::conditional_t<CANON, double, SI>> *in, const int y[4],
                                       unsigned dj, unsigned lj, cx<T> v[12])
{
    if constexpr (CANON) {
        const unsigned b = (unsigned)canon_index(g, y) * 12;
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const cx<double> c = ld32<double, double>(in, b + k);
            v[k] = {static_cast<T>(static_cast<SI>(c.r)), static_cast<T>(static_cast<SI>(c.i))};
        }
    } else {
#pragma unroll
        for (int k = 0; k < 12; k++) v[k] = ld32<T, SI>(in, (dj * 12 + k) * (unsigned)g.Vd + lj);
    }
}

// The right-hand sides of a launch in storage S.  16-bit operands come one at a time,
// and their list is known to hold one when the kernel is compiled (with a list of 16
// a call took half a microsecond longer: FP16 on 8^4 29.7 us, now 29.1).
template <typename S> struct RhsFields {
    enum { MAX = sizeof(S) == 2 ? 1 : A_MAX_RHS };
    const void *in[MAX];
    void *out[MAX];
    int n;
};
// Block and right-hand side of this workgroup.  Workgroup w runs on XCD w mod 8.
// Each XCD sweeps one contiguous eighth of the domain-blocked site order: most
// neighbour spinors and links a workgroup reads were brought into the same
// XCD's L2 by its neighbours (a plain order spreads neighbouring blocks over
// all eight L2s).  The right-hand sides of a block follow one another there, so
// its links and clover blocks come from memory once for all of them.
template <typename S> __device__ __forceinline__ void rhs_block(const RhsFields<S> &io, unsigned &blk, unsigned &rhs)
{
    const unsigned nr = RhsFields<S>::MAX == 1 ? 1 : (unsigned)io.n, nbk = gridDim.x / nr, w = blockIdx.x;
    if (nbk % 8 == 0) {
        const unsigned q = w / 8;
        rhs = q % nr;
        blk = (w % 8) * (nbk / 8) + q / nr;
    } else {
        rhs = w % nr;
        blk = w / nr;
    }
}

// one hop: DIR = +1 forward, -1 backward (CANON: in is the canonical FP64 field)
template <int MU, int DIR, typename T, typename SI, typename G, int NLC, bool CANON>
__device__ __forceinline__ void a_hop(const Geo &g, const int x[4], int d, int loc,
                                      const v2<std::conditional_t<CANON, double, SI>> *in, const v2<G> *links, cx<T> acc[12])
{
    const long Vd = g.Vd;
    int y[4] = {x[0], x[1], x[2], x[3]};
    bool wrap = false;
    if constexpr (DIR > 0) {
        y[MU] = x[MU] + 1;
        if (y[MU] == g.L[MU]) { y[MU] = 0; wrap = true; }
    } else {
        y[MU] = x[MU] - 1;
        if (y[MU] < 0) { y[MU] = g.L[MU] - 1; wrap = true; }
    }
    const long J = encode(g, y);
    const int dj = (int)(J / Vd), lj = (int)(J - (long)dj * Vd);
    cx<T> v[12], h[6], uh[6];
    if constexpr (CANON) a_load<T, SI, CANON>(g, in, y, dj, lj, v);
    else
#pragma unroll
        for (int k = 0; k < 12; k++) v[k] = ld<T, SI>(in, ((long)dj * 12 + k) * Vd + lj);
    if constexpr (DIR > 0) {
        // -1/2 (1 - gamma_mu) U_mu(x) psi(x + mu)
        proj<MU, -1>(v, h);
        su3<T> U = ld_link<T, G, NLC>(links, ((long)d * 4 + MU) * NLC * Vd + loc, Vd);
        su3_mul(U, h, uh);
        recon_acc<MU, -1>(acc, uh, T(wrap ? -0.5 * g.bc[MU] : -0.5));
    } else {
        // -1/2 (1 + gamma_mu) U_mu(x - mu)^dagger psi(x - mu)
        proj<MU, +1>(v, h);
        su3<T> U = ld_link<T, G, NLC>(links, ((long)dj * 4 + MU) * NLC * Vd + lj, Vd);
        su3_dag_mul(U, h, uh);
        recon_acc<MU, +1>(acc, uh, T(wrap ? -0.5 * g.bc[MU] : -0.5));
    }
}

// One thread per site; CANON: in the canonical FP64 fields of the interface.
template <typename T, typename SI, typename SO, typename G, int NLC, bool CANON>
__global__ __launch_bounds__(256) void k_apply_A(Geo g, RhsFields<SI> io, const v2<G> *links, const v2<G> *clov)
{
    typedef std::conditional_t<CANON, double, SI> FI;
    typedef std::conditional_t<CANON, double, SO> FO;
    unsigned blk, rhs;
    rhs_block(io, blk, rhs);
    long I = (long)blk * blockDim.x + threadIdx.x;
    if (I >= g.V) return;
    const v2<FI> *in = global_ptr((const v2<FI> *)io.in[rhs]);
    v2<FO> *out = global_ptr((v2<FO> *)io.out[rhs]);
    int x[4], d, loc;
    decode(g, I, x, d, loc);
    const long Vd = g.Vd;
    cx<T> acc[12];
    {
        cx<T> s[12];
        if constexpr (CANON) a_load<T, SI, CANON>(g, in, x, d, loc, s);
        else
#pragma unroll
            for (int k = 0; k < 12; k++) s[k] = ld<T, SI>(in, ((long)d * 12 + k) * Vd + loc);
        clover_apply<T, G>(clov, (long)d * 36 * Vd + loc, Vd, s, acc);
    }
    // The eight hops one after another (a loop the compiler keeps rolled): only
    // one neighbour's spinor and link are live at a time.  Unrolled, the
    // compiler issues every load of the site up front, which needs several
    // hundred registers and spills to scratch.
#pragma unroll 1
    for (int k = 0; k < 8; k++) {
        switch (k) {
            case 0: a_hop<0, +1, T, SI, G, NLC, CANON>(g, x, d, loc, in, links, acc); break;
            case 1: a_hop<0, -1, T, SI, G, NLC, CANON>(g, x, d, loc, in, links, acc); break;
            case 2: a_hop<1, +1, T, SI, G, NLC, CANON>(g, x, d, loc, in, links, acc); break;
            case 3: a_hop<1, -1, T, SI, G, NLC, CANON>(g, x, d, loc, in, links, acc); break;
            case 4: a_hop<2, +1, T, SI, G, NLC, CANON>(g, x, d, loc, in, links, acc); break;
            case 5: a_hop<2, -1, T, SI, G, NLC, CANON>(g, x, d, loc, in, links, acc); break;
            case 6: a_hop<3, +1, T, SI, G, NLC, CANON>(g, x, d, loc, in, links, acc); break;
            default: a_hop<3, -1, T, SI, G, NLC, CANON>(g, x, d, loc, in, links, acc); break;
        }
    }
    if constexpr (CANON) {
        const unsigned b = (unsigned)canon_index(g, x) * 12;
#pragma unroll
        for (int k = 0; k < 12; k++)
            st32<double, double>(out, b + k, cx<double>{static_cast<double>(static_cast<SO>(acc[k].r)),
                                                        static_cast<double>(static_cast<SO>(acc[k].i))});
    } else {
#pragma unroll
        for (int k = 0; k < 12; k++) st<T, SO>(out, ((long)d * 12 + k) * Vd + loc, acc[k]);
    }
}

// A on whole domains: a workgroup takes NT consecutive sites of the
// domain-blocked order (NT / Vd whole domains), one thread per site.  The
// workgroup's input spinors are staged in LDS, and each site pushes its
// backward term U_mu(x)^+ (1 + gamma_mu) psi(x) to the site x + mu through LDS,
// so inside a domain every link and spinor is read from memory once (by its
// own site); only hops that leave the domain read a neighbour domain's spinor
// (and, backwards, its link).  The hops are summed in the order of k_apply_A
// (per direction: forward, then backward) with the same products, so both
// kernels give the same bits.  Field offsets are 32-bit byte offsets (the host
// checks that every field is under 4 GiB), which keeps an address in one VGPR.
//
// CANON: in and out are the canonical FP64 fields of the interface (SI, SO the
// precision in which the operator takes and returns its values): the domain's
// spinors go from and to memory through LDS as its x-runs (contiguous there),
// a neighbour domain's spinor is 192 contiguous bytes, and no separate layout
// conversions are needed.
//
// Bound by memory.  FP64 on 32^3x64 with 4^4 domains, per right-hand side: in
// canonical fields 786 us alone, 552 us when three share a launch (their
// workgroups follow one another on one XCD, and the links and clover blocks
// come from its L2: 960 + 192 bytes a site instead of 1536); a layout conversion
// each way and one launch per right-hand side take 1059 us.

// Spinors in LDS: [12][NT + 1]; the odd stride keeps the twelve components of
// one site, which consecutive lanes move to and from canonical memory, in
// different banks.
template <int MU, int NT, typename T, typename SI, typename G, int NLC, bool CANON>
__device__ __forceinline__ void a_dom_dir(const Geo &g, const int x[4], int d, int loc, int ts,
                                          const v2<std::conditional_t<CANON, double, SI>> *in, const v2<G> *links,
                                          cx<T> (*sp)[NT + 1], cx<T> (*ex)[NT], cx<T> acc[12])
{
    const unsigned Vd = (unsigned)g.Vd;
    const int base = ts - loc;                // first site of this site's domain in the workgroup
    const int lx = x[MU] % g.b[MU];           // coordinate inside the domain
    cx<T> h[6], uh[6];
    {
        const unsigned lb = ((unsigned)d * 4 + MU) * NLC * Vd + loc;
        const su3<T> U = ld_link_with<T, NLC>([&](int e) { return ld32<T, G>(links, lb + e * Vd); });
        // forward: -1/2 (1 - gamma_mu) U_mu(x) psi(x + mu)
        {
            cx<T> v[12];
            int y[4] = {x[0], x[1], x[2], x[3]};
            bool wrap = false;
            y[MU] = x[MU] + 1;
            if (lx + 1 < g.b[MU]) {
                const int lj = (int)(encode(g, y) - (long)d * Vd);
#pragma unroll
                for (int k = 0; k < 12; k++) v[k] = sp[k][base + lj];
            } else {
                if (y[MU] == g.L[MU]) { y[MU] = 0; wrap = true; }
                const long J = encode(g, y);
                const unsigned dj = (unsigned)(J / Vd), lj = (unsigned)(J - (long)dj * Vd);
                a_load<T, SI, CANON>(g, in, y, dj, lj, v);
            }
            proj<MU, -1>(v, h);
            su3_mul(U, h, uh);
            recon_acc<MU, -1>(acc, uh, T(wrap ? -0.5 * g.bc[MU] : -0.5));
        }
        // push U_mu(x)^+ (1 + gamma_mu) psi(x) for the site x + mu
        {
            cx<T> v[12];
#pragma unroll
            for (int k = 0; k < 12; k++) v[k] = sp[k][ts];
            proj<MU, +1>(v, h);
        }
        su3_dag_mul(U, h, uh);
#pragma unroll
        for (int k = 0; k < 6; k++) ex[k][ts] = uh[k];
    }
    __syncthreads();   // every push of this direction is in LDS
    // backward: -1/2 (1 + gamma_mu) U_mu(x - mu)^+ psi(x - mu)
    if (lx > 0) {
        int y[4] = {x[0], x[1], x[2], x[3]};
        y[MU] = x[MU] - 1;
        const int lj = (int)(encode(g, y) - (long)d * Vd);
#pragma unroll
        for (int k = 0; k < 6; k++) uh[k] = ex[k][base + lj];
        recon_acc<MU, +1>(acc, uh, T(-0.5));
    } else {
        int y[4] = {x[0], x[1], x[2], x[3]};
        y[MU] = x[MU] - 1;
        bool wrap = false;
        if (y[MU] < 0) { y[MU] = g.L[MU] - 1; wrap = true; }
        const long J = encode(g, y);
        const unsigned dj = (unsigned)(J / Vd), lj = (unsigned)(J - (long)dj * Vd);
        cx<T> v[12];
        a_load<T, SI, CANON>(g, in, y, dj, lj, v);
        proj<MU, +1>(v, h);
        const unsigned lb = (dj * 4 + MU) * NLC * Vd + lj;
        const su3<T> W = ld_link_with<T, NLC>([&](int e) { return ld32<T, G>(links, lb + e * Vd); });
        su3_dag_mul(W, h, uh);
        recon_acc<MU, +1>(acc, uh, T(wrap ? -0.5 * g.bc[MU] : -0.5));
    }
    __syncthreads();   // the pushes are consumed before the next direction's
}

template <int NT, typename T, typename SI, typename SO, typename G, int NLC, bool CANON>
__global__ __launch_bounds__(NT, 2) void k_apply_A_dom(Geo g, RhsFields<SI> io, const v2<G> *links, const v2<G> *clov)
{
    typedef std::conditional_t<CANON, double, SI> FI;
    typedef std::conditional_t<CANON, double, SO> FO;
    __shared__ cx<T> sp[12][NT + 1];           // the workgroup's input spinors
    __shared__ cx<T> ex[6][NT];                // backward terms pushed to x + mu
    __shared__ int2 site_of[CANON ? NT : 1];   // lexicographic sites: (canonical index, place in the workgroup)
    unsigned blk, rhs;
    rhs_block(io, blk, rhs);
    const int t = threadIdx.x;
    const long I = (long)blk * NT + t;         // V is a multiple of NT: every thread has a site
    const v2<FI> *in = global_ptr((const v2<FI> *)io.in[rhs]);
    v2<FO> *out = global_ptr((v2<FO> *)io.out[rhs]);
    int x[4], d, loc;
    decode(g, I, x, d, loc);
    const unsigned Vd = (unsigned)g.Vd;
    cx<T> acc[12];
    if constexpr (CANON) {
        site_of[t - loc + local_lex(g, x)] = make_int2((int)canon_index(g, x), t);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 12; i++) {
            const int e = t + i * NT, sl = e / 12, k = e - sl * 12;
            const int2 p = site_of[sl];
            const cx<double> c = ld32<double, double>(in, (unsigned)p.x * 12 + k);
            sp[k][p.y] = {static_cast<T>(static_cast<SI>(c.r)), static_cast<T>(static_cast<SI>(c.i))};
        }
        __syncthreads();
    }
    {
        cx<T> s[12];
        if constexpr (CANON) {
#pragma unroll
            for (int k = 0; k < 12; k++) s[k] = sp[k][t];
        } else {
#pragma unroll
            for (int k = 0; k < 12; k++) s[k] = ld32<T, SI>(in, ((unsigned)d * 12 + k) * Vd + loc);
#pragma unroll
            for (int k = 0; k < 12; k++) sp[k][t] = s[k];
        }
        const unsigned cb = (unsigned)d * 36 * Vd + loc;
        clover_block_with<T>([&](int q) { return ld32<T, G>(clov, cb + q * Vd); }, s, acc);
        clover_block_with<T>([&](int q) { return ld32<T, G>(clov, cb + (18 + q) * Vd); }, s + 6, acc + 6);
    }
    if constexpr (!CANON) __syncthreads();
#pragma unroll 1
    for (int mu = 0; mu < 4; mu++) {
        // the site's indices made opaque per direction: what is formed from
        // them (neighbour indices, offsets) is formed here, not hoisted out of
        // the loop and held in registers through it
        int xs[4] = {x[0], x[1], x[2], x[3]}, ds = d, ls = loc, tss = t;
        asm volatile("" : "+v"(xs[0]), "+v"(xs[1]), "+v"(xs[2]), "+v"(xs[3]), "+v"(ds), "+v"(ls), "+v"(tss));
        switch (mu) {
            case 0: a_dom_dir<0, NT, T, SI, G, NLC, CANON>(g, xs, ds, ls, tss, in, links, sp, ex, acc); break;
            case 1: a_dom_dir<1, NT, T, SI, G, NLC, CANON>(g, xs, ds, ls, tss, in, links, sp, ex, acc); break;
            case 2: a_dom_dir<2, NT, T, SI, G, NLC, CANON>(g, xs, ds, ls, tss, in, links, sp, ex, acc); break;
            default: a_dom_dir<3, NT, T, SI, G, NLC, CANON>(g, xs, ds, ls, tss, in, links, sp, ex, acc); break;
        }
    }
    if constexpr (CANON) {
        // (the last direction's closing barrier: sp has been read)
#pragma unroll
        for (int k = 0; k < 12; k++) sp[k][t] = acc[k];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 12; i++) {
            const int e = t + i * NT, sl = e / 12, k = e - sl * 12;
            const int2 p = site_of[sl];
            const cx<T> c = sp[k][p.y];
            st32<double, double>(out, (unsigned)p.x * 12 + k,
                                 cx<double>{static_cast<double>(static_cast<SO>(c.r)), static_cast<double>(static_cast<SO>(c.i))});
        }
    } else {
        int ds = d, ls = loc;   // output offsets formed here, not held through the hops
        asm volatile("" : "+v"(ds), "+v"(ls));
#pragma unroll
        for (int k = 0; k < 12; k++) st32<T, SO>(out, ((unsigned)ds * 12 + k) * Vd + ls, acc[k]);
    }
}

template <bool DOM, int NT, typename T, typename S, int NLC, bool CANON>
static void launch_A(const Geo &g, const void *const *in, void *const *out, int n, const void *links, const void *clov,
                     hipStream_t s)
{
    RhsFields<S> io{};
    io.n = n;
    for (int q = 0; q < n; q++) {
        io.in[q] = in[q];
        io.out[q] = out[q];
    }
    if constexpr (DOM)
        hipLaunchKernelGGL((k_apply_A_dom<NT, T, S, S, S, NLC, CANON>), (unsigned)(g.V / NT) * n, NT, 0, s, g, io,
                           (const v2<S> *)links, (const v2<S> *)clov);
    else
        hipLaunchKernelGGL((k_apply_A<T, S, S, S, NLC, CANON>), nblocks(g.V, NT) * n, NT, 0, s, g, io,
                           (const v2<S> *)links, (const v2<S> *)clov);
}

// at most 16 right-hand sides (16-bit storage: one)
template <bool DOM, int NT>
static void launch_apply_A(const Geo &g, const void *const *in, void *const *out, int n, const void *links,
                           const void *clov, int prec, bool canon, hipStream_t s)
{
    if (canon && prec == P64) launch_A<DOM, NT, double, double, 9, true>(g, in, out, n, links, clov, s);
    else if (canon) launch_A<DOM, NT, float, float, 6, true>(g, in, out, n, links, clov, s);
    else if (prec == P64) launch_A<DOM, NT, double, double, 9, false>(g, in, out, n, links, clov, s);
    else if (prec == P32) launch_A<DOM, NT, float, float, 6, false>(g, in, out, n, links, clov, s);
    else if (prec == P16) launch_A<DOM, NT, float, half_t, 6, false>(g, in, out, n, links, clov, s);
    else launch_A<DOM, NT, float, bf16_t, 6, false>(g, in, out, n, links, clov, s);
}

// whole domains per workgroup where the domain size divides the workgroup's
// site count (V is then a multiple of it) and every field is under 4 GiB (the
// largest, links and clover, hold 36 complex numbers per site)
static int dom_sites(const Geo &g, int prec)
{
    const size_t elem = prec == P64 ? 16 : prec == P32 ? 8 : 4;
    if ((size_t)g.V * 36 * elem >= ((size_t)1 << 32)) return 0;
    if (g.Vd <= 256 && 256 % g.Vd == 0 && g.V % 256 == 0) return 256;
    if (g.Vd == 512 && g.V % 512 == 0) return 512;
    return 0;
}

// Whole domains per workgroup, or one thread per site: the latter for domains
// without such a kernel (288 sites), and where the launch has at most one
// workgroup per CU, which then lasts as long as one workgroup: without LDS and
// barriers it waits for memory less often (8^4 in canonical fields: FP64 16.9
// against 18.2 us, FP32 14.4 against 17.8; 16^3x32 with three right-hand sides,
// 1536 workgroups: FP64 155 against 102 us for all).  Not in FP16, where the two
// kernels' third link rows are not contracted alike and the bits would depend
// on the number of right-hand sides.
static hipError_t apply_A_rhs(const Geo &g, const void *const *in, void *const *out, int n, const void *links,
                              const void *clov, int prec, bool canon, hipStream_t s)
{
    const int nt = dom_sites(g, prec);
    const int most = prec == P64 || prec == P32 ? (int)A_MAX_RHS : 1;
    for (int k = 0; k < n; k += most) {
        const int take = n - k < most ? n - k : most;
        const bool few = g.V / 256 * take <= 256 && prec != P16;
        if (!nt || few) launch_apply_A<false, 256>(g, in + k, out + k, take, links, clov, prec, canon, s);
        else if (nt == 256) launch_apply_A<true, 256>(g, in + k, out + k, take, links, clov, prec, canon, s);
        else launch_apply_A<true, 512>(g, in + k, out + k, take, links, clov, prec, canon, s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// FP64 and FP32 only: with 16-bit storage the neighbours' FP64 spinors cost as much
// as the conversions or more (one right-hand side on 32^3x64 with 4^4 domains: FP16
// 666 us against 478 with the conversions, BF16 459 against 471; on 24x12x12x24 with
// 6x6x2x4: 54 against 37 and 41 against 35); the field under 4 GiB (32-bit byte
// offsets)
bool apply_A_canonical_fits(const Geo &g, int prec)
{
    return (prec == P64 || prec == P32) && (size_t)g.V * 12 * 16 < ((size_t)1 << 32);
}

hipError_t apply_A_canonical(const Geo &g, const double *in, double *out, int nrhs, const void *links, const void *clov,
                             int prec, hipStream_t s)
{
    if (!apply_A_canonical_fits(g, prec)) return hipErrorInvalidValue;
    const size_t n = (size_t)g.V * 24;
    const void *ins[A_MAX_RHS];
    void *outs[A_MAX_RHS];
    for (int k = 0; k < nrhs; k += A_MAX_RHS) {
        const int take = nrhs - k < A_MAX_RHS ? nrhs - k : A_MAX_RHS;
        for (int q = 0; q < take; q++) {
            ins[q] = in + (size_t)(k + q) * n;
            outs[q] = out + (size_t)(k + q) * n;
        }
        const hipError_t e = apply_A_rhs(g, ins, outs, take, links, clov, prec, true, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t apply_A_multi(const Geo &g, const void *const *in, void *const *out, int n, const void *links, const void *clov,
                         int prec, hipStream_t s)
{
    return apply_A_rhs(g, in, out, n, links, clov, prec, false, s);
}

hipError_t apply_A(const Geo &g, const void *in, void *out, const void *links, const void *clov, int prec,
                   hipStream_t s)
{
    return apply_A_multi(g, &in, &out, 1, links, clov, prec, s);
}

// ===========================================================================
// FP64 linear algebra (deterministic two-stage reductions)
// ===========================================================================

constexpr int BS = 256;

template <int N> __device__ __forceinline__ void block_reduce_store(double (&v)[N], double2 *dst_pairs)
{
    // wave64 butterfly, then the waves of the block through LDS in fixed order
    __shared__ double red[BS / 64][N];
#pragma unroll
    for (int q = 0; q < N; q++)
        for (int o = 32; o > 0; o >>= 1) v[q] += __shfl_xor(v[q], o);
    int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0)
#pragma unroll
        for (int q = 0; q < N; q++) red[w][q] = v[q];
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 0; q + 1 < N + 1; q += 2) {
            double a = 0, b = 0;
            for (int k = 0; k < BS / 64; k++) {
                a += red[k][q];
                if (q + 1 < N) b += red[k][q + 1];
            }
            dst_pairs[q / 2] = make_double2(a, b);
        }
    }
}

// blocks of a BLAS launch over n complex elements: about four elements per
// thread, at most BLAS_NBLK (the size of the partial-sum buffer)
static int blas_blocks(long n)
{
    const long b = (n + 4L * BS - 1) / (4L * BS);
    return (int)(b < 1 ? 1 : b > BLAS_NBLK ? BLAS_NBLK : b);
}

// Stage 2 of a reduction, for every system of a list (blockIdx.y): the sum over
// the system's blocks of partial[b][j], j < m, to result[at + j] (pinned host
// memory, read after the stream is waited for), then what the next kernel needs
// of it, formed here so that the host does not have to be asked in between.
enum Finish {
    FIN_STORE,     // nothing more
    FIN_DOTS,      // coef[j] = <W_j, w> / b_j^2 for the first k; the last of m > k is |w|^2
    FIN_CGS,       // b = |w|, the step's coefficient <w, r> / b^2, whether to repeat
    FIN_BICG_RHO, FIN_BICG_ALPHA, FIN_BICG_OMEGA, FIN_BICG_NEXT
};
// A system's scalars on the device, in Blas::coef: 0..15 coefficients of the
// Gram-Schmidt pass, then
enum { CO_STEP = 16, CO_SKIP = 17, CO_BEFORE = 18, CO_NORMS = 19 };   // norms b_j: two a pair, 8 pairs
// and, during BiCGstab,
enum { CO_RHO = 0, CO_ALPHA = 1, CO_OMEGA = 2, CO_BETA = 3, CO_BETA_OMEGA = 4, CO_STOP = 5 };

__device__ __forceinline__ double2 cdiv(double2 a, double2 b)
{
    // scaled by the power of two of the larger part of b, so that |b|^2 neither
    // overflows nor vanishes
    const int e = -ilogb(fmax(fabs(b.x), fabs(b.y)));
    const double c = ldexp(b.x, e), d = ldexp(b.y, e), q = c * c + d * d;
    return make_double2(ldexp((a.x * c + a.y * d) / q, e), ldexp((a.y * c - a.x * d) / q, e));
}
__device__ __forceinline__ double2 cmul2(double2 a, double2 b)
{
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

template <int FIN> __device__ void finish_scalars(const BlasOp &o, const double2 *sum, int m, int k, bool may_repeat, int at)
{
    double2 *co = o.coef;
    double *norms = (double *)(co + CO_NORMS);
    if constexpr (FIN == FIN_DOTS) {
        for (int j = 0; j < k; j++) {
            const double b = norms[j];
            co[j] = make_double2(sum[j].x / b / b, sum[j].y / b / b);
        }
        if (m > k) co[CO_BEFORE] = sum[k];
    } else if constexpr (FIN == FIN_CGS) {
        const double b = sqrt(sum[0].x);
        const bool repeat = may_repeat && !(sum[0].x > 0.25 * co[CO_BEFORE].x);
        norms[k] = b;
        co[CO_STEP] = make_double2(sum[1].x / b / b, sum[1].y / b / b);
        co[CO_SKIP] = make_double2(repeat || !(b > 0) || !isfinite(b), 0);
        if (repeat) co[CO_BEFORE] = sum[0];
    } else if constexpr (FIN == FIN_BICG_RHO) {
        co[CO_RHO] = co[CO_BETA] = sum[0];   // rho, alpha and omega of the step before are 1
        co[CO_BETA_OMEGA] = make_double2(-sum[0].x, -sum[0].y);
    } else if constexpr (FIN == FIN_BICG_ALPHA) {
        const double2 a = cdiv(co[CO_RHO], sum[0]);
        co[CO_ALPHA] = a;
        co[CO_STOP] = o.result[at + 1] = make_double2(!isfinite(a.x) || !isfinite(a.y), 0);
    } else if constexpr (FIN == FIN_BICG_OMEGA) {
        const bool ok = sum[1].x > 0 && isfinite(sum[0].x) && isfinite(sum[0].y);
        co[CO_OMEGA] = o.result[at + 2] = ok ? make_double2(sum[0].x / sum[1].x, sum[0].y / sum[1].x) : make_double2(0, 0);
    } else if constexpr (FIN == FIN_BICG_NEXT) {
        const double2 beta = cmul2(cdiv(sum[1], co[CO_RHO]), cdiv(co[CO_ALPHA], co[CO_OMEGA]));
        const double2 bo = cmul2(beta, co[CO_OMEGA]);
        co[CO_RHO] = sum[1];
        co[CO_BETA] = beta;
        co[CO_BETA_OMEGA] = make_double2(-bo.x, -bo.y);
    }
}

// the device's clock (wall_clock64, of a fixed rate) into pinned host memory
__global__ void k_stamp(unsigned long long *t) { *t = wall_clock64(); }

hipError_t stamp(unsigned long long *t, hipStream_t s)
{
    hipLaunchKernelGGL(k_stamp, 1, 1, 0, s, t);
    return hipGetLastError();
}

template <int FIN>
__global__ __launch_bounds__(BS) void k_finish(BlasList L, int m, int k, bool may_repeat, int at, unsigned long long *end)
{
    __shared__ double2 red[BS], sum[BLAS_MAXK];
    const BlasOp o = L.op[blockIdx.y];
    for (int j = 0; j < m; j++) {
        double2 s = make_double2(0, 0);
        for (int b = threadIdx.x; b < o.nblk; b += BS) {
            double2 v = o.partial[(long)b * 32 + j];
            s.x += v.x;
            s.y += v.y;
        }
        red[threadIdx.x] = s;
        __syncthreads();
        for (int q = BS / 2; q > 0; q >>= 1) {
            if ((int)threadIdx.x < q) {
                red[threadIdx.x].x += red[threadIdx.x + q].x;
                red[threadIdx.x].y += red[threadIdx.x + q].y;
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) sum[j] = o.result[at + j] = red[0];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        finish_scalars<FIN>(o, sum, m, k, may_repeat, at);
        if (end && blockIdx.y == 0) *end = wall_clock64();
    }
}

template <int FIN> static void launch_finish(const BlasList &L, int ns, int m, int at, hipStream_t s, int k = 0, bool may_repeat = false,
                                            unsigned long long *end = nullptr)
{
    hipLaunchKernelGGL(k_finish<FIN>, dim3(1, ns), BS, 0, s, L, m, k, may_repeat, at, end);
}

// ---- several systems in one launch: blockIdx.y is the system -----------------
// Every system keeps the blocks, and with them the order of its sums, that it
// has alone; a launch has those of the largest.

BlasOp blas_op(const Blas &B, long n)
{
    BlasOp o{};
    o.partial = B.partial;
    o.result = B.result;
    o.coef = B.coef;
    o.n = n;
    o.nblk = blas_blocks(n);
    return o;
}

static hipError_t finish_one(const Blas &B, long n, int m, hipStream_t s)
{
    BlasList L{};
    L.op[0] = blas_op(B, n);
    launch_finish<FIN_STORE>(L, 1, m, 0, s);
    return hipGetLastError();
}

// f(list, systems, grid) for BLAS_LIST systems at a time
template <typename F> static hipError_t for_lists(const std::vector<BlasOp> &ops, F f)
{
    for (size_t i = 0; i < ops.size(); i += BLAS_LIST) {
        BlasList L{};
        const int ns = (int)(ops.size() - i < BLAS_LIST ? ops.size() - i : BLAS_LIST);
        int nb = 1;
        for (int q = 0; q < ns; q++) {
            L.op[q] = ops[i + q];
            if (L.op[q].nblk > nb) nb = L.op[q].nblk;
        }
        f(L, ns, dim3(nb, ns));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// this block's system and its elements: first, past the last, step
#define DD_BLAS_OP(o, i)                                                   \
    const BlasOp o = L.op[blockIdx.y];                                     \
    if ((int)blockIdx.x >= o.nblk) return;                                 \
    const long step = (long)o.nblk * BS;                                   \
    long i = (long)blockIdx.x * BS + threadIdx.x

// <W_j, w>, j < K
template <int K> __global__ __launch_bounds__(BS) void k_multidot(BlasList L)
{
    DD_BLAS_OP(o, i);
    double acc[2 * K];
#pragma unroll
    for (int q = 0; q < 2 * K; q++) acc[q] = 0;
    for (; i < o.n; i += step) {
        double2 b = o.w[i];
#pragma unroll
        for (int j = 0; j < K; j++) {
            double2 a = o.W[j * o.n + i];
            acc[2 * j] += a.x * b.x + a.y * b.y;
            acc[2 * j + 1] += a.x * b.y - a.y * b.x;
        }
    }
    block_reduce_store<2 * K>(acc, o.partial + (long)blockIdx.x * 32);
}

static hipError_t launch_multidot(const BlasList &L, dim3 grid, int k, hipStream_t s)
{
    switch (k) {
#define MD(K) case K: hipLaunchKernelGGL(k_multidot<K>, grid, BS, 0, s, L); break;
        MD(1) MD(2) MD(3) MD(4) MD(5) MD(6) MD(7) MD(8) MD(9) MD(10) MD(11) MD(12) MD(13) MD(14) MD(15) MD(16)
#undef MD
        default: return hipErrorInvalidValue;
    }
    return hipSuccess;
}

hipError_t multidot(Blas &B, const double2 *W, int k, double2 *v, long n, hipStream_t s)
{
    if (k < 1 || k > BLAS_MAXK) return hipErrorInvalidValue;
    BlasOp o = blas_op(B, n);
    o.W = W;
    o.w = v;
    return for_lists({o}, [&](const BlasList &L, int ns, dim3 grid) {
        (void)launch_multidot(L, grid, k, s);
        launch_finish<FIN_STORE>(L, ns, k, 0, s);
    });
}

// w -= sum_j coef[j] W_j; |w|^2 and <w, r>
template <int K> __global__ __launch_bounds__(BS) void k_cgs_update(BlasList L)
{
    DD_BLAS_OP(o, i);
    double2 c[K > 0 ? K : 1];
#pragma unroll
    for (int j = 0; j < K; j++) c[j] = o.coef[j];
    double acc[4] = {0, 0, 0, 0};
    for (; i < o.n; i += step) {
        double2 x = o.w[i];
#pragma unroll
        for (int j = 0; j < K; j++) {
            double2 a = o.W[j * o.n + i];
            x.x -= c[j].x * a.x - c[j].y * a.y;
            x.y -= c[j].x * a.y + c[j].y * a.x;
        }
        if (K > 0) o.w[i] = x;
        double2 b = o.r[i];
        acc[0] += x.x * x.x + x.y * x.y;
        acc[2] += x.x * b.x + x.y * b.y;
        acc[3] += x.x * b.y - x.y * b.x;
    }
    block_reduce_store<4>(acc, o.partial + (long)blockIdx.x * 32);
}

static hipError_t launch_cgs_update(const BlasList &L, dim3 grid, int k, hipStream_t s)
{
    switch (k) {
#define CU(K) case K: hipLaunchKernelGGL(k_cgs_update<K>, grid, BS, 0, s, L); break;
        CU(0) CU(1) CU(2) CU(3) CU(4) CU(5) CU(6) CU(7) CU(8) CU(9) CU(10) CU(11) CU(12) CU(13) CU(14) CU(15) CU(16)
#undef CU
        default: return hipErrorInvalidValue;
    }
    return hipSuccess;
}

hipError_t cgs_update(Blas &B, double2 *w, const double2 *W, int k, double2 *r, long n, hipStream_t s)
{
    if (k < 0 || k > BLAS_MAXK) return hipErrorInvalidValue;
    BlasOp o = blas_op(B, n);
    o.W = W;
    o.w = w;
    o.r = r;
    return for_lists({o}, [&](const BlasList &L, int ns, dim3 grid) {
        (void)launch_cgs_update(L, grid, k, s);
        launch_finish<FIN_STORE>(L, ns, 2, 0, s);
    });
}

// r -= <w, r> / |w|^2 w unless the pass is to be repeated (or w vanished); |r|^2
__global__ __launch_bounds__(BS) void k_residual_update(BlasList L)
{
    DD_BLAS_OP(o, i);
    if (o.coef[CO_SKIP].x != 0) return;
    const double2 c = o.coef[CO_STEP];
    double acc[2] = {0, 0};
    for (; i < o.n; i += step) {
        const double2 x = o.w[i];
        double2 y = o.r[i];
        y.x -= c.x * x.x - c.y * x.y;
        y.y -= c.x * x.y + c.y * x.x;
        o.r[i] = y;
        acc[0] += y.x * y.x + y.y * y.y;
    }
    block_reduce_store<2>(acc, o.partial + (long)blockIdx.x * 32);
}

// One pass of the Gram-Schmidt step of every system and, unless it has to be
// repeated, the residual's update: three reductions whose results are used on
// the device and read by the host together.  With a copy and a wait after each
// reduction and a launch per system, five steps on 4^4 took 180 us more (2810
// us, now 2630) and those of 12 systems on 16^3x32 1.7 ms more (42.6, now 40.9).
hipError_t fgcr_step(const std::vector<BlasOp> &ops, int k, int nd, bool may_repeat, unsigned long long *end, hipStream_t s)
{
    if (k < 0 || k > BLAS_MAXK || nd < k || nd > BLAS_MAXK) return hipErrorInvalidValue;
    return for_lists(ops, [&](const BlasList &L, int ns, dim3 grid) {
        if (nd > 0) {
            (void)launch_multidot(L, grid, nd, s);
            launch_finish<FIN_DOTS>(L, ns, nd, STEP_DOTS, s, k);
        }
        (void)launch_cgs_update(L, grid, k, s);
        launch_finish<FIN_CGS>(L, ns, 2, STEP_W, s, k, may_repeat);
        hipLaunchKernelGGL(k_residual_update, grid, BS, 0, s, L);
        launch_finish<FIN_STORE>(L, ns, 1, STEP_R, s, 0, false, end);
    });
}

struct Coefs {
    double2 c[BLAS_MAXK];
};
template <int K> __global__ __launch_bounds__(BS) void k_axpy_multi(double2 *x, const double2 *Z, Coefs co, long n)
{
    double2 c[K];
#pragma unroll
    for (int j = 0; j < K; j++) c[j] = co.c[j];
    for (long i = (long)blockIdx.x * BS + threadIdx.x; i < n; i += (long)gridDim.x * BS) {
        double2 y = x[i];
#pragma unroll
        for (int j = 0; j < K; j++) {
            double2 a = Z[j * n + i];
            y.x += c[j].x * a.x - c[j].y * a.y;
            y.y += c[j].x * a.y + c[j].y * a.x;
        }
        x[i] = y;
    }
}

hipError_t axpy_multi(double2 *x, const double2 *Z, const double2 *coef, int k, long n, hipStream_t s)
{
    if (k < 1 || k > BLAS_MAXK) return hipErrorInvalidValue;
    Coefs co{};
    for (int j = 0; j < k; j++) co.c[j] = coef[j];
    switch (k) {
#define AX(K) case K: hipLaunchKernelGGL(k_axpy_multi<K>, blas_blocks(n), BS, 0, s, x, Z, co, n); break;
        AX(1) AX(2) AX(3) AX(4) AX(5) AX(6) AX(7) AX(8) AX(9) AX(10) AX(11) AX(12) AX(13) AX(14) AX(15) AX(16)
#undef AX
    }
    return hipGetLastError();
}

// r = b - r (b: the operand w); |r|^2
__global__ __launch_bounds__(BS) void k_residual(BlasList L)
{
    DD_BLAS_OP(o, i);
    double acc[2] = {0, 0};
    for (; i < o.n; i += step) {
        double2 y = o.w[i], a = o.r[i];
        y.x -= a.x;
        y.y -= a.y;
        o.r[i] = y;
        acc[0] += y.x * y.x + y.y * y.y;
    }
    block_reduce_store<2>(acc, o.partial + (long)blockIdx.x * 32);
}

hipError_t residual(const std::vector<BlasOp> &ops, hipStream_t s)
{
    return for_lists(ops, [&](const BlasList &L, int ns, dim3 grid) {
        hipLaunchKernelGGL(k_residual, grid, BS, 0, s, L);
        launch_finish<FIN_STORE>(L, ns, 1, 0, s);
    });
}

hipError_t residual(Blas &B, double2 *b, double2 *r, long n, hipStream_t s)
{
    BlasOp o = blas_op(B, n);
    o.w = b;
    o.r = r;
    return residual({o}, s);
}

__global__ __launch_bounds__(BS) void k_norm2(BlasList L)
{
    DD_BLAS_OP(o, i);
    double acc[2] = {0, 0};
    for (; i < o.n; i += step) {
        double2 y = o.w[i];
        acc[0] += y.x * y.x + y.y * y.y;
    }
    block_reduce_store<2>(acc, o.partial + (long)blockIdx.x * 32);
}

hipError_t norm2(const std::vector<BlasOp> &ops, hipStream_t s)
{
    return for_lists(ops, [&](const BlasList &L, int ns, dim3 grid) {
        hipLaunchKernelGGL(k_norm2, grid, BS, 0, s, L);
        launch_finish<FIN_STORE>(L, ns, 1, 0, s);
    });
}

hipError_t norm2(Blas &B, double2 *v, long n, hipStream_t s)
{
    BlasOp o = blas_op(B, n);
    o.w = v;
    return norm2({o}, s);
}

// ---- BiCGstab: vector updates whose coefficients earlier reductions left on
// the device (coef of the system), so that an iteration is launched as a whole.
// Each is bound by memory; what shares operands shares a pass: 21 vectors are
// moved an iteration besides the operator's.  16^3x32: 196 us an iteration, 285
// with a wait for the host after each of four reductions and 24 vectors moved.

__device__ __forceinline__ double2 axpy2(double2 y, double2 c, double2 x)
{
    y.x += c.x * x.x - c.y * x.y;
    y.y += c.x * x.y + c.y * x.x;
    return y;
}

// p = r + beta (p - omega v)
__global__ __launch_bounds__(BS) void k_bicg_p(BicgVectors V, const double2 *co, long n)
{
    const double2 b = co[CO_BETA], bo = co[CO_BETA_OMEGA];
    for (long i = (long)blockIdx.x * BS + threadIdx.x; i < n; i += (long)gridDim.x * BS)
        V.p[i] = axpy2(axpy2(V.r[i], b, V.p[i]), bo, V.v[i]);
}

// s = r - alpha v
__global__ __launch_bounds__(BS) void k_bicg_s(BicgVectors V, const double2 *co, long n)
{
    const double2 a = co[CO_ALPHA], ma = make_double2(-a.x, -a.y);
    for (long i = (long)blockIdx.x * BS + threadIdx.x; i < n; i += (long)gridDim.x * BS)
        V.s[i] = axpy2(V.r[i], ma, V.v[i]);
}

// <t, s>, |t|^2
__global__ __launch_bounds__(BS) void k_bicg_ts(BicgVectors V, long n, double2 *partial)
{
    double acc[4] = {0, 0, 0, 0};
    for (long i = (long)blockIdx.x * BS + threadIdx.x; i < n; i += (long)gridDim.x * BS) {
        const double2 a = V.t[i], b = V.s[i];
        acc[0] += a.x * b.x + a.y * b.y;
        acc[1] += a.x * b.y - a.y * b.x;
        acc[2] += a.x * a.x + a.y * a.y;
    }
    block_reduce_store<4>(acc, partial + (long)blockIdx.x * 32);
}

// x += alpha p + omega s, r = s - omega t, |r|^2, <r0, r>; nothing where alpha
// is not finite
__global__ __launch_bounds__(BS) void k_bicg_xr(BicgVectors V, const double2 *co, long n, double2 *partial)
{
    if (co[CO_STOP].x != 0) return;
    const double2 a = co[CO_ALPHA], w = co[CO_OMEGA], mw = make_double2(-w.x, -w.y);
    double acc[4] = {0, 0, 0, 0};
    for (long i = (long)blockIdx.x * BS + threadIdx.x; i < n; i += (long)gridDim.x * BS) {
        const double2 sv = V.s[i], y = axpy2(sv, mw, V.t[i]), r0 = V.r0[i];
        V.x[i] = axpy2(axpy2(V.x[i], a, V.p[i]), w, sv);
        V.r[i] = y;
        acc[0] += y.x * y.x + y.y * y.y;
        acc[2] += r0.x * y.x + r0.y * y.y;
        acc[3] += r0.x * y.y - r0.y * y.x;
    }
    block_reduce_store<4>(acc, partial + (long)blockIdx.x * 32);
}

static void bicg_finish(const Blas &B, long n, int fin, int m, int at, hipStream_t s)
{
    BlasList L{};
    L.op[0] = blas_op(B, n);
    switch (fin) {
        case FIN_BICG_RHO: launch_finish<FIN_BICG_RHO>(L, 1, m, at, s); break;
        case FIN_BICG_ALPHA: launch_finish<FIN_BICG_ALPHA>(L, 1, m, at, s); break;
        case FIN_BICG_OMEGA: launch_finish<FIN_BICG_OMEGA>(L, 1, m, at, s); break;
        default: launch_finish<FIN_BICG_NEXT>(L, 1, m, at, s); break;
    }
}

static void bicg_dot(const Blas &B, const double2 *a, double2 *b, long n, int fin, int at, hipStream_t s)
{
    BlasList L{};
    L.op[0] = blas_op(B, n);
    L.op[0].W = a;
    L.op[0].w = b;
    hipLaunchKernelGGL(k_multidot<1>, blas_blocks(n), BS, 0, s, L);
    bicg_finish(B, n, fin, 1, at, s);
}

hipError_t bicg_start(Blas &B, const BicgVectors &V, long n, hipStream_t s)
{
    bicg_dot(B, V.r0, V.r, n, FIN_BICG_RHO, BICG_RHO, s);
    return hipGetLastError();
}

hipError_t bicg_direction(Blas &B, const BicgVectors &V, long n, hipStream_t s)
{
    hipLaunchKernelGGL(k_bicg_p, blas_blocks(n), BS, 0, s, V, B.coef, n);
    return hipGetLastError();
}

hipError_t bicg_half(Blas &B, const BicgVectors &V, long n, hipStream_t s)
{
    bicg_dot(B, V.r0, V.v, n, FIN_BICG_ALPHA, BICG_R0V, s);
    hipLaunchKernelGGL(k_bicg_s, blas_blocks(n), BS, 0, s, V, B.coef, n);
    return hipGetLastError();
}

hipError_t bicg_update(Blas &B, const BicgVectors &V, long n, hipStream_t s)
{
    hipLaunchKernelGGL(k_bicg_ts, blas_blocks(n), BS, 0, s, V, n, B.partial);
    bicg_finish(B, n, FIN_BICG_OMEGA, 2, BICG_TS, s);
    hipLaunchKernelGGL(k_bicg_xr, blas_blocks(n), BS, 0, s, V, B.coef, n, B.partial);
    bicg_finish(B, n, FIN_BICG_NEXT, 2, BICG_RR, s);
    return hipGetLastError();
}

// out = ca a + cb b + cc c (complex coefficients; c may be null; out may alias a, b or c)
__global__ __launch_bounds__(BS) void k_lincomb(double2 *out, const double2 *a, double2 ca, const double2 *b,
                                                double2 cb, const double2 *c, double2 cc, long n)
{
    for (long i = (long)blockIdx.x * BS + threadIdx.x; i < n; i += (long)gridDim.x * BS) {
        const double2 x = a[i], y = b[i];
        double2 o;
        o.x = ca.x * x.x - ca.y * x.y + cb.x * y.x - cb.y * y.y;
        o.y = ca.x * x.y + ca.y * x.x + cb.x * y.y + cb.y * y.x;
        if (c) {
            const double2 z = c[i];
            o.x += cc.x * z.x - cc.y * z.y;
            o.y += cc.x * z.y + cc.y * z.x;
        }
        out[i] = o;
    }
}

hipError_t lincomb(double2 *out, const double2 *a, double2 ca, const double2 *b, double2 cb, const double2 *c,
                   double2 cc, long n, hipStream_t s)
{
    hipLaunchKernelGGL(k_lincomb, blas_blocks(n), BS, 0, s, out, a, ca, b, cb, c, cc, n);
    return hipGetLastError();
}

// ---- FP32 vectors with FP64 accumulation (the inner solve of the
// mixed-precision outer solver) ----------------------------------------------

template <int K>
__global__ __launch_bounds__(BS) void k_multidot32(const float2 *W, long ldw, const float2 *v, long n, double2 *partial)
{
    double acc[2 * K];
#pragma unroll
    for (int q = 0; q < 2 * K; q++) acc[q] = 0;
    for (long i = (long)blockIdx.x * BS + threadIdx.x; i < n; i += (long)gridDim.x * BS) {
        const float2 b = v[i];
#pragma unroll
        for (int j = 0; j < K; j++) {
            const float2 a = W[j * ldw + i];
            acc[2 * j] += (double)a.x * b.x + (double)a.y * b.y;
            acc[2 * j + 1] += (double)a.x * b.y - (double)a.y * b.x;
        }
    }
    block_reduce_store<2 * K>(acc, partial + (long)blockIdx.x * 32);
}

hipError_t multidot32(Blas &B, const float2 *W, long ldw, int k, const float2 *v, long n, hipStream_t s)
{
    switch (k) {
#define MD(K) case K: hipLaunchKernelGGL(k_multidot32<K>, blas_blocks(n), BS, 0, s, W, ldw, v, n, B.partial); break;
        MD(1) MD(2) MD(3) MD(4) MD(5) MD(6) MD(7) MD(8) MD(9) MD(10) MD(11) MD(12) MD(13) MD(14) MD(15) MD(16)
#undef MD
        default: return hipErrorInvalidValue;
    }
    return finish_one(B, n, k, s);
}

template <int K>
__global__ __launch_bounds__(BS) void k_cgs_update32(float2 *w, const float2 *W, long ldw, const double2 *coef, long n,
                                                     double2 *partial)
{
    double2 c[K > 0 ? K : 1];
#pragma unroll
    for (int j = 0; j < K; j++) c[j] = coef[j];
    double acc[2] = {0, 0};
    for (long i = (long)blockIdx.x * BS + threadIdx.x; i < n; i += (long)gridDim.x * BS) {
        const float2 x0 = w[i];
        double xr = x0.x, xi = x0.y;
#pragma unroll
        for (int j = 0; j < K; j++) {
            const float2 a = W[j * ldw + i];
            xr -= c[j].x * a.x - c[j].y * a.y;
            xi -= c[j].x * a.y + c[j].y * a.x;
        }
        const float2 x = make_float2((float)xr, (float)xi);
        w[i] = x;
        acc[0] += (double)x.x * x.x + (double)x.y * x.y;
    }
    block_reduce_store<2>(acc, partial + (long)blockIdx.x * 32);
}

hipError_t cgs_update32(Blas &B, float2 *w, const float2 *W, long ldw, int k, long n, hipStream_t s)
{
    switch (k) {
#define CU(K) case K: hipLaunchKernelGGL(k_cgs_update32<K>, blas_blocks(n), BS, 0, s, w, W, ldw, B.coef, n, B.partial); break;
        CU(0) CU(1) CU(2) CU(3) CU(4) CU(5) CU(6) CU(7) CU(8) CU(9) CU(10) CU(11) CU(12) CU(13) CU(14) CU(15) CU(16)
#undef CU
        default: return hipErrorInvalidValue;
    }
    return finish_one(B, n, 1, s);
}

// w *= inv_b; then result[0] = <w, r>, after which r -= c w with c = that dot
// is left to k_axpy32 (c is only known on the host)
__global__ __launch_bounds__(BS) void k_scale_dot32(float2 *w, double inv_b, const float2 *r, long n, double2 *partial)
{
    double acc[2] = {0, 0};
    for (long i = (long)blockIdx.x * BS + threadIdx.x; i < n; i += (long)gridDim.x * BS) {
        float2 x = w[i];
        x.x = (float)(x.x * inv_b);
        x.y = (float)(x.y * inv_b);
        w[i] = x;
        const float2 b = r[i];
        acc[0] += (double)x.x * b.x + (double)x.y * b.y;
        acc[1] += (double)x.x * b.y - (double)x.y * b.x;
    }
    block_reduce_store<2>(acc, partial + (long)blockIdx.x * 32);
}

hipError_t scale_dot32(Blas &B, float2 *w, double inv_b, const float2 *r, long n, hipStream_t s)
{
    hipLaunchKernelGGL(k_scale_dot32, blas_blocks(n), BS, 0, s, w, inv_b, r, n, B.partial);
    return finish_one(B, n, 1, s);
}

// r -= c w; result[0] = (|r|^2, 0)
__global__ __launch_bounds__(BS) void k_axpy32(float2 *r, double2 c, const float2 *w, long n, double2 *partial)
{
    double acc[2] = {0, 0};
    for (long i = (long)blockIdx.x * BS + threadIdx.x; i < n; i += (long)gridDim.x * BS) {
        const float2 x = w[i];
        float2 y = r[i];
        y.x = (float)(y.x - (c.x * x.x - c.y * x.y));
        y.y = (float)(y.y - (c.x * x.y + c.y * x.x));
        r[i] = y;
        acc[0] += (double)y.x * y.x + (double)y.y * y.y;
    }
    block_reduce_store<2>(acc, partial + (long)blockIdx.x * 32);
}

hipError_t axpy32(Blas &B, float2 *r, double2 c, const float2 *w, long n, hipStream_t s)
{
    hipLaunchKernelGGL(k_axpy32, blas_blocks(n), BS, 0, s, r, c, w, n, B.partial);
    return finish_one(B, n, 1, s);
}

// x += scale * sum_j coef[j] Z_j (FP64 x, FP32 Z)
template <int K>
__global__ __launch_bounds__(BS) void k_axpy_mixed(double2 *x, const float2 *Z, long ldz, const double2 *coef,
                                                   double scale, long n)
{
    double2 c[K];
#pragma unroll
    for (int j = 0; j < K; j++) c[j] = make_double2(scale * coef[j].x, scale * coef[j].y);
    for (long i = (long)blockIdx.x * BS + threadIdx.x; i < n; i += (long)gridDim.x * BS) {
        double2 y = x[i];
#pragma unroll
        for (int j = 0; j < K; j++) {
            const float2 a = Z[j * ldz + i];
            y.x += c[j].x * a.x - c[j].y * a.y;
            y.y += c[j].x * a.y + c[j].y * a.x;
        }
        x[i] = y;
    }
}

hipError_t axpy_mixed(Blas &B, double2 *x, const float2 *Z, long ldz, int k, double scale, long n, hipStream_t s)
{
    switch (k) {
#define AX(K) case K: hipLaunchKernelGGL(k_axpy_mixed<K>, blas_blocks(n), BS, 0, s, x, Z, ldz, B.coef, scale, n); break;
        AX(1) AX(2) AX(3) AX(4) AX(5) AX(6) AX(7) AX(8) AX(9) AX(10) AX(11) AX(12) AX(13) AX(14) AX(15) AX(16)
#undef AX
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// out = s * in, rounded to FP32
__global__ __launch_bounds__(BS) void k_to_f32(const double2 *in, double sc, float2 *out, long n)
{
    for (long i = (long)blockIdx.x * BS + threadIdx.x; i < n; i += (long)gridDim.x * BS) {
        const double2 v = in[i];
        out[i] = make_float2((float)(sc * v.x), (float)(sc * v.y));
    }
}

hipError_t to_f32(const double2 *in, double sc, float2 *out, long n, hipStream_t s)
{
    hipLaunchKernelGGL(k_to_f32, blas_blocks(n), BS, 0, s, in, sc, out, n);
    return hipGetLastError();
}

// out_q = sum_i W_i P[i][q] for q < nq (columns of n complex numbers, W_i =
// W + i*ldw, out_q = out + q*ldo; P row-major nin x nq on the device, nin, nq
// <= RECOMB_MAX).  Each element of the inputs is read once; the outputs of one
// element accumulate in registers.
constexpr int RECOMB_MAX = 24;
__global__ __launch_bounds__(BS) void k_recombine(const double2 *W, long ldw, int nin, const double2 *P, int nq,
                                                  double2 *out, long ldo, long n)
{
    __shared__ double2 sp[RECOMB_MAX * RECOMB_MAX];
    for (int t = threadIdx.x; t < nin * nq; t += BS) sp[t] = P[t];
    __syncthreads();
    for (long e = (long)blockIdx.x * BS + threadIdx.x; e < n; e += (long)gridDim.x * BS) {
        double2 acc[RECOMB_MAX];
#pragma unroll
        for (int q = 0; q < RECOMB_MAX; q++) acc[q] = make_double2(0, 0);
        for (int i = 0; i < nin; i++) {
            const double2 w = W[i * ldw + e];
#pragma unroll
            for (int q = 0; q < RECOMB_MAX; q++) {
                if (q >= nq) break;
                const double2 c = sp[i * nq + q];
                acc[q].x += c.x * w.x - c.y * w.y;
                acc[q].y += c.x * w.y + c.y * w.x;
            }
        }
#pragma unroll
        for (int q = 0; q < RECOMB_MAX; q++) {
            if (q >= nq) break;
            out[q * ldo + e] = acc[q];
        }
    }
}

hipError_t recombine(const double2 *W, long ldw, int nin, const double2 *P, int nq, double2 *out, long ldo, long n,
                     hipStream_t s)
{
    if (nin < 1 || nq < 1 || nin > RECOMB_MAX || nq > RECOMB_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_recombine, blas_blocks(n), BS, 0, s, W, ldw, nin, P, nq, out, ldo, n);
    return hipGetLastError();
}

__global__ void k_zero(double2 *v, long n)
{
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
        v[i] = make_double2(0, 0);
}

hipError_t zero(double2 *v, long n, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero, 2048, 256, 0, s, v, n);
    return hipGetLastError();
}

}  // namespace dd
