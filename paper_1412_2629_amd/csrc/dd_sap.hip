// One half-sweep of the Schwarz alternating procedure (multiplicative
// Schwarz, Sec. II-D and the algorithm of Table I): every domain of one colour
// solves D_Omega delta = rho_Omega approximately and adds delta to the
// solution.  One workgroup per domain, one thread per site; the spinors the
// block solve exchanges between sites live in LDS for the whole solve.
//
// Residual bookkeeping.  After a domain's block solve its residual is known
// exactly: the MR residual on the even sites and zero on the odd sites
// (Sec. II-D, Eq. 5).  Between two solves of a domain only its neighbours
// (the other colour) change the solution, by their own delta, so the domain
// next sees
//     rho = stored block residual - R delta_neighbours .
// Each domain therefore stores, after its solve, its block residual and the
// boundary half-spinors of its delta (the terms of R that its neighbours
// need: (1 - gamma_mu) delta on its -mu face, U_mu^dagger (1 + gamma_mu) delta
// on its +mu face), and gathers its neighbours' at the start of its next
// solve.  This is the paper's packed boundary buffers (Sec. III-A) with the
// gather done by the reading domain, so no two workgroups write the same
// address and no atomics are needed.
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>
#include <unordered_map>

#include "dd_device.h"
#include "dd_internal.h"

namespace dd {

template <int BX, int BY, int BZ, int BT> struct Shape {
    static constexpr int VD = BX * BY * BZ * BT;
    static constexpr int VH = VD / 2;
    static constexpr int B[4] = {BX, BY, BZ, BT};
    static constexpr int FS[4] = {VD / BX, VD / BY, VD / BZ, VD / BT};
    static constexpr int FTOT = 2 * (VD / BX + VD / BY + VD / BZ + VD / BT);
    static_assert(BX % 2 == 0 && BY % 2 == 0 && BZ % 2 == 0 && BT % 2 == 0, "domain extents must be even");

    // face f = 2*mu + side (side 0: l_mu = 0, side 1: l_mu = B_mu - 1)
    static constexpr int foff(int f)
    {
        int o = 0;
        for (int q = 0; q < f; q++) o += FS[q >> 1];
        return o;
    }
    __device__ static void coords(int loc, int l[4])
    {
        int p = loc >= VH;
        int h = loc - p * VH;
        int xh = h % (BX / 2);
        int row = h / (BX / 2);
        l[1] = row % BY;
        row /= BY;
        l[2] = row % BZ;
        l[3] = row / BZ;
        l[0] = 2 * xh + ((p + l[1] + l[2] + l[3]) & 1);
    }
    // index within the half-lattice of the site's own parity
    __device__ static int half_index(const int l[4]) { return (l[0] + BX * (l[1] + BY * (l[2] + BZ * l[3]))) >> 1; }
    template <int MU> __device__ static int face_index(const int l[4])
    {
        if constexpr (MU == 0) return l[1] + BY * (l[2] + BZ * l[3]);
        else if constexpr (MU == 1) return l[0] + BX * (l[2] + BZ * l[3]);
        else if constexpr (MU == 2) return l[0] + BX * (l[1] + BY * l[3]);
        else return l[0] + BX * (l[1] + BY * l[2]);
    }
};

// ---- block reductions over all VD threads (deterministic order) -----------

template <int CTRL> __device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL> __device__ __forceinline__ double dpp(double v)
{
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_value(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_value(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}
// Sum (MAX: maximum) over groups of SEG consecutive lanes (4, 8, 16 or 64), in
// every lane of the group (all lanes active): DPP permutes within each 16-lane
// row (lane ^ 1, lane ^ 2, then the mirrored halves of 8 and of 16 lanes) leave
// every lane with its row's result; the four row results are read out and
// combined.  A permute is an operand of the addition; a shuffle through LDS
// waits a hundred cycles and more at each step.  With the 16-bit epilogue's two
// maxima taken together, a launch on 8^4 went from 28.6 to 27.6 us (FP16, 4^4
// domains), from 26.8 to 25.4 (2^4), in FP64 from 31.4 to 30.0.
template <int SEG, bool MAX, typename T> __device__ __forceinline__ T lanes_reduce(T v)
{
    static_assert(SEG == 4 || SEG == 8 || SEG == 16 || SEG == 64, "lanes of a group");
    auto op = [](T a, T b) { return MAX ? fmax(a, b) : a + b; };
    v = op(v, dpp<0xB1>(v));                           // quad_perm 1,0,3,2
    v = op(v, dpp<0x4E>(v));                           // quad_perm 2,3,0,1
    if constexpr (SEG >= 8) v = op(v, dpp<0x141>(v));   // row_half_mirror
    if constexpr (SEG >= 16) v = op(v, dpp<0x140>(v));  // row_mirror
    if constexpr (SEG == 64)
        v = op(op(lane_value(v, 0), lane_value(v, 16)), op(lane_value(v, 32), lane_value(v, 48)));
    return v;
}

// Sums (MAX: maxima) over the sites of each domain of the workgroup, NW waves;
// every thread joins.  NDW > 1: VH consecutive lanes of a wave belong to one
// domain, sub the calling thread's; NDW == 1: all waves to one.  No closing
// barrier: a call site has its own part of red or barriers pass before its next use.
template <int VH, int NDW, int NW, bool MAX, typename T, int N>
__device__ __forceinline__ void domain_reduce(T (&v)[N], T *red, int sub)
{
    constexpr int SEG = NDW > 1 ? VH : 64;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < N; k++) v[k] = lanes_reduce<SEG, MAX>(v[k]);
    if (lane % SEG == 0)
#pragma unroll
        for (int k = 0; k < N; k++) red[(k * NW + w) * NDW + (NDW > 1 ? lane / SEG : 0)] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N; k++) {
        T s = red[k * NW * NDW + sub];
#pragma unroll
        for (int j = 1; j < NW; j++) {
            const T x = red[(k * NW + j) * NDW + sub];
            s = MAX ? fmax(s, x) : s + x;
        }
        v[k] = s;
    }
}

// smallest power of two >= m (m > 0), 1 for m == 0
template <typename T> __device__ __forceinline__ T pow2_ceil(T m)
{
    if (!(m > T(0))) return T(1);
    int e;
    T f = frexp(m, &e);   // m = f * 2^e, f in [0.5, 1)
    (void)f;
    return ldexp(T(1), e);
}

template <typename T> __device__ __forceinline__ T maxabs12(const cx<T> a[12])
{
    T m = 0;
#pragma unroll
    for (int k = 0; k < 12; k++) m = fmax(m, fmax(fabs(a[k].r), fabs(a[k].i)));
    return m;
}

// ---- in-domain hopping terms from an LDS half-lattice spinor --------------
//
// acc += sum over in-domain neighbours of (1 - gamma_mu) U_mu(x) v(x+mu) and
// (1 + gamma_mu) U_mu(x-mu)^dagger v(x-mu); the -1/2 of Eq. 1 is applied by
// the caller.  v holds the sites of the other parity.

template <class Sh, int MU, typename T, typename G, int NLC>
__device__ __forceinline__ void dom_hop(const cx<T> (*v)[Sh::VH], const int l[4], long lbase, int loc,
                                        const v2<G> *links, cx<T> acc[12], T scale = T(1))
{
    constexpr int VD = Sh::VD;
    int n[4] = {l[0], l[1], l[2], l[3]};
    cx<T> s[12], h[6], uh[6];
    if (l[MU] + 1 < Sh::B[MU]) {
        n[MU] = l[MU] + 1;
        int nh = Sh::half_index(n);
#pragma unroll
        for (int k = 0; k < 12; k++) s[k] = v[k][nh];
        proj<MU, -1>(s, h);
        su3<T> U = ld_link<T, G, NLC>(links, lbase + (long)MU * NLC * VD + loc, VD);
        su3_mul(U, h, uh);
        recon_acc<MU, -1>(acc, uh, scale);
    }
    if (l[MU] > 0) {
        n[MU] = l[MU] - 1;
        int nh = Sh::half_index(n);
        int nloc = (1 - (loc >= Sh::VH)) * Sh::VH + nh;
#pragma unroll
        for (int k = 0; k < 12; k++) s[k] = v[k][nh];
        proj<MU, +1>(s, h);
        su3<T> U = ld_link<T, G, NLC>(links, lbase + (long)MU * NLC * VD + nloc, VD);
        su3_dag_mul(U, h, uh);
        recon_acc<MU, +1>(acc, uh, scale);
    }
}

// A uniform global pointer the compiler must treat as unknown from here on: the
// addresses derived from it are formed at their use instead of being
// precomputed and held in registers across loops.
template <typename P> __device__ __forceinline__ P opaque(P p)
{
    asm volatile("" : "+s"(p));
    return global_ptr(p);
}

// The hop sum of every site of parity po, shared by the site's thread pair:
// the thread of parity po takes directions 0 and 1 of its own site, the thread
// of the other parity with the same half index takes directions 2 and 3 of
// that site (partner coordinates lp, index locp) and hands its partial sum over
// through X ([12][VH] in LDS).  XFREE: nothing reads X during the hops, so the
// partial is written at once; otherwise after a barrier.  Every thread of the
// workgroup calls this (it holds barriers).  The directions are visited in a
// loop that is not unrolled (one direction's temporaries live at a time); the po
// thread's acc (zeroed first if ZERO) gains scale x its share and then the
// helper's; the helper's acc is zeroed and takes its share.
template <class Sh, typename T, typename G, int NLC, bool XFREE, bool ZERO>
__device__ __forceinline__ void pair_hops_rolled(const cx<T> (*v)[Sh::VH], cx<T> (*X)[Sh::VH], int po, int par,
                                                 int hi, const int l[4], int loc, const int lp[4], int locp,
                                                 long lbase, const v2<G> *links, cx<T> acc[12], T scale)
{
    const bool own = par == po, help = par == 1 - po;
    if (ZERO || !own)
#pragma unroll
        for (int k = 0; k < 12; k++) acc[k] = czero<T>();
    if (own || help) {
        int ls[4];
#pragma unroll
        for (int q = 0; q < 4; q++) ls[q] = own ? l[q] : lp[q];
        const int ss = own ? loc : locp;
#pragma unroll 1
        for (int mu = own ? 0 : 2; mu < (own ? 2 : 4); mu++) {
            const v2<G> *lk = opaque(links);
            switch (mu) {
                case 0: dom_hop<Sh, 0, T, G, NLC>(v, ls, lbase, ss, lk, acc, scale); break;
                case 1: dom_hop<Sh, 1, T, G, NLC>(v, ls, lbase, ss, lk, acc, scale); break;
                case 2: dom_hop<Sh, 2, T, G, NLC>(v, ls, lbase, ss, lk, acc, scale); break;
                default: dom_hop<Sh, 3, T, G, NLC>(v, ls, lbase, ss, lk, acc, scale); break;
            }
        }
    }
    if constexpr (XFREE) {
        if (help)
#pragma unroll
            for (int k = 0; k < 12; k++) X[k][hi] = acc[k];
    } else {
        __syncthreads();
        if (help)
#pragma unroll
            for (int k = 0; k < 12; k++) X[k][hi] = acc[k];
    }
    __syncthreads();
    if (own)
#pragma unroll
        for (int k = 0; k < 12; k++) acc[k] = acc[k] + X[k][hi];
}

// ---- boundary terms --------------------------------------------------------

template <class Sh> __device__ __forceinline__ long face_base(int d, int f) { return ((long)d * Sh::FTOT + Sh::foff(f)) * 6; }

// rho += 1/2 phi * (the hop from the neighbouring domain across each face)
template <class Sh, int MU, typename T, typename SS, typename G, int NLC, bool SCALED>
__device__ __forceinline__ void gather_face(const SapArgs &a, const int D[4], int d, const int l[4], int loc,
                                            cx<T> rho[12])
{
    constexpr int VD = Sh::VD;
    const v2<SS> *face = global_ptr((const v2<SS> *)a.face_in);
    int Dn[4] = {D[0], D[1], D[2], D[3]};
    cx<T> h[6];
    if (l[MU] == 0) {
        // backward hop from x - mu, in the -mu neighbour's +mu face
        bool wrap = D[MU] == 0;
        Dn[MU] = wrap ? a.g.n[MU] - 1 : D[MU] - 1;
        int dn = Dn[0] + a.g.n[0] * (Dn[1] + a.g.n[1] * (Dn[2] + a.g.n[2] * Dn[3]));
        T sc = SCALED ? T(global_ptr(a.face_in_scale)[dn]) : T(1);
        long fb = face_base<Sh>(dn, 2 * MU + 1);
        int fi = Sh::template face_index<MU>(l);
#pragma unroll
        for (int k = 0; k < 6; k++) h[k] = scal(sc, ld<T, SS>(face, fb + (long)k * Sh::FS[MU] + fi));
        recon_acc<MU, +1>(rho, h, T(wrap ? 0.5 * a.g.bc[MU] : 0.5));
    } else if (l[MU] == Sh::B[MU] - 1) {
        // forward hop from x + mu, in the +mu neighbour's -mu face
        bool wrap = D[MU] == a.g.n[MU] - 1;
        Dn[MU] = wrap ? 0 : D[MU] + 1;
        int dn = Dn[0] + a.g.n[0] * (Dn[1] + a.g.n[1] * (Dn[2] + a.g.n[2] * Dn[3]));
        T sc = SCALED ? T(global_ptr(a.face_in_scale)[dn]) : T(1);
        long fb = face_base<Sh>(dn, 2 * MU);
        int fi = Sh::template face_index<MU>(l);
#pragma unroll
        for (int k = 0; k < 6; k++) h[k] = scal(sc, ld<T, SS>(face, fb + (long)k * Sh::FS[MU] + fi));
        cx<T> uh[6];
        su3<T> U = ld_link<T, G, NLC>(global_ptr((const v2<G> *)a.links), ((long)d * 4 + MU) * NLC * VD + loc, VD);
        su3_mul(U, h, uh);
        recon_acc<MU, -1>(rho, uh, T(wrap ? 0.5 * a.g.bc[MU] : 0.5));
    }
}

template <class Sh, int MU, typename T, typename SS, typename G, int NLC>
__device__ __forceinline__ void write_face(const SapArgs &a, int d, const int l[4], int loc, const cx<T> delta[12],
                                           T inv_sc)
{
    constexpr int VD = Sh::VD;
    v2<SS> *face = global_ptr((v2<SS> *)a.face);
    cx<T> h[6];
    if (l[MU] == 0) {
        proj<MU, -1>(delta, h);
        long fb = face_base<Sh>(d, 2 * MU);
        int fi = Sh::template face_index<MU>(l);
#pragma unroll
        for (int k = 0; k < 6; k++) st<T, SS>(face, fb + (long)k * Sh::FS[MU] + fi, scal(inv_sc, h[k]));
    } else if (l[MU] == Sh::B[MU] - 1) {
        cx<T> uh[6];
        proj<MU, +1>(delta, h);
        const su3<T> U = ld_link<T, G, NLC>(global_ptr((const v2<G> *)a.links), ((long)d * 4 + MU) * NLC * VD + loc, VD);
        su3_dag_mul(U, h, uh);
        long fb = face_base<Sh>(d, 2 * MU + 1);
        int fi = Sh::template face_index<MU>(l);
#pragma unroll
        for (int k = 0; k < 6; k++) st<T, SS>(face, fb + (long)k * Sh::FS[MU] + fi, scal(inv_sc, uh[k]));
    }
}

// ---- the LDS-resident half-sweep kernels (FP32 arithmetic) ----------------
//
// At the start of the block solve the domain's links are staged once into LDS,
// so the MR steps read no global memory: the hopping terms take the neighbour
// spinor and the link from LDS, the site terms from registers (or, the tile's
// odd sites, from LDS).

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// A spinor of one site and right-hand side in LDS and in the accumulator: six 16-byte entries of two complex components, the entries of one
// component pair contiguous over (site, right-hand side).  16 bytes a lane is
// what LDS moves at its full rate (measured on gfx950: 131 bytes a cycle and CU
// against 67 for 8-byte reads).
typedef f32x4_t c2_t;

template <int STRIDE> __device__ __forceinline__ void ld_c2(const c2_t *p, cx<float> s[12])
{
#pragma unroll
    for (int j = 0; j < 6; j++) {
        const c2_t q = p[j * STRIDE];
        s[2 * j] = {q[0], q[1]};
        s[2 * j + 1] = {q[2], q[3]};
    }
}
template <int STRIDE> __device__ __forceinline__ void st_c2(c2_t *p, const cx<float> s[12])
{
#pragma unroll
    for (int j = 0; j < 6; j++) p[j * STRIDE] = c2_t{s[2 * j].r, s[2 * j].i, s[2 * j + 1].r, s[2 * j + 1].i};
}

// A stored pair of 16-bit values as FP32, converted here: hidden from the
// compiler, so that it does not fold the conversion into mixed-precision
// multiply-adds, which issue at half the rate of FP32 ones (gfx950, two waves
// per SIMD: 4.4 against 2.6 cycles each).  The upper half is shifted down first:
// the conversion that selects it by itself (SDWA) is the slow one.  An SU(3)
// times half-spinor product with the link's nine pairs read from LDS takes 347
// cycles this way, 424 with SDWA conversions, 447 with mixed-precision
// multiply-adds and 299 with FP32 links.
template <typename G> __device__ __forceinline__ cx<float> widen(v2<G> v)
{
    cx<float> c;
    if constexpr (std::is_same<G, half_t>::value) {
        unsigned u = __builtin_bit_cast(unsigned, v), h = u >> 16;
        asm("" : "+v"(h));
        c = {static_cast<float>(__builtin_bit_cast(half_t, (unsigned short)u)),
             static_cast<float>(__builtin_bit_cast(half_t, (unsigned short)h))};
    } else {
        c = {static_cast<float>(v.x), static_cast<float>(v.y)};
    }
    asm("" : "+v"(c.r), "+v"(c.i));
    return c;
}

// out = (packed clover block of 36 pairs, load(q) its pair q) in
template <typename Load> __device__ __forceinline__ void clover_wide(Load load, const cx<float> in[12], cx<float> out[12])
{
    clover_block_with<float>(load, in, out);
    clover_block_with<float>([&](int q) { return load(18 + q); }, in + 6, out + 6);
}

// The block residual of one site in memory: 16-byte entries, [3][VH] of four
// 16-bit complex numbers or [6][VH] of two FP32 ones; scale x the stored values.
template <int VH, typename SS> __device__ __forceinline__ void ld_res(const void *base, long site, float scale, cx<float> s[12])
{
    if constexpr (sizeof(SS) == 2) {
        typedef SS ss8_t __attribute__((ext_vector_type(8)));
        const ss8_t *p = global_ptr((const ss8_t *)base) + site;
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const ss8_t q = p[j * VH];
#pragma unroll
            for (int e = 0; e < 4; e++)
                s[4 * j + e] = {scale * static_cast<float>(q[2 * e]), scale * static_cast<float>(q[2 * e + 1])};
        }
    } else {
        ld_c2<VH>(global_ptr((const c2_t *)base) + site, s);
    }
}
template <int VH, typename SS> __device__ __forceinline__ void st_res(void *base, long site, float inv, const cx<float> s[12])
{
    if constexpr (sizeof(SS) == 2) {
        typedef SS ss8_t __attribute__((ext_vector_type(8)));
        ss8_t *p = global_ptr((ss8_t *)base) + site;
#pragma unroll
        for (int j = 0; j < 3; j++) {
            ss8_t q;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                q[2 * e] = static_cast<SS>(inv * s[4 * j + e].r);
                q[2 * e + 1] = static_cast<SS>(inv * s[4 * j + e].i);
            }
            p[j * VH] = q;
        }
    } else {
        st_c2<VH>(global_ptr((c2_t *)base) + site, s);
    }
}

// A site's links in registers (one right-hand side per workgroup): 16-bit links
// widened to three FP32 rows once at staging, FP32 links as the two stored rows,
// the third rebuilt at each use (its registers go to the FP32 clover block).
template <typename G> struct RegLink {
    su3<float> U;
    __device__ __forceinline__ void put(const v2<G> rows[6])
    {
        U = ld_link_with<float, 6>([&](int e) { return widen<G>(rows[e]); });
        // the third row as the storage type holds it
#pragma unroll
        for (int e = 6; e < 9; e++) {
            v2<G> q;
            q.x = static_cast<G>(U.m[e].r);
            q.y = static_cast<G>(U.m[e].i);
            U.m[e] = widen<G>(q);
        }
    }
    __device__ __forceinline__ su3<float> operator()() const { return U; }
};
template <> struct RegLink<float> {
    float2 m[6];
    __device__ __forceinline__ void put(const float2 rows[6])
    {
#pragma unroll
        for (int e = 0; e < 6; e++) m[e] = rows[e];
    }
    __device__ __forceinline__ su3<float> operator()() const
    {
        return ld_link_with<float, 6>([&](int e) { return cx<float>{m[e].x, m[e].y}; });
    }
};

template <> struct RegLink<double> {
    su3<double> U;
    __device__ __forceinline__ void put(const double2 rows[9])
    {
#pragma unroll
        for (int e = 0; e < 9; e++) U.m[e] = {rows[e].x, rows[e].y};
    }
    __device__ __forceinline__ const su3<double> &operator()() const { return U; }
};

// A domain's 16-bit links in LDS (tiles of right-hand sides) as three rows
// [mu][9][LS], the third rebuilt once at staging; read as FP32 matrices.
template <typename G, int LS> struct LdsLinks {
    const v2<G> *p;
    __device__ __forceinline__ su3<float> operator()(int mu, int site) const
    {
        const v2<G> *q = p + mu * 9 * LS + site;
        su3<float> U;
#pragma unroll
        for (int e = 0; e < 9; e++) U.m[e] = widen<G>(q[e * LS]);
        return U;
    }
    // stages one link from its stored rows
    static __device__ __forceinline__ void put(v2<G> *s, int mu, int site, const v2<G> rows[6])
    {
        const su3<float> U = ld_link<float, G, 6>(rows, 0, 1);
#pragma unroll
        for (int e = 0; e < 9; e++) st<float, G>(s, (mu * 9 + e) * LS + site, U.m[e]);
    }
};

// A site's hop along MU inside the domain; SIGN < 0: from x + mu, SIGN > 0: from
// x - mu.  hop_exists: the neighbour lies in the domain; hop_step: its half
// index relative to the site's (ox: 1 where the site's x is odd), a constant
// except along x.
template <class Sh, int MU, int SIGN> __device__ __forceinline__ bool hop_exists(const int l[4])
{
    return SIGN < 0 ? l[MU] + 1 < Sh::B[MU] : l[MU] > 0;
}
template <class Sh, int MU, int SIGN> __device__ __forceinline__ int hop_step(int ox)
{
    constexpr int STEP = MU == 1 ? Sh::B[0] / 2 : MU == 2 ? Sh::B[0] * Sh::B[1] / 2 : Sh::B[0] * Sh::B[1] * Sh::B[2] / 2;
    return MU == 0 ? (SIGN < 0 ? ox : ox - 1) : SIGN < 0 ? STEP : -STEP;
}

// ---- one right-hand side per workgroup -------------------------------------
//
// One workgroup per domain, one thread per site.  Each thread holds its own
// site's links and clover block (C on even sites, C^-1 on odd sites) in
// registers; x of the even sites and rho/delta of the odd sites stay in the
// registers of the site's own thread, r of the even sites in its LDS entry.
//
// A link is used by its own site's thread only.  In the hop sum of the sites of
// one parity their threads take the forward hops (the neighbour's spinor from
// LDS, their own link), and the threads of the other parity the backward ones:
// each multiplies its own spinor by its own link's adjoint and leaves the half-
// spinor in LDS for the site x + mu.  So both parities' threads work in every
// phase, links need neither LDS nor a conversion at each use, and the LDS
// traffic is that of reading eight neighbour spinors.
// One launch (a colour) with 8x4^3 domains: 45.3 us in FP32 on 16^3x32 (half the
// CUs have one), 377 us with FP16 storage on 32^3x64.  With a pair of threads
// reading all eight neighbours and the links from LDS it took 47.8 and 422 us,
// and 56.4 and 520 us with 8-byte LDS reads, mixed-precision multiply-adds and
// generic loads.  What is left is mostly the issue of FP32 instructions: 8 of 10
// cycles a wave can issue in, at two waves per SIMD (256 registers).
//
// NDW domains share a workgroup (NDW > 1 for domains of fewer than 64 sites):
// wave 0 then holds the even sites and wave 1 the odd sites of all of them,
// so each phase of the even-odd MR step runs one full wave; d is the calling
// thread's domain.

// The forward hop along MU into this site from the other parity's array v
// (at this half index): acc += (1 - gamma_mu) U_mu(x) v(x + mu).
template <class Sh, int MU, typename Link>
__device__ __forceinline__ void lane_fwd(const c2_t *v, const int l[4], int ox, const Link &U, cx<float> acc[12])
{
    if (!hop_exists<Sh, MU, -1>(l)) return;
    cx<float> s[12], h[6], uh[6];
    ld_c2<Sh::VH>(v + hop_step<Sh, MU, -1>(ox), s);
    proj<MU, -1>(s, h);
    su3_mul(U(), h, uh);
    recon_acc<MU, -1>(acc, uh, 1.0f);
}

// X (this half index) = U_mu(x)^dagger (1 + gamma_mu) own, for the site x + mu
template <class Sh, int MU, typename Link>
__device__ __forceinline__ void lane_push(const cx<float> own[12], const int l[4], const Link &U, c2_t *X)
{
    if (!hop_exists<Sh, MU, -1>(l)) return;
    cx<float> h[6], uh[6];
    proj<MU, +1>(own, h);
    su3_dag_mul(U(), h, uh);
#pragma unroll
    for (int j = 0; j < 3; j++) X[(MU * 3 + j) * Sh::VH] = c2_t{uh[2 * j].r, uh[2 * j].i, uh[2 * j + 1].r, uh[2 * j + 1].i};
}

// acc += the half-spinor that x - mu left for this site
template <class Sh, int MU> __device__ __forceinline__ void lane_pull(const c2_t *X, const int l[4], int ox, cx<float> acc[12])
{
    if (!hop_exists<Sh, MU, +1>(l)) return;
    const c2_t *p = X + MU * 3 * Sh::VH + hop_step<Sh, MU, +1>(ox);
    cx<float> uh[6];
#pragma unroll
    for (int j = 0; j < 3; j++) {
        const c2_t q = p[j * Sh::VH];
        uh[2 * j] = {q[0], q[1]};
        uh[2 * j + 1] = {q[2], q[3]};
    }
    recon_acc<MU, +1>(acc, uh, 1.0f);
}

// The hop sum of every site of parity po, in acc of its thread.  v: the other
// parity's spinors in LDS at this half index, own: this thread's own spinor
// (threads of the other parity), X: the half-spinors handed over.  Every thread
// of the workgroup calls this (it holds a barrier, after which v is free); X is
// free after the next one.  HALVES: the forward hops are summed as split_hops
// does, by pairs of directions; the first pair's sum waits in the site's own entry
// of park, which is free after the barrier.
template <class Sh, bool HALVES, typename Link>
__device__ __forceinline__ void lane_hops(const c2_t *v, const cx<float> own[12], c2_t *X, c2_t *park, int po, int par,
                                          const int l[4], const Link (&U)[4], cx<float> acc[12])
{
    const int ox = l[0] & 1;
#pragma unroll
    for (int k = 0; k < 12; k++) acc[k] = czero<float>();
    if (par == po) {
        lane_fwd<Sh, 0>(v, l, ox, U[0], acc);
        lane_fwd<Sh, 1>(v, l, ox, U[1], acc);
        if constexpr (HALVES) {
            st_c2<Sh::VH>(park, acc);
            asm volatile("" ::: "memory");   // read back below, not kept in registers
#pragma unroll
            for (int k = 0; k < 12; k++) acc[k] = czero<float>();
        }
        lane_fwd<Sh, 2>(v, l, ox, U[2], acc);
        lane_fwd<Sh, 3>(v, l, ox, U[3], acc);
        if constexpr (HALVES) {
            cx<float> early[12];
            ld_c2<Sh::VH>(park, early);
#pragma unroll
            for (int k = 0; k < 12; k++) acc[k] = early[k] + acc[k];
        }
    } else if (par == 1 - po) {
        lane_push<Sh, 0>(own, l, U[0], X);
        lane_push<Sh, 1>(own, l, U[1], X);
        lane_push<Sh, 2>(own, l, U[2], X);
        lane_push<Sh, 3>(own, l, U[3], X);
    }
    __syncthreads();
    if (par == po) {
        lane_pull<Sh, 0>(X, l, ox, acc);
        lane_pull<Sh, 1>(X, l, ox, acc);
        lane_pull<Sh, 2>(X, l, ox, acc);
        lane_pull<Sh, 3>(X, l, ox, acc);
    }
}

// The boundary terms of a visit, in two steps so that the loads of every
// direction are in flight together: face_fetch loads the site's boundary
// half-spinor along MU (if it has one) and its weight, face_apply adds its
// contribution.
template <class Sh, int MU, typename T, typename SS, bool SCALED>
__device__ __forceinline__ void face_fetch(const SapArgs &a, const int D[4], const int l[4], cx<T> h[6], T &w, int &side)
{
    const bool bwd = l[MU] == 0, fwd = l[MU] == Sh::B[MU] - 1;
    side = bwd ? 1 : fwd ? 2 : 0;
    if (!(bwd || fwd)) return;
    const v2<SS> *face = global_ptr((const v2<SS> *)a.face_in);
    int Dn[4] = {D[0], D[1], D[2], D[3]};
    const bool wrap = bwd ? D[MU] == 0 : D[MU] == a.g.n[MU] - 1;
    Dn[MU] = bwd ? (wrap ? a.g.n[MU] - 1 : D[MU] - 1) : (wrap ? 0 : D[MU] + 1);
    const int dn = Dn[0] + a.g.n[0] * (Dn[1] + a.g.n[1] * (Dn[2] + a.g.n[2] * Dn[3]));
    // backward hop: the -mu neighbour's +mu face; forward: the +mu neighbour's -mu face
    const long fb = face_base<Sh>(dn, 2 * MU + (bwd ? 1 : 0));
    const int fi = Sh::template face_index<MU>(l);
#pragma unroll
    for (int k = 0; k < 6; k++) h[k] = ld<T, SS>(face, fb + (long)k * Sh::FS[MU] + fi);
    const T sc = SCALED ? T(global_ptr(a.face_in_scale)[dn]) : T(1);
    w = sc * T(wrap ? 0.5 * a.g.bc[MU] : 0.5);
}

template <class Sh, int MU, typename T, typename Link>
__device__ __forceinline__ void face_apply(const Link &U, const cx<T> h[6], T w, int side, cx<T> rho[12])
{
    if (side == 1) {
        recon_acc<MU, +1>(rho, h, w);
    } else if (side == 2) {
        cx<T> uh[6];
        su3_mul(U(), h, uh);
        recon_acc<MU, -1>(rho, uh, w);
    }
}

template <class Sh, int MU, typename T, typename SS, typename Link>
__device__ __forceinline__ void face_write(const SapArgs &a, int d, const int l[4], const cx<T> delta[12], T inv_sc,
                                           const Link &U)
{
    v2<SS> *face = global_ptr((v2<SS> *)a.face);
    cx<T> h[6];
    const bool lo = l[MU] == 0;
    if (!(lo || l[MU] == Sh::B[MU] - 1)) return;
    if (lo) {
        proj<MU, -1>(delta, h);
    } else {
        cx<T> g[6];
        proj<MU, +1>(delta, g);
        su3_dag_mul(U(), g, h);
    }
    const long fb = face_base<Sh>(d, 2 * MU + (lo ? 0 : 1));
    const int fi = Sh::template face_index<MU>(l);
#pragma unroll
    for (int k = 0; k < 6; k++) st<T, SS>(face, fb + (long)k * Sh::FS[MU] + fi, scal(inv_sc, h[k]));
}

// The sums over a domain's sites (one domain a workgroup, its even sites in the
// first half of the NW waves) of the two halves v[0 .. 2] and v[3 .. 5] of three
// values, in the order in which domain_reduce sums them where each half has waves
// of its own.  No closing barrier (see domain_reduce).
template <int NW, typename T> __device__ __forceinline__ void halves_sum(T (&v)[6], T (&out)[3], T *red)
{
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < 6; k++) v[k] = lanes_reduce<64, false>(v[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < 6; k++) red[k * NW + w] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; k++) {
        T s = red[k * NW];
#pragma unroll
        for (int j = 1; j < NW / 2; j++) s += red[k * NW + j];
#pragma unroll
        for (int j = 0; j < NW / 2; j++) s += red[(3 + k) * NW + j];
        out[k] = s;
    }
}

// SS: storage of the block residual and the boundary terms; G: of links (two
// rows) and clover.  The accumulator ([d][6][VD] 16-byte entries, FP32) and the
// block residual are laid out for 16-byte accesses.
// HALVES: every sum in the order of split_block_solve, with the bits that it gives,
// for launches of many systems of small lattices (dd_form.h).  4^4 domains on 16^3x32
// with 12 right-hand sides, 3072 workgroups: 324 us a launch in FP32 and 282 in FP16,
// 14 and 8 % above the kernel's own order, for the first pair's hops going through
// LDS and twice the wave sums; with the pair in registers FP32 spilled 172 bytes and
// took 1.3 times as long.
template <class Sh, int NDW, typename SS, typename G, bool SCALED, bool HALVES>
__device__ __forceinline__ void lds_block_solve(const SapArgs &a, const int d, const Visit f)
{
    using T = float;
    constexpr int VD = Sh::VD, VH = Sh::VH, NLC = 6;
    constexpr int NT = NDW * VD;              // threads of the workgroup
    static_assert(NDW == 1 || NDW * VH == 64, "packed domains: one wave per parity");
    __shared__ c2_t she_all[NDW][6 * VH];     // even sites: r
    __shared__ c2_t sho_all[NDW][6 * VH];     // odd sites: C_o^-1 D_oe r; x in the reconstruction
    __shared__ c2_t shx_all[NDW][4 * 3 * VH]; // half-spinors handed to x + mu
    // FP32 clover blocks leave no registers for A through the MR steps, nor do sums by
    // halves: it waits in LDS (with them, where two workgroups are to share a CU, only
    // the even sites' A; the odd ones' in memory)
    constexpr bool A_LDS = sizeof(v2<G>) == 8 || HALVES;
    constexpr int NA = HALVES ? VH : VD;
    __shared__ c2_t sa_all[A_LDS ? NDW * 6 * NA : 1];
    __shared__ c2_t park_all[HALVES ? 6 * VH : 1];
    constexpr int NW = NT / 64;
    static_assert(NT % 64 == 0, "whole waves");
    static_assert(!HALVES || (NDW == 1 && VH % 64 == 0), "halves: one domain a workgroup, whole waves of each parity");
    __shared__ T red[2][(HALVES ? 6 : 3) * NW * NDW];

    const int par = (int)threadIdx.x / (NDW * VH);
    const int idx = (int)threadIdx.x - par * (NDW * VH);
    const int sub = idx / VH;   // this thread's domain within the workgroup
    const int hi = idx - sub * VH;
    const int loc = par * VH + hi;
    // this half index
    c2_t *const ve = she_all[sub] + hi, *const vo = sho_all[sub] + hi, *const vx = shx_all[sub] + hi;
    c2_t *const vp = park_all + (HALVES ? hi : 0);
    int l[4];
    Sh::coords(loc, l);
    int D[4];
    {
        int r = d;
        D[0] = r % a.g.n[0]; r /= a.g.n[0];
        D[1] = r % a.g.n[1]; r /= a.g.n[1];
        D[2] = r % a.g.n[2];
        D[3] = r / a.g.n[2];
    }
    const v2<G> *glinks = global_ptr((const v2<G> *)a.links);
    const v2<G> *cs = global_ptr((const v2<G> *)a.cs);
    const long sbase = (long)d * 12 * VD + loc;
    c2_t *const psi = global_ptr((c2_t *)a.psi) + (long)d * 6 * VD + loc;
    const long rbase = (long)d * (sizeof(SS) == 2 ? 3 : 6) * VH + hi;

    // ---- the site's links and clover block and the block right-hand side
    // A: even sites x (MR solution), odd sites rho_o then delta_o
    cx<T> A[12], P[12];
    v2<G> lt[4][NLC], cl[36];
    const long lb = (long)d * 4 * NLC * VD + loc;
#pragma unroll
    for (int q = 0; q < 4 * NLC; q++) lt[q / NLC][q % NLC] = glinks[lb + (long)q * VD];
    if (f.first) {
        if (a.io32) {
#pragma unroll
            for (int k = 0; k < 12; k++) A[k] = ld<T, float>(global_ptr((const float2 *)a.eta), sbase + (long)k * VD);
        } else {
#pragma unroll
            for (int k = 0; k < 12; k++) A[k] = ld<T, double>(global_ptr(a.eta), sbase + (long)k * VD);
        }
    } else if (par == 0) {
        ld_res<VH, SS>(a.res, rbase, SCALED ? T(global_ptr(a.res_scale)[d]) : T(1), A);
    } else {
#pragma unroll
        for (int k = 0; k < 12; k++) A[k] = czero<T>();
    }
    cx<T> hf[4][6];
    T wf[4] = {0, 0, 0, 0};
    int sf[4] = {0, 0, 0, 0};
    if (f.faces_in) {
        face_fetch<Sh, 0, T, SS, SCALED>(a, D, l, hf[0], wf[0], sf[0]);
        face_fetch<Sh, 1, T, SS, SCALED>(a, D, l, hf[1], wf[1], sf[1]);
        face_fetch<Sh, 2, T, SS, SCALED>(a, D, l, hf[2], wf[2], sf[2]);
        face_fetch<Sh, 3, T, SS, SCALED>(a, D, l, hf[3], wf[3], sf[3]);
    }
    const long cbase = (long)d * 36 * VD + loc;
#pragma unroll
    for (int q = 0; q < 36; q++) cl[q] = cs[cbase + (long)q * VD];
    RegLink<G> U[4];
#pragma unroll
    for (int mu = 0; mu < 4; mu++) U[mu].put(lt[mu]);
    // this site's clover block (C_e on even sites, C_o^-1 on odd sites) times in
    auto clover = [&](const cx<T> in[12], cx<T> out[12]) {
        if constexpr (sizeof(v2<G>) == 4) clover_wide([&](int q) { return widen<G>(cl[q]); }, in, out);
        else clover_wide([&](int q) { return cx<T>{(T)cl[q].x, (T)cl[q].y}; }, in, out);
    };
    if (f.faces_in) {
        if constexpr (HALVES) {
            cx<T> early[12], late[12];
#pragma unroll
            for (int k = 0; k < 12; k++) early[k] = late[k] = czero<T>();
            face_apply<Sh, 0, T>(U[0], hf[0], wf[0], sf[0], early);
            face_apply<Sh, 1, T>(U[1], hf[1], wf[1], sf[1], early);
            face_apply<Sh, 2, T>(U[2], hf[2], wf[2], sf[2], late);
            face_apply<Sh, 3, T>(U[3], hf[3], wf[3], sf[3], late);
#pragma unroll
            for (int k = 0; k < 12; k++) A[k] = A[k] + (early[k] + late[k]);
        } else {
            face_apply<Sh, 0, T>(U[0], hf[0], wf[0], sf[0], A);
            face_apply<Sh, 1, T>(U[1], hf[1], wf[1], sf[1], A);
            face_apply<Sh, 2, T>(U[2], hf[2], wf[2], sf[2], A);
            face_apply<Sh, 3, T>(U[3], hf[3], wf[3], sf[3], A);
        }
    }

    // ---- even-odd preparation: r = rho_e - D_eo C_o^-1 rho_o, x = 0
    if (par == 1) {
        clover(A, P);
        st_c2<VH>(vo, P);
    }
    __syncthreads();
    // the even-site MR residual r lives in its own slot of she for the whole
    // solve (fewer live registers); x stays in the registers of A
    cx<T> t[12];
    lane_hops<Sh, HALVES>(vo, P, vx, vp, 0, par, l, U, t);
    if (par == 0) {
#pragma unroll
        for (int k = 0; k < 12; k++) {
            P[k] = A[k] + scal(T(0.5), t[k]);
            A[k] = czero<T>();
        }
        st_c2<VH>(ve, P);
    }
    c2_t *const va = sa_all + (A_LDS ? sub * 6 * NA + (HALVES ? hi : loc) : 0);
    v2<T> *const rho_g = global_ptr((v2<T> *)a.rho_tmp) + (long)d * 12 * VH + hi;
    if (HALVES && par == 1) {
#pragma unroll
        for (int k = 0; k < 12; k++) st<T, T>(rho_g, (long)k * VH, A[k]);
    } else if (A_LDS) {
        st_c2<NA>(va, A);
    }
    // C has arrived: without this, a path around the MR loop on which it has
    // not makes the later waits for its registers wait for younger loads
#pragma unroll
    for (int q = 0; q < 36; q++) {
        if constexpr (sizeof(v2<G>) == 4) asm volatile("" : "+v"(cl[q]));
        else asm volatile("" : "+v"(cl[q].x), "+v"(cl[q].y));
    }

    // ---- minimal residual on the Schur complement
#pragma unroll 1
    for (int it = 0; it < a.n_mr; it++) {
        if constexpr (sizeof(v2<G>) == 4) {
            // keep the clover block in its 16-bit storage form: stops the
            // compiler from hoisting its widening out of the loop, which would
            // double the registers it occupies
#pragma unroll
            for (int q = 0; q < 36; q++) asm volatile("" : "+v"(cl[q]));
        }
        __syncthreads();
        if (par == 0) ld_c2<VH>(ve, P);
        lane_hops<Sh, HALVES>(ve, P, vx, vp, 1, par, l, U, t);       // -2 D_oe r
        if (par == 1) {
            clover(t, P);                                // -2 C_o^-1 D_oe r
            st_c2<VH>(vo, P);
        } else if (par == 0) {
            // meanwhile the even sites form C_e r, which needs only r
            ld_c2<VH>(ve, t);
            clover(t, P);
        }
        __syncthreads();
        T dots[3] = {0, 0, 0}, half[6] = {0, 0, 0, 0, 0, 0};
        lane_hops<Sh, HALVES>(vo, P, vx, vp, 0, par, l, U, t);
        cx<T> rr[12];
        if (par == 0) {
            ld_c2<VH>(ve, rr);
#pragma unroll
            for (int k = 0; k < 12; k++) {
                P[k] = P[k] + scal(T(-0.25), t[k]);      // p = C_e r - D_eo C_o^-1 D_oe r
                T *const s = HALVES ? half + k / 6 * 3 : dots;
                s[0] = fmad(P[k].i, rr[k].i, fmad(P[k].r, rr[k].r, s[0]));
                s[1] = fmad(-P[k].i, rr[k].r, fmad(P[k].r, rr[k].i, s[1]));
                s[2] = fmad(P[k].i, P[k].i, fmad(P[k].r, P[k].r, s[2]));
            }
        }
        if constexpr (HALVES) halves_sum<NW>(half, dots, red[0]);
        else domain_reduce<VH, NDW, NW, false>(dots, red[0], sub);
        if (par == 0) {
            cx<T> alpha = dots[2] > T(0) ? cx<T>{dots[0] / dots[2], dots[1] / dots[2]} : czero<T>();
            if (A_LDS) ld_c2<NA>(va, A);
#pragma unroll
            for (int k = 0; k < 12; k++) {
                A[k] = cmac(A[k], alpha, rr[k]);
                P[k] = cmac(rr[k], neg(alpha), P[k]);
            }
            if (A_LDS) st_c2<NA>(va, A);
            st_c2<VH>(ve, P);
        }
    }

    // ---- odd sites: delta_o = C_o^-1 (rho_o - D_oe x); x goes through sho
    // (free since the last reduction), she keeps r for the epilogue.  The
    // accumulator is fetched ahead of it.
    c2_t ps[6];
#pragma unroll
    for (int j = 0; j < 6; j++) ps[j] = c2_t{0.f, 0.f, 0.f, 0.f};
    if (HALVES && par == 1) {
#pragma unroll
        for (int k = 0; k < 12; k++) A[k] = ld<T, T>(rho_g, (long)k * VH);
    } else if (A_LDS) {
        ld_c2<NA>(va, A);
    }
    if (par == 0) st_c2<VH>(vo, A);
    if (!f.first)
#pragma unroll
        for (int j = 0; j < 6; j++) ps[j] = psi[j * VD];
    __syncthreads();
    lane_hops<Sh, HALVES>(vo, A, vx, vp, 1, par, l, U, t);
    if (par == 1) {
#pragma unroll
        for (int k = 0; k < 12; k++) t[k] = A[k] + scal(T(0.5), t[k]);
        clover(t, A);
    }

    // ---- epilogue
#pragma unroll
    for (int j = 0; j < 6; j++) ps[j] += c2_t{A[2 * j].r, A[2 * j].i, A[2 * j + 1].r, A[2 * j + 1].i};
    if (f.last) {
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const cx<T> c = {ps[k / 2][2 * (k & 1)], ps[k / 2][2 * (k & 1) + 1]};
            if (a.io32) st<T, float>(global_ptr((float2 *)a.out), sbase + (long)k * VD, c);
            else st<T, double>(global_ptr(a.out), sbase + (long)k * VD, c);
        }
    } else {
#pragma unroll
        for (int j = 0; j < 6; j++) psi[j * VD] = ps[j];
    }
    T mx[2] = {T(1), T(1)};
    if constexpr (SCALED) {
        if (!f.res_out && !f.faces_out) return;
        cx<T> rr[12];
#pragma unroll
        for (int k = 0; k < 12; k++) rr[k] = czero<T>();
        if (par == 0) ld_c2<VH>(ve, rr);
        mx[0] = maxabs12(rr);
        mx[1] = maxabs12(A);
        domain_reduce<VH, NDW, NW, true>(mx, red[1], sub);
        mx[0] = pow2_ceil(mx[0]);
        mx[1] = T(8) * pow2_ceil(mx[1]);
        if (f.res_out) {
            if (loc == 0) global_ptr(a.res_scale)[d] = (float)mx[0];
            if (par == 0) st_res<VH, SS>(a.res, rbase, T(1) / mx[0], rr);
        }
    } else if (f.res_out && par == 0) {
        cx<T> rr[12];
        ld_c2<VH>(ve, rr);
        st_res<VH, SS>(a.res, rbase, T(1), rr);
    }
    if (f.faces_out) {
        if (SCALED && loc == 0) global_ptr(a.face_scale)[d] = (float)mx[1];
        const T inv = T(1) / mx[1];
        face_write<Sh, 0, T, SS>(a, d, l, A, inv, U[0]);
        face_write<Sh, 1, T, SS>(a, d, l, A, inv, U[1]);
        face_write<Sh, 2, T, SS>(a, d, l, A, inv, U[2]);
        face_write<Sh, 3, T, SS>(a, d, l, A, inv, U[3]);
    }
}


// ---- one right-hand side per workgroup, two threads per site --------------------
//
// The schedule of lds_block_solve for lattices whose colour does not fill the
// device with one thread per site (a launch then lasts as long as one block
// solve), for 6x6x2x4 domains and for FP64 on 2^4 domains (dd_form.h).  Thread (parity, q, half index) holds the
// site's links of directions 2q and 2q + 1 and its clover block q (the spinor's
// components 6q .. 6q + 5, on which C is block diagonal), and owns that half of
// x, r, rho and delta: it takes the forward or backward hops of its directions,
// hands the other half of its partial sum to its twin through LDS, and gathers
// its half of the backward hops of all four directions.  The four groups of
// threads are whole waves, so no wave diverges.
// A block solve is then half as long a chain of instructions per thread, and
// a CU with one workgroup has two waves per SIMD instead of one (one wave
// issues an FP32 instruction every 5.2 cycles, two every 2.6).  Launches of one
// colour: 33.7 us against 40.5 (FP16, 4^4 domains, 16^3x32), about 37 against 58
// (FP32, 6x6x2x4 domains, 12^3x24: 72 workgroups), and in FP64 on 2^4 domains
// 78.6 us against 681 on 16^3x32 (eight threads per domain, links and clover
// blocks read from memory at each use).
// Spinors of precision T in LDS and memory: 16-byte entries of two FP32 or one
// FP64 complex number.
template <typename T> struct SpEntry {
    typedef c2_t type;
    static constexpr int N = 2;   // complex numbers per entry
    static __device__ __forceinline__ c2_t make(const cx<float> *s) { return c2_t{s[0].r, s[0].i, s[1].r, s[1].i}; }
    static __device__ __forceinline__ void split(const c2_t &e, cx<float> *s)
    {
        s[0] = {e[0], e[1]};
        s[1] = {e[2], e[3]};
    }
};
template <> struct SpEntry<double> {
    typedef double2 type;
    static constexpr int N = 1;
    static __device__ __forceinline__ double2 make(const cx<double> *s) { return make_double2(s[0].r, s[0].i); }
    static __device__ __forceinline__ void split(const double2 &e, cx<double> *s) { s[0] = {e.x, e.y}; }
};
// components 0 .. NC - 1 from entries p[0], p[STRIDE], ...
template <int STRIDE, int NC, typename T> __device__ __forceinline__ void ld_sp(const typename SpEntry<T>::type *p, cx<T> *s)
{
#pragma unroll
    for (int j = 0; j < NC / SpEntry<T>::N; j++) SpEntry<T>::split(p[j * STRIDE], s + j * SpEntry<T>::N);
}
template <int STRIDE, int NC, typename T> __device__ __forceinline__ void st_sp(typename SpEntry<T>::type *p, const cx<T> *s)
{
#pragma unroll
    for (int j = 0; j < NC / SpEntry<T>::N; j++) p[j * STRIDE] = SpEntry<T>::make(s + j * SpEntry<T>::N);
}

// the spin halves of recon_acc: out (components 6q .. 6q + 5) += the half q of
// the spinor whose projection is h
template <int Q, int MU, int SG, typename T> __device__ __forceinline__ void recon_half(cx<T> out[6], const cx<T> h[6])
{
#pragma unroll
    for (int c = 0; c < 3; c++) {
        if constexpr (Q == 0) {
            out[c] = out[c] + h[c];
            out[3 + c] = out[3 + c] + h[3 + c];
        } else if constexpr (MU == 0) {
            out[c] = out[c] + (SG < 0 ? times_mi(h[3 + c]) : times_i(h[3 + c]));
            out[3 + c] = out[3 + c] + (SG < 0 ? times_mi(h[c]) : times_i(h[c]));
        } else if constexpr (MU == 1) {
            out[c] = SG < 0 ? out[c] - h[3 + c] : out[c] + h[3 + c];
            out[3 + c] = SG < 0 ? out[3 + c] + h[c] : out[3 + c] - h[c];
        } else if constexpr (MU == 2) {
            out[c] = out[c] + (SG < 0 ? times_mi(h[c]) : times_i(h[c]));
            out[3 + c] = out[3 + c] + (SG < 0 ? times_i(h[3 + c]) : times_mi(h[3 + c]));
        } else {
            out[c] = SG < 0 ? out[c] + h[c] : out[c] - h[c];
            out[3 + c] = SG < 0 ? out[3 + c] + h[3 + c] : out[3 + c] - h[3 + c];
        }
    }
}

// One direction's forward hop, push and pull, as lane_fwd, lane_push, lane_pull.
template <class Sh, int MU, typename T, typename Link>
__device__ __forceinline__ void split_fwd(const typename SpEntry<T>::type *v, const int l[4], int ox, const Link &U, cx<T> acc[12])
{
    if (!hop_exists<Sh, MU, -1>(l)) return;
    cx<T> s[12], h[6], uh[6];
    ld_sp<Sh::VH, 12, T>(v + hop_step<Sh, MU, -1>(ox), s);
    proj<MU, -1>(s, h);
    su3_mul(U(), h, uh);
    recon_acc<MU, -1>(acc, uh, T(1));
}
template <class Sh, int MU, typename T, typename Link>
__device__ __forceinline__ void split_push(const cx<T> own[12], const int l[4], const Link &U, typename SpEntry<T>::type *X)
{
    if (!hop_exists<Sh, MU, -1>(l)) return;
    cx<T> h[6], uh[6];
    proj<MU, +1>(own, h);
    su3_dag_mul(U(), h, uh);
    st_sp<Sh::VH, 6, T>(X + MU * (6 / SpEntry<T>::N) * Sh::VH, uh);
}
template <class Sh, int Q, int MU, typename T>
__device__ __forceinline__ void split_pull(const typename SpEntry<T>::type *X, const int l[4], int ox, cx<T> half[6])
{
    if (!hop_exists<Sh, MU, +1>(l)) return;
    cx<T> uh[6];
    ld_sp<Sh::VH, 6, T>(X + MU * (6 / SpEntry<T>::N) * Sh::VH + hop_step<Sh, MU, +1>(ox), uh);
    recon_half<Q, MU, +1>(half, uh);
}
template <class Sh, int Q, typename T>
__device__ __forceinline__ void split_pulls(const typename SpEntry<T>::type *X, const int l[4], int ox, cx<T> half[6])
{
    split_pull<Sh, Q, 0, T>(X, l, ox, half);
    split_pull<Sh, Q, 1, T>(X, l, ox, half);
    split_pull<Sh, Q, 2, T>(X, l, ox, half);
    split_pull<Sh, Q, 3, T>(X, l, ox, half);
}

// The hop sum of the sites of parity po: this thread's half of it where par ==
// po.  v, own: the other parity's spinors in LDS at this half index and at this
// thread's own site (the same pointer); X, E: handed-over half-spinors and
// twin's halves.  Holds one barrier, after which v is free; X and E are free
// after the next one.
template <class Sh, typename T, typename Link>
__device__ __forceinline__ void split_hops(const typename SpEntry<T>::type *v, typename SpEntry<T>::type *X,
                                           typename SpEntry<T>::type *E, int po, int par, int q, bool live, const int l[4],
                                           const Link (&U)[2], cx<T> half[6])
{
    constexpr int VH = Sh::VH, HE = 6 / SpEntry<T>::N * VH;   // entries of a half
    const int ox = l[0] & 1;
#pragma unroll
    for (int k = 0; k < 6; k++) half[k] = czero<T>();
    if (live && par == po) {
        cx<T> acc[12];
#pragma unroll
        for (int k = 0; k < 12; k++) acc[k] = czero<T>();
        if (q == 0) {
            split_fwd<Sh, 0, T>(v, l, ox, U[0], acc);
            split_fwd<Sh, 1, T>(v, l, ox, U[1], acc);
            st_sp<VH, 6, T>(E + HE, acc + 6);
#pragma unroll
            for (int k = 0; k < 6; k++) half[k] = acc[k];
        } else {
            split_fwd<Sh, 2, T>(v, l, ox, U[0], acc);
            split_fwd<Sh, 3, T>(v, l, ox, U[1], acc);
            st_sp<VH, 6, T>(E, acc);
#pragma unroll
            for (int k = 0; k < 6; k++) half[k] = acc[6 + k];
        }
    } else if (live) {
        cx<T> own[12];
        ld_sp<VH, 12, T>(v, own);
        if (q == 0) {
            split_push<Sh, 0, T>(own, l, U[0], X);
            split_push<Sh, 1, T>(own, l, U[1], X);
        } else {
            split_push<Sh, 2, T>(own, l, U[0], X);
            split_push<Sh, 3, T>(own, l, U[1], X);
        }
    }
    __syncthreads();
    if (live && par == po) {
        cx<T> o[6];
        ld_sp<VH, 6, T>(E + q * HE, o);
#pragma unroll
        for (int k = 0; k < 6; k++) half[k] = half[k] + o[k];
        if (q == 0) split_pulls<Sh, 0, T>(X, l, ox, half);
        else split_pulls<Sh, 1, T>(X, l, ox, half);
    }
}

template <class Sh, int NDW> struct SplitShape {
    static constexpr int GP = (NDW * Sh::VH + 63) / 64 * 64;   // threads of one (parity, q)
    static constexpr int NT = 4 * GP;
    // waves per SIMD the registers are divided among (FP64: all for one)
    template <typename T> static constexpr int waves() { return NT / 64 >= 12 ? 3 : sizeof(T) == 8 ? 1 : 2; }
};

// T: arithmetic; SS: storage of the block residual and boundary terms; G: of
// links and clover.  The accumulator has precision T.
template <class Sh, int NDW, typename T, typename SS, typename G, bool SCALED>
__device__ __forceinline__ void split_block_solve(const SapArgs &a, const int d, const int sub, const Visit f)
{
    constexpr int VD = Sh::VD, VH = Sh::VH, GP = SplitShape<Sh, NDW>::GP, NW = SplitShape<Sh, NDW>::NT / 64;
    constexpr int NLC = sizeof(G) == 8 ? 9 : 6;   // FP64 links are stored whole
    typedef SpEntry<T> E;
    typedef typename E::type e_t;
    constexpr int HE = 6 / E::N * VH, FE = 2 * HE;   // entries of half a spinor array, of a whole one
    // FP64 clover blocks: LDS, read at each use (FP32 and 16-bit ones: registers)
    constexpr bool CL_LDS = sizeof(G) == 8;
    __shared__ e_t se_all[NDW][FE], so_all[NDW][FE], sx_all[NDW][2 * FE], sE_all[NDW][FE];
    __shared__ v2<G> scl_all[CL_LDS ? 4 * 18 * GP : 1];
    __shared__ T red[2][3 * NW * NDW];

    const int grp = __builtin_amdgcn_readfirstlane((int)threadIdx.x / GP);   // whole waves
    const int par = grp >> 1, q = grp & 1, idx = (int)threadIdx.x - grp * GP;
    const bool live = idx < NDW * VH;
    const int hi = live ? idx % VH : 0, loc = par * VH + hi;
    e_t *const ve = se_all[sub] + hi, *const vo = so_all[sub] + hi, *const vx = sx_all[sub] + hi, *const vE = sE_all[sub] + hi;
    int l[4];
    Sh::coords(loc, l);
    int D[4];
    {
        int r = d;
        D[0] = r % a.g.n[0]; r /= a.g.n[0];
        D[1] = r % a.g.n[1]; r /= a.g.n[1];
        D[2] = r % a.g.n[2];
        D[3] = r / a.g.n[2];
    }
    const long sbase = ((long)d * 12 + 6 * q) * VD + loc;

    // ---- this thread's links, clover block and half of the right-hand side
    cx<T> A[6], P[6];   // A: even sites x, odd sites rho_o then delta_o
    v2<G> lt[2][NLC], cl[18];
    {
        const v2<G> *gl = global_ptr((const v2<G> *)a.links) + ((long)d * 4 + 2 * q) * NLC * VD + loc;
        const v2<G> *cs = global_ptr((const v2<G> *)a.cs) + ((long)d * 36 + 18 * q) * VD + loc;
#pragma unroll
        for (int k = 0; k < 2 * NLC; k++) lt[k / NLC][k % NLC] = gl[(long)k * VD];
#pragma unroll
        for (int k = 0; k < 18; k++) cl[k] = cs[(long)k * VD];
    }
    const e_t *const psi_in = global_ptr((const e_t *)a.psi) + ((long)d * (12 / E::N) + q * (6 / E::N)) * VD + loc;
    e_t *const psi_out = const_cast<e_t *>(psi_in);
    v2<SS> *const res = global_ptr((v2<SS> *)a.res) + (long)d * 12 * VH + hi * E::N + q * 6 * VH;   // see below
#pragma unroll
    for (int k = 0; k < 6; k++) A[k] = czero<T>();
    if (f.first) {
        if (a.io32) {
#pragma unroll
            for (int k = 0; k < 6; k++) A[k] = ld<T, float>(global_ptr((const float2 *)a.eta), sbase + (long)k * VD);
        } else {
#pragma unroll
            for (int k = 0; k < 6; k++) A[k] = ld<T, double>(global_ptr(a.eta), sbase + (long)k * VD);
        }
    } else if (par == 0) {
        // stored as the LDS entries are: E::N consecutive components at a time
        const T sc = SCALED ? T(global_ptr(a.res_scale)[d]) : T(1);
#pragma unroll
        for (int k = 0; k < 6; k++) A[k] = scal(sc, ld<T, SS>(res, (long)(k / E::N) * E::N * VH + k % E::N));
    }
    RegLink<G> U[2];
    U[0].put(lt[0]);
    U[1].put(lt[1]);
    if constexpr (CL_LDS) {
#pragma unroll
        for (int k = 0; k < 18; k++) scl_all[k * 4 * GP + threadIdx.x] = cl[k];
    }
    auto clover = [&](const cx<T> in[6], cx<T> out[6]) {
        if constexpr (CL_LDS) clover_block_with<T>([&](int k) { return ld<T, G>(scl_all, k * 4 * GP + (int)threadIdx.x); }, in, out);
        else if constexpr (sizeof(v2<G>) == 4) clover_block_with<T>([&](int k) { return widen<G>(cl[k]); }, in, out);
        else clover_block_with<T>([&](int k) { return cx<T>{(T)cl[k].x, (T)cl[k].y}; }, in, out);
    };
    // the boundary terms of directions 2q and 2q + 1; the twin's half goes
    // through vx, which holds a whole spinor for each parity
    if (f.faces_in) {
        cx<T> rho[12];
#pragma unroll
        for (int k = 0; k < 12; k++) rho[k] = czero<T>();
        if (live) {
            cx<T> hf[2][6];
            T wf[2] = {0, 0};
            int sf[2] = {0, 0};
            if (q == 0) {
                face_fetch<Sh, 0, T, SS, SCALED>(a, D, l, hf[0], wf[0], sf[0]);
                face_fetch<Sh, 1, T, SS, SCALED>(a, D, l, hf[1], wf[1], sf[1]);
                face_apply<Sh, 0, T>(U[0], hf[0], wf[0], sf[0], rho);
                face_apply<Sh, 1, T>(U[1], hf[1], wf[1], sf[1], rho);
                st_sp<VH, 6, T>(vx + par * FE + HE, rho + 6);
            } else {
                face_fetch<Sh, 2, T, SS, SCALED>(a, D, l, hf[0], wf[0], sf[0]);
                face_fetch<Sh, 3, T, SS, SCALED>(a, D, l, hf[1], wf[1], sf[1]);
                face_apply<Sh, 2, T>(U[0], hf[0], wf[0], sf[0], rho);
                face_apply<Sh, 3, T>(U[1], hf[1], wf[1], sf[1], rho);
                st_sp<VH, 6, T>(vx + par * FE, rho);
            }
        }
        __syncthreads();
        if (live) {
            cx<T> o[6];
            ld_sp<VH, 6, T>(vx + par * FE + q * HE, o);
#pragma unroll
            for (int k = 0; k < 6; k++) A[k] = A[k] + ((q == 0 ? rho[k] : rho[6 + k]) + o[k]);
        }
    }

    // ---- even-odd preparation: r = rho_e - D_eo C_o^-1 rho_o, x = 0
    if (par == 1) {
        clover(A, P);
        if (live) st_sp<VH, 6, T>(vo + q * HE, P);
    }
    __syncthreads();
    cx<T> t[6];
    split_hops<Sh, T>(vo, vx, vE, 0, par, q, live, l, U, t);
    if (par == 0) {
#pragma unroll
        for (int k = 0; k < 6; k++) {
            P[k] = A[k] + scal(T(0.5), t[k]);
            A[k] = czero<T>();
        }
        if (live) st_sp<VH, 6, T>(ve + q * HE, P);
    }

    // ---- minimal residual on the Schur complement
#pragma unroll 1
    for (int it = 0; it < a.n_mr; it++) {
        if constexpr (sizeof(v2<G>) == 4) {
            // keep the clover block in its 16-bit storage form (see lds_block_solve)
#pragma unroll
            for (int k = 0; k < 18; k++) asm volatile("" : "+v"(cl[k]));
        }
        __syncthreads();
        split_hops<Sh, T>(ve, vx, vE, 1, par, q, live, l, U, t);   // -2 D_oe r
        cx<T> rr[6];
        if (par == 1) {
            clover(t, P);                                // -2 C_o^-1 D_oe r
            if (live) st_sp<VH, 6, T>(vo + q * HE, P);
        } else {
            // meanwhile the even sites form C_e r, which needs only r
            ld_sp<VH, 6, T>(ve + q * HE, rr);
            clover(rr, P);
        }
        __syncthreads();
        T dots[3] = {0, 0, 0};
        split_hops<Sh, T>(vo, vx, vE, 0, par, q, live, l, U, t);
        if (par == 0 && live) {
#pragma unroll
            for (int k = 0; k < 6; k++) {
                P[k] = P[k] + scal(T(-0.25), t[k]);      // p = C_e r - D_eo C_o^-1 D_oe r
                dots[0] = fmad(P[k].i, rr[k].i, fmad(P[k].r, rr[k].r, dots[0]));
                dots[1] = fmad(-P[k].i, rr[k].r, fmad(P[k].r, rr[k].i, dots[1]));
                dots[2] = fmad(P[k].i, P[k].i, fmad(P[k].r, P[k].r, dots[2]));
            }
        }
        domain_reduce<VH, NDW, NW, false>(dots, red[0], sub);
        if (par == 0) {
            const cx<T> alpha = dots[2] > T(0) ? cx<T>{dots[0] / dots[2], dots[1] / dots[2]} : czero<T>();
#pragma unroll
            for (int k = 0; k < 6; k++) {
                A[k] = cmac(A[k], alpha, rr[k]);
                P[k] = cmac(rr[k], neg(alpha), P[k]);
            }
            if (live) st_sp<VH, 6, T>(ve + q * HE, P);
        }
    }

    // ---- odd sites: delta_o = C_o^-1 (rho_o - D_oe x); x goes through so, se
    // keeps r for the epilogue.  The accumulator is fetched ahead of it.
    e_t ps[6 / E::N];
    {
        const cx<T> z[2] = {czero<T>(), czero<T>()};
#pragma unroll
        for (int j = 0; j < 6 / E::N; j++) ps[j] = E::make(z);
    }
    if (par == 0 && live) st_sp<VH, 6, T>(vo + q * HE, A);
    if (!f.first)
#pragma unroll
        for (int j = 0; j < 6 / E::N; j++) ps[j] = psi_in[(long)j * VD];
    __syncthreads();
    split_hops<Sh, T>(vo, vx, vE, 1, par, q, live, l, U, t);
    if (par == 1) {
#pragma unroll
        for (int k = 0; k < 6; k++) t[k] = A[k] + scal(T(0.5), t[k]);
        clover(t, A);
    }

    // ---- epilogue: psi += delta, stored residual, boundary terms
    if (live) {
        cx<T> c[6];
#pragma unroll
        for (int j = 0; j < 6 / E::N; j++) E::split(ps[j], c + j * E::N);
#pragma unroll
        for (int k = 0; k < 6; k++) c[k] = c[k] + A[k];
        if (f.last) {
#pragma unroll
            for (int k = 0; k < 6; k++) {
                if (a.io32) st<T, float>(global_ptr((float2 *)a.out), sbase + (long)k * VD, c[k]);
                else st<T, double>(global_ptr(a.out), sbase + (long)k * VD, c[k]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 6 / E::N; j++) psi_out[(long)j * VD] = E::make(c + j * E::N);
        }
    }
    if (!f.res_out && !f.faces_out) return;
    cx<T> rr[6];
#pragma unroll
    for (int k = 0; k < 6; k++) rr[k] = czero<T>();
    if (par == 0 && live) ld_sp<VH, 6, T>(ve + q * HE, rr);
    T mx[2] = {0, 0};
    if constexpr (SCALED) {
#pragma unroll
        for (int k = 0; k < 6; k++) {
            mx[0] = fmax(mx[0], fmax(fabs(rr[k].r), fabs(rr[k].i)));
            mx[1] = fmax(mx[1], fmax(fabs(A[k].r), fabs(A[k].i)));
        }
        if (!live) mx[1] = 0;
        T m[2] = {mx[0], mx[1]};
        domain_reduce<VH, NDW, NW, true>(m, red[1], sub);
        mx[0] = pow2_ceil(m[0]);
        mx[1] = T(8) * pow2_ceil(m[1]);
    } else {
        mx[0] = mx[1] = T(1);
        __syncthreads();   // the reconstruction's hops have read so
    }
    if (f.res_out && par == 0 && live) {
        if (SCALED && hi == 0 && q == 0) global_ptr(a.res_scale)[d] = (float)mx[0];
        const T inv = T(1) / mx[0];
#pragma unroll
        for (int k = 0; k < 6; k++) st<T, SS>(res, (long)(k / E::N) * E::N * VH + k % E::N, scal(inv, rr[k]));
    }
    if (f.faces_out) {
        if (SCALED && loc == 0 && q == 0 && live) global_ptr(a.face_scale)[d] = (float)mx[1];
        const T inv = T(1) / mx[1];
        e_t *const vd = par == 0 ? ve : vo;
        if (live) st_sp<VH, 6, T>(vd + q * HE, A);
        __syncthreads();
        if (live) {
            cx<T> delta[12];
            ld_sp<VH, 12, T>(vd, delta);
            if (q == 0) {
                face_write<Sh, 0, T, SS>(a, d, l, delta, inv, U[0]);
                face_write<Sh, 1, T, SS>(a, d, l, delta, inv, U[1]);
            } else {
                face_write<Sh, 2, T, SS>(a, d, l, delta, inv, U[0]);
                face_write<Sh, 3, T, SS>(a, d, l, delta, inv, U[1]);
            }
        }
    }
}


// ---- the FP64 block solve for domains of 256 and more sites -------------------
//
// The same schedule as lds_block_solve (one workgroup per domain, one thread
// per site, Schur complement MR on the even sites), laid out for FP64's
// register cost: the even-site r and x live in LDS, links and clover blocks
// are read from global memory at each use (they stay in the L1/L2 caches
// within a block solve), the odd-site right-hand side is parked in global
// memory until the reconstruction, and the hop directions are visited in a
// loop, so no thread holds more than two 12-component vectors at a time.

template <class Sh>
__device__ __forceinline__ void f64_block_solve(const SapArgs &a, const int d, const Visit f)
{
    using T = double;
    using G = double;
    constexpr int VD = Sh::VD, VH = Sh::VH, NLC = 9;
    __shared__ cx<T> she[12][VH];   // even sites: MR residual r
    __shared__ cx<T> sho[12][VH];   // odd sites: C_o^-1 D_oe r
    __shared__ cx<T> shx[12][VH];   // even sites: MR solution x
    __shared__ T red[3 * (VD / 64)];

    const int loc = threadIdx.x;
    const int par = loc >= VH;
    const int hi = loc - par * VH;
    int l[4];
    Sh::coords(loc, l);
    // the site of the other parity with the same half index (its hops in
    // directions 2 and 3 are this thread's share)
    const int locp = (1 - par) * VH + hi;
    int lp[4];
    Sh::coords(locp, lp);
    int D[4];
    {
        int r = d;
        D[0] = r % a.g.n[0]; r /= a.g.n[0];
        D[1] = r % a.g.n[1]; r /= a.g.n[1];
        D[2] = r % a.g.n[2];
        D[3] = r / a.g.n[2];
    }
    const v2<G> *links = (const v2<G> *)a.links;
    const long lbase = (long)d * 4 * NLC * VD;
    const v2<G> *cs = (const v2<G> *)a.cs;
    const long cbase = (long)d * 36 * VD + loc;
    v2<T> *rho_g = global_ptr((v2<T> *)a.rho_tmp);
    const long sbase = (long)d * 12 * VD + loc;

    // ---- the block right-hand side rho
    cx<T> A[12], P[12];
    if (f.first) {
#pragma unroll
        for (int k = 0; k < 12; k++) A[k] = ld<T, double>(global_ptr(a.eta), sbase + (long)k * VD);
    } else if (par == 0) {
        const v2<T> *res = global_ptr((const v2<T> *)a.res);
#pragma unroll
        for (int k = 0; k < 12; k++) A[k] = ld<T, T>(res, ((long)d * 12 + k) * VH + hi);
    } else {
#pragma unroll
        for (int k = 0; k < 12; k++) A[k] = czero<T>();
    }
    if (f.faces_in) {
        gather_face<Sh, 0, T, T, G, NLC, false>(a, D, d, l, loc, A);
        gather_face<Sh, 1, T, T, G, NLC, false>(a, D, d, l, loc, A);
        gather_face<Sh, 2, T, T, G, NLC, false>(a, D, d, l, loc, A);
        gather_face<Sh, 3, T, T, G, NLC, false>(a, D, d, l, loc, A);
    }

    // ---- even-odd preparation: r = rho_e - D_eo C_o^-1 rho_o, x = 0
    if (par == 1) {
        clover_apply<T, G>(opaque(cs), cbase, VD, A, P);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            sho[k][hi] = P[k];
            st<T, T>(rho_g, ((long)d * 12 + k) * VH + hi, A[k]);
        }
    }
    __syncthreads();
    // she is free until r is written: it carries the odd threads' partial sums
    pair_hops_rolled<Sh, T, G, NLC, true, true>(sho, she, 0, par, hi, l, loc, lp, locp, lbase, links, P, T(0.5));
    if (par == 0) {
#pragma unroll
        for (int k = 0; k < 12; k++) {
            she[k][hi] = A[k] + P[k];
            shx[k][hi] = czero<T>();
        }
    }

    // ---- minimal residual on the Schur complement
#pragma unroll 1
    for (int it = 0; it < a.n_mr; it++) {
        __syncthreads();
        // sho is dead here (its readers passed the reduction's barriers): it
        // carries the even threads' partial sums
        pair_hops_rolled<Sh, T, G, NLC, true, true>(she, sho, 1, par, hi, l, loc, lp, locp, lbase, links, P,
                                                    T(-0.5));   // D_oe r
        if (par == 1) {
            clover_apply<T, G>(opaque(cs), cbase, VD, P, A);                                       // C_o^-1 D_oe r
#pragma unroll
            for (int k = 0; k < 12; k++) sho[k][hi] = A[k];
        } else {
            // meanwhile the even sites form C_e r, which needs only r
#pragma unroll
            for (int k = 0; k < 12; k++) A[k] = she[k][hi];
            clover_apply<T, G>(opaque(cs), cbase, VD, A, P);                                       // C_e r
        }
        __syncthreads();
        T dots[3] = {0, 0, 0};
        pair_hops_rolled<Sh, T, G, NLC, false, false>(sho, sho, 0, par, hi, l, loc, lp, locp, lbase, links, P,
                                                      T(0.5));   // - D_eo C_o^-1 D_oe r
        if (par == 0) {
#pragma unroll
            for (int k = 0; k < 12; k++) {
                const cx<T> rk = she[k][hi];
                dots[0] = fmad(P[k].i, rk.i, fmad(P[k].r, rk.r, dots[0]));
                dots[1] = fmad(-P[k].i, rk.r, fmad(P[k].r, rk.i, dots[1]));
                dots[2] = fmad(P[k].i, P[k].i, fmad(P[k].r, P[k].r, dots[2]));
            }
        }
        domain_reduce<VH, 1, VD / 64, false>(dots, red, 0);
        if (par == 0) {
            const cx<T> alpha = dots[2] > T(0) ? cx<T>{dots[0] / dots[2], dots[1] / dots[2]} : czero<T>();
#pragma unroll
            for (int k = 0; k < 12; k++) {
                const cx<T> rk = she[k][hi];
                shx[k][hi] = cmac(shx[k][hi], alpha, rk);
                she[k][hi] = cmac(rk, neg(alpha), P[k]);
            }
        }
    }
    __syncthreads();

    // ---- delta: x on even sites, C_o^-1 (rho_o - D_oe x) on odd sites
    // x moves to the even threads' registers; shx then carries their partial sums
    if (par == 1) {
#pragma unroll
        for (int k = 0; k < 12; k++) P[k] = ld<T, T>(rho_g, ((long)d * 12 + k) * VH + hi);
    } else {
#pragma unroll
        for (int k = 0; k < 12; k++) A[k] = shx[k][hi];
    }
    pair_hops_rolled<Sh, T, G, NLC, false, false>(shx, shx, 1, par, hi, l, loc, lp, locp, lbase, links, P, T(0.5));
    if (par == 1) clover_apply<T, G>(opaque(cs), cbase, VD, P, A);

    // ---- epilogue: psi += delta, stored residual, boundary terms
    {
        const v2<T> *psi_in = global_ptr((const v2<T> *)a.psi);
        v2<T> *psi_out = global_ptr((v2<T> *)a.psi);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const cx<T> ps = f.first ? A[k] : ld<T, T>(psi_in, sbase + (long)k * VD) + A[k];
            if (f.last) st<T, double>(global_ptr(a.out), sbase + (long)k * VD, ps);
            else st<T, T>(psi_out, sbase + (long)k * VD, ps);
        }
    }
    if (f.res_out && par == 0) {
        v2<T> *res = global_ptr((v2<T> *)a.res);
#pragma unroll
        for (int k = 0; k < 12; k++) st<T, T>(res, ((long)d * 12 + k) * VH + hi, she[k][hi]);
    }
    if (f.faces_out) {
        write_face<Sh, 0, T, T, G, NLC>(a, d, l, loc, A, T(1));
        write_face<Sh, 1, T, T, G, NLC>(a, d, l, loc, A, T(1));
        write_face<Sh, 2, T, T, G, NLC>(a, d, l, loc, A, T(1));
        write_face<Sh, 3, T, T, G, NLC>(a, d, l, loc, A, T(1));
    }
}

// The boundary terms a visit reads (face_in) and writes (face): one buffer for
// the multiplicative schedule (the two colours alternate), two alternating
// buffers for the additive one (all domains read the previous cycle's terms
// while writing their own).
__device__ __forceinline__ void bind_faces(SapArgs &a, const Visit &v)
{
    if (a.face_alt) {
        if (v.flip) {
            a.face_in = a.face;
            a.face_in_scale = a.face_scale;
            a.face = a.face_alt;
            a.face_scale = a.face_scale_alt;
        } else {
            a.face_in = a.face_alt;
            a.face_in_scale = a.face_scale_alt;
        }
    } else {
        a.face_in = a.face;
        a.face_in_scale = a.face_scale;
    }
}

// ---- batched half-sweeps ------------------------------------------------------
//
// One launch covers one colour of one half-sweep for many systems (right-hand
// sides and lattices of one domain shape): workgroup i takes item i = (system,
// domain) and that system's arguments.  Items with system < 0 are padding;
// systems with active == 0 (already converged) are skipped.

// With NDW > 1, items come in runs of NDW domains of one system (the plan
// never splits or pads a run), and workgroup i takes run i.
template <class Sh, int NDW, typename SS, typename G, bool SCALED, bool HALVES>
__global__ __launch_bounds__(Sh::VD * NDW, 2) void k_sap_lds(const SapArgs *args, const int2 *items,
                                                                             Visit v)
{
    const int2 it = items[(long)blockIdx.x * NDW];
    if (it.x < 0) return;
    SapArgs a = args[it.x];
    if (!a.active) return;
    bind_faces(a, v);
    int d = it.y;
    if constexpr (NDW > 1) d = items[(long)blockIdx.x * NDW + ((int)threadIdx.x & 63) / Sh::VH].y;
    lds_block_solve<Sh, NDW, SS, G, SCALED, HALVES>(a, d, v);
}

template <class Sh>
__global__ __launch_bounds__(Sh::VD) void k_sap_f64(const SapArgs *args, const int2 *items, Visit v)
{
    const int2 it = items[blockIdx.x];
    if (it.x < 0) return;
    SapArgs a = args[it.x];
    if (!a.active) return;
    bind_faces(a, v);
    f64_block_solve<Sh>(a, it.y, v);
}

template <class Sh, int NDW, typename T, typename SS, typename G, bool SCALED>
__global__ __launch_bounds__((SplitShape<Sh, NDW>::NT), (SplitShape<Sh, NDW>::template waves<T>())) void k_sap_split(
    const SapArgs *args, const int2 *items, Visit v)
{
    const int2 it = items[(long)blockIdx.x * NDW];
    if (it.x < 0) return;
    SapArgs a = args[it.x];
    if (!a.active) return;
    bind_faces(a, v);
    int d = it.y, sub = 0;
    if constexpr (NDW > 1) {
        sub = ((int)threadIdx.x % SplitShape<Sh, NDW>::GP) / Sh::VH;
        d = items[(long)blockIdx.x * NDW + sub].y;
    }
    split_block_solve<Sh, NDW, T, SS, G, SCALED>(a, d, sub, v);
}

// ---- dispatch ---------------------------------------------------------------

// ---- block solves of a tile of right-hand sides ---------------------------------
//
// One workgroup solves one domain for a tile of up to RT right-hand sides of
// one lattice (systems sys0 .. sys0 + nt - 1), so the domain's links are staged
// into LDS once for the tile and each link entry read from LDS serves all of
// them.  Thread t works on the even and the odd site with half index h = t / RT
// for right-hand side r = t % RT, so the threads of a site are consecutive
// lanes, and every thread is busy in both parity phases of the MR step.
// Spinors in LDS are [component pair][half index][right-hand side]; one such
// array serves both parities, the MR residual r and the solution x stay in the
// even site's registers.
//
// PROD selects the SU(3) product of a hop: VALU (per-thread fused
// multiply-adds, RT = 2), FP32 MFMA (4x4x1, six steps over the inner
// dimension) or BF16-input MFMA with FP32 accumulation (4x4x4, two steps; the
// link and half-spinor rounded to BF16), both RT = 4: the four lanes of a site
// are one 4x4 block of the 16-block MFMA instructions.  There the product U h
// (U the link or its adjoint, h the projected half-spinor) is, in real form, a
// 6x6 matrix (rows Re y_a and Im y_a, columns Re h_b and Im h_b) times a
// 6-vector; for the four right-hand sides and one spin component of h it is a
// 6x6 times 6x4 product, done as two 4-row blocks of the site's quad: lane r
// supplies row r of each block of U and column r (its own half-spinor), and
// receives column r of the result.  Lanes of right-hand sides beyond the tile
// work on zeros and touch no memory.
//
// Two right-hand sides, not four, for the VALU form: at 80 KB of LDS two
// workgroups share a CU, and while one moves its domain's data (some 10 bytes a
// cycle is what one CU gets from beyond its L1) the other one computes.  The
// FP16 launch of one colour for 12 right-hand sides on 32^3x64 (4096 domains of
// 4^4) takes 3.15 ms this way.  With tiles of four (157 KB, one workgroup a CU,
// separate arrays for r and C_o^-1 D_oe r) it took 4.73 ms with 8-byte LDS reads,
// mixed-precision multiply-adds and each site's lanes moving its boundary terms
// and accumulator, and 3.89 ms with 16-byte reads, FP32 multiply-adds and whole
// waves moving the boundary terms.

enum { PROD_VALU = 0, PROD_MFMA_F32 = 1, PROD_MFMA_BF16 = 2 };
constexpr int RT_VALU = 2, RT_MFMA = 4;
template <int PROD> constexpr int tile_rt() { return PROD == PROD_VALU ? RT_VALU : RT_MFMA; }
// Link entries in LDS lie LSTR entries apart.  For the matrix operands VD + 16:
// the four lanes of a quad read four different entries of one site (rows or
// columns of U), and with a stride of VD (a multiple of the 64 banks) all four
// would fall in one bank.
template <class Sh, int PROD> constexpr int tile_lstr() { return PROD == PROD_VALU ? Sh::VD : Sh::VD + 16; }

typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));

// Sum over the lanes of a wave with equal lane % RT, returned to all of them.
template <int RT, bool MAX> __device__ __forceinline__ float rhs_wave_reduce(float v)
{
    auto op = [](float a, float b) { return MAX ? fmax(a, b) : a + b; };
    if constexpr (RT == 2) v = op(v, dpp<0x4E>(v));   // quad_perm 2,3,0,1
    v = op(v, dpp<0x124>(v));                          // row_ror:4
    v = op(v, dpp<0x128>(v));                          // row_ror:8
    v = op(v, __shfl_xor(v, 16));
    v = op(v, __shfl_xor(v, 32));
    return v;
}

// sum of v over the threads of this thread's right-hand side (lanes with equal
// lane % RT), for all NW waves of the workgroup; fixed order, every thread joins
template <int RT, int NW> __device__ __forceinline__ void rhs_sum(float (&v)[3], f32x4_t *red)
{
#pragma unroll
    for (int q = 0; q < 3; q++) v[q] = rhs_wave_reduce<RT, false>(v[q]);
    const int w = threadIdx.x >> 6, r = threadIdx.x % RT;
    if ((threadIdx.x & 63) < RT) red[w * RT + r] = f32x4_t{v[0], v[1], v[2], 0.f};
    __syncthreads();
    f32x4_t s = red[r];
#pragma unroll
    for (int k = 1; k < NW; k++) s += red[k * RT + r];
    v[0] = s[0];
    v[1] = s[1];
    v[2] = s[2];
    // no closing barrier: several barriers pass before red is written again
}

// The maxima of a and b over the workgroup for this lane's right-hand side; no
// closing barrier: the caller (the epilogue) gives it its own part of red.
template <int RT, int NW> __device__ __forceinline__ void rhs_max2(float &a, float &b, f32x4_t *red)
{
    a = rhs_wave_reduce<RT, true>(a);
    b = rhs_wave_reduce<RT, true>(b);
    const int w = threadIdx.x >> 6, r = threadIdx.x % RT;
    if ((threadIdx.x & 63) < RT) red[w * RT + r] = f32x4_t{a, b, 0.f, 0.f};
    __syncthreads();
    f32x4_t m = red[r];
#pragma unroll
    for (int k = 1; k < NW; k++) {
        const f32x4_t q = red[k * RT + r];
        m[0] = fmax(m[0], q[0]);
        m[1] = fmax(m[1], q[1]);
    }
    a = m[0];
    b = m[1];
}

// Row `row` of U (forward hop, SIGN < 0) or of U^dagger (backward hop): u[b] =
// U[row][b], or conj(U[b][row]); links in LDS as three rows [mu][9][VD].
template <class Sh, int SIGN, int PROD, typename G>
__device__ __forceinline__ void link_row(const v2<G> *slink, int mu, int lloc, int row, cx<float> u[3])
{
#pragma unroll
    for (int b = 0; b < 3; b++) {
        const int e = SIGN < 0 ? row * 3 + b : b * 3 + row;
        const v2<G> v = slink[(mu * 9 + e) * tile_lstr<Sh, PROD>() + lloc];
        u[b] = {static_cast<float>(v.x), SIGN < 0 ? static_cast<float>(v.y) : -static_cast<float>(v.y)};
    }
}

// uh = (U or U^dagger) h for the four right-hand sides of the quad (h: this
// lane's half-spinor, both spin components) on the matrix cores.
template <class Sh, int SIGN, int PROD, typename G>
__device__ __forceinline__ void quad_product(const v2<G> *slink, int mu, int lloc, int r, const cx<float> h[6],
                                             cx<float> uh[6])
{
    // block 0 rows: Re y_0, Re y_1, Re y_2, Im y_0; block 1: Im y_1, Im y_2, 0, 0
    cx<float> u0[3], u1[3];
    link_row<Sh, SIGN, PROD, G>(slink, mu, lloc, r < 3 ? r : 0, u0);
    link_row<Sh, SIGN, PROD, G>(slink, mu, lloc, r == 0 ? 1 : 2, u1);
    const bool re0 = r < 3, use1 = r < 2;
    float a0[6], a1[6];
#pragma unroll
    for (int b = 0; b < 3; b++) {
        a0[b] = re0 ? u0[b].r : u0[b].i;
        a0[3 + b] = re0 ? -u0[b].i : u0[b].r;
        a1[b] = use1 ? u1[b].i : 0.f;
        a1[3 + b] = use1 ? u1[b].r : 0.f;
    }
    f32x4_t acc[2][2];
#pragma unroll
    for (int s = 0; s < 2; s++) acc[s][0] = acc[s][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if constexpr (PROD == PROD_MFMA_F32) {
#pragma unroll
        for (int k = 0; k < 6; k++)
#pragma unroll
            for (int s = 0; s < 2; s++) {
                const float bk = k < 3 ? h[s * 3 + k].r : h[s * 3 + k - 3].i;
                acc[s][0] = __builtin_amdgcn_mfma_f32_4x4x1f32(a0[k], bk, acc[s][0], 0, 0, 0);
                acc[s][1] = __builtin_amdgcn_mfma_f32_4x4x1f32(a1[k], bk, acc[s][1], 0, 0, 0);
            }
    } else {
        const bf16x4_t A0lo = {(__bf16)a0[0], (__bf16)a0[1], (__bf16)a0[2], (__bf16)a0[3]};
        const bf16x4_t A0hi = {(__bf16)a0[4], (__bf16)a0[5], (__bf16)0.f, (__bf16)0.f};
        const bf16x4_t A1lo = {(__bf16)a1[0], (__bf16)a1[1], (__bf16)a1[2], (__bf16)a1[3]};
        const bf16x4_t A1hi = {(__bf16)a1[4], (__bf16)a1[5], (__bf16)0.f, (__bf16)0.f};
#pragma unroll
        for (int s = 0; s < 2; s++) {
            const cx<float> *hs = h + 3 * s;
            const bf16x4_t Blo = {(__bf16)hs[0].r, (__bf16)hs[1].r, (__bf16)hs[2].r, (__bf16)hs[0].i};
            const bf16x4_t Bhi = {(__bf16)hs[1].i, (__bf16)hs[2].i, (__bf16)0.f, (__bf16)0.f};
            acc[s][0] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(A0lo, Blo, acc[s][0], 0, 0, 0);
            acc[s][0] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(A0hi, Bhi, acc[s][0], 0, 0, 0);
            acc[s][1] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(A1lo, Blo, acc[s][1], 0, 0, 0);
            acc[s][1] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(A1hi, Bhi, acc[s][1], 0, 0, 0);
        }
    }
#pragma unroll
    for (int s = 0; s < 2; s++) {
        uh[s * 3 + 0] = {acc[s][0][0], acc[s][0][3]};
        uh[s * 3 + 1] = {acc[s][0][1], acc[s][1][0]};
        uh[s * 3 + 2] = {acc[s][0][2], acc[s][1][1]};
    }
}

// acc += the hop into a site along MU: (1 - gamma_mu) U_mu(x) v(x + mu) for
// SIGN < 0, (1 + gamma_mu) U_mu(x - mu)^dagger v(x - mu) for SIGN > 0.  v: this
// right-hand side's spinor of the other parity's site with this site's half
// index hi in LDS ([6][VH][RT]); loc: the site, op: the first site of the other
// parity.  Neighbour offsets are constants (one address register for x, one
// for the other directions), so LDS addresses are immediates.  The link's reads
// stand here, not behind a function that returns it: the compiler then waits
// for them one by one, not for all (32^3x64: 3.13 against 3.24 ms a launch).
// Issuing the next hop's reads ahead of a hop's product gains nothing (3.12 ms
// with FP16, 3.03 against 2.93 with BF16 storage): two waves per SIMD hide them.
template <class Sh, int MU, int SIGN, int PROD, typename G>
__device__ __forceinline__ void tile_hop(const c2_t *v, const int l[4], int loc, int op, int hi, int ox, int r,
                                         const v2<G> *slink, cx<float> acc[12])
{
    constexpr int RT = tile_rt<PROD>(), LS = tile_lstr<Sh, PROD>();
    if constexpr (PROD == PROD_VALU) {
        if (!hop_exists<Sh, MU, SIGN>(l)) return;
        const int dn = hop_step<Sh, MU, SIGN>(ox);
        cx<float> s[12], h[6], uh[6];
        ld_c2<Sh::VH * RT>(v + dn * RT, s);
        proj<MU, SIGN>(s, h);
        const v2<G> *up = slink + MU * 9 * LS + (SIGN < 0 ? loc : op + hi + dn);
        su3<float> U;
#pragma unroll
        for (int e = 0; e < 9; e++) U.m[e] = widen<G>(up[e * LS]);
        if constexpr (SIGN < 0) su3_mul(U, h, uh);
        else su3_dag_mul(U, h, uh);
        recon_acc<MU, SIGN>(acc, uh, 1.0f);
    } else {
        // every lane takes part in the matrix instructions; a site without this
        // neighbour multiplies a finite stand-in (its own index's entry) and
        // adds the product with weight 0
        const bool has = hop_exists<Sh, MU, SIGN>(l);
        const int dn = has ? hop_step<Sh, MU, SIGN>(ox) : 0;
        cx<float> s[12], h[6], uh[6];
        ld_c2<Sh::VH * RT>(v + dn * RT, s);
        proj<MU, SIGN>(s, h);
        quad_product<Sh, SIGN, PROD, G>(slink, MU, SIGN < 0 ? loc : op + hi + dn, r, h, uh);
        recon_acc<MU, SIGN>(acc, uh, has ? 1.0f : 0.0f);
    }
}

template <class Sh, int PROD, typename G>
__device__ __forceinline__ void tile_hops(const c2_t *v, const int l[4], int loc, int op, int hi, int ox, int r,
                                          const v2<G> *slink, cx<float> acc[12])
{
#pragma unroll
    for (int k = 0; k < 12; k++) acc[k] = czero<float>();
    if constexpr (PROD != PROD_VALU) {
        // one hop's operands live at a time (a loop the compiler keeps rolled)
#pragma unroll 1
        for (int k = 0; k < 8; k++) {
            switch (k) {
                case 0: tile_hop<Sh, 0, -1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc); break;
                case 1: tile_hop<Sh, 0, +1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc); break;
                case 2: tile_hop<Sh, 1, -1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc); break;
                case 3: tile_hop<Sh, 1, +1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc); break;
                case 4: tile_hop<Sh, 2, -1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc); break;
                case 5: tile_hop<Sh, 2, +1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc); break;
                case 6: tile_hop<Sh, 3, -1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc); break;
                default: tile_hop<Sh, 3, +1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc); break;
            }
        }
        return;
    }
    tile_hop<Sh, 0, -1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc);
    tile_hop<Sh, 0, +1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc);
    tile_hop<Sh, 1, -1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc);
    tile_hop<Sh, 1, +1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc);
    tile_hop<Sh, 2, -1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc);
    tile_hop<Sh, 2, +1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc);
    tile_hop<Sh, 3, -1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc);
    tile_hop<Sh, 3, +1, PROD, G>(v, l, loc, op, hi, ox, r, slink, acc);
}

// The boundary terms of a face (f = 2 mu + side) for the tile's right-hand
// sides are moved by whole waves, so that every access to the boundary buffers
// is a run of cache lines (by the site's own lanes it is 64-byte pieces, and an
// eighth of the lanes at a time).  A face's places in the buffer are in the
// order (parity, transverse position / 2) of the sites that write them; no
// other kernel reads them.

// The site of the domain with parity p at place (p, j) of face f.
template <class Sh> __device__ __forceinline__ int tile_face_site(int p, int j, int f)
{
    static_assert(Sh::B[0] == 4 && Sh::B[1] == 4 && Sh::B[2] == 4 && Sh::B[3] == 4, "4^4 domains: two bits a coordinate");
    const int sh = f & ~1, l = f & 1 ? 3 : 0;   // 2 mu bits below the face's own coordinate
    int i = 2 * j;                              // transverse position, its lowest bit fixed by the parity
    i |= (l ^ i ^ (i >> 2) ^ (i >> 4) ^ p) & 1;
    const int lex = (i & ((1 << sh) - 1)) | (l << sh) | ((i >> sh) << (sh + 2));
    return lex >> 1;
}

// Loads the neighbour's half-spinors of the place of this lane for every
// right-hand side, and their weights (0 for those that the tile does not hold;
// their loads repeat the first's).  No branches: the loads of all right-hand
// sides are in flight together.
template <class Sh, int RT, typename SS, bool SCALED>
__device__ __forceinline__ void tile_face_fetch(const SapArgs *args, const Visit &v, int nt, const int D[4], int f,
                                                v2<SS> (&raw)[RT][6], float (&w)[RT])
{
    constexpr int FS = Sh::FS[0];
    static_assert(FS == 64 && Sh::FS[1] == 64 && Sh::FS[2] == 64 && Sh::FS[3] == 64, "one lane per face site");
    const Geo &g = args[0].g;
    const int mu = f >> 1, side = f & 1;
    int dn = 0;
    bool wrap = false;
#pragma unroll
    for (int m = 3; m >= 0; m--) {
        int q = D[m];
        if (m == mu) {
            wrap = side ? q == g.n[m] - 1 : q == 0;
            q = side ? (wrap ? 0 : q + 1) : (wrap ? g.n[m] - 1 : q - 1);
        }
        dn = dn * g.n[m] + q;
    }
    const float wb = wrap ? 0.5f * (float)g.bc[mu] : 0.5f;   // bc is +1 or -1
    const long fb = face_base<Sh>(dn, f ^ 1) + (threadIdx.x & 63);
#pragma unroll
    for (int r = 0; r < RT; r++) {
        const SapArgs &a = args[r < nt ? r : 0];
        const bool alt = a.face_alt && !v.flip;
        const v2<SS> *face = global_ptr((const v2<SS> *)(alt ? a.face_alt : a.face));
#pragma unroll
        for (int k = 0; k < 6; k++) raw[r][k] = face[fb + (long)k * FS];
        w[r] = wb;
        if constexpr (SCALED) w[r] *= global_ptr(alt ? a.face_scale_alt : a.face_scale)[dn];
        w[r] = r < nt ? w[r] : 0.f;
    }
}

// Their contribution (weight, and the link on the forward side) to stage [3]
// [FS][RT], by the order of Shape::face_index; the sites of the face add it to
// their right-hand side.
template <class Sh, int RT, int PROD, typename SS, typename G>
__device__ __forceinline__ void tile_face_stage(const v2<SS> (&raw)[RT][6], const float (&w)[RT], int f,
                                                const v2<G> *slink, c2_t *stage)
{
    constexpr int FS = Sh::FS[0], LS = tile_lstr<Sh, PROD>();
    // place of this lane: the neighbour's site of parity q, this domain's of parity 1 - q
    const int q = (threadIdx.x & 63) >> 5, j = threadIdx.x & 31;
    const int h = tile_face_site<Sh>(1 - q, j, f), lex = 2 * h + ((1 - q + (h >> 1) + (h >> 3) + (h >> 5)) & 1);
    const int sh = f & ~1, i = (lex & ((1 << sh) - 1)) | ((lex >> (sh + 2)) << sh);
    su3<float> U;
    if (f & 1) U = LdsLinks<G, LS>{slink}(f >> 1, (1 - q) * Sh::VH + h);
#pragma unroll
    for (int r = 0; r < RT; r++) {
        cx<float> hs[6];
#pragma unroll
        for (int k = 0; k < 6; k++) hs[k] = scal(w[r], widen<SS>(raw[r][k]));
        if (f & 1) {
            cx<float> uh[6];
            su3_mul(U, hs, uh);
#pragma unroll
            for (int k = 0; k < 6; k++) hs[k] = uh[k];
        }
#pragma unroll
        for (int c = 0; c < 3; c++)
            stage[(c * FS + i) * RT + r] = c2_t{hs[2 * c].r, hs[2 * c].i, hs[2 * c + 1].r, hs[2 * c + 1].i};
    }
}

// rho += the staged contribution (stage: both faces of MU) of the site's face
// along MU, if it has one
template <class Sh, int RT, int MU>
__device__ __forceinline__ void tile_face_add(const c2_t *stage, const int l[4], int r, cx<float> rho[12])
{
    constexpr int FS = Sh::FS[MU];
    const bool lo = l[MU] == 0, up = l[MU] == Sh::B[MU] - 1;
    if (!(lo || up)) return;
    const c2_t *p = stage + (up ? 3 * RT * FS : 0) + Sh::template face_index<MU>(l) * RT + r;
    cx<float> h[6];
#pragma unroll
    for (int j = 0; j < 3; j++) {
        const c2_t q = p[j * FS * RT];
        h[2 * j] = {q[0], q[1]};
        h[2 * j + 1] = {q[2], q[3]};
    }
    if (lo) recon_acc<MU, +1>(rho, h, 1.0f);
    else recon_acc<MU, -1>(rho, h, 1.0f);
}

// Writes the domain's own half-spinors of face f at the sites of parity p,
// places j = (64 / RT) sub + lane / RT, from delta of that parity in LDS; inv: 1
// / scale of this lane's right-hand side, whose boundary buffer is face (null:
// nothing to write).
template <class Sh, int RT, int PROD, typename SS, typename G>
__device__ __forceinline__ void tile_face_out(v2<SS> *face, int d, int f, int p, int sub, const c2_t *dl, float inv,
                                              const v2<G> *slink)
{
    constexpr int FS = Sh::FS[0], LS = tile_lstr<Sh, PROD>(), VH = Sh::VH;
    const int lane = threadIdx.x & 63, r = lane % RT, j = sub * (64 / RT) + lane / RT;
    const int h0 = tile_face_site<Sh>(p, j, f);
    cx<float> s[12], h[6];
    ld_c2<VH * RT>(dl + h0 * RT + r, s);
    switch (f) {
        case 0: proj<0, -1>(s, h); break;
        case 1: proj<0, +1>(s, h); break;
        case 2: proj<1, -1>(s, h); break;
        case 3: proj<1, +1>(s, h); break;
        case 4: proj<2, -1>(s, h); break;
        case 5: proj<2, +1>(s, h); break;
        case 6: proj<3, -1>(s, h); break;
        default: proj<3, +1>(s, h); break;
    }
    if (f & 1) {
        cx<float> uh[6];
        su3_dag_mul(LdsLinks<G, LS>{slink}(f >> 1, p * VH + h0), h, uh);
#pragma unroll
        for (int k = 0; k < 6; k++) h[k] = uh[k];
    }
    if (!face) return;
    const long fb = face_base<Sh>(d, f) + p * 32 + j;
#pragma unroll
    for (int k = 0; k < 6; k++) st<float, SS>(face, fb + (long)k * FS, scal(inv, h[k]));
}

// Items: x = first system of the tile | (systems in the tile) << 24, y = domain.
// SS: storage of block residual and boundary terms; G: links and clover (two
// rows stored, three rows in LDS); arithmetic and accumulator FP32.  The
// accumulator and the block residual, which no other kernel reads, are laid
// out for this one: [d][6][VD] and [d][3][VH] 16-byte entries.
template <class Sh, int PROD, typename SS, typename G, bool SCALED>
__global__ __launch_bounds__(Sh::VH * tile_rt<PROD>(), 2) void k_sap_tile(const SapArgs *args, const int2 *items, Visit v)
{
    using T = float;
    constexpr int RT = tile_rt<PROD>();
    constexpr int VD = Sh::VD, VH = Sh::VH, NT = VH * RT, NW = NT / 64, NLC = 6;
    constexpr int FPW = 8 / NW;               // faces per wave
    static_assert(NT % 64 == 0 && NT <= 1024 && (NW == 4 || NW == 8), "one or two faces a wave");
    constexpr int LSTR = tile_lstr<Sh, PROD>();
    __shared__ v2<G> slink[4 * 9 * LSTR];     // [mu][9][LSTR]
    __shared__ v2<G> sclo[36][VH];            // C_o^-1 of the odd sites
    // [6][VH][RT]: what the next hops read (even sites r, odd sites C_o^-1 D_oe r)
    __shared__ c2_t sp[6 * VH * RT];
    __shared__ f32x4_t red[2 * NW * RT];

    const int2 it = items[blockIdx.x];
    if (it.x < 0) return;   // padding (XCD lists of unequal length)
    const int sys0 = it.x & 0xffffff, nt = it.x >> 24, d = it.y;
    const int t = threadIdx.x, hi = t / RT, r = t % RT;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    // this lane's right-hand side; what the tile shares (geometry, links,
    // clover, MR steps) is taken from the first system, so it stays uniform
    const SapArgs *const ta = args + sys0;
    const SapArgs &a0 = ta[0];
    const SapArgs &a = ta[r < nt ? r : 0];
    const bool live = (r < nt) & (a.active != 0);
    const int loc_e = hi, loc_o = VH + hi;
    int le[4], lo[4];
    Sh::coords(loc_e, le);
    Sh::coords(loc_o, lo);
    const int oe = le[0] & 1, oo = lo[0] & 1;
    int D[4];
    {
        int q = d;
        D[0] = q % a0.g.n[0]; q /= a0.g.n[0];
        D[1] = q % a0.g.n[1]; q /= a0.g.n[1];
        D[2] = q % a0.g.n[2];
        D[3] = q / a0.g.n[2];
    }
    const v2<G> *glinks = global_ptr((const v2<G> *)a0.links);
    const v2<G> *cs = global_ptr((const v2<G> *)a0.cs);
    const int n_mr = a0.n_mr;
    const long se = (long)d * 12 * VD + loc_e, so = (long)d * 12 * VD + loc_o;
    c2_t *const pe = global_ptr((c2_t *)a.psi) + (long)d * 6 * VD + loc_e, *const po = pe + VH;
    const long rbase = (long)d * 3 * VH + hi;
    const double2 *const eta = global_ptr(a.eta);
    double2 *const out = global_ptr(a.out);
    const bool io32 = a.io32;
    // this wave's faces: one of each side where it has two
    int face_of[FPW];
#pragma unroll
    for (int q = 0; q < FPW; q++) face_of[q] = FPW == 1 ? wave : q == 0 ? wave : 4 + (wave ^ 1);

    // ---- links and the odd sites' C_o^-1 into LDS, the even site's C_e into
    // registers; every global load before the first LDS store
    v2<G> cle[36];
    cx<T> Ae[12], Ao[12], P[12], tt[12];
    v2<SS> fraw[FPW][RT][6];
    float fw[FPW][RT];
    {
        constexpr int NL = 4 * VD / NT;   // links per thread
        v2<G> lt[NL][NLC];
#pragma unroll
        for (int j = 0; j < NL; j++) {
            const int q = t + j * NT;     // = mu VD + site
#pragma unroll
            for (int e = 0; e < NLC; e++) lt[j][e] = glinks[(((long)d * 4 + q / VD) * NLC + e) * VD + q % VD];
        }
        const long cb = (long)d * 36 * VD;
        constexpr int NCO = 36 * VH / NT;
        static_assert(36 * VH % NT == 0 && 4 * VD % NT == 0, "odd clover entries and links per thread");
        v2<G> ct[NCO];
#pragma unroll
        for (int j = 0; j < NCO; j++) {
            const int i = t + j * NT, k = i / VH;
            ct[j] = cs[cb + (long)k * VD + VH + (i - k * VH)];
        }
        // the block right-hand side of both sites, without the boundary terms
        if (!live) {
#pragma unroll
            for (int k = 0; k < 12; k++) Ae[k] = Ao[k] = czero<T>();
        } else if (v.first && io32) {
#pragma unroll
            for (int k = 0; k < 12; k++) {
                Ae[k] = ld<T, float>((const float2 *)eta, se + (long)k * VD);
                Ao[k] = ld<T, float>((const float2 *)eta, so + (long)k * VD);
            }
        } else if (v.first) {
#pragma unroll
            for (int k = 0; k < 12; k++) {
                Ae[k] = ld<T, double>(eta, se + (long)k * VD);
                Ao[k] = ld<T, double>(eta, so + (long)k * VD);
            }
        } else {
            ld_res<VH, SS>(a.res, rbase, SCALED ? T(global_ptr(a.res_scale)[d]) : T(1), Ae);
#pragma unroll
            for (int k = 0; k < 12; k++) Ao[k] = czero<T>();
        }
        if (v.faces_in)
#pragma unroll
            for (int q = 0; q < FPW; q++) tile_face_fetch<Sh, RT, SS, SCALED>(ta, v, nt, D, face_of[q], fraw[q], fw[q]);
#pragma unroll
        for (int k = 0; k < 36; k++) cle[k] = cs[cb + (long)k * VD + loc_e];
#pragma unroll
        for (int j = 0; j < NCO; j++) {
            const int i = t + j * NT, k = i / VH;
            sclo[k][i - k * VH] = ct[j];
        }
#pragma unroll
        for (int j = 0; j < NL; j++) {
            const int q = t + j * NT;
            LdsLinks<G, LSTR>::put(slink, q / VD, q % VD, lt[j]);
        }
    }
    __syncthreads();   // links staged
    if (v.faces_in) {
        // sp holds four faces at a time: along x and y, then along z and t
#pragma unroll
        for (int h = 0; h < 2; h++) {
#pragma unroll
            for (int q = 0; q < FPW; q++)
                if (face_of[q] >> 2 == h)
                    tile_face_stage<Sh, RT, PROD, SS, G>(fraw[q], fw[q], face_of[q], slink, sp + 3 * RT * 64 * (face_of[q] & 3));
            __syncthreads();
            if (h == 0) {
                tile_face_add<Sh, RT, 0>(sp, le, r, Ae);
                tile_face_add<Sh, RT, 1>(sp + 6 * RT * 64, le, r, Ae);
                tile_face_add<Sh, RT, 0>(sp, lo, r, Ao);
                tile_face_add<Sh, RT, 1>(sp + 6 * RT * 64, lo, r, Ao);
            } else {
                tile_face_add<Sh, RT, 2>(sp, le, r, Ae);
                tile_face_add<Sh, RT, 3>(sp + 6 * RT * 64, le, r, Ae);
                tile_face_add<Sh, RT, 2>(sp, lo, r, Ao);
                tile_face_add<Sh, RT, 3>(sp + 6 * RT * 64, lo, r, Ao);
            }
            __syncthreads();   // sp is written again below
        }
    }
    c2_t *const vs = sp + hi * RT + r;
    auto clover_o = [&](const cx<T> in[12], cx<T> o[12]) {
        clover_wide([&](int q) { return widen<G>(sclo[q][hi]); }, in, o);
    };

    // ---- even-odd preparation: r = rho_e - D_eo C_o^-1 rho_o, x = 0.  With
    // the matrix-instruction products rho_o waits in this right-hand side's
    // global buffer until the reconstruction (their operands leave no room
    // for it in registers); the VALU form keeps it in registers.
    constexpr bool PARK = PROD != PROD_VALU;
    clover_o(Ao, P);
    v2<T> *rho_g = global_ptr((v2<T> *)a.rho_tmp);
    st_c2<VH * RT>(vs, P);
    if (PARK && live)
#pragma unroll
        for (int k = 0; k < 12; k++) st<T, T>(rho_g, ((long)d * 12 + k) * VH + hi, Ao[k]);
    __syncthreads();
    tile_hops<Sh, PROD, G>(vs, le, loc_e, VH, hi, oe, r, slink, tt);
    cx<T> rr[12];
#pragma unroll
    for (int k = 0; k < 12; k++) {
        rr[k] = Ae[k] + scal(T(0.5), tt[k]);
        Ae[k] = czero<T>();
    }
    // C_e has arrived: without this, a path around the MR loop on which it has
    // not makes the later waits for its registers wait for younger loads
#pragma unroll
    for (int q = 0; q < 36; q++) asm volatile("" : "+v"(cle[q]));
    __syncthreads();   // sp has been read
    st_c2<VH * RT>(vs, rr);

    // ---- minimal residual on the Schur complement, per right-hand side
#pragma unroll 1
    for (int itr = 0; itr < n_mr; itr++) {
        if constexpr (sizeof(v2<G>) == 4) {
            // keep the clover blocks in their 16-bit storage form (see k_sap_lds)
#pragma unroll
            for (int q = 0; q < 36; q++) asm volatile("" : "+v"(cle[q]));
        }
        __syncthreads();
        tile_hops<Sh, PROD, G>(vs, lo, loc_o, 0, hi, oo, r, slink, tt);   // -2 D_oe r
        clover_o(tt, P);                                            // -2 C_o^-1 D_oe r
        __syncthreads();   // sp has been read
        st_c2<VH * RT>(vs, P);
        __syncthreads();
        tile_hops<Sh, PROD, G>(vs, le, loc_e, VH, hi, oe, r, slink, tt);
        clover_wide([&](int q) { return widen<G>(cle[q]); }, rr, P);   // C_e r
        T dots[3] = {0, 0, 0};
#pragma unroll
        for (int k = 0; k < 12; k++) {
            P[k] = P[k] + scal(T(-0.25), tt[k]);                    // p = C_e r - D_eo C_o^-1 D_oe r
            dots[0] = fmad(P[k].i, rr[k].i, fmad(P[k].r, rr[k].r, dots[0]));
            dots[1] = fmad(-P[k].i, rr[k].r, fmad(P[k].r, rr[k].i, dots[1]));
            dots[2] = fmad(P[k].i, P[k].i, fmad(P[k].r, P[k].r, dots[2]));
        }
        rhs_sum<RT, NW>(dots, red);   // its barrier: sp has been read
        const cx<T> alpha = dots[2] > T(0) ? cx<T>{dots[0] / dots[2], dots[1] / dots[2]} : czero<T>();
#pragma unroll
        for (int k = 0; k < 12; k++) {
            Ae[k] = cmac(Ae[k], alpha, rr[k]);
            rr[k] = cmac(rr[k], neg(alpha), P[k]);
        }
        st_c2<VH * RT>(vs, rr);
    }

    // ---- odd sites: delta_o = C_o^-1 (rho_o - D_oe x).  The accumulator is
    // fetched ahead of it (where registers allow).
    c2_t pse[6], pso[6];
#pragma unroll
    for (int j = 0; j < 6; j++) pse[j] = pso[j] = c2_t{0.f, 0.f, 0.f, 0.f};
    auto fetch_psi = [&] {
        if (live && !v.first)
#pragma unroll
            for (int j = 0; j < 6; j++) {
                pse[j] = pe[j * VD];
                pso[j] = po[j * VD];
            }
    };
    st_c2<VH * RT>(vs, Ae);   // r there was this thread's own entry, not read since
    if constexpr (!PARK) fetch_psi();
    __syncthreads();
    tile_hops<Sh, PROD, G>(vs, lo, loc_o, 0, hi, oo, r, slink, tt);
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const cx<T> ro = !PARK ? Ao[k] : live ? ld<T, T>(rho_g, ((long)d * 12 + k) * VH + hi) : czero<T>();
        tt[k] = ro + scal(T(0.5), tt[k]);
    }
    clover_o(tt, Ao);                                               // Ao = delta_o, Ae = delta_e = x
    if constexpr (PARK) fetch_psi();

    // ---- epilogue: psi += delta, stored residual, boundary terms
    if (live) {
#pragma unroll
        for (int j = 0; j < 6; j++) {
            pse[j] += c2_t{Ae[2 * j].r, Ae[2 * j].i, Ae[2 * j + 1].r, Ae[2 * j + 1].i};
            pso[j] += c2_t{Ao[2 * j].r, Ao[2 * j].i, Ao[2 * j + 1].r, Ao[2 * j + 1].i};
        }
        if (v.last) {
#pragma unroll
            for (int k = 0; k < 12; k++) {
                const cx<T> ce = {pse[k / 2][2 * (k & 1)], pse[k / 2][2 * (k & 1) + 1]};
                const cx<T> co = {pso[k / 2][2 * (k & 1)], pso[k / 2][2 * (k & 1) + 1]};
                if (io32) {
                    st<T, float>((float2 *)out, se + (long)k * VD, ce);
                    st<T, float>((float2 *)out, so + (long)k * VD, co);
                } else {
                    st<T, double>(out, se + (long)k * VD, ce);
                    st<T, double>(out, so + (long)k * VD, co);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < 6; j++) {
                pe[j * VD] = pse[j];
                po[j * VD] = pso[j];
            }
        }
    }
    if (!v.res_out && !v.faces_out) return;
    T rsc = T(1), fsc = T(1);
    if constexpr (SCALED) {
        T mr = maxabs12(rr), mf = fmax(maxabs12(Ae), maxabs12(Ao));
        rhs_max2<RT, NW>(mr, mf, red + NW * RT);
        rsc = pow2_ceil(mr);
        fsc = T(8) * pow2_ceil(mf);
    }
    if (v.res_out && live) {
        if (SCALED && hi == 0) global_ptr(a.res_scale)[d] = (float)rsc;
        st_res<VH, SS>(a.res, rbase, T(1) / rsc, rr);
    }
    if (v.faces_out) {
        const bool alt = a.face_alt && v.flip;
        if (SCALED && hi == 0 && live) global_ptr(alt ? a.face_scale_alt : a.face_scale)[d] = (float)fsc;
        v2<SS> *const face = live ? global_ptr((v2<SS> *)(alt ? a.face_alt : a.face)) : nullptr;
        const T inv = T(1) / fsc;
        if (!SCALED) __syncthreads();   // the reconstruction's hops have read sp (SCALED: rhs_max2's barrier)
        // lane % RT is the right-hand side there too: inv and face are this lane's
#pragma unroll
        for (int p = 0; p < 2; p++) {
            if (p) __syncthreads();     // the even sites' delta has been read
            st_c2<VH * RT>(vs, p ? Ao : Ae);
            __syncthreads();
#pragma unroll 1
            for (int side = 0; side < 2; side++)
                tile_face_out<Sh, RT, PROD, SS, G>(face, d, 2 * (wave / (RT / 2)) + side, p, wave % (RT / 2), sp, inv, slink);
        }
    }
}

// Every block-solve launch goes through here: the workgroup size must not
// exceed the kernel's launch bound (the register allocation is made for that
// bound), which is read from the code object once per kernel and checked on
// the host before the launch.
template <typename... P, typename... A>
static hipError_t launch_bounded(void (*kernel)(P...), unsigned grid, unsigned block, hipStream_t s, A... args)
{
    static std::mutex mu;
    static std::unordered_map<const void *, int> bound;
    const void *key = reinterpret_cast<const void *>(kernel);
    int maxt;
    {
        std::lock_guard<std::mutex> lock(mu);
        auto it = bound.find(key);
        if (it == bound.end()) {
            hipFuncAttributes at;
            const hipError_t e = hipFuncGetAttributes(&at, key);
            if (e != hipSuccess) return e;
            it = bound.emplace(key, at.maxThreadsPerBlock).first;
        }
        maxt = it->second;
    }
    if (block == 0 || (int)block > maxt) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(block), 0, s, args...);
    return hipGetLastError();
}

// one thread per site, FP32 arithmetic
template <class Sh, int NDW, bool HALVES>
static hipError_t launch_lds(const SapArgs *args, const int2 *items, int nitems, int prec, Visit v, hipStream_t s)
{
    constexpr int NT = Sh::VD * NDW;
    if (prec == P32)
        return launch_bounded(k_sap_lds<Sh, NDW, float, float, false, HALVES>, nitems / NDW, NT, s, args, items, v);
    else if (prec == P16)
        return launch_bounded(k_sap_lds<Sh, NDW, half_t, half_t, true, HALVES>, nitems / NDW, NT, s, args, items, v);
    else
        return launch_bounded(k_sap_lds<Sh, NDW, bf16_t, bf16_t, false, HALVES>, nitems / NDW, NT, s, args, items, v);
}

template <class Sh>
static hipError_t launch_batch(const SapArgs *args, const int2 *items, int nitems, int prec, int product, Visit v,
                               hipStream_t s)
{
    if (product >= PRODUCT_TILE_VALU && product <= PRODUCT_TILE_MFMA_BF16) {
        // a tile of right-hand sides per workgroup: 4^4 domains, FP16 storage
        if constexpr (std::is_same<Sh, Shape<4, 4, 4, 4>>::value) {
            constexpr int NT = Sh::VH * RT_MFMA, NTV = Sh::VH * RT_VALU;
            if (prec == PB16) {
                switch (product) {
                    case PRODUCT_TILE_VALU:
                        return launch_bounded(k_sap_tile<Sh, PROD_VALU, bf16_t, bf16_t, false>, nitems, NTV, s, args,
                                              items, v);
                    case PRODUCT_TILE_MFMA_F32:
                        return launch_bounded(k_sap_tile<Sh, PROD_MFMA_F32, bf16_t, bf16_t, false>, nitems, NT, s, args,
                                              items, v);
                    case PRODUCT_TILE_MFMA_BF16:
                        return launch_bounded(k_sap_tile<Sh, PROD_MFMA_BF16, bf16_t, bf16_t, false>, nitems, NT, s,
                                              args, items, v);
                    default: return hipErrorInvalidValue;
                }
            }
            if (prec != P16) return hipErrorInvalidValue;
            switch (product) {
                case PRODUCT_TILE_VALU:
                    return launch_bounded(k_sap_tile<Sh, PROD_VALU, half_t, half_t, true>, nitems, NTV, s, args, items, v);
                case PRODUCT_TILE_MFMA_F32:
                    return launch_bounded(k_sap_tile<Sh, PROD_MFMA_F32, half_t, half_t, true>, nitems, NT, s, args, items,
                                          v);
                case PRODUCT_TILE_MFMA_BF16:
                    return launch_bounded(k_sap_tile<Sh, PROD_MFMA_BF16, half_t, half_t, true>, nitems, NT, s, args,
                                          items, v);
                default: return hipErrorInvalidValue;
            }
        }
        return hipErrorInvalidValue;
    }
    constexpr int NDW = Sh::VD < 64 ? 128 / Sh::VD : 1;
    if (nitems % NDW) return hipErrorInvalidValue;
    if (product == PRODUCT_LANE_HALVES) {
        if constexpr (Sh::VD == 256)
            if (prec != P64) return launch_lds<Sh, NDW, true>(args, items, nitems, prec, v, s);
        return hipErrorInvalidValue;
    }
    if (product == PRODUCT_LANE_SPLIT) {
        if constexpr (Sh::VD < 512) {
            constexpr int NT = SplitShape<Sh, NDW>::NT;
            if constexpr (Sh::VD == 16)
                if (prec == P64)
                    return launch_bounded(k_sap_split<Sh, NDW, double, double, double, false>, nitems / NDW, NT, s, args, items, v);
            if (prec == P32)
                return launch_bounded(k_sap_split<Sh, NDW, float, float, float, false>, nitems / NDW, NT, s, args, items, v);
            if (prec == P16)
                return launch_bounded(k_sap_split<Sh, NDW, float, half_t, half_t, true>, nitems / NDW, NT, s, args, items, v);
            if (prec == PB16)
                return launch_bounded(k_sap_split<Sh, NDW, float, bf16_t, bf16_t, false>, nitems / NDW, NT, s, args, items, v);
        }
        return hipErrorInvalidValue;
    }
    if (prec == P64) {
        // whole waves only
        if constexpr (Sh::VD >= 64 && Sh::VD % 64 == 0)
            return launch_bounded(k_sap_f64<Sh>, nitems, Sh::VD, s, args, items, v);
        else
            return hipErrorInvalidValue;
    } else if constexpr (Sh::VD * NDW % 64 == 0) {
        return launch_lds<Sh, NDW, false>(args, items, nitems, prec, v, s);
    } else {
        return hipErrorInvalidValue;   // two threads per site (dd_form.h)
    }
}

int sap_domains_per_workgroup(int shape, int prec, int product)
{
    return shape == 0 ? 8 : 1;   // only one-right-hand-side kernels take 2^4 domains
}

int sap_rhs_per_workgroup(int product)
{
    switch (product) {
        case PRODUCT_TILE_VALU: return RT_VALU;
        case PRODUCT_TILE_MFMA_F32:
        case PRODUCT_TILE_MFMA_BF16: return RT_MFMA;
        default: return 1;
    }
}

bool sap_product_supported(const int b[4], int prec, int product)
{
    if (product == PRODUCT_LANE) return sap_prec_supported(b, prec);
    if (product < PRODUCT_TILE_VALU || product > PRODUCT_TILE_MFMA_BF16) return false;
    return sap_shape_id(b) == 1 && (prec == P16 || prec == PB16);
}

int sap_lattice_form(const Geo &g, int prec, int product)
{
    return sap_kernel_form(g.Vd, prec, product, g.nd / 2 / sap_domains_per_workgroup(sap_shape_id(g.b), prec, product));
}

int sap_shape_id(const int b[4])
{
    if (b[0] == 2 && b[1] == 2 && b[2] == 2 && b[3] == 2) return 0;
    if (b[0] == 4 && b[1] == 4 && b[2] == 4 && b[3] == 4) return 1;
    if (b[0] == 8 && b[1] == 4 && b[2] == 4 && b[3] == 4) return 2;
    if (b[0] == 4 && b[1] == 4 && b[2] == 4 && b[3] == 8) return 3;
    if (b[0] == 6 && b[1] == 6 && b[2] == 2 && b[3] == 4) return 4;
    return -1;
}

int sap_shape_count() { return 5; }

void sap_shape_extents(int shape, int b[4])
{
    static const int E[5][4] = {{2, 2, 2, 2}, {4, 4, 4, 4}, {8, 4, 4, 4}, {4, 4, 4, 8}, {6, 6, 2, 4}};
    for (int m = 0; m < 4; m++) b[m] = E[shape][m];
}

bool sap_shape_supported(const int b[4]) { return sap_shape_id(b) >= 0; }

// FP64 block solves need 16 sites or whole waves of one thread per site
bool sap_prec_supported(const int b[4], int prec)
{
    const int id = sap_shape_id(b);
    if (id < 0 || prec < P64 || prec > PB16) return false;
    const int vd = b[0] * b[1] * b[2] * b[3];
    return prec != P64 || vd == 16 || vd % 64 == 0;
}

long sap_face_sites(const int b[4])
{
    long Vd = (long)b[0] * b[1] * b[2] * b[3];
    return 2 * (Vd / b[0] + Vd / b[1] + Vd / b[2] + Vd / b[3]);
}

// item i < nd/2: the i-th black domain (item.x = x), item nd/2 + i: the i-th
// white one, in increasing domain number.  The domain grid's x extent is even,
// so domains 2i and 2i + 1 lie in one x row and have opposite colours: the
// i-th domain of colour c is the one of that pair with colour c.
__global__ void k_schedule_items(Geo g, int x, int2 *items)
{
    const int half = g.nd / 2;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.nd) return;
    const int c = i >= half, j = i - c * half;
    const int d0 = 2 * j;
    const int rest = d0 / g.n[0];
    const int D1 = rest % g.n[1], D2 = (rest / g.n[1]) % g.n[2], D3 = rest / (g.n[1] * g.n[2]);
    const int colour0 = (D1 + D2 + D3) & 1;   // colour of domain 2j (its x coordinate is even)
    items[i] = make_int2(x, d0 + ((c + colour0) & 1));
}

__global__ void k_put_args(SapArgs a, SapArgs *dst) { *dst = a; }

hipError_t sap_schedule_items(const Geo &g, int x, int2 *items, hipStream_t s)
{
    hipLaunchKernelGGL(k_schedule_items, (g.nd + 255) / 256, 256, 0, s, g, x, items);
    return hipGetLastError();
}

hipError_t sap_put_args(const SapArgs &a, SapArgs *dst, hipStream_t s)
{
    hipLaunchKernelGGL(k_put_args, 1, 1, 0, s, a, dst);
    return hipGetLastError();
}

hipError_t sap_sweep_batch(const SapArgs *args, const int2 *items, int nitems, int shape, int prec, int product,
                           Visit v, hipStream_t s)
{
    if (nitems <= 0) return hipSuccess;
    switch (shape) {
        case 0: return launch_batch<Shape<2, 2, 2, 2>>(args, items, nitems, prec, product, v, s);
        case 1: return launch_batch<Shape<4, 4, 4, 4>>(args, items, nitems, prec, product, v, s);
        case 2: return launch_batch<Shape<8, 4, 4, 4>>(args, items, nitems, prec, product, v, s);
        case 3: return launch_batch<Shape<4, 4, 4, 8>>(args, items, nitems, prec, product, v, s);
        case 4: return launch_batch<Shape<6, 6, 2, 4>>(args, items, nitems, prec, product, v, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace dd
