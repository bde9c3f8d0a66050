// Kernels of a refinement level solved with the mask scheme (Sec. V), double precision.
//
// The level is the periodic N^3 grid of its resolution.  A cell with mask > 0 is active and
// relaxed; a cell with mask <= 0 keeps a fixed value w (the coarser level's solution
// interpolated there).  A masked neighbour nb of an active cell i enters the operator as
// the ghost value u_g = (1 - r) u_b + r u_i, r = m_nb / m_i (eq. u_i-1jk), with the boundary
// value u_b = (m_i w_nb - m_nb w_i) / (m_i - m_nb) fixed where the linearly interpolated mask
// vanishes (eq. phi_b), and b_g = exp(u_g) (b is not interpolated): eq. bc_modified_fR_op
// and eq. bc_modified_fR_dop.  Coarse levels carry the 8-child means of the masks and of w.
// The residual is restricted from active children (masked ones count zero) into active coarse
// cells, R u from all 8 children; the coarse correction is zero in masked coarse cells and
// is prolongated into active fine cells only (Sec. V.A.2, V.A.3, V.B.2).
//
// On the finest level a mask that only holds +1 and -1 is read as one byte per cell (bit 0:
// active, bit 1: active with a masked neighbour).
#include "device_fp64.h"

#include <type_traits>

namespace mgfr {
namespace {

constexpr int kB = 256;
constexpr int kMaxParts = 8192;

using dev::OpVal;
using dev::at;
using dev::bounded;
using u8 = unsigned char;

// mask value of cell q: the float mask, or a byte flag standing for +1 / -1
__device__ __forceinline__ double mval(const float* __restrict__ m, long long q) { return m[q]; }
__device__ __forceinline__ double mval(const u8* __restrict__ m, long long q) { return (m[q] & 1) ? 1.0 : -1.0; }

// The term of a masked neighbour (mask ratio r = m_nb / m_i <= 0, fixed value wn) in L_i and
// dL_i/du_i of an active cell of value ui, b_i = bi and fixed value wi: with the boundary value
// u_b = (m_i wn - m_nb wi) / (m_i - m_nb) the ghost u_g = (1 - r) u_b + r ui is wn + r (ui - wi), and
// b_g = exp(u_g) (eq. phi_b, eq. u_i-1jk, eq. bc_modified_fR_op, eq. bc_modified_fR_dop).
__device__ __forceinline__ void masked_face(double r, double wn, double wi, double ui, double bi, double& L, double& dL)
{
    const double ug = fma(r, ui - wi, wn);
    const double bg = dev::exp_(ug), du = ug - ui;
    L = fma(bg + bi, du, L);
    // chain rule: du_g/du_i = r, db_g/du_i = r b_g
    dL += (r * bg + bi) * du + (bg + bi) * (r - 1.0);
}

// ---- masks of +1 and -1 ---------------------------------------------------------------------
// A cell's value travels with b = exp(u), its sign set where the cell is masked (then u is its fixed
// value w, which it keeps for the whole solve).  An active cell's is clear, also in the NaN of a
// diverged one, as exp_ has it.
__device__ __forceinline__ double signed_b(double u, int active)
{
    const double b = dev::exp_(u);
    return __hiloint2double(__double2hiint(b) | (active ? 0 : (int)0x80000000), __double2loint(b));
}
__device__ __forceinline__ bool masked_b(double b) { return __double2hiint(b) < 0; }

// L_i - f and dL_i/du_i of an active cell of fixed value wi.  With r = -1 and u_b = (w_nb + w_i)/2
// the ghost is u_g = w_nb + w_i - u_i, so b_g = exp(w_nb) exp(w_i - u_i): one exponential serves
// all ghosts of the cell, and a ghost is a neighbour of value u_nb + (w_i - u_i) and b_g whose
// derivative has the further term -(b_g + b_i) - b_g (u_g - u_i).  A wavefront without a masked
// neighbour skips what ghosts need; the other cells' results are the same bits either way.
__device__ __forceinline__ OpVal masked_op_pm1(const Grid& g, double ui, double bi, const double (&un)[6],
                                               const double (&bn)[6], double f, double wi)
{
    double su = 0.0, sb = 0.0, sbu = 0.0, sg = 0.0;
    bool any = false;
#pragma unroll
    for (int v = 0; v < 6; ++v) any = any || masked_b(bn[v]);
    if (__any(any)) {
        const double shift = any ? wi - ui : 0.0;
        const double E = dev::exp_(shift);
#pragma unroll
        for (int v = 0; v < 6; ++v) {
            const bool gh = masked_b(bn[v]);
            const double b = gh ? -bn[v] * E : bn[v];
            const double du = (un[v] - ui) + (gh ? shift : 0.0);
            su += du;
            sb += b;
            sbu = fma(b, du, sbu);
            if (gh) sg += fma(b, du, b) + bi;
        }
    } else {
#pragma unroll
        for (int v = 0; v < 6; ++v) {
            const double du = un[v] - ui;
            su += du;
            sb += bn[v];
            sbu = fma(bn[v], du, sbu);
        }
    }
    const double S = dev::curvature(g, ui, bi);
    OpVal o;
    o.L = fma(g.C, fma(bi, su, sbu), S) - f;
    o.dL = fma(g.C, fma(-6.0, bi, fma(bi, su, -sb)) - sg, -S * g.inv_np1);
    return o;
}

// The same with every value read where it is; w only where a neighbour is masked.
__device__ __forceinline__ OpVal masked_op(const Grid& g, const u8* __restrict__ flags, const double* __restrict__ w,
                                           const double* __restrict__ u, int i, int j, int k, double ui, double,
                                           double f)
{
    const int m = g.n - 1;
    const long long qn[6] = {at(g, (i - 1) & m, j, k), at(g, (i + 1) & m, j, k), at(g, i, (j - 1) & m, k),
                             at(g, i, (j + 1) & m, k), at(g, i, j, (k - 1) & m), at(g, i, j, (k + 1) & m)};
    double un[6], bn[6];
#pragma unroll
    for (int v = 0; v < 6; ++v) {
        un[v] = u[qn[v]];
        bn[v] = signed_b(un[v], flags[qn[v]] & 1);
    }
    const long long q = at(g, i, j, k);
    const double wi = (flags[q] & 2) ? w[q] : 0.0;
    return masked_op_pm1(g, ui, dev::exp_(ui), un, bn, f, wi);
}

// L_i - f and dL_i/du_i at active cell (i,j,k) of value ui, mask mi.
template <class M>
__device__ __forceinline__ OpVal masked_op(const Grid& g, const M* __restrict__ mask,
                                           const double* __restrict__ w, const double* __restrict__ u,
                                           int i, int j, int k, double ui, double mi, double f)
{
    const int m = g.n - 1;
    const long long qn[6] = {at(g, (i - 1) & m, j, k), at(g, (i + 1) & m, j, k), at(g, i, (j - 1) & m, k),
                             at(g, i, (j + 1) & m, k), at(g, i, j, (k - 1) & m), at(g, i, j, (k + 1) & m)};
    const double bi = dev::exp_(ui);
    double L = 0.0, dL = 0.0, wi = 0.0;
    bool have_wi = false;
#pragma unroll
    for (int v = 0; v < 6; ++v) {
        const double mn = mval(mask, qn[v]);
        if (mn > 0.0) {
            const double un = u[qn[v]], bn = dev::exp_(un), du = un - ui;
            L = fma(bn + bi, du, L);
            dL += bi * du - bn - bi;
        } else {
            if (!have_wi) {
                wi = w[at(g, i, j, k)];
                have_wi = true;
            }
            masked_face(mn / mi, w[qn[v]], wi, ui, bi, L, dL);
        }
    }
    const double S = dev::curvature(g, ui, bi);
    OpVal o;
    o.L = fma(g.C, L, S) - f;
    o.dL = fma(g.C, dL, -S * g.inv_np1);
    return o;
}

// The same from values at hand: the neighbours' u (a masked one's fixed value), signed b and mask.
// A wavefront without a masked neighbour runs no ghost terms.
__device__ __forceinline__ OpVal masked_op_at(const Grid& g, double ui, double bi, const double (&un)[6],
                                              const double (&bn)[6], const float (&mn)[6], float mi, double f, double wi)
{
    double L = 0.0, dL = 0.0;
    bool any = false;
#pragma unroll
    for (int v = 0; v < 6; ++v) {
        const bool gh = masked_b(bn[v]);
        any = any || gh;
        const double b = gh ? 0.0 : bn[v], du = gh ? 0.0 : un[v] - ui, bb = gh ? 0.0 : bi;
        L = fma(b + bb, du, L);
        dL += fma(bb, du, -b) - bb;
    }
    if (__any(any)) {
        const double im = 1.0 / (double)mi;
#pragma unroll
        for (int v = 0; v < 6; ++v)
            if (masked_b(bn[v])) masked_face((double)mn[v] * im, un[v], wi, ui, bi, L, dL);
    }
    const double S = dev::curvature(g, ui, bi);
    OpVal o;
    o.L = fma(g.C, L, S) - f;
    o.dL = fma(g.C, dL, -S * g.inv_np1);
    return o;
}

// Summed magnitudes of the terms of L_i - f at an active cell: C (b_nb + b_i)|u_nb - u_i| per
// face (the ghost's for a masked neighbour), the curvature term and |f|.
__device__ double masked_mag(const Grid& g, const float* mask, const double* w, const double* u, int i, int j, int k,
                             double ui, double mi, double f)
{
    const int m = g.n - 1;
    const long long qn[6] = {at(g, (i - 1) & m, j, k), at(g, (i + 1) & m, j, k), at(g, i, (j - 1) & m, k),
                             at(g, i, (j + 1) & m, k), at(g, i, j, (k - 1) & m), at(g, i, j, (k + 1) & m)};
    const double bi = dev::exp_(ui), wi = w[at(g, i, j, k)];
    double t = 0.0;
    for (int v = 0; v < 6; ++v) {
        const double mn = mask[qn[v]];
        double un;
        if (mn > 0.0) {
            un = u[qn[v]];
        } else {
            const double r = mn / mi;
            un = (1.0 - r) * ((mi * w[qn[v]] - mn * wi) / (mi - mn)) + r * ui;
        }
        t += g.C * (dev::exp_(un) + bi) * fabs(un - ui);
    }
    return t + g.A * dev::exp_(-ui * g.inv_np1) + fabs(f);
}

__device__ __forceinline__ void cell_of(const Grid& g, long long q, int& i, int& j, int& k)
{
    i = (int)(q >> (2 * g.lg));
    j = (int)((q >> g.lg) & (g.n - 1));
    k = (int)(q & (g.n - 1));
}

// Block reduction over kB threads in a fixed order: a summed, b maxed (NaN propagates).
__device__ __forceinline__ void block_sum_max(double& a, double& b, double* sa, double* sb)
{
    sa[threadIdx.x] = a;
    sb[threadIdx.x] = b;
    __syncthreads();
    for (int s = kB / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            sa[threadIdx.x] += sa[threadIdx.x + s];
            const double o = sb[threadIdx.x + s];
            if (!(sb[threadIdx.x] >= o)) sb[threadIdx.x] = o;
        }
        __syncthreads();
    }
    a = sa[0];
    b = sb[0];
    __syncthreads();
}

// Block reduction over kB threads in a fixed order: a and b both summed.
__device__ __forceinline__ void block_sum2(double& a, double& b, double* sa, double* sb)
{
    sa[threadIdx.x] = a;
    sb[threadIdx.x] = b;
    __syncthreads();
    for (int s = kB / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            sa[threadIdx.x] += sa[threadIdx.x + s];
            sb[threadIdx.x] += sb[threadIdx.x + s];
        }
        __syncthreads();
    }
    a = sa[0];
    b = sb[0];
    __syncthreads();
}

// One colour of a red-black Newton-Gauss-Seidel sweep; one thread per cell of the colour,
// masked cells untouched.
template <class M>
__global__ void __launch_bounds__(kB) km_ngs_colour(Grid g, const M* __restrict__ mask,
                                                    const double* __restrict__ w, double* __restrict__ u,
                                                    const double* __restrict__ src, int colour)
{
    const long long half = 1LL << (3 * g.lg - 1);
    const long long t = (long long)blockIdx.x * kB + threadIdx.x;
    if (t >= half) return;
    const int hk = g.n >> 1;
    const int s = (int)(t & (hk - 1));
    const long long row = t >> (g.lg - 1);
    const int i = (int)(row >> g.lg), j = (int)(row & (g.n - 1));
    const int k = 2 * s + ((i + j + colour) & 1);
    const long long q = at(g, i, j, k);
    const double mi = mval(mask, q);
    if (!(mi > 0.0)) return;
    const double ui = u[q];
    const OpVal r = masked_op(g, mask, w, u, i, j, k, ui, mi, dev::rhs_value(g, src[q]));
    u[q] = ui + bounded(-r.L / r.dL, g.max_step);
}

// ---- fused red-black sweep of a level (n >= 64), of byte flags or of a float mask -----------
// The domain's fused sweep (sweep_fp64.hip: red cells of plane p, then black cells of plane p-1,
// in one pass over HBM, out of place from uin to uout, (u, b) of the planes in LDS, one tile
// column pair per thread with the ring and the halo as extra columns) with the mask scheme: a
// masked cell carries -b, is never updated and is copied to uout unchanged.  The density is
// loaded for active cells and w for those with a masked neighbour.  On byte flags every update sees
// the operands of the two-colour sweep in the same order.  A float mask (the coarse levels') is
// staged beside (u, b).
// Bound by its double-precision arithmetic, the ghosts' on top of the domain sweep's.  Measured at
// 512^3 with 61% of the cells active: 1.26 ms per sweep; with the loads behind branches and a 64-bit
// address each 1.31, with the column pairs laid over tile and halo (704 threads) and an exponential and
// a branch per masked neighbour 2.19 ms.  Float mask at 256^3, half of the cells active: 231 us, the two
// colour launches 358 us.
constexpr int kMK = 64;  // tile width along k

// A flag byte or a mask value: whether the cell is active, and whether its update needs w.
__device__ __forceinline__ bool is_active(int fl) { return fl & 1; }
__device__ __forceinline__ bool is_active(float m) { return m > 0.0f; }
__device__ __forceinline__ bool needs_w(int fl) { return fl & 2; }
__device__ __forceinline__ bool needs_w(float m) { return m > 0.0f; }
template <class M>
using MaskVal = typename std::conditional<std::is_same<M, float>::value, float, int>::type;

// A column's value on a plane: a scalar plane pointer and the column's byte offset, which fits in 32
// bits (n <= 1024); both are opaque, or the compiler keeps a 64-bit pointer per column and array and
// adds to it.
template <class T>
__device__ __forceinline__ auto plane_ref(T* f, int lg, int p, unsigned col) -> auto&
{
    using U = std::remove_const_t<T>;
    using gptr = __attribute__((address_space(1))) char*;
    gptr b = (gptr)(f + ((size_t)p << (2 * lg)));
    unsigned d = col * (unsigned)sizeof(U);
    asm("" : "+s"(b));
    asm("" : "+v"(d));
    return *(__attribute__((address_space(1))) U*)(b + d);
}

template <class V>
struct ColM {
    double u1, b1, vr, br, ru[2], fr, fb, wr, wb;
    V m1, rm[2];    // flag or mask of plane p+1 and, raw, of planes p+2 and p+3
    V mr;           // mask of the cell (vr, br)
    unsigned col;   // (j,k) offset within a plane
    int c, cl;      // LDS cell and its k-neighbour below (the one above follows it)
};

template <int TJ, int TK, class M>
__global__ void __launch_bounds__(TJ * TK / 2) __attribute__((amdgpu_waves_per_eu(4)))
km_ngs_fused(Grid g, const M* __restrict__ flags, const double* __restrict__ w, const double* __restrict__ uin,
             double* __restrict__ uout, const double* __restrict__ src, FusedSweep a)
{
    using V = MaskVal<M>;
    using Col = ColM<V>;
    constexpr bool FM = std::is_same<M, float>::value;
    constexpr int NT = TJ * TK / 2;
    constexpr int LJ = TJ + 4, LK = TK + 4, HK = LK / 2, NL = LJ * LK;
    constexpr int NR = 2 * (TK + 2) + 2 * TJ;
    constexpr int NH = 2 * (TK + 4) + 2 * (TJ + 2);
    constexpr int NR2 = NR / 2, R1 = (NR2 + 63) / 64 * 64;
    static_assert(R1 + NR2 <= NT && NR + NH <= NT, "one extra column per thread");
    __shared__ double2 lv[3][NL];
    __shared__ float lm[FM ? 3 : 1][FM ? NL : 1];
    const int nb = gridDim.x;
    int lid = blockIdx.x;
    if ((nb & 7) == 0) lid = (lid & 7) * (nb >> 3) + (lid >> 3);
    const int tk = lid % a.ntk;
    lid /= a.ntk;
    const int tj = lid % a.ntj;
    const int ci = lid / a.ntj;
    const int i0 = ci * a.ti, j0 = tj * TJ, k0 = tk * TK;
    const int lg = g.lg, m = g.n - 1;
    const int last = i0 + a.ti + 1;  // last plane read
    const int t = threadIdx.x;

    // a row's even columns before its odd ones
    auto place = [](Col& q, int jj, int kk) {
        q.c = jj * LK + (kk & 1) * HK + (kk >> 1);
        q.cl = jj * LK + ((kk & 1) ? kk >> 1 : HK + (kk >> 1) - 1);
    };
    // X is the column of the pair with the red cell on plane i0-1, Y the other
    Col X{}, Y{}, E{};
    {
        const int jj = 2 + t / (TK / 2), kk = 2 + 2 * (t - (jj - 2) * (TK / 2));
        const int gj = (j0 - 2 + jj) & m, gk = (k0 - 2 + kk) & m;
        const int sx = (i0 - 1 + gj + gk) & 1;
        X.col = (unsigned)((gj << lg) | (gk + sx));
        Y.col = (unsigned)((gj << lg) | (gk + 1 - sx));
        place(X, jj, kk + sx);
        place(Y, jj, kk + 1 - sx);
    }
    // E: a ring or halo cell of some of the threads, as in the domain's sweep
    bool eon, ering;
    int epar;
    {
        int x = -1;
        if (t < NR2) x = 2 * t;
        else if (t >= R1 && t < R1 + NR2) x = 2 * (t - R1) + 1;
        ering = x >= 0;
        if (!ering) x = t < R1 ? t - NR2 : t - 2 * NR2;
        eon = ering || x < NH;
        const int o = ering ? 1 : 0, ra = LJ - 2 * o, rb = LK - 2 * o;
        int ej, ek;
        if (x < rb) { ej = 0; ek = x; }
        else if (x < rb + ra - 1) { ej = x - rb + 1; ek = rb - 1; }
        else if (x < 2 * rb + ra - 2) { ej = ra - 1; ek = rb - 2 - (x - (rb + ra - 1)); }
        else { ej = ra - 2 - (x - (2 * rb + ra - 2)); ek = 0; }
        if (!eon) { ej = 0; ek = 0; }
        ej += o;
        ek += o;
        const int gj = (j0 - 2 + ej) & m, gk = (k0 - 2 + ek) & m;
        E.col = (unsigned)((gj << lg) | gk);
        place(E, ej, ek);
        epar = (gj + gk) & 1;
    }

    auto ref = [&](auto* f, int p, unsigned col) -> auto& { return plane_ref(f, lg, p & m, col); };
    auto buf = [&](int p) { return (p - i0 + 3) % 3; };
    // the density and w of a cell of flag byte fl on plane p, where an update needs them, else the
    // tile's corner's: no load stands behind a branch (but for a float mask, whose registers
    // would spill: 5% slower at 256^3)
    const unsigned corner = (unsigned)((j0 << lg) | k0);
    auto fetch = [&](int p, const Col& q, V fl, double& fv, double& wv) {
        if constexpr (FM) {
            if (is_active(fl)) {
                fv = ref(src, p, q.col);
                wv = ref(w, p, q.col);
            }
            return;
        }
        fv = ref(src, p, is_active(fl) ? q.col : corner);
        wv = ref(w, p, needs_w(fl) ? q.col : corner);
    };
    auto prologue = [&](Col& q) {
        const double um2 = ref(uin, i0 - 2, q.col), um1 = ref(uin, i0 - 1, q.col);
        const V fm2 = ref(flags, i0 - 2, q.col), fm1 = ref(flags, i0 - 1, q.col);
        q.u1 = ref(uin, i0, q.col);
        q.m1 = ref(flags, i0, q.col);
        q.ru[1] = ref(uin, i0 + 1, q.col);
        q.rm[1] = ref(flags, i0 + 1, q.col);
        q.b1 = signed_b(q.u1, is_active(q.m1));
        lv[buf(i0 - 2)][q.c] = make_double2(um2, signed_b(um2, is_active(fm2)));
        lv[buf(i0 - 1)][q.c] = make_double2(um1, signed_b(um1, is_active(fm1)));
        if constexpr (FM) {
            lm[buf(i0 - 2)][q.c] = fm2;
            lm[buf(i0 - 1)][q.c] = fm1;
        }
        return fm1;
    };
    {
        const V fx = prologue(X);
        fetch(i0 - 1, X, fx, X.fr, X.wr);
        prologue(Y);
        fetch(i0, Y, Y.m1, Y.fr, Y.wr);
        if (eon) {
            const V fe = prologue(E);
            if (ering) {
                // of the plane on which the cell is red first
                double f1, w1;
                fetch(i0 - 1, E, fe, E.fr, E.wr);
                fetch(i0, E, E.m1, f1, w1);
                if ((i0 - 1 + epar) & 1) {
                    E.fr = f1;
                    E.wr = w1;
                }
            }
        }
    }
    __syncthreads();

    const double ms = g.max_step;
    // BLACK: the step has a black cell in the chunk (the first two do not)
    auto step = [&](auto N2c, auto Bc, int p, Col& A, Col& B) {
        constexpr int N2 = decltype(N2c)::value, N3 = N2 ^ 1;
        constexpr bool BLACK = decltype(Bc)::value;
        double2* L0 = lv[buf(p)];
        const double2* Lm = lv[buf(p - 1)];
        double2* L1 = lv[buf(p + 1)];
        auto Lf = [&](int pp) -> float* { return lm[FM ? buf(pp) : 0]; };
        // past the last plane that one again
        const int p3 = p + 3 < last ? p + 3 : last;
        auto load = [&](Col& q) {
            q.ru[N3] = ref(uin, p3, q.col);
            q.rm[N3] = ref(flags, p3, q.col);
        };
        load(A);
        load(B);
        load(E);
        // the operator at the cell of column q on plane pp (its mask from LDS; below and above: the
        // masks of its i-neighbours)
        auto op = [&](const Col& q, int pp, const double (&un)[6], const double (&bn)[6], float below, V above,
                      const double2& own, double fv, double wv) -> OpVal {
            if constexpr (FM) {
                const float* l = Lf(pp);
                const float mn[6] = {below, above, l[q.c - LK], l[q.c + LK], l[q.cl], l[q.cl + 1]};
                return masked_op_at(g, own.x, own.y, un, bn, mn, l[q.c], dev::rhs_value(g, fv), wv);
            } else {
                return masked_op_pm1(g, own.x, own.y, un, bn, dev::rhs_value(g, fv), wv);
            }
        };
        // red cell of plane p, if active
        auto red = [&](const Col& q, const double2& m1, const double2& p0) -> double2 {
            const int c = q.c;
            const double2 jm = L0[c - LK], jp = L0[c + LK], km = L0[q.cl], kp = L0[q.cl + 1];
            const double un[6] = {m1.x, q.u1, jm.x, jp.x, km.x, kp.x};
            const double bn[6] = {m1.y, q.b1, jm.y, jp.y, km.y, kp.y};
            const OpVal r = op(q, p, un, bn, Lf(p - 1)[FM ? c : 0], q.m1, p0, q.fr, q.wr);
            const double v = p0.x + bounded(-r.L / r.dL, ms);
            return make_double2(v, dev::exp_(v));
        };
        {
            const int c = A.c;
            const double2 m1 = Lm[c];
            double2 v = L0[c];
            if (!masked_b(v.y)) {
                v = red(A, m1, v);
                L0[c] = v;
            }
            // black cell of plane p-1, if active; plane p-1 is then final in both columns
            if constexpr (BLACK) {
                double un1 = m1.x;
                if (!masked_b(m1.y)) {
                    const double2 jm = Lm[c - LK], jp = Lm[c + LK], km = Lm[A.cl], kp = Lm[A.cl + 1];
                    const double un[6] = {A.vr, v.x, jm.x, jp.x, km.x, kp.x};
                    const double bn[6] = {A.br, v.y, jm.y, jp.y, km.y, kp.y};
                    const OpVal r = op(A, p - 1, un, bn, (float)A.mr, FM ? (V)Lf(p)[FM ? c : 0] : V(0), m1, A.fb, A.wb);
                    un1 = m1.x + bounded(-r.L / r.dL, ms);
                }
                ref(uout, p - 1, A.col) = un1;
                ref(uout, p - 1, B.col) = B.vr;
            }
            A.vr = v.x;
            A.br = v.y;
            if constexpr (FM) A.mr = Lf(p)[c];
        }
        const bool ered = ering && ((p + epar) & 1) == 0;
        if (ered) {
            const double2 p0 = L0[E.c];
            if (!masked_b(p0.y)) L0[E.c] = red(E, Lm[E.c], p0);
        }
        // stage plane p+1; plane p+2 follows in the registers, and with its flags known the
        // right-hand sides and fixed values of A's next active step (p+2) are loaded
        const V mA = A.m1;
        auto advance = [&](Col& q) {
            L1[q.c] = make_double2(q.u1, q.b1);
            if constexpr (FM) Lf(p + 1)[q.c] = q.m1;
            q.u1 = q.ru[N2];
            q.m1 = q.rm[N2];
            q.b1 = signed_b(q.u1, is_active(q.m1));
        };
        advance(A);
        advance(B);
        if (eon) advance(E);
        const int pf = p + 2 < last ? p + 2 : last - 1;
        fetch(pf, A, A.m1, A.fr, A.wr);
        fetch(p + 1, A, mA, A.fb, A.wb);
        if (ered) fetch(pf, E, E.m1, E.fr, E.wr);
        __syncthreads();
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    step(I1{}, std::false_type{}, i0 - 1, X, Y);
    step(I0{}, std::false_type{}, i0, Y, X);
    for (int p = i0 + 1; p <= i0 + a.ti; p += 2) {
        step(I1{}, std::true_type{}, p, X, Y);
        step(I0{}, std::true_type{}, p + 1, Y, X);
    }
}

// One thread per coarse cell: R u of all 8 children and R d of the active ones into active
// coarse cells; masked coarse cells take their fixed value and a zero right-hand side.
template <class M>
__global__ void __launch_bounds__(kB) km_resid_restrict(Grid g, const M* __restrict__ mask,
                                                        const double* __restrict__ w, const double* __restrict__ u,
                                                        const double* __restrict__ src,
                                                        const float* __restrict__ maskc,
                                                        const double* __restrict__ wc, double* __restrict__ uc,
                                                        double* __restrict__ uhat, double* __restrict__ fc)
{
    const int lgc = g.lg - 1, nc = g.n >> 1;
    const long long tc = (long long)blockIdx.x * kB + threadIdx.x;
    if (tc >= (1LL << (3 * lgc))) return;
    if (!(maskc[tc] > 0.0f)) {
        uc[tc] = wc[tc];
        uhat[tc] = wc[tc];
        fc[tc] = 0.0;
        return;
    }
    const int I = (int)(tc >> (2 * lgc)), J = (int)((tc >> lgc) & (nc - 1)), K = (int)(tc & (nc - 1));
    double su = 0.0, sd = 0.0;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int i = 2 * I + a, j = 2 * J + b, k = 2 * K + c;
                const long long q = at(g, i, j, k);
                const double ui = u[q], mi = mval(mask, q);
                su += ui;
                if (mi > 0.0) sd += masked_op(g, mask, w, u, i, j, k, ui, mi, dev::rhs_value(g, src[q])).L;
            }
    uc[tc] = 0.125 * su;
    uhat[tc] = 0.125 * su;
    fc[tc] = 0.125 * sd;
}

// FAS right-hand side at active coarse cells: f = L^H(R u) - R d.
__global__ void __launch_bounds__(kB) km_fas_rhs(Grid g, const float* __restrict__ mask,
                                                 const double* __restrict__ w, const double* __restrict__ uhat,
                                                 double* __restrict__ f)
{
    const long long q = (long long)blockIdx.x * kB + threadIdx.x;
    if (q >= (1LL << (3 * g.lg))) return;
    const double mi = mask[q];
    if (!(mi > 0.0)) return;
    int i, j, k;
    cell_of(g, q, i, j, k);
    f[q] = masked_op(g, mask, w, uhat, i, j, k, uhat[q], mi, 0.0).L - f[q];
}

// Coarse correction u^H - R u^h at active coarse cells, zero at masked ones (no correction
// comes from a cell that is not a valid multigrid cell), written over uhat.
__global__ void __launch_bounds__(kB) km_coarse_diff(long long n, const float* __restrict__ maskc,
                                                     const double* __restrict__ uc, double* __restrict__ uhat)
{
    const long long q = (long long)blockIdx.x * kB + threadIdx.x;
    if (q >= n) return;
    uhat[q] = maskc[q] > 0.0f ? uc[q] - uhat[q] : 0.0;
}

// Block partials (sum d^2, max |d|) over the active cells.  A thread takes one 2x2x2 block of
// cells, the eight cells unrolled so that their loads overlap; one partial pair per workgroup.
template <class M>
__global__ void __launch_bounds__(kB) km_norm(Grid g, const M* __restrict__ mask,
                                              const double* __restrict__ w, const double* __restrict__ u,
                                              const double* __restrict__ src, double* __restrict__ partial)
{
    __shared__ double sa[kB], sb[kB];
    const int lgc = g.lg - 1, nc = g.n >> 1;
    const long long nblk = 1LL << (3 * lgc);
    double s = 0.0, mx = 0.0;
    const long long t = (long long)blockIdx.x * kB + threadIdx.x;
    if (t < nblk) {
        const int I = (int)(t >> (2 * lgc)), J = (int)((t >> lgc) & (nc - 1)), K = (int)(t & (nc - 1));
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int z = 0; z < 2; ++z) {
                    const int i = 2 * I + x, j = 2 * J + y, k = 2 * K + z;
                    const long long q = at(g, i, j, k);
                    const double mi = mval(mask, q);
                    if (mi > 0.0) {
                        const double d = masked_op(g, mask, w, u, i, j, k, u[q], mi, dev::rhs_value(g, src[q])).L;
                        s += d * d;
                        const double a = fabs(d);
                        if (!(mx >= a)) mx = a;
                    }
                }
    }
    block_sum_max(s, mx, sa, sb);
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = s;
        partial[2 * blockIdx.x + 1] = mx;
    }
}

// A level of byte flags or of a float mask (n >= 64), streamed: a workgroup owns a tile of TJ x TK
// columns and a chunk of ti planes (even); per plane it stages (u, signed b) of the tile and a
// one-cell ring in LDS (a float mask's values too), keeps the i-neighbours in registers and has the
// next two planes in flight, so each value and exponential is fetched and formed once.  RESTRICT:
// R u of all 8 children and R d of the active ones into active coarse cells; masked coarse cells take
// their fixed value and a zero right-hand side.  FAS: f = L(u) - f at active cells (fc holds f).
// NORM: the partial (sum d^2, max |d|) of the workgroup, summed in a fixed order.
// The columns lie as in the domain's residual (resid_fp64.hip: two of a thread, neighbours in j, a
// coarse cell's eight children in two lanes; the ring is an extra column of the first threads), and
// no load stands behind a branch: a cell that needs no density or w reads that of the tile's
// corner instead.
// Bound by its arithmetic.  Measured at 512^3, 61% active: norm 0.72 ms, restriction 0.80 ms; one
// column per thread of 8 x 32 tiles (384 threads, loads behind branches, restriction through LDS)
// 1.25 and 1.67.  Float masks at 256^3: restriction 170 us (286), FAS right-hand side 168 us (243).
// What km_stream does with d = L(u) - f.
enum { kNorm, kRestrict, kFas };

template <class V>
struct ColS {
    double um, u0, up, bm, b0, bp;  // planes p-1, p, p+1
    double ru[2];                   // plane q, raw, in [(q - i0) & 1]
    double f[2], w[2];              // density (FAS: f) and w, same slots
    double uq, dq;                  // of the plane before, for the restriction
    V mm, m0, mp, rm[2];
    unsigned col;                   // (j,k) offset within a plane
    int c;                          // LDS cell
};

// the value of the lane whose k differs in its last bit
__device__ __forceinline__ double k_pair(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0xb1, 0xf, 0xf, true);  // quad_perm [1,0,3,2]
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0xb1, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

template <int TJ, int TK, int NT, int MODE, class M>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4)))
km_stream(Grid g, const M* __restrict__ flags, const double* __restrict__ w, const double* __restrict__ u,
          const double* __restrict__ src, double* __restrict__ partial, const float* __restrict__ maskc,
          const double* __restrict__ wc, double* __restrict__ uc, double* __restrict__ uhat, double* __restrict__ fc,
          int ti)
{
    using V = MaskVal<M>;
    using Col = ColS<V>;
    constexpr bool FM = std::is_same<M, float>::value;
    constexpr int LJ = TJ + 2, LK = TK + 2, NL = LJ * LK, NH = 2 * LK + 2 * TJ;
    static_assert(NT == TJ * TK / 2 && NH <= NT, "two columns and one ring cell per thread");
    __shared__ double2 lv[2][NL];
    __shared__ float lm[FM ? 2 : 1][FM ? NL : 1];
    const int ntk = g.n / TK, ntj = g.n / TJ;
    const int nb = gridDim.x;
    int lid = blockIdx.x;
    if ((nb & 7) == 0) lid = (lid & 7) * (nb >> 3) + (lid >> 3);
    const int tk = lid % ntk;
    lid /= ntk;
    const int tj = lid % ntj;
    const int i0 = (lid / ntj) * ti, j0 = tj * TJ, k0 = tk * TK;
    const int lg = g.lg, m = g.n - 1;
    const int last = i0 + ti;  // last plane read
    const int t = threadIdx.x;

    auto ref = [&](auto* f, int p, unsigned col) -> auto& { return plane_ref(f, lg, p & m, col); };
    auto request = [&](Col& q, int N, int p) {
        q.ru[N] = ref(u, p, q.col);
        q.rm[N] = ref(flags, p, q.col);
    };
    // density (FAS: f) and w of plane p, of mask mp
    const unsigned corner = (unsigned)((j0 << lg) | k0);
    auto request_f = [&](Col& q, int N, int p, V mp) {
        q.f[N] = ref(MODE == kFas ? fc : src, p, is_active(mp) ? q.col : corner);
        q.w[N] = ref(w, p, needs_w(mp) ? q.col : corner);
    };

    Col X{}, Y{}, E{};
    const bool ring = t < NH;
    {
        auto setup = [&](Col& q, int j, int k) {
            q.col = (unsigned)((((j0 - 1 + j) & m) << lg) | ((k0 - 1 + k) & m));
            q.c = j * LK + k;
        };
        const int r = t - 2 * LK;
        setup(X, 1 + 2 * (t / TK), 1 + t % TK);
        setup(Y, 2 + 2 * (t / TK), 1 + t % TK);
        if (t < LK) setup(E, 0, t);
        else if (t < 2 * LK) setup(E, LJ - 1, t - LK);
        else if (ring) setup(E, 1 + (r >> 1), (r & 1) * (LK - 1));
        else E.col = X.col;  // loads its own column again, in vain
    }
    auto prologue = [&](Col& q) {
        q.um = ref(u, i0 - 1, q.col);
        q.u0 = ref(u, i0, q.col);
        q.up = ref(u, i0 + 1, q.col);
        q.mm = ref(flags, i0 - 1, q.col);
        q.m0 = ref(flags, i0, q.col);
        q.mp = ref(flags, i0 + 1, q.col);
        request(q, 0, i0 + 2);
    };
    auto staged = [&](Col& q) {
        q.b0 = signed_b(q.u0, is_active(q.m0));
        q.bp = signed_b(q.up, is_active(q.mp));
        lv[0][q.c] = make_double2(q.u0, q.b0);
        if constexpr (FM) lm[0][q.c] = q.m0;
    };
    prologue(X);
    prologue(Y);
    prologue(E);
    request_f(X, 0, i0, X.m0);
    request_f(Y, 0, i0, Y.m0);
    X.bm = signed_b(X.um, is_active(X.mm));
    Y.bm = signed_b(Y.um, is_active(Y.mm));
    staged(X);
    staged(Y);
    if (ring) staged(E);
    __syncthreads();

    double s = 0.0, mx = 0.0, cw = 0.0;
    float cm = 0.0f;
    // One plane, N = (p - i0) & 1 fixed at compile time: the slots of the loads in flight rotate by
    // renaming (a copy would wait for them).
    auto step = [&](auto Nc, int p) {
        constexpr int N = decltype(Nc)::value, O = N ^ 1;
        // the coarse cell of this and the next plane, ahead of the planes' loads: waiting for the
        // youngest load waits for all
        const long long qc = ((((long long)((p & m) >> 1) << (lg - 1)) + (j0 >> 1) + t / TK) << (lg - 1)) +
                             ((k0 + t % TK) >> 1);
        if constexpr (MODE == kRestrict && N == 0) {
            cm = maskc[qc];
            cw = wc[qc];
        }
        const int p3 = p + 3 < last ? p + 3 : last, p1 = p + 1 < last ? p + 1 : last - 1;
        request(X, O, p3);
        request(Y, O, p3);
        request(E, O, p3);
        request_f(X, O, p1, X.mp);
        request_f(Y, O, p1, Y.mp);
        const double2* L = lv[N];
        const float* l = lm[FM ? N : 0];
        auto residual = [&](Col& q, double2 jm, double2 jp, float mjm, float mjp) -> double {
            double d = 0.0;
            if (!masked_b(q.b0)) {
                const double2 km = L[q.c - 1], kp = L[q.c + 1];
                const double un[6] = {q.um, q.up, jm.x, jp.x, km.x, kp.x};
                const double bn[6] = {q.bm, q.bp, jm.y, jp.y, km.y, kp.y};
                const double f = MODE == kFas ? 0.0 : dev::rhs_value(g, q.f[N]);
                if constexpr (FM) {
                    const float mn[6] = {(float)q.mm, (float)q.mp, mjm, mjp, l[q.c - 1], l[q.c + 1]};
                    d = masked_op_at(g, q.u0, q.b0, un, bn, mn, q.m0, f, q.w[N]).L;
                } else {
                    d = masked_op_pm1(g, q.u0, q.b0, un, bn, f, q.w[N]).L;
                }
            }
            asm volatile("" : "+v"(d));  // one column after the other: interleaved, they spill
            if constexpr (MODE == kFas) {
                if (!masked_b(q.b0)) ref(fc, p, q.col) = d - q.f[N];
            } else if constexpr (MODE == kNorm) {
                s += d * d;
                const double ad = fabs(d);
                if (!(mx >= ad)) mx = ad;
            }
            return d;
        };
        const double dx = residual(X, L[X.c - LK], make_double2(Y.u0, Y.b0), l[FM ? X.c - LK : 0], Y.m0);
        const double dy = residual(Y, make_double2(X.u0, X.b0), L[Y.c + LK], X.m0, l[FM ? Y.c + LK : 0]);
        if constexpr (MODE == kRestrict && N == 0) {
            X.uq = X.u0;
            X.dq = dx;
            Y.uq = Y.u0;
            Y.dq = dy;
        } else if constexpr (MODE == kRestrict) {
            const double ux = X.uq + X.u0, uy = Y.uq + Y.u0, ex = X.dq + dx, ey = Y.dq + dy;
            const double su = ux + k_pair(ux) + uy + k_pair(uy);
            const double sd = ex + k_pair(ex) + ey + k_pair(ey);
            if (!(t & 1)) {
                const double v = cm > 0.0f ? 0.125 * su : cw;
                uc[qc] = v;
                uhat[qc] = v;
                fc[qc] = cm > 0.0f ? 0.125 * sd : 0.0;
            }
        }
        // stage plane p+1 and shift the planes
        auto advance = [&](Col& q) {
            lv[O][q.c] = make_double2(q.up, q.bp);
            if constexpr (FM) lm[O][q.c] = q.mp;
            q.mm = q.m0;
            q.m0 = q.mp;
            q.um = q.u0;
            q.bm = q.b0;
            q.u0 = q.up;
            q.b0 = q.bp;
            q.up = q.ru[N];
            q.mp = q.rm[N];
            q.bp = signed_b(q.up, is_active(q.mp));
        };
        advance(X);
        advance(Y);
        if (ring) advance(E);
        __syncthreads();
    };
    for (int p = i0; p < i0 + ti; p += 2) {
        step(std::integral_constant<int, 0>{}, p);
        step(std::integral_constant<int, 1>{}, p + 1);
    }
    if constexpr (MODE == kNorm) {
        double* ra = (double*)&lv[0][0];
        double* rb = ra + NT;
        ra[t] = s;
        rb[t] = mx;
        __syncthreads();
        for (int h = NT / 2; h > 0; h >>= 1) {
            if (t < h) {
                ra[t] += ra[t + h];
                const double o = rb[t + h];
                if (!(rb[t] >= o)) rb[t] = o;
            }
            __syncthreads();
        }
        if (t == 0) {
            partial[2 * blockIdx.x] = ra[0];
            partial[2 * blockIdx.x + 1] = rb[0];
        }
    }
}

constexpr int kSJ = 8, kSK = 64, kST = 256;  // tile and threads of km_stream

template <int MODE, class M>
hipError_t stream(const Grid& g, const M* flags, const double* w, const double* u, const double* src, double* partial,
                  const float* maskc, const double* wc, double* uc, double* uhat, double* fc, int ti, hipStream_t s)
{
    const unsigned nb = (unsigned)((g.n / ti) * (g.n / kSJ) * (g.n / kSK));
    hipLaunchKernelGGL((km_stream<kSJ, kSK, kST, MODE, M>), dim3(nb), dim3(kST), 0, s, g, flags, w, u, src, partial, maskc,
                       wc, uc, uhat, fc, ti);
    return hipGetLastError();
}

// Planes per workgroup of the streamed passes: enough workgroups for three on every compute unit.
int stream_planes(int n) { return n >= 512 ? 64 : n >= 256 ? 32 : 8; }

// Block partials (number of active cells, max |mask|; NaN propagates).
__global__ void __launch_bounds__(kB) km_count(const float* __restrict__ mask, long long n,
                                               double* __restrict__ partial)
{
    __shared__ double sa[kB], sb[kB];
    double s = 0.0, mx = 0.0;
    for (long long q = (long long)blockIdx.x * kB + threadIdx.x; q < n; q += (long long)gridDim.x * kB) {
        const float m = mask[q];
        if (m > 0.0f) s += 1.0;
        const double a = fabs((double)m);
        if (!(mx >= a)) mx = a;
    }
    block_sum_max(s, mx, sa, sb);
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = s;
        partial[2 * blockIdx.x + 1] = mx;
    }
}

// Byte flags of a mask (1 where > 0) and block partials of the number of cells whose mask is
// neither +1 nor -1 (the flags stand for the mask only when there is none).
__global__ void __launch_bounds__(kB) km_flags(const float* __restrict__ mask, long long n, u8* __restrict__ flags,
                                               double* __restrict__ partial)
{
    __shared__ double sa[kB], sb[kB];
    double s = 0.0, mx = 0.0;
    for (long long q = (long long)blockIdx.x * kB + threadIdx.x; q < n; q += (long long)gridDim.x * kB) {
        const float m = mask[q];
        flags[q] = m > 0.0f ? 1 : 0;
        if (m != 1.0f && m != -1.0f) s += 1.0;
    }
    block_sum_max(s, mx, sa, sb);
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = s;
        partial[2 * blockIdx.x + 1] = mx;
    }
}

// Bit 1 of the flags of active cells with a masked neighbour (bit 0, which is all that is read of
// the neighbours, does not change).
__global__ void __launch_bounds__(kB) km_boundary(Grid g, u8* flags)
{
    const long long q = (long long)blockIdx.x * kB + threadIdx.x;
    if (q >= (1LL << (3 * g.lg)) || !(flags[q] & 1)) return;
    int i, j, k;
    cell_of(g, q, i, j, k);
    const int m = g.n - 1;
    const int all = flags[at(g, (i - 1) & m, j, k)] & flags[at(g, (i + 1) & m, j, k)] & flags[at(g, i, (j - 1) & m, k)] &
                    flags[at(g, i, (j + 1) & m, k)] & flags[at(g, i, j, (k - 1) & m)] & flags[at(g, i, j, (k + 1) & m)];
    if (!(all & 1)) flags[q] = 3;
}

// Coarse mask and fixed values: 8-child means.
__global__ void __launch_bounds__(kB) km_restrict_setup(int lgc, const float* __restrict__ maskf,
                                                        const double* __restrict__ wf, float* __restrict__ maskc,
                                                        double* __restrict__ wc)
{
    const int lg = lgc + 1, nc = 1 << lgc;
    const long long tc = (long long)blockIdx.x * kB + threadIdx.x;
    if (tc >= (1LL << (3 * lgc))) return;
    const int I = (int)(tc >> (2 * lgc)), J = (int)((tc >> lgc) & (nc - 1)), K = (int)(tc & (nc - 1));
    double sm = 0.0, sw = 0.0;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const long long q = ((((long long)(2 * I + a) << lg) + 2 * J + b) << lg) + 2 * K + c;
                sm += maskf[q];
                sw += wf[q];
            }
    maskc[tc] = (float)(0.125 * sm);
    wc[tc] = 0.125 * sw;
}

// Coarsest level (n <= 8) in one workgroup, through LDS: relax the active cells until the rms
// residual over them is <= rtol x its initial value or its rounding floor, or cap sweeps.
__global__ void __launch_bounds__(kB) km_coarsest(Grid g, const float* __restrict__ mask,
                                                  const double* __restrict__ w, double* __restrict__ u,
                                                  const double* __restrict__ f, int cap, double rtol,
                                                  long long* __restrict__ sweeps_done)
{
    __shared__ double su[512], sw[512], sf[512];
    __shared__ float sm[512];
    __shared__ double sa[kB], sb[kB];
    const int nc = 1 << (3 * g.lg);
    for (int q = threadIdx.x; q < nc; q += kB) {
        su[q] = u[q];
        sw[q] = w[q];
        sf[q] = dev::rhs_value(g, f[q]);
        sm[q] = mask[q];
    }
    __syncthreads();
    // rms residual over the active cells, and its rounding floor: per cell one unit in the
    // last place of u times |dL/du| plus one of the summed magnitudes of the terms
    __shared__ double sc[kB];
    auto rms = [&](double& floor) {
        double s = 0.0, fl = 0.0, cnt = 0.0;
        for (int q = threadIdx.x; q < nc; q += kB) {
            const double mi = sm[q];
            if (!(mi > 0.0)) continue;
            int i, j, k;
            cell_of(g, q, i, j, k);
            const OpVal r = masked_op(g, sm, sw, su, i, j, k, su[q], mi, sf[q]);
            s += r.L * r.L;
            const double f1 = 2.220446049250313e-16 *
                              (fabs(r.dL) * fabs(su[q]) + masked_mag(g, sm, sw, su, i, j, k, su[q], mi, sf[q]));
            fl += f1 * f1;
            cnt += 1.0;
        }
        block_sum2(s, fl, sa, sb);
        sc[threadIdx.x] = cnt;
        __syncthreads();
        for (int w2 = kB / 2; w2 > 0; w2 >>= 1) {
            if (threadIdx.x < w2) sc[threadIdx.x] += sc[threadIdx.x + w2];
            __syncthreads();
        }
        cnt = sc[0];
        __syncthreads();
        floor = cnt > 0.0 ? sqrt(fl / cnt) : 0.0;
        return cnt > 0.0 ? sqrt(s / cnt) : 0.0;
    };
    double floor0 = 0.0;
    const double r0 = rtol > 0.0 ? rms(floor0) : 0.0;
    int sweep = 0;
    for (; sweep < cap; ++sweep) {
        if (rtol > 0.0) {
            // stop once reduced by rtol or down to the rounding floor
            double floor;
            const double r = rms(floor);
            if (r <= rtol * r0 || r <= floor) break;
        }
        for (int colour = 0; colour < 2; ++colour) {
            for (int q = threadIdx.x; q < nc; q += kB) {
                const double mi = sm[q];
                int i, j, k;
                cell_of(g, q, i, j, k);
                if (((i + j + k) & 1) != colour || !(mi > 0.0)) continue;
                const double ui = su[q];
                const OpVal r = masked_op(g, sm, sw, su, i, j, k, ui, mi, sf[q]);
                su[q] = ui + bounded(-r.L / r.dL, g.max_step);
            }
            __syncthreads();
        }
    }
    for (int q = threadIdx.x; q < nc; q += kB) u[q] = su[q];
    if (threadIdx.x == 0 && sweeps_done) sweeps_done[0] += sweep;
}

inline unsigned blocks(long long work) { return (unsigned)((work + kB - 1) / kB); }

inline unsigned rblocks(long long work)
{
    const long long b = (work + kB - 1) / kB;
    return (unsigned)(b < kMaxParts ? (b < 1 ? 1 : b) : kMaxParts);
}

}  // namespace

hipError_t masked_count(const float* mask, long long n, double* partial, int* nparts, hipStream_t s)
{
    const unsigned nb = rblocks(n);
    hipLaunchKernelGGL(km_count, dim3(nb), dim3(kB), 0, s, mask, n, partial);
    *nparts = (int)nb;
    return hipGetLastError();
}

hipError_t masked_restrict_setup(const Grid& gc, const float* maskf, const double* wf, float* maskc, double* wc,
                                 hipStream_t s)
{
    hipLaunchKernelGGL(km_restrict_setup, dim3(blocks(cells(gc))), dim3(kB), 0, s, gc.lg, maskf, wf, maskc, wc);
    return hipGetLastError();
}

hipError_t masked_flags(const float* mask, long long n, unsigned char* flags, double* partial, int* nparts,
                        hipStream_t s)
{
    const unsigned nb = rblocks(n);
    hipLaunchKernelGGL(km_flags, dim3(nb), dim3(kB), 0, s, mask, n, flags, partial);
    *nparts = (int)nb;
    return hipGetLastError();
}

hipError_t masked_boundary(const Grid& g, unsigned char* flags, hipStream_t s)
{
    hipLaunchKernelGGL(km_boundary, dim3(blocks(cells(g))), dim3(kB), 0, s, g, flags);
    return hipGetLastError();
}

template <class M>
hipError_t ngs_t(const Grid& g, const M* mask, const double* w, double* u, const double* src, hipStream_t s)
{
    if (g.n < 2) return hipErrorInvalidValue;
    const long long half = cells(g) / 2;
    for (int colour = 0; colour < 2; ++colour) {
        hipLaunchKernelGGL(km_ngs_colour<M>, dim3(blocks(half)), dim3(kB), 0, s, g, mask, w, u, src, colour);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t masked_ngs(const Grid& g, const float* mask, const double* w, double* u, const double* src, hipStream_t s)
{
    return ngs_t(g, mask, w, u, src, s);
}

hipError_t masked_ngs(const Grid& g, const unsigned char* flags, const double* w, double* u, const double* src,
                      hipStream_t s)
{
    return ngs_t(g, flags, w, u, src, s);
}

template <class M>
hipError_t ngs_fused_t(const Grid& g, const M* mask, const double* w, const double* uin, double* uout, const double* src,
                       int ti, hipStream_t s)
{
    if (g.n < kMK || g.n > 1024 || uin == uout || ti < 4 || (ti & 3) || ti > g.n || (g.n % ti) != 0)
        return hipErrorInvalidValue;
    constexpr int TJ = 16;
    FusedSweep a{};
    a.ti = ti;
    a.ntj = g.n / TJ;
    a.ntk = g.n / kMK;
    const unsigned nb = (unsigned)((g.n / ti) * a.ntj * a.ntk);
    hipLaunchKernelGGL((km_ngs_fused<TJ, kMK, M>), dim3(nb), dim3(TJ * kMK / 2), 0, s, g, mask, w, uin, uout, src, a);
    return hipGetLastError();
}

hipError_t masked_ngs_fused(const Grid& g, const unsigned char* flags, const double* w, const double* uin, double* uout,
                            const double* src, int ti, hipStream_t s)
{
    return ngs_fused_t(g, flags, w, uin, uout, src, ti, s);
}

hipError_t masked_ngs_fused(const Grid& g, const float* mask, const double* w, const double* uin, double* uout,
                            const double* src, int ti, hipStream_t s)
{
    return ngs_fused_t(g, mask, w, uin, uout, src, ti, s);
}

template <class M>
hipError_t resid_restrict_t(const Grid& g, const M* mask, const double* w, const double* u, const double* src,
                            const float* maskc, const double* wc, double* uc, double* uhat, double* fc, hipStream_t s)
{
    if (g.n < 2) return hipErrorInvalidValue;
    hipLaunchKernelGGL(km_resid_restrict<M>, dim3(blocks(cells(g) / 8)), dim3(kB), 0, s, g, mask, w, u, src, maskc,
                       wc, uc, uhat, fc);
    return hipGetLastError();
}

hipError_t masked_resid_restrict(const Grid& g, const float* mask, const double* w, const double* u,
                                 const double* src, const float* maskc, const double* wc, double* uc, double* uhat,
                                 double* fc, hipStream_t s)
{
    if (g.n < kMK) return resid_restrict_t(g, mask, w, u, src, maskc, wc, uc, uhat, fc, s);
    return stream<kRestrict>(g, mask, w, u, src, nullptr, maskc, wc, uc, uhat, fc, stream_planes(g.n), s);
}

hipError_t masked_resid_restrict(const Grid& g, const unsigned char* flags, const double* w, const double* u,
                                 const double* src, const float* maskc, const double* wc, double* uc, double* uhat,
                                 double* fc, hipStream_t s)
{
    if (g.n < kMK) return resid_restrict_t(g, flags, w, u, src, maskc, wc, uc, uhat, fc, s);
    return stream<kRestrict>(g, flags, w, u, src, nullptr, maskc, wc, uc, uhat, fc, stream_planes(g.n), s);
}

hipError_t masked_fas_rhs(const Grid& gc, const float* maskc, const double* wc, const double* uhat, double* f,
                          hipStream_t s)
{
    if (gc.n >= kMK)
        return stream<kFas>(gc, maskc, wc, uhat, (const double*)nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, f,
                            stream_planes(gc.n), s);
    hipLaunchKernelGGL(km_fas_rhs, dim3(blocks(cells(gc))), dim3(kB), 0, s, gc, maskc, wc, uhat, f);
    return hipGetLastError();
}

hipError_t masked_prolong(const Grid& gc, const float* maskc, const double* uc, double* uhat, const float* maskf,
                          double* uf, hipStream_t s)
{
    // the correction, then the streaming 27/9/3/1 prolongation into the active fine cells
    hipLaunchKernelGGL(km_coarse_diff, dim3(blocks(cells(gc))), dim3(kB), 0, s, cells(gc), maskc, uc, uhat);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return prolong_add_masked(gc, uf, uhat, maskf, s);
}

long long masked_norm_partials(const Grid& g) { return (long long)blocks(cells(g) / 8); }

template <class M>
hipError_t norm_t(const Grid& g, const M* mask, const double* w, const double* u, const double* src, double* partial,
                  int* nparts, hipStream_t s)
{
    if (g.n < 2) return hipErrorInvalidValue;
    const unsigned nb = blocks(cells(g) / 8);
    hipLaunchKernelGGL(km_norm<M>, dim3(nb), dim3(kB), 0, s, g, mask, w, u, src, partial);
    *nparts = (int)nb;
    return hipGetLastError();
}

// Streamed from 64^3 up: with one thread per cell every neighbour's exponential is formed again.  A
// float mask's at 512^3, 2% of the cells active: 0.55 ms, 1.92 per cell; 256^3 98 against 220 us.
template <class M>
hipError_t norm_any(const Grid& g, const M* mask, const double* w, const double* u, const double* src, double* partial,
                    int* nparts, hipStream_t s)
{
    if (g.n < kMK) return norm_t(g, mask, w, u, src, partial, nparts, s);
    const int ti = stream_planes(g.n);
    const long long nb = (long long)(g.n / ti) * (g.n / kSJ) * (g.n / kSK);
    if (nb > masked_norm_partials(g)) return hipErrorInvalidValue;
    *nparts = (int)nb;
    return stream<kNorm>(g, mask, w, u, src, partial, nullptr, nullptr, nullptr, nullptr, nullptr, ti, s);
}

hipError_t masked_norm(const Grid& g, const float* mask, const double* w, const double* u, const double* src,
                       double* partial, int* nparts, hipStream_t s)
{
    return norm_any(g, mask, w, u, src, partial, nparts, s);
}

hipError_t masked_norm(const Grid& g, const unsigned char* flags, const double* w, const double* u,
                       const double* src, double* partial, int* nparts, hipStream_t s)
{
    return norm_any(g, flags, w, u, src, partial, nparts, s);
}

hipError_t masked_coarsest(const Grid& g, const float* mask, const double* w, double* u, const double* f, int cap,
                           double rtol, long long* sweeps, hipStream_t s)
{
    if (cells(g) > 512) return hipErrorInvalidValue;
    hipLaunchKernelGGL(km_coarsest, dim3(1), dim3(kB), 0, s, g, mask, w, u, f, cap, rtol, sweeps);
    return hipGetLastError();
}

}  // namespace mgfr
