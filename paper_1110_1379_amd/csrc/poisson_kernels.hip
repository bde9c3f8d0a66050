// Kernels of the modified Poisson solve (eq. discrete_poisson): the potential phi of the
// density and of delta R of the scalaron,
//   (1/h^2) [sum of the 6 neighbours of phi - 6 phi] = S - mean(S),
//   S = 2 Om a (rho~ - 1) - (1/2) (A exp(-u/(n+1)) - Sbar)
// with A = (1/3) Om a^4 (n a^2 xi)^(1/(n+1)) and Sbar = Om a^4 (a^-3 + 4 OL/Om), so that the
// bracket of the paper's delta R term, times Om a^4 / 6, is (A exp(-u/(n+1)) - Sbar) / 2.
// Linear multigrid (Sec. V.A.3, correction scheme): red-black Gauss-Seidel, x_i =
// (sum_nb x_nb - h^2 b_i) / 6, the residual restricted by 8-child means, the coarse
// correction prolongated 27/9/3/1 (prolong.hip).  Every level is periodic.
#include <type_traits>

#include "device_fp64.h"

namespace mgfr {
namespace {

constexpr int kB = 256;
constexpr int kTK = 64;

__device__ __forceinline__ unsigned at3(int lg, int i, int j, int k)
{
    return ((((unsigned)i << lg) + (unsigned)j) << lg) + (unsigned)k;
}

// ---- source and its mean -----------------------------------------------------------------
__global__ void __launch_bounds__(kB) kp_source(PoissonSource c, long long n3, const double* __restrict__ rho,
                                                const double* __restrict__ u, double* __restrict__ S,
                                                double* __restrict__ partial)
{
    __shared__ double rs[kB], rm[kB];
    double s = 0.0, mx = 0.0;
    for (long long q = (long long)blockIdx.x * kB + threadIdx.x; q < n3; q += (long long)gridDim.x * kB) {
        const double v = 2.0 * c.D * (rho[q] - 1.0) - 0.5 * (c.A * dev::exp_(-u[q] * c.inv_np1) - c.Sbar);
        S[q] = v;
        s += v;
        const double av = fabs(v);
        if (!(mx >= av)) mx = av;  // NaN propagates
    }
    rs[threadIdx.x] = s;
    rm[threadIdx.x] = mx;
    __syncthreads();
    for (int w = kB / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            rs[threadIdx.x] += rs[threadIdx.x + w];
            const double o = rm[threadIdx.x + w];
            if (!(rm[threadIdx.x] >= o)) rm[threadIdx.x] = o;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = rs[0];
        partial[2 * blockIdx.x + 1] = rm[0];
    }
}

// ---- residual norm: r = b - bmean - lap x (x null: r = b - bmean) --------------------------
__global__ void __launch_bounds__(kB) kp_resid_norm(PGrid g, const double* __restrict__ x, const double* __restrict__ b,
                                                    double bmean, double* __restrict__ partial)
{
    __shared__ double rs[kB], rm[kB];
    const int m = g.n - 1;
    const long long n3 = 1LL << (3 * g.lg);
    double s = 0.0, mx = 0.0;
    for (long long q = (long long)blockIdx.x * kB + threadIdx.x; q < n3; q += (long long)gridDim.x * kB) {
        double r = b[q] - bmean;
        if (x) {
            const int i = (int)(q >> (2 * g.lg)), j = (int)((q >> g.lg) & m), k = (int)(q & m);
            const double lap = (x[at3(g.lg, (i + 1) & m, j, k)] + x[at3(g.lg, (i - 1) & m, j, k)] +
                                x[at3(g.lg, i, (j + 1) & m, k)] + x[at3(g.lg, i, (j - 1) & m, k)] +
                                x[at3(g.lg, i, j, (k + 1) & m)] + x[at3(g.lg, i, j, (k - 1) & m)] - 6.0 * x[q]) *
                               g.inv_hh;
            r -= lap;
        }
        s += r * r;
        const double ar = fabs(r);
        if (!(mx >= ar)) mx = ar;
    }
    rs[threadIdx.x] = s;
    rm[threadIdx.x] = mx;
    __syncthreads();
    for (int w = kB / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            rs[threadIdx.x] += rs[threadIdx.x + w];
            const double o = rm[threadIdx.x + w];
            if (!(rm[threadIdx.x] >= o)) rm[threadIdx.x] = o;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = rs[0];
        partial[2 * blockIdx.x + 1] = rm[0];
    }
}

// ---- one colour of a Gauss-Seidel sweep, in place (levels of 32^3; single sweeps below 256^3) ----
__global__ void __launch_bounds__(kB) kp_ngs_colour(PGrid g, double* __restrict__ x, const double* __restrict__ b,
                                                    double bmean, int colour)
{
    const long long half = 1LL << (3 * g.lg - 1);
    const long long t = (long long)blockIdx.x * kB + threadIdx.x;
    if (t >= half) return;
    const int m = g.n - 1, hk = g.n >> 1;
    const int s = (int)(t & (hk - 1));
    const long long row = t >> (g.lg - 1);
    const int i = (int)(row >> g.lg), j = (int)(row & m);
    const int k = 2 * s + ((i + j + colour) & 1);
    const double sum = x[at3(g.lg, (i + 1) & m, j, k)] + x[at3(g.lg, (i - 1) & m, j, k)] + x[at3(g.lg, i, (j + 1) & m, k)] +
                       x[at3(g.lg, i, (j - 1) & m, k)] + x[at3(g.lg, i, j, (k + 1) & m)] + x[at3(g.lg, i, j, (k - 1) & m)];
    const unsigned q = at3(g.lg, i, j, k);
    x[q] = (sum - g.hh * (b[q] - bmean)) * (1.0 / 6.0);
}

// ---- fused red-black sweep (n >= 64; the solver's single sweeps from 256^3 up), out of place ----
// Same scheme as the nonlinear fused sweep: a workgroup streams the planes of a TJ x 64
// tile; per plane the tile plus a 2-cell in-plane halo is staged in LDS (three buffers, one
// barrier per plane), the i-neighbours stay in registers; at step p the red cells of plane
// p (tile + ring) and then the black cells of plane p-1 (tile) are updated; the ring is
// recomputed from the same old values by every tile that sees it, so the sweep equals the
// two-pass red-then-black sweep.
template <int TJ, int NT>
__global__ void __launch_bounds__(NT) kp_fused(PGrid g, const double* __restrict__ xin, double* __restrict__ xout,
                                               const double* __restrict__ b, double bmean, int ti, int ntj, int ntk)
{
    constexpr int LJ = TJ + 4, LK = kTK + 4, NL = LJ * LK;
    constexpr int NS = (NL + NT - 1) / NT;
    __shared__ double lx[3][NL];
    const int nb = gridDim.x;
    int lid = blockIdx.x;
    if ((nb & 7) == 0) lid = (lid & 7) * (nb >> 3) + (lid >> 3);
    const int tk = lid % ntk;
    lid /= ntk;
    const int tj = lid % ntj;
    const int ci = lid / ntj;
    const int i0 = ci * ti, j0 = tj * TJ, k0 = tk * kTK;
    const int lg = g.lg, m = g.n - 1;
    const int last = i0 + ti + 1;  // last plane read
    const double hh = g.hh;

    unsigned col[NS];
    int par[NS], fl[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int c = threadIdx.x + s * NT;
        col[s] = 0;
        par[s] = 0;
        fl[s] = 0;
        if (c < NL) {
            const int jj = c / LK, kk = c - jj * LK;
            const int gj = (j0 - 2 + jj) & m, gk = (k0 - 2 + kk) & m;
            col[s] = (unsigned)((gj << lg) | gk);
            par[s] = (gj + gk) & 1;
            fl[s] = 1;
            if (jj >= 1 && jj <= LJ - 2 && kk >= 1 && kk <= LK - 2) fl[s] |= 2;
            if (jj >= 2 && jj <= LJ - 3 && kk >= 2 && kk <= LK - 3) fl[s] |= 4;
        }
    }
    // element offsets fit in 32 bits (n <= 1024)
    auto offset = [&](int p, int s) -> unsigned { return ((unsigned)(p & m) << (2 * lg)) + col[s]; };
    auto buf = [&](int p) { return (p - i0 + 3) % 3; };

    // x of planes p-2 .. p+1, the right-hand side (minus its mean, times h^2) of planes
    // p-1 .. p+1, and the raw loads of plane p+2
    double xm2[NS], xm1[NS], x0[NS], xp1[NS], bm1[NS], b0[NS], bp1[NS], xn2[NS], bn2[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        xm2[s] = xm1[s] = x0[s] = xp1[s] = bm1[s] = b0[s] = bp1[s] = xn2[s] = bn2[s] = 0.0;
        if (fl[s]) {
            xm1[s] = xin[offset(i0 - 2, s)];
            x0[s] = xin[offset(i0 - 1, s)];
            xp1[s] = xin[offset(i0, s)];
            xn2[s] = xin[offset(i0 + 1, s)];
            bm1[s] = hh * (b[offset(i0 - 2, s)] - bmean);
            b0[s] = hh * (b[offset(i0 - 1, s)] - bmean);
            bp1[s] = hh * (b[offset(i0, s)] - bmean);
            bn2[s] = b[offset(i0 + 1, s)];
            lx[buf(i0 - 1)][threadIdx.x + s * NT] = x0[s];
        }
    }
    __syncthreads();
    for (int p = i0 - 1; p <= i0 + ti; ++p) {
        const bool more3 = p + 3 <= last;
        double xn3[NS], bn3[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            xn3[s] = bn3[s] = 0.0;
            if (more3 && fl[s]) {
                xn3[s] = xin[offset(p + 3, s)];
                bn3[s] = b[offset(p + 3, s)];
            }
        }
        double* LA = lx[buf(p)];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int c = threadIdx.x + s * NT;
            if ((fl[s] & 2) && ((p + par[s]) & 1) == 0) {
                const double v = (xm1[s] + xp1[s] + LA[c - LK] + LA[c + LK] + LA[c - 1] + LA[c + 1] - b0[s]) * (1.0 / 6.0);
                x0[s] = v;
                LA[c] = v;
            }
        }
        if (p - 1 >= i0) {
            const double* LB = lx[buf(p - 1)];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int c = threadIdx.x + s * NT;
                if (fl[s] & 4) {
                    if (((p - 1 + par[s]) & 1) == 1)
                        xm1[s] = (xm2[s] + x0[s] + LB[c - LK] + LB[c + LK] + LB[c - 1] + LB[c + 1] - bm1[s]) * (1.0 / 6.0);
                    xout[offset(p - 1, s)] = xm1[s];
                }
            }
        }
        double* LC = lx[buf(p + 1)];
        const bool more2 = p + 2 <= last;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (fl[s]) LC[threadIdx.x + s * NT] = xp1[s];
            xm2[s] = xm1[s];
            xm1[s] = x0[s];
            bm1[s] = b0[s];
            x0[s] = xp1[s];
            b0[s] = bp1[s];
            if (more2 && fl[s]) {
                xp1[s] = xn2[s];
                bp1[s] = hh * (bn2[s] - bmean);
            }
            xn2[s] = xn3[s];
            bn2[s] = bn3[s];
        }
        __syncthreads();
    }
}

// ---- two fused red-black sweeps per pass, out of place -------------------------------------
// Temporal blocking of the sweep above: one pass over the planes applies two complete
// red-black sweeps, A then B, so x and b come from HBM once for both.  At plane step p:
//   A red on plane p (tile + 3-cell ring), A black on plane p-1 (tile + 2-cell ring),
//   B red on plane p-2 (tile + 1-cell ring), B black on plane p-3 (tile),
// each reading exactly the values that the one-sweep kernel would have at that point (the
// rings are recomputed from identical values by every tile that sees them), with the same
// arithmetic, so the pass equals two one-sweep launches bit for bit.  The tile carries a
// 4-cell in-plane halo; a plane's LDS buffer serves, in turn, as the staged plane, A's red
// and black planes, then B's red and black planes (five buffers, one barrier per plane).
// The planes i0-4 .. i0+ti+3 are read and i0 .. i0+ti-1 written.
//
// A thread owns two k-adjacent columns of the tile and its halo.  At step p the one whose cell on
// plane p is red makes all four updates of the step, the other none, and the roles alternate:
// every lane updates.  No update of a step reads a cell that the step writes for another column,
// so the LDS reads run ahead of the updates and the writes come last.  The planes below p+1 are in
// LDS (a row's even columns before its odd ones, so the lanes' active columns are neighbours); a
// column keeps its planes p+1 and p+2, the last value of its second sweep and its right-hand
// sides, each used by A and two steps later by B.  A ring too far out for an update gets a value
// that nothing valid reads: a cell's validity shrinks by one ring per update, and the tile is
// written after four.
// Bound by latency: a step of 14 wavefronts is one barrier, four dependent updates and the wait for
// the loads of two steps before (vector units busy 17 - 20%, LDS conflicts 12 - 14% of the cycles).
// 97 VGPRs let one workgroup run on a compute unit; at 64 for a second one it spills (1.06 ms), 8 x
// 64 and 16 x 32 tiles at two or three a unit re-read more halo (1.07 ms), and 32 x 64 with two pairs
// per thread spills (1.02 ms).  Measured at 512^3: 0.853 ms per pass, 3.8 TB/s of the 3.2 GB it cannot
// do without; with a slot for every cell of tile and halo, half of them idle in each phase, and
// six planes of x in registers (157 VGPRs) 1.18 ms.  256^3: 0.112 against 0.154 ms.
struct Col2 {
    double xr[2], vr;     // plane q of x in xr[(q - p0) & 1]; the last value of sweep B
    double bR[2], bK[2];  // right-hand sides of this active step's red and black cell and of the last one's
    unsigned col;         // byte offset of (j,k) within a plane
    int c, cu, cl;        // LDS cell staged and cell updated; the latter's k-neighbour below, the one above follows it
    bool own;             // in the tile
};

// PROL: the pass starts from x + P(xc), xc the correction of the level below (trilinear, 27/9/3/1
// over 64: in-plane interpolants of a column on the two nearest coarse planes, blended 3:1), added to
// each value of x as its plane is staged, instead of in a pass of its own over x.  i0 is even, so
// planes p0+1, p0+3, .. are even: their two coarse planes are at hand, and the plane after each
// needs the next one.  512^3: 0.908 ms, the pass and the correction by itself 0.832 + 0.412; 256^3
// 123 us, 116 + 52.
struct ColC {
    double cur, prev;  // interpolants on the coarse plane of the plane staged, and on the one before
    unsigned jk, jnk;  // offsets of the coarse neighbours across k on the two coarse rows
};

template <int TJ, int TK, int NT, bool PROL>
__global__ void __launch_bounds__(NT)
kp_fused2(PGrid g, const double* __restrict__ xin, double* __restrict__ xout, const double* __restrict__ b, double bmean,
          int ti, int ntj, int ntk, const double* __restrict__ xc)
{
    constexpr int H = 4, LJ = TJ + 2 * H, LK = TK + 2 * H, HK = LK / 2, NL = LJ * LK, NP = NL / 2;
    static_assert(NP <= NT, "one column pair per thread");
    // the cell past a plane's tile is the one of the columns that stage or update none
    constexpr int NB = NL + 2;
    __shared__ double lx[5 * NB + LK];
    const int nb = gridDim.x;
    int lid = blockIdx.x;
    if ((nb & 7) == 0) lid = (lid & 7) * (nb >> 3) + (lid >> 3);
    const int tk = lid % ntk;
    lid /= ntk;
    const int tj = lid % ntj;
    const int ci = lid / ntj;
    const int i0 = ci * ti, j0 = tj * TJ, k0 = tk * TK;
    const int lg = g.lg, m = g.n - 1;
    const int p0 = i0 - H + 1;  // first step
    const double hh = g.hh;

    // X is the column of a pair with the red cell on plane p0, Y the other
    Col2 X{}, Y{};
    // a plane's base is scalar, a column's byte offset fits in 32 bits; planes past the last one read
    // are loaded, wrapped, and not used
    // (both opaque: the compiler would keep a 64-bit pointer per column and add to it)
    using gptr = __attribute__((address_space(1))) char*;
    auto plane = [&](const double* f, int p) -> gptr {
        gptr q = (gptr)(f + ((size_t)(p & m) << (2 * lg)));
        asm("" : "+s"(q));
        return q;
    };
    using gval = __attribute__((address_space(1))) double*;
    auto place = [&](unsigned o) -> unsigned {
        asm("" : "+v"(o));
        return o;
    };
    auto at = [&](const double* f, int p, const Col2& q) -> double { return *(gval)(plane(f, p) + place(q.col)); };
    auto put = [&](int p, const Col2& q, double v) { *(gval)(plane(xout, p) + place(q.col)) = v; };
    // LDS bases of the planes p+1 .. p-3
    int u1 = NB, u0 = 0, d1 = 4 * NB, d2 = 3 * NB, d3 = 2 * NB;
    // PROL: X's and Y's interpolants, the coarse values they share (rows J and Jn at K), and all six of
    // the next coarse plane, in flight
    ColC CX{}, CY{};
    unsigned c0 = 0, c1 = 0;
    double r0 = 0.0, r1 = 0.0, rx0 = 0.0, rx1 = 0.0, ry0 = 0.0, ry1 = 0.0;
    const int lgc = lg - 1, mc = m >> 1;
    auto coarse = [&](int I, unsigned o) -> double {
        gptr q = (gptr)(xc + ((size_t)(I & mc) << (2 * lgc)));
        asm("" : "+s"(q));
        return *(gval)(q + place(o));
    };
    auto request_c = [&](int I) {
        r0 = coarse(I, c0);
        r1 = coarse(I, c1);
        rx0 = coarse(I, CX.jk);
        rx1 = coarse(I, CX.jnk);
        ry0 = coarse(I, CY.jk);
        ry1 = coarse(I, CY.jnk);
    };
    // the interpolant on the next coarse plane, from the values in flight
    auto next_c = [&](ColC& q, double s0, double s1) {
        q.prev = q.cur;
        q.cur = (9.0 / 16.0) * r0 + (3.0 / 16.0) * (r1 + s0) + (1.0 / 16.0) * s1;
    };
    {
        const int t = threadIdx.x;
        const bool on = t < NP;
        const int jj = on ? t / HK : 0, kk = on ? 2 * (t - jj * HK) : 0;
        const int gj = (j0 - H + jj) & m, gk = (k0 - H + kk) & m;
        const int sx = (p0 + gj + gk) & 1;
        double ex0 = 0.0, ex1 = 0.0, ey0 = 0.0, ey1 = 0.0;  // the corrections of planes p0-1 and p0
        if constexpr (PROL) {
            const int J = gj >> 1, Jn = (J + ((gj & 1) ? 1 : -1)) & mc, K = gk >> 1;
            const int KX = (K + (sx ? 1 : -1)) & mc, KY = (K + (sx ? -1 : 1)) & mc;
            auto cell = [&](int j, int k) { return (unsigned)((j << lgc) | k) * (unsigned)sizeof(double); };
            c0 = cell(J, K);
            c1 = cell(Jn, K);
            CX.jk = cell(J, KX);
            CX.jnk = cell(Jn, KX);
            CY.jk = cell(J, KY);
            CY.jnk = cell(Jn, KY);
            const int I = (p0 - 1) >> 1;  // of planes p0-1 and p0
            for (int d = -1; d <= 1; ++d) {
                request_c(I + d);
                next_c(CX, rx0, rx1);
                next_c(CY, ry0, ry1);
                if (d == 0) {
                    ex0 = 0.75 * CX.cur + 0.25 * CX.prev;
                    ey0 = 0.75 * CY.cur + 0.25 * CY.prev;
                }
            }
            ex1 = 0.75 * CX.prev + 0.25 * CX.cur;
            ey1 = 0.75 * CY.prev + 0.25 * CY.cur;
            request_c(I + 2);
        }
        auto setup = [&](Col2& q, int d, double e0, double e1) {
            const int k = kk + d;
            q.col = (unsigned)((gj << lg) | (gk + d)) * sizeof(double);
            q.c = on ? jj * LK + (k & 1) * HK + (k >> 1) : NL;
            const int rj = jj < LJ - 1 - jj ? jj : LJ - 1 - jj, rk = k < LK - 1 - k ? k : LK - 1 - k;
            const int r = on ? (rj < rk ? rj : rk) : 0;
            q.cu = r >= 1 ? q.c : NL;
            q.cl = r >= 1 ? jj * LK + ((k & 1) ? k >> 1 : HK + (k >> 1) - 1) : NL;
            q.own = r >= H;
            lx[d1 + q.c] = at(xin, p0 - 1, q) + e0;
            lx[u0 + q.c] = at(xin, p0, q) + e1;
            q.xr[1] = at(xin, p0 + 1, q);
            q.xr[0] = at(xin, p0 + 2, q);
        };
        setup(X, sx, ex0, ex1);
        setup(Y, 1 - sx, ey0, ey1);
        // the first steps need only the red cells' sides: X's on p0, Y's on p0+1
        X.bR[0] = at(b, p0, X);
        Y.bR[0] = at(b, p0 + 1, Y);
    }
    __syncthreads();

    // The slots are compile-time constants (N1: of plane p+1, and of p+3; S: of this active step's
    // right-hand sides, the other one of the last one's and of the next one's): a copy of a register
    // whose load is in flight would wait for it.
    auto step = [&](auto N1c, auto Sc, int p, Col2& A, Col2& B, ColC& CA, ColC& CB) {
        constexpr int N1 = decltype(N1c)::value, S = decltype(Sc)::value, T = S ^ 1;
        struct Nb {
            double m, jm, jp, km, kp;
        };
        // the cell below (plane dm) and the in-plane neighbours (plane d)
        auto gather = [&](const Col2& q, int dm, int d) -> Nb {
            return {lx[dm + q.cu], lx[d + q.cu - LK], lx[d + q.cu + LK], lx[d + q.cl], lx[d + q.cl + 1]};
        };
        auto relax = [&](const Nb& q, double xm, double xp, double bv) -> double {
            // hh is a power of two, so the fma rounds as the product and difference do; the
            // result is rounded before the next update adds it
#pragma clang fp contract(off)
            return __builtin_fma(-hh, bv - bmean, xm + xp + q.jm + q.jp + q.km + q.kp) * (1.0 / 6.0);
        };
        // plane p+1 of x; PROL: an odd one lies between its own coarse plane and the next
        double xa = A.xr[N1], xb = B.xr[N1];
        if constexpr (PROL && N1 == 1) {
            xa += 0.75 * CA.cur + 0.25 * CA.prev;
            xb += 0.75 * CB.cur + 0.25 * CB.prev;
        } else if constexpr (PROL) {
            next_c(CX, rx0, rx1);
            next_c(CY, ry0, ry1);
            request_c(((p + 1) >> 1) + 2);
            xa += 0.75 * CA.prev + 0.25 * CA.cur;
            xb += 0.75 * CB.prev + 0.25 * CB.cur;
        }
        const Nb q0 = gather(A, d1, u0), q1 = gather(A, d2, d1);
        const double a0 = relax(q0, q0.m, xa, A.bR[S]);  // A red, plane p
        const Nb q2 = gather(A, d3, d2);
        const double a1 = relax(q1, q1.m, a0, A.bK[S]);  // A black, plane p-1
        const Nb q3 = gather(A, d3, d3);
        const double a2 = relax(q2, q2.m, a1, A.bR[T]);  // B red, plane p-2
        const double a3 = relax(q3, A.vr, a2, A.bK[T]);  // B black, plane p-3
        lx[u0 + A.cu] = a0;
        lx[d1 + A.cu] = a1;
        lx[d2 + A.cu] = a2;
        A.vr = a2;
        // A is active again at step p+2
        A.bR[T] = at(b, p + 2, A);
        A.bK[T] = at(b, p + 1, A);
        // stage plane p+1 and request p+3
        lx[u1 + A.c] = xa;
        lx[u1 + B.c] = xb;
        A.xr[N1] = at(xin, p + 3, A);
        B.xr[N1] = at(xin, p + 3, B);
        if (A.own && (unsigned)(p - 3 - i0) < (unsigned)ti) {  // the tile of plane p-3 is final
            put(p - 3, A, a3);
            put(p - 3, B, B.vr);
        }
        const int f = d3;
        d3 = d2;
        d2 = d1;
        d1 = u0;
        u0 = u1;
        u1 = f;
        __syncthreads();
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    const int steps = ti + 2 * H - 2;  // one more for an odd ti
    for (int p = p0;; p += 4) {
        step(I1{}, I0{}, p, X, Y, CX, CY);
        step(I0{}, I0{}, p + 1, Y, X, CY, CX);
        if (p + 2 >= p0 + steps) break;
        step(I1{}, I1{}, p + 2, X, Y, CX, CY);
        step(I0{}, I1{}, p + 3, Y, X, CY, CX);
        if (p + 4 >= p0 + steps) break;
    }
}

// ---- residual restricted to the coarse level: bc = R (b - bmean - lap x) ---------------------
__global__ void __launch_bounds__(kB) kp_resid_restrict(PGrid g, const double* __restrict__ x,
                                                        const double* __restrict__ b, double bmean,
                                                        double* __restrict__ bc)
{
    const int lgc = g.lg - 1, nc = g.n >> 1, m = g.n - 1;
    const long long tc = (long long)blockIdx.x * kB + threadIdx.x;
    if (tc >= (1LL << (3 * lgc))) return;
    const int I = (int)(tc >> (2 * lgc)), J = (int)((tc >> lgc) & (nc - 1)), K = (int)(tc & (nc - 1));
    double s = 0.0;
    for (int a = 0; a < 2; ++a)
        for (int bb = 0; bb < 2; ++bb)
            for (int z = 0; z < 2; ++z) {
                const int i = 2 * I + a, j = 2 * J + bb, k = 2 * K + z;
                const unsigned q = at3(g.lg, i, j, k);
                const double lap = (x[at3(g.lg, (i + 1) & m, j, k)] + x[at3(g.lg, (i - 1) & m, j, k)] +
                                    x[at3(g.lg, i, (j + 1) & m, k)] + x[at3(g.lg, i, (j - 1) & m, k)] +
                                    x[at3(g.lg, i, j, (k + 1) & m)] + x[at3(g.lg, i, j, (k - 1) & m)] - 6.0 * x[q]) *
                                   g.inv_hh;
                s += b[q] - bmean - lap;
            }
    bc[tc] = 0.125 * s;
}

// ---- streaming residual (n >= 64): norm partials or restriction ----------------------------
// r = b - bmean - lap x.  A workgroup owns a TJ x 64 tile of columns and a chunk of ti planes
// (ti even): x of the tile plus a one-cell in-plane halo is staged in LDS per plane (two
// buffers, one barrier per plane), the i-neighbours stay in registers, and the loads run two
// planes ahead.  NORM: per-workgroup (sum r^2, max |r|); RESTRICT: 8-child means into bc.
template <int TJ, int NT, bool RESTRICT>
__global__ void __launch_bounds__(NT) kp_resid_stream(PGrid g, const double* __restrict__ x,
                                                      const double* __restrict__ b, double bmean, int ti, int ntj,
                                                      int ntk, double* __restrict__ out)
{
    constexpr int LJ = TJ + 2, LK = kTK + 2, NL = LJ * LK;
    constexpr int NS = (NL + NT - 1) / NT;
    __shared__ double lx[2][NL];
    __shared__ double rr[RESTRICT ? TJ * kTK : 1];
    __shared__ double red_s[NT], red_m[NT];
    const int nb = gridDim.x;
    int lid = blockIdx.x;
    if ((nb & 7) == 0) lid = (lid & 7) * (nb >> 3) + (lid >> 3);
    const int tk = lid % ntk;
    lid /= ntk;
    const int tj = lid % ntj;
    const int ci = lid / ntj;
    const int i0 = ci * ti, j0 = tj * TJ, k0 = tk * kTK;
    const int lg = g.lg, m = g.n - 1;
    const int last = i0 + ti;  // last plane read
    unsigned col[NS];
    int fl[NS], li[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int c = threadIdx.x + s * NT;
        col[s] = 0;
        fl[s] = li[s] = 0;
        if (c < NL) {
            const int jj = c / LK, kk = c - jj * LK;
            col[s] = (unsigned)((((j0 - 1 + jj) & m) << lg) | ((k0 - 1 + kk) & m));
            fl[s] = 1;
            if (jj >= 1 && jj <= TJ && kk >= 1 && kk <= kTK) {
                fl[s] |= 2;
                li[s] = (jj - 1) * kTK + (kk - 1);
            }
        }
    }
    auto offset = [&](int p, int s) -> unsigned { return ((unsigned)(p & m) << (2 * lg)) + col[s]; };
    // x of planes p-1, p, p+1 and b of plane p in registers; x of p+2 (and b of p+1) in flight
    double xm1[NS], x0[NS], xp1[NS], xn2[NS], b0[NS], prev[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        xm1[s] = x0[s] = xp1[s] = xn2[s] = b0[s] = prev[s] = 0.0;
        if (fl[s] & 2) b0[s] = b[offset(i0, s)];
        if (fl[s]) {
            xm1[s] = x[offset(i0 - 1, s)];
            x0[s] = x[offset(i0, s)];
            xp1[s] = x[offset(i0 + 1, s)];
            xn2[s] = x[offset(i0 + 2, s)];
            lx[0][threadIdx.x + s * NT] = x0[s];
        }
    }
    __syncthreads();
    double acc = 0.0, mx = 0.0;
    for (int p = i0; p < i0 + ti; ++p) {
        const bool more3 = p + 3 <= last, moreb = p + 1 < last;
        double xn3[NS], b1[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            xn3[s] = b1[s] = 0.0;
            if (fl[s] && more3) xn3[s] = x[offset(p + 3, s)];
            if ((fl[s] & 2) && moreb) b1[s] = b[offset(p + 1, s)];
        }
        const double* LX = lx[(p - i0) & 1];
        const bool second = RESTRICT && ((p - i0) & 1);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int c = threadIdx.x + s * NT;
            if (fl[s] & 2) {
                const double lap =
                    (xm1[s] + xp1[s] + LX[c - LK] + LX[c + LK] + LX[c - 1] + LX[c + 1] - 6.0 * x0[s]) * g.inv_hh;
                const double r = b0[s] - bmean - lap;
                if (!RESTRICT) {
                    acc += r * r;
                    const double ar = fabs(r);
                    if (!(mx >= ar)) mx = ar;
                } else if (second) {
                    rr[li[s]] = prev[s] + r;
                } else {
                    prev[s] = r;
                }
            }
        }
        if (second) {
            __syncthreads();
            const int lgc = lg - 1;
            for (int t = threadIdx.x; t < (TJ / 2) * (kTK / 2); t += NT) {
                const int cj = t / (kTK / 2), ck = t - cj * (kTK / 2);
                const int q = (2 * cj) * kTK + 2 * ck;
                const double sr = rr[q] + rr[q + 1] + rr[q + kTK] + rr[q + kTK + 1];
                out[at3(lgc, (p & m) >> 1, (j0 >> 1) + cj, (k0 >> 1) + ck)] = 0.125 * sr;
            }
        }
        double* NX = lx[(p + 1 - i0) & 1];
        const bool more2 = p + 2 <= last;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (fl[s]) NX[threadIdx.x + s * NT] = xp1[s];
            xm1[s] = x0[s];
            x0[s] = xp1[s];
            if (more2) xp1[s] = xn2[s];
            xn2[s] = xn3[s];
            b0[s] = b1[s];
        }
        __syncthreads();
    }
    if (!RESTRICT) {
        const int t = threadIdx.x;
        red_s[t] = acc;
        red_m[t] = mx;
        __syncthreads();
        for (int w = NT / 2; w > 0; w >>= 1) {
            if (t < w) {
                red_s[t] += red_s[t + w];
                const double o = red_m[t + w];
                if (!(red_m[t] >= o)) red_m[t] = o;
            }
            __syncthreads();
        }
        if (t == 0) {
            out[2 * blockIdx.x] = red_s[0];
            out[2 * blockIdx.x + 1] = red_m[0];
        }
    }
}

__global__ void __launch_bounds__(kB) kp_add(double* __restrict__ x, double v, long long n)
{
    for (long long q = (long long)blockIdx.x * kB + threadIdx.x; q < n; q += (long long)gridDim.x * kB) x[q] += v;
}

unsigned grid_for(long long n)
{
    long long b = (n + kB - 1) / kB;
    if (b > 8192) b = 8192;
    return (unsigned)(b < 1 ? 1 : b);
}

}  // namespace

int poisson_partials(long long n) { return (int)grid_for(n); }

hipError_t poisson_source(const PoissonSource& c, long long n3, const double* rho, const double* u, double* S,
                          double* partial, hipStream_t s)
{
    hipLaunchKernelGGL(kp_source, dim3(grid_for(n3)), dim3(kB), 0, s, c, n3, rho, u, S, partial);
    return hipGetLastError();
}

// Streaming residual launch geometry: TJ x 64 tiles, ti planes per workgroup (even, dividing
// n), few enough workgroups for the partial-sum scratch.
constexpr int kRTJ = 8, kRNT = 256;

int resid_planes(int n)
{
    const long long tiles = (long long)(n / kRTJ) * (n / kTK);
    int ti = 8;
    while (ti < n && tiles * (n / ti) > 8192) ti *= 2;
    return ti;
}

hipError_t poisson_resid_norm(const PGrid& g, const double* x, const double* b, double bmean, double* partial,
                              int* nparts, hipStream_t s)
{
    if (x && g.n >= kTK && g.n <= 1024) {
        const int ti = resid_planes(g.n), ntj = g.n / kRTJ, ntk = g.n / kTK;
        const unsigned nb = (unsigned)((g.n / ti) * ntj * ntk);
        *nparts = (int)nb;
        hipLaunchKernelGGL((kp_resid_stream<kRTJ, kRNT, false>), dim3(nb), dim3(kRNT), 0, s, g, x, b, bmean, ti, ntj,
                           ntk, partial);
        return hipGetLastError();
    }
    const unsigned nb = grid_for(1LL << (3 * g.lg));
    *nparts = (int)nb;
    hipLaunchKernelGGL(kp_resid_norm, dim3(nb), dim3(kB), 0, s, g, x, b, bmean, partial);
    return hipGetLastError();
}

hipError_t poisson_ngs(const PGrid& g, double* x, const double* b, double bmean, hipStream_t s)
{
    const long long half = 1LL << (3 * g.lg - 1);
    for (int colour = 0; colour < 2; ++colour)
        hipLaunchKernelGGL(kp_ngs_colour, dim3((unsigned)((half + kB - 1) / kB)), dim3(kB), 0, s, g, x, b, bmean,
                           colour);
    return hipGetLastError();
}

// below 256 a level has too few tiles to fill the chip for a single sweep; the two-sweep pass, whose
// alternative is four launches, is the faster one wherever its tile fits: 128^3 19 against 42 us,
// 64^3 10.5 against 16.3 us
int poisson_fused_min_n() { return 4 * kTK; }
int poisson_fused2_min_n() { return kTK; }

hipError_t poisson_ngs_fused(const PGrid& g, const double* xin, double* xout, const double* b, double bmean, int ti,
                             hipStream_t s)
{
    constexpr int TJ = 16, NT = 512;
    if (g.n < kTK || g.n > 1024 || xin == xout || ti < 1 || ti > g.n || (g.n % ti) != 0) return hipErrorInvalidValue;
    const int ntj = g.n / TJ, ntk = g.n / kTK;
    const unsigned nb = (unsigned)((g.n / ti) * ntj * ntk);
    hipLaunchKernelGGL((kp_fused<TJ, NT>), dim3(nb), dim3(NT), 0, s, g, xin, xout, b, bmean, ti, ntj, ntk);
    return hipGetLastError();
}

// One workgroup per compute unit and pass where the level has the tiles for it (n <= 512), and as
// few of the 6 planes that a chunk computes again as that allows: 512^3 with 512 planes 0.853 ms,
// with 128 0.916; 256^3 with 64 0.112, with 32 0.120 and with 128 0.176.
int poisson_fused2_planes(int n)
{
    const int ti = (n / 16) * (n / 64) * n / 256;
    return ti < 2 ? 2 : ti < n ? ti : n;
}

hipError_t poisson_ngs_fused2(const PGrid& g, const double* xin, double* xout, const double* b, double bmean, int ti,
                              const double* xc, hipStream_t s)
{
    constexpr int TJ = 16, TK = 64, NT = 896;  // 24 x 72 cells with the halo: 864 column pairs
    if (g.n < TK || g.n > 1024 || xin == xout || ti < 1 || ti > g.n || (g.n % ti) != 0 || (xc && (ti & 1)))
        return hipErrorInvalidValue;
    const int ntj = g.n / TJ, ntk = g.n / TK;
    const unsigned nb = (unsigned)((g.n / ti) * ntj * ntk);
    if (xc)
        hipLaunchKernelGGL((kp_fused2<TJ, TK, NT, true>), dim3(nb), dim3(NT), 0, s, g, xin, xout, b, bmean, ti, ntj, ntk, xc);
    else
        hipLaunchKernelGGL((kp_fused2<TJ, TK, NT, false>), dim3(nb), dim3(NT), 0, s, g, xin, xout, b, bmean, ti, ntj, ntk, xc);
    return hipGetLastError();
}

hipError_t poisson_resid_restrict(const PGrid& g, const double* x, const double* b, double bmean, double* bc,
                                  hipStream_t s)
{
    if (g.n >= kTK && g.n <= 1024) {
        const int ti = resid_planes(g.n), ntj = g.n / kRTJ, ntk = g.n / kTK;
        const unsigned nb = (unsigned)((g.n / ti) * ntj * ntk);
        hipLaunchKernelGGL((kp_resid_stream<kRTJ, kRNT, true>), dim3(nb), dim3(kRNT), 0, s, g, x, b, bmean, ti, ntj,
                           ntk, bc);
        return hipGetLastError();
    }
    const long long ncell = 1LL << (3 * (g.lg - 1));
    hipLaunchKernelGGL(kp_resid_restrict, dim3((unsigned)((ncell + kB - 1) / kB)), dim3(kB), 0, s, g, x, b, bmean, bc);
    return hipGetLastError();
}

hipError_t poisson_add(double* x, double v, long long n, hipStream_t s)
{
    hipLaunchKernelGGL(kp_add, dim3(grid_for(n)), dim3(kB), 0, s, x, v, n);
    return hipGetLastError();
}

}  // namespace mgfr
