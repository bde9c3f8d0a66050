// Single-precision kernels of the defect-correction (mixed precision) domain solver.
//
// The outer double-precision loop holds u and its residual d = L(u) - f.  In between, a
// single-precision FAS multigrid solves N(e) = r for the correction e of u, in the
// correction form of device_fp32.h (r = -d, base ub = u rounded to single precision).
// The coarse levels of this inner multigrid use the restricted base R ub.  Smoother:
// red-black Newton-Gauss-Seidel on N (Sec. V.B.1 applied to the correction equation).
#include "device_fp32.h"
#include "fused_fp32.h"

#include <type_traits>

namespace mgfr {
namespace {

using dev32::em1f;
using dev32::make_v;
using dev32::newton32;
using dev32::Op32;
using dev32::op32;
using dev32::Res32;
using dev32::V32;

constexpr int kBlock = 256;
constexpr int kTK = 64;

__device__ __forceinline__ long long at(int lg, int i, int j, int k)
{
    return ((((long long)i << lg) + j) << lg) + k;
}

__device__ __forceinline__ void nbr_index(int lg, int i, int j, int k, long long (&q)[6])
{
    const int m = (1 << lg) - 1;
    q[0] = at(lg, (i - 1) & m, j, k);
    q[1] = at(lg, (i + 1) & m, j, k);
    q[2] = at(lg, i, (j - 1) & m, k);
    q[3] = at(lg, i, (j + 1) & m, k);
    q[4] = at(lg, i, j, (k - 1) & m);
    q[5] = at(lg, i, j, (k + 1) & m);
}

// ---- per-colour sweep, in place (small levels) ------------------------------------------
__global__ void __launch_bounds__(kBlock) k32_ngs_colour(Grid g, const float* __restrict__ ub, float* __restrict__ e,
                                                         const float* __restrict__ f, int colour)
{
    if (g.halt && *g.halt) return;
    const Op32 o = op32(g);
    const long long half = 1LL << (3 * g.lg - 1);
    const long long t = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (t >= half) return;
    const int hk = g.n >> 1;
    const int s = (int)(t & (hk - 1));
    const long long row = t >> (g.lg - 1);
    const int i = (int)(row >> g.lg), j = (int)(row & (g.n - 1));
    const int k = 2 * s + ((i + j + colour) & 1);
    const long long q = at(g.lg, i, j, k);
    long long qn[6];
    nbr_index(g.lg, i, j, k, qn);
    V32 nb[6];
#pragma unroll
    for (int v = 0; v < 6; ++v) nb[v] = make_v(ub[qn[v]], e[qn[v]]);
    const V32 c = make_v(ub[q], e[q]);
    const Res32 r = dev32::corr_op(o, c, nb, f[q]);
    e[q] = c.e + newton32(r, o.max_step);
}

// ---- fused red-black sweep (n >= 64), same scheme as the double-precision one ----------
// Three LDS plane buffers, one barrier per plane, the red ring recomputed per tile.  A thread
// owns a pair of k-adjacent columns: at every plane step exactly one column of each pair
// holds the cells to update (red on plane p, black on plane p-1), and the two swap at the
// next step, so with the step loop unrolled by two every lane updates a cell at every step.
using fused32::Col32;

template <int TJ, int TK, int NT>
__global__ void __launch_bounds__(NT) k32_fused(Grid g, const float* __restrict__ ub, const float* __restrict__ ein,
                                                float* __restrict__ eout, const float* __restrict__ f,
                                                FusedSweep32 a)
{
    if (g.halt && *g.halt) return;
    constexpr int LJ = TJ + 4, LK = TK + 4, NL = LJ * LK, NP = NL / 2;
    static_assert(NP <= NT, "one column pair per thread");
    __shared__ V32 lv[3][NL];
    const Op32 o = op32(g);
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

    // X: the column of the pair whose cell on plane i0-1 is red; Y: the other one
    Col32 X{}, Y{};
    const int pc = threadIdx.x;
    if (pc < NP) {
        const int jj = pc / (LK / 2), kk0 = 2 * (pc - jj * (LK / 2));
        const int gj = (j0 - 2 + jj) & m, gk0 = (k0 - 2 + kk0) & m;
        const int sx = (i0 - 1 + gj + gk0) & 1;
        auto setup = [&](Col32& q, int d) {
            const int kk = kk0 + d;
            q.col = (unsigned)((gj << lg) | (gk0 + d));
            q.c = jj * LK + kk;
            q.fl = 1;
            if (jj >= 1 && jj <= LJ - 2 && kk >= 1 && kk <= LK - 2) q.fl |= 2;
            if (jj >= 2 && jj <= LJ - 3 && kk >= 2 && kk <= LK - 3) q.fl |= 4;
        };
        setup(X, sx);
        setup(Y, 1 - sx);
    }
    // element offsets fit in 32 bits (n <= 1024)
    auto offset = [&](int p, const Col32& q) -> unsigned { return ((unsigned)(p & m) << (2 * lg)) + q.col; };
    auto buf = [&](int p) { return (p - i0 + 3) % 3; };
    auto prologue = [&](Col32& q) {
        if (!q.fl) return;
        // planes i0-2, i0-1, i0 in slots 1, 2, 3; plane i0+1 raw in slot 1
        q.v[1] = make_v(ub[offset(i0 - 2, q)], ein[offset(i0 - 2, q)]);
        q.v[2] = make_v(ub[offset(i0 - 1, q)], ein[offset(i0 - 1, q)]);
        q.v[3] = make_v(ub[offset(i0, q)], ein[offset(i0, q)]);
        q.f[1] = f[offset(i0 - 2, q)];
        q.f[2] = f[offset(i0 - 1, q)];
        q.f[3] = f[offset(i0, q)];
        q.rub[1] = ub[offset(i0 + 1, q)];
        q.re[1] = ein[offset(i0 + 1, q)];
        q.rf[1] = f[offset(i0 + 1, q)];
        lv[buf(i0 - 1)][q.c] = q.v[2];
    };
    prologue(X);
    prologue(Y);
    __syncthreads();

    // One plane step, R = (p - i0 + 1) mod 4 fixed at compile time so that the register
    // planes rotate by renaming.  A holds the red cell of plane p and the black cell of
    // plane p-1.
    auto step = [&](auto Rc, int p, Col32& A, Col32& B) {
        constexpr int R = decltype(Rc)::value;
        constexpr int M2 = R, M1 = (R + 1) & 3, P0 = (R + 2) & 3, P1 = (R + 3) & 3;
        constexpr int N2 = (R + 1) & 1, N3 = R & 1;  // raw slots of planes p+2, p+3
        if (p + 3 <= last) {
            if (A.fl) {
                A.rub[N3] = ub[offset(p + 3, A)];
                A.re[N3] = ein[offset(p + 3, A)];
                A.rf[N3] = f[offset(p + 3, A)];
            }
            if (B.fl) {
                B.rub[N3] = ub[offset(p + 3, B)];
                B.re[N3] = ein[offset(p + 3, B)];
                B.rf[N3] = f[offset(p + 3, B)];
            }
        }
        V32* LA = lv[buf(p)];
        if (A.fl & 2) {
            const int c = A.c;
            const V32 nbv[6] = {A.v[M1], A.v[P1], LA[c - LK], LA[c + LK], LA[c - 1], LA[c + 1]};
            const Res32 r = dev32::corr_op(o, A.v[P0], nbv, A.f[P0]);
            A.v[P0] = dev32::remake_v(A.v[P0], A.v[P0].e + newton32(r, o.max_step));
            LA[c] = A.v[P0];
        }
        if (p - 1 >= i0) {
            if (A.fl & 4) {
                const V32* LB = lv[buf(p - 1)];
                const int c = A.c;
                const V32 nbv[6] = {A.v[M2], A.v[P0], LB[c - LK], LB[c + LK], LB[c - 1], LB[c + 1]};
                const Res32 r = dev32::corr_op(o, A.v[M1], nbv, A.f[M1]);
                A.v[M1].e = A.v[M1].e + newton32(r, o.max_step);
                eout[offset(p - 1, A)] = A.v[M1].e;
            }
            if (B.fl & 4) eout[offset(p - 1, B)] = B.v[M1].e;
        }
        V32* LC = lv[buf(p + 1)];
        const bool more2 = p + 2 <= last;
        auto advance = [&](Col32& q) {
            if (q.fl) {
                LC[q.c] = q.v[P1];
                if (more2) {  // plane p+2 takes the slot of plane p-2
                    q.v[M2] = make_v(q.rub[N2], q.re[N2]);
                    q.f[M2] = q.rf[N2];
                }
            }
        };
        advance(A);
        advance(B);
        __syncthreads();
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    // a.ti + 2 steps (a.ti a multiple of 4): two, then groups of four so that the register
    // planes and the column roles are back in place at the end of every iteration.  X holds
    // the red cells of planes i0-1, i0+1, ...
    step(I0{}, i0 - 1, X, Y);
    step(I1{}, i0, Y, X);
    for (int p = i0 + 1; p <= i0 + a.ti; p += 4) {
        step(I2{}, p, X, Y);
        step(I3{}, p + 1, Y, X);
        step(I0{}, p + 2, X, Y);
        step(I1{}, p + 3, Y, X);
    }
}

// ---- fused red-black sweep, one tile column pair per thread -------------------------------
// The tile sweep itself is in fused_fp32.h (shared with the batched solves).
template <int TJ, int TK>
__global__ void __launch_bounds__(TJ * TK / 2) k32_fused2(Grid g, const float* __restrict__ ub,
                                                         const float* __restrict__ ein, float* __restrict__ eout,
                                                         const float* __restrict__ f, FusedSweep32 a)
{
    if (g.halt && *g.halt) return;
    __shared__ V32 lv[3][(TJ + 4) * (TK + 4)];
    const int nb = gridDim.x;
    int lid = blockIdx.x;
    if ((nb & 7) == 0) lid = (lid & 7) * (nb >> 3) + (lid >> 3);
    const int tk = lid % a.ntk;
    lid /= a.ntk;
    const int tj = lid % a.ntj;
    const int ci = lid / a.ntj;
    fused32::sweep_tile<TJ, TK>(op32(g), g.n, g.lg, ci * a.ti, tj * TJ, tk * TK, a.ti, ub, ein, eout, f, lv);
}

// ---- streaming residual + restriction (n >= 64) ----------------------------------------
// Per plane the tile's cell values (ub, e, B, M) plus a one-cell in-plane halo sit in LDS and
// the i-neighbours in registers, so each cell's values are formed once.  8-child means of e and of
// d = N(e) - f into the coarse level: ec = ehat = R e, fc = R d.
// Thread t owns the columns of rows 2 (t / 64) and 2 (t / 64) + 1 of the tile at k = t mod 64 and the
// first threads a halo cell each; every lane evaluates the operator twice per plane, and a coarse
// cell's eight children are in two lanes, the other's fetched by a lane exchange.  Requests run two
// planes ahead and stand behind no branch (past the chunk's last plane they read that one
// again): where the compiler cannot count the loads in flight it waits for all of them.
// Measured at 512^3: 0.427 ms (4.2 TB/s); with the tile and its halo in three slots of a thread and the loads
// behind branches 0.508.
struct ColR32 {
    V32 vm, v0, vp;                        // planes p-1, p, p+1
    float ru[2], re[2], f[2], eq, dq;      // plane q of ub, e (raw) and f in [(q - i0) & 1]; the plane before
    unsigned col;                          // (j,k) offset within a plane
    int c;                                 // LDS cell
};

struct HaloR32 {
    V32 vp;
    float ru[2], re[2];
    unsigned col;
    int c;
};

// the value of the lane whose k differs in its last bit
__device__ __forceinline__ float k_pair(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xb1, 0xf, 0xf, true));  // [1,0,3,2]
}

// FAS: instead of the restriction fc = N(e) - fc in place, the right-hand side of a coarse level (f is
// not read): 256^3 64 us, 142 with one thread per cell.
template <int TJ, int NT, bool FAS = false>
__global__ void __launch_bounds__(NT) k32_resid_stream(Grid g, const float* __restrict__ ub, const float* __restrict__ e,
                                                       const float* __restrict__ f, float* __restrict__ ec,
                                                       float* __restrict__ ehat, float* __restrict__ fc, int ti,
                                                       int ntj, int ntk)
{
    if (g.halt && *g.halt) return;
    const Op32 o = op32(g);
    constexpr int LJ = TJ + 2, LK = kTK + 2, NL = LJ * LK, NH = 2 * LK + 2 * TJ;
    static_assert(NT == TJ * kTK / 2 && NH <= NT, "two columns and one halo cell per thread");
    __shared__ V32 lv[2][NL];
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
    const int t = threadIdx.x;
    const float* fsrc = FAS ? fc : f;

    // A plane's pointer is scalar and a column's byte offset fits in 32 bits (n <= 1024); both are
    // opaque, or the compiler keeps a 64-bit pointer per column and array and adds to it.
    auto at2 = [&](const float* a, int p, unsigned col) -> auto& {
        using gptr = __attribute__((address_space(1))) char*;
        gptr b = (gptr)(a + ((size_t)(p & m) << (2 * lg)));
        unsigned d = col * (unsigned)sizeof(float);
        asm("" : "+s"(b));
        asm("" : "+v"(d));
        return *(__attribute__((address_space(1))) float*)(b + d);
    };
    auto request = [&](auto& q, int N, int p) {
        q.ru[N] = at2(ub, p, q.col);
        q.re[N] = at2(e, p, q.col);
    };
    ColR32 X{}, Y{};
    HaloR32 E{};
    const bool halo = t < NH;
    {
        auto setup = [&](auto& q, int j, int k) {
            q.col = (unsigned)((((j0 - 1 + j) & m) << lg) | ((k0 - 1 + k) & m));
            q.c = j * LK + k;
        };
        const int jj = 1 + 2 * (t / kTK), kk = 1 + t % kTK, r = t - 2 * LK;
        setup(X, jj, kk);
        setup(Y, jj + 1, kk);
        if (t < LK) setup(E, 0, t);
        else if (t < 2 * LK) setup(E, LJ - 1, t - LK);
        else if (halo) setup(E, 1 + (r >> 1), (r & 1) * (LK - 1));
        else E.col = X.col;  // loads its own column again, in vain
    }
    auto prologue = [&](ColR32& q) {
        q.vm = make_v(at2(ub, i0 - 1, q.col), at2(e, i0 - 1, q.col));
        q.v0 = make_v(at2(ub, i0, q.col), at2(e, i0, q.col));
        q.vp = make_v(at2(ub, i0 + 1, q.col), at2(e, i0 + 1, q.col));
        request(q, 0, i0 + 2);
        q.f[0] = at2(fsrc, i0, q.col);
        q.f[1] = at2(fsrc, i0 + 1, q.col);
        lv[0][q.c] = q.v0;
    };
    prologue(X);
    prologue(Y);
    {
        const V32 v0 = make_v(at2(ub, i0, E.col), at2(e, i0, E.col));
        E.vp = make_v(at2(ub, i0 + 1, E.col), at2(e, i0 + 1, E.col));
        request(E, 0, i0 + 2);
        if (halo) lv[0][E.c] = v0;
    }
    __syncthreads();

    // One plane, N = (p - i0) & 1 fixed at compile time: the slots of the loads in flight rotate by
    // renaming (a copy would wait for them).
    auto step = [&](auto Nc, int p) {
        constexpr int N = decltype(Nc)::value, M = N ^ 1;
        const int p3 = p + 3 < last ? p + 3 : last;
        request(X, M, p3);
        request(Y, M, p3);
        request(E, M, p3);
        const V32* L = lv[N];
        auto residual = [&](const ColR32& q, const V32& jm, const V32& jp) -> float {
            const V32 nbv[6] = {q.vm, q.vp, jm, jp, L[q.c - 1], L[q.c + 1]};
            const float d = dev32::corr_op(o, q.v0, nbv, FAS ? 0.0f : q.f[N]).N;
            if constexpr (FAS) at2(fc, p, q.col) = d - q.f[N];
            return d;
        };
        const float dx = residual(X, L[X.c - LK], Y.v0);
        const float dy = residual(Y, X.v0, L[Y.c + LK]);
        const int pf = p + 2 < last ? p + 2 : last - 1;
        X.f[N] = at2(fsrc, pf, X.col);
        Y.f[N] = at2(fsrc, pf, Y.col);
        if constexpr (FAS) {
        } else if constexpr (N == 0) {
            X.eq = X.v0.e;
            X.dq = dx;
            Y.eq = Y.v0.e;
            Y.dq = dy;
        } else {
            const float ex = X.eq + X.v0.e, ey = Y.eq + Y.v0.e, rx = X.dq + dx, ry = Y.dq + dy;
            const float se = ex + k_pair(ex) + ey + k_pair(ey);
            const float sd = rx + k_pair(rx) + ry + k_pair(ry);
            if (!(t & 1)) {
                const long long qc = at(lg - 1, (p & m) >> 1, (j0 >> 1) + t / kTK, (k0 + t % kTK) >> 1);
                ec[qc] = 0.125f * se;
                ehat[qc] = 0.125f * se;
                fc[qc] = 0.125f * sd;
            }
        }
        // stage plane p+1 and shift the planes
        auto advance = [&](auto& q) {
            lv[M][q.c] = q.vp;
            if constexpr (std::is_same<decltype(q), ColR32&>::value) {
                q.vm = q.v0;
                q.v0 = q.vp;
            }
            q.vp = make_v(q.ru[N], q.re[N]);
        };
        advance(X);
        advance(Y);
        if (halo) advance(E);
        __syncthreads();
    };
    for (int p = i0; p < i0 + ti; p += 2) {
        step(std::integral_constant<int, 0>{}, p);
        step(std::integral_constant<int, 1>{}, p + 1);
    }
}

// ---- residual + restriction, FAS right-hand side, transfers ----------------------------
__global__ void __launch_bounds__(kBlock) k32_resid_restrict(Grid g, const float* __restrict__ ub,
                                                             const float* __restrict__ e,
                                                             const float* __restrict__ f,
                                                             float* __restrict__ ec, float* __restrict__ ehat,
                                                             float* __restrict__ fc)
{
    if (g.halt && *g.halt) return;
    const Op32 o = op32(g);
    const int lgc = g.lg - 1, nc = g.n >> 1;
    const long long tc = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (tc >= (1LL << (3 * lgc))) return;
    const int I = (int)(tc >> (2 * lgc)), J = (int)((tc >> lgc) & (nc - 1)), K = (int)(tc & (nc - 1));
    float se = 0.0f, sd = 0.0f;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int z = 0; z < 2; ++z) {
                const int i = 2 * I + x, j = 2 * J + y, k = 2 * K + z;
                const long long q = at(g.lg, i, j, k);
                long long qn[6];
                nbr_index(g.lg, i, j, k, qn);
                V32 nb[6];
#pragma unroll
                for (int v = 0; v < 6; ++v) nb[v] = make_v(ub[qn[v]], e[qn[v]]);
                const V32 c = make_v(ub[q], e[q]);
                se += c.e;
                sd += dev32::corr_op(o, c, nb, f[q]).N;
            }
    ec[tc] = 0.125f * se;
    ehat[tc] = 0.125f * se;
    fc[tc] = 0.125f * sd;
}

__global__ void __launch_bounds__(kBlock) k32_fas_rhs(Grid g, const float* __restrict__ ub,
                                                      const float* __restrict__ ehat, float* __restrict__ f)
{
    if (g.halt && *g.halt) return;
    const Op32 o = op32(g);
    const long long q = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (q >= (1LL << (3 * g.lg))) return;
    const int i = (int)(q >> (2 * g.lg)), j = (int)((q >> g.lg) & (g.n - 1)), k = (int)(q & (g.n - 1));
    long long qn[6];
    nbr_index(g.lg, i, j, k, qn);
    V32 nb[6];
#pragma unroll
    for (int v = 0; v < 6; ++v) nb[v] = make_v(ub[qn[v]], ehat[qn[v]]);
    f[q] = dev32::corr_op(o, make_v(ub[q], ehat[q]), nb, 0.0f).N - f[q];
}

__global__ void __launch_bounds__(kBlock) k32_restrict_mean(int lgc, const float* __restrict__ fine,
                                                            float* __restrict__ coarse)
{
    const long long tc = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (tc >= (1LL << (3 * lgc))) return;
    const int nc = 1 << lgc, lg = lgc + 1;
    const int I = (int)(tc >> (2 * lgc)), J = (int)((tc >> lgc) & (nc - 1)), K = (int)(tc & (nc - 1));
    float s = 0.0f;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int z = 0; z < 2; ++z) s += fine[at(lg, 2 * I + x, 2 * J + y, 2 * K + z)];
    coarse[tc] = 0.125f * s;
}

__global__ void __launch_bounds__(kBlock) k32_fill(float* __restrict__ x, float v, long long n)
{
    for (long long q = (long long)blockIdx.x * kBlock + threadIdx.x; q < n; q += (long long)gridDim.x * kBlock) x[q] = v;
}
inline unsigned blocks_for(long long work) { return (unsigned)((work + kBlock - 1) / kBlock); }

}  // namespace

hipError_t ngs_sweep32(const Grid& g, const float* ub, float* e, const float* f, hipStream_t s)
{
    const long long half = cells(g) / 2;
    for (int colour = 0; colour < 2; ++colour)
        hipLaunchKernelGGL(k32_ngs_colour, dim3(blocks_for(half)), dim3(kBlock), 0, s, g, ub, e, f, colour);
    return hipGetLastError();
}

hipError_t ngs_sweep32_fused(const Grid& g, const float* ub, const float* ein, float* eout, const float* f,
                             int ti, int tile, hipStream_t s)
{
    if (g.n < kTK || g.n > 1024 || ein == eout || ti < 4 || (ti & 3) || ti > g.n || (g.n % ti) != 0)
        return hipErrorInvalidValue;
    if (tile != kTile32Paired) {
        // one tile column pair per thread
        FusedSweep32 a{};
        a.ti = ti;
        auto launch = [&](auto kern, int TJ, int TK) {
            if (g.n % TJ || g.n % TK) return hipErrorInvalidValue;
            a.ntj = g.n / TJ;
            a.ntk = g.n / TK;
            const unsigned nb = (unsigned)((g.n / ti) * a.ntj * a.ntk);
            hipLaunchKernelGGL(kern, dim3(nb), dim3(TJ * TK / 2), 0, s, g, ub, ein, eout, f, a);
            return hipGetLastError();
        };
        if (tile == kTile32x32) return launch(k32_fused2<32, 32>, 32, 32);
        if (tile == kTile16x64) return launch(k32_fused2<16, 64>, 16, 64);
        if (tile == kTile32x64) return launch(k32_fused2<32, 64>, 32, 64);
        return launch(k32_fused2<16, 32>, 16, 32);
    }
    // 216 column pairs per 12 x 36 tile.  With 90 VGPRs a SIMD holds 5 wavefronts, so five
    // 4-wavefront workgroups share a CU: narrower tiles re-read more halo than 8 x 64 tiles
    // of 7 wavefronts, but the extra resident waves hide more of the per-plane barrier and
    // load latency (0.90 against 0.95 ms per 512^3 sweep).
    constexpr int TJ = 8, TK = 32, NT = 256;
    FusedSweep32 a{};
    a.ti = ti;
    a.ntj = g.n / TJ;
    a.ntk = g.n / TK;
    const unsigned nb = (unsigned)((g.n / ti) * a.ntj * a.ntk);
    hipLaunchKernelGGL((k32_fused<TJ, TK, NT>), dim3(nb), dim3(NT), 0, s, g, ub, ein, eout, f, a);
    return hipGetLastError();
}

template <bool FAS>
hipError_t stream32(const Grid& g, const float* ub, const float* e, const float* f, float* ec, float* ehat, float* fc,
                    hipStream_t s)
{
    constexpr int TJ = 8, NT = 256;
    const int ntj = g.n / TJ, ntk = g.n / kTK;
    int ti = 8;
    while (ti < g.n && (long long)ntj * ntk * (g.n / ti) > 8192) ti *= 2;
    const unsigned nb = (unsigned)((g.n / ti) * ntj * ntk);
    hipLaunchKernelGGL((k32_resid_stream<TJ, NT, FAS>), dim3(nb), dim3(NT), 0, s, g, ub, e, f, ec, ehat, fc, ti, ntj, ntk);
    return hipGetLastError();
}

hipError_t resid_restrict32(const Grid& g, const float* ub, const float* e, const float* f, float* ec,
                            float* ehat, float* fc, hipStream_t s)
{
    if (g.n >= kTK) return stream32<false>(g, ub, e, f, ec, ehat, fc, s);
    hipLaunchKernelGGL(k32_resid_restrict, dim3(blocks_for(cells(g) / 8)), dim3(kBlock), 0, s, g, ub, e, f, ec,
                       ehat, fc);
    return hipGetLastError();
}

hipError_t fas_rhs32(const Grid& gc, const float* ubc, const float* ehat, float* f, hipStream_t s)
{
    // one thread per cell forms seven cells' exponentials; streamed each cell's are formed once.  At
    // 64^3 the 64 workgroups of that are too few (a solve at 128^3 1.97 ms against 1.93).
    if (gc.n >= 2 * kTK) return stream32<true>(gc, ubc, ehat, nullptr, nullptr, nullptr, f, s);
    hipLaunchKernelGGL(k32_fas_rhs, dim3(blocks_for(cells(gc))), dim3(kBlock), 0, s, gc, ubc, ehat, f);
    return hipGetLastError();
}

hipError_t restrict_mean32(const Grid& gc, const float* fine, float* coarse, hipStream_t s)
{
    hipLaunchKernelGGL(k32_restrict_mean, dim3(blocks_for(cells(gc))), dim3(kBlock), 0, s, gc.lg, fine, coarse);
    return hipGetLastError();
}

hipError_t fill32(float* x, float v, long long n, hipStream_t s)
{
    long long b = (n + kBlock - 1) / kBlock;
    if (b > 4096) b = 4096;
    if (b < 1) b = 1;
    hipLaunchKernelGGL(k32_fill, dim3((unsigned)b), dim3(kBlock), 0, s, x, v, n);
    return hipGetLastError();
}

}  // namespace mgfr
