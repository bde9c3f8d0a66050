// Streaming residual of a double-precision level, for n >= 64.
//
// d_i = L_i(u) - f_i (the operator of device_fp64.h).  Each workgroup owns a TJ x 64 tile of
// (j,k) columns and a chunk of planes; per plane it stages u and b = exp(u) of the tile plus
// a one-cell in-plane halo in LDS, and keeps the i-neighbours in registers, so every cell's
// exponential is evaluated once.  What is done with d is chosen at compile time:
//   NORM      per-workgroup partial sum of d^2 and max |d| (NaN-propagating)
//   RESTRICT  8-child means of u and d into the coarse level: uc = uhat = R u, fc = R d
//   UPDATE    u = uin + e (e single precision, the correction of the defect-correction
//             loop) for every loaded cell; the updated tile is written to uout
//   CAST      r = -d and ub = u rounded to single precision (right-hand side and base of
//             the next single-precision correction solve)
//   FAS       f = L(u) - f in place (fc), the right-hand side of a coarse level
#include <type_traits>

#include "device_fp64.h"

namespace mgfr {
namespace {

constexpr int kTK = 64;

// A column of a thread: u and exp(u) of planes p-1, p, p+1, the loads in flight, and of the plane
// before, for the restriction, u and d.
struct ColR {
    double um, u0, up, bm, b0, bp;
    double ru[2], f[2], uq, dq;  // plane q of u (raw) and f in [(q - i0) & 1]
    float re[2];                 // and of the correction
    unsigned col;                // (j,k) offset within a plane
    int c;                       // LDS cell
};

// A halo cell of a thread: only staged.
struct HaloR {
    double up, bp, ru[2];
    float re[2];
    unsigned col;
    int c;
};

// the value of the lane whose k differs in its last bit
__device__ __forceinline__ double k_pair(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0xb1, 0xf, 0xf, true);  // quad_perm [1,0,3,2]
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0xb1, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// Thread t owns the two columns of rows 2 (t / 64) and 2 (t / 64) + 1 of the tile at k = t mod 64, so
// that every lane evaluates the operator twice per plane, a wavefront's accesses are whole rows, and
// the eight children of a coarse cell are in two lanes, the other's fetched by a lane exchange; the
// halo is an extra column of the first threads.  Requests run two planes ahead and stand behind no
// branch (those past the chunk's last plane read that one again): where the compiler cannot count
// the loads in flight it waits for all of them.
// Bound by HBM.  Measured at 512^3: norm 0.418 ms (5.1 TB/s), restriction 0.525 ms (4.9 TB/s), norm and
// cast 0.730 ms, with the correction 1.002 ms (4.4 and 4.8 TB/s); with the tile and its halo in three
// slots of a thread, a third of whose lanes evaluated nothing, and the loads behind branches 0.655,
// 0.779, 0.908 and 1.129 ms.
template <int TJ, int NT, bool NORM, bool RESTRICT, bool UPDATE, bool CAST, bool FAS = false>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4)))
k_resid_stream(Grid g, const double* __restrict__ uin, const double* __restrict__ src, ResidStream a)
{
    if (g.halt && *g.halt) return;
    constexpr int LJ = TJ + 2, LK = kTK + 2, NL = LJ * LK, NH = 2 * LK + 2 * TJ;
    static_assert(NT == TJ * kTK / 2 && NH <= NT, "two columns and one halo cell per thread");
    __shared__ double2 lv[2][NL];  // (u, exp u)

    const int nb = gridDim.x;
    int lid = blockIdx.x;
    if ((nb & 7) == 0) lid = (lid & 7) * (nb >> 3) + (lid >> 3);
    const int tk = lid % a.ntk;
    lid /= a.ntk;
    const int tj = lid % a.ntj;
    const int ci = lid / a.ntj;
    const int i0 = ci * a.ti, j0 = tj * TJ, k0 = tk * kTK;
    const int lg = g.lg, m = g.n - 1;
    const int last = i0 + a.ti;  // last plane read
    const int t = threadIdx.x;
    const double* fsrc = FAS ? a.fc : src;

    // A plane's pointer is scalar and a column's byte offset fits in 32 bits (n <= 1024); both are
    // opaque, or the compiler keeps a 64-bit pointer per column and array and adds to it.
    auto ref = [&](auto* f, int p, unsigned col) -> auto& {
        using T = std::remove_const_t<std::remove_pointer_t<decltype(f)>>;
        using gptr = __attribute__((address_space(1))) char*;
        gptr b = (gptr)(f + ((size_t)(p & m) << (2 * lg)));
        unsigned d = col * (unsigned)sizeof(T);
        asm("" : "+s"(b));
        asm("" : "+v"(d));
        return *(__attribute__((address_space(1))) T*)(b + d);
    };
    auto load_u = [&](int p, unsigned col) -> double {
        double v = ref(uin, p, col);
        if constexpr (UPDATE) v += (double)ref(a.e32, p, col);
        return v;
    };
    // the correction of a prefetched plane is kept apart and added when the plane is used,
    // so that issuing the loads does not wait for them
    auto request = [&](auto& q, int N, int p) {
        q.ru[N] = ref(uin, p, q.col);
        if constexpr (UPDATE) q.re[N] = ref(a.e32, p, q.col);
    };

    ColR X{}, Y{};
    HaloR E{};
    const bool halo = t < NH;
    {
        const int jj = 1 + 2 * (t / kTK), kk = 1 + t % kTK;
        auto setup = [&](auto& q, int j, int k) {
            q.col = (unsigned)((((j0 - 1 + j) & m) << lg) | ((k0 - 1 + k) & m));
            q.c = j * LK + k;
        };
        setup(X, jj, kk);
        setup(Y, jj + 1, kk);
        const int r = t - 2 * LK;
        if (t < LK) setup(E, 0, t);
        else if (t < 2 * LK) setup(E, LJ - 1, t - LK);
        else if (halo) setup(E, 1 + (r >> 1), (r & 1) * (LK - 1));
        else E.col = X.col;  // loads its own column again, in vain
    }
    auto prologue = [&](ColR& q) {
        q.um = load_u(i0 - 1, q.col);
        q.u0 = load_u(i0, q.col);
        q.up = load_u(i0 + 1, q.col);
        request(q, 0, i0 + 2);
        q.f[0] = ref(fsrc, i0, q.col);
        q.f[1] = ref(fsrc, i0 + 1, q.col);
        q.bm = dev::exp_(q.um);
        q.b0 = dev::exp_(q.u0);
        q.bp = dev::exp_(q.up);
        lv[0][q.c] = make_double2(q.u0, q.b0);
    };
    prologue(X);
    prologue(Y);
    {
        const double u0 = load_u(i0, E.col);
        E.up = load_u(i0 + 1, E.col);
        request(E, 0, i0 + 2);
        E.bp = dev::exp_(E.up);
        if (halo) lv[0][E.c] = make_double2(u0, dev::exp_(u0));
    }
    __syncthreads();

    double acc = 0.0, mx = 0.0;
    // One plane, N = (p - i0) & 1 fixed at compile time: the slots of the loads in flight rotate by
    // renaming (a copy would wait for them).
    auto step = [&](auto Nc, int p) {
        constexpr int N = decltype(Nc)::value, M = N ^ 1;
        const int p3 = p + 3 < last ? p + 3 : last;
        request(X, M, p3);
        request(Y, M, p3);
        request(E, M, p3);
        const double2* L = lv[N];
        auto residual = [&](ColR& q, double2 jm, double2 jp) -> double {
            const double2 km = L[q.c - 1], kp = L[q.c + 1];
            const double un[6] = {q.um, q.up, jm.x, jp.x, km.x, kp.x};
            const double bn[6] = {q.bm, q.bp, jm.y, jp.y, km.y, kp.y};
            double d = dev::cell_op_b(g, q.u0, q.b0, un, bn, FAS ? 0.0 : dev::rhs_value(g, q.f[N])).L;
            asm volatile("" : "+v"(d));  // one column after the other: interleaved, they spill
            if constexpr (FAS) ref(a.fc, p, q.col) = d - q.f[N];
            if constexpr (NORM) {
                acc += d * d;
                const double ad = fabs(d);
                if (!(mx >= ad)) mx = ad;
            }
            if constexpr (UPDATE) ref(a.uout, p, q.col) = q.u0;
            if constexpr (CAST) {
                ref(a.r32, p, q.col) = (float)(-d);
                ref(a.ub32, p, q.col) = (float)q.u0;
            }
            return d;
        };
        const double dx = residual(X, L[X.c - LK], make_double2(Y.u0, Y.b0));
        const double dy = residual(Y, make_double2(X.u0, X.b0), L[Y.c + LK]);
        const int pf = p + 2 < last ? p + 2 : last - 1;
        X.f[N] = ref(fsrc, pf, X.col);
        Y.f[N] = ref(fsrc, pf, Y.col);
        if constexpr (RESTRICT) {
            if constexpr (N == 0) {
                X.uq = X.u0;
                X.dq = dx;
                Y.uq = Y.u0;
                Y.dq = dy;
            } else {
                const double ux = X.uq + X.u0, uy = Y.uq + Y.u0, ex = X.dq + dx, ey = Y.dq + dy;
                const double su = ux + k_pair(ux) + uy + k_pair(uy);
                const double sd = ex + k_pair(ex) + ey + k_pair(ey);
                if (!(t & 1)) {
                    const int lgc = lg - 1;
                    const long long qc = ((((long long)((p & m) >> 1) << lgc) + ((j0 >> 1) + t / kTK)) << lgc) +
                                         ((k0 + t % kTK) >> 1);
                    a.uc[qc] = 0.125 * su;
                    a.uhat[qc] = 0.125 * su;
                    a.fc[qc] = 0.125 * sd;
                }
            }
        }
        // stage plane p+1 and shift the planes
        auto advance = [&](auto& q) {
            lv[M][q.c] = make_double2(q.up, q.bp);
            if constexpr (std::is_same<decltype(q), ColR&>::value) {
                q.um = q.u0;
                q.bm = q.b0;
                q.u0 = q.up;
                q.b0 = q.bp;
            }
            q.up = UPDATE ? q.ru[N] + (double)q.re[N] : q.ru[N];
            q.bp = dev::exp_(q.up);
        };
        advance(X);
        advance(Y);
        if (halo) advance(E);
        __syncthreads();
    };
#pragma unroll 1
    for (int p = i0; p < i0 + a.ti; p += 2) {
        step(std::integral_constant<int, 0>{}, p);
        step(std::integral_constant<int, 1>{}, p + 1);
    }
    if (NORM) {
        double* red_s = (double*)&lv[0][0];
        double* red_m = red_s + NT;
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
            a.partial[2 * blockIdx.x] = red_s[0];
            a.partial[2 * blockIdx.x + 1] = red_m[0];
        }
    }
}

constexpr int kTJ = 8, kNT = 256;

template <bool NORM, bool RESTRICT, bool UPDATE, bool CAST>
hipError_t launch(const Grid& g, const double* uin, const double* src, ResidStream a, hipStream_t s)
{
    a.ntj = g.n / kTJ;
    a.ntk = g.n / kTK;
    const unsigned nb = (unsigned)((g.n / a.ti) * a.ntj * a.ntk);
    hipLaunchKernelGGL((k_resid_stream<kTJ, kNT, NORM, RESTRICT, UPDATE, CAST>), dim3(nb), dim3(kNT), 0, s, g,
                       uin, src, a);
    return hipGetLastError();
}

}  // namespace

int resid_stream_planes(int n)
{
    // even, dividing n, and few enough workgroups for the partial-sum scratch
    const long long tiles = (long long)(n / kTJ) * (n / kTK);
    int ti = 8;
    while (ti < n && tiles * (n / ti) > 8192) ti *= 2;
    return ti;
}

long long resid_stream_blocks(int n) { return (long long)(n / resid_stream_planes(n)) * (n / kTJ) * (n / kTK); }

hipError_t fas_stream(const Grid& g, const double* uhat, double* f, hipStream_t s)
{
    ResidStream a{};
    a.ti = resid_stream_planes(g.n);
    a.fc = f;
    a.ntj = g.n / kTJ;
    a.ntk = g.n / kTK;
    hipLaunchKernelGGL((k_resid_stream<kTJ, kNT, false, false, false, false, true>),
                       dim3((unsigned)resid_stream_blocks(g.n)), dim3(kNT), 0, s, g, uhat, (const double*)nullptr, a);
    return hipGetLastError();
}

hipError_t resid_stream(const Grid& g, const double* uin, const double* src, ResidStream a, hipStream_t s)
{
    if (g.n < kTK || g.n > 1024 || a.ti < 2 || (a.ti & 1) || g.n % a.ti) return hipErrorInvalidValue;
    const bool norm = a.partial != nullptr, restr = a.uc != nullptr, upd = a.e32 != nullptr,
               cast = a.r32 != nullptr;
    if (upd && (a.uout == nullptr || a.uout == uin)) return hipErrorInvalidValue;
    if (norm && !restr && !upd && !cast) return launch<true, false, false, false>(g, uin, src, a, s);
    if (!norm && restr && !upd && !cast) return launch<false, true, false, false>(g, uin, src, a, s);
    if (norm && !restr && upd && cast) return launch<true, false, true, true>(g, uin, src, a, s);
    if (norm && !restr && !upd && cast) return launch<true, false, false, true>(g, uin, src, a, s);
    return hipErrorInvalidValue;
}

}  // namespace mgfr
