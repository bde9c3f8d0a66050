// The levels of side <= 16 of the Poisson V-cycle, one workgroup in one launch with every level in
// LDS: sweeps, restriction of the residual, the coarsest solve and the corrections, with the updates
// of the launches they replace (poisson_kernels.hip) in the same order.
//
// A launch on these levels takes 3.5 - 4.5 us and as long again until the next one, whatever it
// does, and a V-cycle had 34 of them.  Bound by latency: a colour sweep is one LDS round and a barrier.
// A Poisson solve of 16^3 takes 0.39 ms, 0.76 in launches, 32^3 0.69 and 0.92, 128^3 1.35 and 1.56, 512^3
// 26.9 and 27.2.
#include "mgfr_impl.h"

namespace mgfr {
namespace {

constexpr int kPT = 512;   // threads
constexpr int kTop = 16;   // side of the largest level
constexpr int kCells = kTop * kTop * kTop * 8 / 7 + 8;  // cells of all levels

struct Lin {
    double* x;
    double* b;
    int lg;
    double hh, inv_hh;
    __device__ int at(int i, int j, int k) const
    {
        const int m = (1 << lg) - 1;
        return ((((i & m) << lg) + (j & m)) << lg) + (k & m);
    }
    __device__ int cells() const { return 1 << (3 * lg); }
    __device__ void cell(int q, int& i, int& j, int& k) const
    {
        const int m = (1 << lg) - 1;
        i = q >> (2 * lg);
        j = (q >> lg) & m;
        k = q & m;
    }
    __device__ double nsum(int i, int j, int k) const
    {
        return x[at(i + 1, j, k)] + x[at(i - 1, j, k)] + x[at(i, j + 1, k)] + x[at(i, j - 1, k)] + x[at(i, j, k + 1)] +
               x[at(i, j, k - 1)];
    }
};

__device__ void sweep(const Lin& l)
{
    const int hk = 1 << (l.lg - 1), half = l.cells() / 2;
    for (int colour = 0; colour < 2; ++colour) {
        for (int t = threadIdx.x; t < half; t += kPT) {
            const int row = t >> (l.lg - 1), i = row >> l.lg, j = row & ((1 << l.lg) - 1);
            const int k = 2 * (t & (hk - 1)) + ((i + j + colour) & 1);
            const int q = l.at(i, j, k);
            l.x[q] = (l.nsum(i, j, k) - l.hh * l.b[q]) * (1.0 / 6.0);
        }
        __syncthreads();
    }
}

// z.b = R (residual of l), z.x = 0
__device__ void coarsen(const Lin& l, const Lin& z)
{
    for (int q = threadIdx.x; q < z.cells(); q += kPT) {
        int I, J, K;
        z.cell(q, I, J, K);
        double s = 0.0;
        for (int a = 0; a < 8; ++a) {
            const int i = 2 * I + (a >> 2), j = 2 * J + ((a >> 1) & 1), k = 2 * K + (a & 1), c = l.at(i, j, k);
            s += l.b[c] - (l.nsum(i, j, k) - 6.0 * l.x[c]) * l.inv_hh;
        }
        z.b[q] = 0.125 * s;
        z.x[q] = 0.0;
    }
    __syncthreads();
}

// l.x += P z.x (27/9/3/1 over 64)
__device__ void correct(const Lin& l, const Lin& z)
{
    for (int q = threadIdx.x; q < l.cells(); q += kPT) {
        int i, j, k;
        l.cell(q, i, j, k);
        const int I = i >> 1, J = j >> 1, K = k >> 1;
        const int In = I + ((i & 1) ? 1 : -1), Jn = J + ((j & 1) ? 1 : -1), Kn = K + ((k & 1) ? 1 : -1);
        auto plane = [&](int a) -> double {
            return (9.0 / 16.0) * z.x[z.at(a, J, K)] + (3.0 / 16.0) * (z.x[z.at(a, Jn, K)] + z.x[z.at(a, J, Kn)]) +
                   (1.0 / 16.0) * z.x[z.at(a, Jn, Kn)];
        };
        l.x[q] += 0.75 * plane(I) + 0.25 * plane(In);
    }
    __syncthreads();
}

__device__ __forceinline__ double wave_sum(double v)
{
    for (int w = 32; w > 0; w >>= 1) v += __shfl_xor(v, w);
    return v;
}

// Gauss-Seidel until rms(residual) <= rtol x initial, or down to its rounding floor, or cap sweeps
// (rtol = 0: exactly cap).  The constant null mode and the mean of x are irrelevant (the potential's
// mean is fixed last).  At most 64 cells: one wavefront, a cell per lane, neighbours by lane reads.
__device__ void coarsest(const Lin& l, int cap, double rtol, double* red)
{
    const int nc = l.cells();
    constexpr double eps = 2.220446049250313e-16;
    auto terms = [&](double ns, double x, double b, double& r2, double& f2) {
        const double r = b - (ns - 6.0 * x) * l.inv_hh;
        const double f = eps * ((fabs(ns) + 6.0 * fabs(x)) * l.inv_hh + fabs(b));
        r2 += r * r;
        f2 += f * f;
    };
    if (nc <= 64) {
        if (threadIdx.x < 64) {
            const int q = threadIdx.x < nc ? threadIdx.x : 0;
            const bool on = threadIdx.x < nc;
            int i, j, k;
            l.cell(q, i, j, k);
            const int n[6] = {l.at(i + 1, j, k), l.at(i - 1, j, k), l.at(i, j + 1, k),
                              l.at(i, j - 1, k), l.at(i, j, k + 1), l.at(i, j, k - 1)};
            double x = l.x[q];
            const double b = l.b[q];
            auto nsum = [&]() -> double {
                return __shfl(x, n[0]) + __shfl(x, n[1]) + __shfl(x, n[2]) + __shfl(x, n[3]) + __shfl(x, n[4]) +
                       __shfl(x, n[5]);
            };
            auto rms = [&](double& floor) -> double {
                double r2 = 0.0, f2 = 0.0;
                terms(nsum(), x, b, r2, f2);
                floor = sqrt(wave_sum(on ? f2 : 0.0) / nc);
                return sqrt(wave_sum(on ? r2 : 0.0) / nc);
            };
            double fl;
            const double r0 = rtol > 0.0 ? rms(fl) : 0.0;
            for (int s = 0; s < cap; ++s) {
                if (rtol > 0.0) {
                    const double r = rms(fl);
                    if (r <= rtol * r0 || r <= fl) break;
                }
                for (int colour = 0; colour < 2; ++colour) {
                    const double v = (nsum() - l.hh * b) * (1.0 / 6.0);
                    if (((i + j + k) & 1) == colour) x = v;
                }
            }
            if (on) l.x[q] = x;
        }
        __syncthreads();
        return;
    }
    auto rms = [&](double& floor) -> double {
        double r2 = 0.0, f2 = 0.0;
        for (int q = threadIdx.x; q < nc; q += kPT) {
            int i, j, k;
            l.cell(q, i, j, k);
            terms(l.nsum(i, j, k), l.x[q], l.b[q], r2, f2);
        }
        r2 = wave_sum(r2);
        f2 = wave_sum(f2);
        constexpr int NW = kPT / 64;
        if ((threadIdx.x & 63) == 0) {
            red[threadIdx.x >> 6] = r2;
            red[NW + (threadIdx.x >> 6)] = f2;
        }
        __syncthreads();
        double a = 0.0, c = 0.0;
        for (int w = 0; w < NW; ++w) {
            a += red[w];
            c += red[NW + w];
        }
        __syncthreads();
        floor = sqrt(c / nc);
        return sqrt(a / nc);
    };
    double fl;
    const double r0 = rtol > 0.0 ? rms(fl) : 0.0;
    for (int s = 0; s < cap; ++s) {
        if (rtol > 0.0) {
            const double r = rms(fl);
            if (r <= rtol * r0 || r <= fl) break;
        }
        sweep(l);
    }
}

// One V-cycle of the nl levels from g (side <= kTop) down; x from zero if `zero`.
__global__ void __launch_bounds__(kPT) kp_tail(PGrid g, double* __restrict__ x, const double* __restrict__ b, double bmean,
                                               bool zero, int nl, int pre, int post, int cap, double rtol)
{
    __shared__ double sx[kCells], sb[kCells];
    __shared__ double red[2 * kPT / 64];
    auto level = [&](int d) -> Lin {
        int at = 0;
        double s = 1.0;
        for (int k = 0; k < d; ++k) {
            at += 1 << (3 * (g.lg - k));
            s *= 4.0;
        }
        return Lin{sx + at, sb + at, g.lg - d, g.hh * s, g.inv_hh / s};
    };
    const Lin top = level(0);
    for (int q = threadIdx.x; q < top.cells(); q += kPT) {
        top.x[q] = zero ? 0.0 : x[q];
        top.b[q] = b[q] - bmean;
    }
    __syncthreads();
    for (int d = 0; d + 1 < nl; ++d) {
        const Lin l = level(d);
        for (int k = 0; k < pre; ++k) sweep(l);
        coarsen(l, level(d + 1));
    }
    coarsest(level(nl - 1), cap, rtol, red);
    for (int d = nl - 2; d >= 0; --d) {
        const Lin l = level(d);
        correct(l, level(d + 1));
        for (int k = 0; k < post; ++k) sweep(l);
    }
    for (int q = threadIdx.x; q < top.cells(); q += kPT) x[q] = top.x[q];
}

}  // namespace

int poisson_tail_n() { return kTop; }

hipError_t poisson_tail(const PGrid& g, double* x, const double* b, double bmean, bool zero, int nl, int pre, int post,
                        int cap, double rtol, hipStream_t s)
{
    if (g.n > kTop || nl < 1 || (g.n >> (nl - 1)) < 2 || (g.n >> (nl - 1)) > 8) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kp_tail, dim3(1), dim3(kPT), 0, s, g, x, b, bmean, zero, nl, pre, post, cap, rtol);
    return hipGetLastError();
}

}  // namespace mgfr
