// The levels of side <= 16 of a domain solve's V-cycle, by one workgroup in one launch with
// every level in LDS (resident.h): the V-cycle from the level of side W down, in both precisions.
//
// One launch per phase takes 2 - 7 us each on these levels whatever their size: some 30 launches
// and the coarsest level's 15 - 27 us made a third of a 128^3 V-cycle.
#include "resident.h"

namespace mgfr {
namespace {

using res::cube;

template <int S>
__device__ __forceinline__ int element(int q)
{
    int i, j, k;
    res::cell_at<S>(q, i, j, k);
    return (i * S + j) * S + k;
}

// u of the level (side W, right-hand side from src as g says) after one V-cycle of its nl levels;
// the coarsest level's sweeps are added to *sweeps.
template <int W>
__global__ void __launch_bounds__(res::threads(W)) kd_tail64(Grid g, double* __restrict__ u,
                                                            const double* __restrict__ src, bool fas, int nl,
                                                            res::Cfg cfg, long long* __restrict__ sweeps)
{
    if (g.halt && *g.halt) return;
    constexpr int NT = res::threads(W);
    __shared__ res::Lds64<W, true> m;
    for (int q = threadIdx.x; q < cube(W); q += NT) {
        const int e = element<W>(q);
        const double v = u[e];
        m.top.v[q] = make_double2(v, dev::exp_(v));
        m.top.f[q] = dev::rhs_value(g, src[e]);
    }
    __syncthreads();
    const res::Op64 o{g.C, g.A, g.inv_np1, g.max_step};
    if (fas) {  // L(R u) - R d
        for (int q = threadIdx.x; q < cube(W); q += NT) {
            int i, j, k;
            res::cell_at<W>(q, i, j, k);
            m.top.f[q] = res::cell64<W, true>(o, m.top.v, nullptr, q, i, j, k, m.top.f[q]).L;
        }
        __syncthreads();
    }
    const int done = res::vcycle64<W, true, NT>(o, cfg, nl, m.top, m.below, m.red);
    for (int q = threadIdx.x; q < cube(W); q += NT) u[element<W>(q)] = m.top.v[q].x;
    if (threadIdx.x == 0) *sweeps += done;
}

// e of the level after one V-cycle of the correction equation; the bases of the levels below are
// formed from ub.
template <int W>
__global__ void __launch_bounds__(res::threads(W)) kd_tail32(Grid g, const float* __restrict__ ub, float* __restrict__ e,
                                                            const float* __restrict__ f, bool fas, int nl,
                                                            res::Cfg cfg)
{
    if (g.halt && *g.halt) return;
    constexpr int NT = res::threads(W);
    __shared__ res::Lds32<W, true> m;
    const dev32::Op32 o = dev32::op32(g);
    for (int q = threadIdx.x; q < cube(W); q += NT) {
        const int at = element<W>(q);
        const float b = ub[at];
        m.top.v[q] = res::make_v4(b, __expf(b), e[at]);
        m.top.f[q] = f[at];
        m.top.S_[q] = o.A * __expf(-b * o.inv_np1);
    }
    __syncthreads();
    if (fas) {  // N(R e) - R d
        for (int q = threadIdx.x; q < cube(W); q += NT) {
            int i, j, k;
            res::cell_at<W>(q, i, j, k);
            m.top.f[q] = res::cell32<W, true>(o, m.top.v, m.top.S_, nullptr, q, i, j, k, m.top.f[q]).N;
        }
        __syncthreads();
    }
    res::bases32<W, true, NT>(o, nl, m.top, m.below);
    res::vcycle32<W, true, NT>(o, cfg, nl, m.top, m.below, m.red);
    for (int q = threadIdx.x; q < cube(W); q += NT) e[element<W>(q)] = m.top.v[q].y;
}

}  // namespace

int domain_tail_n() { return 16; }

hipError_t domain_tail(const Grid& g, double* u, const double* src, bool fas, int nl, int pre, int post, int cap, double rtol,
                       long long* sweeps, hipStream_t s)
{
    const res::Cfg cfg{pre, post, cap, rtol};
    auto go = [&](auto kern, int nt) {
        hipLaunchKernelGGL(kern, dim3(1), dim3(nt), 0, s, g, u, src, fas, nl, cfg, sweeps);
        return hipGetLastError();
    };
    switch (g.n) {
    case 2: return go(kd_tail64<2>, res::threads(2));
    case 4: return go(kd_tail64<4>, res::threads(4));
    case 8: return go(kd_tail64<8>, res::threads(8));
    case 16: return go(kd_tail64<16>, res::threads(16));
    default: return hipErrorInvalidValue;
    }
}

hipError_t domain_tail32(const Grid& g, const float* ub, float* e, const float* f, bool fas, int nl, int pre, int post, int cap,
                         double rtol, hipStream_t s)
{
    const res::Cfg cfg{pre, post, cap, rtol};
    auto go = [&](auto kern, int nt) {
        hipLaunchKernelGGL(kern, dim3(1), dim3(nt), 0, s, g, ub, e, f, fas, nl, cfg);
        return hipGetLastError();
    };
    switch (g.n) {
    case 2: return go(kd_tail32<2>, res::threads(2));
    case 4: return go(kd_tail32<4>, res::threads(4));
    case 8: return go(kd_tail32<8>, res::threads(8));
    case 16: return go(kd_tail32<16>, res::threads(16));
    default: return hipErrorInvalidValue;
    }
}

}  // namespace mgfr
