// Two red-black sweeps of a small level in one launch, with what stands beside them in the
// V-cycle: before the coarse step the residual and its restriction, after it the coarse
// correction.  Every workgroup relaxes a block of B^3 cells: the block and a halo as wide as the
// values reach (one cell per colour sweep, one more for the residual) are loaded into LDS, the
// halo is relaxed again from the same old values by every block that sees it, and only the block
// is written, out of place.  The updates are those of the colour launches in the same order.
//
// At 32^3 a colour launch takes 3.5 us and the host four more between two of them, whatever
// they do: the eight launches and the two transfers of a V-cycle there are these two passes.
// Bound by the latency of its four colour sweeps.  Measured: 32^3 11 and 9.5 us in double precision, 10
// and 8 in single; 64^3 23 and 20, 23 and 17.  A double-precision solve at 32^3 takes 0.62 ms,
// 0.83 in launches; mixed at 64^3 0.90 and 1.25, at 128^3 1.94 and 2.24.
#include <type_traits>

#include "device_fp32.h"
#include "device_fp64.h"

namespace mgfr {
namespace {

// Double precision: a cell holds (u, exp u); f is the level's right-hand side.
struct B64 {
    using T = double;
    using V = double2;
    Grid g;
    __device__ V make(const T*, unsigned, T u) const { return make_double2(u, dev::exp_(u)); }
    __device__ static T value(const V& v) { return v.x; }
    __device__ T rhs(T src) const { return dev::rhs_value(g, src); }
    __device__ dev::OpVal op(const V& c, const V (&nb)[6], T f) const
    {
        const double un[6] = {nb[0].x, nb[1].x, nb[2].x, nb[3].x, nb[4].x, nb[5].x};
        const double bn[6] = {nb[0].y, nb[1].y, nb[2].y, nb[3].y, nb[4].y, nb[5].y};
        return dev::cell_op_b(g, c.x, c.y, un, bn, f);
    }
    __device__ V relax(const V& c, const V (&nb)[6], T f) const
    {
        const dev::OpVal r = op(c, nb, f);
        return make(nullptr, 0, c.x + dev::bounded(-r.L / r.dL, g.max_step));
    }
    __device__ T residual(const V& c, const V (&nb)[6], T f) const { return op(c, nb, f).L; }
};

// Single precision, the correction equation: a cell holds its base and (e, B, M).
struct B32 {
    using T = float;
    using V = dev32::V32;
    dev32::Op32 o;
    __device__ V make(const T* ub, unsigned q, T e) const { return dev32::make_v(ub[q], e); }
    __device__ static T value(const V& v) { return v.e; }
    __device__ T rhs(T f) const { return f; }
    __device__ V relax(const V& c, const V (&nb)[6], T f) const
    {
        return dev32::make_v(c.ub, c.e + dev32::newton32(dev32::corr_op(o, c, nb, f), o.max_step));
    }
    __device__ T residual(const V& c, const V (&nb)[6], T f) const { return dev32::corr_op(o, c, nb, f).N; }
};

__device__ __forceinline__ B64 policy(const Grid& g, double) { return B64{g}; }
__device__ __forceinline__ B32 policy(const Grid& g, float) { return B32{dev32::op32(g)}; }

// PRE: two sweeps of `in` into `out`, then uc = uhat = R out, fc = R (residual).  Otherwise in +
// P(uc - uhat), then two sweeps into `out`.  in and out are never the same array.
template <class P, int B, int NT, bool PRE>
__global__ void __launch_bounds__(NT) k_block(Grid g, const typename P::T* __restrict__ ub,
                                              const typename P::T* __restrict__ in, typename P::T* __restrict__ out,
                                              const typename P::T* __restrict__ src, typename P::T* __restrict__ uc,
                                              typename P::T* __restrict__ uhat, typename P::T* __restrict__ fc)
{
    if (g.halt && *g.halt) return;
    using T = typename P::T;
    using V = typename P::V;
    constexpr int H = PRE ? 5 : 4, R = B + 2 * H, NC = R * R * R;
    constexpr int RC = PRE ? 1 : R / 2 + 2;  // side of the coarse cells around the block and its halo
    __shared__ V v[NC];
    __shared__ T f[NC];
    __shared__ T ce[RC * RC * RC];
    const P pol = policy(g, T(0));
    const int lg = g.lg, m = g.n - 1, nb = g.n / B;
    const int b = blockIdx.x;
    const int k0 = (b % nb) * B - H, j0 = (b / nb % nb) * B - H, i0 = (b / (nb * nb)) * B - H;
    auto at = [&](int i, int j, int k) -> unsigned {
        return (((((unsigned)((i0 + i) & m)) << lg) + (unsigned)((j0 + j) & m)) << lg) + (unsigned)((k0 + k) & m);
    };
    if constexpr (!PRE) {
        // the correction of the coarse cells; i0, j0 and k0 are even
        const int mc = m >> 1, lgc = lg - 1;
        for (int c = threadIdx.x; c < RC * RC * RC; c += NT) {
            const int i = c / (RC * RC), j = c / RC % RC, k = c % RC;
            const unsigned q = (((((unsigned)(((i0 >> 1) - 1 + i) & mc)) << lgc) + (unsigned)(((j0 >> 1) - 1 + j) & mc))
                                << lgc) + (unsigned)(((k0 >> 1) - 1 + k) & mc);
            ce[c] = uc[q] - uhat[q];
        }
        __syncthreads();
    }
    for (int c = threadIdx.x; c < NC; c += NT) {
        const int i = c / (R * R), j = c / R % R, k = c % R;
        const unsigned q = at(i, j, k);
        T x = in[q];
        if constexpr (!PRE) {
            // 27/9/3/1 over 64: the bilinear part of the two nearest coarse planes, blended
            const int I = (i >> 1) + 1, J = (j >> 1) + 1, K = (k >> 1) + 1;
            const int I2 = I + ((i & 1) ? 1 : -1), J2 = J + ((j & 1) ? 1 : -1), K2 = K + ((k & 1) ? 1 : -1);
            auto plane = [&](int a) -> T {
                const T* e = ce + a * RC * RC;
                return T(9.0 / 16.0) * e[J * RC + K] + T(3.0 / 16.0) * (e[J2 * RC + K] + e[J * RC + K2]) +
                       T(1.0 / 16.0) * e[J2 * RC + K2];
            };
            x += T(0.75) * plane(I) + T(0.25) * plane(I2);
        }
        v[c] = pol.make(ub, q, x);
        f[c] = pol.rhs(src[q]);
    }
    __syncthreads();

    auto neighbours = [&](int c, V (&n)[6]) {
        n[0] = v[c - R * R];
        n[1] = v[c + R * R];
        n[2] = v[c - R];
        n[3] = v[c + R];
        n[4] = v[c - 1];
        n[5] = v[c + 1];
    };
    // one colour of the cells at least MG cells inside
    auto sweep = [&](auto Mc, int colour) {
        constexpr int MG = decltype(Mc)::value, W = R - 2 * MG, HW = W / 2;
        for (int t = threadIdx.x; t < W * W * HW; t += NT) {
            const int s = t % HW, j = t / HW % W, i = t / (HW * W);
            const int k = 2 * s + ((i + j + MG + H + colour) & 1);  // i0, j0 and k0 are H from an even cell
            const int c = ((MG + i) * R + MG + j) * R + MG + k;
            V n[6];
            neighbours(c, n);
            v[c] = pol.relax(v[c], n, f[c]);
        }
        __syncthreads();
    };
    sweep(std::integral_constant<int, 1>{}, 0);
    sweep(std::integral_constant<int, 2>{}, 1);
    sweep(std::integral_constant<int, 3>{}, 0);
    sweep(std::integral_constant<int, 4>{}, 1);

    for (int t = threadIdx.x; t < B * B * B; t += NT) {
        const int i = H + t / (B * B), j = H + t / B % B, k = H + t % B;
        const int c = (i * R + j) * R + k;
        out[at(i, j, k)] = P::value(v[c]);
        if constexpr (PRE) {
            V n[6];
            neighbours(c, n);
            f[c] = pol.residual(v[c], n, f[c]);
        }
    }
    if constexpr (PRE) {
        __syncthreads();
        constexpr int BC = B / 2;
        for (int t = threadIdx.x; t < BC * BC * BC; t += NT) {
            const int i = H + 2 * (t / (BC * BC)), j = H + 2 * (t / BC % BC), k = H + 2 * (t % BC);
            T su = T(0), sd = T(0);
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const int c = ((i + (x >> 2)) * R + j + ((x >> 1) & 1)) * R + k + (x & 1);
                su += P::value(v[c]);
                sd += f[c];
            }
            const unsigned q = (((((unsigned)((i0 + i) >> 1)) << (lg - 1)) + (unsigned)((j0 + j) >> 1)) << (lg - 1)) +
                               (unsigned)((k0 + k) >> 1);
            uc[q] = T(0.125) * su;
            uhat[q] = T(0.125) * su;
            fc[q] = T(0.125) * sd;
        }
    }
}

template <class P, bool PRE>
hipError_t pass(const Grid& g, const typename P::T* ub, const typename P::T* in, typename P::T* out,
                const typename P::T* src, typename P::T* uc, typename P::T* uhat, typename P::T* fc, hipStream_t s)
{
    if (!block_level(g.n) || in == out) return hipErrorInvalidValue;
    // 4^3 blocks fill the chip at 32^3 (512 of them; 8^3 blocks take as long); at 64^3 8^3 blocks do,
    // and relax a third as many halo cells (double precision 23 and 20 us, 4^3 blocks 66 and 44)
    if (g.n == 32)
        hipLaunchKernelGGL((k_block<P, 4, 512, PRE>), dim3(8 * 8 * 8), dim3(512), 0, s, g, ub, in, out, src, uc, uhat, fc);
    else
        hipLaunchKernelGGL((k_block<P, 8, 1024, PRE>), dim3(8 * 8 * 8), dim3(1024), 0, s, g, ub, in, out, src, uc, uhat,
                           fc);
    return hipGetLastError();
}

}  // namespace

// Levels that take the block passes: below 32 the V-cycle is one launch (tail.hip), from 128 up a
// sweep's launches are no longer what it costs and the halos are (with 8^3 blocks the first pass relaxes
// 4.7 cells for each of its own and the second 2.9).
bool block_level(int n) { return n == 32 || n == 64; }

hipError_t block_pre(const Grid& g, const double* in, double* out, const double* src, double* uc, double* uhat,
                     double* fc, hipStream_t s)
{
    return pass<B64, true>(g, nullptr, in, out, src, uc, uhat, fc, s);
}

hipError_t block_post(const Grid& g, const double* in, double* out, const double* src, const double* uc,
                      const double* uhat, hipStream_t s)
{
    return pass<B64, false>(g, nullptr, in, out, src, const_cast<double*>(uc), const_cast<double*>(uhat), nullptr, s);
}

hipError_t block_pre32(const Grid& g, const float* ub, const float* in, float* out, const float* f, float* ec,
                       float* ehat, float* fc, hipStream_t s)
{
    return pass<B32, true>(g, ub, in, out, f, ec, ehat, fc, s);
}

hipError_t block_post32(const Grid& g, const float* ub, const float* in, float* out, const float* f, const float* ec,
                        const float* ehat, hipStream_t s)
{
    return pass<B32, false>(g, ub, in, out, f, const_cast<float*>(ec), const_cast<float*>(ehat), nullptr, s);
}

}  // namespace mgfr
