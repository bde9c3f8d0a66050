// Coarse-grid correction u^h += P(u^H - R u^h) (Sec. V.B.3), double and single precision.
//
// P is the cell-centred trilinear interpolation with weights 27/9/3/1 over 64 (Sec. V.A.3),
// periodic.  It factors into an in-plane bilinear part (9/16, 3/16, 3/16, 1/16) on each
// coarse plane and a 3/4, 1/4 blend of the two coarse planes nearest the fine plane.  A
// thread owns the two fine columns (j, 2K) and (j, 2K+1), which read and write together and share
// two of their coarse columns, and a chunk of fine planes: it forms the in-plane interpolants once
// per coarse plane and reuses them for the two fine planes that need them.  The difference e =
// u^H - R u^h is formed on the fly from the two coarse arrays (FAS); the linear correction scheme
// passes the correction itself (no second array).
// Bound by HBM (u once each way).  Measured at 512^3: 0.577 ms (4.2 TB/s) in
// double precision with the difference formed, 0.412 ms without (5.5 TB/s), 0.257 ms in single; one fine
// column per thread, eight coarse reads for every two cells, 0.758, 0.490 and 0.285.
#include "mgfr_impl.h"

namespace mgfr {
namespace {

constexpr int kPT = 256;  // threads (pairs of fine columns) per workgroup

// Two neighbouring values, no further aligned than one (a caller's field may start anywhere): one
// access all the same, the hardware takes any multiple of four bytes.
template <typename T>
struct Pair {
    T x, y;
};

// DIFF: the correction is uc - uhat (else uc itself).  maskf (may be null): add only where
// the fine mask is positive (the active cells of a masked level).
template <typename T, int PI, bool DIFF>
__global__ void __launch_bounds__(kPT) k_prolong_stream(int lgc, T* __restrict__ uf, const T* __restrict__ uc,
                                                        const T* __restrict__ uhat, const float* __restrict__ maskf,
                                                        int ncolblk, const int* __restrict__ halt)
{
    if (halt && *halt) return;
    const int lg = lgc + 1, mc = (1 << lgc) - 1;
    const int nb = gridDim.x;
    int lid = blockIdx.x;
    if ((nb & 7) == 0) lid = (lid & 7) * (nb >> 3) + (lid >> 3);
    const int cb = lid % ncolblk, chunk = lid / ncolblk;
    const unsigned pair = (unsigned)cb * kPT + threadIdx.x;
    if (pair >= (1u << (2 * lg - 1))) return;
    const int j = (int)(pair >> lgc), K = (int)(pair & (unsigned)mc);
    const int J = j >> 1, Jn = (J + ((j & 1) ? 1 : -1)) & mc, Km = (K - 1) & mc, Kp = (K + 1) & mc;
    const unsigned row = (unsigned)J << lgc, rown = (unsigned)Jn << lgc;
    const int i0 = chunk * PI;

    // element offsets fit in 32 bits (n <= 1024)
    using P2 = Pair<T>;
    auto fine = [&](int i) -> unsigned { return ((unsigned)i << (2 * lg)) + 2 * pair; };
    P2 v[PI];
#pragma unroll
    for (int t = 0; t < PI; ++t) v[t] = *(const P2*)(uf + fine(i0 + t));

    // the in-plane interpolants of the two columns on coarse plane I
    auto inplane = [&](int I) -> P2 {
        const unsigned base = (unsigned)(I & mc) << (2 * lgc);
        auto E = [&](unsigned c) -> T { return DIFF ? uc[base + c] - uhat[base + c] : uc[base + c]; };
        const T c0 = E(row + K), c1 = E(rown + K);
        P2 e;
        e.x = T(9.0 / 16.0) * c0 + T(3.0 / 16.0) * (c1 + E(row + Km)) + T(1.0 / 16.0) * E(rown + Km);
        e.y = T(9.0 / 16.0) * c0 + T(3.0 / 16.0) * (c1 + E(row + Kp)) + T(1.0 / 16.0) * E(rown + Kp);
        return e;
    };
    auto add = [&](int t, const P2& near, const P2& far) {
        const unsigned q = fine(i0 + t);
        P2 r{v[t].x + (T(0.75) * near.x + T(0.25) * far.x), v[t].y + (T(0.75) * near.y + T(0.25) * far.y)};
        if (maskf) {
            const Pair<float> m = *(const Pair<float>*)(maskf + q);
            if (!(m.x > 0.0f) && !(m.y > 0.0f)) return;  // 512^3, 2% active 0.404 ms, 0.539 if stored
            if (!(m.x > 0.0f)) r.x = v[t].x;
            if (!(m.y > 0.0f)) r.y = v[t].y;
        }
        *(P2*)(uf + q) = r;
    };
    // fine planes 2I and 2I+1 lie nearest coarse plane I and next to I-1 and I+1
    P2 below = inplane((i0 >> 1) - 1), at = inplane(i0 >> 1);
#pragma unroll
    for (int t = 0; t < PI; t += 2) {
        const P2 above = inplane((i0 >> 1) + t / 2 + 1);
        add(t, at, below);
        add(t + 1, at, above);
        below = at;
        at = above;
    }
}

template <typename T, bool DIFF>
hipError_t launch(const Grid& gc, T* uf, const T* uc, const T* uhat, hipStream_t s, const float* maskf = nullptr)
{
    const int n = gc.n * 2;
    if (gc.n < 2 || n > 1024) return hipErrorInvalidValue;
    const int ncolblk = (n * n / 2 + kPT - 1) / kPT;
    // of two coarse arrays on the largest levels 16 planes per thread, which read fewer coarse planes
    // twice: 512^3 double 0.577 against 0.605 ms, single 0.257 against 0.278; of one array 0.417 against
    // 0.412
    if (DIFF && n >= 512) {
        const unsigned nb = (unsigned)(ncolblk * (n / 16));
        hipLaunchKernelGGL((k_prolong_stream<T, 16, DIFF>), dim3(nb), dim3(kPT), 0, s, gc.lg, uf, uc, uhat, maskf,
                           ncolblk, gc.halt);
    } else if (n >= 8) {
        const unsigned nb = (unsigned)(ncolblk * (n / 8));
        hipLaunchKernelGGL((k_prolong_stream<T, 8, DIFF>), dim3(nb), dim3(kPT), 0, s, gc.lg, uf, uc, uhat, maskf,
                           ncolblk, gc.halt);
    } else {
        hipLaunchKernelGGL((k_prolong_stream<T, 4, DIFF>), dim3((unsigned)ncolblk), dim3(kPT), 0, s, gc.lg, uf, uc, uhat,
                           maskf, ncolblk, gc.halt);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t prolong_correct(const Grid& gc, double* uf, const double* uc, const double* uhat, hipStream_t s)
{
    return launch<double, true>(gc, uf, uc, uhat, s);
}

hipError_t prolong_correct32(const Grid& gc, float* ef, const float* ec, const float* ehat, hipStream_t s)
{
    return launch<float, true>(gc, ef, ec, ehat, s);
}

hipError_t prolong_add_direct(const Grid& gc, double* uf, const double* ec, hipStream_t s)
{
    return launch<double, false>(gc, uf, ec, nullptr, s);
}

hipError_t prolong_add_masked(const Grid& gc, double* uf, const double* ec, const float* maskf, hipStream_t s)
{
    return launch<double, false>(gc, uf, ec, nullptr, s, maskf);
}

}  // namespace mgfr
