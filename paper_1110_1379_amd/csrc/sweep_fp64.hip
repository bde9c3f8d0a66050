// Fused red-black Newton-Gauss-Seidel sweep, double precision, for levels with n >= 64.
//
// One sweep (red cells, then black cells, Sec. V.B.1) in one pass over HBM: each workgroup
// owns a TJ x TK tile of (j,k) columns and a chunk of planes i, and streams the planes in
// order.  Per plane it stages u and b = exp(u) of the tile plus an in-plane halo of two
// cells in LDS (three plane buffers, so one barrier per plane suffices).  At step p it updates
// the red cells of plane p (tile + 1-cell ring), then the black cells of plane p-1 (tile
// only), whose red neighbours are all final by then, and stages plane p+1:
//   red(p)   needs black(p-1), black(p+1), black in-plane            (all old)
//   black(p-1) needs red(p-2), red(p), red in-plane incl. the ring  (all new)
// The ring's red values are recomputed from the same old values by both tiles that see
// them, so they are bit-identical to the owner's, and the sweep equals the two-pass
// red-then-black sweep cell for cell.  The sweep reads `uin` and writes `uout` (never the
// same array) so that halo reads always see the values from before the sweep.
//
// A thread owns two k-adjacent columns.  At step p the column whose cell on plane p is red
// does both updates of the step (red on plane p, black on plane p-1, the same column); the
// other column has nothing to do until the next step.  The roles alternate, so every lane
// updates at every step.
#include "device_fp64.h"

#include <type_traits>

namespace mgfr {
namespace {

using dev::OpVal;

// One column of a thread's pair between steps p-1 and p: u and b = exp(u) of plane p+1, the red
// value it updated last (plane p-2 for the column with the red cell of plane p, p-1 for the
// other), the raw loads of planes p+2 and p+3 (plane q in slot (q - i0) & 1), and the raw
// right-hand sides of the red and the black cell of its next active step.  The planes p-1 and
// p are in LDS.
struct Col64 {
    double u1, b1, vr, br, ru[2], fr, fb;
    unsigned col;  // (j,k) offset within a plane
    int c;         // LDS cell
};

// An extra column of a thread: a cell of the red ring around the tile (updated on the planes
// where it is red) or of the halo around that (only staged).
struct Edge64 {
    double u1, b1, ru[2], fr;
    unsigned col;
    int c, cm, cp;   // LDS cells: its own and its k-neighbours' of the ring
    bool on, ring;
};

// Thread t < TJ TK / 2 owns the pair t of k-adjacent tile columns; the ring and the halo are
// extra columns of some of the threads, the ring cells of one parity side by side so that the
// wavefronts that update them are full.  A plane's values are (u, b) pairs, a row's even
// columns before its odd ones: the active columns of neighbouring lanes are then neighbours
// in LDS, and a neighbour is one 16-byte read.
// At 16 x 64: 512 threads, 65 KB of LDS and at most 128 VGPRs, so that two workgroups share a
// compute unit and one computes while the other waits at its barrier; with the pairs laid over
// the tile and its halo (704 threads) and four planes of (u, b, f) in registers it was one.
// Bound by its double-precision arithmetic (24 B of traffic per cell).  Measured at 512^3, 128
// planes: 0.794 ms per sweep (4.06 TB/s at 24 B per cell); with the loads behind branches and a 64-bit
// address each 0.835, in the layout before 1.045 ms; at 256^3 106, 111 and 153 us.
template <int TJ, int TK, int NT>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4)))
k_ngs_fused(Grid g, const double* __restrict__ uin, double* __restrict__ uout, const double* __restrict__ src,
            FusedSweep a)
{
    if (g.halt && *g.halt) return;
    constexpr int LJ = TJ + 4, LK = TK + 4, HK = LK / 2, NL = LJ * LK, NP = TJ * TK / 2;
    constexpr int NR = 2 * (TK + 2) + 2 * TJ;             // ring around the tile
    constexpr int NH = 2 * (TK + 4) + 2 * (TJ + 2);       // halo around the ring
    constexpr int NR2 = NR / 2, R1 = (NR2 + 63) / 64 * 64;  // ring cells of one parity; first thread of the second
    static_assert(NP == NT && R1 + NR2 <= NT && NR + NH <= NT, "one pair and one extra column per thread");
    // three plane buffers: plane p-1 (black update), plane p (red update), plane p+1 (staged)
    __shared__ double2 lv[3][NL];

    // workgroup -> (plane chunk, j tile, k tile); consecutive workgroups go to different
    // XCDs, so hand each XCD a contiguous range of tiles (their halos share its L2)
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

    // LDS cell of tile cell (jj, kk), 0 <= jj < LJ, 0 <= kk < LK
    auto cell = [&](int jj, int kk) { return jj * LK + (kk & 1) * HK + (kk >> 1); };
    // X is the column of the pair with the red cell on plane i0-1, Y the other
    Col64 X{}, Y{};
    int xm, xp, ym, yp;  // LDS cells of their k-neighbours
    {
        const int jj = 2 + t / (TK / 2), kk = 2 + 2 * (t - (jj - 2) * (TK / 2));
        const int gj = (j0 - 2 + jj) & m, gk = (k0 - 2 + kk) & m;
        const int sx = (i0 - 1 + gj + gk) & 1;
        X.col = (unsigned)((gj << lg) | (gk + sx));
        Y.col = (unsigned)((gj << lg) | (gk + 1 - sx));
        X.c = cell(jj, kk + sx);
        xm = cell(jj, kk + sx - 1);
        xp = cell(jj, kk + sx + 1);
        Y.c = cell(jj, kk + 1 - sx);
        ym = cell(jj, kk - sx);
        yp = cell(jj, kk + 2 - sx);
    }
    // E: the ring cells in the order of a walk around it, whose parity alternates: even ones
    // to threads 0 .., odd ones to threads R1 ..; the halo cells to the threads left over
    Edge64 E{};
    int epar = 0;  // parity of (j + k) of E's column
    {
        int w = -1;
        if (t < NR2) w = 2 * t;
        else if (t >= R1 && t < R1 + NR2) w = 2 * (t - R1) + 1;
        E.ring = w >= 0;
        if (!E.ring) w = t < R1 ? t - NR2 : t - 2 * NR2;
        E.on = E.ring || w < NH;
        // rectangle of ra x rb cells starting at (o, o)
        const int o = E.ring ? 1 : 0, ra = LJ - 2 * o, rb = LK - 2 * o;
        int ej, ek;
        if (w < rb) { ej = 0; ek = w; }
        else if (w < rb + ra - 1) { ej = w - rb + 1; ek = rb - 1; }
        else if (w < 2 * rb + ra - 2) { ej = ra - 1; ek = rb - 2 - (w - (rb + ra - 1)); }
        else { ej = ra - 2 - (w - (2 * rb + ra - 2)); ek = 0; }
        if (!E.on) { ej = 0; ek = 0; }
        ej += o;
        ek += o;
        const int gj = (j0 - 2 + ej) & m, gk = (k0 - 2 + ek) & m;
        E.col = (unsigned)((gj << lg) | gk);
        E.c = cell(ej, ek);
        E.cm = cell(ej, ek > 0 ? ek - 1 : 0);
        E.cp = cell(ej, ek < LK - 1 ? ek + 1 : LK - 1);
        epar = (gj + gk) & 1;
    }

    // A plane's pointer is scalar and a column's byte offset fits in 32 bits (n <= 1024); both are
    // opaque, or the compiler keeps a 64-bit pointer per column and array and adds to it.
    auto ref = [&](const double* f, int p, unsigned col) -> auto& {
        using gptr = __attribute__((address_space(1))) char*;
        gptr b = (gptr)(f + ((size_t)(p & m) << (2 * lg)));
        unsigned d = col * (unsigned)sizeof(double);
        asm("" : "+s"(b));
        asm("" : "+v"(d));
        return *(__attribute__((address_space(1))) double*)(b + d);
    };
    auto buf = [&](int p) { return (p - i0 + 3) % 3; };
    auto prologue = [&](auto& q) {
        // planes i0-2 and i0-1 to LDS, plane i0 in (u1, b1), plane i0+1 raw
        const double um2 = ref(uin, i0 - 2, q.col), um1 = ref(uin, i0 - 1, q.col);
        q.u1 = ref(uin, i0, q.col);
        q.ru[1] = ref(uin, i0 + 1, q.col);
        q.b1 = dev::exp_(q.u1);
        lv[buf(i0 - 2)][q.c] = make_double2(um2, dev::exp_(um2));
        lv[buf(i0 - 1)][q.c] = make_double2(um1, dev::exp_(um1));
    };
    X.fr = ref(src, i0 - 1, X.col);
    Y.fr = ref(src, i0, Y.col);
    prologue(X);
    prologue(Y);
    if (E.on) {
        // the right-hand side of the plane on which the cell is red first
        const double f0 = ref(src, i0 - 1, E.col), f1 = ref(src, i0, E.col);
        E.fr = ((i0 - 1 + epar) & 1) ? f1 : f0;
        prologue(E);
    }
    __syncthreads();

    const double ms = g.max_step;
    // One plane step.  N2 = (p - i0) & 1 is fixed at compile time (the raw slots rotate by
    // renaming).  A holds the red cell of plane p and the black cell of plane p-1, which the first
    // two steps do not have in the chunk (BLACK false).  The loads stand behind no branch, those
    // past the chunk's last plane read that one again: where the compiler cannot count the loads in
    // flight it waits for all of them.
    auto step = [&](auto N2c, auto Bc, int p, Col64& A, Col64& B, int am, int ap) {
        constexpr int N2 = decltype(N2c)::value, N3 = N2 ^ 1;  // raw slots of planes p+2, p+3
        constexpr bool BLACK = decltype(Bc)::value;
        double2* L0 = lv[buf(p)];
        const double2* Lm = lv[buf(p - 1)];
        double2* L1 = lv[buf(p + 1)];
        // the loads of plane p+3, two steps ahead of their use
        const int p3 = p + 3 < last ? p + 3 : last;
        A.ru[N3] = ref(uin, p3, A.col);
        B.ru[N3] = ref(uin, p3, B.col);
        E.ru[N3] = ref(uin, p3, E.col);
        const int pf = p + 2 < last ? p + 2 : last - 1;
        {
            const int c = A.c;
            // red cell of plane p; its black neighbours are all old
            const double2 m1 = Lm[c], p0 = L0[c];
            double v, bv;
            {
                const double2 jm = L0[c - LK], jp = L0[c + LK], km = L0[am], kp = L0[ap];
                const double un[6] = {m1.x, A.u1, jm.x, jp.x, km.x, kp.x};
                const double bn[6] = {m1.y, A.b1, jm.y, jp.y, km.y, kp.y};
                const OpVal r = dev::cell_op_b(g, p0.x, p0.y, un, bn, dev::rhs_value(g, A.fr));
                v = p0.x + dev::bounded(-r.L / r.dL, ms);
                bv = dev::exp_(v);
                L0[c] = make_double2(v, bv);
            }
            // black cell of plane p-1; its red neighbours are all new.  Plane p-1 is then final
            // in both columns.
            if constexpr (BLACK) {
                const double2 jm = Lm[c - LK], jp = Lm[c + LK], km = Lm[am], kp = Lm[ap];
                const double un[6] = {A.vr, v, jm.x, jp.x, km.x, kp.x};
                const double bn[6] = {A.br, bv, jm.y, jp.y, km.y, kp.y};
                const OpVal r = dev::cell_op_b(g, m1.x, m1.y, un, bn, dev::rhs_value(g, A.fb));
                ref(uout, p - 1, A.col) = m1.x + dev::bounded(-r.L / r.dL, ms);
                ref(uout, p - 1, B.col) = B.vr;
            }
            A.vr = v;
            A.br = bv;
            // A is active again at step p+2
            A.fr = ref(src, pf, A.col);
            A.fb = ref(src, p + 1, A.col);
        }
        if (E.ring && ((p + epar) & 1) == 0) {
            const int c = E.c;
            const double2 m1 = Lm[c], p0 = L0[c], jm = L0[c - LK], jp = L0[c + LK], km = L0[E.cm], kp = L0[E.cp];
            const double un[6] = {m1.x, E.u1, jm.x, jp.x, km.x, kp.x};
            const double bn[6] = {m1.y, E.b1, jm.y, jp.y, km.y, kp.y};
            const OpVal r = dev::cell_op_b(g, p0.x, p0.y, un, bn, dev::rhs_value(g, E.fr));
            const double v = p0.x + dev::bounded(-r.L / r.dL, ms);
            L0[c] = make_double2(v, dev::exp_(v));
            E.fr = ref(src, pf, E.col);
        }
        // stage plane p+1 for the next step; plane p+2 follows in the registers
        auto advance = [&](auto& q) {
            L1[q.c] = make_double2(q.u1, q.b1);
            q.u1 = q.ru[N2];
            q.b1 = dev::exp_(q.u1);
        };
        advance(A);
        advance(B);
        if (E.on) advance(E);
        __syncthreads();
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    // a.ti + 2 steps (a.ti even), two by two so that the column roles and the raw slots are
    // back in place at the end of every iteration
    step(I1{}, std::false_type{}, i0 - 1, X, Y, xm, xp);
    step(I0{}, std::false_type{}, i0, Y, X, ym, yp);
    for (int p = i0 + 1; p <= i0 + a.ti; p += 2) {
        step(I1{}, std::true_type{}, p, X, Y, xm, xp);
        step(I0{}, std::true_type{}, p + 1, Y, X, ym, yp);
    }
}

template <int TJ, int TK, int NT>
hipError_t launch(const Grid& g, const double* uin, double* uout, const double* src, FusedSweep a,
                  hipStream_t s)
{
    a.ntj = g.n / TJ;
    a.ntk = g.n / TK;
    const int nti = g.n / a.ti;
    const unsigned nb = (unsigned)(nti * a.ntj * a.ntk);
    hipLaunchKernelGGL((k_ngs_fused<TJ, TK, NT>), dim3(nb), dim3(NT), 0, s, g, uin, uout, src, a);
    return hipGetLastError();
}

}  // namespace

int fused_sweep_min_n() { return 64; }

int fused_sweep_planes(int n)
{
    // Planes per workgroup: long enough to amortise the 4 planes a chunk reads beyond its own,
    // short enough to fill the chip (two workgroups of 512 threads to each of 256 compute
    // units).  Measured, us per sweep: 128^3 with 4 / 8 / 16 planes 23.0 / 21.4 / 30.3, 256^3 with 16 /
    // 32 / 64 115 / 106 / 110, 512^3 with 64 / 128 / 256 / 512 801 / 792 / 801 / 827.
    return n <= 128 ? 8 : n == 256 ? 32 : 128;
}

hipError_t ngs_sweep_fused(const Grid& g, const double* uin, double* uout, const double* src, int ti, int tile,
                           hipStream_t s)
{
    if (g.n < 64 || g.n > 1024 || uin == uout || ti < 4 || (ti & 3) || ti > g.n || (g.n % ti) != 0)
        return hipErrorInvalidValue;
    FusedSweep a{};
    a.ti = ti;
    if (tile == kTile64x16x32) return launch<16, 32, 256>(g, uin, uout, src, a, s);
    return launch<16, 64, 512>(g, uin, uout, src, a, s);
}

}  // namespace mgfr
