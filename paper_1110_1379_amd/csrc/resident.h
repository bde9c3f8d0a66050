// V-cycles of a small grid (side <= 16) by one workgroup with every level in LDS, in both
// precisions, for the workgroup-per-unit kernels of the batched solves and for the lower
// levels of a domain solve.  PER: the grid is periodic; otherwise it is a cube patch with
// ghost faces (batch_dev.h).
//
// One compute unit does all the work of a level, so its vector instructions and its LDS reads
// bound it; what each choice saves is theirs:
//  - the level's side is a template parameter (cells and neighbours are found with constant
//    shifts), and the periodic form has no face tests;
//  - what a visit needs of a neighbour is one 16-byte LDS word: (u, b = exp(u)), or in single
//    precision (ub, e, b = exp(ub), M = b expm1(e)), whose last part is formed once per update
//    instead of at each of the six visits;
//  - a row's even columns lie before its odd ones, so the lanes of one colour read
//    neighbouring words;
//  - the residuals of a 4^3 block of fine cells are summed into its eight coarse cells within
//    one wavefront, without a barrier of the workgroup;
//  - the coarsest level of at most 64 cells is relaxed by one wavefront, which uses the
//    residuals of its stop test for the red update that follows it, and sums them with
//    cross-lane moves.
// Measured, with the separate arrays, run-time sides and restriction rounds of before in
// brackets: the V-cycle from one 16^3 level down 50 us in double precision (seven boxes; 115) and
// 52 us in single (ten patches; 125); the whole double-precision solves of 61 boxes of 16^3 0.74
// ms (2.36), the mixed ones of some 240 patches of 16^3 1.87 ms (5.8).
#pragma once

#include "batch_dev.h"

namespace mgfr {
namespace res {

using bdev::kR;
using bdev::kR32;
using bdev::wave_sync;
using dev::OpVal;
using dev32::em1f;
using dev32::newton32;
using dev32::Op32;
using dev32::Res32;

constexpr int cube(int s) { return s * s * s; }

// Workgroup of the resident kernels: at side 16 the levels fill a compute unit's LDS, so one
// workgroup runs on it and takes all the wavefronts its registers allow.
// (Two wavefronts at least: a single one's barriers are left out, and with them the separation
// of one unit's end from the next one's start in the persistent kernels.)
constexpr int threads(int W) { return W >= 16 ? 1024 : W == 8 ? 256 : 128; }

// threadIdx.x, not known to be the same from one call to the next: otherwise the cell and
// neighbour indices of every level and colour are formed once before a solve's loops and kept,
// in several times the registers there are.
__device__ __forceinline__ int thread_index()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Storage index of cell (i, j, k) of a level of side S.
template <int S>
__device__ __forceinline__ int place(int i, int j, int k)
{
    return (i * S + j) * S + (k & 1) * (S / 2) + (k >> 1);
}
// The cell at storage index q.
template <int S>
__device__ __forceinline__ void cell_at(int q, int& i, int& j, int& k)
{
    const int r = q & (S - 1);
    k = 2 * (r & (S / 2 - 1)) + (r / (S / 2));
    j = (q / S) & (S - 1);
    i = q / (S * S);
}
// Cell t of a colour (red: i + j + k even), t < S^3 / 2, and its storage index.
template <int S>
__device__ __forceinline__ int coloured(int t, int colour, int& i, int& j, int& k)
{
    const int kk = t & (S / 2 - 1), row = t / (S / 2);
    i = row / S;
    j = row & (S - 1);
    const int par = (i + j + colour) & 1;
    k = 2 * kk + par;
    return row * S + par * (S / 2) + kk;
}

// Storage indices of the six neighbours of the cell at q (periodic; on a patch the ones
// outside are meaningless but inside the level).
template <int S>
__device__ __forceinline__ void neighbours(int q, int i, int j, int k, int (&n)[6])
{
    constexpr int P = S * S, H = S / 2;
    n[0] = i == 0 ? q + (S - 1) * P : q - P;
    n[1] = i == S - 1 ? q - (S - 1) * P : q + P;
    n[2] = j == 0 ? q + (S - 1) * S : q - S;
    n[3] = j == S - 1 ? q - (S - 1) * S : q + S;
    const int row = q & ~(S - 1), kk = k >> 1;
    n[4] = (k & 1) ? row + kk : row + H + ((kk - 1) & (H - 1));
    n[5] = (k & 1) ? row + ((kk + 1) & (H - 1)) : row + H + kk;
}

// For a cell of a patch, the ghost face of an axis (at most one), or -1.
template <int S>
__device__ __forceinline__ int ghost_face(int axis, int c)
{
    return c == 0 ? 2 * axis : c == S - 1 ? 2 * axis + 1 : -1;
}

// v + the value w lanes above, within rows of 16 lanes.
template <int W>
__device__ __forceinline__ double add_above(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x100 + W, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x100 + W, 0xf, 0xf, true);
    return v + __hiloint2double(hi, lo);
}
template <int W>
__device__ __forceinline__ float add_above(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x100 + W, 0xf, 0xf, true));
}
__device__ __forceinline__ double lane0(double v)
{
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                            __builtin_amdgcn_readfirstlane(__double2loint(v)));
}
__device__ __forceinline__ float lane0(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
// Sum over the wavefront; every lane gets it.
template <class T>
__device__ __forceinline__ T wave_sum(T v)
{
    v = v + __shfl_down(v, 32);
    v = v + __shfl_down(v, 16);
    v = add_above<8>(v);
    v = add_above<4>(v);
    v = add_above<2>(v);
    v = add_above<1>(v);
    return lane0(v);
}
// Sum over a workgroup of NT threads (red: NT / 64 entries); every thread gets it.  red may be
// used again after the workgroup's next barrier.
template <int NT, class T>
__device__ __forceinline__ T group_sum(T v, T* red)
{
    v = wave_sum(v);
    if constexpr (NT > 64) {
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        v = red[0];
        for (int w = 1; w < NT / 64; ++w) v += red[w];
    }
    return v;
}

// What the multigrid cycle needs of the solver's settings.
struct Cfg {
    int pre, post, cap;
    double rtol;
};

// ---- double precision ---------------------------------------------------------------------
struct Op64 {
    double C, A, inv_np1, max_step;
};

// S = A exp(-u/(n+1)): for n = 1 through 1 / sqrt(b), as dev::curvature, but from u itself where b
// is denormal or zero (u < -708), whose root has lost what u still holds.  The wavefront branches,
// not the lane: 40 boxes of 32^3 2.50 ms against 2.53, 300 of 16^3 1.445 against 1.451 (without the
// test 1.440).
__device__ __forceinline__ double curvature(const Op64& o, double u, double b)
{
    if (o.inv_np1 == 0.5) {
        double y = __builtin_amdgcn_rsq(b);
        double e = fma(-b * y, y, 1.0);
        y = fma(0.5 * y, e, y);
        e = fma(-b * y, y, 1.0);
        y = fma(0.5 * y, e, y);
        const bool small = b < 2.2250738585072014e-308;
        if (__builtin_expect(__any(small), 0)) y = small ? dev::exp_(-0.5 * u) : y;
        return o.A * y;
    }
    return o.A * dev::exp_(-u * o.inv_np1);
}

// -L / dL, bounded.
__device__ __forceinline__ double newton64(const OpVal& r, double ms)
{
    double y = __builtin_amdgcn_rcp(r.dL);
    y = fma(fma(-r.dL, y, 1.0), y, y);
    y = fma(fma(-r.dL, y, 1.0), y, y);
    return dev::bounded(-r.L * y, ms);
}

// A level in LDS: (u, b), the right-hand side, and for levels below the top R u of the finer
// one; a patch's boundary values [6][S][S].
template <int S, bool PER>
struct Level64 {
    double2 v[cube(S)];
    double f[cube(S)];
    double uh[cube(S)];
    double fc[PER ? 1 : 6 * S * S];
};
template <int S, bool PER>
struct Top64 {
    double2 v[cube(S)];
    double f[cube(S)];
    double fc[PER ? 1 : 6 * S * S];
};
// The levels below side S.
template <int S, bool PER>
struct Below64 {
    Level64<S / 2, PER> lv;
    Below64<S / 2, PER> below;
};
template <bool PER>
struct Below64<2, PER> {};
template <int W, bool PER>
struct Lds64 {
    Top64<W, PER> top;
    Below64<W, PER> below;
    double red[threads(W)];   // residuals of the restriction blocks; sums
};

template <int S, bool PER>
__device__ __forceinline__ OpVal cell64(const Op64& o, const double2* v, const double* fc, int q, int i, int j, int k,
                                        double f)
{
    int n[6];
    neighbours<S>(q, i, j, k, n);
    const double2 c = v[q];
    const double S_ = curvature(o, c.x, c.y);
    OpVal r;
    if constexpr (PER) {
        const double2 n0 = v[n[0]];
        double su = n0.x - c.x, sb = n0.y, sbu = n0.y * su;
#pragma unroll
        for (int x = 1; x < 6; ++x) {
            const double2 nb = v[n[x]];
            const double du = nb.x - c.x;
            su += du;
            sb += nb.y;
            sbu = fma(nb.y, du, sbu);
        }
        r.L = o.C * fma(c.y, su, sbu) + S_ - f;
        r.dL = o.C * (fma(c.y, su, -sb) - 6.0 * c.y) - S_ * o.inv_np1;
    } else {
        double su = 0.0, sb = 0.0, sbu = 0.0, lg = 0.0, dlg = 0.0, nreg = 6.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int ca = a == 0 ? i : a == 1 ? j : k;
            const int face = ghost_face<S>(a, ca);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double2 nb = v[n[2 * a + h]];
                const bool in = face != 2 * a + h;
                const double du = in ? nb.x - c.x : 0.0, bn = in ? nb.y : 0.0;
                su += du;
                sb += bn;
                sbu = fma(bn, du, sbu);
            }
            if (face >= 0) {
                const int p0 = a == 0 ? j : i, p1 = a == 2 ? j : k;
                const double ug = (1.0 - kR) * fc[(face * S + p0) * S + p1] + kR * c.x;
                const double bg = dev::exp_(ug);
                lg += (bg + c.y) * (ug - c.x);
                dlg += (kR * bg + c.y) * (ug - c.x) + (bg + c.y) * (kR - 1.0);
                nreg -= 1.0;
            }
        }
        r.L = o.C * (fma(c.y, su, sbu) + lg) + S_ - f;
        r.dL = o.C * (fma(c.y, su, -sb) - nreg * c.y + dlg) - S_ * o.inv_np1;
    }
    return r;
}

template <int S, bool PER, int NT>
__device__ void sweep64(const Op64& o, double2* v, const double* f, const double* fc)
{
#pragma unroll
    for (int colour = 0; colour < 2; ++colour) {
        for (int t = thread_index(); t < cube(S) / 2; t += NT) {
            int i, j, k;
            const int q = coloured<S>(t, colour, i, j, k);
            const OpVal r = cell64<S, PER>(o, v, fc, q, i, j, k, f[q]);
            const double u = v[q].x + newton64(r, o.max_step);
            v[q] = make_double2(u, dev::exp_(u));
        }
        __syncthreads();
    }
}

// Into the level below: u = uh = R u with b = exp(u), and f = L^H(R u) - R d.  A wavefront takes
// a 4^3 block of fine cells (one per lane) and its eight coarse cells; their sums run in (i, j, k)
// order.
template <int S, bool PER, int NT, class LowerLevel>
__device__ void coarsen64(const Op64& o, const double2* v, const double* f, const double* fc, LowerLevel& z, double* red)
{
    constexpr int B = S / 4 > 0 ? S / 4 : 1;   // blocks per side
    constexpr int Q = S >= 4 ? 4 : S;          // cells of a block per side
    const int tid = thread_index(), lane = tid & 63, wave = tid >> 6;
    double* mine = red + 64 * wave;
    for (int b = wave; b < B * B * B; b += NT / 64) {
        const int bi = b / (B * B) * Q, bj = b / B % B * Q, bk = b % B * Q;
        if (lane < Q * Q * Q) {
            const int i = bi + lane / (Q * Q), j = bj + lane / Q % Q, k = bk + lane % Q;
            const int q = place<S>(i, j, k);
            mine[lane] = cell64<S, PER>(o, v, fc, q, i, j, k, f[q]).L;
        }
        wave_sync();
        // lanes 0 .. 7 sum the residuals, lanes 8 .. 15 the values of the coarse cells
        constexpr int C = Q / 2, NC = C * C * C;
        const int cc = lane & (NC - 1), part = lane / NC;
        if (part < 2) {
            const int x = cc / (C * C), y = cc / C % C, w = cc % C;
            double s = 0.0;
#pragma unroll
            for (int a = 0; a < 8; ++a) {
                const int fx = 2 * x + (a >> 2), fy = 2 * y + ((a >> 1) & 1), fw = 2 * w + (a & 1);
                s += part == 0 ? mine[(fx * Q + fy) * Q + fw] : v[place<S>(bi + fx, bj + fy, bk + fw)].x;
            }
            s *= 0.125;
            const int qc = place<S / 2>(bi / 2 + x, bj / 2 + y, bk / 2 + w);
            if (part == 0) {
                z.f[qc] = s;
            } else {
                z.v[qc] = make_double2(s, dev::exp_(s));
                z.uh[qc] = s;
            }
        }
        wave_sync();
    }
    __syncthreads();
    Op64 oc = o;
    oc.C = 0.25 * o.C;
    for (int q = thread_index(); q < cube(S / 2); q += NT) {
        int i, j, k;
        cell_at<S / 2>(q, i, j, k);
        z.f[q] = cell64<S / 2, PER>(oc, z.v, z.fc, q, i, j, k, 0.0).L - z.f[q];
    }
    __syncthreads();
}

// P(e) at fine cell (i, j, k): 27/9/3/1 over 64 of the coarse cells around it, of side SC; outside a
// patch a coarse cell contributes zero.
template <int SC, bool PER, class T>
__device__ __forceinline__ T interpolate(const T* e, int i, int j, int k)
{
    const int I = i >> 1, J = j >> 1, K = k >> 1;
    const int In = I + ((i & 1) ? 1 : -1), Jn = J + ((j & 1) ? 1 : -1), Kn = K + ((k & 1) ? 1 : -1);
    auto at = [&](int x, int y, int w) -> T {
        const T val = e[place<SC>(x & (SC - 1), y & (SC - 1), w & (SC - 1))];
        if constexpr (PER) return val;
        else return (x < 0 || x >= SC || y < 0 || y >= SC || w < 0 || w >= SC) ? T(0) : val;
    };
    return T(27.0 / 64.0) * at(I, J, K) + T(9.0 / 64.0) * (at(In, J, K) + at(I, Jn, K) + at(I, J, Kn)) +
           T(3.0 / 64.0) * (at(In, Jn, K) + at(In, J, Kn) + at(I, Jn, Kn)) + T(1.0 / 64.0) * at(In, Jn, Kn);
}

// u += P(u^H - R u), with its b.
template <int S, bool PER, int NT, class LowerLevel>
__device__ void correct64(double2* v, LowerLevel& z)
{
    for (int q = thread_index(); q < cube(S / 2); q += NT) z.uh[q] = z.v[q].x - z.uh[q];
    __syncthreads();
    for (int q = thread_index(); q < cube(S); q += NT) {
        int i, j, k;
        cell_at<S>(q, i, j, k);
        const double u = v[q].x + interpolate<S / 2, PER>(z.uh, i, j, k);
        v[q] = make_double2(u, dev::exp_(u));
    }
    __syncthreads();
}

// The coarsest level: sweeps until rms(L - f) <= rtol x initial, or its rounding floor (one unit
// in the last place of |dL||u| + |f| + S per cell), or cap sweeps (rtol = 0: exactly cap).  Returns
// the sweeps done (of the first wavefront's count where it works alone).
template <int S, bool PER, int NT>
__device__ int coarsest64(const Op64& o, const Cfg& cfg, double2* v, const double* f, const double* fc, double* red)
{
    constexpr int NC = cube(S);
    constexpr bool WAVE = NC <= 64;
    constexpr int T = WAVE ? 64 : NT, PT = (NC + T - 1) / T;
    int sweep = 0;
    if (!WAVE || threadIdx.x < 64) {
        int qs[PT], ii[PT], jj[PT], kk[PT];
        double fv[PT];
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            qs[p] = thread_index() + p * T;
            cell_at<S>(qs[p] & (NC - 1), ii[p], jj[p], kk[p]);
            fv[p] = qs[p] < NC ? f[qs[p]] : 0.0;
        }
        auto sync = [] {
            if constexpr (WAVE) wave_sync();
            else __syncthreads();
        };
        auto sum = [&](double a) -> double {
            if constexpr (WAVE) {
                return wave_sum(a);
            } else {
                const double s = group_sum<NT>(a, red);
                __syncthreads();
                return s;
            }
        };
        double r0 = 0.0;
        for (;; ++sweep) {
            OpVal r[PT];
            double s = 0.0, fl = 0.0;
#pragma unroll
            for (int p = 0; p < PT; ++p)
                if (qs[p] < NC) {
                    r[p] = cell64<S, PER>(o, v, fc, qs[p], ii[p], jj[p], kk[p], fv[p]);
                    s += r[p].L * r[p].L;
                    const double2 c = v[qs[p]];
                    const double f1 = 2.220446049250313e-16 *
                                      (fabs(r[p].dL) * fabs(c.x) + fabs(fv[p]) + curvature(o, c.x, c.y));
                    fl += f1 * f1;
                }
            if (cfg.rtol > 0.0) {
                // the norms' squares, compared as such
                const double ts = sum(s), tf = sum(fl);
                if (sweep == 0) r0 = cfg.rtol * cfg.rtol * ts;
                if (ts <= r0 || ts <= tf) break;
            }
            if (sweep >= cfg.cap) break;
            // red: the residuals just formed; black: from the new red values
#pragma unroll
            for (int p = 0; p < PT; ++p)
                if (qs[p] < NC && ((ii[p] + jj[p] + kk[p]) & 1) == 0) {
                    const double u = v[qs[p]].x + newton64(r[p], o.max_step);
                    v[qs[p]] = make_double2(u, dev::exp_(u));
                }
            sync();
#pragma unroll
            for (int p = 0; p < PT; ++p)
                if (qs[p] < NC && ((ii[p] + jj[p] + kk[p]) & 1) == 1) {
                    const OpVal rb = cell64<S, PER>(o, v, fc, qs[p], ii[p], jj[p], kk[p], fv[p]);
                    const double u = v[qs[p]].x + newton64(rb, o.max_step);
                    v[qs[p]] = make_double2(u, dev::exp_(u));
                }
            sync();
        }
    }
    __syncthreads();
    return sweep;
}

// One V-cycle of the nl levels from side S down; returns the sweeps of the coarsest level (in
// the first wavefront).
template <int S, bool PER, int NT, class L, class Below>
__device__ int vcycle64(const Op64& o, const Cfg& cfg, int nl, L& l, Below& below, double* red)
{
    if (nl == 1) {
        if constexpr (S <= 8) return coarsest64<S, PER, NT>(o, cfg, l.v, l.f, l.fc, red);
        return 0;
    }
    int done = 0;
    if constexpr (S > 2) {
        for (int s = 0; s < cfg.pre; ++s) sweep64<S, PER, NT>(o, l.v, l.f, l.fc);
        coarsen64<S, PER, NT>(o, l.v, l.f, l.fc, below.lv, red);
        Op64 oc = o;
        oc.C = 0.25 * o.C;
        done = vcycle64<S / 2, PER, NT>(oc, cfg, nl - 1, below.lv, below.below, red);
        correct64<S, PER, NT>(l.v, below.lv);
        for (int s = 0; s < cfg.post; ++s) sweep64<S, PER, NT>(o, l.v, l.f, l.fc);
    }
    return done;
}

template <int S, bool PER, int NT, class L>
__device__ double rms64(const Op64& o, const L& l, double* red)
{
    double s = 0.0;
    for (int q = thread_index(); q < cube(S); q += NT) {
        int i, j, k;
        cell_at<S>(q, i, j, k);
        const double d = cell64<S, PER>(o, l.v, l.fc, q, i, j, k, l.f[q]).L;
        s += d * d;
    }
    s = group_sum<NT>(s, red);
    __syncthreads();
    return sqrt(s / (double)cube(S));
}

// ---- single precision -----------------------------------------------------------------------
// (ub, e, b = exp(ub), M = b expm1(e)) in one word; S = A exp(-ub/(n+1)) fixed with the base.
template <int S, bool PER>
struct Level32 {
    float4 v[cube(S)];
    float f[cube(S)], S_[cube(S)], eh[cube(S)];
    float fc[PER ? 1 : 6 * S * S];
};
template <int S, bool PER>
struct Top32 {
    float4 v[cube(S)];
    float f[cube(S)], S_[cube(S)];
    float fc[PER ? 1 : 6 * S * S];
};
template <int S, bool PER>
struct Below32 {
    Level32<S / 2, PER> lv;
    Below32<S / 2, PER> below;
};
template <bool PER>
struct Below32<2, PER> {};
template <int W, bool PER>
struct Lds32 {
    Top32<W, PER> top;
    Below32<W, PER> below;
    float red[threads(W)];
    double sum[16];
};

__device__ __forceinline__ float4 make_v4(float ub, float b, float e)
{
    return make_float4(ub, e, b, b * em1f(e));
}

template <int S, bool PER>
__device__ __forceinline__ Res32 cell32(const Op32& o, const float4* v, const float* S_, const float* fc, int q, int i,
                                        int j, int k, float f)
{
    int n[6];
    neighbours<S>(q, i, j, k, n);
    const float4 c = v[q];
    const float cB = c.z + c.w, cM = c.w;
    float t1 = 0.0f, t2 = 0.0f, su = 0.0f, se = 0.0f, sB = 0.0f, nreg = 6.0f, lg = 0.0f, dlg = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int face = PER ? -1 : ghost_face<S>(a, a == 0 ? i : a == 1 ? j : k);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float4 nb = v[n[2 * a + h]];
            const bool in = PER || face != 2 * a + h;
            const float du = in ? nb.x - c.x : 0.0f, de = in ? nb.y - c.y : 0.0f;
            const float nM = nb.w, nB = in ? nb.z + nb.w : 0.0f;
            t1 = fmaf(nM, du, t1);
            t2 = fmaf(nB, de, t2);
            su += du;
            se += de;
            sB += nB;
        }
        if constexpr (!PER) {
            if (face >= 0) {
                const int p0 = a == 0 ? j : i, p1 = a == 2 ? j : k;
                const float ubg = (1.0f - kR32) * fc[(face * S + p0) * S + p1] + kR32 * c.x;
                const float eg = kR32 * c.y;
                const float bg = __expf(ubg);
                const float Mg = bg * em1f(eg), Bg = bg + Mg;
                const float du = ubg - c.x, de = eg - c.y;
                lg += (Mg + cM) * du + (Bg + cB) * de;
                dlg += (kR32 * Bg + cB) * (du + de) + (Bg + cB) * (kR32 - 1.0f);
                nreg -= 1.0f;
            }
        }
    }
    const float Sq = S_[q];
    const float x = em1f(-c.y * o.inv_np1);
    Res32 r;
    r.N = o.C * (fmaf(cM, su, t1) + fmaf(cB, se, t2) + lg) + Sq * x - f;
    r.dN = o.C * (cB * (su + se) - sB - nreg * cB + dlg) - Sq * o.inv_np1 * (1.0f + x);
    return r;
}

// e of the cell at q replaced.
__device__ __forceinline__ void put32(float4* v, int q, float e)
{
    const float b = v[q].z;
    v[q].y = e;
    v[q].w = b * em1f(e);
}

template <int S, bool PER, int NT>
__device__ void sweep32(const Op32& o, float4* v, const float* f, const float* S_, const float* fc)
{
#pragma unroll
    for (int colour = 0; colour < 2; ++colour) {
        for (int t = thread_index(); t < cube(S) / 2; t += NT) {
            int i, j, k;
            const int q = coloured<S>(t, colour, i, j, k);
            const Res32 r = cell32<S, PER>(o, v, S_, fc, q, i, j, k, f[q]);
            put32(v, q, v[q].y + newton32(r, o.max_step));
        }
        __syncthreads();
    }
}

// As coarsen64: e = eh = R e and f = N^H(R e) - R N on the level below, whose base is in place.
template <int S, bool PER, int NT, class LowerLevel>
__device__ void coarsen32(const Op32& o, const float4* v, const float* f, const float* S_, const float* fc, LowerLevel& z,
                          float* red)
{
    constexpr int B = S / 4 > 0 ? S / 4 : 1;
    constexpr int Q = S >= 4 ? 4 : S;
    const int tid = thread_index(), lane = tid & 63, wave = tid >> 6;
    float* mine = red + 64 * wave;
    for (int b = wave; b < B * B * B; b += NT / 64) {
        const int bi = b / (B * B) * Q, bj = b / B % B * Q, bk = b % B * Q;
        if (lane < Q * Q * Q) {
            const int i = bi + lane / (Q * Q), j = bj + lane / Q % Q, k = bk + lane % Q;
            const int q = place<S>(i, j, k);
            mine[lane] = cell32<S, PER>(o, v, S_, fc, q, i, j, k, f[q]).N;
        }
        wave_sync();
        constexpr int C = Q / 2, NC = C * C * C;
        const int cc = lane & (NC - 1), part = lane / NC;
        if (part < 2) {
            const int x = cc / (C * C), y = cc / C % C, w = cc % C;
            float s = 0.0f;
#pragma unroll
            for (int a = 0; a < 8; ++a) {
                const int fx = 2 * x + (a >> 2), fy = 2 * y + ((a >> 1) & 1), fw = 2 * w + (a & 1);
                s += part == 0 ? mine[(fx * Q + fy) * Q + fw] : v[place<S>(bi + fx, bj + fy, bk + fw)].y;
            }
            s *= 0.125f;
            const int qc = place<S / 2>(bi / 2 + x, bj / 2 + y, bk / 2 + w);
            if (part == 0) {
                z.f[qc] = s;
            } else {
                put32(z.v, qc, s);
                z.eh[qc] = s;
            }
        }
        wave_sync();
    }
    __syncthreads();
    Op32 oc = o;
    oc.C = 0.25f * o.C;
    for (int q = thread_index(); q < cube(S / 2); q += NT) {
        int i, j, k;
        cell_at<S / 2>(q, i, j, k);
        z.f[q] = cell32<S / 2, PER>(oc, z.v, z.S_, z.fc, q, i, j, k, 0.0f).N - z.f[q];
    }
    __syncthreads();
}

template <int S, bool PER, int NT, class LowerLevel>
__device__ void correct32(float4* v, LowerLevel& z)
{
    for (int q = thread_index(); q < cube(S / 2); q += NT) z.eh[q] = z.v[q].y - z.eh[q];
    __syncthreads();
    for (int q = thread_index(); q < cube(S); q += NT) {
        int i, j, k;
        cell_at<S>(q, i, j, k);
        put32(v, q, v[q].y + interpolate<S / 2, PER>(z.eh, i, j, k));
    }
    __syncthreads();
}

// As coarsest64; the floor is one single-precision unit in the last place of |dN||e| + |f|.
template <int S, bool PER, int NT>
__device__ int coarsest32(const Op32& o, const Cfg& cfg, float4* v, const float* f, const float* S_, const float* fc,
                          float* red)
{
    constexpr int NC = cube(S);
    constexpr bool WAVE = NC <= 64;
    constexpr int T = WAVE ? 64 : NT, PT = (NC + T - 1) / T;
    int sweep = 0;
    if (!WAVE || threadIdx.x < 64) {
        int qs[PT], ii[PT], jj[PT], kk[PT];
        float fv[PT];
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            qs[p] = thread_index() + p * T;
            cell_at<S>(qs[p] & (NC - 1), ii[p], jj[p], kk[p]);
            fv[p] = qs[p] < NC ? f[qs[p]] : 0.0f;
        }
        auto sync = [] {
            if constexpr (WAVE) wave_sync();
            else __syncthreads();
        };
        auto sum = [&](float a) -> float {
            if constexpr (WAVE) {
                return wave_sum(a);
            } else {
                const float s = group_sum<NT>(a, red);
                __syncthreads();
                return s;
            }
        };
        const float rtol = (float)cfg.rtol;
        float r0 = 0.0f;
        for (;; ++sweep) {
            Res32 r[PT];
            float s = 0.0f, fl = 0.0f;
#pragma unroll
            for (int p = 0; p < PT; ++p)
                if (qs[p] < NC) {
                    r[p] = cell32<S, PER>(o, v, S_, fc, qs[p], ii[p], jj[p], kk[p], fv[p]);
                    s += r[p].N * r[p].N;
                    const float f1 = 1.1920929e-7f * (fabsf(r[p].dN) * fabsf(v[qs[p]].y) + fabsf(fv[p]));
                    fl += f1 * f1;
                }
            if (rtol > 0.0f) {
                const float ts = sqrtf(sum(s)), tf = sqrtf(sum(fl));
                if (sweep == 0) r0 = rtol * ts;
                if (ts <= r0 || ts <= tf) break;
            }
            if (sweep >= cfg.cap) break;
#pragma unroll
            for (int p = 0; p < PT; ++p)
                if (qs[p] < NC && ((ii[p] + jj[p] + kk[p]) & 1) == 0)
                    put32(v, qs[p], v[qs[p]].y + newton32(r[p], o.max_step));
            sync();
#pragma unroll
            for (int p = 0; p < PT; ++p)
                if (qs[p] < NC && ((ii[p] + jj[p] + kk[p]) & 1) == 1) {
                    const Res32 rb = cell32<S, PER>(o, v, S_, fc, qs[p], ii[p], jj[p], kk[p], fv[p]);
                    put32(v, qs[p], v[qs[p]].y + newton32(rb, o.max_step));
                }
            sync();
        }
    }
    __syncthreads();
    return sweep;
}

template <int S, bool PER, int NT, class L, class Below>
__device__ int vcycle32(const Op32& o, const Cfg& cfg, int nl, L& l, Below& below, float* red)
{
    if (nl == 1) {
        if constexpr (S <= 8) return coarsest32<S, PER, NT>(o, cfg, l.v, l.f, l.S_, l.fc, red);
        return 0;
    }
    int done = 0;
    if constexpr (S > 2) {
        for (int s = 0; s < cfg.pre; ++s) sweep32<S, PER, NT>(o, l.v, l.f, l.S_, l.fc);
        coarsen32<S, PER, NT>(o, l.v, l.f, l.S_, l.fc, below.lv, red);
        Op32 oc = o;
        oc.C = 0.25f * o.C;
        done = vcycle32<S / 2, PER, NT>(oc, cfg, nl - 1, below.lv, below.below, red);
        correct32<S, PER, NT>(l.v, below.lv);
        for (int s = 0; s < cfg.post; ++s) sweep32<S, PER, NT>(o, l.v, l.f, l.S_, l.fc);
    }
    return done;
}

// Bases of the nl - 1 levels below side S: ub = R ub, b and S, from the level above (e and M are
// written by the restriction).
template <int S, bool PER, int NT, class L, class Below>
__device__ void bases32(const Op32& o, int nl, const L& l, Below& below)
{
    if constexpr (S > 2) {
        if (nl == 1) return;
        auto& z = below.lv;
        for (int q = thread_index(); q < cube(S / 2); q += NT) {
            int I, J, K;
            cell_at<S / 2>(q, I, J, K);
            float s = 0.0f;
#pragma unroll
            for (int a = 0; a < 8; ++a)
                s += l.v[place<S>(2 * I + (a >> 2), 2 * J + ((a >> 1) & 1), 2 * K + (a & 1))].x;
            const float ub = 0.125f * s;
            z.v[q] = make_float4(ub, 0.0f, __expf(ub), 0.0f);
            z.S_[q] = o.A * __expf(-ub * o.inv_np1);
        }
        __syncthreads();
        bases32<S / 2, PER, NT>(o, nl - 1, z, below.below);
    }
}

}  // namespace res
}  // namespace mgfr
