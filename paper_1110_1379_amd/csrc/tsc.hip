// Triangle-shaped-cloud (TSC) density assignment and force interpolation (Sec. VI.C),
// double precision, and their C entry points.
//
// Box units, periodic: cell i of the N^3 grid covers [i/N, (i+1)/N).  A particle at x has
// s = x N (modulo N), nearest cell floor(s) and offset d = s - floor(s) - 1/2; the cells
// floor(s) - 1, floor(s), floor(s) + 1 get the weights (1/2 - d)^2 / 2, 3/4 - d^2,
// (1/2 + d)^2 / 2 per axis, their product in 3-D.  Interpolation applies the same weights to
// the cell accelerations -grad phi, taken by central differences, so the pair conserves
// momentum.  Contraction into fused multiply-adds is switched off in the weight, product and
// sum arithmetic, so every operation rounds as written.
//
// Assignment is a gather, not a scatter: the particles are sorted by the key of their nearest
// cell (radix sort), a table gives each cell's range in that order, and every cell sums the
// contributions of the particles whose nearest cell is one of its 27 neighbours, through
// per-cell moments of each neighbour row (k_tsc_density), in a fixed order, so the density
// is the same bits on every call.  No atomics: in the clumps a scatter would put many lanes
// of a wavefront on the same few addresses.
//
// Interpolation reads the potential directly where consecutive particles lie near each other,
// and from tiles of it staged in LDS, the particles sorted by tile, where they are scattered
// (mgfr_tsc_force has the rule).
#include <algorithm>
#include <cstring>

#include <rocprim/rocprim.hpp>

#include "host_internal.h"

using namespace mgfr_host;

namespace mgfr {
namespace {

constexpr int kB = 256;

#pragma clang fp contract(off)

// Workgroup index remapped so that each of the 8 XCDs (which take workgroups round robin)
// runs one contiguous eighth of the grid: neighbouring cells and particles then share an L2.
__device__ __forceinline__ long long xcd_block()
{
    const unsigned nb = gridDim.x, b = blockIdx.x;
    if (nb & 7) return b;
    return (long long)(b & 7) * (nb >> 3) + (b >> 3);
}

// Nearest cell index and the three weights per axis of the particle at p[0..2].
__device__ __forceinline__ void tsc_weights(const double* __restrict__ p, int N, int (&c)[3], double (&w)[3][3])
{
    const double Nd = (double)N, inv = 1.0 / Nd;  // N is a power of two: s * inv is s / N exactly
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        double s = p[ax] * Nd;
        s = s - Nd * floor(s * inv);
        if (s >= Nd) s -= Nd;
        const double fl = floor(s);
        const double d = s - fl - 0.5;
        c[ax] = (int)fl & (N - 1);
        const double tl = 0.5 - d, tr = 0.5 + d;
        w[ax][0] = 0.5 * (tl * tl);
        w[ax][1] = 0.75 - d * d;
        w[ax][2] = 0.5 * (tr * tr);
    }
}

// Block partials of one pass over the particles: the number of non-finite coordinates and the
// number of particles that jump: that lie far (over kNear cells along i or j, 4 kNear along k) along
// two axes or all from the particle before them in their wavefront.  (A step along one axis alone
// is the order's own: few particles sorted by cell lie far apart in their rows, and share the
// cache lines of the rows beside.)  KEYS: also the key (flat index of the nearest
// cell) and identity index of every particle; a non-finite one gets some key of the grid.
// Reading the positions bounds it (3.2 GB at 512^3 particles): one pass where the check and
// the keys took one each (0.61 + 0.74 -> 0.88 ms).
constexpr int kNear = 4;

template <bool KEYS>
__global__ void __launch_bounds__(kB) k_tsc_scan(const double* __restrict__ pos, long long np, int N, int lg,
                                                 unsigned* __restrict__ key, unsigned* __restrict__ idx,
                                                 double* __restrict__ partial)
{
    __shared__ int bad[kB / 64], far[kB / 64];
    const int lane = threadIdx.x & 63, m = N - 1;
    int nbad = 0, nfar = 0;
    const long long rounds = (np + (long long)gridDim.x * kB - 1) / ((long long)gridDim.x * kB);
    for (long long r = 0; r < rounds; ++r) {
        const long long p = (r * gridDim.x + blockIdx.x) * kB + threadIdx.x;
        const bool live = p < np;
        int c[3] = {0, 0, 0};
        if (live) {
            const double Nd = (double)N, inv = 1.0 / Nd;  // N is a power of two: s * inv is s / N exactly
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const double x = pos[3 * p + ax];
                if (!isfinite(x)) ++nbad;
                double s = x * Nd;
                s = s - Nd * floor(s * inv);
                if (s >= Nd) s -= Nd;
                c[ax] = (int)floor(s) & m;
            }
            if (KEYS) {
                key[p] = ((unsigned)c[0] << (2 * lg)) | ((unsigned)c[1] << lg) | (unsigned)c[2];
                idx[p] = (unsigned)p;
            }
        }
        if (!KEYS) {
            // distance to the lane below, modulo N
            int away = 0;
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const int d = (c[ax] - __shfl_up(c[ax], 1)) & m, near = ax < 2 ? kNear : 4 * kNear;
                away += d > near && d < N - near;
            }
            if (live && lane > 0 && away >= 2) ++nfar;
        }
    }
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) {
        nbad += __shfl_xor(nbad, w);
        nfar += __shfl_xor(nfar, w);
    }
    if (lane == 0) {
        bad[threadIdx.x >> 6] = nbad;
        far[threadIdx.x >> 6] = nfar;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sb = 0.0, sf = 0.0;
        for (int w = 0; w < kB / 64; ++w) {
            sb += (double)bad[w];
            sf += (double)far[w];
        }
        partial[2 * blockIdx.x] = sf;
        partial[2 * blockIdx.x + 1] = sb;
    }
}

// Offsets d (x, y, z) of the particles from their nearest cell centre, in key order: the
// weights of a particle follow from d alone, and its nearest cell from its key.
__global__ void __launch_bounds__(kB) k_tsc_gather(const double* __restrict__ pos, const unsigned* __restrict__ idx,
                                                   long long np, int N, double* __restrict__ dsorted)
{
    const long long t = (long long)blockIdx.x * kB + threadIdx.x;
    if (t >= np) return;
    const long long p = idx[t];
    const double Nd = (double)N, inv = 1.0 / Nd;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        double s = pos[3 * p + ax] * Nd;
        s = s - Nd * floor(s * inv);
        if (s >= Nd) s -= Nd;
        dsorted[3 * t + ax] = s - floor(s) - 0.5;
    }
}

// The TSC weight of offset o in {0, 1, 2} (cells -1, 0, +1 from the nearest) at offset d.
__device__ __forceinline__ double tsc_w(double d, int o)
{
    if (o == 1) return 0.75 - d * d;
    const double t = o == 0 ? 0.5 - d : 0.5 + d;
    return 0.5 * (t * t);
}

// start[c] = first position in key order of a particle with key >= c, for c = 0 .. ncell
// (start[ncell] = np): the particles of cell c are start[c] .. start[c+1] - 1.
__global__ void __launch_bounds__(kB) k_tsc_cell_start(const unsigned* __restrict__ key, long long np,
                                                       long long ncell, unsigned* __restrict__ start)
{
    const long long t = (long long)blockIdx.x * kB + threadIdx.x;
    if (t >= np) return;
    const long long k = key[t];
    const long long prev = t > 0 ? (long long)key[t - 1] : -1;
    for (long long c = prev + 1; c <= k; ++c) start[c] = (unsigned)t;
    if (t == np - 1)
        for (long long c = k + 1; c <= ncell; ++c) start[c] = (unsigned)np;
}

__global__ void __launch_bounds__(kB) k_tsc_fill_start(unsigned* __restrict__ start, long long n)
{
    const long long t = (long long)blockIdx.x * kB + threadIdx.x;
    if (t < n) start[t] = 0u;
}

// Density of cell (i,j,k): the sum over the particles whose nearest cell is (i+a, j+b, k+c),
// a, b, c in {-1, 0, 1}, of mass x their weight for offset (-a, -b, -c).  A workgroup owns a
// segment of S = min(N, kB) cells of one row.  For each of the 9 neighbour rows (a, b) in
// turn:
//  - the particles of the source cells k0-1 .. k0+S of that row are taken kCH at a time, in
//    up to three key ranges: the wrapped cell N-1 (when k0 = 0), the cells
//    max(k0-1, 0) .. min(k0+S, N-1), the wrapped cell 0 (when k0 + S = N); every thread
//    evaluates mass x w_x(-a) x w_y(-b) x w_z(o) for the three z offsets o of its particles
//    of the chunk into LDS, so that the weights cost the same in every lane;
//  - one thread per source cell sums those terms over the cell's particles in key order
//    (three moments, kept in LDS);
//  - every cell adds the moments of its source cells k-1, k, k+1 for the offsets that reach
//    it.
// Each particle's weights are evaluated once per neighbour row rather than once per target
// cell, and the serial walk over a dense cell's particles is one lane's three additions per
// particle.  The order of
// every sum is fixed, so the density is the same bits on every call.
constexpr int kCH = 512;

__global__ void __launch_bounds__(kB) k_tsc_density(const double* __restrict__ dsorted,
                                                    const unsigned* __restrict__ start, int N, int lg, double mass,
                                                    double* __restrict__ rho)
{
    __shared__ double cw[3][kCH];                // per particle of the chunk: its three terms
    __shared__ double mom[3][kB + 2];            // moments of source cell k0-1+sc for z offsets 0, 1, 2
    const int m = N - 1;
    const int S = N < kB ? N : kB;               // cells per segment
    const int nseg = N / S;                      // segments per row
    const long long wg = xcd_block();
    const long long rowid = wg / nseg;           // (i, j)
    const int k0 = (int)(wg % nseg) * S;
    const int i = (int)(rowid >> lg), j = (int)(rowid & m);
    const int tid = threadIdx.x;
    const bool live = tid < S;
    double sum = 0.0;
    for (int ab = 0; ab < 9; ++ab) {
        const int a = ab / 3 - 1, b = ab % 3 - 1;
        const unsigned row = ((unsigned)((i + a) & m) << (2 * lg)) | ((unsigned)((j + b) & m) << lg);
        // the source cells of this thread (slots tid and tid + kB): particle range and the
        // key range (0, 1, 2 as above; -1 none) that holds it
        unsigned lo[2], hi[2];
        int rg[2];
        double mm[2][3];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int sc = tid + q * kB;
            lo[q] = hi[q] = 0;
            rg[q] = -1;
            if (sc < S + 2) {
                const unsigned key = row | (unsigned)((k0 - 1 + sc) & m);
                lo[q] = start[key];
                hi[q] = start[key + 1];
                rg[q] = (sc == 0 && k0 == 0) ? 0 : (sc == S + 1 && k0 + S == N) ? 2 : 1;
            }
            mm[q][0] = mm[q][1] = mm[q][2] = 0.0;
        }
        for (int sg = 0; sg < 3; ++sg) {
            unsigned g0, g1;
            if (sg == 0) {
                if (k0 != 0) continue;
                g0 = start[row + N - 1];
                g1 = start[row + N];
            } else if (sg == 1) {
                g0 = start[row + (k0 > 0 ? k0 - 1 : 0)];
                g1 = start[row + (k0 + S < N ? k0 + S + 1 : N)];
            } else {
                if (k0 + S != N) continue;
                g0 = start[row];
                g1 = start[row + 1];
            }
            for (unsigned c0 = g0; c0 < g1; c0 += kCH) {
                const unsigned c1 = c0 + kCH < g1 ? c0 + kCH : g1;
                __syncthreads();
                for (unsigned t = c0 + tid; t < c1; t += kB) {
                    const double* d = dsorted + 3 * (long long)t;
                    const double wxy = mass * tsc_w(d[0], 1 - a) * tsc_w(d[1], 1 - b);
                    const double dz = d[2];
                    cw[0][t - c0] = wxy * tsc_w(dz, 0);
                    cw[1][t - c0] = wxy * tsc_w(dz, 1);
                    cw[2][t - c0] = wxy * tsc_w(dz, 2);
                }
                __syncthreads();
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (rg[q] != sg) continue;
                    const unsigned t0 = lo[q] > c0 ? lo[q] : c0, t1 = hi[q] < c1 ? hi[q] : c1;
                    for (unsigned t = t0; t < t1; ++t) {
                        const unsigned l = t - c0;
                        mm[q][0] = mm[q][0] + cw[0][l];
                        mm[q][1] = mm[q][1] + cw[1][l];
                        mm[q][2] = mm[q][2] + cw[2][l];
                    }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int sc = tid + q * kB;
            if (sc < S + 2) {
                mom[0][sc] = mm[q][0];
                mom[1][sc] = mm[q][1];
                mom[2][sc] = mm[q][2];
            }
        }
        __syncthreads();
        // source cells k-1, k, k+1 are slots tid, tid+1, tid+2; they reach cell k with the
        // z weights of offsets +1, 0, -1 (o = 2, 1, 0)
        if (live) {
            sum = sum + mom[2][tid];
            sum = sum + mom[1][tid + 1];
            sum = sum + mom[0][tid + 2];
        }
        __syncthreads();  // the next row rewrites mom (it may stage nothing before that)
    }
    if (live) rho[((long long)rowid << lg) + k0 + tid] = sum;
}

// acc = sum over the 27 cells of weight x (-grad phi), -grad phi by central differences.
// phi_at(x, y, z): the potential at offsets x - 2, y - 2, z - 2 from the nearest cell.
template <class Phi>
__device__ __forceinline__ void tsc_force(const double (&w)[3][3], double half, Phi phi_at, double* __restrict__ acc)
{
    double fx = 0.0, fy = 0.0, fz = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
            for (int z = 0; z < 3; ++z) {
                // cell (c0 + a - 1, c1 + b - 1, c2 + z - 1) is index a+1, b+1, z+1 of the 5-wide ranges
                const double wt = w[0][a] * w[1][b] * w[2][z];
                const double gx = -(phi_at(a + 2, b + 1, z + 1) - phi_at(a, b + 1, z + 1)) * half;
                const double gy = -(phi_at(a + 1, b + 2, z + 1) - phi_at(a + 1, b, z + 1)) * half;
                const double gz = -(phi_at(a + 1, b + 1, z + 2) - phi_at(a + 1, b + 1, z)) * half;
                fx = fx + wt * gx;
                fy = fy + wt * gy;
                fz = fz + wt * gz;
            }
    acc[0] = fx;
    acc[1] = fy;
    acc[2] = fz;
}

// One thread per particle, the potential read through the caches.
__global__ void __launch_bounds__(kB) k_tsc_force(const double* __restrict__ phi, int N, int lg,
                                                  const double* __restrict__ pos, long long np,
                                                  double* __restrict__ acc)
{
    const long long p = xcd_block() * kB + threadIdx.x;
    if (p >= np) return;
    int c[3];
    double w[3][3];
    tsc_weights(pos + 3 * p, N, c, w);
    const int m = N - 1;
    const double half = (double)N / 2.0;
    // offsets of the planes c0-2 .. c0+2, rows c1-2 .. c1+2 and columns c2-2 .. c2+2
    unsigned pi[5], rj[5], ck[5];
#pragma unroll
    for (int t = 0; t < 5; ++t) {
        pi[t] = (unsigned)((c[0] + t - 2) & m) << (2 * lg);
        rj[t] = (unsigned)((c[1] + t - 2) & m) << lg;
        ck[t] = (unsigned)((c[2] + t - 2) & m);
    }
    tsc_force(
        w, half, [&](int x, int y, int z) { return phi[pi[x] + rj[y] + ck[z]]; }, acc + 3 * p);
}

// The same for scattered particles: they are taken in the order of their 16^3-cell tile (key,
// idx: the sorted tile keys and particle indices; start: each tile's first place in that
// order), kFP to a workgroup, and the potential of each tile met and of the two cells around it
// is staged in LDS once, so that a particle's 81 values cost LDS reads instead of some 25 cache
// lines of their own.  Each particle's sum is the direct kernel's, bit for bit, in any order.
// 62.5 KB of LDS: two workgroups of 8 wavefronts on a compute unit.  Bound by the LDS reads and
// the double-precision arithmetic; at 512^3 particles in lattice order with 30% moved into
// clumps it takes 6.2 ms, 9.8 with the check, its keys and sort, and the direct kernel 37.2 ms.
constexpr int kFT = 16, kFH = kFT + 4, kFB = 512, kFP = 4096;

__global__ void __launch_bounds__(kB) k_tsc_tile_keys(const double* __restrict__ pos, long long np, int N, int lg,
                                                      unsigned* __restrict__ key, unsigned* __restrict__ idx)
{
    const long long p = (long long)blockIdx.x * kB + threadIdx.x;
    if (p >= np) return;
    const double Nd = (double)N, inv = 1.0 / Nd;
    unsigned k = 0;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        double s = pos[3 * p + ax] * Nd;
        s = s - Nd * floor(s * inv);
        if (s >= Nd) s -= Nd;
        k = (k << (lg - 4)) | (unsigned)(((int)floor(s) & (N - 1)) >> 4);
    }
    key[p] = k;
    idx[p] = (unsigned)p;
}

__global__ void __launch_bounds__(kFB) k_tsc_force_tiles(const double* __restrict__ phi, int N, int lg,
                                                         const double* __restrict__ pos,
                                                         const unsigned* __restrict__ key,
                                                         const unsigned* __restrict__ idx,
                                                         const unsigned* __restrict__ start, long long np,
                                                         double* __restrict__ acc)
{
    __shared__ double tile[kFH * kFH * kFH];
    const int m = N - 1, nt = N / kFT, lt = lg - 4;
    const double half = (double)N / 2.0;
    long long t = xcd_block() * kFP;
    const long long t1 = t + kFP < np ? t + kFP : np;
    while (t < t1) {  // uniform over the workgroup
        const unsigned k = key[t];
        const long long e = start[k + 1] < t1 ? start[k + 1] : t1;
        // first cell of the staged block
        const int b0 = (int)(k >> (2 * lt)) * kFT - 2, b1 = (int)((k >> lt) & (nt - 1)) * kFT - 2,
                  b2 = (int)(k & (nt - 1)) * kFT - 2;
        __syncthreads();
        for (int q = threadIdx.x; q < kFH * kFH * kFH; q += kFB) {
            const int x = q / (kFH * kFH), y = q / kFH % kFH, z = q % kFH;
            tile[q] = phi[((((size_t)((b0 + x) & m) << lg) + ((b1 + y) & m)) << lg) + ((b2 + z) & m)];
        }
        __syncthreads();
        for (long long q = t + threadIdx.x; q < e; q += kFB) {
            const long long p = idx[q];
            int c[3];
            double w[3][3];
            tsc_weights(pos + 3 * p, N, c, w);
            const double* at = tile + ((c[0] - b0 - 2) * kFH + (c[1] - b1 - 2)) * kFH + (c[2] - b2 - 2);
            tsc_force(
                w, half, [&](int x, int y, int z) { return at[(x * kFH + y) * kFH + z]; }, acc + 3 * p);
        }
        t = e;
    }
}

#pragma clang fp contract(fast)

inline unsigned blocks(long long n) { return (unsigned)((n + kB - 1) / kB); }

int check_args(mgfr_ctx* c, const double* pos, long long np, int N)
{
    if (!is_pow2(N) || N < 4 || N > 1024) return c->fail(MGFR_EINVAL, "N=%d must be a power of two in [4, 1024]", N);
    if (np < 0 || np > (1LL << 36)) return c->fail(MGFR_EINVAL, "particle count %lld out of range", np);
    if (np > 0 && !pos) return c->fail(MGFR_EINVAL, "pos is NULL");
    return MGFR_OK;
}

// The pass over the positions (k_tsc_scan): non-finite ones would give arbitrary cells and are
// refused; *far gets the number of particles that jump, counted where no keys are asked for
// (synchronises).
int scan_positions(mgfr_ctx* c, const double* pos, long long np, int N, unsigned* key, unsigned* idx, double* far,
                   hipStream_t s)
{
    *far = 0.0;
    if (np == 0) return MGFR_OK;
    MGFR_TRY(ensure_scratch(c));
    const unsigned nb = (unsigned)std::min<long long>(blocks(np), 4096);
    if (key)
        hipLaunchKernelGGL(k_tsc_scan<true>, dim3(nb), dim3(kB), 0, s, pos, np, N, ilog2(N), key, idx, c->partial);
    else
        hipLaunchKernelGGL(k_tsc_scan<false>, dim3(nb), dim3(kB), 0, s, pos, np, N, ilog2(N), key, idx, c->partial);
    MGFR_TRY(hip_check(c, hipGetLastError(), "k_tsc_scan"));
    MGFR_TRY(hip_check(c, fold_sums(c->partial, (int)nb, c->red, s), "position check"));
    double r[2];
    MGFR_TRY(read_reduction(c, s, r));
    *far = r[0];
    if (r[1] != 0.0) return c->fail(MGFR_ENONFINITE, "%.0f non-finite particle coordinates", r[1]);
    return MGFR_OK;
}

inline size_t al(size_t b) { return (b + 255) & ~(size_t)255; }

// Grows the context's particle scratch to `need` bytes and orders the call's use of it on s
// after the last call's, which may have been queued on another stream; false if the device has
// not that much.
bool tsc_scratch(mgfr_ctx* c, size_t need, hipStream_t s)
{
    if (!c->tsc_ev && hipEventCreateWithFlags(&c->tsc_ev, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        c->tsc_ev = nullptr;
        return false;
    }
    if (c->tsc && hipStreamWaitEvent(s, c->tsc_ev, 0) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    if (c->tsc_bytes >= need) return true;
    (void)hipStreamSynchronize(s);
    (void)hipFree(c->tsc);
    c->tsc = nullptr;
    c->tsc_bytes = 0;
    if (hipMalloc(&c->tsc, need) != hipSuccess) {
        (void)hipGetLastError();
        c->tsc = nullptr;
        return false;
    }
    c->tsc_bytes = need;
    return true;
}

// The sort's buffers for np particles and a table of `cells` first places, carved from one
// block: keys and indices twice, the table, and rocPRIM's temporary storage.
struct SortBuffers {
    unsigned *key, *key2, *idx, *idx2, *start;
    void* tmp;
    size_t tmp_bytes, bytes;
};

hipError_t sort_buffers(long long np, long long cells, int bits, hipStream_t s, SortBuffers* b)
{
    b->tmp_bytes = 0;
    if (np > 0) {
        const hipError_t e = rocprim::radix_sort_pairs(nullptr, b->tmp_bytes, (unsigned*)nullptr, (unsigned*)nullptr,
                                                       (unsigned*)nullptr, (unsigned*)nullptr, (size_t)np, 0, bits, s);
        if (e != hipSuccess) return e;
    }
    b->bytes = 4 * al(sizeof(unsigned) * (size_t)np) + al(sizeof(unsigned) * (size_t)(cells + 1)) + al(b->tmp_bytes);
    return hipSuccess;
}

void place(SortBuffers* b, void* base, long long np, long long cells)
{
    const size_t ub = al(sizeof(unsigned) * (size_t)np);
    char* p = (char*)base;
    b->key = (unsigned*)p;
    b->key2 = (unsigned*)(p + ub);
    b->idx = (unsigned*)(p + 2 * ub);
    b->idx2 = (unsigned*)(p + 3 * ub);
    b->start = (unsigned*)(p + 4 * ub);
    b->tmp = p + 4 * ub + al(sizeof(unsigned) * (size_t)(cells + 1));
}

// key2, idx2 = the pairs sorted by key, and start from them.
int sort_and_table(mgfr_ctx* c, SortBuffers& b, long long np, long long cells, int bits, hipStream_t s)
{
    MGFR_TRY(hip_check(c, rocprim::radix_sort_pairs(b.tmp, b.tmp_bytes, b.key, b.key2, b.idx, b.idx2, (size_t)np, 0,
                                                    bits, s),
                       "radix_sort_pairs"));
    hipLaunchKernelGGL(k_tsc_cell_start, dim3(blocks(np)), dim3(kB), 0, s, b.key2, np, cells, b.start);
    return hip_check(c, hipGetLastError(), "k_tsc_cell_start");
}

}  // namespace
}  // namespace mgfr

extern "C" {

int mgfr_tsc_density(mgfr_ctx* c, const double* pos, long long np, int N, double mass, double* rho, void* stream)
{
    if (!c) return MGFR_EINVAL;
    c->err.clear();
    MGFR_TRY(mgfr::check_args(c, pos, np, N));
    if (np >= (1LL << 31)) return c->fail(MGFR_EINVAL, "assignment takes at most 2^31 - 1 particles (%lld)", np);
    if (!rho) return c->fail(MGFR_EINVAL, "rho is NULL");
    if (!std::isfinite(mass)) return c->fail(MGFR_EINVAL, "mass must be finite");
    MGFR_TRY(hip_check(c, hipSetDevice(c->device), "hipSetDevice"));
    hipStream_t s = (hipStream_t)stream;
    const int lg = ilog2(N);
    const long long ncell = (long long)N * N * N;
    mgfr::SortBuffers b;
    MGFR_TRY(hip_check(c, mgfr::sort_buffers(np, ncell, 3 * lg, s, &b), "radix_sort_pairs (size query)"));
    // the offsets in key order, then the sort's buffers: one block kept in the context
    const size_t ob = mgfr::al(sizeof(double) * 3 * (size_t)np);
    if (!mgfr::tsc_scratch(c, ob + b.bytes, s))
        return c->fail(MGFR_ENOMEM, "hipMalloc of %zu bytes failed", ob + b.bytes);
    double* sorted = (double*)c->tsc;
    mgfr::place(&b, (char*)c->tsc + ob, np, ncell);
    double far;
    MGFR_TRY(mgfr::scan_positions(c, pos, np, N, b.key, b.idx, &far, s));
    if (np > 0) {
        MGFR_TRY(mgfr::sort_and_table(c, b, np, ncell, 3 * lg, s));
        hipLaunchKernelGGL(mgfr::k_tsc_gather, dim3(mgfr::blocks(np)), dim3(mgfr::kB), 0, s, pos, b.idx2, np, N, sorted);
        MGFR_TRY(hip_check(c, hipGetLastError(), "k_tsc_gather"));
    } else {
        hipLaunchKernelGGL(mgfr::k_tsc_fill_start, dim3(mgfr::blocks(ncell + 1)), dim3(mgfr::kB), 0, s, b.start, ncell + 1);
        MGFR_TRY(hip_check(c, hipGetLastError(), "k_tsc_fill_start"));
    }
    const long long segs = (long long)N * N * (N < mgfr::kB ? 1 : N / mgfr::kB);
    hipLaunchKernelGGL(mgfr::k_tsc_density, dim3((unsigned)segs), dim3(mgfr::kB), 0, s, sorted, b.start, N, lg, mass, rho);
    MGFR_TRY(hip_check(c, hipGetLastError(), "k_tsc_density"));
    return hip_check(c, hipEventRecord(c->tsc_ev, s), "hipEventRecord");
}

int mgfr_tsc_force(mgfr_ctx* c, const double* phi, int N, const double* pos, long long np, double* acc, void* stream)
{
    if (!c) return MGFR_EINVAL;
    c->err.clear();
    MGFR_TRY(mgfr::check_args(c, pos, np, N));
    if (!phi || (np > 0 && !acc)) return c->fail(MGFR_EINVAL, "phi or acc is NULL");
    MGFR_TRY(hip_check(c, hipSetDevice(c->device), "hipSetDevice"));
    hipStream_t s = (hipStream_t)stream;
    double far;
    MGFR_TRY(mgfr::scan_positions(c, pos, np, N, nullptr, nullptr, &far, s));
    const int lg = ilog2(N);
    const long long ntile = (long long)(N / mgfr::kFT) * (N / mgfr::kFT) * (N / mgfr::kFT);
    // Scattered particles go through the tiles.  A jump costs the direct kernel 0.25 (128^3) to 1.1
    // ns (512^3, no order at all) for cache lines of its own; the tiles cost the sort, 0.13 ms up to
    // 2^20 particles and a fraction of that from there on, where it takes its faster form, and the
    // staging, 7.5 ps for every cell of the grid however few particles it holds, and save 0.17 ns a
    // particle besides.  So, direct and tile times in ms for one side and the other of each line:
    //  - 375 thousand jumps: lattice order with clumps, 1.05 M particles, 64^3 with 169 thousand jumps
    //    0.128, 0.144 and with 452 thousand 0.190, 0.146; 256^3 with 194 thousand 0.279, 0.313 and
    //    with 522 thousand 0.391, 0.342; and 1% of the particles (in cell order 134 M at 512^3 take
    //    6.45, 7.24, with 1% jumps among them 10.0, 7.52);
    //  - a jump for every 50 cells, less 0.4 for every particle: 512^3 with 4 M particles and 0.75 M jumps
    //    1.11, 1.19, with 1.41 M 1.45, 1.28; 1.05 M without order 1.17, 1.61, 2 M 2.17, 1.11; 1024^3 with
    //    30 M and 5.6 M jumps 7.37, 8.41, with 15 M 12.8, 8.90;
    //  - below 2^20 particles nine tenths of them and 128 particles to a tile, and none at 64^3: 256^3
    //    with 800 thousand in lattice order with clumps, 82% jumps 0.40, 0.59, without order 0.87,
    //    0.41, with 600 thousand 0.67, 0.45, with 400 thousand 0.46, 0.55; 64^3 without order 0.28, 0.24,
    //    with assignment before it 400 thousand 0.41, 0.46.
    bool tiles = N >= 64 && np < (1LL << 31) && far >= 375000.0 && far > 0.01 * (double)np &&
                 far >= 0.02 * (double)N * N * N - 0.4 * (double)np &&
                 (np >= (1LL << 20) || (N > 64 && far >= 0.9 * (double)np && np >= 128 * ntile));
    mgfr::SortBuffers b;
    if (tiles) {
        MGFR_TRY(hip_check(c, mgfr::sort_buffers(np, ntile, 3 * (lg - 4), s, &b), "radix_sort_pairs (size query)"));
        // the direct kernel needs no scratch: it takes over where there is none
        tiles = mgfr::tsc_scratch(c, b.bytes, s);
    }
    if (tiles) {
        mgfr::place(&b, c->tsc, np, ntile);
        hipLaunchKernelGGL(mgfr::k_tsc_tile_keys, dim3(mgfr::blocks(np)), dim3(mgfr::kB), 0, s, pos, np, N, lg, b.key,
                           b.idx);
        MGFR_TRY(hip_check(c, hipGetLastError(), "k_tsc_tile_keys"));
        MGFR_TRY(mgfr::sort_and_table(c, b, np, ntile, 3 * (lg - 4), s));
        hipLaunchKernelGGL(mgfr::k_tsc_force_tiles, dim3((unsigned)((np + mgfr::kFP - 1) / mgfr::kFP)), dim3(mgfr::kFB), 0,
                           s, phi, N, lg, pos, b.key2, b.idx2, b.start, np, acc);
        MGFR_TRY(hip_check(c, hipGetLastError(), "k_tsc_force_tiles"));
        MGFR_TRY(hip_check(c, hipEventRecord(c->tsc_ev, s), "hipEventRecord"));
    } else if (np > 0) {
        hipLaunchKernelGGL(mgfr::k_tsc_force, dim3(mgfr::blocks(np)), dim3(mgfr::kB), 0, s, phi, N, ilog2(N), pos, np,
                           acc);
        MGFR_TRY(hip_check(c, hipGetLastError(), "k_tsc_force"));
    }
    return MGFR_OK;
}

}  // extern "C"
