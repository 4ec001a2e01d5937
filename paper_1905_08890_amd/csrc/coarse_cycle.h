// The coarse levels of a V-cycle run by one workgroup (device code shared by
// the single-grid kernels and the batched ones).  Included inside namespace
// grmg::detail after stencil_ops.h.
#pragma once

#include "stencil_ops.h"

namespace grmg {
namespace detail {

// The V-cycle below (and including) level ls, run by one workgroup: every
// level is small enough to live in L2, so one launch with block barriers
// replaces the ~10 launches per level of the multi-kernel path.  Same steps,
// same order: nu1 sweeps, residual + restriction, coarse source, ..., 32
// sweeps and mean projection at the coarsest, prolongation, nu2 sweeps.
// FAS kinds: phi0 = R phi, f^H = L^H(R phi) - R eps.  Linearised kinds
// (correction scheme): b^H = R(b - J e), e^H = 0.
constexpr int kCoarseThreads = 1024;

template <int KIND, typename T>
__device__ void cv_sweep(T *__restrict__ phi, const T *__restrict__ f, const T *__restrict__ c1,
                         const T *__restrict__ c2, int n, T inv_h2, OpConst oc, T Fb, T fs)
{
    const int half = n >> 1, tot = n * n * half;
    const SmallDiv dh(half, tot), dn(n);
    const T rJ = poisson_inv_diag(inv_h2);
    for (int colour = 0; colour < 2; ++colour) {
        for (int t = threadIdx.x; t < tot; t += kCoarseThreads) {
            const int r = dh.div(t), z = dn.div(r);
            const int x2 = t - r * half, y = r - z * n;
            const int i = 2 * x2 + ((y + z + colour) & 1);
            const long p = lin(i, y, z, n);
            const T ph = phi[p];
            T J;
            const T L = op_point<KIND, T>(ph, nb_sum(phi, i, y, z, n), inv_h2, load_c1<KIND>(c1, p),
                                          load_c2<KIND>(c2, p), oc, Fb, J);
            phi[p] = newton_update<KIND, T>(ph, L, f[p] - fs, J, rJ);
        }
        __syncthreads();
    }
}

__device__ double cv_block_sum(double v)
{
    __shared__ double sh[kCoarseThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if (lane == 0) sh[wave] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < kCoarseThreads / 64; ++w) s += sh[w];
    __syncthreads();
    return s; // every thread gets the same fixed-order sum
}

template <int KIND, typename T>
__device__ void coarse_vcycle_body(const CoarseLevelsT<T> &C, int nu1, int nu2, OpConst oc, const T Fb0,
                                   const T fs0) // frozen scalars of C's first level (zero unless the finest)
{
    constexpr bool LIN = KIND >= K_LIN_POISSON;
    const int L = C.nl;
    for (int i = 0; i < L - 1; ++i) {
        const int n = C.n[i], m = n >> 1;
        const T inv_h2 = T(C.inv_h2[i]);
        const T Fb = i == 0 ? Fb0 : T(0), fs = i == 0 ? fs0 : T(0);
        for (int it = 0; it < nu1; ++it) cv_sweep<KIND, T>(C.phi[i], C.f[i], C.c1[i], C.c2[i], n, inv_h2, oc, Fb, fs);
        const int M = m * m * m;
        const SmallDiv dm(m);
        for (int q = threadIdx.x; q < M; q += kCoarseThreads) {
            const int r = dm.div(q), Z = dm.div(r);
            const int X = q - r * m, Y = r - Z * m;
            T sr = 0, sp = 0;
            for (int c = 0; c < 8; ++c) {
                const int a = 2 * X + (c & 1), b = 2 * Y + ((c >> 1) & 1), d = 2 * Z + (c >> 2);
                const long p = lin(a, b, d, n);
                const T ph = C.phi[i][p];
                T Jd;
                const T Lv = op_point<KIND, T>(ph, nb_sum(C.phi[i], a, b, d, n), inv_h2, load_c1<KIND>(C.c1[i], p),
                                               load_c2<KIND>(C.c2[i], p), oc, Fb, Jd);
                sr += Lv - (C.f[i][p] - fs);
                sp += ph;
            }
            if constexpr (LIN) {
                C.f[i + 1][q] = -sr / T(8);
                C.phi[i + 1][q] = T(0);
            } else {
                const T rp = sp / T(8);
                C.phi[i + 1][q] = rp;
                C.phi0[i + 1][q] = rp;
                C.tmp[i + 1][q] = sr / T(8);
            }
        }
        __syncthreads();
        if constexpr (!LIN) {
            const T inv_H2 = T(C.inv_h2[i + 1]);
            for (int q = threadIdx.x; q < M; q += kCoarseThreads) {
                const int r = dm.div(q), Z = dm.div(r);
                const int X = q - r * m, Y = r - Z * m;
                T Jd;
                const T Lv = op_point<KIND, T>(C.phi[i + 1][q], nb_sum(C.phi[i + 1], X, Y, Z, m), inv_H2,
                                               load_c1<KIND>(C.c1[i + 1], q), load_c2<KIND>(C.c2[i + 1], q), oc, T(0),
                                               Jd);
                C.f[i + 1][q] = Lv - C.tmp[i + 1][q];
            }
            __syncthreads();
        }
    }
    if (C.n[L - 1] * C.n[L - 1] * C.n[L - 1] <= 64) {
        // coarsest level of at most 64 points: one wavefront, one point per lane,
        // neighbours by lane shuffles (no block barriers between the sweeps)
        const int i = L - 1, n = C.n[i], N = n * n * n;
        if (threadIdx.x < 64) {
            const int lane = threadIdx.x;
            const bool on = lane < N;
            const int a = lane % n, b = (lane / n) % n, d = lane / (n * n);
            const int xp = (int)lin(wrapi(a + 1, n), b, d, n), xm = (int)lin(wrapi(a - 1, n), b, d, n);
            const int yp = (int)lin(a, wrapi(b + 1, n), d, n), ym = (int)lin(a, wrapi(b - 1, n), d, n);
            const int zp = (int)lin(a, b, wrapi(d + 1, n), n), zm = (int)lin(a, b, wrapi(d - 1, n), n);
            const T inv_h2 = T(C.inv_h2[i]);
            const T Fb = i == 0 ? Fb0 : T(0), fs = i == 0 ? fs0 : T(0);
            T ph = on ? C.phi[i][lane] : T(0);
            const T fv = on ? C.f[i][lane] : T(0);
            const T cv1 = on ? load_c1<KIND>(C.c1[i], lane) : T(0);
            const T cv2 = on ? load_c2<KIND>(C.c2[i], lane) : T(0);
            const T old = ph;
            const int par = (a + b + d) & 1;
            for (int it = 0; it < kCoarseSweeps; ++it)
                for (int colour = 0; colour < 2; ++colour) {
                    const T nbs = __shfl(ph, on ? xp : lane, 64) + __shfl(ph, on ? xm : lane, 64) +
                                  __shfl(ph, on ? yp : lane, 64) + __shfl(ph, on ? ym : lane, 64) +
                                  __shfl(ph, on ? zp : lane, 64) + __shfl(ph, on ? zm : lane, 64);
                    if (on && par == colour) {
                        T J;
                        const T Lv = op_point<KIND, T>(ph, nbs, inv_h2, cv1, cv2, oc, Fb, J);
                        ph = newton_update<KIND, T>(ph, Lv, fv - fs, J, poisson_inv_diag(inv_h2));
                    }
                }
            double dsum = on ? (double)(ph - old) : 0.0;
            for (int off = 1; off < 64; off <<= 1) dsum += __shfl_xor(dsum, off, 64);
            ph -= T(dsum / (double)N);
            if (on) C.phi[i][lane] = ph;
        }
        __syncthreads();
    } else { // coarsest: sweeps, then remove the mean of the correction
        const int i = L - 1, n = C.n[i], N = n * n * n;
        const T inv_h2 = T(C.inv_h2[i]);
        const T Fb = i == 0 ? Fb0 : T(0), fs = i == 0 ? fs0 : T(0);
        for (int q = threadIdx.x; q < N; q += kCoarseThreads) C.tmp[i][q] = C.phi[i][q];
        __syncthreads();
        for (int it = 0; it < kCoarseSweeps; ++it)
            cv_sweep<KIND, T>(C.phi[i], C.f[i], C.c1[i], C.c2[i], n, inv_h2, oc, Fb, fs);
        double d = 0.0;
        for (int q = threadIdx.x; q < N; q += kCoarseThreads) d += (double)(C.phi[i][q] - C.tmp[i][q]);
        const T mean = T(cv_block_sum(d) / (double)N);
        for (int q = threadIdx.x; q < N; q += kCoarseThreads) C.phi[i][q] -= mean;
        __syncthreads();
    }
    for (int i = L - 2; i >= 0; --i) {
        const int n = C.n[i], m = n >> 1, N = n * n * n;
        const T inv_h2 = T(C.inv_h2[i]);
        const T Fb = i == 0 ? Fb0 : T(0), fs = i == 0 ? fs0 : T(0);
        const SmallDiv dn(n);
        for (int p = threadIdx.x; p < N; p += kCoarseThreads) {
            const int r = dn.div(p), d = dn.div(r);
            const int a = p - r * n, b = r - d * n;
            const int I = a >> 1, J = b >> 1, K = d >> 1;
            const int Is[2] = {I, wrapi(I + ((a & 1) ? 1 : -1), m)};
            const int Js[2] = {J, wrapi(J + ((b & 1) ? 1 : -1), m)};
            const int Ks[2] = {K, wrapi(K + ((d & 1) ? 1 : -1), m)};
            T v = 0;
            for (int c = 0; c < 8; ++c) {
                const int ox = c & 1, oy = (c >> 1) & 1, oz = c >> 2;
                const T w = (ox ? T(0.25) : T(0.75)) * (oy ? T(0.25) : T(0.75)) * (oz ? T(0.25) : T(0.75));
                const long q = lin(Is[ox], Js[oy], Ks[oz], m);
                v += w * (LIN ? C.phi[i + 1][q] : C.phi[i + 1][q] - C.phi0[i + 1][q]);
            }
            C.phi[i][p] += v;
        }
        __syncthreads();
        for (int it = 0; it < nu2; ++it) cv_sweep<KIND, T>(C.phi[i], C.f[i], C.c1[i], C.c2[i], n, inv_h2, oc, Fb, fs);
    }
}

// ---- the same cycle with every level held in LDS ----
//
// Levels up to 16^3: the first level's iterate, source and all levels'
// coefficients are copied in, the first level's iterate is copied back.  One
// workgroup's cycle is bound by what its four SIMDs issue (four clocks a wavefront
// instruction) and by the latency of ~20 short phases between barriers.  So:
// 32-bit indices into one LDS array (addresses kept in a table in LDS made every
// access a flat one); a thread owns x-pairs of cells, whose indices, sources and
// coefficients it forms once per visit of a level (~27 instructions a point instead
// of ~85); the four pairs of a coarse cell sit in adjacent lanes, so restriction
// sums by DPP; the coarsest sweeps run in one wavefront without barriers, and on
// 2^3 in registers.  Per cycle from 16^3, Poisson (FP32 arrays, three streams) 57.9 ->
// 28.8 us; from 8^3, Hamiltonian 38.6 -> 20.6 us; patches from 9-16^3 81 -> 43 us.
//
// BC = kPeriodic: dense n^3 levels, neighbours wrap.  BC = kFaces: Dirichlet
// patch levels, the iterate padded by one cell whose values are the face values
// (patch_ops.h), read from the caller's arrays on every level.
// TG is the type of the arrays in global memory, T the type the cycle computes
// in (FP64 also for the FP32 correction cycles: their coarsest levels and mean
// constraint are solved in FP64).
constexpr int kPeriodic = 0, kFaces = 1;
constexpr size_t kCoarseLdsBytes = 150 * 1024;
constexpr size_t kCoarseLdsSmall = 20 * 1024; // enough for levels up to 8^3 of every kind
constexpr int kCoarseLdsN = 16;                   // largest level: 2 pairs per thread of 1024
constexpr int kCoarseLdsWideN = 20;               // the same with 4 pairs per thread
constexpr int kCoarseNT = 1024, kCoarseNTSmall = 256;
static_assert(kCoarseLdsN * kCoarseLdsN * kCoarseLdsN / 2 <= 2 * kCoarseNT &&
                  kCoarseLdsWideN * kCoarseLdsWideN * kCoarseLdsWideN / 2 <= 4 * kCoarseNT && 8 * 8 * 8 / 2 <= kCoarseNTSmall,
              "a thread has a place for each of its pairs");
static_assert(kCoarseSweeps >= 20, "the closed form of the 2^3 Poisson sweeps");

// Offsets (in values) of one level's arrays in LDS.
struct LdsLevel {
    int n, phi, phi0, f, c1, c2, end;
};
template <int KIND, int BC>
__host__ __device__ __forceinline__ LdsLevel lds_level(int n0, int i)
{
    constexpr bool LIN = KIND >= K_LIN_POISSON;
    constexpr int NC = kNumCoef<KIND>();
    LdsLevel V{};
    int off = 0;
    for (int l = 0; l <= i; ++l) {
        const int n = n0 >> l, N = n * n * n, W = n + 2 * BC;
        V.n = n;
        V.phi = off;
        off += W * W * W;
        V.phi0 = off;
        off += (l >= 1 && !LIN) ? N : 0;
        V.f = off;
        off += N;
        V.c1 = off;
        off += NC >= 1 ? N : 0;
        V.c2 = off;
        off += NC >= 2 ? N : 0;
        V.end = off;
    }
    return V;
}

// bytes the cycle of levels n0, n0 / 2, ... (nl of them) needs
template <int KIND, int BC> __host__ __device__ inline size_t coarse_lds_bytes(int n0, int nl)
{
    return (size_t)lds_level<KIND, BC>(n0, nl - 1).end * sizeof(double);
}

// bytes of LDS, or 0 where the cycle does not fit (largest: the side that the threads take)
template <int KIND, int BC> __host__ __device__ inline size_t coarse_lds_need(int n0, int nl, int largest = kCoarseLdsN)
{
    if (n0 > largest) return 0;
    const size_t b = coarse_lds_bytes<KIND, BC>(n0, nl);
    return b <= kCoarseLdsBytes ? b : 0;
}

template <int BC> __device__ __forceinline__ int lds_idx(int i, int j, int k, int n)
{
    return BC == kPeriodic ? (k * n + j) * n + i : ((k + 1) * (n + 2) + j + 1) * (n + 2) + i + 1;
}

// t / d of small non-negative integers (t < 2^16, d <= 64) by a reciprocal
__device__ __forceinline__ int div_small(int t, float rd) { return (int)(((float)t + 0.5f) * rd); }
__device__ __forceinline__ float rcp_small(int d) { return __builtin_amdgcn_rcpf((float)d); }

// An x-pair of cells (2 x2, 2 x2 + 1) of row (y, z): LDS index of the even cell,
// offsets to the y and z neighbours, the pair's outer x neighbours, the dense
// index of the even cell; par = colour of the even cell.  An odd side's last pair
// has no odd cell.
struct LdsPair {
    int p, ym, yp, zm, zp, xm, xp, q, par;
    bool on, odd;  // the pair and its odd cell exist
    int fy, fz;    // kFaces: -1, 0, 1 = the face the cells touch
    bool fx0, fx1; // kFaces: the even cell touches x- / the last cell touches x+
};
template <int BC> __device__ __forceinline__ LdsPair lds_pair(int x2, int y, int z, int n, bool on)
{
    LdsPair P;
    const int sy = n + 2 * BC, sz = sy * sy;
    P.on = on;
    if (!on) x2 = y = z = 0;
    P.p = lds_idx<BC>(2 * x2, y, z, n);
    P.q = (z * n + y) * n + 2 * x2;
    P.ym = -sy;
    P.yp = sy;
    P.zm = -sz;
    P.zp = sz;
    P.xm = P.p - 1;
    P.xp = P.p + 2;
    P.par = (y + z) & 1;
    P.odd = 2 * x2 + 1 < n;
    P.fy = P.fz = 0;
    P.fx0 = P.fx1 = false;
    if constexpr (BC == kPeriodic) {
        if (y == 0) P.ym += n * sy;
        if (y == n - 1) P.yp -= n * sy;
        if (z == 0) P.zm += n * sz;
        if (z == n - 1) P.zp -= n * sz;
        if (x2 == 0) P.xm += n;
        if (2 * x2 + 2 == n) P.xp -= n;
    } else {
        P.fy = y == 0 ? -1 : (y == n - 1 ? 1 : 0);
        P.fz = z == 0 ? -1 : (z == n - 1 ? 1 : 0);
        P.fx0 = x2 == 0;
        P.fx1 = 2 * x2 + 2 >= n;
    }
    return P;
}

// L(phi) at cell `w` (0 even, 1 odd) of a pair, dL/dphi there, the iterate and
// (kFaces) the number of boundary faces; the order of the neighbours and the face
// terms are those of nb_sum and patch_op
template <int KIND, int BC, typename T>
__device__ __forceinline__ T pair_op(const T *phi, const LdsPair &P, int w, T inv_h2, T c1, T c2, OpConst oc, T Fb, T &J,
                                     T &ph, int &nf)
{
    const int p = P.p + w;
    ph = phi[p];
    const T vxm = phi[w ? P.p : P.xm], vxp = phi[w ? P.xp : P.p + 1];
    const T vym = phi[p + P.ym], vyp = phi[p + P.yp], vzm = phi[p + P.zm], vzp = phi[p + P.zp];
    T nbs = vxm + vxp + vym + vyp + vzm + vzp;
    nf = 0;
    if constexpr (BC == kFaces) { // across a boundary face 2b - phi (sides are at least 3: one face per axis)
        const bool x0 = !w && P.fx0, x1 = P.fx1 && (w || !P.odd);
        if (x0 || x1) {
            nbs += (x0 ? vxm : vxp) - ph;
            ++nf;
        }
        if (P.fy) {
            nbs += (P.fy < 0 ? vym : vyp) - ph;
            ++nf;
        }
        if (P.fz) {
            nbs += (P.fz < 0 ? vzm : vzp) - ph;
            ++nf;
        }
    }
    const T L = op_point<KIND, T>(ph, nbs, inv_h2, c1, c2, oc, Fb, J);
    if constexpr (BC == kFaces)
        if (nf) J -= T(nf) * inv_h2 * (KIND == GR_KIND_HAMILTONIAN ? T(1) - T(oc.kappa) * ph : T(1));
    return L;
}

// pair t of a level.  QUADS (even sides): the four pairs of a coarse cell in
// adjacent lanes, t = 4 (coarse cell) + dy + 2 dz; else rows of pairs in order.
template <int BC, bool QUADS> __device__ __forceinline__ LdsPair lds_pair_of(int t, int n, float rhalf, float rn, float rm)
{
    const int half = (n + 1) >> 1;
    if constexpr (QUADS) {
        const int q = t >> 2, r = div_small(q, rm), Z = div_small(r, rm);
        return lds_pair<BC>(q - r * half, 2 * (r - Z * half) + (t & 1), 2 * Z + ((t >> 1) & 1), n, t < n * n * half);
    } else {
        const int r = div_small(t, rhalf), z = div_small(r, rn);
        return lds_pair<BC>(t - r * half, r - z * n, z, n, t < n * n * half);
    }
}

// Sum of the six neighbours of cell w of a pair (its own value ph: across a boundary
// face the neighbour is 2 b - ph, added as b + (b - ph))
template <int BC, typename T> __device__ __forceinline__ T pair_nbs(const T *phi, const LdsPair &P, int w, T ph)
{
    const int p = P.p + w;
    const T vxm = phi[w ? P.p : P.xm], vxp = phi[w ? P.xp : P.p + 1];
    const T vym = phi[p + P.ym], vyp = phi[p + P.yp], vzm = phi[p + P.zm], vzp = phi[p + P.zp];
    T nbs = vxm + vxp + vym + vyp + vzm + vzp;
    if constexpr (BC == kFaces) {
        const bool x0 = !w && P.fx0, x1 = P.fx1 && (w || !P.odd);
        if (x0 || x1) nbs += (x0 ? vxm : vxp) - ph;
        if (P.fy) nbs += (P.fy < 0 ? vym : vyp) - ph;
        if (P.fz) nbs += (P.fz < 0 ? vzm : vzp) - ph;
    }
    return nbs;
}

// `sweeps` red-black sweeps of a level by NTH threads, CPL pairs each.  NTH = 64:
// one wavefront, whose LDS accesses are done in order, so a phase needs no barrier.
// One division per cell and visit, by the diagonal D = 6 a / h^2 - c (plus 1 / h^2 per
// face).  The corrections (which start from zero) take the Gauss-Seidel value itself,
// (a nbs / h^2 - f) / D, as alpha nbs + beta: six dependent operations a phase
// instead of ten (phases are latency-bound).  The FAS kinds hold the whole field, whose
// smooth part alpha's rounding would damp (converged FP64 Poisson solves were 1.4 to 4
// times further from the exact ones): they add the change alpha (nbs - 6 ph) + beta,
// whose first difference is exact for smooth fields: eight operations.
template <int KIND, int BC, int CPL, int NTH, bool QUADS, typename T>
__device__ __forceinline__ void lds_sweeps(T *s, const LdsLevel &V, int sweeps, T inv_h2, OpConst oc, T Fb, T fs)
{
    constexpr int NC = kNumCoef<KIND>();
    constexpr bool HAM = KIND == GR_KIND_HAMILTONIAN, FAS = KIND < K_LIN_POISSON, CMC = KIND == GR_KIND_CMC;
    const int n = V.n;
    const float rhalf = rcp_small((n + 1) >> 1), rn = rcp_small(n);
    T *phi = s + V.phi;
    LdsPair P[CPL];
    T u[CPL][2], v[CPL][2]; // per cell: alpha and beta; Hamiltonian: f and the coefficient
    T m[CPL][2];            // CMC: the mass term's share of the change, -m2 / D
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        P[c] = lds_pair_of<BC, QUADS>(threadIdx.x + NTH * c, n, rhalf, rn, rhalf);
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const int q = P[c].q + (P[c].odd ? w : 0);
            const T f = s[V.f + q] - fs, c1 = NC >= 1 ? s[V.c1 + q] : T(0);
            if constexpr (HAM) {
                u[c][w] = f;
                v[c][w] = c1;
            } else {
                const T a = KIND == K_LIN_HAM ? s[V.c2 + q] : T(1);
                T D = T(6) * a * inv_h2 + (KIND == GR_KIND_CMC ? c1 : -c1);
                if constexpr (BC == kFaces) {
                    const bool x0 = !w && P[c].fx0, x1 = P[c].fx1 && (w || !P[c].odd);
                    const int nf = ((x0 || x1) ? 1 : 0) + (P[c].fy ? 1 : 0) + (P[c].fz ? 1 : 0);
                    D += T(nf) * inv_h2;
                }
                const T rD = T(1) / D;
                u[c][w] = a * inv_h2 * rD;
                v[c][w] = -f * rD;
                if (CMC) m[c][w] = -c1 * rD;
            }
        }
    }
#pragma unroll 1
    for (int h = 0; h < 2 * sweeps; ++h) {
        T x[CPL];
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const int w = P[c].par ^ (h & 1);
            const T uc = w ? u[c][1] : u[c][0], vc = w ? v[c][1] : v[c][0];
            if constexpr (HAM) {
                T J, ph;
                int nf;
                const T L = pair_op<KIND, BC, T>(phi, P[c], w, inv_h2, vc, T(0), oc, Fb, J, ph, nf);
                x[c] = ph - (L - uc) / J;
            } else if constexpr (FAS) {
                const T ph = phi[P[c].p + w];
                const T d = pair_nbs<BC, T>(phi, P[c], w, ph) - T(6) * ph;
                const T b = CMC ? (w ? m[c][1] : m[c][0]) * ph + vc : vc;
                x[c] = ph + (uc * d + b);
            } else {
                x[c] = uc * pair_nbs<BC, T>(phi, P[c], w, T(0)) + vc;
            }
        }
        if (NTH == 64) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); // no reordering by the compiler
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const int w = P[c].par ^ (h & 1);
            if (P[c].on && (!w || P[c].odd)) phi[P[c].p + w] = x[c];
        }
        if (NTH == 64) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
    }
}

// value of the lane whose number differs in bit b (0, 1, 2), by DPP
template <int B> __device__ __forceinline__ double lane_xor(double v)
{
    union {
        double d;
        int i[2];
    } a, r;
    a.d = v;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        if constexpr (B == 0) r.i[w] = __builtin_amdgcn_mov_dpp(a.i[w], 0xb1, 0xf, 0xf, true); // quad [1,0,3,2]
        else if constexpr (B == 1) r.i[w] = __builtin_amdgcn_mov_dpp(a.i[w], 0x4e, 0xf, 0xf, true); // quad [2,3,0,1]
        else { // within 8 lanes: reversed (7 - l), then the quad reversed (l ^ 3)
            const int m = __builtin_amdgcn_mov_dpp(a.i[w], 0x141, 0xf, 0xf, true); // row_half_mirror
            r.i[w] = __builtin_amdgcn_mov_dpp(m, 0x1b, 0xf, 0xf, true);            // quad [3,2,1,0]
        }
    }
    return r.d;
}
// value of lane l ^ 1 and l ^ 2 added: sums over the four lanes of a quad, to all of them
__device__ __forceinline__ double quad_sum(double v)
{
    v += lane_xor<0>(v);
    return v + lane_xor<1>(v);
}
template <int B> __device__ __forceinline__ double walsh_stage(double v, int lane)
{
    const double u = lane_xor<B>(v);
    return (lane >> B) & 1 ? u - v : v + u;
}

// The 32 sweeps on the 2^3 torus, in one wavefront's registers; the Poisson kinds
// in closed form: the sweeps contract
// every pair of Walsh modes s, s + (1,1,1) by 1/9 each, so 32 sweeps leave the
// exact solution to below one rounding (9^-32), except the pair of the constant
// and the checkerboard mode, whose sweeps end with phi_even - phi_odd = h^2 <f_odd>
// / 6 whatever they started from and a constant that the mean constraint replaces.
// 2^3 periodic, one point per lane 0..7 (the other lanes repeat them); ends with
// the mean of the correction removed
template <int KIND, typename T>
__device__ void coarsest_two(T *s, const LdsLevel &V, T inv_h2, OpConst oc, T Fb, T fs)
{
    constexpr int NC = kNumCoef<KIND>();
    constexpr bool POI = KIND == GR_KIND_POISSON || KIND == K_LIN_POISSON;
    const int l = threadIdx.x & 7;
    const bool odd = __popc(l) & 1;
    T ph = s[V.phi + l];
    const T old = ph;
    const T f = s[V.f + l] - fs;
    if constexpr (POI) {
        T F = walsh_stage<2>(walsh_stage<1>(walsh_stage<0>(f, l), l), l); // F_s of mode s = lane
        const T M = walsh_stage<2>(walsh_stage<1>(walsh_stage<0>(ph, l), l), l);
        const T F0 = __shfl(F, 0, 8), h2 = T(1) / inv_h2;
        T c;
        if (l == 0) c = M / T(8);                                  // the old mean
        else if (l == 7) c = (F0 - F) * h2 / T(96);                // checkerboard: h^2 <f_odd> / 12
        else c = F * h2 / (T(-32) * T(__popc(l)));                 // F_s / (8 lambda_s), lambda_s = -4 |s| / h^2
        ph = walsh_stage<2>(walsh_stage<1>(walsh_stage<0>(c, l), l), l);
    } else {
        const T c1 = NC >= 1 ? s[V.c1 + l] : T(0), c2 = NC >= 2 ? s[V.c2 + l] : T(0);
        T al = T(0), be = T(0), ma = T(0); // as lds_sweeps
        if constexpr (KIND != GR_KIND_HAMILTONIAN) {
            const T a = KIND == K_LIN_HAM ? c2 : T(1), rD = T(1) / (T(6) * a * inv_h2 + (KIND == GR_KIND_CMC ? c1 : -c1));
            al = a * inv_h2 * rD;
            be = -f * rD;
            ma = -c1 * rD;
        }
        for (int it = 0; it < kCoarseSweeps; ++it)
#pragma unroll
            for (int colour = 0; colour < 2; ++colour) {
                const T x = lane_xor<0>(ph), y = lane_xor<1>(ph), z = lane_xor<2>(ph);
                const T nbs = x + x + y + y + z + z; // both neighbours of an axis are the same cell
                T v;
                if constexpr (KIND == GR_KIND_HAMILTONIAN) {
                    T J;
                    const T L = op_point<KIND, T>(ph, nbs, inv_h2, c1, c2, oc, Fb, J);
                    v = ph - (L - f) / J;
                } else if constexpr (KIND == GR_KIND_CMC) {
                    const T d = nbs - T(6) * ph;
                    v = ph + (al * d + (ma * ph + be));
                } else {
                    v = al * nbs + be;
                }
                ph = (odd == (colour == 1)) ? v : ph;
            }
        T d = ph - old;
        d += lane_xor<0>(d);
        d += lane_xor<1>(d);
        d += lane_xor<2>(d);
        ph -= d / T(8);
    }
    if (threadIdx.x < 8) s[V.phi + l] = ph;
}

// sum of v over the first wavefront's lanes (every lane gets it)
__device__ __forceinline__ double wave_sum(double v)
{
    for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// CPL: pairs per thread of the largest level (2 for 16^3 and 4 for 20^3 with 1024 threads, 1 for 8^3 with 256)
template <int KIND, int BC, int NT, int CPL, typename TG, typename T>
__device__ void coarse_cycle_body(T *s, const CoarseLevelsT<TG> &G, int nu1, int nu2, OpConst oc, const T Fb0,
                                  const T fs0)
{
    constexpr bool LIN = KIND >= K_LIN_POISSON;
    constexpr int NC = kNumCoef<KIND>();
    const int L = G.nl, n0 = G.n[0];
    // down to the coarsest level and back up in one loop: every phase's code is there once
#pragma unroll 1
    for (int step = 0; step < 2 * L - 1; ++step) {
        const bool up = step >= L, coarsest = step == L - 1;
        const int i = up ? 2 * L - 2 - step : step;
        const LdsLevel V = lds_level<KIND, BC>(n0, i), C = lds_level<KIND, BC>(n0, i + 1);
        const int n = V.n, N = n * n * n, m = C.n, M = m * m * m;
        const T inv_h2 = T(G.inv_h2[i]), Fb = i == 0 ? Fb0 : T(0), fs = i == 0 ? fs0 : T(0);
        const float rm = rcp_small(m), rn = rcp_small(n);
        if (up) { // phi += P e, e = phi^H - R phi (correction scheme: e = phi^H)
            if constexpr (!LIN) { // e over R phi
                for (int q = threadIdx.x; q < M; q += NT) {
                    const int r = div_small(q, rm), Z = div_small(r, rm);
                    s[C.phi0 + q] = s[C.phi + lds_idx<BC>(q - r * m, r - Z * m, Z, m)] - s[C.phi0 + q];
                }
                __syncthreads();
            }
            const T *e = s + (LIN ? C.phi : C.phi0);
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                const int t = threadIdx.x + NT * c;
                if (t >= 4 * M) break;
                const int q = t >> 2, r = div_small(q, rm), Z = div_small(r, rm), X = q - r * m, Y = r - Z * m;
                const int dy = t & 1, dz = (t >> 1) & 1;
                int Xs[3] = {X - 1, X, X + 1}, Ys[2] = {Y, Y + (dy ? 1 : -1)}, Zs[2] = {Z, Z + (dz ? 1 : -1)};
                T gx[3] = {1, 1, 1}, gy = 1, gz = 1; // kFaces: the correction is odd across every face
                if constexpr (BC == kPeriodic) {
                    Xs[0] = wrapi(Xs[0], m);
                    Xs[2] = wrapi(Xs[2], m);
                    Ys[1] = wrapi(Ys[1], m);
                    Zs[1] = wrapi(Zs[1], m);
                } else {
                    if (Xs[0] < 0) { Xs[0] = X; gx[0] = -1; }
                    if (Xs[2] >= m) { Xs[2] = X; gx[2] = -1; }
                    if ((unsigned)Ys[1] >= (unsigned)m) { Ys[1] = Y; gy = -1; }
                    if ((unsigned)Zs[1] >= (unsigned)m) { Zs[1] = Z; gz = -1; }
                }
                T v[2] = {0, 0};
#pragma unroll
                for (int oz = 0; oz < 2; ++oz)
#pragma unroll
                    for (int oy = 0; oy < 2; ++oy) {
                        const int row = (Zs[oz] * m + Ys[oy]) * m;
                        T wyz = (oy ? T(0.25) : T(0.75)) * (oz ? T(0.25) : T(0.75));
                        if constexpr (BC == kFaces) wyz *= (oy ? gy : T(1)) * (oz ? gz : T(1));
                        const T a = e[row + Xs[0]], b = e[row + Xs[1]], d = e[row + Xs[2]];
                        v[0] += T(0.75) * wyz * b;
                        v[0] += T(0.25) * wyz * (BC == kFaces ? gx[0] * a : a);
                        v[1] += T(0.75) * wyz * b;
                        v[1] += T(0.25) * wyz * (BC == kFaces ? gx[2] * d : d);
                    }
                const int p = V.phi + lds_idx<BC>(2 * X, 2 * Y + dy, 2 * Z + dz, n);
                s[p] += v[0];
                s[p + 1] += v[1];
            }
            __syncthreads();
        }
        if (!coarsest) {
            lds_sweeps<KIND, BC, CPL, NT, true, T>(s, V, up ? nu2 : nu1, inv_h2, oc, Fb, fs);
        } else if (BC == kPeriodic && n == 2) {
            if constexpr (BC == kPeriodic)
                if (threadIdx.x < 64) coarsest_two<KIND, T>(s, V, inv_h2, oc, Fb, fs);
            __syncthreads();
        } else if (n <= 6) { // at most 108 pairs
            if (threadIdx.x < 64) lds_sweeps<KIND, BC, 2, 64, false, T>(s, V, kCoarseSweeps, inv_h2, oc, Fb, fs);
            __syncthreads();
        } else {
            lds_sweeps<KIND, BC, CPL, NT, false, T>(s, V, kCoarseSweeps, inv_h2, oc, Fb, fs);
        }
        if (coarsest && BC == kPeriodic && n != 2) { // the mean of the correction removed
            // the iterate before the sweeps: R phi (FAS), zero (correction scheme), or the caller's array
            auto before = [&](int q) { return i == 0 ? T(G.phi[0][q]) : (LIN ? T(0) : s[V.phi0 + q]); };
            __shared__ double mean;
            if (threadIdx.x < 64) {
                double d = 0.0;
                for (int q = threadIdx.x; q < N; q += 64) d += (double)(s[V.phi + q] - before(q));
                d = wave_sum(d) / (double)N;
                if (threadIdx.x == 0) mean = d;
            }
            __syncthreads();
            for (int q = threadIdx.x; q < N; q += NT) s[V.phi + q] -= T(mean);
            __syncthreads();
        }
        if (up || coarsest) continue;
        // R phi and R eps (correction scheme: b^H = R(b - J e)): a pair per thread, the four
        // pairs of a coarse cell summed over their quad of lanes
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const int t = threadIdx.x + NT * c;
            const LdsPair P = lds_pair_of<BC, true>(t, n, rm, rn, rm);
            T sr = 0, sp = 0;
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const int q = P.q + w;
                T J, ph;
                int nf;
                const T Lv = pair_op<KIND, BC, T>(s + V.phi, P, w, inv_h2, NC >= 1 ? s[V.c1 + q] : T(0),
                                                  NC >= 2 ? s[V.c2 + q] : T(0), oc, Fb, J, ph, nf);
                sr += Lv - (s[V.f + q] - fs);
                sp += ph;
            }
            sr = quad_sum(sr);
            if constexpr (!LIN) sp = quad_sum(sp);
            if (!P.on || (t & 3)) continue;
            const int q = t >> 2;
            if constexpr (LIN) {
                s[C.f + q] = -sr / T(8);
                s[C.phi + q] = T(0);
            } else {
                const int r = div_small(q, rm), Z = div_small(r, rm);
                const T rp = sp / T(8);
                s[C.phi + lds_idx<BC>(q - r * m, r - Z * m, Z, m)] = rp;
                s[C.phi0 + q] = rp;
                s[C.f + q] = sr / T(8);
            }
        }
        __syncthreads();
        if constexpr (!LIN) { // f^H = L^H(R phi) - R eps; every cell of a pair (odd coarse sides too)
            const T inv_H2 = T(G.inv_h2[i + 1]);
            const int mh = (m + 1) >> 1;
            const LdsPair P = lds_pair_of<BC, false>(threadIdx.x, m, rcp_small(mh), rm, rm);
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                if (!P.on || (w && !P.odd)) continue;
                const int q = P.q + w;
                T J, ph;
                int nf;
                const T Lv = pair_op<KIND, BC, T>(s + C.phi, P, w, inv_H2, NC >= 1 ? s[C.c1 + q] : T(0),
                                                  NC >= 2 ? s[C.c2 + q] : T(0), oc, T(0), J, ph, nf);
                s[C.f + q] = Lv - s[C.f + q];
            }
            __syncthreads();
        }
    }
}

// s: the workgroup's LDS, at least coarse_lds_bytes; called by NT threads.  Only for
// levels that coarse_lds_need accepts: a larger first level has more pairs than the threads
// take and runs past the LDS.
template <int KIND, int BC, int NT, typename TG, typename T, int CPL = (NT >= 1024 ? 2 : 1)>
__device__ void coarse_cycle_lds(T *s, const CoarseLevelsT<TG> &G, int nu1, int nu2, OpConst oc, T Fb0, T fs0)
{
    constexpr int NC = kNumCoef<KIND>();
#pragma unroll 1
    for (int i = 0; i < G.nl; ++i) {
        const LdsLevel V = lds_level<KIND, BC>(G.n[0], i);
        const int N = V.n * V.n * V.n, W = V.n + 2 * BC, P = W * W * W;
        if (i == 0 || BC == kFaces) {
#pragma unroll 4
            for (int q = threadIdx.x; q < P; q += NT) s[V.phi + q] = T(G.phi[i][q]);
        }
#pragma unroll 4
        for (int q = threadIdx.x; q < N; q += NT) {
            if (i == 0) s[V.f + q] = T(G.f[0][q]);
            if (NC >= 1) s[V.c1 + q] = T(G.c1[i][q]);
            if (NC >= 2) s[V.c2 + q] = T(G.c2[i][q]);
        }
    }
    __syncthreads();
    coarse_cycle_body<KIND, BC, NT, CPL, TG, T>(s, G, nu1, nu2, oc, Fb0, fs0);
    const int W0 = G.n[0] + 2 * BC, P0 = W0 * W0 * W0;
    for (int q = threadIdx.x; q < P0; q += NT) G.phi[0][q] = TG(s[q]);
}

// The coarsest correction level alone, of any side: for levels that the cycle above does
// not take (a coarsest side above 16 is twice an odd number: 18, 22, 26, ...).  The same 32
// sweeps and mean, computed in FP64, cells strided over the NT = kCoarseThreads threads.
// x: N values for the iterate, LDS (sides up to 26) or global memory; e: the correction.
template <int KIND, typename TG>
__device__ __forceinline__ void coarsest_wide(double *x, int n, double inv_h2, OpConst oc, const TG *__restrict__ f,
                                              const TG *__restrict__ c1, const TG *__restrict__ c2, TG *__restrict__ e)
{
    const int n2 = n * n, N = n2 * n, half = n >> 1, tot = n2 * half;
    const SmallDiv dh(half, tot), dn(n);
    const double rJ = poisson_inv_diag(inv_h2);
    for (int q = threadIdx.x; q < N; q += kCoarseThreads) x[q] = (double)e[q];
    __syncthreads();
    for (int h = 0; h < 2 * kCoarseSweeps; ++h) {
        for (int t = threadIdx.x; t < tot; t += kCoarseThreads) {
            const int r = dh.div(t), z = dn.div(r), y = r - z * n;
            const int i = 2 * (t - r * half) + ((y + z + h) & 1), p = r * n + i; // below 2^31
            const double ph = x[p];
            const double nbs = x[i ? p - 1 : p + n - 1] + x[i < n - 1 ? p + 1 : p - i] + x[y ? p - n : p + n2 - n] +
                               x[y < n - 1 ? p + n : p - n2 + n] + x[z ? p - n2 : p + N - n2] +
                               x[z < n - 1 ? p + n2 : p - N + n2];
            double J;
            const double L = op_point<KIND, double>(ph, nbs, inv_h2, (double)load_c1<KIND>(c1, p),
                                                    (double)load_c2<KIND>(c2, p), oc, 0.0, J);
            x[p] = newton_update<KIND, double>(ph, L, (double)f[p], J, rJ);
        }
        __syncthreads();
    }
    double d = 0.0;
    for (int q = threadIdx.x; q < N; q += kCoarseThreads) d += x[q] - (double)e[q];
    const double mean = cv_block_sum(d) / (double)N;
    for (int q = threadIdx.x; q < N; q += kCoarseThreads) e[q] = TG(x[q] - mean);
}

} // namespace detail
} // namespace grmg
