// One leg of the V-cycle on a small level in one launch.
//
// On levels of at most 64^3 the time of a V-cycle is the number of launches: a
// colour of a red-black sweep takes 3.3-4.6 us there whatever it computes, and a level
// takes eleven.  k_small_down does the pre-smoothing sweeps, the residual, the
// restriction and the FAS coarse source of a level, k_small_up the prolongation and
// the post-smoothing sweeps.  A workgroup owns a tile and holds it in LDS with
// a halo wide enough that every half-sweep of the leg can be recomputed from the old
// values of its neighbours (one cell less per half-sweep), so tiles never wait for
// each other; the iterate is written out of place.  The point updates are those of
// the per-colour kernels, in the same order: the same bits.
//
// What bounds it: the redundant updates (7200 instead of 1024 for an 8^3 tile and two
// sweeps), i.e. instruction issue.  Tiles of 8 x 4 x 4 fill the chip up to 32^3; above,
// 8^3 tiles do less redundant work in all.  Measured (Hamiltonian, 32^3): a leg down
// 12.9 and up 9.6 us for 40 us in 11 launches; solves of the ten fields at 48^3 13.6 ->
// 10.5 ms, at 128^3 (64^3 and 32^3 levels) 18.9 -> 16.5 ms.  Beyond 64^3 the tiles queue:
// with a 96^3 limit the same solves take as long or longer.
#include "stencil_ops.h"

namespace grmg {
namespace {

using namespace detail;

constexpr int ST = 8;    // tile side in x
constexpr int SNT = 512; // threads
constexpr int kSmallTileN = 32; // largest side with the small tile

// Row r of a region of side TS + 2 H in y and z: rows are numbered by their distance
// from the tile (ring d holds rows (TS - 2 + 2 d)^2 .. (TS + 2 d)^2 - 1), so the rows
// that a half-sweep still has to update are a prefix.
template <int H, int TS> __device__ __forceinline__ void region_row(int r, int &y, int &z)
{
    const int q = (int)(__builtin_amdgcn_sqrtf((float)r) + 1e-3f); // floor of the root: r < 400
    const int d = q < TS ? 0 : (q - TS + 2) >> 1, side = TS + 2 * d;
    if (d == 0) {
        y = H + (r & (TS - 1));
        z = H + (r / TS);
        return;
    }
    int k = r - (side - 2) * (side - 2);
    if (k < 2 * side) { // the ring's first and last plane
        const bool hi = k >= side;
        y = H - d + (hi ? k - side : k);
        z = hi ? H + TS - 1 + d : H - d;
    } else { // the ends of the planes between
        k -= 2 * side;
        y = (k & 1) ? H + TS - 1 + d : H - d;
        z = H - d + 1 + (k >> 1);
    }
}

template <typename T> struct Pair2;
template <> struct Pair2<double> {
    typedef double2 type;
};
template <> struct Pair2<float> {
    typedef float2 type;
};

// The region of one 8 x TS x TS tile: R = 8 + 2 H wide, RY = TS + 2 H in y and z,
// x-pairs over threads.  CPL pairs per thread, those of the rows nearest the tile first.
template <int H, int TS> struct Region {
    static constexpr int R = ST + 2 * H, RY = TS + 2 * H, SZ = R * RY, RP = R / 2, PAIRS = RY * RY * RP;
    static constexpr int CPL = (PAIRS + SNT - 1) / SNT;
    // rows within distance d of the tile
    static constexpr int rows(int d) { return (TS + 2 * d) * (TS + 2 * d); }
};

// Red-black sweeps on a region in LDS: half-sweep h updates the cells within
// distance MARGIN - h of the tile (the region's first cell has even coordinates).
// f, a, b: source and coefficients of the pairs' even (0) and odd (1) cells.
template <int KIND, typename T, int H, int TS, int MARGIN, int HALF>
__device__ __forceinline__ void region_sweeps(T *s, const int (&off)[Region<H, TS>::CPL], const T (&f0)[Region<H, TS>::CPL],
                                              const T (&f1)[Region<H, TS>::CPL], const T (&a0)[Region<H, TS>::CPL],
                                              const T (&a1)[Region<H, TS>::CPL], const T (&b0)[Region<H, TS>::CPL],
                                              const T (&b1)[Region<H, TS>::CPL], T inv_h2, OpConst oc, T Fb, T fs)
{
    using G = Region<H, TS>;
    constexpr int R = G::R;
    const T rJ = poisson_inv_diag(inv_h2);
#pragma unroll 1
    for (int h = 0; h < HALF; ++h) {
        const int d = MARGIN - h, pairs = G::rows(d) * G::RP;
#pragma unroll
        for (int c = 0; c < G::CPL; ++c) {
            if (SNT * c >= G::rows(MARGIN) * G::RP || SNT * c >= pairs) continue; // uniform: these rows are done
            const int t = threadIdx.x + SNT * c;
            // off = LDS index of the even cell, its row's parity in the sign bit's place (see prepare)
            const int p0 = off[c] & 0x3fff, par = (off[c] >> 14) & 1, x2 = off[c] >> 15;
            const int w = par ^ (h & 1); // the cell of colour h & 1
            const int x = 2 * x2 + w;
            if (t < pairs && x >= H - d && x < H + ST + d) {
                const int p = p0 + w;
                const T ph = s[p];
                const T nbs = s[p - 1] + s[p + 1] + s[p - R] + s[p + R] + s[p - G::SZ] + s[p + G::SZ];
                T J;
                const T L = op_point<KIND, T>(ph, nbs, inv_h2, w ? a1[c] : a0[c], w ? b1[c] : b0[c], oc, Fb, J);
                s[p] = newton_update<KIND, T>(ph, L, (w ? f1[c] : f0[c]) - fs, J, rJ);
            }
        }
        __syncthreads();
    }
}

struct TileAt {
    int x, y, z;
};
// tiles in contiguous runs per XCD where the grid allows it
template <int TS> __device__ __forceinline__ TileAt tile_at(int n)
{
    const int ntx = (n + ST - 1) / ST, nt = (n + TS - 1) / TS;
    const int G = gridDim.x;
    int b = blockIdx.x;
    if ((G & 7) == 0) b = (b & 7) * (G >> 3) + (b >> 3);
    return {ST * (b % ntx), TS * ((b / ntx) % nt), TS * (b / (ntx * nt))};
}

// Pair c of this thread: its place in LDS (packed: index, row parity, x2), the
// global index of its even cell.
template <int H, int TS> __device__ __forceinline__ bool region_pair(int t, const TileAt &o, int n, int &off, long &g)
{
    using G = Region<H, TS>;
    const bool on = t < G::PAIRS;
    const int row = on ? t / G::RP : 0, x2 = on ? t - row * G::RP : 0;
    int y, z;
    region_row<H, TS>(row, y, z);
    off = (z * G::SZ + y * G::R + 2 * x2) | (((y + z) & 1) << 14) | (x2 << 15);
    g = lin(wrapi(o.x - H + 2 * x2, n), wrapi(o.y - H + y, n), wrapi(o.z - H + z, n), n);
    return on;
}

// Sums of NC values per thread over a workgroup, to every thread.
template <int NC, int NT>
__device__ __forceinline__ void block_sum_all(double (&v)[NC])
{
    __shared__ double sh[NC][NT / 64];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        double x = v[c];
        for (int k = 32; k > 0; k >>= 1) x += __shfl_down(x, k, 64);
        if ((threadIdx.x & 63) == 0) sh[c][threadIdx.x >> 6] = x;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        v[c] = 0.0;
        for (int w = 0; w < NT / 64; ++w) v[c] += sh[c][w];
    }
    __syncthreads();
}
// Sums of NC values per thread over a grid of at most 4096 workgroups, in a fixed order:
// each workgroup leaves its partial sums and the one that arrives last adds them
// all (thread t adds slots t, t + NT, ..., then a tree).  True in that workgroup,
// whose thread 0 has the sums.  The counter is left at zero.
// Partials and counter are relaxed atomics of device scope: on gfx950 such a store is
// written through and such a load is taken from where all eight L2s agree, and s_waitcnt
// vmcnt(0) returns when the stores have got there, so the count cannot be seen before
// them.  (The language would ask for release and acquire; their fences write back
// and invalidate a whole L2: 5 us instead of 1.)
template <int NC, int NT>
__device__ __forceinline__ bool grid_sum(double (&v)[NC], double *partials, unsigned *count, int nblocks, int block)
{
    __shared__ bool last;
    block_sum_all<NC, NT>(v);
    if (threadIdx.x == 0) {
        for (int c = 0; c < NC; ++c)
            __hip_atomic_store(partials + c * kReduceBlocks + block, v[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        last = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)nblocks - 1u;
    }
    __syncthreads();
    if (!last) return false;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        v[c] = 0.0;
        for (int b = threadIdx.x; b < nblocks; b += NT)
            v[c] += __hip_atomic_load(partials + c * kReduceBlocks + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    block_sum_all<NC, NT>(v);
    if (threadIdx.x == 0) __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// Sum of a coarse cell's eight children, in the order of the per-launch restriction at
// this size (plane-marching from 64^3: z, x, then y pairs; below: one after another), so
// that the two paths give the same bits.
template <typename T> __device__ __forceinline__ T child_sum8(const T (&v)[8], bool pairs)
{
    T r = v[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) r += v[k];
    const T t = ((v[0] + v[4]) + (v[1] + v[5])) + ((v[2] + v[6]) + (v[3] + v[7]));
    return pairs ? t : r;
}
template <typename T> __device__ __forceinline__ T child_sum(T v, bool pairs) // one child per lane
{
    T a[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] = __shfl(v, k, 8);
    return child_sum8(a, pairs);
}

// nu = NU sweeps of level n from phi_in (null: zero) to phi_out, then
//   FAS kinds: R phi -> phi_c, phi0_c and f^H = L^H(R phi) - R eps -> f_c;
//   correction kinds: b^H = R(b - J e) -> f_c, e^H = 0 -> phi_c.
template <int KIND, typename T, int NU, int TS>
__global__ void __launch_bounds__(SNT) k_small_down(const T *__restrict__ phi_in, T *__restrict__ phi_out,
                                                    const T *__restrict__ f, const T *__restrict__ c1,
                                                    const T *__restrict__ c2, int n, T inv_h2, OpConst oc,
                                                    const double *__restrict__ fbar, const double *__restrict__ fshift,
                                                    T *__restrict__ phi_c, T *__restrict__ phi0_c, T *__restrict__ f_c,
                                                    const T *__restrict__ coef_c, const int *__restrict__ stop)
{
    constexpr bool LIN = KIND >= K_LIN_POISSON;
    constexpr int NC = kNumCoef<KIND>(), H = 2 * NU + 2;
    using G = Region<H, TS>;
    typedef typename Pair2<T>::type T2;
    constexpr int CM = ST / 2 + 2, CMY = TS / 2 + 2; // coarse cells of the tile and one around it
    __shared__ __align__(16) T s[G::RY * G::SZ];
    __shared__ T rp[CM * CMY * CMY];
    const TileAt o = tile_at<TS>(n);
    const T Fb = T(*fbar), fs = T(*fshift);
    const int stopped = stop ? *stop : 0;
    int off[G::CPL];
    T f0[G::CPL], f1[G::CPL], a0[G::CPL], a1[G::CPL], b0[G::CPL], b1[G::CPL];
    T2 ph[G::CPL];
    constexpr int SWEPT = G::rows(H - 1) * G::RP; // pairs that a half-sweep updates
#pragma unroll
    for (int c = 0; c < G::CPL; ++c) {
        long g;
        const bool on = region_pair<H, TS>(threadIdx.x + SNT * c, o, n, off[c], g);
        ph[c] = T2{T(0), T(0)};
        if (on && phi_in) ph[c] = *reinterpret_cast<const T2 *>(phi_in + g);
        T2 a{T(0), T(0)}, b{T(0), T(0)}, d{T(0), T(0)};
        if (SNT * c < SWEPT) { // compile-time
            a = *reinterpret_cast<const T2 *>(f + g);
            if (NC >= 1) b = *reinterpret_cast<const T2 *>(c1 + g);
            if (NC >= 2) d = *reinterpret_cast<const T2 *>(c2 + g);
        }
        f0[c] = a.x, f1[c] = a.y;
        a0[c] = b.x, a1[c] = b.y;
        b0[c] = d.x, b1[c] = d.y;
    }
    // the child cell of this thread in the restriction: coarse cell t >> 3 of the tile, child t & 7
    const int q = threadIdx.x >> 3, ch = threadIdx.x & 7;
    const int X = q & 3, Y = (q >> 2) % (TS / 2), Z = (q >> 2) / (TS / 2);
    const int cx = 2 * X + (ch & 1), cy = 2 * Y + ((ch >> 1) & 1), cz = 2 * Z + (ch >> 2);
    const bool inside = Z < TS / 2 && o.x + cx < n && o.y + cy < n && o.z + cz < n; // the last tiles of a side that 8 does not divide
    const long gc = inside ? lin(o.x + cx, o.y + cy, o.z + cz, n) : 0;
    const T fr = f[gc], r1 = NC >= 1 ? c1[gc] : T(0), r2 = NC >= 2 ? c2[gc] : T(0);
    const int m = n >> 1;
    const long qc = inside ? lin((o.x >> 1) + X, (o.y >> 1) + Y, (o.z >> 1) + Z, m) : 0;
    const T k1 = !LIN && NC >= 1 ? coef_c[qc] : T(0);
    if (stopped) return; // looked at after the loads above are on their way
#pragma unroll
    for (int c = 0; c < G::CPL; ++c)
        if (threadIdx.x + SNT * c < G::PAIRS) *reinterpret_cast<T2 *>(s + (off[c] & 0x3fff)) = ph[c];
    __syncthreads();
    region_sweeps<KIND, T, H, TS, H - 1, 2 * NU>(s, off, f0, f1, a0, a1, b0, b1, inv_h2, oc, Fb, fs);
    // the tile written out (its rows come first)
#pragma unroll
    for (int c = 0; c < G::CPL; ++c) {
        if (SNT * c >= G::rows(0) * G::RP) continue; // compile-time
        const int t = threadIdx.x + SNT * c, p0 = off[c] & 0x3fff, x = 2 * (off[c] >> 15) - H;
        const int y = p0 % G::SZ / G::R - H, z = p0 / G::SZ - H;
        if (t < G::rows(0) * G::RP && x >= 0 && x < ST && o.x + x < n && o.y + y < n && o.z + z < n)
            *reinterpret_cast<T2 *>(phi_out + lin(o.x + x, o.y + y, o.z + z, n)) = T2{s[p0], s[p0 + 1]};
    }
    const int p = Z < TS / 2 ? (cz + H) * G::SZ + (cy + H) * G::R + cx + H : G::SZ + G::R + 1; // in bounds for every thread
    T J;
    const T phc = s[p];
    const T L = op_point<KIND, T>(phc, s[p - 1] + s[p + 1] + s[p - G::R] + s[p + G::R] + s[p - G::SZ] + s[p + G::SZ],
                                  inv_h2, r1, r2, oc, Fb, J);
    const bool pairs = n >= 64;
    const T sr = child_sum(LIN ? fr - L : L - (fr - fs), pairs);
    if constexpr (LIN) {
        if (ch == 0 && inside) {
            f_c[qc] = sr / T(8);
            phi_c[qc] = T(0);
        }
    } else {
        // R phi of the tile's coarse cells and the ring around them (H >= 4 covers it)
        for (int t = threadIdx.x; t < CM * CMY * CMY; t += SNT) {
            const int a = t % CM, b = (t / CM) % CMY, d = t / (CM * CMY);
            const int e = (2 * d + H - 2) * G::SZ + (2 * b + H - 2) * G::R + 2 * a + H - 2;
            T sp[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) sp[k] = s[e + (k & 1) + ((k >> 1) & 1) * G::R + (k >> 2) * G::SZ];
            rp[t] = child_sum8(sp, pairs) / T(8);
        }
        __syncthreads();
        if (ch == 0 && inside) {
            const int r = ((Z + 1) * CMY + Y + 1) * CM + X + 1;
            T Jc;
            const T pc = rp[r];
            const T Lc = op_point<KIND, T>(pc, rp[r - 1] + rp[r + 1] + rp[r - CM] + rp[r + CM] + rp[r - CM * CMY] + rp[r + CM * CMY],
                                           inv_h2 * T(0.25), k1, T(0), oc, T(0), Jc);
            phi_c[qc] = pc;
            phi0_c[qc] = pc;
            f_c[qc] = Lc - sr / T(8);
        }
    }
}

// phi_in + P e (e = phi_c - phi0_c, correction kinds e = phi_c), then NU sweeps, to phi_out
template <int KIND, typename T, int NU, int TS>
__global__ void __launch_bounds__(SNT) k_small_up(const T *__restrict__ phi_in, T *__restrict__ phi_out,
                                                  const T *__restrict__ f, const T *__restrict__ c1,
                                                  const T *__restrict__ c2, int n, T inv_h2, OpConst oc,
                                                  const double *__restrict__ fbar, const double *__restrict__ fshift,
                                                  const T *__restrict__ phi_c, const T *__restrict__ phi0_c,
                                                  SmallSum sum, const int *__restrict__ stop)
{
    constexpr bool LIN = KIND >= K_LIN_POISSON;
    constexpr int NC = kNumCoef<KIND>(), H = 2 * NU;
    using G = Region<H, TS>;
    typedef typename Pair2<T>::type T2;
    constexpr int CE = G::R / 2 + 2, CEY = G::RY / 2 + 2; // coarse cells under the region and one around them
    __shared__ __align__(16) T s[G::RY * G::SZ];
    __shared__ T e[CE * CEY * CEY];
    const TileAt o = tile_at<TS>(n);
    const T Fb = T(*fbar), fs = T(*fshift);
    const int m = n >> 1;
    const int stopped = stop ? *stop : 0;
    int off[G::CPL];
    T f0[G::CPL], f1[G::CPL], a0[G::CPL], a1[G::CPL], b0[G::CPL], b1[G::CPL];
    T2 ph[G::CPL];
#pragma unroll
    for (int c = 0; c < G::CPL; ++c) {
        long g;
        (void)region_pair<H, TS>(threadIdx.x + SNT * c, o, n, off[c], g); // a place is always valid
        ph[c] = *reinterpret_cast<const T2 *>(phi_in + g);
        const T2 a = *reinterpret_cast<const T2 *>(f + g);
        T2 b{T(0), T(0)}, d{T(0), T(0)};
        if (NC >= 1) b = *reinterpret_cast<const T2 *>(c1 + g);
        if (NC >= 2) d = *reinterpret_cast<const T2 *>(c2 + g);
        f0[c] = a.x, f1[c] = a.y;
        a0[c] = b.x, a1[c] = b.y;
        b0[c] = d.x, b1[c] = d.y;
    }
    for (int t = threadIdx.x; t < CE * CEY * CEY; t += SNT) {
        const int a = t % CE, b = (t / CE) % CEY, d = t / (CE * CEY);
        const long qc = lin(wrapi((o.x >> 1) - H / 2 - 1 + a, m), wrapi((o.y >> 1) - H / 2 - 1 + b, m),
                            wrapi((o.z >> 1) - H / 2 - 1 + d, m), m);
        e[t] = LIN ? phi_c[qc] : phi_c[qc] - phi0_c[qc];
    }
    if (stopped) return;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < G::CPL; ++c) {
        const int t = threadIdx.x + SNT * c;
        if (t >= G::PAIRS) continue;
        const int p0 = off[c] & 0x3fff, x2 = off[c] >> 15, y = p0 % G::SZ / G::R, z = p0 / G::SZ;
        // H is even, so the parity of a cell in the region is its own
        const int X = x2 + 1, Y = (y >> 1) + 1, Z = (z >> 1) + 1;
        const int Y1 = Y + ((y & 1) ? 1 : -1), Z1 = Z + ((z & 1) ? 1 : -1);
        T v[2] = {T(0), T(0)};
#pragma unroll
        for (int oz = 0; oz < 2; ++oz)
#pragma unroll
            for (int oy = 0; oy < 2; ++oy) {
                const int row = ((oz ? Z1 : Z) * CEY + (oy ? Y1 : Y)) * CE + X;
                const T w = (oy ? T(0.25) : T(0.75)) * (oz ? T(0.25) : T(0.75));
                const T a = e[row - 1], b = e[row], d = e[row + 1];
                v[0] += T(0.75) * w * b;
                v[0] += T(0.25) * w * a;
                v[1] += T(0.75) * w * b;
                v[1] += T(0.25) * w * d;
            }
        *reinterpret_cast<T2 *>(s + p0) = T2{ph[c].x + v[0], ph[c].y + v[1]};
    }
    __syncthreads();
    region_sweeps<KIND, T, H, TS, H - 1, 2 * NU>(s, off, f0, f1, a0, a1, b0, b1, inv_h2, oc, Fb, fs);
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < G::CPL; ++c) {
        if (SNT * c >= G::rows(0) * G::RP) continue; // compile-time
        const int t = threadIdx.x + SNT * c, p0 = off[c] & 0x3fff, x = 2 * (off[c] >> 15) - H;
        const int y = p0 % G::SZ / G::R - H, z = p0 / G::SZ - H;
        if (t < G::rows(0) * G::RP && x >= 0 && x < ST && o.x + x < n && o.y + y < n && o.z + z < n) {
            *reinterpret_cast<T2 *>(phi_out + lin(o.x + x, o.y + y, o.z + z, n)) = T2{s[p0], s[p0 + 1]};
            acc += (double)s[p0] + (double)s[p0 + 1];
        }
    }
    if (sum.partials) {
        double v[1] = {acc};
        if (grid_sum<1, SNT>(v, sum.partials, sum.count, gridDim.x, blockIdx.x) && threadIdx.x == 0) *sum.out = v[0] * sum.scale;
    }
}

// ---- the end of a cycle of a small grid: two launches instead of six ----
// Latency: 4.6 us (pin) and 7 us (norms) at 32^3, about 3 of them the launch; the sums
// are finished by the workgroup that arrives last, not by a launch of their own.

// F = (f - A(chi^6 - 1))/chi + AA chi^-7/4 (Hamiltonian regulariser) at one point
__device__ __forceinline__ double frozen_F(double psi, double f, double AA, OpConst oc)
{
    const double chi = 1.0 - oc.kappa * psi;
    const double chi2 = chi * chi;
    const double chi6 = chi2 * chi2 * chi2;
    const double chim7 = 1.0 / (chi6 * chi);
    return (f - oc.A * (chi6 - 1.0)) / chi + 0.25 * AA * chim7;
}

// phi -= *mean (pinned), and the frozen mean of the next cycle from it: <F>
// (Hamiltonian) or add + <coef phi> (CMC)
template <int KIND>
__global__ void __launch_bounds__(256) k_pin_frozen(double *__restrict__ phi, const double *__restrict__ f,
                                                    const double *__restrict__ coef, long N, OpConst oc,
                                                    const double *__restrict__ mean, const double *__restrict__ add,
                                                    SmallSum sum, const int *__restrict__ stop)
{
    if (*stop) return;
    const double m = *mean;
    double v[1] = {0.0};
    for (long q = (long)blockIdx.x * 256 + threadIdx.x; q < N / 2; q += (long)gridDim.x * 256) {
        double2 a = reinterpret_cast<const double2 *>(phi)[q];
        const double2 c = reinterpret_cast<const double2 *>(coef)[q];
        a.x -= m;
        a.y -= m;
        reinterpret_cast<double2 *>(phi)[q] = a;
        if constexpr (KIND == GR_KIND_HAMILTONIAN) {
            const double2 b = reinterpret_cast<const double2 *>(f)[q];
            v[0] += frozen_F(a.x, b.x, c.x, oc);
            v[0] += frozen_F(a.y, b.y, c.y, oc);
        } else {
            v[0] += c.x * a.x;
            v[0] += c.y * a.y;
        }
    }
    if (grid_sum<1, 256>(v, sum.partials, sum.count, gridDim.x, blockIdx.x) && threadIdx.x == 0)
        *sum.out = (add ? *add : 0.0) + sum.scale * v[0];
}

// The stopping norms <eps^2>, <(f - fshift)^2>, and the decision whether the solve
// goes on, left on the device (later cycles that are already queued then do nothing)
// and in page-locked host memory.
template <int KIND>
__global__ void __launch_bounds__(256) k_norms_decide(const double *__restrict__ phi, const double *__restrict__ f,
                                                      const double *__restrict__ coef, int n, double inv_h2, OpConst oc,
                                                      const double *__restrict__ fbar, const double *__restrict__ fshift,
                                                      SmallSum sum, SolveControl *__restrict__ ctl,
                                                      double *__restrict__ host)
{
    if (ctl->stop) return;
    const double Fb = *fbar, fs = *fshift;
    const long N = (long)n * n * n;
    double v[2] = {0.0, 0.0};
    const float rn = __builtin_amdgcn_rcpf((float)n); // p / n by a reciprocal: p < 2^18, n <= 64
    for (int p = blockIdx.x * 256 + threadIdx.x; p < (int)N; p += gridDim.x * 256) {
        const int r = (int)(((float)p + 0.5f) * rn), z = (int)(((float)r + 0.5f) * rn), x = p - r * n, y = r - z * n;
        double J;
        const double L = op_point<KIND, double>(phi[p], nb_sum(phi, x, y, z, n), inv_h2, load_c1<KIND>(coef, p), 0.0, oc,
                                                Fb, J);
        const double fe = f[p] - fs, e = L - fe;
        v[0] += e * e;
        v[1] += fe * fe;
    }
    if (!grid_sum<2, 256>(v, sum.partials, sum.count, gridDim.x, blockIdx.x) || threadIdx.x != 0) return;
    const double r2 = v[0] * sum.scale, f2 = v[1] * sum.scale;
    sum.out[0] = r2;
    sum.out[1] = f2;
    // the host's own test (solve_one)
    const double rr = sqrt(r2), fn = sqrt(f2), rel = rr / (fn > 0.0 ? fn : 1.0);
    const bool met = ctl->rtol > 0.0 && (rel <= ctl->rtol || rr == 0.0);
    const int cyc = ctl->cycle, stop = !isfinite(rel) || met || cyc >= ctl->max_cycles;
    double *slot = host + 4 * (cyc & 1); // the next cycle's result goes to the other slot
    slot[0] = r2;
    slot[1] = f2;
    slot[2] = stop;
    __threadfence_system();
    __hip_atomic_store(slot + 3, (double)(cyc + 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); // what the host waits for
    ctl->cycle = cyc + 1;
    ctl->stop = stop;
}

__global__ void k_solve_begin(SolveControl *ctl, double rtol, int max_cycles, unsigned *count, double *fbar, double *fshift)
{
    ctl->rtol = rtol;
    ctl->max_cycles = max_cycles;
    ctl->cycle = 0;
    ctl->stop = 0;
    *count = 0;
    *fbar = 0.0;
    *fshift = 0.0;
}

// workgroups of the passes over n^3 points: two points a thread, at most 256
unsigned tail_blocks(long N)
{
    const long b = (N + 511) / 512;
    return (unsigned)(b < 256 ? b : 256);
}

// Tiles of 8 x 4 x 4 cells up to 32^3 (at most a tile per CU: the fewer redundant
// updates of a small tile count), 8^3 above (the tiles queue: their sum counts).
template <int TS> unsigned small_grid(int n)
{
    const int ntx = (n + ST - 1) / ST, nt = (n + TS - 1) / TS;
    return (unsigned)(ntx * nt * nt);
}
template <int KIND, typename T, int NU, int TS>
void down_t(hipStream_t s, const SmallLeg<T> &L, OpConst oc, const double *fbar, const double *fshift)
{
    k_small_down<KIND, T, NU, TS><<<small_grid<TS>(L.n), SNT, 0, s>>>(L.in, L.out, L.f, L.c1, L.c2, L.n,
                                                                      T(1.0 / (L.h * L.h)), oc, fbar, fshift, L.phi_c,
                                                                      L.phi0_c, L.f_c, L.coef_c, L.stop);
}
template <int KIND, typename T, int NU, int TS>
void up_t(hipStream_t s, const SmallLeg<T> &L, OpConst oc, const double *fbar, const double *fshift)
{
    k_small_up<KIND, T, NU, TS><<<small_grid<TS>(L.n), SNT, 0, s>>>(L.in, L.out, L.f, L.c1, L.c2, L.n,
                                                                    T(1.0 / (L.h * L.h)), oc, fbar, fshift, L.phi_c,
                                                                    L.phi0_c, L.sum, L.stop);
}
template <int KIND, typename T>
void down(hipStream_t s, const SmallLeg<T> &L, int nu, OpConst oc, const double *fbar, const double *fshift)
{
    if (L.n <= kSmallTileN) nu == 2 ? down_t<KIND, T, 2, 4>(s, L, oc, fbar, fshift) : down_t<KIND, T, 1, 4>(s, L, oc, fbar, fshift);
    else nu == 2 ? down_t<KIND, T, 2, 8>(s, L, oc, fbar, fshift) : down_t<KIND, T, 1, 8>(s, L, oc, fbar, fshift);
}
template <int KIND, typename T>
void up(hipStream_t s, const SmallLeg<T> &L, int nu, OpConst oc, const double *fbar, const double *fshift)
{
    if (L.n <= kSmallTileN) nu == 2 ? up_t<KIND, T, 2, 4>(s, L, oc, fbar, fshift) : up_t<KIND, T, 1, 4>(s, L, oc, fbar, fshift);
    else nu == 2 ? up_t<KIND, T, 2, 8>(s, L, oc, fbar, fshift) : up_t<KIND, T, 1, 8>(s, L, oc, fbar, fshift);
}

} // namespace

void launch_small_down(int kind, hipStream_t s, const SmallLeg<double> &L, int nu, OpConst oc, const double *fbar,
                       const double *fshift)
{
    if (kind == GR_KIND_POISSON) down<GR_KIND_POISSON>(s, L, nu, oc, fbar, fshift);
    else if (kind == GR_KIND_HAMILTONIAN) down<GR_KIND_HAMILTONIAN>(s, L, nu, oc, fbar, fshift);
    else down<GR_KIND_CMC>(s, L, nu, oc, fbar, fshift);
}

void launch_small_up(int kind, hipStream_t s, const SmallLeg<double> &L, int nu, OpConst oc, const double *fbar,
                     const double *fshift)
{
    if (kind == GR_KIND_POISSON) up<GR_KIND_POISSON>(s, L, nu, oc, fbar, fshift);
    else if (kind == GR_KIND_HAMILTONIAN) up<GR_KIND_HAMILTONIAN>(s, L, nu, oc, fbar, fshift);
    else up<GR_KIND_CMC>(s, L, nu, oc, fbar, fshift);
}

void launch_small_down_f32(int kind, hipStream_t s, const SmallLeg<float> &L, int nu, OpConst oc, const double *zero)
{
    if (kind == K_LIN_POISSON) down<K_LIN_POISSON>(s, L, nu, oc, zero, zero);
    else if (kind == K_LIN_HAM) down<K_LIN_HAM>(s, L, nu, oc, zero, zero);
    else down<K_LIN_CMC>(s, L, nu, oc, zero, zero);
}

void launch_small_up_f32(int kind, hipStream_t s, const SmallLeg<float> &L, int nu, OpConst oc, const double *zero)
{
    if (kind == K_LIN_POISSON) up<K_LIN_POISSON>(s, L, nu, oc, zero, zero);
    else if (kind == K_LIN_HAM) up<K_LIN_HAM>(s, L, nu, oc, zero, zero);
    else up<K_LIN_CMC>(s, L, nu, oc, zero, zero);
}

void launch_solve_begin(hipStream_t s, SolveControl *ctl, double rtol, int max_cycles, unsigned *count, double *fbar,
                        double *fshift)
{
    k_solve_begin<<<1, 1, 0, s>>>(ctl, rtol, max_cycles, count, fbar, fshift);
}

void launch_pin_frozen(int kind, hipStream_t s, double *phi, const double *f, const double *coef, long N, OpConst oc,
                       const double *mean, const double *add, const SmallSum &sum, const int *stop)
{
    const unsigned g = tail_blocks(N);
    if (kind == GR_KIND_HAMILTONIAN)
        k_pin_frozen<GR_KIND_HAMILTONIAN><<<g, 256, 0, s>>>(phi, f, coef, N, oc, mean, add, sum, stop);
    else
        k_pin_frozen<GR_KIND_CMC><<<g, 256, 0, s>>>(phi, f, coef, N, oc, mean, add, sum, stop);
}

void launch_norms_decide(int kind, hipStream_t s, const double *phi, const double *f, const double *coef, int n, double h,
                         OpConst oc, const double *fbar, const double *fshift, const SmallSum &sum, SolveControl *ctl,
                         double *host)
{
    const unsigned g = tail_blocks((long)n * n * n);
    const double ih2 = 1.0 / (h * h);
    if (kind == GR_KIND_POISSON)
        k_norms_decide<GR_KIND_POISSON><<<g, 256, 0, s>>>(phi, f, coef, n, ih2, oc, fbar, fshift, sum, ctl, host);
    else if (kind == GR_KIND_HAMILTONIAN)
        k_norms_decide<GR_KIND_HAMILTONIAN><<<g, 256, 0, s>>>(phi, f, coef, n, ih2, oc, fbar, fshift, sum, ctl, host);
    else
        k_norms_decide<GR_KIND_CMC><<<g, 256, 0, s>>>(phi, f, coef, n, ih2, oc, fbar, fshift, sum, ctl, host);
}

} // namespace grmg
