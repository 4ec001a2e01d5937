// Source and coefficient builders for the ten field equations, the CIC
// matter deposit, and the derived fields (paper sec. 4.1.2, 4.3, 4.5).
#include "sources_ops.h"

#include <algorithm>

namespace grmg {

namespace {

constexpr int TPB = 256;
using namespace detail;

__device__ __forceinline__ int wrap_any(long i, int n)
{
    long r = i % n;
    return (int)(r < 0 ? r + n : r);
}

// ------------------------------------------------------------------- CIC

// Cell-centred CIC: g = x/h - 1/2, i0 = floor(g), t = g - i0, weights (1-t, t) on cells
// (i0, i0+1), periodic.  chi at the particle from the CIC-interpolated Psi;
// W^2 = c^2 + a^-2 chi^-4 u.u.
//
// (Small counts and grids: k_chain_tile.)
// The grid points are cut into tiles of 8^3.  A particle is listed with every tile that
// its cloud reaches (1.4 on average, at most 8): the entries are counted per tile, the
// counts scanned, and the particles' numbers written to their tiles' lists.  A workgroup
// then takes a tile, adds its particles' charges in LDS and stores every point once.  The
// sums of a point are taken in no fixed order.
//
// Why: memory atomics run at about 26e9 a second on this card whatever they add (they
// pass the eight L2s), so 40 a particle, or two a particle for a sort by cell, were what
// the deposit cost; and a gather per point walks the lists of a dense lump alone.  LDS
// takes both: the tile counters are first gathered per workgroup in LDS.  Against the
// sort by cell and the gather per point, and above n^3 particles the scatter with memory
// atomics (us): 128^3, 2.1e6 even particles 330 -> 170 (counting 25, lists 38, tiles 100);
// 1.5e6, 40 % of them in lumps 500 -> 227; 256^3, 16.8e6 3210 -> 1280; 192^3, 8e6 12000
// -> 750; 32^3, 3e4 60 -> 36.  Bound: the LDS adds, 17 clocks each with their conflicts.

constexpr int DT = 8, DP = DT * DT * DT;         // tile side and points
constexpr int DS = DT + 2;                       // Psi under the tile's clouds: one cell more on each side
constexpr int BNT = 1024;                // threads of the binning kernels
constexpr int BHASH = 8192, BPROBE = 32;         // hash table; entries that find no place count in memory

__device__ __forceinline__ void cic_cells(const double *__restrict__ pos, long q, int n, int *i0, int *i1, double *t)
{
    for (int d = 0; d < 3; ++d) {
        const double g = pos[3 * q + d] * n - 0.5;
        const double fl = floor(g);
        t[d] = g - fl;
        // any finite position wraps; the others count as cell 0
        const long il = isfinite(fl) ? (long)fl : 0;
        i0[d] = il >= 0 && il < n ? (int)il : wrap_any(il, n);
        i1[d] = i0[d] + 1 == n ? 0 : i0[d] + 1;
    }
}

// Tile coordinates of the lower and upper cells of a particle's cloud, 10 bits each
// (n <= 1024); no particle: the lower ones are all ones.
struct TileSpan {
    unsigned lo, hi;
};
__device__ __forceinline__ TileSpan cic_span(const double *__restrict__ pos, long q, long np, int n)
{
    if (q >= np) return {~0u, ~0u};
    int i0[3], i1[3];
    double t[3];
    cic_cells(pos, q, n, i0, i1, t);
    return {(unsigned)(i0[0] / DT) | (unsigned)(i0[1] / DT) << 10 | (unsigned)(i0[2] / DT) << 20,
            (unsigned)(i1[0] / DT) | (unsigned)(i1[1] / DT) << 10 | (unsigned)(i1[2] / DT) << 20};
}
// f(tile) for every tile of the span, once
template <typename F> __device__ __forceinline__ void for_tiles(const TileSpan s, int nt, F f)
{
    if (s.lo == ~0u) return;
    const unsigned diff = s.lo ^ s.hi;
    const int nx = diff & 1023u ? 2 : 1, ny = (diff >> 10) & 1023u ? 2 : 1, nz = diff >> 20 ? 2 : 1;
    for (int c = 0; c < nx * ny * nz; ++c) {
        const int cx = nx == 2 ? c & 1 : 0, r = nx == 2 ? c >> 1 : c, cy = ny == 2 ? r & 1 : 0, cz = ny == 2 ? r >> 1 : r;
        const int x = (cx ? s.hi : s.lo) & 1023u, y = ((cy ? s.hi : s.lo) >> 10) & 1023u, z = (cz ? s.hi : s.lo) >> 20;
        f((z * nt + y) * nt + x);
    }
}

// The slot of `key` in the workgroup's hash table, -1 if none is near; INSERT: taken if free.
template <bool INSERT> __device__ __forceinline__ int table_slot(int *keys, int key)
{
    unsigned s = ((unsigned)key * 2654435769u) >> 19; // 13 bits: BHASH
    for (int p = 0; p < BPROBE; ++p, s = (s + 1) & (BHASH - 1)) {
        int k = __hip_atomic_load(keys + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (INSERT && k == -1) k = atomicCAS(keys + s, -1, key) == -1 ? key : keys[s];
        if (k == key) return (int)s;
        if (!INSERT && k == -1) return -1;
    }
    return -1;
}

// Entries per tile (PLACE = false, at = counts) or the entries themselves (at = the
// tiles' next free places): each tile that a workgroup's particles reach costs one
// memory atomic, not each particle.  HASH = false: at most BSLOT tiles, a counter each.
template <bool PLACE, bool HASH, int BSLOT, int BPT>
__global__ void __launch_bounds__(BNT) k_cic_bin(int n, int nt, const double *__restrict__ pos, long np,
                                                 unsigned *__restrict__ at, unsigned *__restrict__ list)
{
    __shared__ int keys[HASH ? BSLOT : 1];
    __shared__ unsigned cnt[BSLOT];
    const int slots = HASH ? BSLOT : nt * nt * nt;
    const long q0 = (long)blockIdx.x * (BNT * BPT) + threadIdx.x;
    TileSpan span[BPT];
#pragma unroll
    for (int i = 0; i < BPT; ++i) span[i] = cic_span(pos, q0 + i * BNT, np, n);
    for (int i = threadIdx.x; i < slots; i += BNT) {
        if (HASH) keys[i] = -1;
        cnt[i] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < BPT; ++i)
        for_tiles(span[i], nt, [&](int k) {
            const int s = HASH ? table_slot<true>(keys, k) : k;
            if (s >= 0) atomicAdd(cnt + s, 1u);
            else if (!PLACE) atomicAdd(at + k, 1u);
        });
    __syncthreads();
    for (int i = threadIdx.x; i < slots; i += BNT)
        if (cnt[i]) {
            const unsigned b = atomicAdd(at + (HASH ? keys[i] : i), cnt[i]);
            if (PLACE) cnt[i] = b;
        }
    if constexpr (PLACE) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < BPT; ++i)
            for_tiles(span[i], nt, [&](int k) {
                const int s = HASH ? table_slot<false>(keys, k) : k;
                list[s >= 0 ? atomicAdd(cnt + s, 1u) : atomicAdd(at + k, 1u)] = (unsigned)(q0 + i * BNT);
            });
    }
}

// Exclusive scan of cnt[0..nt3) into start[0..nt3] and next[0..nt3), one workgroup; and the
// tiles with long lists, up to `room` of them (heavy[0]: how many), cnt: whether listed.
// The arrays are 16-byte aligned.
constexpr int SCNT = 1024, SCPT = 8;
constexpr int DNT = 512;
constexpr unsigned DLONG = 2 * DNT;
__global__ void __launch_bounds__(SCNT) k_cic_scan(unsigned *__restrict__ cnt, int nt3, unsigned *__restrict__ start,
                                                   unsigned *__restrict__ next, unsigned *__restrict__ heavy,
                                                   unsigned room)
{
    __shared__ unsigned wsum[SCNT / 64];
    __shared__ unsigned nheavy;
    if (threadIdx.x == 0) nheavy = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    unsigned carry = 0;
    for (int b0 = 0; b0 < nt3; b0 += SCNT * SCPT) {
        const int base = b0 + threadIdx.x * SCPT;
        const bool full = base + SCPT <= nt3;
        unsigned v[SCPT], sum = 0;
        if (full) {
#pragma unroll
            for (int i = 0; i < SCPT; i += 4) *reinterpret_cast<uint4 *>(v + i) = *reinterpret_cast<const uint4 *>(cnt + base + i);
        } else {
#pragma unroll
            for (int i = 0; i < SCPT; ++i) v[i] = base + i < nt3 ? cnt[base + i] : 0u;
        }
#pragma unroll
        for (int i = 0; i < SCPT; ++i) sum += v[i];
        unsigned x = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[w] = x;
        __syncthreads();
        unsigned run = carry + x - sum, all = 0;
        for (int i = 0; i < SCNT / 64; ++i) {
            if (i < w) run += wsum[i];
            all += wsum[i];
        }
        carry += all;
        unsigned out[SCPT], mark[SCPT];
#pragma unroll
        for (int i = 0; i < SCPT; ++i) {
            unsigned at = room;
            if (v[i] > DLONG) at = atomicAdd(&nheavy, 1u);
            if (at < room) heavy[1 + at] = (unsigned)(base + i);
            mark[i] = at < room;
            out[i] = run;
            run += v[i];
        }
        if (full) {
#pragma unroll
            for (int i = 0; i < SCPT; i += 4) {
                *reinterpret_cast<uint4 *>(start + base + i) = *reinterpret_cast<const uint4 *>(out + i);
                *reinterpret_cast<uint4 *>(next + base + i) = *reinterpret_cast<const uint4 *>(out + i);
                *reinterpret_cast<uint4 *>(cnt + base + i) = *reinterpret_cast<const uint4 *>(mark + i);
            }
        } else {
#pragma unroll
            for (int i = 0; i < SCPT; ++i)
                if (base + i < nt3) {
                    start[base + i] = next[base + i] = out[i];
                    cnt[base + i] = mark[i];
                }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        start[nt3] = carry;
        heavy[0] = nheavy < room ? nheavy : room;
    }
}

// One tile: the sources of its points from particles handed to `take` (which calls its
// argument with each particle's number), summed in LDS.  Bound by the LDS adds (40 a
// particle).  Each point is stored; ADD: added to what is there; SPLIT: other
// workgroups add to it at the same time.
struct CicVolume { // c h^3 and its reciprocal
    double v, r;
};
template <bool ADD, bool SPLIT, class Take>
__device__ __forceinline__ void cic_tile(int b, int n, int nt, double a, double c, double kap, CicVolume V,
                                         const double *__restrict__ pos, const double *__restrict__ u, double mass,
                                         const double *__restrict__ psi, double *const (&out)[5], Take take)
{
    __shared__ double acc[5][DP];
    __shared__ double ps[DS * DS * DS];
    const int T[3] = {b % nt, (b / nt) % nt, b / (nt * nt)};
    for (int i = threadIdx.x; i < 5 * DP; i += DNT) (&acc[0][0])[i] = 0.0;
    for (int i = threadIdx.x; i < DS * DS * DS; i += DNT) {
        int x[3] = {i % DS, (i / DS) % DS, i / (DS * DS)};
        for (int d = 0; d < 3; ++d) {
            x[d] += DT * T[d] - 1;
            if (x[d] < 0) x[d] += n;
            else if (x[d] >= n) x[d] %= n;
        }
        ps[i] = psi[lin(x[0], x[1], x[2], n)];
    }
    __syncthreads();
    take([&](long q) {
        int i0[3], i1[3], at[3];
        double t[3];
        cic_cells(pos, q, n, i0, i1, t);
        const double ux = u[3 * q], uy = u[3 * q + 1], uz = u[3 * q + 2];
        bool in[3][2];
        int p[3][2];
        for (int d = 0; d < 3; ++d) {
            in[d][0] = i0[d] / DT == T[d];
            in[d][1] = i1[d] / DT == T[d];
            p[d][0] = i0[d] % DT;
            p[d][1] = i1[d] % DT;
            at[d] = in[d][0] ? p[d][0] + 1 : 0;
        }
        double psi_p = 0.0;
        for (int cc = 0; cc < 8; ++cc) {
            const int ox = cc & 1, oy = (cc >> 1) & 1, oz = cc >> 2;
            const double w = (ox ? t[0] : 1.0 - t[0]) * (oy ? t[1] : 1.0 - t[1]) * (oz ? t[2] : 1.0 - t[2]);
            psi_p += w * ps[((at[2] + oz) * DS + at[1] + oy) * DS + at[0] + ox];
        }
        const double chi = 1.0 - kap * psi_p;
        const double chi2 = chi * chi;
        const double g_uu = (ux * ux + uy * uy + uz * uz) / (a * a * chi2 * chi2); // gamma^ij u_i u_j
        const double W = sqrt(c * c + g_uu);
        const double Q[5] = {W, ux, uy, uz, g_uu / W}; // times mass / (c h^3); the last: stress trace gamma^ij s_ij
#pragma unroll
        for (int cc = 0; cc < 8; ++cc) {
            const int ox = cc & 1, oy = (cc >> 1) & 1, oz = cc >> 2;
            if (!(in[0][ox] && in[1][oy] && in[2][oz])) continue;
            const double w = (ox ? t[0] : 1.0 - t[0]) * (oy ? t[1] : 1.0 - t[1]) * (oz ? t[2] : 1.0 - t[2]);
            const int r = (p[2][oz] * DT + p[1][oy]) * DT + p[0][ox];
#pragma unroll
            for (int f = 0; f < 5; ++f) unsafeAtomicAdd(&acc[f][r], w * Q[f]);
        }
    });
    __syncthreads();
    // The common factor m / (c h^3) once a point, not rounded into one number: a lattice of particles at
    // rest gives exactly 1.  The quotient by V.v = c h^3 from its rounded reciprocal and one
    // correction, which rounds as the division does (Markstein).
    for (int r = threadIdx.x; r < DP; r += DNT) {
        const int x = DT * T[0] + r % DT, y = DT * T[1] + (r / DT) % DT, z = DT * T[2] + r / (DT * DT);
        if (x >= n || y >= n || z >= n) continue;
        const long g = lin(x, y, z, n);
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            const double t = mass * acc[f][r], q = t * V.r;
            const double v = isfinite(q) ? __builtin_fma(__builtin_fma(-q, V.v, t), V.r, q) : q;
            if constexpr (SPLIT) {
                if (v != 0.0) unsafeAtomicAdd(out[f] + g, v); // NaN too
            } else {
                out[f][g] = ADD ? out[f][g] + v : v;
            }
        }
    }
}

// The tiles' particles from their lists; the first `room` workgroups take the dense
// lumps, which would otherwise be the tail.
template <bool ADD>
__global__ void __launch_bounds__(DNT) k_cic_tile(int n, int nt, double a, double c, double kap, CicVolume V,
                                                  const double *__restrict__ pos, const double *__restrict__ u,
                                                  double mass, const double *__restrict__ psi,
                                                  const unsigned *__restrict__ start, const unsigned *__restrict__ list,
                                                  const unsigned *__restrict__ listed,
                                                  const unsigned *__restrict__ heavy, int room, double *__restrict__ s0, double *__restrict__ sx,
                                                  double *__restrict__ sy, double *__restrict__ sz,
                                                  double *__restrict__ sm)
{
    int b = blockIdx.x;
    if (b < room) {
        if ((unsigned)b >= heavy[0]) return;
        b = (int)heavy[1 + b];
    } else {
        const int G = gridDim.x - room;
        b -= room;
        if ((G & 7) == 0) b = (b & 7) * (G >> 3) + (b >> 3); // runs of tiles per XCD: neighbours share particles
        if (listed[b]) return;
    }
    const unsigned first = start[b], last = start[b + 1];
    double *const out[5] = {s0, sx, sy, sz, sm};
    cic_tile<ADD, false>(b, n, nt, a, c, kap, V, pos, u, mass, psi, out, [&](auto put) {
        for (unsigned e = first + threadIdx.x; e < last; e += DNT) put((long)list[e]);
    });
}

// ---- few particles on a small grid: chains instead of lists ----
//
// Counting, scanning and placing are three passes of a few latencies each, which is all
// that 3e4 particles cost.  Here every tile has 512 chains (512 `parts` of them), one a thread
// of its workgroups: a particle is put at the head of a chain of each tile it reaches,
// by a hash of its number, in one pass with one memory atomic an entry.  `parts`
// workgroups share a tile where the tiles are too few for the chip (measured: chains_ok).
__global__ void k_chain_begin(unsigned *__restrict__ head, long nh, long N, double *__restrict__ s0, double *__restrict__ sx,
                              double *__restrict__ sy, double *__restrict__ sz, double *__restrict__ sm)
{
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < nh) head[p] = ~0u;
    if (p < N) s0[p] = sx[p] = sy[p] = sz[p] = sm[p] = 0.0; // N = 0: the tiles store every point
}
// entry e = 8 q + c: particle q in the c-th of its tiles; next[e]: the entry behind it
__global__ void __launch_bounds__(TPB) k_chain_place(int n, int nt, int chains, const double *__restrict__ pos, long np,
                                                     unsigned *__restrict__ head, unsigned *__restrict__ next)
{
    const long q = (long)blockIdx.x * TPB + threadIdx.x;
    if (q >= np) return;
    const unsigned h = (unsigned)(((unsigned long long)((unsigned)q * 2654435769u) * (unsigned)chains) >> 32);
    unsigned e = 8u * (unsigned)q;
    for_tiles(cic_span(pos, q, np, n), nt, [&](int k) {
        next[e] = atomicExch(head + (unsigned)k * (unsigned)chains + h, e);
        ++e;
    });
}
template <bool ADD, bool SPLIT>
__global__ void __launch_bounds__(DNT) k_chain_tile(int n, int nt, double a, double c, double kap, CicVolume V,
                                                    const double *__restrict__ pos, const double *__restrict__ u,
                                                    double mass, const double *__restrict__ psi,
                                                    const unsigned *__restrict__ head, const unsigned *__restrict__ next,
                                                    int parts, double *__restrict__ s0, double *__restrict__ sx,
                                                    double *__restrict__ sy, double *__restrict__ sz, double *__restrict__ sm)
{
    const int b = SPLIT ? (int)blockIdx.x / parts : (int)blockIdx.x;
    unsigned e = head[(long)blockIdx.x * DNT + threadIdx.x];
    double *const out[5] = {s0, sx, sy, sz, sm};
    cic_tile<ADD, SPLIT>(b, n, nt, a, c, kap, V, pos, u, mass, psi, out, [&](auto put) {
        while (e != ~0u) {
            const unsigned q = e >> 3;
            e = next[e];
            put((long)q);
        }
    });
}

__global__ void k_fill_u32(unsigned *__restrict__ x, long N)
{
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < N) x[p] = 0;
}

// ----------------------------------------------------------------- builders

__global__ void k_shift_scale(double *__restrict__ out, const double *__restrict__ in, long N, double scale,
                              const double *__restrict__ mean)
{
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < N) out[p] = scale * (in[p] - *mean);
}

// -1/4 d_j g^j
__global__ void k_div_quarter(double *__restrict__ out, const double *__restrict__ gx,
                              const double *__restrict__ gy, const double *__restrict__ gz, int n, double inv2h)
{
    const long N = (long)n * n * n;
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    const int i = (int)(p % n), j = (int)((p / n) % n), k = (int)(p / ((long)n * n));
    out[p] = div_quarter_point(gx, gy, gz, i, j, k, n, inv2h);
}

struct A6Ptrs {
    double *c[6];
};

// A_ij and A_ijA^ij at every point
__global__ void __launch_bounds__(TPB) k_build_Aij(A6Ptrs A6, double *__restrict__ AA,
                                                   const double *__restrict__ Vx, const double *__restrict__ Vy,
                                                   const double *__restrict__ Vz, const double *__restrict__ U,
                                                   int n, double h)
{
    const long N = (long)n * n * n;
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    const int i = (int)(p % n), j = (int)((p / n) % n), k = (int)(p / ((long)n * n));
    double A[6];
    AA[p] = aij_point(Vx, Vy, Vz, U, i, j, k, n, h, A);
    for (int c = 0; c < 6; ++c) A6.c[c][p] = A[c];
}

__global__ void k_ham_rhs(double *__restrict__ f, const double *__restrict__ s0, long N, double A)
{
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < N) f[p] = A * (s0[p] - 1.0);
}

// CMC coefficient m2 and source f at every point
__global__ void k_build_cmc(double *__restrict__ m2, double *__restrict__ f, const double *__restrict__ psi,
                            const double *__restrict__ s0, const double *__restrict__ sm,
                            const double *__restrict__ AA, long N, double a, double om, double c)
{
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    cmc_point(psi[p], s0[p], sm[p], AA[p], a, om, c, m2[p], f[p]);
}

// sources of the three B^i equations at every point
__global__ void __launch_bounds__(TPB) k_shift_source(double *__restrict__ fBx, double *__restrict__ fBy,
                                                      double *__restrict__ fBz, const double *__restrict__ psi,
                                                      const double *__restrict__ xi, A6Ptrs A6, int n, double h,
                                                      double a, double c)
{
    const long N = (long)n * n * n;
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    const int i = (int)(p % n), j = (int)((p / n) % n), k = (int)(p / ((long)n * n));
    double out[3];
    shift_source_point(psi, xi, A6.c, i, j, k, n, h, a, c, out);
    fBx[p] = out[0];
    fBy[p] = out[1];
    fBz[p] = out[2];
}

// derived fields: 0 Phi = xi/chi, 1 alpha = 1 + Phi/(a^2c^2), 2 psi = a^(1/2) chi,
// 3 beta component = B + d_dir b (dir passed as which-3)
__global__ void k_derived(int which, double *__restrict__ out, const double *__restrict__ psi,
                          const double *__restrict__ xi, const double *__restrict__ Bc,
                          const double *__restrict__ b, int n, double h, double a, double c)
{
    const long N = (long)n * n * n;
    const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    const double kap = 1.0 / (2.0 * a * a * c * c);
    if (which <= 2) {
        const double chi = 1.0 - kap * psi[p];
        if (which == 0) out[p] = xi[p] / chi;
        else if (which == 1) out[p] = 1.0 + (xi[p] / chi) / (a * a * c * c);
        else out[p] = sqrt(a) * chi;
    } else {
        const int dir = which - 3;
        const int i = (int)(p % n), j = (int)((p / n) % n), k = (int)(p / ((long)n * n));
        out[p] = Bc[p] + dcen(b, dir, i, j, k, n, 1.0 / (2.0 * h));
    }
}

inline unsigned blocks_for(long count) { return (unsigned)((count + TPB - 1) / TPB); }

} // namespace

// Particles that one pass takes: as many as the lists hold in the worst case (every cloud
// over eight tiles).  Twice the cells, so that a usual run needs one pass, and 65536 on
// small grids (small: not there, so that the scratch stays below 76 bytes a cell and 2 KB).
long cic_pass(int n, bool small) { return std::min(std::max(2L * n * n * n, small ? 64L : 1L << 16), 1L << 28); }
static long cic_tiles(int n)
{
    const long nt = (n + DT - 1) / DT;
    return nt * nt * nt;
}
// tiles with long lists that are taken first
static unsigned cic_room(long nt3) { return (unsigned)std::min(1 + nt3 / 8, 4096L); }

size_t cic_bytes(int n, long pass)
{
    return sizeof(unsigned) * (size_t)(8 * pass + 3 * (cic_tiles(n) + 4) + 1 + cic_room(cic_tiles(n)));
}

// Workgroups a tile of the chains: 256 particles each, together at most 24, whose adds to memory
// (2560 each) stay below 3 us, and chain heads in at most half of the scratch.
static int cic_parts(long nt3, long np, long pass)
{
    return (int)std::max(1L, std::min({np / (256 * nt3), 24 / nt3, 4 * pass / (DNT * nt3)}));
}
// particles of a pass by chains, next to the heads of as many chains as a tile can have
static long chain_pass(long nt3, long pass) { return pass - nt3 * DNT * cic_parts(nt3, pass, pass) / 8; }
// Chains where there are few tiles, or few particles on a small grid.  Measured back to back (us;
// sort by cell or scatter of the first version / lists / chains):
//   8^3      5120 particles   24.7 / 71.7 / 15.1;  1e6   1913 / 8549 / 701
//   16^3     4096             30.3 / 36.3 / 23.0;  1e6   1638 / 1957 / 1089
//   32^3    32768             32.7 / 36.8 / 30.0;  65000  123 / 42.4 / as lists (no room for the heads)
//   64^3    65000             39.0 / 33.9 / 29.8;  1e6   1728 /  150 / as lists
// Lists from 24^3 and 65536 particles on: 24^3 130000 123 / 150, and their heads cost a pass
// over 4096 tiles at 128^3.
constexpr long kChainFewTiles = 8, kChainTiles = 512, kChainMax = 1L << 16;
static bool chains_ok(long nt3, long np, long pass)
{
    return 4 * pass >= nt3 * DNT &&
           (nt3 <= kChainFewTiles || (nt3 <= kChainTiles && np <= std::min(kChainMax, chain_pass(nt3, pass))));
}

// A table with a counter per tile up to 32768 of them (256^3, 128 KB of LDS), a hash table
// beyond.  8192 particles a workgroup from 2^20 on, so that few workgroups count into the
// same tile, 2048 below, so that the chip has enough workgroups.
template <bool PLACE>
static void cic_bin(hipStream_t s, int n, int nt, const double *pos, long np, unsigned *at, unsigned *list)
{
    if (np <= 0) return;
    const long nt3 = cic_tiles(n);
    auto run = [&](auto k, int per_thread) {
        k<<<(unsigned)((np + BNT * per_thread - 1) / (BNT * per_thread)), BNT, 0, s>>>(n, nt, pos, np, at, list);
    };
    if (nt3 <= 8192 && np < (1L << 20)) run(k_cic_bin<PLACE, false, 8192, 2>, 2);
    else if (nt3 <= 8192) run(k_cic_bin<PLACE, false, 8192, 8>, 8);
    else if (nt3 <= 32768) run(k_cic_bin<PLACE, false, 32768, 8>, 8);
    else run(k_cic_bin<PLACE, true, BHASH, 8>, 8);
}

void launch_cic_deposit(hipStream_t s, int n, double a, double c_tilde, const double *pos, const double *u,
                        double mass, long np, const double *psi, void *scratch, long pass, double *s0, double *sx,
                        double *sy, double *sz, double *sm)
{
    const double kap = 1.0 / (2.0 * a * a * c_tilde * c_tilde), h = 1.0 / n, vol = c_tilde * (h * h * h);
    const CicVolume V{vol, 1.0 / vol};
    const int nt = (n + DT - 1) / DT;
    const long nt3 = cic_tiles(n);
    const long row = (nt3 + 4) / 4 * 4; // nt3 + 1 at least
    const unsigned room = cic_room(nt3);
    unsigned *list = static_cast<unsigned *>(scratch), *cnt = list + 8 * pass, *next = cnt + row, *start = next + row,
             *heavy = start + row;
    if (chains_ok(nt3, np, pass)) {
        const long most = std::max(1L, std::min(np, chain_pass(nt3, pass))); // no particle: one round too
        for (long q = 0; q == 0 || q < np; q += most) {
            const long m = std::min(most, np - q);
            const double *x = m > 0 ? pos + 3 * q : nullptr, *v = m > 0 ? u + 3 * q : nullptr;
            const int parts = cic_parts(nt3, m, pass);
            const long nh = nt3 * DNT * parts, zero = q == 0 && parts > 1 ? (long)n * n * n : 0;
            unsigned *head = list + 8 * m;
            k_chain_begin<<<blocks_for(std::max(nh, zero)), TPB, 0, s>>>(head, nh, zero, s0, sx, sy, sz, sm);
            if (m > 0) k_chain_place<<<blocks_for(m), TPB, 0, s>>>(n, nt, DNT * parts, x, m, head, list);
            auto tile = [&](auto k) {
                k<<<(unsigned)(nt3 * parts), DNT, 0, s>>>(n, nt, a, c_tilde, kap, V, x, v, mass, psi, head, list, parts, s0, sx,
                                                          sy, sz, sm);
            };
            if (parts > 1) tile(k_chain_tile<false, true>);
            else if (q == 0) tile(k_chain_tile<false, false>);
            else tile(k_chain_tile<true, false>);
        }
        return;
    }
    for (long q = 0; q == 0 || q < np; q += pass) {
        const long m = std::min(pass, np - q);
        const double *x = m > 0 ? pos + 3 * q : nullptr, *v = m > 0 ? u + 3 * q : nullptr;
        k_fill_u32<<<blocks_for(nt3), TPB, 0, s>>>(cnt, nt3);
        cic_bin<false>(s, n, nt, x, m, cnt, nullptr);
        k_cic_scan<<<1, SCNT, 0, s>>>(cnt, (int)nt3, start, next, heavy, room);
        cic_bin<true>(s, n, nt, x, m, next, list);
        if (q == 0)
            k_cic_tile<false><<<(unsigned)nt3 + room, DNT, 0, s>>>(n, nt, a, c_tilde, kap, V, x, v, mass, psi, start, list, cnt, heavy, (int)room, s0, sx,
                                                            sy, sz, sm);
        else
            k_cic_tile<true><<<(unsigned)nt3 + room, DNT, 0, s>>>(n, nt, a, c_tilde, kap, V, x, v, mass, psi, start, list, cnt, heavy, (int)room, s0, sx,
                                                           sy, sz, sm);
    }
}

void launch_shift_scale(hipStream_t s, double *out, const double *in, long N, double scale, const double *mean)
{
    k_shift_scale<<<blocks_for(N), TPB, 0, s>>>(out, in, N, scale, mean);
}

void launch_div_quarter(hipStream_t s, double *out, const double *gx, const double *gy, const double *gz, int n,
                        double h)
{
    k_div_quarter<<<blocks_for((long)n * n * n), TPB, 0, s>>>(out, gx, gy, gz, n, 1.0 / (2.0 * h));
}

void launch_build_Aij(hipStream_t s, double *const A6[6], double *AA, const double *Vx, const double *Vy,
                      const double *Vz, const double *U, int n, double h)
{
    A6Ptrs P;
    for (int c = 0; c < 6; ++c) P.c[c] = A6[c];
    k_build_Aij<<<blocks_for((long)n * n * n), TPB, 0, s>>>(P, AA, Vx, Vy, Vz, U, n, h);
}

void launch_ham_rhs(hipStream_t s, double *f, const double *s0, long N, double A)
{
    k_ham_rhs<<<blocks_for(N), TPB, 0, s>>>(f, s0, N, A);
}

void launch_build_cmc(hipStream_t s, double *m2, double *f, const double *psi, const double *s0, const double *sm,
                      const double *AA, long N, double a, double om, double c_tilde)
{
    k_build_cmc<<<blocks_for(N), TPB, 0, s>>>(m2, f, psi, s0, sm, AA, N, a, om, c_tilde);
}

void launch_shift_source(hipStream_t s, double *fB[3], const double *psi, const double *xi, double *const A6[6],
                         int n, double h, double a, double c_tilde)
{
    A6Ptrs P;
    for (int c = 0; c < 6; ++c) P.c[c] = A6[c];
    k_shift_source<<<blocks_for((long)n * n * n), TPB, 0, s>>>(fB[0], fB[1], fB[2], psi, xi, P, n, h, a, c_tilde);
}

void launch_derived(hipStream_t s, int which, double *out, const double *psi, const double *xi, const double *Bc,
                    const double *b, int n, double h, double a, double c_tilde)
{
    k_derived<<<blocks_for((long)n * n * n), TPB, 0, s>>>(which, out, psi, xi, Bc, b, n, h, a, c_tilde);
}

} // namespace grmg
