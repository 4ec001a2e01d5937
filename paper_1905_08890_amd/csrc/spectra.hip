// Vector-mode extraction (paper sec. 6.2): the shift beta^i -- likewise B^i
// and the momentum density s_i -- carries a scalar and a vector mode; the
// discrete curl removes the scalar one, and k^2 P_V(k) = P_curl(k) gives the
// vector mode's power.  Spectra are binned in |k| shells up to a quarter of
// the Nyquist wave number.
//
// Steps, all on the device:
//   1. curl and divergence by 3-point central differences, packed as two
//      complex fields z1 = curl_x + i curl_y, z2 = curl_z + i div (two real
//      transforms for the price of one complex transform each), formed by the
//      first transform pass as it reads the three input fields;
//   2. 3-D FFT of z1 and z2, one pass per axis, each pass keeping only the modes
//      |m_i| <= nbins that a shell can hold;
//   3. per mode of the cube |m_i| <= nbins: separate the four transforms with
//      F[a](m) = (Z(m) + conj Z(-m)) / 2, F[b](m) = (Z(m) - conj Z(-m)) / (2i),
//      form the curl and divergence power and their ratio to |k_eff|^2, and
//      add them to the mode's shell in a fixed order (per shell and plane m_z, then
//      over the planes).
// gr_spectra_fft, the whole transform of a caller's array, moves line bundles
// through LDS with radix-2 stages.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <new>
#include <string>

#include <hip/hip_runtime.h>

#include "gr.h"

namespace {

constexpr int TPB = 256;
constexpr int kFftLds = 4096;  // complex doubles of line data per workgroup (64 KiB)
constexpr int kMaxN = 1024;    // twiddle table in LDS: n / 2 entries
constexpr int kRows = 6;       // k, count, P_curl, P_div, P_vector, P_scalar

__device__ __forceinline__ int wrapi(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// tw[j] = exp(-2 pi i j / n), j < n / 2
__global__ void k_twiddles(double2 *__restrict__ tw, int n)
{
    const int j = blockIdx.x * TPB + threadIdx.x;
    if (j >= n / 2) return;
    double s, c;
    sincospi(-2.0 * j / n, &s, &c);
    tw[j] = double2{c, s};
}

// In-place forward transform of every line along AXIS (0 = x, 1 = y, 2 = z)
// of an n^3 complex array; a workgroup takes lb lines (lb * n <= kFftLds).
template <int AXIS>
__global__ void __launch_bounds__(TPB) k_fft_lines(double2 *__restrict__ data, int n, int logn, int loglb,
                                                   const double2 *__restrict__ tw)
{
    __shared__ double2 s[kFftLds];
    __shared__ double2 stw[kMaxN / 2];
    const int tid = threadIdx.x;
    const int lb = 1 << loglb, half = n >> 1, tot = lb << logn;
    for (int j = tid; j < half; j += TPB) stw[j] = tw[j];
    const long n2 = (long)n * n;
    long base, lstride, jstride;
    if (AXIS == 0) {
        base = (long)blockIdx.x * tot;
        lstride = n;
        jstride = 1;
    } else {
        const int nxb = n >> loglb;
        const long x0 = (long)(blockIdx.x % nxb) << loglb, other = blockIdx.x / nxb;
        base = AXIS == 1 ? other * n2 + x0 : other * n + x0;
        lstride = 1;
        jstride = AXIS == 1 ? n : n2;
    }
    const int shift = 32 - logn;
    for (int idx = tid; idx < tot; idx += TPB) {
        const int l = AXIS == 0 ? idx >> logn : idx & (lb - 1);
        const int j = AXIS == 0 ? idx & (n - 1) : idx >> loglb;
        s[(l << logn) + (int)(__brev((unsigned)j) >> shift)] = data[base + l * lstride + j * jstride];
    }
    __syncthreads();
    // radix-2 stages in pairs (one LDS round trip and barrier per pair): the
    // same butterflies and twiddles as stage after stage; an odd first stage alone
    int ls = 0;
    if (logn & 1) {
        for (int bi = tid; bi < (tot >> 1); bi += TPB) {
            const int l = bi >> (logn - 1), t = bi & (half - 1);
            const int i0 = (l << logn) + (t << 1), i1 = i0 + 1;
            const double2 a = s[i0], c = s[i1]; // twiddle 1
            s[i0] = double2{a.x + c.x, a.y + c.y};
            s[i1] = double2{a.x - c.x, a.y - c.y};
        }
        __syncthreads();
        ls = 1;
    }
    for (; ls < logn; ls += 2) {
        const int hs = 1 << ls, t1 = logn - 1 - ls, t2 = logn - 2 - ls;
        for (int gi = tid; gi < (tot >> 2); gi += TPB) {
            const int l = gi >> (logn - 2), t = gi & ((n >> 2) - 1);
            const int k = t & (hs - 1), grp = t >> ls;
            const int i0 = (l << logn) + (grp << (ls + 2)) + k;
            const double2 a0 = s[i0], a1 = s[i0 + hs], a2 = s[i0 + 2 * hs], a3 = s[i0 + 3 * hs];
            const double2 w1 = stw[k << t1];
            const double b1x = a1.x * w1.x - a1.y * w1.y, b1y = a1.x * w1.y + a1.y * w1.x;
            const double b3x = a3.x * w1.x - a3.y * w1.y, b3y = a3.x * w1.y + a3.y * w1.x;
            const double2 c0{a0.x + b1x, a0.y + b1y}, c1{a0.x - b1x, a0.y - b1y};
            const double2 c2{a2.x + b3x, a2.y + b3y}, c3{a2.x - b3x, a2.y - b3y};
            const double2 w2 = stw[k << t2], w3 = stw[(k + hs) << t2];
            const double d2x = c2.x * w2.x - c2.y * w2.y, d2y = c2.x * w2.y + c2.y * w2.x;
            const double d3x = c3.x * w3.x - c3.y * w3.y, d3y = c3.x * w3.y + c3.y * w3.x;
            s[i0] = double2{c0.x + d2x, c0.y + d2y};
            s[i0 + 2 * hs] = double2{c0.x - d2x, c0.y - d2y};
            s[i0 + hs] = double2{c1.x + d3x, c1.y + d3y};
            s[i0 + 3 * hs] = double2{c1.x - d3x, c1.y - d3y};
        }
        __syncthreads();
    }
    for (int idx = tid; idx < tot; idx += TPB) {
        const int l = AXIS == 0 ? idx >> logn : idx & (lb - 1);
        const int j = AXIS == 0 ? idx & (n - 1) : idx >> loglb;
        data[base + l * lstride + j * jstride] = s[(l << logn) + j];
    }
}

// ---- the pruned transform of the two packed fields ----
//
// Only the modes |m_i| <= R (R = nbins <= n / 4) reach a shell, so every axis
// pass keeps S = 2 R + 1 of its n outputs: the y pass then transforms S / n and
// the z pass (S / n)^2 of the lines of a full transform, and no pass writes what
// is not read.  Each pass writes its kept modes with the next axis fastest
// (x pass [a][z][sx][y], y pass [a][sx][sy][z], z pass [a][sz][sx][sy], a = the
// array z1 or z2, s = m + R), so every pass reads contiguous lines.
//
// A line of n = R1 R2 points (R1 = R2 or 2 R2) is transformed in two rounds by R2
// threads: R1-point transforms in registers over x = R2 j1 + j2, a twiddle, one
// exchange through LDS, R2-point transforms, mode k1 + R1 k2.  One LDS round trip
// per point instead of one per two radix-2 stages: the LDS traffic of a pass falls
// from ~210 to ~50 bytes per point.  At 256^3 with 32 shells one field's
// extraction took 1.43 ms with full transforms of separately written curls (curl
// 297 us, six passes of 150-176 us, serial shell sums 165 us) and takes 0.34 ms
// here: x pass 252 us (bound by the L2: 18 neighbour reads a cell), y 36 us, z 13 us,
// shells 29 us.
template <int LOGN> struct FftSplit {
    static constexpr int N = 1 << LOGN, R1 = 1 << ((LOGN + 1) / 2), R2 = 1 << (LOGN / 2);
    static constexpr int LINES = TPB / R2, PITCH = LINES + 1; // lines per workgroup; LDS pitch in points
};

__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return double2{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}

// In-register R-point transform, decimation in frequency; v[i] ends as mode
// bitrev(i).  w[j] = exp(-2 pi i j / n), n the table's length of the whole line.
template <int R, int N> __device__ __forceinline__ void fft_reg(double2 (&v)[R], const double2 *__restrict__ w)
{
#pragma unroll
    for (int len = R; len > 1; len >>= 1)
#pragma unroll
        for (int b = 0; b < R; b += len)
#pragma unroll
            for (int i = 0; i < len / 2; ++i) {
                const double2 p = v[b + i], q = v[b + i + len / 2];
                v[b + i] = double2{p.x + q.x, p.y + q.y};
                const double2 d{p.x - q.x, p.y - q.y};
                if (i == 0) v[b + i + len / 2] = d;
                else if (4 * i == len) v[b + i + len / 2] = double2{d.y, -d.x}; // times -i
                else v[b + i + len / 2] = cmul(d, w[i * (N / len)]);
            }
}
template <int R> __device__ __forceinline__ constexpr int bitrev(int i)
{
    int r = 0;
    for (int b = 1; b < R; b <<= 1) r = 2 * r + ((i / b) & 1);
    return r;
}

struct Fields {
    const double *vx, *vy, *vz;
};

// Points R2 j + j2 (j < R1) of row (y, z) of array A by 3-point central
// differences: A = 0 curl_x + i curl_y, A = 1 curl_z + i div.  Row pointers and
// compile-time offsets; only the first and the last x neighbour can wrap.
template <int A, int R1, int R2>
__device__ __forceinline__ void curl_row(const Fields &F, int y, int z, int j2, double2 (&v)[R1])
{
    constexpr int N = R1 * R2;
    const double f = 0.5 * N;
    auto row = [&](const double *p, int yy, int zz) { return p + ((long)zz * N + yy) * N + j2; };
    const int yp = wrapi(y + 1, N), ym = wrapi(y - 1, N), zp = wrapi(z + 1, N), zm = wrapi(z - 1, N);
    const int first = j2 == 0 ? N - 1 : -1;                 // x - 1 of j = 0, from the row's j2
    const int last = j2 == R2 - 1 ? 1 - N : 1;              // x + 1 of j = R1 - 1, from its x
    auto dx = [&](const double *p, int j) {
        return (p[R2 * j + (j == R1 - 1 ? last : 1)] - p[R2 * j + (j == 0 ? first : -1)]) * f;
    };
    if constexpr (A == 0) {
        const double *zyp = row(F.vz, yp, z), *zym = row(F.vz, ym, z), *yzp = row(F.vy, y, zp);
        const double *yzm = row(F.vy, y, zm), *xzp = row(F.vx, y, zp), *xzm = row(F.vx, y, zm);
        const double *zc = row(F.vz, y, z);
#pragma unroll
        for (int j = 0; j < R1; ++j) {
            const double dyvz = (zyp[R2 * j] - zym[R2 * j]) * f, dzvy = (yzp[R2 * j] - yzm[R2 * j]) * f;
            const double dzvx = (xzp[R2 * j] - xzm[R2 * j]) * f, dxvz = dx(zc, j);
            v[j] = double2{dyvz - dzvy, dzvx - dxvz};
        }
    } else {
        const double *xyp = row(F.vx, yp, z), *xym = row(F.vx, ym, z), *yyp = row(F.vy, yp, z);
        const double *yym = row(F.vy, ym, z), *zzp = row(F.vz, y, zp), *zzm = row(F.vz, y, zm);
        const double *xc = row(F.vx, y, z), *yc = row(F.vy, y, z);
#pragma unroll
        for (int j = 0; j < R1; ++j) {
            const double dxvy = dx(yc, j), dyvx = (xyp[R2 * j] - xym[R2 * j]) * f;
            const double dxvx = dx(xc, j), dyvy = (yyp[R2 * j] - yym[R2 * j]) * f;
            const double dzvz = (zzp[R2 * j] - zzm[R2 * j]) * f;
            v[j] = double2{dxvy - dyvx, dxvx + dyvy + dzvz};
        }
    }
}

// One pass over lines [0, nlines) of the array a = blockIdx.x % 2 of a pair (the
// two workgroups of one group of lines run side by side: they read the same rows
// of v).  AXIS 0 forms its input from the fields; the others read `in`, a line's n
// points contiguous.
//   AXIS 0: line r = z n + y           -> out[a][z][s][y]
//   AXIS 1: line r = s n + z           (in [a][z][s][:])       -> out[a][s][sy][z]
//   AXIS 2: line r = sx S + sy         (in [a][r][:])          -> out[a][sz][r]
template <int LOGN, int AXIS>
__global__ void __launch_bounds__(TPB, LOGN <= 8 ? 2 : 1) k_fft_pruned(Fields src, const double2 *__restrict__ in,
                                                                       double2 *__restrict__ out, long nlines, int R,
                                                                       const double2 *__restrict__ tw)
{
    using F = FftSplit<LOGN>;
    constexpr int N = F::N, R1 = F::R1, R2 = F::R2, LINES = F::LINES, PITCH = F::PITCH, PER = R1 / R2;
    __shared__ double2 s[N * PITCH];
    const int S = 2 * R + 1;
    // contiguous runs of lines per XCD: the rows that neighbouring groups share stay in one L2
    const unsigned G = gridDim.x;
    const unsigned w = G % 8 == 0 ? (blockIdx.x & 7) * (G >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    const int a = w & 1;
    const long line0 = (long)(w >> 1) * LINES;
    const int j2 = threadIdx.x % R2, la = threadIdx.x / R2;          // round 1: consecutive threads along the line
    const int lb = threadIdx.x % LINES, kq = threadIdx.x / LINES;    // round 2: consecutive threads across lines
    const long ra = line0 + la, rb = line0 + lb;
    if (ra < nlines) {
        double2 v[R1];
        if constexpr (AXIS == 0) {
            const int y = (int)(ra % N), z = (int)(ra / N);
            if (a == 0) curl_row<0, R1, R2>(src, y, z, j2, v);
            else curl_row<1, R1, R2>(src, y, z, j2, v);
        } else {
            const long row = AXIS == 1 ? (a * (long)N + ra % N) * S + ra / N : a * (long)S * S + ra;
            const double2 *p = in + row * N + j2;
#pragma unroll
            for (int j = 0; j < R1; ++j) v[j] = p[R2 * j];
        }
        fft_reg<R1, N>(v, tw);
#pragma unroll
        for (int i = 0; i < R1; ++i) {
            const int k1 = bitrev<R1>(i), e = j2 * k1; // e < N
            double2 t = tw[e & (N / 2 - 1)];
            if (e >= N / 2) t = double2{-t.x, -t.y};
            s[(k1 * R2 + j2) * PITCH + la] = cmul(v[i], t);
        }
    }
    __syncthreads();
    if (rb < nlines) {
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const int k1 = kq + p * R2;
            double2 u[R2];
#pragma unroll
            for (int j = 0; j < R2; ++j) u[j] = s[(k1 * R2 + j) * PITCH + lb];
            fft_reg<R2, N>(u, tw);
#pragma unroll
            for (int i = 0; i < R2; ++i) {
                const int k = k1 + R1 * bitrev<R2>(i);
                const int m = k <= R ? k + R : k - N + R; // kept: 0 .. R and N - R .. N - 1
                if (k > R && m < 0) continue;
                long o;
                if (AXIS == 0) o = ((a * (long)N + rb / N) * S + m) * N + rb % N;
                else if (AXIS == 1) o = ((a * (long)S + rb / N) * S + m) * N + rb % N;
                else o = (a * (long)S + m) * S * S + rb;
                out[o] = u[i];
            }
        }
    }
}

// Fixed-order sum over a workgroup (wavefront shuffles, then the waves in order).
__device__ __forceinline__ double block_sum(double v, double *sh)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    for (int w = 0; w < TPB / 64; ++w) t += sh[w];
    __syncthreads();
    return t;
}

// Sums of shell b's modes in the plane mz (blockIdx = (mz + R, b)): thread my (and
// my + 256, ...) runs over the mx of its ring, so a mode is visited once and the
// order of every addition is fixed.  part[b][plane][row].
__global__ void __launch_bounds__(TPB) k_bin_modes(const double2 *__restrict__ cube, int n, int nbins,
                                                   double *__restrict__ part)
{
    __shared__ double sh[TPB / 64];
    const int R = nbins, S = 2 * R + 1, b = blockIdx.y, mz = (int)blockIdx.x - R;
    const double N = (double)n * n * n, invN2 = 1.0 / (N * N), twopi = 6.283185307179586476925286766559;
    const double2 *z1 = cube, *z2 = cube + (long)S * S * S;
    double v[kRows] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    double sx, sy, sz, cc;
    sincospi(2.0 * mz / n, &sz, &cc);
    for (int q = threadIdx.x; q < S; q += TPB) {
        const int my = q - R;
        // |m| in [b + 1/2, b + 3/2): |mx| between these, one to spare on either side
        const double lo = (b + 0.5) * (b + 0.5) - (double)(mz * mz + my * my);
        const double hi = (b + 1.5) * (b + 1.5) - (double)(mz * mz + my * my);
        if (hi < 0.0) continue;
        const int x0 = lo > 1.0 ? (int)sqrt(lo) - 1 : 0;
        int x1 = (int)sqrt(hi) + 1;
        x1 = x1 > R ? R : x1;
        sincospi(2.0 * my / n, &sy, &cc);
        for (int ax = x0; ax <= x1; ++ax)
            for (int sg = 0; sg < (ax ? 2 : 1); ++sg) {
                const int mx = sg ? -ax : ax;
                const double mag = sqrt((double)(mx * mx + my * my + mz * mz));
                if ((int)floor(mag + 0.5) - 1 != b) continue;
                const long ip = ((long)(mz + R) * S + mx + R) * S + my + R;
                const long im = ((long)(R - mz) * S + R - mx) * S + R - my;
                const double2 ap = z1[ip], am = z1[im], bp = z2[ip], bm = z2[im];
                // F[curl_x] = (ap + conj am) / 2, F[curl_y] = (ap - conj am) / (2i), likewise curl_z, div from z2
                const double fxr = 0.5 * (ap.x + am.x), fxi = 0.5 * (ap.y - am.y);
                const double fyr = 0.5 * (ap.y + am.y), fyi = -0.5 * (ap.x - am.x);
                const double fzr = 0.5 * (bp.x + bm.x), fzi = 0.5 * (bp.y - bm.y);
                const double fdr = 0.5 * (bp.y + bm.y), fdi = -0.5 * (bp.x - bm.x);
                const double pc = ((fxr * fxr + fxi * fxi) + (fyr * fyr + fyi * fyi) + (fzr * fzr + fzi * fzi)) * invN2;
                const double pd = (fdr * fdr + fdi * fdi) * invN2;
                sincospi(2.0 * mx / n, &sx, &cc);
                const double keff2 = (n * sx) * (n * sx) + (n * sy) * (n * sy) + (n * sz) * (n * sz);
                v[0] += twopi * mag;
                v[1] += 1.0;
                v[2] += pc;
                v[3] += pd;
                v[4] += pc / keff2;
                v[5] += pd / keff2;
            }
    }
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const double t = block_sum(v[r], sh);
        if (threadIdx.x == 0) part[((long)b * S + blockIdx.x) * kRows + r] = t;
    }
}

// out[row][bin] = sum over the planes (thread t adds planes t, t + 256, ..., then
// a fixed tree); one workgroup per bin
__global__ void __launch_bounds__(TPB) k_bin_reduce(const double *__restrict__ part, int nbins, int S,
                                                    double *__restrict__ out)
{
    __shared__ double sh[TPB / 64];
    const int b = blockIdx.x;
    for (int r = 0; r < kRows; ++r) {
        double v = 0.0;
        for (int p = threadIdx.x; p < S; p += TPB) v += part[((long)b * S + p) * kRows + r];
        v = block_sum(v, sh);
        if (threadIdx.x == 0) out[r * nbins + b] = v;
    }
}

thread_local std::string s_err;
int sfail(int code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
int sfail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    s_err = buf;
    return code;
}
#define SHIP(expr)                                                                                    \
    do {                                                                                              \
        hipError_t e_ = (expr);                                                                       \
        if (e_ != hipSuccess) return sfail(GR_EDEVICE, "%s: %s", #expr, hipGetErrorString(e_));       \
    } while (0)
#define SLAUNCH() SHIP(hipGetLastError())

size_t al256(size_t b) { return (b + 255) / 256 * 256; }

int ilog2(int v)
{
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
}

} // namespace

struct gr_spectra_s {
    int n = 0, logn = 0, nbins = 0;
    size_t off_a = 0, off_b = 0, off_tw = 0, off_out = 0, bytes = 0;
    char *ws = nullptr;
    hipStream_t stream = nullptr;
    bool bound = false;
};

namespace {

int fft3(gr_spectra S, double2 *d)
{
    const int n = S->n, logn = S->logn;
    const int lb = n < kFftLds / n ? n : kFftLds / n, loglb = ilog2(lb);
    const unsigned grid = (unsigned)((long)n * n / lb);
    const double2 *tw = reinterpret_cast<const double2 *>(S->ws + S->off_tw);
    k_fft_lines<0><<<grid, TPB, 0, S->stream>>>(d, n, logn, loglb, tw);
    k_fft_lines<1><<<grid, TPB, 0, S->stream>>>(d, n, logn, loglb, tw);
    k_fft_lines<2><<<grid, TPB, 0, S->stream>>>(d, n, logn, loglb, tw);
    SLAUNCH();
    return GR_OK;
}

// the three pruned passes: fields -> a [2][z][S][y] -> b [2][S][S][z] -> a [2][S][S][S]
template <int LOGN>
void pruned_passes(hipStream_t st, const Fields &src, double2 *a, double2 *b, int R, const double2 *tw)
{
    constexpr int LINES = FftSplit<LOGN>::LINES;
    const long n = 1 << LOGN, S = 2L * R + 1;
    auto grid = [](long lines) { return (unsigned)(2 * ((lines + LINES - 1) / LINES)); };
    k_fft_pruned<LOGN, 0><<<grid(n * n), TPB, 0, st>>>(src, nullptr, a, n * n, R, tw);
    k_fft_pruned<LOGN, 1><<<grid(n * S), TPB, 0, st>>>(src, a, b, n * S, R, tw);
    k_fft_pruned<LOGN, 2><<<grid(S * S), TPB, 0, st>>>(src, b, a, S * S, R, tw);
}

} // namespace

extern "C" {

const char *gr_spectra_last_error(void) { return s_err.c_str(); }

int gr_create_spectra(int n, int nbins, gr_spectra *out)
{
    if (!out) return sfail(GR_EINVAL, "null argument");
    *out = nullptr;
    if (n < 8 || n > kMaxN || (n & (n - 1))) return sfail(GR_EINVAL, "n = %d must be a power of two in [8, %d]", n, kMaxN);
    if (nbins < 1 || nbins > n / 4) return sfail(GR_EINVAL, "nbins = %d must be in [1, n/4 = %d]", nbins, n / 4);
    gr_spectra S = new (std::nothrow) gr_spectra_s;
    if (!S) return sfail(GR_EDEVICE, "out of host memory");
    S->n = n;
    S->logn = ilog2(n);
    S->nbins = nbins;
    const size_t side = 2 * (size_t)nbins + 1;
    size_t off = 0;
    S->off_a = off; // x pass output, then the mode cube
    off += al256(2 * (size_t)n * n * side * sizeof(double2));
    S->off_b = off; // y pass output, then (the z pass has read it) the shells' partial sums
    off += std::max(al256(2 * (size_t)n * side * side * sizeof(double2)), al256(side * kRows * nbins * sizeof(double)));
    off = std::max(off, 2 * al256((size_t)n * n * n * sizeof(double2))); // the size callers have always been told
    S->off_tw = off;
    off += al256((size_t)(n / 2) * sizeof(double2));
    S->off_out = off;
    off += al256((size_t)kRows * nbins * sizeof(double));
    S->bytes = off;
    *out = S;
    return GR_OK;
}

int gr_spectra_workspace_bytes(gr_spectra S, size_t *bytes)
{
    if (!S || !bytes) return sfail(GR_EINVAL, "null argument");
    *bytes = S->bytes;
    return GR_OK;
}

int gr_spectra_bind(gr_spectra S, void *d_ws, size_t bytes, void *stream)
{
    if (!S || !d_ws) return sfail(GR_EINVAL, "null argument");
    if (bytes < S->bytes) return sfail(GR_EINVAL, "workspace %zu bytes < required %zu", bytes, S->bytes);
    if (reinterpret_cast<uintptr_t>(d_ws) % 256) return sfail(GR_EINVAL, "workspace not 256-byte aligned");
    S->ws = reinterpret_cast<char *>(d_ws);
    S->stream = reinterpret_cast<hipStream_t>(stream);
    k_twiddles<<<(unsigned)((S->n / 2 + TPB - 1) / TPB), TPB, 0, S->stream>>>(
        reinterpret_cast<double2 *>(S->ws + S->off_tw), S->n);
    SLAUNCH();
    S->bound = true;
    return GR_OK;
}

int gr_spectra_fft(gr_spectra S, double *d_data)
{
    if (!S || !d_data) return sfail(GR_EINVAL, "null argument");
    if (!S->bound) return sfail(GR_ESTATE, "spectra handle not bound");
    if (reinterpret_cast<uintptr_t>(d_data) % 16) return sfail(GR_EINVAL, "data not 16-byte aligned");
    return fft3(S, reinterpret_cast<double2 *>(d_data));
}

int gr_vector_spectra(gr_spectra S, const double *d_vx, const double *d_vy, const double *d_vz, double *h_out)
{
    if (!S || !d_vx || !d_vy || !d_vz || !h_out) return sfail(GR_EINVAL, "null argument");
    if (!S->bound) return sfail(GR_ESTATE, "spectra handle not bound");
    const int n = S->n, nb = S->nbins, side = 2 * nb + 1, cells = kRows * nb;
    double2 *bufa = reinterpret_cast<double2 *>(S->ws + S->off_a);
    double2 *bufb = reinterpret_cast<double2 *>(S->ws + S->off_b);
    const double2 *tw = reinterpret_cast<const double2 *>(S->ws + S->off_tw);
    double *part = reinterpret_cast<double *>(S->ws + S->off_b);
    double *out = reinterpret_cast<double *>(S->ws + S->off_out);
    const Fields src{d_vx, d_vy, d_vz};
    switch (S->logn) {
    case 3: pruned_passes<3>(S->stream, src, bufa, bufb, nb, tw); break;
    case 4: pruned_passes<4>(S->stream, src, bufa, bufb, nb, tw); break;
    case 5: pruned_passes<5>(S->stream, src, bufa, bufb, nb, tw); break;
    case 6: pruned_passes<6>(S->stream, src, bufa, bufb, nb, tw); break;
    case 7: pruned_passes<7>(S->stream, src, bufa, bufb, nb, tw); break;
    case 8: pruned_passes<8>(S->stream, src, bufa, bufb, nb, tw); break;
    case 9: pruned_passes<9>(S->stream, src, bufa, bufb, nb, tw); break;
    default: pruned_passes<10>(S->stream, src, bufa, bufb, nb, tw); break;
    }
    SLAUNCH();
    k_bin_modes<<<dim3((unsigned)side, (unsigned)nb), TPB, 0, S->stream>>>(bufa, n, nb, part);
    k_bin_reduce<<<(unsigned)nb, TPB, 0, S->stream>>>(part, nb, side, out);
    SLAUNCH();
    SHIP(hipMemcpyAsync(h_out, out, (size_t)cells * sizeof(double), hipMemcpyDeviceToHost, S->stream));
    SHIP(hipStreamSynchronize(S->stream));
    // sums -> means over each shell's modes
    for (int b = 0; b < nb; ++b) {
        const double c = h_out[nb + b];
        if (c > 0)
            for (int r = 0; r < kRows; ++r)
                if (r != 1) h_out[r * nb + b] /= c;
    }
    return GR_OK;
}

int gr_destroy_spectra(gr_spectra S)
{
    delete S;
    return GR_OK;
}

} // extern "C"
