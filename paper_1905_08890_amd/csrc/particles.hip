// Particle evolution with the solved metric (paper sec. 4.4, and the leapfrog
// of the appendix on time evolution): the kick, split into five ordered
// substeps over the force contributions, and the drift with the coordinate
// velocity.  One thread per particle; the metric quantities at a particle are
// the cloud-in-cell interpolation (the deposit's cell-centred weights and
// periodic wrap) of the grid values and of their 3-point central-difference
// gradients, evaluated at the eight cloud corners from the grid arrays.
#include <cmath>

#include "gr_internal.h"

namespace grmg {
namespace {

constexpr int TPB = 256;

__device__ __forceinline__ int wrapc(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// The metric at the grid points, packed for the gathers: {Phi, Psi}, {beta^x,
// beta^y} and beta^z, so a point costs two 16-byte loads and one 8-byte load.
struct Metric {
    const double2 *pp, *bxy;
    const double *bz;
    int n;
    double inv2h;
};

// One thread per grid point: Phi = xi / chi and beta^i = B^i + d_i b (one pass of
// 0.26 ms at 256^3, 5.9 TB/s, instead of four of 0.08 ms that left five arrays).
__global__ void __launch_bounds__(TPB) k_pack_metric(double2 *__restrict__ pp, double2 *__restrict__ bxy,
                                                     double *__restrict__ bz, const double *__restrict__ psi,
                                                     const double *__restrict__ xi, const double *__restrict__ Bx,
                                                     const double *__restrict__ By, const double *__restrict__ Bz,
                                                     const double *__restrict__ b, int n, double kap, double inv2h)
{
    const int x = blockIdx.x * blockDim.x + threadIdx.x, y = blockIdx.y * blockDim.y + threadIdx.y, z = blockIdx.z;
    if (x >= n || y >= n) return;
    const long plane = (long)n * n, row = z * plane + (long)y * n, p = row + x;
    const double ps = psi[p];
    pp[p] = double2{xi[p] / (1.0 - kap * ps), ps};
    const double dx = (b[row + wrapc(x + 1, n)] - b[row + wrapc(x - 1, n)]) * inv2h;
    const double dy = (b[z * plane + (long)wrapc(y + 1, n) * n + x] - b[z * plane + (long)wrapc(y - 1, n) * n + x]) * inv2h;
    const double dz = (b[wrapc(z + 1, n) * plane + (long)y * n + x] - b[wrapc(z - 1, n) * plane + (long)y * n + x]) * inv2h;
    bxy[p] = double2{Bx[p] + dx, By[p] + dy};
    bz[p] = Bz[p] + dz;
}

// The cloud of a particle along one axis: the wrapped indices of the cells
// i0 - 1 .. i0 + 2 (the cloud's corners are 1 and 2) and the corners' weights.  The
// interpolated central difference, (f(c + 1) - f(c - 1)) summed over the corners c,
// weights the four cells by -w0, -w1, w0, w1.
struct Axis {
    int i[4];
    double w[2];
    __device__ __forceinline__ Axis(double x, int n)
    {
        const double g = x * (double)n - 0.5;
        const double fl = floor(g);
        const double t = g - fl;
        i[1] = wrapc((int)fl, n);
        i[0] = wrapc(i[1] - 1, n);
        i[2] = wrapc((int)fl + 1, n);
        i[3] = wrapc(i[2] + 1, n);
        w[0] = 1.0 - t;
        w[1] = t;
    }
};

// Visits the 32 cells that the interpolated values and central differences of a
// particle touch: the 8 cloud corners as corner(p, w, wx, wy, wz), the weights
// of the value and of the three differences, and per axis the 8 outer cells as
// outer(axis, p, w).  (Corner by corner the differences would read 8 x 6 cells.)
// The weights of a difference sum to zero, so the callers take the values relative to
// the cloud's first corner: they then round like differences of neighbours, not
// like the values themselves.
// One z plane per trip of a loop that is kept: with all 32 cells' loads in flight
// the kick needs 354 registers (one wavefront per SIMD).
template <class C, class O>
__device__ __forceinline__ void visit_cloud(const Axis &X, const Axis &Y, const Axis &Z, int n, C corner, O outer)
{
    const long row[4] = {(long)Y.i[0] * n, (long)Y.i[1] * n, (long)Y.i[2] * n, (long)Y.i[3] * n};
    const long plane = (long)n * n;
    // plane index and z weights by rotation (an indexed array would go to memory)
    int z0 = Z.i[0], z1 = Z.i[1], z2 = Z.i[2], z3 = Z.i[3];
    double d0 = -Z.w[0], d1 = -Z.w[1], d2 = Z.w[0], d3 = Z.w[1];
#pragma unroll 1
    for (int c = 0; c < 4; ++c) {
        const long base = plane * z0;
        const double dz = d0;
        if (c == 0 || c == 3) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int a = 0; a < 2; ++a) outer(2, base + row[1 + b] + X.i[1 + a], X.w[a] * Y.w[b] * dz);
        } else {
            const double wz = d1; // the corner's weight: w0 at c = 1, w1 at c = 2
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const double wyz = Y.w[b] * wz;
                outer(0, base + row[1 + b] + X.i[0], -X.w[0] * wyz);
#pragma unroll
                for (int a = 0; a < 2; ++a)
                    corner(base + row[1 + b] + X.i[1 + a], X.w[a] * wyz, (a ? X.w[0] : -X.w[1]) * wyz,
                           X.w[a] * (b ? Y.w[0] : -Y.w[1]) * wz, X.w[a] * Y.w[b] * dz);
                outer(0, base + row[1 + b] + X.i[3], X.w[1] * wyz);
            }
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                outer(1, base + row[0] + X.i[1 + a], X.w[a] * -Y.w[0] * wz);
                outer(1, base + row[3] + X.i[1 + a], X.w[a] * Y.w[1] * wz);
            }
        }
        z0 = z1;
        z1 = z2;
        z2 = z3;
        d0 = d1;
        d1 = d2;
        d2 = d3;
    }
}

// Particle of this thread, in contiguous runs of workgroups per XCD (the grid is
// a multiple of 8): particles kept near lattice order then gather from one slab
// of the grid per L2.  side > 0 (np = side^3, a set that may be in lattice order): a
// workgroup takes a 16 x 4 x 4 block of the lattice instead of 256 in a row.
__device__ __forceinline__ long particle_index(int side)
{
    const long b = (long)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (side == 0) return b * TPB + threadIdx.x;
    const int sx = side >> 4, sy = side >> 2, t = threadIdx.x;
    const int bx = (int)(b % sx), r = (int)(b / sx), by = r % sy, bz = r / sy;
    return ((long)(4 * bz + (t >> 6)) * side + 4 * by + ((t >> 4) & 3)) * side + 16 * bx + (t & 15);
}

__device__ __forceinline__ double lorentz_W(double a, double c, double Psi, const double u[3])
{
    const double chi = 1.0 - Psi / (2.0 * a * a * c * c);
    const double chi2 = chi * chi;
    const double uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    return sqrt(c * c + uu / (a * a * chi2 * chi2));
}

// Five substeps of u_i += dt c_j (f_j)_i (see gr_kick); c_j from the velocity
// as updated by the substeps before it.  Bound by the gathers: 32 cells of 40
// bytes a particle, no two neighbours alike once displaced, so the L1 serves one access
// a clock from end to end (842e6 in 1.46 ms; it waits for a miss in a third of the
// clocks).  256^3 particles on 256^3: 4.79 ms gathering
// five arrays corner by corner (8 x 35 values), 2.22 ms over the packed cells with all
// loads in flight (one wavefront per SIMD), 1.92 ms plane by plane (three), 1.70 ms
// with 16 x 4 x 4 blocks of a lattice, 1.46 ms with values relative to the first corner.
__global__ void __launch_bounds__(TPB) k_kick(Metric M, double a, double c, const double *__restrict__ pos,
                                              double *__restrict__ u, long np, double dt, int order, int side)
{
    const long q = particle_index(side);
    if (q >= np) return;
    const Axis X(pos[3 * q], M.n), Y(pos[3 * q + 1], M.n), Z(pos[3 * q + 2], M.n);
    double uq[3] = {u[3 * q], u[3 * q + 1], u[3 * q + 2]};
    double Phi = 0.0, Psi = 0.0;
    double g[5][3] = {}; // d_i of Phi, Psi, beta^x, beta^y, beta^z, times 2h
    const long p0 = X.i[1] + ((long)Z.i[1] * M.n + Y.i[1]) * M.n;
    const double2 s0 = M.pp[p0], v0 = M.bxy[p0];
    const double z0 = M.bz[p0];
    visit_cloud(
        X, Y, Z, M.n,
        [&](long p, double w, double wx, double wy, double wz) {
            const double2 s = M.pp[p], v = M.bxy[p];
            const double f[5] = {s.x - s0.x, s.y - s0.y, v.x - v0.x, v.y - v0.y, M.bz[p] - z0};
            Phi += w * s.x;
            Psi += w * s.y;
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                g[k][0] += wx * f[k];
                g[k][1] += wy * f[k];
                g[k][2] += wz * f[k];
            }
        },
        [&](int d, long p, double w) {
            const double2 s = M.pp[p], v = M.bxy[p];
            const double f[5] = {s.x - s0.x, s.y - s0.y, v.x - v0.x, v.y - v0.y, M.bz[p] - z0};
#pragma unroll
            for (int k = 0; k < 5; ++k) g[k][d] += w * f[k];
        });
#pragma unroll
    for (int s = 0; s < 5; ++s) {
        const int j = order == GR_KICK_FORWARD ? s + 1 : 5 - s;
        double cj, f[3];
        if (j <= 3) {
            cj = j == 1 ? uq[0] : (j == 2 ? uq[1] : uq[2]); // -u_j times -d_i beta^j
#pragma unroll
            for (int i = 0; i < 3; ++i) f[i] = j == 1 ? g[2][i] : (j == 2 ? g[3][i] : g[4][i]);
        } else {
            const double W = lorentz_W(a, c, Psi, uq);
            if (j == 4)
                cj = -(W * W - c * c) / (W * c) * (1.0 + Phi / (a * a * c * c)) / (1.0 - Psi / (2.0 * a * a * c * c));
            else
                cj = -W / c;
#pragma unroll
            for (int i = 0; i < 3; ++i) f[i] = j == 4 ? g[1][i] : g[0][i];
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) uq[i] += dt * cj * (f[i] * M.inv2h);
    }
    for (int i = 0; i < 3; ++i) u[3 * q + i] = uq[i];
}

// x^i += dt V^i with the fields at the old position, wrapped into [0, 1)
// (256^3 particles: 0.92 -> 0.75 ms; the L1 waits for misses in two thirds of the clocks)
__global__ void __launch_bounds__(TPB) k_drift(Metric M, double a, double c, double *__restrict__ pos,
                                               const double *__restrict__ u, long np, double dt, int side)
{
    const long q = particle_index(side);
    if (q >= np) return;
    double x[3] = {pos[3 * q], pos[3 * q + 1], pos[3 * q + 2]};
    const double uq[3] = {u[3 * q], u[3 * q + 1], u[3 * q + 2]};
    const Axis X(x[0], M.n), Y(x[1], M.n), Z(x[2], M.n);
    double Phi = 0.0, Psi = 0.0, beta[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int cc = 0; cc < 8; ++cc) {
        const int ox = cc & 1, oy = (cc >> 1) & 1, oz = cc >> 2;
        const double w = X.w[ox] * Y.w[oy] * Z.w[oz];
        const long p = ((long)Z.i[1 + oz] * M.n + Y.i[1 + oy]) * M.n + X.i[1 + ox];
        const double2 s = M.pp[p], v = M.bxy[p];
        Phi += w * s.x;
        Psi += w * s.y;
        beta[0] += w * v.x;
        beta[1] += w * v.y;
        beta[2] += w * M.bz[p];
    }
    const double W = lorentz_W(a, c, Psi, uq);
    const double chi = 1.0 - Psi / (2.0 * a * a * c * c);
    const double chi2 = chi * chi;
    const double fac = (1.0 + Phi / (a * a * c * c)) / (chi2 * chi2) * (c / W);
    for (int d = 0; d < 3; ++d) {
        const double v = fac * uq[d] - beta[d];
        double y = x[d] + dt * v;
        y -= floor(y);
        if (y >= 1.0) y = 0.0;
        pos[3 * q + d] = y;
    }
}

// Newtonian kick of the temporary synchronisation: u_i -= dt d_i Phi_N (CIC
// interpolation of the central difference at the eight cloud corners)
__global__ void __launch_bounds__(TPB) k_newton_kick(int n, const double *__restrict__ phiN, double inv2h,
                                                     const double *__restrict__ pos, double *__restrict__ u, long np,
                                                     double dt, int side)
{
    const long q = particle_index(side);
    if (q >= np) return;
    const Axis X(pos[3 * q], n), Y(pos[3 * q + 1], n), Z(pos[3 * q + 2], n);
    double grad[3] = {0.0, 0.0, 0.0};
    const double f0 = phiN[X.i[1] + ((long)Z.i[1] * n + Y.i[1]) * n];
    visit_cloud(
        X, Y, Z, n,
        [&](long p, double, double wx, double wy, double wz) {
            const double f = phiN[p] - f0;
            grad[0] += wx * f;
            grad[1] += wy * f;
            grad[2] += wz * f;
        },
        [&](int d, long p, double w) { grad[d] += w * (phiN[p] - f0); });
    for (int d = 0; d < 3; ++d) u[3 * q + d] -= dt * (grad[d] * inv2h);
}

// side of a cube of particles that 16 x 4 x 4 blocks tile, else 0
inline int lattice_side(long np)
{
    const long s = std::lround(std::cbrt((double)np));
    return s * s * s == np && s % 16 == 0 && s < 32768 ? (int)s : 0;
}

// workgroups for np particles, a multiple of 8
inline unsigned particle_blocks(long np) { return (unsigned)(((np + TPB - 1) / TPB + 7) / 8 * 8); }

} // namespace

void launch_newton_kick(hipStream_t s, int n, const double *phiN, const double *pos, double *u, long np, double dt)
{
    if (np <= 0) return;
    k_newton_kick<<<particle_blocks(np), TPB, 0, s>>>(n, phiN, 0.5 * n, pos, u, np, dt, lattice_side(np));
}

void launch_pack_metric(hipStream_t s, int n, double h, double a, double c, const double *psi, const double *xi,
                        const double *const B[3], const double *b, double *pp, double *bxy, double *bz)
{
    const int bx = n < 64 ? n : 64, by = TPB / bx;
    k_pack_metric<<<dim3((unsigned)((n + bx - 1) / bx), (unsigned)((n + by - 1) / by), (unsigned)n),
                    dim3((unsigned)bx, (unsigned)by), 0, s>>>(
        reinterpret_cast<double2 *>(pp), reinterpret_cast<double2 *>(bxy), bz, psi, xi, B[0], B[1], B[2], b, n,
        1.0 / (2.0 * a * a * c * c), 1.0 / (2.0 * h));
}

void launch_kick(hipStream_t s, int n, double a, double c, const double *pp, const double *bxy, const double *bz,
                 const double *pos, double *u, long np, double dt, int order)
{
    if (np <= 0) return;
    const Metric M{reinterpret_cast<const double2 *>(pp), reinterpret_cast<const double2 *>(bxy), bz, n, 0.5 * n};
    k_kick<<<particle_blocks(np), TPB, 0, s>>>(M, a, c, pos, u, np, dt, order, lattice_side(np));
}

void launch_drift(hipStream_t s, int n, double a, double c, const double *pp, const double *bxy, const double *bz,
                  double *pos, const double *u, long np, double dt)
{
    if (np <= 0) return;
    const Metric M{reinterpret_cast<const double2 *>(pp), reinterpret_cast<const double2 *>(bxy), bz, n, 0.5 * n};
    k_drift<<<particle_blocks(np), TPB, 0, s>>>(M, a, c, pos, u, np, dt, lattice_side(np));
}

} // namespace grmg
