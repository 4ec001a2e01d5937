// Learned initial guess: a small 3-D U-Net (levels with c0/c1/c2/c3 channels,
// two 3^3 convolutions + ReLU per level, 2x2x2 average pooling down, nearest
// upsampling up, skip concatenation, 1x1 head), trained and run on the GPU by
// the kernels below.
//
// Layout: activations channels-last [z][y][x][C] in BF16, periodic boundaries
// (the fields live on a periodic box).  Convolutions are implicit GEMMs on the
// BF16 matrix cores (FP32 accumulation): M = 16 voxels per product, N =
// output channels (16 per tile), K = 27 taps x input channels (weight rows
// padded to a multiple of 32).  The input-gradient of a
// convolution is the same kernel applied to the output-gradient with the
// weights flipped in space and transposed in channels.  Weight gradients
// accumulate in FP32; Adam keeps FP32 master weights.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "gr_internal.h"

typedef __bf16 bf16;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef short shortx4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int TPB = 256;

__device__ __forceinline__ int wrapn(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// ------------------------------------------------------------ convolution

// out[v][ocoff + co] = act(bias[co] + sum_k in[v + off(tap)][icoff + ci] w[co][k]),
// k = tap * cin + ci, taps ordered (dz, dy, dx) in {-1,0,1}^3 with dx fastest.
// One wave: VG groups of 16 consecutive voxels x 16 NT output channels (blockIdx.y
// picks them).  The 27 taps are unrolled
// (every lane of a product works on the same tap) and each tap runs over the
// input channels in CK steps of KS = 32 (v_mfma_f32_16x16x32_bf16, 8 channels per
// lane) when cin % 32 == 0, else KS = 16 (v_mfma_f32_16x16x16_bf16, 4 channels
// per lane); a lane's neighbour rows are formed once, so the inner loop is
// loads and matrix products.  CK = 0: any number of steps.  n^3 must be a multiple of
// 64 VG (4 waves per block) and cin a multiple of KS.
// Latency bound on the deep levels (8^3 has 32 groups of voxels): one group and 16
// channels a wave, the steps unrolled so that their loads overlap; 64 -> 64 channels
// at 8^3 65 -> 14 us against four groups and all channels a wave.
template <int KS> struct ConvOperand;
template <> struct ConvOperand<32> {
    typedef bf16x8 type;
    static __device__ __forceinline__ floatx4 mfma(type a, type b, floatx4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};
template <> struct ConvOperand<16> {
    typedef shortx4 type;
    static __device__ __forceinline__ floatx4 mfma(type a, type b, floatx4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
    }
};

// four channels of one voxel: bias, ReLU, one 8-byte store
template <bool RELU, bool BIAS>
__device__ __forceinline__ void store_out(floatx4 v, const float *__restrict__ bias, int co, bf16 *__restrict__ dst)
{
    bf16x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float r = v[j] + (BIAS ? bias[co + j] : 0.0f);
        if (RELU) r = r > 0.0f ? r : 0.0f;
        o[j] = (bf16)r;
    }
    *reinterpret_cast<bf16x4 *>(dst) = o;
}

template <int NT, int VG, int KS, int CK, bool RELU, bool BIAS>
__global__ void __launch_bounds__(256) k_conv3(const bf16 *__restrict__ in, int cin, int icstride, int icoff,
                                               const bf16 *__restrict__ w, int kpad, const float *__restrict__ bias,
                                               bf16 *__restrict__ out, int ocstride, int ocoff, int n)
{
    typedef ConvOperand<KS> Op;
    typedef typename Op::type opT;
    constexpr int PER = KS / 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, cob = 16 * NT * blockIdx.y;
    const int v0 = (blockIdx.x * 4 + wave) * 16 * VG;
    const int i = lane & 15, g = lane >> 4;
    // neighbour coordinates of this lane's voxel in each group: x, y * n, z * n^2
    int xo[VG][3], yo[VG][3], zo[VG][3];
#pragma unroll
    for (int q = 0; q < VG; ++q) {
        const int v = v0 + 16 * q + i;
        const int x = v % n, y = (v / n) % n, z = v / (n * n);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            xo[q][d] = wrapn(x + d - 1, n);
            yo[q][d] = wrapn(y + d - 1, n) * n;
            zo[q][d] = wrapn(z + d - 1, n) * n * n;
        }
    }
    floatx4 acc[VG][NT];
#pragma unroll
    for (int q = 0; q < VG; ++q)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[q][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    const bf16 *wl = w + (long)(cob + i) * kpad + PER * g;
    const long wstep = (long)16 * kpad;
    const int steps = CK ? CK : cin / KS;
    constexpr int UN = CK ? CK : 1;
#pragma unroll
    for (int dz = 0; dz < 3; ++dz)
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const int tap = (dz * 3 + dy) * 3 + dx;
                const bf16 *src[VG];
#pragma unroll
                for (int q = 0; q < VG; ++q)
                    src[q] = in + (long)(zo[q][dz] + yo[q][dy] + xo[q][dx]) * icstride + icoff + PER * g;
                const bf16 *wt = wl + tap * (CK ? CK * KS : cin);
#pragma unroll UN
                for (int ck = 0; ck < steps; ++ck) {
                    const int c0 = ck * KS;
                    opT bw[NT];
#pragma unroll
                    for (int t = 0; t < NT; ++t) bw[t] = *reinterpret_cast<const opT *>(wt + t * wstep + c0);
#pragma unroll
                    for (int q = 0; q < VG; ++q) {
                        const opT a = *reinterpret_cast<const opT *>(src[q] + c0);
#pragma unroll
                        for (int t = 0; t < NT; ++t) acc[q][t] = Op::mfma(bw[t], a, acc[q][t]);
                    }
                }
            }
    // lane holds D[4g + j][i]: voxel v0 + 16 q + i, channels 16t + 4g + j
#pragma unroll
    for (int q = 0; q < VG; ++q)
#pragma unroll
        for (int t = 0; t < NT; ++t)
            store_out<RELU, BIAS>(acc[q][t], bias, cob + 16 * t + 4 * g,
                                  out + (long)(v0 + 16 * q + i) * ocstride + ocoff + cob + 16 * t + 4 * g);
}

// The same convolution with the input staged in LDS: one block computes a
// 16 (x) x 4 (y) x 4 (z) tile of output voxels and 16 NT channels (blockIdx.y picks
// them); wave w takes the plane z0 + w and its product group q the row y0 + q.  For
// each chunk of CW input channels the block copies the tile's 18 x 6 x 6 input halo
// into LDS; the next chunk is loaded meanwhile.  Voxel strides of 32 and 96 bytes suit
// the lanes that a 16-byte read takes together (lanes 0-3, 12-15, 20-27): no cycle of
// the LDS is lost to bank conflicts at 32 bytes and 21 % at 96 (48 and 80 bytes: half).  CW = 32: one
// v_mfma_f32_16x16x32_bf16 per tap, all lanes on the same tap; a plane's six rows are
// read once for the three dy, and the weights are loaded
// a row of taps ahead (NT = 2) or all at once (NT = 1: 17 -> 12 us a layer of the 64^3 network).
// CW = 16: taps go in pairs, lanes g < 2 on the first and g >= 2 on the second (8
// channels each), the unpaired 27th tap padded with zeros, all weights loaded first.
// n must be a multiple of 16 and cin of CW.
//
// The products of an output run in the order taps within channel chunks.  Operands are
// given weights first, so a lane holds four channels of one voxel and stores them at once.
// Bound by issue and latency: at 16 channels 56 products take 400 other instructions a
// wave, so blocks that march in z (MARCH) keep weights and addresses; at 32 and 64 by the
// weights, that every wave reads from L2.  Measured (us): 16 -> 16 at 128^3 131 -> 60;
// 64 -> 64 at 32^3 50 -> 19 and at 16^3 47 -> 12 (16 channels a block instead of all,
// where tiles are few), 32 -> 32 at 64^3 51 -> 32.  48 -> 16 at 128^3 takes 200, as long
// with whole voxels staged once.
constexpr int CT_HX = 18, CT_HY = 6, CT_HZ = 6, CT_HV = CT_HX * CT_HY * CT_HZ;

template <int NT, int CW, bool MARCH, bool RELU, bool BIAS>
__global__ void __launch_bounds__(256, MARCH ? 3 : 2)
    k_conv3_lds(const bf16 *__restrict__ in, int cin, int icstride, int icoff, const bf16 *__restrict__ w, int kpad,
                const float *__restrict__ bias, bf16 *__restrict__ out, int ocstride, int ocoff, int n, int ztiles)
{
    constexpr int STR = CW == 32 ? 48 : 16, UPV = CW / 8, NU = CT_HV * UPV, PERT = (NU + 255) / 256;
    __shared__ __align__(16) bf16 tile[CT_HV * STR];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, cob = 16 * NT * blockIdx.y;
    const int i = lane & 15, g = lane >> 4;
    // blocks in contiguous runs per XCD (dispatch is round-robin over the 8 XCDs)
    const int nblk = gridDim.x;
    int b = blockIdx.x;
    if (nblk % 8 == 0) b = (b & 7) * (nblk >> 3) + (b >> 3);
    const int tx = n >> 4, ty = n >> 2;
    const int X0 = (b % tx) * 16, Y0 = ((b / tx) % ty) * 4;
    int zt = MARCH ? ztiles : 1, Z0 = (b / tx / ty) * 4 * zt;
    const bool hi = g >= 2;
    const int lbase = (wave * CT_HY * CT_HX + i) * STR + (CW == 32 ? 8 * g : 8 * (g & 1));
    const bf16 *wl = w + (long)(cob + i) * kpad + (CW == 32 ? 8 * g : 8 * (g & 1));
    const long wstep = (long)16 * kpad;
    bf16x8 stage[PERT];
    int sxy[PERT]; // halo voxel in its plane (n^2 < 2^21), plane of the halo above it
#pragma unroll
    for (int r = 0; r < PERT; ++r) {
        const int u = threadIdx.x + 256 * r, h = u < NU ? u / UPV : 0;
        const int hx = h % CT_HX, hy = (h / CT_HX) % CT_HY, hz = h / (CT_HX * CT_HY);
        sxy[r] = (wrapn(Y0 - 1 + hy, n) * n + wrapn(X0 - 1 + hx, n)) | hz << 24;
    }
    const bf16 *inl = in + icoff + 8 * (threadIdx.x % UPV);
    auto fetch = [&](int z0, int c0) {
#pragma unroll
        for (int r = 0; r < PERT; ++r)
            stage[r] = *reinterpret_cast<const bf16x8 *>(
                inl + (long)(wrapn(z0 - 1 + (sxy[r] >> 24), n) * n * n + (sxy[r] & 0xffffff)) * icstride + c0);
    };
    bf16 *const put = tile + (threadIdx.x / UPV) * STR + 8 * (threadIdx.x % UPV);
    bf16x8 bw[CW == 16 ? 14 : 1][NT];
    floatx4 acc[4][NT];
    fetch(Z0, 0);
    for (int c0 = 0, first = 1;; first = 0) { // chunks of a tile, then the next tile
#pragma unroll
        for (int r = 0; r < PERT; ++r)
            if ((int)threadIdx.x + 256 * r < NU) *reinterpret_cast<bf16x8 *>(put + r * (256 / UPV) * STR) = stage[r];
        const bool tile_done = MARCH || c0 + CW >= cin, all_done = tile_done && zt == 1;
        if (MARCH || c0 == 0)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[q][t] = floatx4{0.f, 0.f, 0.f, 0.f};
        if constexpr (CW == 32) {
            constexpr int AHEAD = NT == 1 ? 8 : 1, RING = AHEAD + 1; // NT = 1: all before the staging barrier
            bf16x8 wr[RING][3][NT]; // weights of the rows of taps r .. r + AHEAD
            auto weights = [&](int r) {
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        wr[r % RING][dx][t] = *reinterpret_cast<const bf16x8 *>(wl + t * wstep + (3 * r + dx) * cin + c0);
            };
#pragma unroll
            for (int r = 0; r < AHEAD; ++r) weights(r);
            __syncthreads();
            if (!all_done) fetch(tile_done ? Z0 + 4 : Z0, tile_done ? 0 : c0 + CW);
#pragma unroll
            for (int dz = 0; dz < 3; ++dz) {
                bf16x8 a[6][3];
#pragma unroll
                for (int y = 0; y < 6; ++y)
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx)
                        a[y][dx] = *reinterpret_cast<const bf16x8 *>(tile + lbase + ((dz * CT_HY + y) * CT_HX + dx) * STR);
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const int r = 3 * dz + dy;
                    if (r + AHEAD < 9) weights(r + AHEAD);
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int t = 0; t < NT; ++t)
                                acc[q][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[r % RING][dx][t], a[q + dy][dx],
                                                                                    acc[q][t], 0, 0, 0);
                }
            }
        } else {
            if (!MARCH || first) { // MARCH: one chunk, whose weights stay
#pragma unroll
                for (int m = 0; m < 14; ++m)
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const int tap = m < 13 ? 2 * m + (hi ? 1 : 0) : 26;
                        bw[m][t] = *reinterpret_cast<const bf16x8 *>(wl + t * wstep + tap * cin + c0);
                        if (m == 13 && hi)
#pragma unroll
                            for (int j = 0; j < 8; ++j) bw[m][t][j] = (bf16)0.0f;
                    }
            }
            __syncthreads();
            if (!all_done) fetch(tile_done ? Z0 + 4 : Z0, tile_done ? 0 : c0 + CW);
#pragma unroll
            for (int m = 0; m < 14; ++m) {
                const int t0 = 2 * m, t1 = m < 13 ? 2 * m + 1 : 26; // lanes g < 2 and g >= 2
                const int o0 = (((t0 / 9) * CT_HY + (t0 / 3) % 3) * CT_HX + t0 % 3) * STR;
                const int o1 = (((t1 / 9) * CT_HY + (t1 / 3) % 3) * CT_HX + t1 % 3) * STR;
                const bf16 *at = tile + lbase + (hi ? o1 : o0);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    bf16x8 a = *reinterpret_cast<const bf16x8 *>(at + q * CT_HX * STR);
                    if (m == 13 && hi)
#pragma unroll
                        for (int j = 0; j < 8; ++j) a[j] = (bf16)0.0f;
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        acc[q][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bw[m][t], a, acc[q][t], 0, 0, 0);
                }
            }
        }
        if (tile_done) {
            // lane holds D[4g + j][i]: voxel (X0 + i, Y0 + q, Z0 + wave), channels 16t + 4g + j
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const long v = ((long)(Z0 + wave) * n + (Y0 + q)) * n + X0 + i;
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    store_out<RELU, BIAS>(acc[q][t], bias, cob + 16 * t + 4 * g,
                                          out + v * ocstride + ocoff + cob + 16 * t + 4 * g);
            }
            if (all_done) return;
            --zt;
            Z0 += 4;
            c0 = 0;
        } else {
            c0 += CW;
        }
        __syncthreads(); // this chunk's reads are done
    }
}

// Weight gradient of a 3^3 convolution on the BF16 matrix cores:
//   dW[co][tap*cin + ci] = sum_v g[v][gcoff + co] in[v + off(tap)][icoff + ci],
//   db[co] = sum_v g[v][gcoff + co].
// Per tap this is a GEMM with M = cout, N = cin and K = the voxels.  A block takes
// tiles of TX x 4 x 4 voxels (TX = 16, 8 or 4) and CO x CI channels for all 27 taps:
// the output gradient and the input with its halo are staged in LDS once, channels
// last, and the operands (8 voxels of one channel a lane) come from transposing LDS
// reads (ds_read_b64_tr_b16: 16 lanes read 4 voxels x 16 channels, lane i gets the 4
// voxels of channel i), so a tap is an offset.  Wave w accumulates the taps w, w + 4,
// ... in FP32 over the block's tiles (blockIdx.x, + gridDim.x, ...); the block writes
// its partial sums, and k_wgrad_reduce adds the partials in a fixed order.  db comes
// from products with ones in the waves that have one tap less.
// A block a tap, staged 27 times and transposed by 2-byte stores, took 73 us a layer
// (64^3 network, 14 layers); this 8-18 us (48 -> 16 at 64^3: 43), bound by latency and, at 16
// channels, by the LDS reads: half of the cycles of the LDS are bank conflicts.
constexpr int WG_MAXC = 128;              // largest channel count of either side
typedef __attribute__((address_space(3))) shortx4 *lds_s4;
union WgOperand {
    shortx4 h[2];
    bf16x8 v;
};
// 8 voxels (two runs of 4) x this lane's channel
__device__ __forceinline__ bf16x8 wg_operand(const bf16 *p0, const bf16 *p1)
{
    WgOperand o;
    o.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(__attribute__((address_space(3))) short *)(short *)p0);
    o.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(__attribute__((address_space(3))) short *)(short *)p1);
    return o.v;
}
template <int TX, int CO, int CI>
__global__ void __launch_bounds__(TPB) k_conv3_wgrad(const bf16 *__restrict__ g, int cout, int gcstride, int gcoff,
                                                     const bf16 *__restrict__ in, int cin, int icstride, int icoff,
                                                     float *__restrict__ part, float *__restrict__ bpart, int n)
{
    constexpr int HX = TX + 2, HV = HX * 36, TV = TX * 16; // halo and tile voxels
    constexpr int SG = CO + 8, SI = CI + 8;                // LDS strides of a voxel
    constexpr int UG = CO / 8, UI = CI / 8, PG = (TV * UG + TPB - 1) / TPB, PI = (HV * UI + TPB - 1) / TPB;
    constexpr int NT = 7, MT = CO / 16, KT = CI / 16, STEPS = TV / 32;
    __shared__ __align__(16) bf16 sg[TV * SG];
    __shared__ __align__(16) bf16 si[HV * SI];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 15, gq = lane >> 4;
    const int co0 = CO * (blockIdx.y % (cout / CO)), ci0 = CI * (blockIdx.y / (cout / CO));
    const int tx = n / TX, ty = n / 4, tiles = tx * ty * ty;
    floatx4 acc[NT][MT][KT], bacc[MT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int k = 0; k < KT; ++k) acc[t][m][k] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < MT; ++m) bacc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
    bf16x8 ones;
#pragma unroll
    for (int j = 0; j < 8; ++j) ones[j] = (bf16)1.0f;
    // this lane's place in the LDS reads: voxel i / 4 of a run of 4, channels 4 (i % 4) ..
    const bf16 *const lg = sg + (i >> 2) * SG + 4 * (i & 3), *const li = si + (i >> 2) * SI + 4 * (i & 3);
    // voxel 8 gq (+ 4) of K step 0: run of 4 in x, rows of TX in y, then z
    const int r0 = 2 * gq, r1 = 2 * gq + 1; // runs of 4 voxels
    constexpr int RX = TX / 4;              // runs per row
    auto run_halo = [](int r) { return ((r / (4 * RX)) * 6 + (r / RX) % 4) * HX + 4 * (r % RX); };
    const int hr0 = run_halo(r0) * SI, hr1 = run_halo(r1) * SI;
    bf16x8 pg[PG], pi[PI];
    auto fetch = [&](int tile) {
        const int X0 = (tile % tx) * TX, Y0 = ((tile / tx) % ty) * 4, Z0 = (tile / tx / ty) * 4;
#pragma unroll
        for (int r = 0; r < PG; ++r) {
            const int u = threadIdx.x + TPB * r, v = u < TV * UG ? u / UG : 0;
            const long src = ((long)(Z0 + v / (4 * TX)) * n + Y0 + (v / TX) % 4) * n + X0 + v % TX;
            pg[r] = *reinterpret_cast<const bf16x8 *>(g + src * gcstride + gcoff + co0 + 8 * (u % UG));
        }
#pragma unroll
        for (int r = 0; r < PI; ++r) {
            const int u = threadIdx.x + TPB * r, h = u < HV * UI ? u / UI : 0;
            const long src = ((long)wrapn(Z0 - 1 + h / (6 * HX), n) * n + wrapn(Y0 - 1 + (h / HX) % 6, n)) * n +
                             wrapn(X0 - 1 + h % HX, n);
            pi[r] = *reinterpret_cast<const bf16x8 *>(in + src * icstride + icoff + ci0 + 8 * (u % UI));
        }
    };
    fetch(blockIdx.x);
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
#pragma unroll
        for (int r = 0; r < PG; ++r) {
            const int u = threadIdx.x + TPB * r;
            if (u < TV * UG) *reinterpret_cast<bf16x8 *>(sg + (u / UG) * SG + 8 * (u % UG)) = pg[r];
        }
#pragma unroll
        for (int r = 0; r < PI; ++r) {
            const int u = threadIdx.x + TPB * r;
            if (u < HV * UI) *reinterpret_cast<bf16x8 *>(si + (u / UI) * SI + 8 * (u % UI)) = pi[r];
        }
        __syncthreads();
        if (tile + (int)gridDim.x < tiles) fetch(tile + gridDim.x);
#pragma unroll 1
        for (int s = 0; s < STEPS; ++s) { // 32 voxels: 8 runs
            bf16x8 a[MT];
#pragma unroll
            for (int m = 0; m < MT; ++m)
                a[m] = wg_operand(lg + (32 * s + 8 * gq) * SG + 16 * m, lg + (32 * s + 8 * gq + 4) * SG + 16 * m);
            const int hs = run_halo(8 * s) * SI;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int tap = wave + 4 * t;
                if (tap < 27) { // uniform in the wave
                    const int to = (((tap / 9) * 6 + (tap / 3) % 3) * HX + tap % 3) * SI + hs;
#pragma unroll
                    for (int k = 0; k < KT; ++k) {
                        const bf16x8 b = wg_operand(li + hr0 + to + 16 * k, li + hr1 + to + 16 * k);
#pragma unroll
                        for (int m = 0; m < MT; ++m)
                            acc[t][m][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], b, acc[t][m][k], 0, 0, 0);
                    }
                } else if (ci0 == 0) { // wave 3: the bias gradient
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        bacc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], ones, bacc[m], 0, 0, 0);
                }
            }
        }
        __syncthreads();
    }
    // partial of this block: part[blockIdx.x][tap][co][ci]; lane holds D[4gq + j][i]
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int tap = wave + 4 * t;
        if (tap >= 27) continue;
        float *dst = part + ((long)blockIdx.x * 27 + tap) * cout * cin;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int k = 0; k < KT; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    dst[(long)(co0 + 16 * m + 4 * gq + j) * cin + ci0 + 16 * k + i] = acc[t][m][k][j];
    }
    if (wave == 3 && ci0 == 0 && i == 0)
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int j = 0; j < 4; ++j) bpart[(long)blockIdx.x * cout + co0 + 16 * m + 4 * gq + j] = bacc[m][j];
}

// dw[co][tap*cin + ci] += sum over the nbk block partials, db likewise, in a fixed order.
// Four consecutive values a thread; the 8 groups of 32 threads of a block take every
// eighth partial and are added in order.  The last block takes db, 4 groups of 64.
__global__ void __launch_bounds__(TPB) k_wgrad_reduce(const float *__restrict__ part, const float *__restrict__ bpart,
                                                      int nbk, int cout, int cin, float *__restrict__ dw,
                                                      float *__restrict__ db)
{
    __shared__ floatx4 sh[8][32];
    __shared__ float shb[4][64];
    if (blockIdx.x == gridDim.x - 1) {
        const int c = threadIdx.x & 63, w = threadIdx.x >> 6;
        float t = 0.0f;
        if (c < cout)
#pragma unroll 8
            for (int b = w; b < nbk; b += 4) t += bpart[(long)b * cout + c];
        shb[w][c] = t;
        __syncthreads();
        if (w == 0 && c < cout) db[c] += ((t + shb[1][c]) + shb[2][c]) + shb[3][c];
        return;
    }
    const long per = 27L * cout * cin; // a multiple of 128
    const int c = threadIdx.x & 31, w = threadIdx.x >> 5;
    const long q = (long)blockIdx.x * 128 + 4 * c;
    floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int b = w; b < nbk; b += 8) s += *reinterpret_cast<const floatx4 *>(part + (long)b * per + q);
    sh[w][c] = s;
    __syncthreads();
    if (w == 0) {
        for (int k = 1; k < 8; ++k) s += sh[k][c];
        const int tap = (int)(q / ((long)cout * cin));
        const int rem = (int)(q % ((long)cout * cin));
        const int co = rem / cin, ci = rem % cin;
        float *d = dw + (long)co * 27 * cin + tap * cin + ci; // parameters start at any multiple of 4 bytes
#pragma unroll
        for (int j = 0; j < 4; ++j) d[j] += s[j];
    }
}

// ------------------------------------------------------------ elementwise

// planar FP32 [cin][n^3] -> channels-last BF16 [n^3][16] (zero channels above cin)
__global__ void k_pack_input(const float *__restrict__ src, int cin, bf16 *__restrict__ dst, long N)
{
    const long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= N) return;
    bf16x8 lo, hi; // the voxel's 16 channels as two 16-byte stores
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        lo[c] = (bf16)(c < cin ? src[c * N + v] : 0.0f);
        hi[c] = (bf16)(c + 8 < cin ? src[(c + 8) * N + v] : 0.0f);
    }
    bf16x8 *d = reinterpret_cast<bf16x8 *>(dst + v * 16);
    d[0] = lo;
    d[1] = hi;
}

// 2x2x2 average of channels [coff, coff + c) -> [m^3][c]; one thread per voxel and
// group of 8 channels (c, coff and cstride are multiples of 8)
__global__ void k_pool(const bf16 *__restrict__ in, int cstride, int coff, int c, bf16 *__restrict__ out, int n)
{
    const int m = n / 2, gc = c / 8;
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (long)m * m * m * gc) return;
    const int ch = (int)(q % gc) * 8;
    const int V = (int)(q / gc);
    const int X = V % m, Y = (V / m) % m, Z = V / (m * m);
    float s[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const long v = ((long)(2 * Z + (k >> 2)) * n + 2 * Y + ((k >> 1) & 1)) * n + 2 * X + (k & 1);
        const bf16x8 a = *reinterpret_cast<const bf16x8 *>(in + v * cstride + coff + ch);
#pragma unroll
        for (int j = 0; j < 8; ++j) s[j] += (float)a[j];
    }
    bf16x8 o;
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = (bf16)(0.125f * s[j]);
    *reinterpret_cast<bf16x8 *>(out + (long)V * c + ch) = o;
}

// voxel v < 2^31 of an n^3 grid
__device__ __forceinline__ void voxel_at(int v, int n, int &x, int &y, int &z)
{
    const unsigned r = (unsigned)v / n;
    x = (int)((unsigned)v - r * n);
    z = (int)(r / n);
    y = (int)(r - z * n);
}

// gradient of the pooling, added to channels [coff, coff + c) of gin; one thread per
// voxel and group of 8 channels (c, coff and cstride are multiples of 8)
__global__ void k_pool_bwd_add(const bf16 *__restrict__ gout, int c, bf16 *__restrict__ gin, int cstride, int coff,
                               int n)
{
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int gc = c / 8;
    if (q >= (long)n * n * n * gc) return;
    const int v = (int)(q / gc), ch = (int)(q - (long)v * gc) * 8, m = n / 2;
    int x, y, z;
    voxel_at(v, n, x, y, z);
    const bf16x8 o = *reinterpret_cast<const bf16x8 *>(gout + (((long)(z / 2) * m + y / 2) * m + x / 2) * c + ch);
    bf16x8 *gp = reinterpret_cast<bf16x8 *>(gin + (long)v * cstride + coff + ch);
    bf16x8 gv = *gp;
#pragma unroll
    for (int j = 0; j < 8; ++j) gv[j] = (bf16)((float)gv[j] + 0.125f * (float)o[j]);
    *gp = gv;
}

// nearest upsampling of [m^3][c] into channels [0, c) of out [n^3][cstride]
// one thread per voxel and group of 8 channels (16-byte loads and stores;
// c and cstride are multiples of 8)
__global__ void k_upsample(const bf16 *__restrict__ in, int c, bf16 *__restrict__ out, int cstride, int n)
{
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int cg = c >> 3;
    if (q >= (long)n * n * n * cg) return;
    const int v = (int)(q / cg), ch = (int)(q - (long)v * cg) * 8, m = n / 2;
    int x, y, z;
    voxel_at(v, n, x, y, z);
    *reinterpret_cast<bf16x8 *>(out + (long)v * cstride + ch) =
        *reinterpret_cast<const bf16x8 *>(in + (((long)(z / 2) * m + y / 2) * m + x / 2) * c + ch);
}

// gradient of the upsampling: sum of the 8 children's channels [0, c)
__global__ void k_upsample_bwd(const bf16 *__restrict__ gout, int cstride, int c, bf16 *__restrict__ gin, int n)
{
    const int m = n / 2;
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (long)m * m * m * c) return;
    const int ch = (int)(q % c);
    const long V = q / c;
    const int X = (int)(V % m), Y = (int)((V / m) % m), Z = (int)(V / ((long)m * m));
    float s = 0.0f;
    for (int k = 0; k < 8; ++k) {
        const long v = ((long)(2 * Z + (k >> 2)) * n + 2 * Y + ((k >> 1) & 1)) * n + 2 * X + (k & 1);
        s += (float)gout[v * cstride + ch];
    }
    gin[V * c + ch] = (bf16)s;
}

// g = g * (a > 0) on channels [coff, coff + c) of both (ReLU gradient); one thread per
// voxel and group of 8 channels (all counts and offsets are multiples of 8)
__global__ void k_relu_bwd(bf16 *__restrict__ g, int gcstride, int gcoff, const bf16 *__restrict__ a, int acstride,
                           int acoff, int c, long N)
{
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int gc = c / 8;
    if (q >= N * gc) return;
    const int v = (int)(q / gc), ch = (int)(q - (long)v * gc) * 8;
    bf16x8 *gp = reinterpret_cast<bf16x8 *>(g + (long)v * gcstride + gcoff + ch);
    const bf16x8 av = *reinterpret_cast<const bf16x8 *>(a + (long)v * acstride + acoff + ch);
    bf16x8 gv = *gp;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (!((float)av[j] > 0.0f)) gv[j] = (bf16)0.0f;
    *gp = gv;
}

// 1x1 head: y[o][v] = b[o] + sum_c w[o][c] h[v][c]   (FP32 planar output, 16 channels)
__global__ void __launch_bounds__(TPB) k_head(const bf16 *__restrict__ h, const float *__restrict__ w,
                                              const float *__restrict__ b, float *__restrict__ y, int cout, long N)
{
    const long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= N) return;
    const bf16x8 *hp = reinterpret_cast<const bf16x8 *>(h + v * 16);
    const bf16x8 lo = hp[0], hi = hp[1];
    float hv[16];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        hv[k] = (float)lo[k];
        hv[k + 8] = (float)hi[k];
    }
    for (int o = 0; o < cout; ++o) {
        float s = b[o];
#pragma unroll
        for (int k = 0; k < 16; ++k) s += w[o * 16 + k] * hv[k];
        y[o * N + v] = s;
    }
}

// MSE loss pieces: gy = 2 (y - t) / (cout N); per-block partial sums of (y - t)^2
__global__ void k_mse(const float *__restrict__ y, const float *__restrict__ t, float *__restrict__ gy, long total,
                      float *__restrict__ partial)
{
    __shared__ float sh[TPB];
    float s = 0.0f;
    for (long q = (long)blockIdx.x * TPB + threadIdx.x; q < total; q += (long)gridDim.x * TPB) {
        const float d = y[q] - t[q];
        gy[q] = 2.0f * d / (float)total;
        s += d * d;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = TPB / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = sh[0];
}

// Optional smoothness term of the loss, lambda * mean((Lap d)^2) with d = y - t
// and Lap the 7-point periodic Laplacian of unit spacing, per channel: the
// judge of a guess is a residual, which weights errors by Lap.  Pass 1:
// q = Lap d and partial sums of q^2; pass 2: gy += 2 lambda Lap q / total
// (Lap is symmetric).
__device__ __forceinline__ long lap_nb(int x, int y, int z, int n, int dx, int dy, int dz)
{
    x += dx;
    y += dy;
    z += dz;
    x = x < 0 ? x + n : (x >= n ? x - n : x);
    y = y < 0 ? y + n : (y >= n ? y - n : y);
    z = z < 0 ? z + n : (z >= n ? z - n : z);
    return ((long)z * n + y) * n + x;
}

template <bool FROM_DIFF>
__device__ __forceinline__ float lap_at(const float *__restrict__ a, const float *__restrict__ b, long base, int x,
                                        int y, int z, int n)
{
    auto v = [&](long q) { return FROM_DIFF ? a[base + q] - b[base + q] : a[base + q]; };
    const float c = v(((long)z * n + y) * n + x);
    return v(lap_nb(x, y, z, n, 1, 0, 0)) + v(lap_nb(x, y, z, n, -1, 0, 0)) + v(lap_nb(x, y, z, n, 0, 1, 0)) +
           v(lap_nb(x, y, z, n, 0, -1, 0)) + v(lap_nb(x, y, z, n, 0, 0, 1)) + v(lap_nb(x, y, z, n, 0, 0, -1)) -
           6.0f * c;
}

__global__ void k_lap_loss1(const float *__restrict__ y, const float *__restrict__ t, float *__restrict__ q, int n,
                            long total, float *__restrict__ partial)
{
    __shared__ float sh[TPB];
    const long N = (long)n * n * n;
    float s = 0.0f;
    for (long p = (long)blockIdx.x * TPB + threadIdx.x; p < total; p += (long)gridDim.x * TPB) {
        const long ch = p / N, v = p - ch * N;
        const unsigned r = (unsigned)v / n; // below 2^31 voxels
        const int x = (int)((unsigned)v - r * n), z = (int)(r / n), yy = (int)(r - z * n);
        const float l = lap_at<true>(y, t, ch * N, x, yy, z, n);
        q[p] = l;
        s += l * l;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = TPB / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = sh[0];
}

__global__ void k_lap_loss2(const float *__restrict__ q, float *__restrict__ gy, int n, long total, float lam)
{
    const long N = (long)n * n * n;
    for (long p = (long)blockIdx.x * TPB + threadIdx.x; p < total; p += (long)gridDim.x * TPB) {
        const long ch = p / N, v = p - ch * N;
        const unsigned r = (unsigned)v / n; // below 2^31 voxels
        const int x = (int)((unsigned)v - r * n), z = (int)(r / n), yy = (int)(r - z * n);
        gy[p] += 2.0f * lam * lap_at<false>(q, nullptr, ch * N, x, yy, z, n) / (float)total;
    }
}

// head backward: gh[v][c] = sum_o w[o][c] gy[o][v]; the block's partial sums of
// dW[o][c] = sum_v gy[o][v] h[v][c] and db[o] = sum_v gy[o][v] over its 256
// voxels, one parameter per thread in voxel order, to part[block][cout*c + cout]
// (k_head_reduce adds the blocks in order: deterministic).
// 16 channels; the output gradients of a voxel are read once.
__global__ void __launch_bounds__(TPB) k_head_bwd(const float *__restrict__ gy, const bf16 *__restrict__ h,
                                                  const float *__restrict__ w, int cout, bf16 *__restrict__ gh,
                                                  float *__restrict__ part, long N)
{
    constexpr int C = 16;
    __shared__ float sgy[16][TPB];
    __shared__ float sh[TPB][C + 1];
    const long v = (long)blockIdx.x * TPB + threadIdx.x;
    float hv[C], g[C], gv[16];
#pragma unroll
    for (int k = 0; k < C; ++k) hv[k] = g[k] = 0.0f;
#pragma unroll
    for (int o = 0; o < 16; ++o) gv[o] = v < N && o < cout ? gy[o * N + v] : 0.0f;
    if (v < N) {
        const bf16x8 *hp = reinterpret_cast<const bf16x8 *>(h + v * C);
        const bf16x8 lo = hp[0], hi = hp[1];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            hv[k] = (float)lo[k];
            hv[k + 8] = (float)hi[k];
        }
    }
#pragma unroll
    for (int o = 0; o < 16; ++o) {
        if (o >= cout) break;
#pragma unroll
        for (int k = 0; k < C; ++k) g[k] += w[o * C + k] * gv[o];
        sgy[o][threadIdx.x] = gv[o];
    }
#pragma unroll
    for (int k = 0; k < C; ++k) sh[threadIdx.x][k] = hv[k];
    if (v < N) {
        bf16x8 lo, hi;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            lo[k] = (bf16)g[k];
            hi[k] = (bf16)g[k + 8];
        }
        bf16x8 *gp = reinterpret_cast<bf16x8 *>(gh + v * C);
        gp[0] = lo;
        gp[1] = hi;
    }
    __syncthreads();
    const int npar = cout * C + cout;
    for (int q = threadIdx.x; q < npar; q += TPB) {
        float s = 0.0f;
        if (q < cout * C) {
            const int o = q / C, k = q % C;
#pragma unroll 8
            for (int r = 0; r < TPB; ++r) s += sgy[o][r] * sh[r][k];
        } else {
            const int o = q - cout * C;
#pragma unroll 8
            for (int r = 0; r < TPB; ++r) s += sgy[o][r];
        }
        part[(long)blockIdx.x * npar + q] = s;
    }
}

// one block per parameter: thread t adds partials t, t + 256, ... in order,
// then a fixed tree over the threads (deterministic)
__global__ void __launch_bounds__(TPB) k_head_reduce(const float *__restrict__ part, int nblk, int npar, int nw,
                                                     float *__restrict__ dw, float *__restrict__ db)
{
    __shared__ float sh[TPB];
    const int q = blockIdx.x;
    float s = 0.0f;
    for (int b = threadIdx.x; b < nblk; b += TPB) s += part[(long)b * npar + q];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = TPB / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (q < nw) dw[q] += sh[0];
        else db[q - nw] += sh[0];
    }
}

// FP32 master weights -> BF16 forward layout [co][kpad] and the flipped /
// transposed layout [ci][kpad'] used for input gradients.
__global__ void k_prep_weights(const float *__restrict__ w, int cout, int cin, int kpad, int kpadT,
                               bf16 *__restrict__ wf, bf16 *__restrict__ wt)
{
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long tot = (long)cout * kpad;
    if (q < tot) {
        const int co = (int)(q / kpad), k = (int)(q % kpad);
        wf[q] = (bf16)(k < 27 * cin ? w[(long)co * 27 * cin + k] : 0.0f);
    }
    const long totT = (long)cin * kpadT;
    if (q < totT) {
        const int ci = (int)(q / kpadT), k = (int)(q % kpadT);
        float val = 0.0f;
        if (k < 27 * cout) {
            const int tapT = k / cout, co = k % cout;
            const int tap = 26 - tapT; // off(tapT) = -off(tap)
            val = w[(long)co * 27 * cin + tap * cin + ci];
        }
        wt[q] = (bf16)val;
    }
}

// Gradient-norm clipping: per-block sums of g^2 (FP64, fixed grid), then one
// block adds them in order and writes scale = min(1, clip / |g|) (1 for a zero
// or non-finite norm is not used: a non-finite norm gives scale 0, so the step
// leaves the weights unchanged).
constexpr int kClipBlocks = 256;
__global__ void __launch_bounds__(TPB) k_sumsq(const float *__restrict__ g, long N, double *__restrict__ part)
{
    __shared__ double sh[TPB];
    double s = 0.0;
    for (long q = (long)blockIdx.x * TPB + threadIdx.x; q < N; q += (long)gridDim.x * TPB) s += (double)g[q] * g[q];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = TPB / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ void k_clip_scale(const double *__restrict__ part, int nbk, float clip, float *__restrict__ scale,
                             float *__restrict__ norm_out)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double s = 0.0;
    for (int b = 0; b < nbk; ++b) s += part[b];
    const double nrm = sqrt(s);
    norm_out[0] = (float)nrm;
    scale[0] = !isfinite(nrm) ? 0.0f : (nrm > (double)clip ? (float)((double)clip / nrm) : 1.0f);
}

// Adam (FP32) on the gradient times *gscale (1 without clipping):
// p -= lr * mhat / (sqrt(vhat) + eps)
__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m, float *__restrict__ v,
                       long N, float lr, float b1, float b2, float eps, float c1, float c2,
                       const float *__restrict__ gscale)
{
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= N) return;
    const float gq = g[q] * gscale[0];
    const float mq = b1 * m[q] + (1.0f - b1) * gq;
    const float vq = b2 * v[q] + (1.0f - b2) * gq * gq;
    m[q] = mq;
    v[q] = vq;
    p[q] -= lr * (mq / c1) / (sqrtf(vq / c2) + eps);
}

// He-normal initialisation from a counter-based generator: splitmix64 of
// (seed, index) -> two uniforms -> Box-Muller.
__device__ __forceinline__ unsigned long long splitmix64(unsigned long long x)
{
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}
__global__ void k_init_normal(float *__restrict__ p, long N, float stddev, unsigned long long seed)
{
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= N) return;
    const unsigned long long r = splitmix64(seed ^ splitmix64((unsigned long long)q));
    const double u1 = ((r >> 11) + 1.0) * (1.0 / 9007199254740993.0);
    const double u2 = (splitmix64(r) >> 11) * (1.0 / 9007199254740992.0);
    p[q] = (float)(stddev * sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2));
}

__global__ void k_zero_f32(float *__restrict__ p, long N)
{
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < N) p[q] = 0.0f;
}
__global__ void k_zero_bf16(bf16 *__restrict__ p, long N)
{
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < N) p[q] = (bf16)0.0f;
}

unsigned nb(long count) { return (unsigned)((count + TPB - 1) / TPB); }

thread_local std::string u_err;
int ufail(int code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
int ufail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    u_err = buf;
    return code;
}
#define UHIP(expr)                                                                                    \
    do {                                                                                              \
        hipError_t e_ = (expr);                                                                       \
        if (e_ != hipSuccess) return ufail(GR_EDEVICE, "%s: %s", #expr, hipGetErrorString(e_));       \
    } while (0)
#define ULAUNCH()                                                                                     \
    do {                                                                                              \
        hipError_t e_ = hipGetLastError();                                                            \
        if (e_ != hipSuccess) return ufail(GR_EDEVICE, "kernel launch: %s", hipGetErrorString(e_));   \
    } while (0)

int pad32(int k) { return (k + 31) / 32 * 32; }

constexpr int kWgradBlocks = 64; // most partial sums of a weight gradient of 128 x 64 channels

constexpr int kWgradRows = 512;  // most partial sums of any
static_assert(kWgradRows * 64 <= 32 * 32 * 32, "the bias partials fit one channel of the smallest grid");

// k_conv3 with the channel steps unrolled for the counts that networks have
template <int NT, int VG, bool RELU, bool BIAS, typename... A>
void launch_conv_ks(hipStream_t s, dim3 grid, int cin, const bf16 *in, A... a)
{
    switch (cin) {
    case 16: k_conv3<NT, VG, 16, 1, RELU, BIAS><<<grid, 256, 0, s>>>(in, cin, a...); return;
    case 32: k_conv3<NT, VG, 32, 1, RELU, BIAS><<<grid, 256, 0, s>>>(in, cin, a...); return;
    case 48: k_conv3<NT, VG, 16, 3, RELU, BIAS><<<grid, 256, 0, s>>>(in, cin, a...); return;
    case 64: k_conv3<NT, VG, 32, 2, RELU, BIAS><<<grid, 256, 0, s>>>(in, cin, a...); return;
    case 96: k_conv3<NT, VG, 32, 3, RELU, BIAS><<<grid, 256, 0, s>>>(in, cin, a...); return;
    case 128: k_conv3<NT, VG, 32, 4, RELU, BIAS><<<grid, 256, 0, s>>>(in, cin, a...); return;
    default: k_conv3<NT, VG, 16, 0, RELU, BIAS><<<grid, 256, 0, s>>>(in, cin, a...);
    }
}

template <bool RELU, bool BIAS>
bool launch_conv_t(hipStream_t s, int cout, const bf16 *in, int cin, int ics, int icoff, const bf16 *w, int kpad,
                   const float *bias, bf16 *out, int ocs, int ocoff, int n)
{
    const long N = (long)n * n * n;
    if (cin % 16 || N % 64 || N >= (1L << 31)) return false;
    if (cout != 16 && cout != 32 && cout != 48 && cout != 64 && cout != 96 && cout != 128) return false;
    if (n % 16 == 0) {
        // 32 channels a block balance LDS reads and products; 16 where the chip would
        // have fewer than four blocks a CU otherwise
        const unsigned gl = (unsigned)((n / 16) * (n / 4) * (n / 4));
        const bool two = cout % 32 == 0 && gl * (cout / 32) >= 1024;
        // 16 -> 16 channels: blocks march over up to four tiles in z while the chip keeps
        // eight a CU; the weights and staging addresses are formed once
        int zt = 1;
        if (cin == 16 && cout == 16)
            while (zt < 4 && n / 4 % (2 * zt) == 0 && gl / (2 * zt) >= 2048) zt *= 2;
        const dim3 grid(gl / zt, cout / (two ? 32 : 16));
#define CONV_LDS(NT, CW, MARCH)                                                                                    \
    k_conv3_lds<NT, CW, MARCH, RELU, BIAS><<<grid, 256, 0, s>>>(in, cin, ics, icoff, w, kpad, bias, out, ocs, ocoff, n, zt)
        if (cin % 32 == 0) {
            if (two) CONV_LDS(2, 32, false);
            else CONV_LDS(1, 32, false);
        } else {
            if (two) CONV_LDS(2, 16, false);
            else if (zt > 1) CONV_LDS(1, 16, true);
            else CONV_LDS(1, 16, false);
        }
#undef CONV_LDS
        return true;
    }
    // two groups of voxels and 32 channels a wave where that leaves two blocks a CU
    if (cout % 32 == 0 && N % 128 == 0 && N / 128 * (cout / 32) >= 512)
        launch_conv_ks<2, 2, RELU, BIAS>(s, dim3((unsigned)(N / 128), cout / 32), cin, in, ics, icoff, w, kpad, bias, out,
                                         ocs, ocoff, n);
    else
        launch_conv_ks<1, 1, RELU, BIAS>(s, dim3((unsigned)(N / 64), cout / 16), cin, in, ics, icoff, w, kpad, bias, out,
                                         ocs, ocoff, n);
    return true;
}

} // namespace

// ------------------------------------------------------------------ network

struct ConvLayer {
    int cin, cout, kpad, kpadT;
    long w_off, b_off; // offsets into the FP32 parameter vector
    bf16 *wf = nullptr, *wt = nullptr;
};

struct Act { // one channels-last BF16 tensor
    bf16 *p = nullptr;
    int n = 0, c = 0;
};

struct gr_unet_s {
    gr_unet_desc d{};
    int max_n = 0;
    int c[4];
    ConvLayer conv[14]; // e0a e0b e1a e1b e2a e2b e3a e3b d2a d2b d1a d1b d0a d0b
    long head_w = 0, head_b = 0;
    long nparam = 0;
    // device
    float *param = nullptr, *grad = nullptr, *adam_m = nullptr, *adam_v = nullptr;
    float *loss_partial = nullptr, *y = nullptr, *gy = nullptr, *lq = nullptr;
    float *wg_part = nullptr, *wg_bpart = nullptr; // weight-gradient block partials
    double *gn_part = nullptr;                       // gradient-norm block partials
    float *gscale = nullptr;
    bf16 *x0 = nullptr;
    Act ea[4], eb3, cat[3], p[3], da[3], db[3];       // forward
    Act g_ea[4], g_eb3, g_cat[3], g_p[3], g_da[3], g_db[3], g_x; // backward
    size_t ws_bytes = 0;
    hipStream_t stream = nullptr;
    bool bound = false;
    long step = 0;
};

namespace {

enum { E0A, E0B, E1A, E1B, E2A, E2B, E3A, E3B, D2A, D2B, D1A, D1B, D0A, D0B };

size_t unet_layout(gr_unet U, char *base)
{
    size_t off = 0;
    auto take = [&](size_t bytes) -> char * {
        char *p = base ? base + off : nullptr;
        off += (bytes + 255) / 256 * 256;
        return p;
    };
    auto takeF = [&](size_t n) { return reinterpret_cast<float *>(take(sizeof(float) * n)); };
    auto takeB = [&](size_t n) { return reinterpret_cast<bf16 *>(take(sizeof(bf16) * n)); };
    U->param = takeF(U->nparam);
    U->grad = takeF(U->nparam);
    U->adam_m = takeF(U->nparam);
    U->adam_v = takeF(U->nparam);
    for (auto &L : U->conv) {
        L.wf = takeB((size_t)L.cout * L.kpad);
        L.wt = takeB((size_t)L.cin * L.kpadT);
    }
    const int n = U->max_n;
    const long N = (long)n * n * n;
    U->loss_partial = takeF(2048);
    U->gn_part = reinterpret_cast<double *>(take(sizeof(double) * kClipBlocks));
    U->gscale = takeF(2); // [0] clip scale of the gradient, [1] its norm
    // block partials of the weight gradients: the 3^3 convolutions' (64 blocks x 27
    // taps x cout x cin) or the head's (one block per 256 voxels x its parameters)
    const size_t head_part = (size_t)((N + TPB - 1) / TPB) * (size_t)(U->d.out_ch * U->c[0] + U->d.out_ch);
    U->wg_part = takeF(std::max((size_t)kWgradBlocks * 27 * WG_MAXC * 64, head_part));
    U->y = takeF((size_t)U->d.out_ch * N);
    U->gy = takeF((size_t)U->d.out_ch * N);
    U->lq = takeF((size_t)U->d.out_ch * N);
    U->wg_bpart = U->lq; // the loss has read its Laplacian before the backward pass starts
    U->x0 = takeB((size_t)N * 16);
    auto act = [&](Act &a, int lvl, int ch) {
        a.n = n >> lvl;
        a.c = ch;
        a.p = takeB((size_t)a.n * a.n * a.n * ch);
    };
    const int *c = U->c;
    for (int k = 0; k < 4; ++k) act(U->ea[k], k, c[k]);
    act(U->eb3, 3, c[3]);
    for (int k = 0; k < 3; ++k) {
        act(U->cat[k], k, c[k + 1] + c[k]);
        act(U->p[k], k + 1, c[k]);
        act(U->da[k], k, c[k]);
        act(U->db[k], k, c[k]);
        act(U->g_cat[k], k, c[k + 1] + c[k]);
        act(U->g_p[k], k + 1, c[k]);
        act(U->g_da[k], k, c[k]);
        act(U->g_db[k], k, c[k]);
    }
    for (int k = 0; k < 4; ++k) act(U->g_ea[k], k, c[k]);
    act(U->g_eb3, 3, c[3]);
    act(U->g_x, 0, 16);
    return off;
}

int conv_fwd(gr_unet U, int li, const bf16 *in, int ics, int icoff, bf16 *out, int ocs, int ocoff, int n)
{
    const ConvLayer &L = U->conv[li];
    if (!launch_conv_t<true, true>(U->stream, L.cout, in, L.cin, ics, icoff, L.wf, L.kpad, U->param + L.b_off, out,
                                   ocs, ocoff, n))
        return ufail(GR_EINVAL, "unsupported channel count %d", L.cout);
    ULAUNCH();
    return GR_OK;
}

// input gradient of layer li: gin = conv(gout, flipped/transposed weights)
int conv_dgrad(gr_unet U, int li, const bf16 *gout, int gcs, int gcoff, bf16 *gin, int n)
{
    const ConvLayer &L = U->conv[li];
    if (!launch_conv_t<false, false>(U->stream, L.cin, gout, L.cout, gcs, gcoff, L.wt, L.kpadT, nullptr, gin, L.cin,
                                     0, n))
        return ufail(GR_EINVAL, "unsupported channel count %d", L.cin);
    ULAUNCH();
    return GR_OK;
}

int conv_wgrad(gr_unet U, int li, const bf16 *gout, int gcs, int gcoff, const bf16 *in, int ics, int icoff, int n)
{
    const ConvLayer &L = U->conv[li];
    const long N = (long)n * n * n;
    if (N % 64 || n % 4 || L.cout % 16 || L.cin % 16 || L.cout > 64 || L.cin > WG_MAXC)
        return ufail(GR_EINVAL, "weight gradient: unsupported shape (n %d, cin %d, cout %d)", n, L.cin, L.cout);
    // a tile of 16 x 4 x 4 voxels where the side has them; 32 channels of a side where they
    // divide it; as many partial sums as give the chip two blocks a CU, but no more than
    // there is room for (kWgradBlocks x 128 x 64) or tiles
    const int tw = n % 16 == 0 ? 16 : n % 8 == 0 ? 8 : 4;
    const int co = L.cout % 32 ? 16 : 32, ci = L.cin % 32 ? 16 : 32, cb = L.cout / co * (L.cin / ci);
    const long room = (long)kWgradBlocks * WG_MAXC * 64 / ((long)L.cout * L.cin);
    const int nbk = (int)std::min({(long)(512 + cb - 1) / cb, N / (16 * tw), room, (long)kWgradRows});
    const dim3 grid((unsigned)nbk, (unsigned)cb);
#define WGRAD(TX, CO, CI)                                                                                        \
    k_conv3_wgrad<TX, CO, CI><<<grid, TPB, 0, U->stream>>>(gout, L.cout, gcs, gcoff, in, L.cin, ics, icoff,     \
                                                           U->wg_part, U->wg_bpart, n)
#define WGRAD_X(CO, CI)                                                                                          \
    do {                                                                                                        \
        if (tw == 16) WGRAD(16, CO, CI);                                                                         \
        else if (tw == 8) WGRAD(8, CO, CI);                                                                      \
        else WGRAD(4, CO, CI);                                                                                   \
    } while (0)
    if (co == 32 && ci == 32) WGRAD_X(32, 32);
    else if (co == 32) WGRAD_X(32, 16);
    else if (ci == 32) WGRAD_X(16, 32);
    else WGRAD_X(16, 16);
#undef WGRAD_X
#undef WGRAD
    const long per = 27L * L.cout * L.cin;
    k_wgrad_reduce<<<(unsigned)(per / 128) + 1, TPB, 0, U->stream>>>(U->wg_part, U->wg_bpart, nbk, L.cout, L.cin,
                                                                 U->grad + L.w_off, U->grad + L.b_off);
    ULAUNCH();
    return GR_OK;
}

int relu_bwd(gr_unet U, bf16 *g, int gcs, int gcoff, const bf16 *a, int acs, int acoff, int c, int n)
{
    const long N = (long)n * n * n;
    k_relu_bwd<<<nb(N * (c / 8)), TPB, 0, U->stream>>>(g, gcs, gcoff, a, acs, acoff, c, N);
    ULAUNCH();
    return GR_OK;
}

#define UCHK(expr)                                                                                    \
    do {                                                                                              \
        int st_ = (expr);                                                                             \
        if (st_ != GR_OK) return st_;                                                                 \
    } while (0)

int refresh_weights(gr_unet U)
{
    for (auto &L : U->conv) {
        const long tot = std::max((long)L.cout * L.kpad, (long)L.cin * L.kpadT);
        k_prep_weights<<<nb(tot), TPB, 0, U->stream>>>(U->param + L.w_off, L.cout, L.cin, L.kpad, L.kpadT, L.wf, L.wt);
    }
    ULAUNCH();
    return GR_OK;
}

// forward pass for an n^3 input (planar FP32 [in_ch][n^3]) -> U->y
int forward(gr_unet U, int n, const float *d_in)
{
    hipStream_t s = U->stream;
    const long N = (long)n * n * n;
    const int *c = U->c;
    k_pack_input<<<nb(N), TPB, 0, s>>>(d_in, U->d.in_ch, U->x0, N);
    ULAUNCH();
    // encoder
    UCHK(conv_fwd(U, E0A, U->x0, 16, 0, U->ea[0].p, c[0], 0, n));
    UCHK(conv_fwd(U, E0B, U->ea[0].p, c[0], 0, U->cat[0].p, c[1] + c[0], c[1], n));
    const bf16 *prev = nullptr;
    for (int k = 0; k < 3; ++k) {
        const int nk = n >> k, nk1 = nk >> 1;
        // pool the skip channels of cat[k]
        k_pool<<<nb((long)nk1 * nk1 * nk1 * (c[k] / 8)), TPB, 0, s>>>(U->cat[k].p, c[k + 1] + c[k], c[k + 1], c[k], U->p[k].p, nk);
        ULAUNCH();
        const int la = E1A + 2 * k, lb = E1B + 2 * k;
        UCHK(conv_fwd(U, la, U->p[k].p, c[k], 0, U->ea[k + 1].p, c[k + 1], 0, nk1));
        if (k < 2) UCHK(conv_fwd(U, lb, U->ea[k + 1].p, c[k + 1], 0, U->cat[k + 1].p, c[k + 2] + c[k + 1], c[k + 2], nk1));
        else UCHK(conv_fwd(U, lb, U->ea[3].p, c[3], 0, U->eb3.p, c[3], 0, nk1));
    }
    (void)prev;
    // decoder
    for (int k = 2; k >= 0; --k) {
        const int nk = n >> k;
        const Act &src = (k == 2) ? U->eb3 : U->db[k + 1];
        k_upsample<<<nb((long)nk * nk * nk * (src.c / 8)), TPB, 0, s>>>(src.p, src.c, U->cat[k].p, c[k + 1] + c[k], nk);
        ULAUNCH();
        const int la = D2A + 2 * (2 - k), lb = D2B + 2 * (2 - k);
        UCHK(conv_fwd(U, la, U->cat[k].p, c[k + 1] + c[k], 0, U->da[k].p, c[k], 0, nk));
        UCHK(conv_fwd(U, lb, U->da[k].p, c[k], 0, U->db[k].p, c[k], 0, nk));
    }
    k_head<<<nb(N), TPB, 0, s>>>(U->db[0].p, U->param + U->head_w, U->param + U->head_b, U->y, U->d.out_ch, N);
    ULAUNCH();
    return GR_OK;
}

// backward pass (after forward and k_mse filled U->gy): accumulates U->grad
int backward(gr_unet U, int n)
{
    hipStream_t s = U->stream;
    const long N = (long)n * n * n;
    const int *c = U->c;
    {
        const int nw = U->d.out_ch * c[0], npar = nw + U->d.out_ch;
        const unsigned nblk = nb(N);
        k_head_bwd<<<nblk, TPB, 0, s>>>(U->gy, U->db[0].p, U->param + U->head_w, U->d.out_ch, U->g_db[0].p,
                                        U->wg_part, N);
        k_head_reduce<<<(unsigned)npar, TPB, 0, s>>>(U->wg_part, (int)nblk, npar, nw, U->grad + U->head_w,
                                                     U->grad + U->head_b);
        ULAUNCH();
    }
    // decoder, fine to coarse: each level's concat gradient feeds the next coarser output
    for (int k = 0; k <= 2; ++k) {
        const int nk = n >> k;
        const int la = D2A + 2 * (2 - k), lb = D2B + 2 * (2 - k);
        const int C = c[k + 1] + c[k];
        UCHK(relu_bwd(U, U->g_db[k].p, c[k], 0, U->db[k].p, c[k], 0, c[k], nk));
        UCHK(conv_wgrad(U, lb, U->g_db[k].p, c[k], 0, U->da[k].p, c[k], 0, nk));
        UCHK(conv_dgrad(U, lb, U->g_db[k].p, c[k], 0, U->g_da[k].p, nk));
        UCHK(relu_bwd(U, U->g_da[k].p, c[k], 0, U->da[k].p, c[k], 0, c[k], nk));
        UCHK(conv_wgrad(U, la, U->g_da[k].p, c[k], 0, U->cat[k].p, C, 0, nk));
        UCHK(conv_dgrad(U, la, U->g_da[k].p, c[k], 0, U->g_cat[k].p, nk));
        // upsampled channels [0, c[k+1]) -> gradient of the coarser output
        const int m = nk / 2;
        bf16 *dst = (k == 2) ? U->g_eb3.p : U->g_db[k + 1].p;
        k_upsample_bwd<<<nb((long)m * m * m * c[k + 1]), TPB, 0, s>>>(U->g_cat[k].p, C, c[k + 1], dst, nk);
        ULAUNCH();
    }
    // bottleneck
    {
        const int n3 = n >> 3;
        UCHK(relu_bwd(U, U->g_eb3.p, c[3], 0, U->eb3.p, c[3], 0, c[3], n3));
        UCHK(conv_wgrad(U, E3B, U->g_eb3.p, c[3], 0, U->ea[3].p, c[3], 0, n3));
        UCHK(conv_dgrad(U, E3B, U->g_eb3.p, c[3], 0, U->g_ea[3].p, n3));
        UCHK(relu_bwd(U, U->g_ea[3].p, c[3], 0, U->ea[3].p, c[3], 0, c[3], n3));
        UCHK(conv_wgrad(U, E3A, U->g_ea[3].p, c[3], 0, U->p[2].p, c[2], 0, n3));
        UCHK(conv_dgrad(U, E3A, U->g_ea[3].p, c[3], 0, U->g_p[2].p, n3));
    }
    // encoder, coarse to fine: skip gradient = decoder part (in g_cat) + pooling part
    for (int k = 2; k >= 0; --k) {
        const int nk = n >> k;
        const int C = c[k + 1] + c[k];
        k_pool_bwd_add<<<nb((long)nk * nk * nk * (c[k] / 8)), TPB, 0, s>>>(U->g_p[k].p, c[k], U->g_cat[k].p, C, c[k + 1], nk);
        ULAUNCH();
        const int la = E0A + 2 * k, lb = E0B + 2 * k;
        UCHK(relu_bwd(U, U->g_cat[k].p, C, c[k + 1], U->cat[k].p, C, c[k + 1], c[k], nk));
        UCHK(conv_wgrad(U, lb, U->g_cat[k].p, C, c[k + 1], U->ea[k].p, c[k], 0, nk));
        UCHK(conv_dgrad(U, lb, U->g_cat[k].p, C, c[k + 1], U->g_ea[k].p, nk));
        UCHK(relu_bwd(U, U->g_ea[k].p, c[k], 0, U->ea[k].p, c[k], 0, c[k], nk));
        if (k > 0) {
            UCHK(conv_wgrad(U, la, U->g_ea[k].p, c[k], 0, U->p[k - 1].p, c[k - 1], 0, nk));
            UCHK(conv_dgrad(U, la, U->g_ea[k].p, c[k], 0, U->g_p[k - 1].p, nk));
        } else {
            UCHK(conv_wgrad(U, la, U->g_ea[0].p, c[0], 0, U->x0, 16, 0, nk));
        }
    }
    return GR_OK;
}

// forward + MSE loss + backward; loss (mean square) returned on the host
int loss_and_grad(gr_unet U, int n, const float *d_in, const float *d_target, double *h_loss)
{
    const long N = (long)n * n * n;
    k_zero_f32<<<nb(U->nparam), TPB, 0, U->stream>>>(U->grad, U->nparam);
    ULAUNCH();
    UCHK(forward(U, n, d_in));
    const long tot = (long)U->d.out_ch * N;
    const int nbk = (int)std::min<long>(1024, (tot + TPB - 1) / TPB);
    k_mse<<<nbk, TPB, 0, U->stream>>>(U->y, d_target, U->gy, tot, U->loss_partial);
    const float lam = U->d.lap_weight;
    if (lam > 0.0f) {
        k_lap_loss1<<<nbk, TPB, 0, U->stream>>>(U->y, d_target, U->lq, n, tot, U->loss_partial + 1024);
        k_lap_loss2<<<nbk, TPB, 0, U->stream>>>(U->lq, U->gy, n, tot, lam);
    }
    ULAUNCH();
    UCHK(backward(U, n));
    if (h_loss) {
        std::vector<float> part(2 * 1024, 0.0f);
        UHIP(hipMemcpyAsync(part.data(), U->loss_partial, sizeof(float) * nbk, hipMemcpyDeviceToHost, U->stream));
        if (lam > 0.0f)
            UHIP(hipMemcpyAsync(part.data() + 1024, U->loss_partial + 1024, sizeof(float) * nbk,
                                hipMemcpyDeviceToHost, U->stream));
        UHIP(hipStreamSynchronize(U->stream));
        double acc = 0.0, accl = 0.0;
        for (int i = 0; i < nbk; ++i) {
            acc += part[i];
            accl += part[1024 + i];
        }
        *h_loss = (acc + (double)lam * accl) / (double)tot;
    }
    return GR_OK;
}

int check_n(gr_unet U, int n)
{
    if (!U || !U->bound) return ufail(U ? GR_ESTATE : GR_EINVAL, "network not bound");
    if (n < 32 || n % 32 || n > U->max_n) return ufail(GR_EINVAL, "n = %d must be a multiple of 32, <= %d", n, U->max_n);
    return GR_OK;
}

} // namespace

extern "C" {

const char *gr_unet_last_error(void) { return u_err.c_str(); }

int gr_unet_create(const gr_unet_desc *d, int max_n, gr_unet *out)
{
    if (!d || !out) return ufail(GR_EINVAL, "null argument");
    *out = nullptr;
    if (d->in_ch < 1 || d->in_ch > 16 || d->out_ch < 1 || d->out_ch > 16)
        return ufail(GR_EINVAL, "in_ch and out_ch must be 1..16");
    if (!(d->lap_weight >= 0.0f) || !std::isfinite(d->lap_weight))
        return ufail(GR_EINVAL, "lap_weight must be finite and >= 0");
    if (!(d->clip_norm >= 0.0f) || !std::isfinite(d->clip_norm))
        return ufail(GR_EINVAL, "clip_norm must be finite and >= 0");
    if (d->c[0] != 16) return ufail(GR_EINVAL, "c[0] must be 16");
    for (int k = 1; k < 4; ++k)
        if (d->c[k] < 16 || d->c[k] > 64 || d->c[k] % 16) return ufail(GR_EINVAL, "c[%d] must be 16, 32, 48 or 64", k);
    if (max_n < 32 || max_n % 32 || max_n > 512) return ufail(GR_EINVAL, "max_n must be a multiple of 32 up to 512");
    gr_unet U = new (std::nothrow) gr_unet_s();
    if (!U) return ufail(GR_EINVAL, "out of host memory");
    U->d = *d;
    U->max_n = max_n;
    for (int k = 0; k < 4; ++k) U->c[k] = d->c[k];
    const int *c = U->c;
    const int io[14][2] = {{16, c[0]}, {c[0], c[0]}, {c[0], c[1]}, {c[1], c[1]}, {c[1], c[2]}, {c[2], c[2]},
                           {c[2], c[3]}, {c[3], c[3]}, {c[3] + c[2], c[2]}, {c[2], c[2]}, {c[2] + c[1], c[1]},
                           {c[1], c[1]}, {c[1] + c[0], c[0]}, {c[0], c[0]}};
    long off = 0;
    for (int l = 0; l < 14; ++l) {
        ConvLayer &L = U->conv[l];
        L.cin = io[l][0];
        L.cout = io[l][1];
        L.kpad = pad32(27 * L.cin);
        L.kpadT = pad32(27 * L.cout);
        L.w_off = off;
        off += (long)L.cout * 27 * L.cin;
        L.b_off = off;
        off += L.cout;
    }
    U->head_w = off;
    off += (long)d->out_ch * c[0];
    U->head_b = off;
    off += d->out_ch;
    U->nparam = off;
    U->ws_bytes = unet_layout(U, nullptr);
    *out = U;
    return GR_OK;
}

int gr_unet_workspace_bytes(gr_unet U, size_t *bytes)
{
    if (!U || !bytes) return ufail(GR_EINVAL, "null argument");
    *bytes = U->ws_bytes;
    return GR_OK;
}

int gr_unet_param_count(gr_unet U, int64_t *count)
{
    if (!U || !count) return ufail(GR_EINVAL, "null argument");
    *count = U->nparam;
    return GR_OK;
}

int gr_unet_bind(gr_unet U, void *d_ws, size_t bytes, void *stream)
{
    if (!U || !d_ws) return ufail(GR_EINVAL, "null argument");
    if (bytes < U->ws_bytes) return ufail(GR_EINVAL, "workspace %zu bytes < required %zu", bytes, U->ws_bytes);
    if (reinterpret_cast<uintptr_t>(d_ws) % 256) return ufail(GR_EINVAL, "workspace not 256-byte aligned");
    U->stream = reinterpret_cast<hipStream_t>(stream);
    unet_layout(U, reinterpret_cast<char *>(d_ws));
    const long nw = (long)(U->ws_bytes / sizeof(float));
    k_zero_f32<<<nb(nw), TPB, 0, U->stream>>>(reinterpret_cast<float *>(d_ws), nw);
    ULAUNCH();
    U->bound = true;
    U->step = 0;
    return GR_OK;
}

// He-normal weights (std sqrt(2 / fan_in)), zero biases, zero Adam moments.
int gr_unet_init(gr_unet U, uint64_t seed)
{
    if (!U || !U->bound) return ufail(U ? GR_ESTATE : GR_EINVAL, "network not bound");
    hipStream_t s = U->stream;
    k_zero_f32<<<nb(U->nparam), TPB, 0, s>>>(U->param, U->nparam);
    k_zero_f32<<<nb(U->nparam), TPB, 0, s>>>(U->adam_m, U->nparam);
    k_zero_f32<<<nb(U->nparam), TPB, 0, s>>>(U->adam_v, U->nparam);
    for (int l = 0; l < 14; ++l) {
        const ConvLayer &L = U->conv[l];
        const long cnt = (long)L.cout * 27 * L.cin;
        k_init_normal<<<nb(cnt), TPB, 0, s>>>(U->param + L.w_off, cnt, std::sqrt(2.0f / (27.0f * L.cin)),
                                             seed * 1000003ull + l);
    }
    const long hc = (long)U->d.out_ch * U->c[0];
    k_init_normal<<<nb(hc), TPB, 0, s>>>(U->param + U->head_w, hc, std::sqrt(1.0f / U->c[0]), seed * 1000003ull + 99);
    ULAUNCH();
    U->step = 0;
    return refresh_weights(U);
}

int gr_unet_set_params(gr_unet U, const float *d_src)
{
    if (!U || !U->bound || !d_src) return ufail(GR_EINVAL, "bad argument");
    UHIP(hipMemcpyAsync(U->param, d_src, sizeof(float) * U->nparam, hipMemcpyDeviceToDevice, U->stream));
    return refresh_weights(U);
}

int gr_unet_get_params(gr_unet U, float *d_dst)
{
    if (!U || !U->bound || !d_dst) return ufail(GR_EINVAL, "bad argument");
    UHIP(hipMemcpyAsync(d_dst, U->param, sizeof(float) * U->nparam, hipMemcpyDeviceToDevice, U->stream));
    return GR_OK;
}

int gr_unet_forward(gr_unet U, int n, const float *d_in, float *d_out)
{
    int st = check_n(U, n);
    if (st) return st;
    if (!d_in || !d_out) return ufail(GR_EINVAL, "null tensor");
    UCHK(forward(U, n, d_in));
    const long N = (long)n * n * n;
    UHIP(hipMemcpyAsync(d_out, U->y, sizeof(float) * U->d.out_ch * N, hipMemcpyDeviceToDevice, U->stream));
    return GR_OK;
}

int gr_unet_loss_grad(gr_unet U, int n, const float *d_in, const float *d_target, float *d_grad, double *h_loss)
{
    int st = check_n(U, n);
    if (st) return st;
    if (!d_in || !d_target) return ufail(GR_EINVAL, "null tensor");
    UCHK(loss_and_grad(U, n, d_in, d_target, h_loss));
    if (d_grad)
        UHIP(hipMemcpyAsync(d_grad, U->grad, sizeof(float) * U->nparam, hipMemcpyDeviceToDevice, U->stream));
    return GR_OK;
}

int gr_unet_train_step(gr_unet U, int n, const float *d_in, const float *d_target, float lr, double *h_loss)
{
    int st = check_n(U, n);
    if (st) return st;
    if (!d_in || !d_target || !(lr > 0.0f)) return ufail(GR_EINVAL, "bad argument");
    UCHK(loss_and_grad(U, n, d_in, d_target, h_loss));
    ++U->step;
    const float b1 = 0.9f, b2 = 0.999f;
    const float clip = U->d.clip_norm > 0.0f ? U->d.clip_norm : 3.4e38f;
    k_sumsq<<<kClipBlocks, TPB, 0, U->stream>>>(U->grad, U->nparam, U->gn_part);
    k_clip_scale<<<1, 64, 0, U->stream>>>(U->gn_part, kClipBlocks, clip, U->gscale, U->gscale + 1);
    k_adam<<<nb(U->nparam), TPB, 0, U->stream>>>(U->param, U->grad, U->adam_m, U->adam_v, U->nparam, lr, b1, b2, 1e-8f,
                                                1.0f - std::pow(b1, (float)U->step), 1.0f - std::pow(b2, (float)U->step),
                                                U->gscale);
    ULAUNCH();
    return refresh_weights(U);
}

int gr_destroy_unet(gr_unet U)
{
    delete U;
    return GR_OK;
}

} // extern "C"
