// Learned correction kernels: 3-D convolutions on MFMA (bfloat16 in, FP32
// accumulate), weight gradients, loss, packing and Adam.
//
// MFMA tile (v_mfma_f32_16x16x16_bf16, one wavefront): A is 16 x 16 (rows x
// k), B is 16 x 16 (k x cols), D = A B + C is 16 x 16 FP32.  Lane l holds
// A[l % 16][4 (l / 16) + 0..3], B[4 (l / 16) + 0..3][l % 16] and
// D[4 (l / 16) + 0..3][l % 16].
//
// Convolution as 27 accumulated tile products: rows = the 16 output channels,
// k = the 16 input channels at one tap, cols = 16 consecutive cells along x.
// A wavefront owns one 16-cell segment of an x-row; each lane keeps its
// weights of the layer in registers.  The padding
// layer of every activation buffer is zero, so taps that leave the grid read
// zeros; cells past the ragged row end are neither read nor written.

#include <algorithm>

#include "learned.h"

namespace dm {
namespace {

constexpr int kT = 256;  // threads per block (4 wavefronts)

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// A workgroup computes one tile of 16 x kTileY x kTileZ cells: the input
// cells of the tile and its one-cell halo (18 x (kTileY + 2) x (kTileZ + 2),
// 16 channels each) are staged in LDS once, so each activation is fetched
// from memory about twice instead of once per tap; wave w then takes the
// x-segments of y-row w, one z-plane after another.  Cells outside the padded
// grid are staged as zeros (the padding layer itself holds zeros).  Each
// wave keeps the layer's weights for its lanes in registers (27 x 8 bytes),
// and staged cells sit 48 bytes apart, so that the 8-byte reads of half a
// wavefront (16 cells x 2 channel groups) fall on 64 distinct banks.
constexpr int kTileY = 4, kTileZ = 8;
constexpr int kTileCells = 18 * (kTileY + 2) * (kTileZ + 2);
constexpr int kCellStride = 3;   // in 16-byte units (32 bytes of data, 16 of padding)

template <int MODE>
__global__ void __launch_bounds__(kT)
k_net_conv(Grid g, const uint16_t *__restrict__ in, const uint16_t *__restrict__ w,
           const uint16_t *__restrict__ mask, uint16_t *__restrict__ out_bf, float *__restrict__ out_f) {
    static_assert(kT / 64 == kTileY, "one wave per y-row of the tile");
    __shared__ uint4 xs[kTileCells * kCellStride];
    const int nsx = (g.nx + 15) >> 4, nty = (g.ny + kTileY - 1) / kTileY;
    // each XCD (workgroups reach them round-robin) takes one run of tiles, so
    // that neighbours share their halos in its L2
    const uint32_t per = gridDim.x / 8, b = blockIdx.x % 8 * per + blockIdx.x / 8;
    const int sx = (int)(b % nsx), rest = (int)(b / nsx);
    const int j0 = rest % nty * kTileY, k0 = rest / nty * kTileZ;
    if (k0 >= g.nz) return;   // the grid is padded to a multiple of 8
    const int i0 = sx * 16;
    // a wave stages every fourth row of the tile: 18 cells are 576 contiguous
    // bytes, 36 lanes of 16; all its rows are in flight before the first is
    // written (cells outside the padded grid are zero)
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    constexpr int kRows = (kTileY + 2) * (kTileZ + 2), kMine = (kRows + kT / 64 - 1) / (kT / 64);
    static_assert(kRows % (kT / 64) == 0, "rows dealt evenly to the waves");
    const bool on = lane < 36 && i0 - 1 + (lane >> 1) <= g.nx;
    uint4 rows[kMine];
#pragma unroll
    for (int m = 0; m < kMine; ++m) {
        const int r = wv + m * (kT / 64), j = j0 - 1 + r % (kTileY + 2), k = k0 - 1 + r / (kTileY + 2);
        rows[m] = make_uint4(0u, 0u, 0u, 0u);
        if (on && j <= g.ny && k <= g.nz)
            rows[m] = reinterpret_cast<const uint4 *>(in + pidx(g, i0 - 1, j, k) * kNetCh)[lane];
    }
    // this lane's A operands: output channel col, input channels 4 kg .. 4 kg + 3, every tap
    const int col = lane & 15, kg = lane >> 4;
    uint2 wr[27];
#pragma unroll
    for (int t = 0; t < 27; ++t) wr[t] = *reinterpret_cast<const uint2 *>(w + t * 256 + col * 16 + 4 * kg);
    if (lane < 36)
#pragma unroll
        for (int m = 0; m < kMine; ++m)
            xs[((wv + m * (kT / 64)) * 18 + (lane >> 1)) * kCellStride + (lane & 1)] = rows[m];
    __syncthreads();
    const int j = j0 + wv;
    if (j >= g.ny) return;
    const int ia = i0 + col;
    const bool va = ia < g.nx;
    const uint2 *xs2 = reinterpret_cast<const uint2 *>(xs);
    // D = W X: rows the output channels (A = the tap's weights, row = output
    // channel, k = input channel), columns the 16 cells (B = the inputs, k =
    // input channel, column = cell); lane (col, kg) ends with output channels
    // 4 kg .. 4 kg + 3 of cell i0 + col, stored as one 8-byte write (a
    // wavefront writes the segment's 512 contiguous bytes).
    // The wave marches through the input planes of its y-row: the nine
    // operands of a plane (three rows, three shifts along x) are read once and
    // serve the last nine taps of the output plane below, the middle nine of
    // the plane itself and the first nine of the one above, three independent
    // chains of products; each output still sums its taps in order.  Reading
    // all 27 operands per output plane kept the LDS as busy as the matrix
    // cores (72 us per layer at 128^3, 61 with this); staging by rows instead
    // of by cells, with its index arithmetic in scalars, took it to 49 us.
    auto load = [&](uint2 *v, int zp) __attribute__((always_inline)) {   // input plane k0 - 1 + zp
#pragma unroll
        for (int r = 0; r < 9; ++r)
            v[r] = xs2[((col + r % 3) + 18 * ((wv + r / 3) + (kTileY + 2) * zp)) * (2 * kCellStride) + kg];
    };
    auto store = [&](const f32x4 &a, int k) __attribute__((always_inline)) {
        if (!va) return;
        const int64_t p = pidx(g, ia, j, k);
        if (MODE == NET_LINEAR) {
            if (kg == 0) *reinterpret_cast<float4 *>(out_f + p * 4) = make_float4(a[0], a[1], a[2], a[3]);
            return;
        }
        uint16_t o[4];
        if (MODE == NET_RELU) {
#pragma unroll
            for (int r = 0; r < 4; ++r) o[r] = f2bf(a[r] > 0.f ? a[r] : 0.f);
        } else {
            const uint2 mraw = *reinterpret_cast<const uint2 *>(mask + p * kNetCh + 4 * kg);
            const uint16_t *m = reinterpret_cast<const uint16_t *>(&mraw);
#pragma unroll
            for (int r = 0; r < 4; ++r) o[r] = f2bf(bf2f(m[r]) > 0.f ? a[r] : 0.f);
        }
        *reinterpret_cast<uint2 *>(out_bf + p * kNetCh + 4 * kg) =
            make_uint2((uint32_t)o[0] | ((uint32_t)o[1] << 16), (uint32_t)o[2] | ((uint32_t)o[3] << 16));
    };
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 below = zero, here = zero;   // output planes zp - 2 and zp - 1 (of the tile) when plane zp is read
    uint2 v[2][9];
    load(v[0], 0);
#pragma unroll
    for (int zp = 0; zp < kTileZ + 2; ++zp) {
        if (zp + 1 < kTileZ + 2) load(v[(zp + 1) & 1], zp + 1);
        f32x4 above = zero;
#pragma unroll
        for (int r = 0; r < 9; ++r) {
            const bf16x4 bx = *reinterpret_cast<const bf16x4 *>(&v[zp & 1][r]);
            if (zp >= 2)
                below = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const bf16x4 *>(&wr[18 + r]), bx,
                                                                  below, 0, 0, 0);
            if (zp >= 1 && zp <= kTileZ)
                here = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const bf16x4 *>(&wr[9 + r]), bx,
                                                                 here, 0, 0, 0);
            if (zp < kTileZ)
                above = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const bf16x4 *>(&wr[r]), bx, above,
                                                                  0, 0, 0);
        }
        if (zp >= 2 && k0 + zp - 2 < g.nz) store(below, k0 + zp - 2);
        below = here;
        here = above;
    }
}

// Weight gradient: per tap, D[c][o] += sum over 16 cells of x[cell + off][c] d[cell][o]
// (A = x^T: rows c, k = cells; B = d: k = cells, cols o).  The products take
// consecutive cells of one channel per lane, while memory holds consecutive
// channels of one cell, so a workgroup transposes a tile (that of the
// convolution, x with its halo) into LDS once, channel rows of 24 values
// (48 bytes: a wavefront's 8-byte reads fall on distinct banks), and every
// operand is an aligned read; the two taps shifted along x come from the
// same read and its neighbours by 16-bit funnel shifts.  A wave takes one
// y-row of the tile and keeps the 27 products in registers over all its
// tiles; the four waves are summed in LDS, so a workgroup leaves one partial.
// Gathering the cells lane by lane from memory (four 2-byte loads per tap)
// took 105 us per layer at 64^3, and summing its 1,024 partials 15 us; now
// 19 and 5.5 us.
constexpr int kGradRow = 24;   // values per channel row: cells i0 - 1 .. i0 + 16 at 3 .. 20

__global__ void __launch_bounds__(kT, 2)
k_net_wgrad(Grid g, const uint16_t *__restrict__ x, const uint16_t *__restrict__ d, float *__restrict__ part) {
    constexpr int kRowsX = (kTileY + 2) * (kTileZ + 2), kRowsD = kTileY * kTileZ;
    __shared__ __align__(16) uint16_t xs[kRowsX * 16 * kGradRow], ds[kRowsD * 16 * kGradRow];
    static_assert(sizeof(xs) >= 27 * 256 * sizeof(float), "the waves' sum reuses the tile");
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 15, kg = lane >> 4;
    const int nsx = (g.nx + 15) >> 4, nty = (g.ny + kTileY - 1) / kTileY, ntz = (g.nz + kTileZ - 1) / kTileZ;
    const int ntiles = nsx * nty * ntz;
    f32x4 acc[27];
#pragma unroll
    for (int t = 0; t < 27; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int i0 = (tile % nsx) * 16, rest = tile / nsx, j0 = (rest % nty) * kTileY, k0 = (rest / nty) * kTileZ;
        __syncthreads();   // the tile before is used up
        for (int e = threadIdx.x; e < kTileCells * 2; e += kT) {
            const int c = e >> 1, half = e & 1;
            const int xi = c % 18, row = c / 18, yi = row % (kTileY + 2), zi = row / (kTileY + 2);
            const int i = i0 - 1 + xi, j = j0 - 1 + yi, k = k0 - 1 + zi;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (i <= g.nx && j <= g.ny && k <= g.nz)
                v = reinterpret_cast<const uint4 *>(x + pidx(g, i, j, k) * kNetCh)[half];
            uint16_t *dst = xs + (row * 16 + 8 * half) * kGradRow + xi + 3;
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int m = 0; m < 8; ++m) dst[m * kGradRow] = (uint16_t)(w[m >> 1] >> (16 * (m & 1)));
        }
        for (int e = threadIdx.x; e < 16 * kRowsD * 2; e += kT) {
            const int c = e >> 1, half = e & 1;
            const int xi = c & 15, row = c >> 4, i = i0 + xi, j = j0 + row % kTileY, k = k0 + row / kTileY;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (i < g.nx && j < g.ny && k < g.nz)
                v = reinterpret_cast<const uint4 *>(d + pidx(g, i, j, k) * kNetCh)[half];
            uint16_t *dst = ds + (row * 16 + 8 * half) * kGradRow + xi;
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int m = 0; m < 8; ++m) dst[m * kGradRow] = (uint16_t)(w[m >> 1] >> (16 * (m & 1)));
        }
        __syncthreads();
        for (int zz = 0; zz < kTileZ; ++zz) {
            const uint2 draw = *reinterpret_cast<const uint2 *>(ds + ((wv + kTileY * zz) * 16 + col) * kGradRow + 4 * kg);
            const bf16x4 b = *reinterpret_cast<const bf16x4 *>(&draw);
#pragma unroll
            for (int r9 = 0; r9 < 9; ++r9) {
                const int dy = r9 % 3 - 1, dz = r9 / 3 - 1, row = (wv + 1 + dy) + (kTileY + 2) * (zz + 1 + dz);
                const uint16_t *src = xs + (row * 16 + col) * kGradRow + 4 + 4 * kg;
                const uint2 own = *reinterpret_cast<const uint2 *>(src);
                const uint32_t prev = *reinterpret_cast<const uint32_t *>(src - 2);
                const uint32_t next = *reinterpret_cast<const uint32_t *>(src + 4);
                const uint32_t mid = __builtin_amdgcn_alignbit(own.y, own.x, 16);
                const uint2 lo = make_uint2(__builtin_amdgcn_alignbit(own.x, prev, 16), mid);
                const uint2 hi = make_uint2(mid, __builtin_amdgcn_alignbit(next, own.y, 16));
                acc[3 * r9] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const bf16x4 *>(&lo), b,
                                                                        acc[3 * r9], 0, 0, 0);
                acc[3 * r9 + 1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const bf16x4 *>(&own), b,
                                                                            acc[3 * r9 + 1], 0, 0, 0);
                acc[3 * r9 + 2] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const bf16x4 *>(&hi), b,
                                                                            acc[3 * r9 + 2], 0, 0, 0);
            }
        }
    }
    float *red = reinterpret_cast<float *>(xs);
    for (int w = 0; w < kT / 64; ++w) {
        __syncthreads();
        if (wv == w) {
#pragma unroll
            for (int t = 0; t < 27; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float *q = red + t * 256 + (4 * kg + r) * 16 + col;
                    *q = w ? *q + acc[t][r] : acc[t][r];
                }
        }
    }
    __syncthreads();
    float *dst = part + (int64_t)blockIdx.x * 27 * 256;
    for (int e = threadIdx.x; e < 27 * 256; e += kT) dst[e] = red[e];
}

// grad of one layer from its partials: a workgroup per (tap, input channel),
// 16 threads along the output channels times 16 along the partials
__global__ void __launch_bounds__(kT)
k_net_wgrad_reduce(const float *__restrict__ part, int nparts, int cin, int cout, float *__restrict__ grad) {
    const int t = blockIdx.x / 16, c = blockIdx.x % 16, o = threadIdx.x & 15, q = threadIdx.x >> 4;
    if (c >= cin) return;
    __shared__ float red[16][17];
    float s = 0.f;
#pragma unroll 8
    for (int w = q; w < nparts; w += 16) s += part[(int64_t)w * 27 * 256 + t * 256 + c * 16 + o];
    red[q][o] = s;
    __syncthreads();
    if (q == 0 && o < cout) {
        float tot = 0.f;
#pragma unroll
        for (int w = 0; w < 16; ++w) tot += red[w][o];
        grad[(t * cin + c) * cout + o] = tot;
    }
}

template <class T>
__global__ void __launch_bounds__(kT)
k_net_pack_r(Grid g, const T *__restrict__ r, double inv_s, const double *__restrict__ ss, double inv_cnt,
             uint16_t *__restrict__ x0) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    const int64_t t = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (t >= n) return;
    if (ss) {
        // the scale from a sum of squares on the device: s = sqrt(ss * inv_cnt)
        const double sc = sqrt(ss[0] * inv_cnt);
        inv_s = sc > 0.0 ? 1.0 / sc : 0.0;
    }
    const int i = (int)(t % g.nx);
    const int64_t q = t / g.nx;
    const int j = (int)(q % g.ny), k = (int)(q / g.ny);
    const int64_t p = pidx(g, i, j, k);
#pragma unroll
    for (int c = 0; c < 3; ++c) x0[p * kNetCh + c] = f2bf((float)((double)r[c * g.P + p] * inv_s));
}

template <class T>
__global__ void __launch_bounds__(kT)
k_net_unpack(Grid g, const T *__restrict__ coef, const float *__restrict__ y, double scale,
             const double *__restrict__ ss, double inv_cnt, T *__restrict__ out) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    const int64_t t = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (t >= n) return;
    if (ss) scale *= sqrt(ss[0] * inv_cnt);
    const int i = (int)(t % g.nx);
    const int64_t q = t / g.nx;
    const int j = (int)(q % g.ny), k = (int)(q / g.ny);
    const int64_t p = pidx(g, i, j, k);
#pragma unroll
    for (int c = 0; c < 3; ++c)
        put_face<T>(g, out + c * g.P, c, i, j, k, p,
                    coef[c * g.P + p] != T(0) ? (T)((double)y[p * 4 + c] * scale) : T(0));
}

__global__ void __launch_bounds__(kT)
k_net_loss(Grid g, const double *__restrict__ coef, const float *__restrict__ y, const double *__restrict__ e,
           double t_scale, double inv_norm, uint16_t *__restrict__ dy, double *__restrict__ part, int pass) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    double s_err = 0.0, s_t = 0.0;
    for (int64_t t = (int64_t)blockIdx.x * kT + threadIdx.x; t < n; t += (int64_t)gridDim.x * kT) {
        const int i = (int)(t % g.nx);
        const int64_t q = t / g.nx;
        const int j = (int)(q % g.ny), k = (int)(q / g.ny);
        const int64_t p = pidx(g, i, j, k);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if (coef[c * g.P + p] == 0.0) {
                if (pass == 1) dy[p * kNetCh + c] = 0;
                continue;
            }
            const double tv = e[c * g.P + p] * t_scale;
            if (pass == 0) {
                s_t += tv * tv;
            } else {
                const double diff = (double)y[p * 4 + c] - tv;
                s_err += diff * diff;
                dy[p * kNetCh + c] = f2bf((float)(2.0 * diff * inv_norm));
            }
        }
    }
    __shared__ double red[2][kT];
    red[0][threadIdx.x] = s_err;
    red[1][threadIdx.x] = s_t;
    __syncthreads();
    for (int w = kT / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            red[0][threadIdx.x] += red[0][threadIdx.x + w];
            red[1][threadIdx.x] += red[1][threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = red[0][0];
        part[2 * blockIdx.x + 1] = red[1][0];
    }
}

// dy channel c = bf16(g_c * factor) on active faces, 0 elsewhere
__global__ void __launch_bounds__(kT)
k_net_dy_from_face(Grid g, const double *__restrict__ coef, const double *__restrict__ gv, double factor,
                   uint16_t *__restrict__ dy) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    const int64_t t = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (t >= n) return;
    const int i = (int)(t % g.nx);
    const int64_t q = t / g.nx;
    const int j = (int)(q % g.ny), k = (int)(q / g.ny);
    const int64_t p = pidx(g, i, j, k);
#pragma unroll
    for (int c = 0; c < 3; ++c)
        dy[p * kNetCh + c] = coef[c * g.P + p] != 0.0 ? f2bf((float)(gv[c * g.P + p] * factor)) : (uint16_t)0;
}

// wf[l][t][o][c] = bf16(W_l[t][c][o]);  wb[l][t][c][o] = bf16(W_l[26 - t][c][o])
// (the data gradient is the forward conv of d with the flipped taps and the
// roles of in and out channels exchanged); zero-padded to 16 x 16.
__global__ void __launch_bounds__(kT)
k_net_pack_weights(const float *__restrict__ w32, uint16_t *__restrict__ wf, uint16_t *__restrict__ wb) {
    const int l = blockIdx.x / 27, t = blockIdx.x % 27;
    const int a = threadIdx.x / 16, b = threadIdx.x % 16;   // row, column of the 16 x 16 tile
    const int cin = kNetIn[l], cout = kNetOut[l];
    int64_t base = 0;
    for (int q = 0; q < l; ++q) base += 27 * kNetIn[q] * kNetOut[q];
    // forward: row = out channel a, column = in channel b
    const float vf = (b < cin && a < cout) ? w32[base + (t * cin + b) * cout + a] : 0.f;
    wf[((int64_t)l * 27 + t) * 256 + a * 16 + b] = f2bf(vf);
    // data gradient: row = in channel a of the layer (its output), column = out channel b
    const float vb = (a < cin && b < cout) ? w32[base + ((26 - t) * cin + a) * cout + b] : 0.f;
    wb[((int64_t)l * 27 + t) * 256 + a * 16 + b] = f2bf(vb);
}

// Adam (Kingma & Ba, Algorithm 1); c1 = 1 - b1^step, c2 = 1 - b2^step
__global__ void __launch_bounds__(kT)
k_net_adam(const float *__restrict__ g, float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
           int n, float lr, float b1, float b2, float eps, float c1, float c2) {
    const int q = blockIdx.x * kT + threadIdx.x;
    if (q >= n) return;
    const float gq = g[q];
    const float mq = b1 * m[q] + (1.f - b1) * gq;
    const float vq = b2 * v[q] + (1.f - b2) * gq * gq;
    m[q] = mq;
    v[q] = vq;
    w[q] -= lr * (mq / c1) / (sqrtf(vq / c2) + eps);
}

}  // namespace

namespace {
inline int net_tiles(const Grid &g) {
    return (int)(ceil_div(g.nx, 16) * ceil_div(g.ny, kTileY) * ceil_div(g.nz, kTileZ));
}
inline int net_parts(const Grid &g) { return std::min(kNetParts, net_tiles(g)); }
}  // namespace

void launch_net_conv(int mode, const Grid &g, const uint16_t *in, const uint16_t *w, const uint16_t *mask,
                     uint16_t *out_bf, float *out_f, hipStream_t s) {
    // one workgroup per tile of 16 x kTileY x kTileZ cells, padded to the XCDs
    const dim3 grid((unsigned)(ceil_div(net_tiles(g), 8) * 8));
    if (mode == NET_RELU)
        hipLaunchKernelGGL(k_net_conv<NET_RELU>, grid, dim3(kT), 0, s, g, in, w, mask, out_bf, out_f);
    else if (mode == NET_MASKED)
        hipLaunchKernelGGL(k_net_conv<NET_MASKED>, grid, dim3(kT), 0, s, g, in, w, mask, out_bf, out_f);
    else
        hipLaunchKernelGGL(k_net_conv<NET_LINEAR>, grid, dim3(kT), 0, s, g, in, w, mask, out_bf, out_f);
}

void launch_net_wgrad(const Grid &g, const uint16_t *x, const uint16_t *d, float *part, hipStream_t s) {
    hipLaunchKernelGGL(k_net_wgrad, dim3((unsigned)net_parts(g)), dim3(kT), 0, s, g, x, d, part);
}

void launch_net_wgrad_reduce(const Grid &g, const float *part, int cin, int cout, float *grad, hipStream_t s) {
    hipLaunchKernelGGL(k_net_wgrad_reduce, dim3(27 * 16), dim3(kT), 0, s, part, net_parts(g), cin, cout, grad);
}

template <class T>
void launch_net_pack_r(const Grid &g, const T *r, double inv_s, uint16_t *x0, hipStream_t s) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    hipLaunchKernelGGL(k_net_pack_r<T>, dim3((unsigned)ceil_div(n, kT)), dim3(kT), 0, s, g, r, inv_s,
                       (const double *)nullptr, 0.0, x0);
}

void launch_net_pack_r_dev(const Grid &g, const double *r, const double *ss, double inv_cnt, uint16_t *x0,
                           hipStream_t s) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    hipLaunchKernelGGL(k_net_pack_r<double>, dim3((unsigned)ceil_div(n, kT)), dim3(kT), 0, s, g, r, 0.0, ss,
                       inv_cnt, x0);
}

template <class T>
void launch_net_unpack(const Grid &g, const T *coef, const float *y, double scale, T *out, hipStream_t s) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    hipLaunchKernelGGL(k_net_unpack<T>, dim3((unsigned)ceil_div(n, kT)), dim3(kT), 0, s, g, coef, y, scale,
                       (const double *)nullptr, 0.0, out);
}

void launch_net_unpack_dev(const Grid &g, const double *coef, const float *y, double h2, const double *ss,
                           double inv_cnt, double *out, hipStream_t s) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    hipLaunchKernelGGL(k_net_unpack<double>, dim3((unsigned)ceil_div(n, kT)), dim3(kT), 0, s, g, coef, y, h2, ss,
                       inv_cnt, out);
}

// The residual judge on the device: d[0] = |v - M z|^2, d[1] = |v - M (z +
// dz)|^2; z += dz when the correction lowers the residual (or the residual
// is already zero, where dz is zero as well); flag = whether it was kept.
// One workgroup per kThreads entries; every workgroup reads the same two
// numbers, workgroup 0 writes the flag.
__global__ void __launch_bounds__(kT)
k_net_accept(int64_t n, const double *__restrict__ d, const double *__restrict__ dz, double *__restrict__ z,
             int *__restrict__ flag) {
    const bool keep = d[1] < d[0] || d[0] == 0.0;
    const int64_t t = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (t == 0) *flag = keep ? 1 : 0;
    if (keep && t < n) z[t] += dz[t];
}

void launch_net_accept(int64_t n, const double *d, const double *dz, double *z, int *flag, hipStream_t s) {
    hipLaunchKernelGGL(k_net_accept, dim3((unsigned)ceil_div(n, kT)), dim3(kT), 0, s, n, d, dz, z, flag);
}

void launch_net_loss(const Grid &g, const double *coef, const float *y, const double *e, double t_scale,
                     double inv_norm, uint16_t *dy, double *part, int nblocks, int pass, hipStream_t s) {
    hipLaunchKernelGGL(k_net_loss, dim3(nblocks), dim3(kT), 0, s, g, coef, y, e, t_scale, inv_norm, dy, part, pass);
}

void launch_net_dy_from_face(const Grid &g, const double *coef, const double *gv, double factor, uint16_t *dy,
                             hipStream_t s) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    hipLaunchKernelGGL(k_net_dy_from_face, dim3((unsigned)ceil_div(n, kT)), dim3(kT), 0, s, g, coef, gv, factor, dy);
}

void launch_net_pack_weights(const float *w32, uint16_t *wf, uint16_t *wb, hipStream_t s) {
    hipLaunchKernelGGL(k_net_pack_weights, dim3(3 * 27), dim3(kT), 0, s, w32, wf, wb);
}

void launch_net_adam(const float *g, float *w, float *m, float *v, int n, float lr, float b1, float b2,
                     float eps, float c1, float c2, hipStream_t s) {
    hipLaunchKernelGGL(k_net_adam, dim3((unsigned)ceil_div(n, kT)), dim3(kT), 0, s, g, w, m, v, n, lr, b1, b2,
                       eps, c1, c2);
}

template void launch_net_pack_r<double>(const Grid &, const double *, double, uint16_t *, hipStream_t);
template void launch_net_pack_r<float>(const Grid &, const float *, double, uint16_t *, hipStream_t);
template void launch_net_unpack<double>(const Grid &, const double *, const float *, double, double *,
                                        hipStream_t);
template void launch_net_unpack<float>(const Grid &, const float *, const float *, double, float *, hipStream_t);

}  // namespace dm
