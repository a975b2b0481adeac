// Kernels of the learned initial-guess network (gfx950).
//
// Network: conv3x3x3(2->16) -> ReLU -> conv3x3x3(16->16) -> ReLU ->
// conv3x3x3(16->1), zero padding, same-size output.  Activations are
// channel-last [batch][z][y][x][c]; the weights of a layer are bfloat16
// [27 taps][cout][cin] with taps ordered (dz, dy, dx), dx fastest, offsets
// -1..1; biases FP32.  Training keeps FP32 master weights (Adam) and runs the
// convolutions with the bfloat16 weights and FP32 activations and
// accumulation; inference of the 16->16 layer runs on the matrix cores
// (bfloat16 x bfloat16 -> FP32 MFMA).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <mutex>
#include <type_traits>

#include "../../include/nested_poisson.h"
#include "np_internal.h"

namespace np {

namespace {

constexpr int kNB = 256;

__host__ __device__ inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// round to nearest even; NaN stays NaN
__device__ __forceinline__ uint16_t f32_to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x7fffffu)) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

template <typename T>
__device__ __forceinline__ float ld(const T* p);
template <>
__device__ __forceinline__ float ld<float>(const float* p) { return *p; }
template <>
__device__ __forceinline__ float ld<uint16_t>(const uint16_t* p) { return bf16_to_f32(*p); }

template <typename T>
__device__ __forceinline__ void st(T* p, float v);
template <>
__device__ __forceinline__ void st<float>(float* p, float v) { *p = v; }
template <>
__device__ __forceinline__ void st<uint16_t>(uint16_t* p, float v) { *p = f32_to_bf16(v); }

// ------------------------------------------------------------------ convolution, FP32 accumulate
// Thread per output voxel; the layer's weights are staged in LDS as FP32.
template <typename TI, typename TO>
__global__ void __launch_bounds__(kNB) k_conv_fwd(const TI* __restrict__ in, int cin, const uint16_t* __restrict__ w,
                                                 const float* __restrict__ bias, int cout, int relu, int B, int Z, int Y,
                                                 int X, TO* __restrict__ out)
{
    __shared__ float ws[27 * 16 * 16];
    const int nw = 27 * cout * cin;
    for (int i = threadIdx.x; i < nw; i += kNB) ws[i] = bf16_to_f32(w[i]);
    __syncthreads();
    const long nvox = (long)B * Z * Y * X;
    const long v = (long)blockIdx.x * kNB + threadIdx.x;
    if (v >= nvox) return;
    const int x = (int)(v % X);
    long r = v / X;
    const int y = (int)(r % Y);
    r /= Y;
    const int z = (int)(r % Z);
    const int b = (int)(r / Z);
    float acc[16];
    for (int o = 0; o < cout; o++) acc[o] = bias[o];
    int t = 0;
    for (int dz = -1; dz <= 1; dz++)
        for (int dy = -1; dy <= 1; dy++)
            for (int dx = -1; dx <= 1; dx++, t++) {
                const int zz = z + dz, yy = y + dy, xx = x + dx;
                if (zz < 0 || zz >= Z || yy < 0 || yy >= Y || xx < 0 || xx >= X) continue;
                const TI* src = in + ((((long)b * Z + zz) * Y + yy) * X + xx) * cin;
                const float* wt = ws + t * cout * cin;
                for (int i = 0; i < cin; i++) {
                    const float a = ld(src + i);
                    for (int o = 0; o < cout; o++) acc[o] = fmaf(wt[o * cin + i], a, acc[o]);
                }
            }
    TO* dst = out + v * cout;
    for (int o = 0; o < cout; o++) st(dst + o, relu ? fmaxf(acc[o], 0.0f) : acc[o]);
}

// The same convolution for the network's own channel counts, fixed at compile
// time: the accumulators stay in registers, the input channels of a tap come in
// with 8- to 16-byte loads and the outputs leave the same way.  Same
// arithmetic in the same order as k_conv_fwd.
template <int N, typename T>
__device__ __forceinline__ void ld_vec(const T* p, float (&a)[N])
{
    if constexpr (sizeof(T) == 2 && N % 8 == 0) {
#pragma unroll
        for (int q = 0; q < N / 8; q++) {
            const uint4 u = ((const uint4*)p)[q];
            const uint32_t w4[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int e = 0; e < 4; e++) {
                a[8 * q + 2 * e] = __uint_as_float(w4[e] << 16);
                a[8 * q + 2 * e + 1] = __uint_as_float(w4[e] & 0xffff0000u);
            }
        }
    } else if constexpr (sizeof(T) == 2 && N == 2) {
        const uint32_t u = *(const uint32_t*)p;
        a[0] = __uint_as_float(u << 16);
        a[1] = __uint_as_float(u & 0xffff0000u);
    } else if constexpr (sizeof(T) == 4 && N % 4 == 0) {
#pragma unroll
        for (int q = 0; q < N / 4; q++) {
            const float4 u = ((const float4*)p)[q];
            a[4 * q] = u.x;
            a[4 * q + 1] = u.y;
            a[4 * q + 2] = u.z;
            a[4 * q + 3] = u.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < N; i++) a[i] = ld(p + i);
    }
}

template <int N, typename T>
__device__ __forceinline__ void st_vec(T* p, const float (&a)[N])
{
    if constexpr (sizeof(T) == 2 && N % 8 == 0) {
#pragma unroll
        for (int q = 0; q < N / 8; q++) {
            uint32_t w4[4];
#pragma unroll
            for (int e = 0; e < 4; e++)
                w4[e] = (uint32_t)f32_to_bf16(a[8 * q + 2 * e]) | ((uint32_t)f32_to_bf16(a[8 * q + 2 * e + 1]) << 16);
            ((uint4*)p)[q] = make_uint4(w4[0], w4[1], w4[2], w4[3]);
        }
    } else if constexpr (sizeof(T) == 4 && N % 4 == 0) {
#pragma unroll
        for (int q = 0; q < N / 4; q++) ((float4*)p)[q] = make_float4(a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]);
    } else {
#pragma unroll
        for (int i = 0; i < N; i++) st(p + i, a[i]);
    }
}

template <int CIN, int COUT, typename TI, typename TO>
__global__ void __launch_bounds__(kNB) k_conv_fwd_t(const TI* __restrict__ in, const uint16_t* __restrict__ w,
                                                   const float* __restrict__ bias, int relu, int B, int Z, int Y, int X,
                                                   TO* __restrict__ out)
{
    __shared__ float ws[27 * COUT * CIN];
    for (int i = threadIdx.x; i < 27 * COUT * CIN; i += kNB) ws[i] = bf16_to_f32(w[i]);
    __syncthreads();
    const long nvox = (long)B * Z * Y * X;
    const long v = (long)blockIdx.x * kNB + threadIdx.x;
    if (v >= nvox) return;
    const int x = (int)(v % X);
    long r = v / X;
    const int y = (int)(r % Y);
    r /= Y;
    const int z = (int)(r % Z);
    const int b = (int)(r / Z);
    float acc[COUT];
#pragma unroll
    for (int o = 0; o < COUT; o++) acc[o] = bias[o];
    int t = 0;
    for (int dz = -1; dz <= 1; dz++)
        for (int dy = -1; dy <= 1; dy++)
            for (int dx = -1; dx <= 1; dx++, t++) {
                const int zz = z + dz, yy = y + dy, xx = x + dx;
                if (zz < 0 || zz >= Z || yy < 0 || yy >= Y || xx < 0 || xx >= X) continue;
                float a[CIN];
                ld_vec<CIN>(in + ((((long)b * Z + zz) * Y + yy) * X + xx) * CIN, a);
                const float* wt = ws + t * COUT * CIN;
#pragma unroll
                for (int i = 0; i < CIN; i++)
#pragma unroll
                    for (int o = 0; o < COUT; o++) acc[o] = fmaf(wt[o * CIN + i], a[i], acc[o]);
            }
    if (relu) {
#pragma unroll
        for (int o = 0; o < COUT; o++) acc[o] = fmaxf(acc[o], 0.0f);
    }
    st_vec<COUT>(out + v * COUT, acc);
}

// Data gradient: gin[v][i] = sum_taps sum_o w[t][o][i] * gout[v - tap][o].
__global__ void __launch_bounds__(kNB) k_conv_bwd_data(const float* __restrict__ gout, int cout,
                                                      const uint16_t* __restrict__ w, int cin, int B, int Z, int Y, int X,
                                                      float* __restrict__ gin)
{
    __shared__ float ws[27 * 16 * 16];
    const int nw = 27 * cout * cin;
    for (int i = threadIdx.x; i < nw; i += kNB) ws[i] = bf16_to_f32(w[i]);
    __syncthreads();
    const long nvox = (long)B * Z * Y * X;
    const long v = (long)blockIdx.x * kNB + threadIdx.x;
    if (v >= nvox) return;
    const int x = (int)(v % X);
    long r = v / X;
    const int y = (int)(r % Y);
    r /= Y;
    const int z = (int)(r % Z);
    const int b = (int)(r / Z);
    float acc[16];
    for (int i = 0; i < cin; i++) acc[i] = 0.0f;
    int t = 0;
    for (int dz = -1; dz <= 1; dz++)
        for (int dy = -1; dy <= 1; dy++)
            for (int dx = -1; dx <= 1; dx++, t++) {
                const int zz = z - dz, yy = y - dy, xx = x - dx;
                if (zz < 0 || zz >= Z || yy < 0 || yy >= Y || xx < 0 || xx >= X) continue;
                const float* g = gout + ((((long)b * Z + zz) * Y + yy) * X + xx) * cout;
                const float* wt = ws + t * cout * cin;
                for (int o = 0; o < cout; o++) {
                    const float go = g[o];
                    for (int i = 0; i < cin; i++) acc[i] = fmaf(wt[o * cin + i], go, acc[i]);
                }
            }
    float* dst = gin + v * cin;
    for (int i = 0; i < cin; i++) dst[i] = acc[i];
}

// Weight and bias gradients, first stage: block `blk` sums over the voxel rows
// blk, blk + gridDim.x, ... and writes its partial (27*cout*cin weights, then
// cout biases) to part[blk].  Each thread owns weight entries
// e = threadIdx.x, threadIdx.x + 256, ...; the row's inputs (3x3 neighbour
// rows with a one-voxel halo) and output gradients are staged in LDS.
constexpr int kRowMax = 64;  // longest row segment staged at once (longer rows are split)

__global__ void __launch_bounds__(kNB) k_conv_bwd_weight_part(const float* __restrict__ in, int cin,
                                                             const float* __restrict__ gout, int cout, int B, int Z,
                                                             int Y, int X, float* __restrict__ part)
{
    __shared__ float sin[9][kRowMax + 2][16];
    __shared__ float sg[kRowMax][16];
    const int nw = 27 * cout * cin;
    const int ne = nw + cout;
    float acc[28];  // ceil((27*16*16 + 16) / 256) = 28 entries per thread at most
    for (int q = 0; q < 28; q++) acc[q] = 0.0f;
    const int nseg = (X + kRowMax - 1) / kRowMax;
    const long nrows = (long)B * Z * Y * nseg;
    for (long row = blockIdx.x; row < nrows; row += gridDim.x) {
        const int seg = (int)(row % nseg);
        long rr = row / nseg;
        const int y = (int)(rr % Y);
        rr /= Y;
        const int z = (int)(rr % Z);
        const int b = (int)(rr / Z);
        const int x0 = seg * kRowMax;
        const int len = min(kRowMax, X - x0);
        __syncthreads();
        // stage 9 neighbour rows (dz, dy) with x in [x0-1, x0+len] and the output gradients
        for (int idx = threadIdx.x; idx < 9 * (len + 2) * cin; idx += kNB) {
            const int i = idx % cin;
            const int xs = (idx / cin) % (len + 2);
            const int nr = idx / (cin * (len + 2));
            const int zz = z + nr / 3 - 1, yy = y + nr % 3 - 1, xx = x0 + xs - 1;
            float vv = 0.0f;
            if (zz >= 0 && zz < Z && yy >= 0 && yy < Y && xx >= 0 && xx < X)
                vv = in[((((long)b * Z + zz) * Y + yy) * X + xx) * cin + i];
            sin[nr][xs][i] = vv;
        }
        for (int idx = threadIdx.x; idx < len * cout; idx += kNB) {
            const int o = idx % cout, xs = idx / cout;
            sg[xs][o] = gout[((((long)b * Z + z) * Y + y) * X + x0 + xs) * cout + o];
        }
        __syncthreads();
        int q = 0;
        for (int e = threadIdx.x; e < ne; e += kNB, q++) {
            float s = 0.0f;
            if (e < nw) {
                const int i = e % cin;
                const int o = (e / cin) % cout;
                const int t = e / (cin * cout);
                const int nr = t / 3, dx = t % 3;  // (dz, dy) row index and x offset + 1
                for (int xs = 0; xs < len; xs++) s = fmaf(sg[xs][o], sin[nr][xs + dx][i], s);
            } else {
                const int o = e - nw;
                for (int xs = 0; xs < len; xs++) s += sg[xs][o];
            }
            acc[q] += s;
        }
    }
    int q = 0;
    for (int e = threadIdx.x; e < ne; e += kNB, q++) part[(long)blockIdx.x * ne + e] = acc[q];
}

__global__ void k_relu_bwd(const float* __restrict__ act, float* __restrict__ g, long n)
{
    const long i = (long)blockIdx.x * kNB + threadIdx.x;
    if (i < n && !(act[i] > 0.0f)) g[i] = 0.0f;
}

// Masked mean squared error: grad = 2 mask (pred - target) / sum(mask), and
// per-block partial sums of mask (pred - target)^2 and of mask.
__global__ void k_mse(const float* __restrict__ pred, const float* __restrict__ target, const float* __restrict__ mask,
                      long n, float inv_count, float* __restrict__ grad, float* __restrict__ part)
{
    __shared__ float red[kNB];
    const long i = (long)blockIdx.x * kNB + threadIdx.x;
    float d = 0.0f;
    if (i < n) {
        const float m = mask ? mask[i] : 1.0f;
        const float diff = (pred[i] - target[i]) * m;
        grad[i] = 2.0f * diff * inv_count;
        d = diff * diff;
    }
    red[threadIdx.x] = d;
    __syncthreads();
    for (int s = kNB / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// out = scale * (part[0] + part[1] + ...), added one after another in that
// order by one wavefront: 64 partials at a time are loaded together and passed
// to the running sum lane by lane (a thread that loaded and added took 346 us
// for the 8583 partials of a 130^3 sample, all of it load latency).
__global__ void __launch_bounds__(64) k_sum(const float* __restrict__ part, int n, float scale, float* __restrict__ out)
{
    const int lane = threadIdx.x;
    float s = 0.0f, next = lane < n ? part[lane] : 0.0f;
    for (int i0 = 0; i0 < n; i0 += 64) {
        const float v = next;
        if (i0 + 64 + lane < n) next = part[i0 + 64 + lane];
        const int m = n - i0 < 64 ? n - i0 : 64;
        if (m == 64) {
#pragma unroll
            for (int e = 0; e < 64; e++) s += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), e));
        } else {
            for (int e = 0; e < m; e++) s += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), e));
        }
    }
    if (lane == 0) out[0] = s * scale;
}

// Adam (Kingma & Ba) with bias correction on FP32 master weights; the
// bfloat16 copy used by the convolutions is refreshed.
__global__ void k_adam(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
                       long n, float lr, float b1, float b2, float eps, float c1, float c2, uint16_t* __restrict__ wb)
{
    const long i = (long)blockIdx.x * kNB + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    w[i] = wi;
    if (wb) wb[i] = f32_to_bf16(wi);
}

__global__ void k_to_bf16(const float* __restrict__ a, uint16_t* __restrict__ b, long n)
{
    const long i = (long)blockIdx.x * kNB + threadIdx.x;
    if (i < n) b[i] = f32_to_bf16(a[i]);
}

// a = bfloat16(a), kept in FP32 storage: the training forward pass rounds its
// inputs and hidden activations as the bfloat16 inference path stores them
__global__ void k_round_bf16(float* __restrict__ a, long n)
{
    const long i = (long)blockIdx.x * kNB + threadIdx.x;
    if (i < n) a[i] = bf16_to_f32(f32_to_bf16(a[i]));
}

// out = h^2 lap(in) with the 7-point stencil of eqn:Laplacian3D (the sum of
// the six face neighbours minus six times the centre), zero outside the box;
// one channel, [batch][z][y][x].  The stencil is symmetric, so the same kernel
// applies its transpose in the backward pass of the residual objective.
__global__ void k_lap7(const float* __restrict__ in, int B, int Z, int Y, int X, float* __restrict__ out)
{
    const long v = (long)blockIdx.x * kNB + threadIdx.x;
    const long nv = (long)B * Z * Y * X;
    if (v >= nv) return;
    const int x = (int)(v % X);
    long r = v / X;
    const int y = (int)(r % Y);
    r /= Y;
    const int z = (int)(r % Z);
    float s = x > 0 ? in[v - 1] : 0.0f;
    s += x + 1 < X ? in[v + 1] : 0.0f;
    s += y > 0 ? in[v - X] : 0.0f;
    s += y + 1 < Y ? in[v + X] : 0.0f;
    s += z > 0 ? in[v - (long)X * Y] : 0.0f;
    s += z + 1 < Z ? in[v + (long)X * Y] : 0.0f;
    out[v] = s - 6.0f * in[v];
}

// ------------------------------------------------------------------ inference on the matrix cores
// v_mfma_f32_16x16x32 bf16: lane l = 16 q + r supplies A[row r][k 8q..+7] and
// B[k 8q..+7][col r], and receives D[rows 4q..+3][col r].  Rows are output channels
// (A: weights), columns 16 voxels along x (B: activations), so a lane ends with four
// neighbouring channels of a voxel and a wavefront stores 16 voxels in one piece.
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

// A layer of the inference path.  A wavefront owns 16 voxels along x and R rows and
// marches along z with the outputs of three planes in flight: the input rows of
// a plane come from memory straight into the B operand and are used for every
// output that they reach (three planes, up to three rows), so nothing is staged in
// LDS and no wavefront waits for another.  A row past an edge of the volume is a
// buffer of no bytes and a voxel past it an offset outside its row: they read zero.
//   CIN = 16: an input row is two operands, the taps dx = 0 and 1 (lanes q < 2 and
//     q >= 2, 8 channels each) and the tap dx = 2 (the other half zero); 72 products
//     per plane for 4 rows.
//   CIN = 2: the three input rows of an output row are one operand (q: dy, then dx and
//     channel; the fourth dx and q = 3 are zero): 12 products per plane.
// COUT = 1 pads the weight rows with zeros and writes FP32; COUT = 16 writes bfloat16.
//
// What bounds it: with 16 input channels the matrix cores (316 GFLOP issued per 258^3
// voxels, a third of it the zero halves and edges of blocks: 270 us at the 1.17 PFLOP/s
// that a large bf16 product reaches here) and, as much, memory (64 or 36 B per voxel);
// with 2 channels memory (36 B).  Measured, 2 -> 16 / 16 -> 16 / 16 -> 1 channels: 258^3
// voxels 208 / 360 / 243 us, 66^3 8.7 / 11.3 / 9.5, 18^3 4.7 / 4.5 / 4.6 (blocks of 16 x 4 x 4
// voxels staged in LDS, products of K = 16, a store per channel: 450 / 560 / 520,
// 8.7 / 15 / 19, 4.9 / 5.7 / 6.5 us).
constexpr int kCvWaves = 4;
constexpr unsigned kCvOob = 0x80000000u;
// With 16 input channels four rows per wavefront read 1.5 input rows per output row, two
// rows 2, but two give twice the wavefronts: from this many pieces of 16 x 16 voxels on
// four are faster (16 -> 16, two / four rows: 66^3 voxels, 1650 pieces, 11.1 / 12.7 us;
// 130^3, 10530, 48.7 / 41.4 us).  With 2 channels the rows share nothing: two.
constexpr long kCvLarge = 4096;

template <int CIN, int COUT, int R, typename TO>
__global__ void __launch_bounds__(64 * kCvWaves, CIN == 16 ? 2 : 6)
k_conv_mfma(const uint16_t* __restrict__ in, const uint16_t* __restrict__ w, const float* __restrict__ bias, int relu,
            int Z, int Y, int X, TO* __restrict__ out, int ntx, int nty, int ntz, int kz)
{
    constexpr int NA = CIN == 16 ? 18 : 3;           // A operands: (dz, dy, half) or dz
    constexpr int NF = CIN == 16 ? 2 * (R + 2) : R;  // B operands of a plane
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int t = (int)blockIdx.x;
    const int bx = t % ntx;
    t /= ntx;
    const int by = t % nty;
    t /= nty;
    const int bz = t % ntz, b = t / ntz;
    const int x0 = 16 * bx, y0 = R * (kCvWaves * by + wave), z0 = kz * bz, z1 = min(z0 + kz, Z) - 1;
    if (y0 >= Y) return;
    const bool wide = ((uintptr_t)out & 7) == 0;  // a voxel's four channels in one store

    // byte offsets of the lane's voxels: CIN = 16 in an input row, CIN = 2 in the rows of a
    // plane that the wavefront reads (voxels x0 + r - 1 .. + 2 of row y0 + j - 1 + q)
    constexpr int VB = CIN * 2;
    const unsigned row_bytes = (unsigned)X * VB;
    const auto x_off = [&](int x, bool on) -> unsigned { return on && x >= 0 && x < X ? (unsigned)(x * VB) : kCvOob; };
    const unsigned o01 = x_off(x0 + r - 1 + (q >> 1), true) + 16 * (q & 1), o2 = x_off(x0 + r + 1, q < 2) + 16 * (q & 1);
    const bool x_edge = x0 == 0 || x0 + 18 > X;
    const auto load = [&](v4u (&f)[NF], int iz) {
        const bool zin = iz >= 0 && iz < Z;
        const uint16_t* const plane = in + ((long)b * Z + iz) * (long)Y * X * CIN;
        if constexpr (CIN == 16) {
#pragma unroll
            for (int j = 0; j < R + 2; j++) {
                const int iy = y0 - 1 + j;
                const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)(plane + (long)iy * X * CIN), 0,
                                                                  zin && iy >= 0 && iy < Y ? (int)row_bytes : 0, 0x00027000);
                f[2 * j] = __builtin_amdgcn_raw_buffer_load_b128(rs, o01, 0, 0);
                f[2 * j + 1] = __builtin_amdgcn_raw_buffer_load_b128(rs, o2, 0, 0);
            }
        } else {
            const int yb = max(y0 - 1, 0), ny = min(y0 + R + 1, Y) - yb;
            const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)(plane + (long)yb * X * CIN), 0,
                                                              zin ? (int)(row_bytes * ny) : 0, 0x00027000);
#pragma unroll
            for (int j = 0; j < R; j++) {
                const int iy = y0 + j - 1 + q;
                const bool yin = q < 3 && iy >= 0 && iy < Y;
                if (x_edge) {
#pragma unroll
                    for (int e = 0; e < 3; e++) {
                        const unsigned o = x_off(x0 + r - 1 + e, yin);
                        f[j][e] = __builtin_amdgcn_raw_buffer_load_b32(rs, o == kCvOob ? o : o + (unsigned)(iy - yb) * row_bytes, 0, 0);
                    }
                } else {
                    // (the fourth voxel, outside the taps, is dropped before the product)
                    f[j] = __builtin_amdgcn_raw_buffer_load_b128(
                        rs, yin ? (unsigned)(iy - yb) * row_bytes + (unsigned)(x0 + r - 1) * VB : kCvOob, 0, 0);
                }
            }
        }
    };
    v4u fa[NF], fb[NF];
    load(fa, z0 - 1);
    load(fb, z0);

    // weights [tap][cout][cin]; the rows of channels past COUT zero
    v8bf aw[NA];
    const int wr = min(r, COUT - 1);
#pragma unroll
    for (int a = 0; a < NA; a++) {
        v4u u = {0, 0, 0, 0};
        if constexpr (CIN == 16) {
            const int tap = (a >> 1) * 3 + ((a & 1) ? 2 : q >> 1);  // a >> 1 = 3 dz + dy
            __builtin_memcpy(&u, w + (tap * COUT + wr) * 16 + 8 * (q & 1), 16);
            if ((a & 1) && q >= 2) u = v4u{0, 0, 0, 0};
        } else {
            for (int dx = 0; dx < 3; dx++) __builtin_memcpy((char*)&u + 4 * dx, w + ((9 * a + 3 * min(q, 2) + dx) * COUT + wr) * 2, 4);
            if (q == 3) u = v4u{0, 0, 0, 0};
        }
        if (r >= COUT) u = v4u{0, 0, 0, 0};
        aw[a] = __builtin_bit_cast(v8bf, u);
    }
    float bo[4];
#pragma unroll
    for (int k = 0; k < 4; k++) bo[k] = 4 * q + k < COUT ? bias[4 * q + k] : 0.0f;

    // outputs of planes iz - 1, iz and iz + 1
    v4f acc[3][R];
#pragma unroll
    for (int s = 0; s < 3; s++)
#pragma unroll
        for (int y = 0; y < R; y++) acc[s][y] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    const auto plane = [&](v4u (&f)[NF], int iz) {
        if constexpr (CIN == 2) {
#pragma unroll
            for (int y = 0; y < R; y++) f[y][3] = 0;
        }
#pragma unroll
        for (int s = 0; s < 3; s++) {
            if (iz - 1 + s < z0 || iz - 1 + s > z1) continue;  // another workgroup's plane
            if constexpr (CIN == 16) {
#pragma unroll
                for (int j = 0; j < R + 2; j++)
#pragma unroll
                    for (int h = 0; h < 2; h++)
#pragma unroll
                        for (int dy = 0; dy < 3; dy++) {
                            const int y = j - dy;
                            if (y < 0 || y >= R) continue;
                            acc[s][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[2 * (3 * (2 - s) + dy) + h],
                                                                                 __builtin_bit_cast(v8bf, f[2 * j + h]),
                                                                                 acc[s][y], 0, 0, 0);
                        }
            } else {
#pragma unroll
                for (int y = 0; y < R; y++)
                    acc[s][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[2 - s], __builtin_bit_cast(v8bf, f[y]), acc[s][y],
                                                                         0, 0, 0);
            }
        }
        const int z = iz - 1, x = x0 + r;
#pragma unroll
        for (int y = 0; y < R; y++) {
            const bool on = z >= z0 && z <= z1 && y0 + y < Y;
            TO* const row = out + (((long)b * Z + z) * Y + y0 + y) * (long)X * COUT;
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; k++) {
                v[k] = acc[0][y][k] + bo[k];
                if (relu) v[k] = fmaxf(v[k], 0.0f);
            }
            const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)row, 0, on ? (int)(X * COUT * sizeof(TO)) : 0, 0x00027000);
            if constexpr (COUT == 1) {
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[0]), rs, q == 0 && x < X ? (unsigned)x * 4 : kCvOob, 0, 0);
            } else if (wide) {
                const v4bf u = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, u), rs, x < X ? (unsigned)(x * 32 + 8 * q) : kCvOob, 0, 0);
            } else if (on && x < X) {
#pragma unroll
                for (int k = 0; k < 4; k++) st(row + x * COUT + 4 * q + k, v[k]);
            }
            acc[0][y] = acc[1][y];
            acc[1][y] = acc[2][y];
            acc[2][y] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        }
    };
    for (int iz = z0 - 1;; iz += 2) {
        plane(fa, iz);
        if (iz > z1) break;
        load(fa, iz + 2);
        plane(fb, iz + 1);
        if (iz + 1 > z1) break;
        load(fb, iz + 3);
    }
}

// ------------------------------------------------------------------ training on the FP32 matrix cores
// The convolutions of a training step with FP32 activations and gradients, for
// the network's own channel counts.  v_mfma_f32_16x16x4_f32 is a chain of four
// FP32 fused multiply-adds in the order of k (checked bit for bit against
// fmaf), so a forward output formed tap by tap and channel by channel has the
// bits of k_conv_fwd_t's: the activations that are rounded to bfloat16 next
// keep their values.  FP32 matrix products run at twice the rate of the vector
// unit (153 TFLOP/s measured), and one LDS read feeds 16 of them.
//
// Operand layout: lane l = 16 q + r supplies A[row r][k q] and B[k q][col r]
// and receives D[rows 4q .. 4q+3][col r].  Rows are output channels and columns
// 16 voxels along x, so a lane ends with four neighbouring channels of a voxel.
//
// A workgroup produces blocks of 16 (x) x 4 (y) x 4 (z) voxels, 4 rows of 16
// per wavefront, from a block of 18 x 6 x 6 voxels in LDS (zero outside the volume).
// Taps outside the volume are products with zero instead of being skipped; with a
// non-finite weight that would make NaN, so then the block is formed voxel by
// voxel as in k_conv_fwd_t (conv_voxel).
constexpr int kTSX = 18, kTSY = 6, kTSZ = 6, kTNV = kTSX * kTSY * kTSZ;
constexpr long kTrainBlocks = 768;  // three workgroups per CU (52 KB of LDS each) for 16 channels

struct ConvTile {
    int b, x0, y0, z0;
};

__device__ __forceinline__ ConvTile conv_tile(long id, int Z, int Y, int X)
{
    const int ntx = (X + 15) >> 4, nty = (Y + 3) >> 2, ntz = (Z + 3) >> 2;
    const int bx = (int)(id % ntx);
    id /= ntx;
    const int by = (int)(id % nty);
    id /= nty;
    return ConvTile{(int)(id / ntz), bx * 16, by * 4, (int)(id % ntz) * 4};
}

__host__ __device__ inline long conv_tiles(int B, int Z, int Y, int X)
{
    return (long)B * ((Z + 3) / 4) * ((Y + 3) / 4) * ((X + 15) / 16);
}

// element index of voxel lv (0 .. kTNV-1) of a block's input region, or -1 outside the volume
__device__ __forceinline__ long region_voxel(const ConvTile& T, int lv, int Z, int Y, int X)
{
    const int lx = lv % kTSX, ly = (lv / kTSX) % kTSY, lz = lv / (kTSX * kTSY);
    const int x = T.x0 - 1 + lx, y = T.y0 - 1 + ly, z = T.z0 - 1 + lz;
    if (x < 0 || x >= X || y < 0 || y >= Y || z < 0 || z >= Z) return -1;
    return (((long)T.b * Z + z) * Y + y) * X + x;
}

// Weight of output channel o from input channel i at the tap that reads the
// input at offset t (dz, dy, dx): the layer's own (forward), or for the data
// gradient, whose input is gout (channel i of it) and output gin (channel o),
// the mirrored tap of the transposed weights.
template <int CI, int CO, bool BWD>
__device__ __forceinline__ float tap_weight(const uint16_t* __restrict__ w, int t, int o, int i)
{
    return bf16_to_f32(BWD ? w[((26 - t) * CI + i) * CO + o] : w[(t * CO + o) * CI + i]);
}

// One channel of one output voxel by scalar arithmetic, taps outside the volume skipped.
template <int CI, int CO, bool BWD>
__device__ __forceinline__ float conv_voxel(const float* __restrict__ in, const uint16_t* __restrict__ w,
                                            const float* __restrict__ bias, int Z, int Y, int X, int b, int z, int y,
                                            int x, int o)
{
    float acc = BWD ? 0.0f : bias[o];
#pragma unroll 1
    for (int t = 0; t < 27; t++) {
        const int zz = z + t / 9 - 1, yy = y + t / 3 % 3 - 1, xx = x + t % 3 - 1;
        if (zz < 0 || zz >= Z || yy < 0 || yy >= Y || xx < 0 || xx >= X) continue;
        const float* src = in + ((((long)b * Z + zz) * Y + yy) * X + xx) * CI;
#pragma unroll 1
        for (int i = 0; i < CI; i++) acc = fmaf(tap_weight<CI, CO, BWD>(w, t, o, i), src[i], acc);
    }
    return acc;
}

// What follows the sums of a training convolution: forward, ReLU and the
// rounding to bfloat16 (kept in FP32) of a hidden layer; data gradient, the mask
// of the ReLU that produced the layer's input (act, may be null).
struct ConvPost {
    int relu, round;
    const float* act;
};

__device__ __forceinline__ float conv_post(float v, const ConvPost& P, float act)
{
    if (P.relu) v = fmaxf(v, 0.0f);
    if (P.round) v = bf16_to_f32(f32_to_bf16(v));
    if (P.act && !(act > 0.0f)) v = 0.0f;
    return v;
}

// the block voxel by voxel (a thread each): only with non-finite weights
template <int CI, int CO, bool BWD>
__device__ __forceinline__ void conv_block_scalar(const ConvTile& T, const float* __restrict__ in,
                                                  const uint16_t* __restrict__ w, const float* __restrict__ bias,
                                                  int Z, int Y, int X, const ConvPost& P, float* __restrict__ out)
{
    const int x = T.x0 + (int)(threadIdx.x & 15), y = T.y0 + (int)(threadIdx.x >> 4 & 3), z = T.z0 + (int)(threadIdx.x >> 6);
    if (x >= X || y >= Y || z >= Z) return;
    const long base = ((((long)T.b * Z + z) * Y + y) * X + x) * CO;
#pragma unroll 1
    for (int o = 0; o < CO; o++)
        out[base + o] = conv_post(conv_voxel<CI, CO, BWD>(in, w, bias, Z, Y, X, T.b, z, y, x, o), P,
                                  P.act ? P.act[base + o] : 0.0f);
}

__device__ __forceinline__ void store_row16(const ConvTile& T, int rid, int q, int r, int Z, int Y, int X, const v4f& acc,
                                            const ConvPost& P, float* __restrict__ out)
{
    const int x = T.x0 + r, y = T.y0 + (rid & 3), z = T.z0 + (rid >> 2);
    if (x >= X || y >= Y || z >= Z) return;
    const long base = ((((long)T.b * Z + z) * Y + y) * X + x) * 16 + 4 * q;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    if (P.act) a = *(const float4*)(P.act + base);
    *(float4*)(out + base) = make_float4(conv_post(acc[0], P, a.x), conv_post(acc[1], P, a.y), conv_post(acc[2], P, a.z),
                                         conv_post(acc[3], P, a.w));
}

// 16 -> 16 channels: the layer's forward pass, or its data gradient (BWD).  The
// 27 x 16 x 16 weights stay in registers (108 per lane) over the blocks a
// workgroup runs; a voxel's channels lie in LDS in the order 4 q + s for
// channel 4 s + q, so that one 16-byte read gives a lane its operands of four
// products.  Bound by the matrix cores (108 products of 32 cycles per row of 16
// voxels: 0.22 ms at 130^3 with the padding of its rows to 16): forward 592 ->
// 301 us, data gradient 2690 -> 288 us there, launch included.
constexpr int kTVS = 20;  // LDS floats per voxel: 16 channels, padded so that 8 voxels in a row meet different banks

template <bool BWD>
__global__ void __launch_bounds__(256, 3) k_conv16_mfma_f32(const float* __restrict__ in, const uint16_t* __restrict__ w,
                                                            const float* __restrict__ bias, int B, int Z, int Y, int X,
                                                            ConvPost P, float* __restrict__ out, long per_block)
{
    __shared__ __align__(16) float tile[kTNV * kTVS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, q = lane >> 4, r = lane & 15;
    float aw[27][4];
    bool bad = false;
    // the weights pass through LDS (read directly, a lane's 108 two-byte loads are strided)
    uint16_t* const wl = (uint16_t*)tile;
    for (int e = threadIdx.x; e < 27 * 256; e += 256) wl[e] = w[e];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 27; t++)
#pragma unroll
        for (int s = 0; s < 4; s++) {
            aw[t][s] = tap_weight<16, 16, BWD>(wl, t, r, 4 * s + q);
            bad = bad || !(fabsf(aw[t][s]) < INFINITY);
        }
    const bool scalar = __any(bad);  // the same in every wavefront
    v4f b0 = {0.f, 0.f, 0.f, 0.f};
    if (!BWD) b0 = v4f{bias[4 * q], bias[4 * q + 1], bias[4 * q + 2], bias[4 * q + 3]};
    const long ntiles = conv_tiles(B, Z, Y, X);
    const long first = (long)blockIdx.x * per_block;
    const long last = first + per_block < ntiles ? first + per_block : ntiles;
    for (long id = first; id < last; id++) {
        const ConvTile T = conv_tile(id, Z, Y, X);
        if (scalar) {
            conv_block_scalar<16, 16, BWD>(T, in, w, bias, Z, Y, X, P, out);
            continue;
        }
        __syncthreads();  // the previous block's operands have been read
        for (int v = threadIdx.x; v < kTNV; v += 256) {
            const long g = region_voxel(T, v, Z, Y, X);
            float4 c0 = make_float4(0.f, 0.f, 0.f, 0.f), c1 = c0, c2 = c0, c3 = c0;
            if (g >= 0) {
                const float4* src = (const float4*)(in + g * 16);
                c0 = src[0];
                c1 = src[1];
                c2 = src[2];
                c3 = src[3];
            }
            float4* dst = (float4*)(tile + v * kTVS);
            dst[0] = make_float4(c0.x, c1.x, c2.x, c3.x);
            dst[1] = make_float4(c0.y, c1.y, c2.y, c3.y);
            dst[2] = make_float4(c0.z, c1.z, c2.z, c3.z);
            dst[3] = make_float4(c0.w, c1.w, c2.w, c3.w);
        }
        __syncthreads();
        // the wavefront's four rows (y = 0 .. 3 of plane `wave`), two at a time
#pragma unroll 1
        for (int p = 0; p < 4; p += 2) {
            const float* t0 = tile + ((wave * kTSY + p) * kTSX + r) * kTVS + 4 * q;
            v4f acc0 = b0, acc1 = b0;
#pragma unroll
            for (int t = 0; t < 27; t++) {
                const int off = ((t / 9 * kTSY + t / 3 % 3) * kTSX + t % 3) * kTVS;
                const v4f u0 = *(const v4f*)(t0 + off), u1 = *(const v4f*)(t0 + off + kTSX * kTVS);
#pragma unroll
                for (int s = 0; s < 4; s++) {
                    acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(aw[t][s], u0[s], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(aw[t][s], u1[s], acc1, 0, 0, 0);
                }
            }
            store_row16(T, wave * 4 + p, q, r, Z, Y, X, acc0, P, out);
            store_row16(T, wave * 4 + p + 1, q, r, Z, Y, X, acc1, P, out);
        }
    }
}

// 1 or 2 -> 16 channels: forward of the first layer (CI = 2), data gradient of
// the last (CI = 1).  K is (tap, channel), four per product: 14 or 7 products per
// row of 16 voxels; a lane's tap differs by q, so it keeps the LDS offset of
// each of its products.  Bound by the 16-channel output (141 MB at 130^3): forward 99 ->
// 76 us, data gradient 249 -> 44 us.
template <int CI, bool BWD>
__global__ void __launch_bounds__(256) k_conv_few_to16_mfma_f32(const float* __restrict__ in, const uint16_t* __restrict__ w,
                                                                const float* __restrict__ bias, int B, int Z, int Y, int X,
                                                                ConvPost P, float* __restrict__ out, long per_block)
{
    constexpr int NK = (27 * CI + 3) / 4;
    __shared__ float tile[kTNV * CI];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, q = lane >> 4, r = lane & 15;
    float aw[NK];
    int off[NK];
    bool bad = false;
#pragma unroll
    for (int s = 0; s < NK; s++) {
        const int k = 4 * s + q, t = k / CI, i = k % CI;
        // past the last tap: zero times zero
        aw[s] = t < 27 ? tap_weight<CI, 16, BWD>(w, t, r, i) : 0.0f;
        off[s] = t < 27 ? ((t / 9 * kTSY + t / 3 % 3) * kTSX + t % 3) * CI + i : 0;
        bad = bad || !(fabsf(aw[s]) < INFINITY);
    }
    const bool scalar = __any(bad);
    v4f b0 = {0.f, 0.f, 0.f, 0.f};
    if (!BWD) b0 = v4f{bias[4 * q], bias[4 * q + 1], bias[4 * q + 2], bias[4 * q + 3]};
    const long ntiles = conv_tiles(B, Z, Y, X);
    const long first = (long)blockIdx.x * per_block;
    const long last = first + per_block < ntiles ? first + per_block : ntiles;
    for (long id = first; id < last; id++) {
        const ConvTile T = conv_tile(id, Z, Y, X);
        if (scalar) {
            conv_block_scalar<CI, 16, BWD>(T, in, w, bias, Z, Y, X, P, out);
            continue;
        }
        __syncthreads();
        for (int v = threadIdx.x; v < kTNV; v += 256) {
            const long g = region_voxel(T, v, Z, Y, X);
#pragma unroll
            for (int i = 0; i < CI; i++) tile[v * CI + i] = g >= 0 ? in[g * CI + i] : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int p = 0; p < 4; p++) {
            const float* t0 = tile + ((wave * kTSY + p) * kTSX + r) * CI;
            v4f acc = b0;
#pragma unroll
            for (int s = 0; s < NK; s++) {
                const float h = 4 * s + q < 27 * CI ? t0[off[s]] : 0.0f;
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(aw[s], h, acc, 0, 0, 0);
            }
            store_row16(T, wave * 4 + p, q, r, Z, Y, X, acc, P, out);
        }
    }
}

// 16 -> 1 or 2 channels: forward of the last layer (CO = 1), data gradient of the
// first (CO = 2).  Too few output channels for a matrix product (15 of 16 rows
// would be padding), so a thread owns one (x, y) column of a 32 x 8 block and
// marches along z: each input plane is staged in LDS once and its 3 x 3
// neighbourhood feeds the sums of three output planes, which sit in registers.
// A voxel's sum runs over its taps in order, channel by channel, as in
// k_conv_fwd_t.  The weights come as scalar loads of bfloat16 pairs (w is 4-byte
// aligned) unpacked on the scalar unit: read from LDS they were three quarters of
// the LDS traffic.  Forward 213 -> 97 us at 130^3, data gradient 1872 -> 189 us.
// zch: output planes of a workgroup
constexpr int kFewX = 32, kFewY = 8;
static_assert(kFewX * kFewY == 256, "a thread per column");

template <int CO, bool BWD>
__global__ void __launch_bounds__(256) k_conv16_to_few_f32(const float* __restrict__ in, const uint16_t* __restrict__ w,
                                                           const float* __restrict__ bias, int B, int Z, int Y, int X,
                                                           ConvPost P, float* __restrict__ out, int zch)
{
    constexpr int SX = kFewX + 2, SY = kFewY + 2, NV = SX * SY;
    __shared__ __align__(16) float tile[NV * kTVS];
    bool bad = false;
    for (int e = threadIdx.x; e < 27 * CO * 16; e += 256) bad = bad || !(fabsf(bf16_to_f32(w[e])) < INFINITY);
    const bool scalar = __syncthreads_or(bad);
    const int nbx = (X + kFewX - 1) / kFewX, nby = (Y + kFewY - 1) / kFewY, nbz = (Z + zch - 1) / zch;
    int id = blockIdx.x;
    const int bx = id % nbx;
    id /= nbx;
    const int by = id % nby;
    id /= nby;
    const int z0 = (id % nbz) * zch, b = id / nbz;
    const int lx = threadIdx.x & (kFewX - 1), ly = threadIdx.x / kFewX;
    const int x = bx * kFewX + lx, y = by * kFewY + ly;
    const bool live = x < X && y < Y;
    const int z1 = z0 + zch < Z ? z0 + zch : Z;
    const auto store = [&](int z, float (&a)[CO]) {
        const long base = ((((long)b * Z + z) * Y + y) * X + x) * CO;
#pragma unroll
        for (int o = 0; o < CO; o++) out[base + o] = conv_post(a[o], P, P.act ? P.act[base + o] : 0.0f);
    };
    if (scalar) {
        if (live)
            for (int z = z0; z < z1; z++) {
                float a[CO];
#pragma unroll
                for (int o = 0; o < CO; o++) a[o] = conv_voxel<16, CO, BWD>(in, w, bias, Z, Y, X, b, z, y, x, o);
                store(z, a);
            }
        return;
    }
    // acc[d]: the sums of output plane zi + 1 - d, which input plane zi enters as its tap plane d
    float acc[3][CO] = {};
    for (int zi = z0 - 1; zi <= z1; zi++) {
        __syncthreads();
        for (int v = threadIdx.x; v < NV; v += 256) {
            const int gx = bx * kFewX - 1 + v % SX, gy = by * kFewY - 1 + v / SX;
            const bool inside = zi >= 0 && zi < Z && gx >= 0 && gx < X && gy >= 0 && gy < Y;
            const float4* src = (const float4*)(in + ((((long)b * Z + zi) * Y + gy) * X + gx) * 16);
            float4* dst = (float4*)(tile + v * kTVS);
#pragma unroll
            for (int s = 0; s < 4; s++) dst[s] = inside ? src[s] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        __syncthreads();
        // output plane zi + 1 starts here (its tap row dz = -1)
#pragma unroll
        for (int o = 0; o < CO; o++) {
            acc[2][o] = acc[1][o];
            acc[1][o] = acc[0][o];
            acc[0][o] = BWD ? 0.0f : bias[o];
        }
        // (a plane outside the volume adds products with zero; unrolled whole, the
        // loop would hold every weight at once)
#pragma unroll 1
        for (int t2 = 0; t2 < 9; t2++) {
            const float4* src = (const float4*)(tile + ((ly + t2 / 3) * SX + lx + t2 % 3) * kTVS);
            float a[16];
#pragma unroll
            for (int s = 0; s < 4; s++) {
                const float4 c = src[s];
                a[4 * s] = c.x;
                a[4 * s + 1] = c.y;
                a[4 * s + 2] = c.z;
                a[4 * s + 3] = c.w;
            }
#pragma unroll
            for (int d = 0; d < 3; d++) {
                // the tap's 16 CO weights, pairs in scalar registers: CO = 1 two channels, CO = 2 two outputs
                const uint32_t* wt = (const uint32_t*)w + (BWD ? 26 - (9 * d + t2) : 9 * d + t2) * 8 * CO;
#pragma unroll
                for (int e = 0; e < 8 * CO; e++) {
                    const uint32_t u = wt[e];
                    const float lo = __uint_as_float(u << 16), hi = __uint_as_float(u & 0xffff0000u);
                    if constexpr (CO == 1) {
                        acc[d][0] = fmaf(lo, a[2 * e], acc[d][0]);
                        acc[d][0] = fmaf(hi, a[2 * e + 1], acc[d][0]);
                    } else {
                        acc[d][0] = fmaf(lo, a[e], acc[d][0]);
                        acc[d][1] = fmaf(hi, a[e], acc[d][1]);
                    }
                }
            }
        }
        if (live && zi - 1 >= z0) store(zi - 1, acc[2]);
    }
}

// Weight and bias gradients on the FP32 matrix cores, first stage: a workgroup
// sums over its range of 16 x 4 x 4 blocks of voxels and writes one partial
// (27 * CO * CI weights, then CO biases).  The voxels are the K dimension, four
// along x per product.
//   16 -> 16: rows output channels (gout), columns input channels, one product
//             per tap: 27 accumulators per lane set, bound by the matrix cores;
//   2 -> 16:  rows output channels, columns (tap, input channel) pairs, 4 products;
//   16 -> 1:  rows taps (gout at the voxel minus the tap), columns input channels, 2
//             products.  Here the voxels are those of the input, and a gout outside
//             the volume enters as zero; an input that is not finite is left out
//             of the products and its pairs are added one by one.
// The four wavefronts' sums meet in LDS in a fixed order.  At 130^3 with the
// second stage: 5136 -> 450, 1341 -> 109 and 1885 -> 93 us.
// A running sum over a workgroup's whole range would round more the larger the volume (258^3
// voxels, gradients of either sign: 2.3e-6, 1.1e-6 and 1.5e-6 of the largest gradient from 64
// bits in the order above; voxel rows summed by k_conv_bwd_weight_part 4.3e-7, 3.3e-7 and 4.6e-7).
// So with few accumulators the sums of kWgStep blocks of voxels are added to a second set; the 27
// of 16 -> 16 leave no registers for one, and where a workgroup has more than 2 kWgRun
// blocks (130^3 voxels: 20), runs of kWgRun are added to its partial: 4.0e-7, 3.1e-7 and
// 3.7e-7, for 2 to 5 % of the time.
constexpr int kWgBlocks = 512;
constexpr long kWgStep = 4, kWgRun = 10;

template <int CI, int CO>
__global__ void __launch_bounds__(256, 2) k_conv_bwd_weight_mfma(const float* __restrict__ in, const float* __restrict__ gout,
                                                                 int B, int Z, int Y, int X, float* __restrict__ part,
                                                                 long per_block)
{
    constexpr bool LAST = CO == 1;                            // the roles of halo and block swap
    constexpr int NA = CI == 2 ? 4 : (LAST ? 2 : 27);         // accumulators (products per four voxels)
    constexpr int HC = LAST ? 1 : CI, BC = LAST ? CI : CO;    // channels of the halo and of the block array
    constexpr int NE = 27 * CI * CO + CO;
    constexpr int NL = kTNV * HC + 256 * BC > NE ? kTNV * HC + 256 * BC : NE;
    __shared__ __align__(16) float lds[NL];
    __shared__ float extra[LAST ? 27 * 16 : 1];
    float* const halo = lds;
    float* const blk = lds + kTNV * HC;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, q = lane >> 4, r = lane & 15;
    constexpr bool TWO = NA <= 4;                             // a second set of accumulators
    v4f acc[NA], sum[TWO ? NA : 1];
    float accb;
    double sumb;  // (one addition per block of voxels)
    // halo offset of the lane's row or column in each product
    int hoff[LAST || CI == 2 ? NA : 1];
    bool hlive[LAST || CI == 2 ? NA : 1];
    if constexpr (LAST || CI == 2) {
#pragma unroll
        for (int a = 0; a < NA; a++) {
            const int e = 16 * a + r, t = LAST ? e : e >> 1;
            hlive[a] = t < 27;
            const int tt = LAST ? 26 - t : t;  // LAST: gout at the voxel minus the tap
            hoff[a] = hlive[a] ? ((tt / 9 * kTSY + tt / 3 % 3) * kTSX + tt % 3) * HC + (LAST ? 0 : e & 1) : 0;
        }
    }
    if constexpr (LAST)
        for (int e = threadIdx.x; e < 27 * 16; e += 256) extra[e] = 0.0f;  // (a barrier follows in the loop)
    const float* const hsrc = LAST ? gout : in;
    const float* const bsrc = LAST ? in : gout;
    const long ntiles = conv_tiles(B, Z, Y, X);
    const long first = (long)blockIdx.x * per_block;
    const long last = first + per_block < ntiles ? first + per_block : ntiles;
    // The next block's values are loaded into registers while the current block is
    // multiplied (HV + 4 vectors per thread), so its load latency is hidden.
    constexpr int HV = HC == 16 ? 4 : 1, NR = (kTNV + 255) / 256;
    constexpr int KU = NA > 4 ? 1 : 4;  // (27 products unrolled four times spill)
    float4 nh[NR][HV], nc[4];
    const int cv = threadIdx.x;  // the thread's voxel of the block
    const auto fetch = [&](const ConvTile& T) {
#pragma unroll
        for (int j = 0; j < NR; j++) {
            const int v = (int)threadIdx.x + 256 * j;
            const long g = v < kTNV ? region_voxel(T, v, Z, Y, X) : -1;
#pragma unroll
            for (int s = 0; s < HV; s++) {
                nh[j][s] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (g < 0) continue;
                if constexpr (HC == 16) {
                    nh[j][s] = ((const float4*)(hsrc + g * 16))[s];
                } else {
                    nh[j][s].x = hsrc[g * HC];
                    if (HC == 2) nh[j][s].y = hsrc[g * HC + 1];
                }
            }
        }
        const int x = T.x0 + (cv & 15), y = T.y0 + (cv >> 4 & 3), z = T.z0 + (cv >> 6);
        const bool inside = x < X && y < Y && z < Z;
        const float4* src = (const float4*)(bsrc + ((((long)T.b * Z + z) * Y + y) * X + x) * 16);
#pragma unroll
        for (int s = 0; s < 4; s++) nc[s] = inside ? src[s] : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    const auto clear = [](auto& v) {
#pragma unroll
        for (v4f& x : v) x = v4f{0.f, 0.f, 0.f, 0.f};
    };
    const long len = TWO || last - first <= 2 * kWgRun ? last - first : kWgRun;
    for (long run = first; run < last; run += len) {
        const long end = run + len < last ? run + len : last;
        clear(acc);
        clear(sum);
        accb = 0.0f;
        sumb = 0.0;
        fetch(conv_tile(run, Z, Y, X));
        for (long id = run; id < end; id++) {
            const ConvTile T = conv_tile(id, Z, Y, X);
            __syncthreads();  // the previous block's operands have been read
#pragma unroll
            for (int j = 0; j < NR; j++) {
                const int v = (int)threadIdx.x + 256 * j;
                if (v >= kTNV) break;
                if constexpr (HC == 16) {
#pragma unroll
                    for (int s = 0; s < HV; s++) ((float4*)(halo + v * 16))[s] = nh[j][s];
                } else {
                    halo[v * HC] = nh[j][0].x;
                    if (HC == 2) halo[v * HC + 1] = nh[j][0].y;
                }
            }
            if constexpr (LAST) {
                const int x = T.x0 + (cv & 15), y = T.y0 + (cv >> 4 & 3), z = T.z0 + (cv >> 6);
                if (x < X && y < Y && z < Z) {
                    float* const c16 = &nc[0].x;
                    const long g = (((long)T.b * Z + z) * Y + y) * X + x;
                    const float g0 = gout[g];
                    const bool gfin = fabsf(g0) < INFINITY;
#pragma unroll
                    for (int i = 0; i < 16; i++) {
                        const float a = c16[i];
                        const bool fin = fabsf(a) < INFINITY;
                        if (!fin) c16[i] = 0.0f;
                        if (fin && gfin) continue;
                        // (inf and NaN: the order of these additions does not matter)
#pragma unroll 1
                        for (int t = 0; t < 27; t++) {
                            const int dz = t / 9 - 1, dy = t / 3 % 3 - 1, dx = t % 3 - 1;
                            const auto in_volume = [&](int zz, int yy, int xx) {
                                return zz >= 0 && zz < Z && yy >= 0 && yy < Y && xx >= 0 && xx < X;
                            };
                            if (!fin && in_volume(z - dz, y - dy, x - dx))
                                atomicAdd(&extra[t * 16 + i],
                                          a * gout[(((long)T.b * Z + z - dz) * Y + y - dy) * X + x - dx]);
                            if (!gfin && !in_volume(z + dz, y + dy, x + dx)) atomicAdd(&extra[t * 16 + i], g0 * 0.0f);
                        }
                    }
                }
            }
#pragma unroll
            for (int s = 0; s < 4; s++) ((float4*)(blk + cv * 16))[s] = nc[s];
            __syncthreads();
            if (id + 1 < end) fetch(conv_tile(id + 1, Z, Y, X));
            // a voxel past the row's end: gout is zero there, and so is what it multiplies
#pragma unroll 1
            for (int p = 0; p < 4; p++) {
                if (T.z0 + wave >= Z || T.y0 + p >= Y) break;
                const float* h0 = halo + ((wave * kTSY + p) * kTSX + q) * HC;
                const float* c0 = blk + ((wave * 4 + p) * 16 + q) * BC + r;
#pragma unroll KU
                for (int k4 = 0; k4 < 4; k4++, h0 += 4 * HC, c0 += 4 * BC) {
                    const float g = *c0;
                    const bool vox = T.x0 + 4 * k4 + q < X;
                    if constexpr (!LAST) accb += g;
#pragma unroll
                    for (int a = 0; a < NA; a++) {
                        if constexpr (LAST) {
                            const float h = hlive[a] && vox ? h0[hoff[a]] : 0.0f;
                            acc[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(h, g, acc[a], 0, 0, 0);
                            if (a == 0 && r == 13) accb += h;  // the centre tap's row: gout of the voxel itself
                        } else if constexpr (CI == 2) {
                            const float h = hlive[a] && vox ? h0[hoff[a]] : 0.0f;
                            acc[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(g, h, acc[a], 0, 0, 0);
                        } else {
                            const float h = h0[((a / 9 * kTSY + a / 3 % 3) * kTSX + a % 3) * 16 + r];
                            acc[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(g, vox ? h : 0.0f, acc[a], 0, 0, 0);
                        }
                    }
                }
            }
            sumb += (double)accb;
            accb = 0.0f;
            if (TWO && ((id - run) % kWgStep == kWgStep - 1 || id + 1 == end)) {
#pragma unroll
                for (int a = 0; a < (TWO ? NA : 0); a++) sum[a] += acc[a];
                clear(acc);
            }
        }
        // the wavefronts' sums into the workgroup's partial; bias: the four voxel lanes of a
        // channel first
        sumb += __shfl_xor(sumb, 16, 64);
        sumb += __shfl_xor(sumb, 32, 64);
        v4f(&tot)[NA] = [&]() -> v4f(&)[NA] {
            if constexpr (TWO) return sum;
            else return acc;
        }();
        for (int wv = 0; wv < 4; wv++) {
            __syncthreads();
            if (wave != wv) continue;
#pragma unroll
            for (int a = 0; a < NA; a++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const int m = 4 * q + e;  // row
                    int at;
                    if constexpr (LAST) at = 16 * a + m < 27 ? (16 * a + m) * 16 + r : -1;
                    else if constexpr (CI == 2) at = 16 * a + r < 54 ? ((16 * a + r) / 2 * 16 + m) * 2 + (r & 1) : -1;
                    else at = (a * 16 + m) * 16 + r;
                    if (at >= 0) lds[at] = wv == 0 ? tot[a][e] : lds[at] + tot[a][e];
                }
            const bool mine = LAST ? lane == 13 : lane < 16;
            if (mine) {
                const int at = 27 * CI * CO + (LAST ? 0 : lane);
                lds[at] = wv == 0 ? (float)sumb : lds[at] + (float)sumb;
            }
        }
        __syncthreads();
        for (int e = threadIdx.x; e < NE; e += 256) {
            float v = lds[e];
            float* const p = part + (long)blockIdx.x * NE + e;
            if (run != first) v += *p;
            if constexpr (LAST)
                if (end == last && e < 27 * 16) v += extra[e];
            *p = v;
        }
    }
}

// Second stage: gw/gb = sum over the partials, in a fixed order: 16 groups of
// partials per weight, then the groups (one thread per weight over all 2048
// partials took 517 us).
constexpr int kSumGroups = 16;

__global__ void __launch_bounds__(64 * kSumGroups) k_sum_parts(const float* __restrict__ part, int nparts, int ne, int nw,
                                                               float* __restrict__ gw, float* __restrict__ gb)
{
    __shared__ float red[kSumGroups][64];
    const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + lane;
    float s = 0.0f;
    if (e < ne) {
#pragma unroll 8
        for (int p = grp; p < nparts; p += kSumGroups) s += part[(long)p * ne + e];
    }
    red[grp][lane] = s;
    __syncthreads();
    if (grp || e >= ne) return;
    s = 0.0f;
#pragma unroll
    for (int g = 0; g < kSumGroups; g++) s += red[g][lane];
    if (e < nw) gw[e] = s;
    else gb[e - nw] = s;
}

// ------------------------------------------------------------------ solver glue
// Features of a nested level's Gamma ((n+2)^3 points, channel-last, 2 channels):
// f / ||f|| and r0 / ||f|| with r0 = f - lap(phi) of the interpolated guess.
template <typename TA>
__global__ void __launch_bounds__(kNB) k_net_features(SGrid g, const double* __restrict__ phi,
                                                     const double* __restrict__ f, double inv_fnorm, double inv_h2,
                                                     TA* __restrict__ x)
{
    const int mx = g.nx - 2, my = g.ny - 2, mz = g.nz - 2;
    const long nv = (long)mx * my * mz;
    const long v = (long)blockIdx.x * kNB + threadIdx.x;
    if (v >= nv) return;
    const int i = (int)(v % mx) + 1;
    const int j = (int)((v / mx) % my) + 1;
    const int k = (int)(v / ((long)mx * my)) + 1;
    auto at = [&](const double* a, int pi, int pj, int pk) {
        return a[(size_t)((pi + pj + pk + 3) & 1) * g.cs + ((size_t)pk * g.ps + (size_t)pj * g.hx) + (pi >> 1)];
    };
    const double lap = (at(phi, i - 1, j, k) + at(phi, i + 1, j, k) + at(phi, i, j - 1, k) + at(phi, i, j + 1, k) +
                        at(phi, i, j, k - 1) + at(phi, i, j, k + 1) - 6.0 * at(phi, i, j, k)) * inv_h2;
    const double fv = at(f, i, j, k);
    st(x + 2 * v, (float)(fv * inv_fnorm));
    st(x + 2 * v + 1, (float)((fv - lap) * inv_fnorm));
}

// phi += s * out on Gamma (out: (n+2)^3 FP32)
__global__ void __launch_bounds__(kNB) k_net_apply(SGrid g, double* __restrict__ phi, const float* __restrict__ out,
                                                  double s)
{
    const int mx = g.nx - 2, my = g.ny - 2, mz = g.nz - 2;
    const long nv = (long)mx * my * mz;
    const long v = (long)blockIdx.x * kNB + threadIdx.x;
    if (v >= nv) return;
    const int i = (int)(v % mx) + 1;
    const int j = (int)((v / mx) % my) + 1;
    const int k = (int)(v / ((long)mx * my)) + 1;
    phi[(size_t)((i + j + k + 3) & 1) * g.cs + ((size_t)k * g.ps + (size_t)j * g.hx) + (i >> 1)] += s * (double)out[v];
}

// target = (phi_a - phi_b) * inv_s on Gamma
__global__ void __launch_bounds__(kNB) k_net_target(SGrid g, const double* __restrict__ pa,
                                                   const double* __restrict__ pb, double inv_s, float* __restrict__ t)
{
    const int mx = g.nx - 2, my = g.ny - 2, mz = g.nz - 2;
    const long nv = (long)mx * my * mz;
    const long v = (long)blockIdx.x * kNB + threadIdx.x;
    if (v >= nv) return;
    const int i = (int)(v % mx) + 1;
    const int j = (int)((v / mx) % my) + 1;
    const int k = (int)(v / ((long)mx * my)) + 1;
    const size_t p = (size_t)((i + j + k + 3) & 1) * g.cs + ((size_t)k * g.ps + (size_t)j * g.hx) + (i >> 1);
    t[v] = (float)((pa[p] - pb[p]) * inv_s);
}

}  // namespace

// ------------------------------------------------------------------ launchers
constexpr int kNetParts = 2048;  // blocks (partial sums) of the weight-gradient reduction

// The network's layer shapes (2 -> 16, 16 -> 16, 16 -> 1) run on the
// compile-time kernel; returns false for other shapes.
template <typename TI, typename TO>
static bool conv_fwd_fixed(hipStream_t st, const TI* in, int cin, const uint16_t* w, const float* bias, int cout, int relu,
                    int B, int Z, int Y, int X, TO* out)
{
    const dim3 grid(cdiv((long)B * Z * Y * X, kNB));
    if (cin == 2 && cout == 16)
        hipLaunchKernelGGL((k_conv_fwd_t<2, 16, TI, TO>), grid, dim3(kNB), 0, st, in, w, bias, relu, B, Z, Y, X, out);
    else if (cin == 16 && cout == 16)
        hipLaunchKernelGGL((k_conv_fwd_t<16, 16, TI, TO>), grid, dim3(kNB), 0, st, in, w, bias, relu, B, Z, Y, X, out);
    else if (cin == 16 && cout == 1)
        hipLaunchKernelGGL((k_conv_fwd_t<16, 1, TI, TO>), grid, dim3(kNB), 0, st, in, w, bias, relu, B, Z, Y, X, out);
    else
        return false;
    return true;
}

// The FP32 matrix-core kernels move a voxel's 16 channels in 16-byte accesses:
// they take the network's layer shapes with 16-byte aligned arrays, the other
// calls go to the thread-per-voxel kernels.
static bool aligned16(const void* a, const void* b, const void* c)
{
    return (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c) & 15) == 0;
}

// planes per workgroup of the few-channel kernel: 8 (1.25 times the input read)
// where that gives two workgroups per CU, else 2 for shorter chains
static int few_planes(int B, int Z, int Y, int X)
{
    return (long)B * cdiv(X, kFewX) * cdiv(Y, kFewY) * cdiv(Z, 8) >= 512 ? 8 : 2;
}

static long few_workgroups(int B, int Z, int Y, int X)
{
    return (long)B * cdiv(X, kFewX) * cdiv(Y, kFewY) * cdiv(Z, few_planes(B, Z, Y, X));
}

// Whether a layer's forward pass is faster in blocks than with a thread per voxel (the results
// are the same).  A block takes its time however many of its voxels lie in the volume, and a
// chain of planes its time however few blocks there are; a thread per voxel has neither.
// Measured, a thread per voxel / blocks: 16 -> 1 channels (0.092 ns a voxel; 22 ns a workgroup
// of 2 planes after 12 us, 52 ns one of 8 after 24 us): 18^3 voxels 8.6 / 16.2 us, 50^3
// 15.2 / 19.1, 58^3 23.2 / 18.8, 130^3 208 / 99, 130 x 130 x 6 14.6 / 31.6, x 16 31.7 / 33.8, x 20
// 40.1 / 34.3; 2 -> 16: 130 x 130 x 6 10.5 / 13.6, x 14 16.2 / 14.4, x 17 18.7 / 22.0, x 26 26.6 / 22.3,
// 66^3 18.8 / 16.5; 16 -> 16: 130 x 130 x 6 41.8 / 49.8, x 10 58.8 / 50.7, 66^3 91.5 / 53.4.
// (The passes that round or mask as well, which a thread per voxel does in a second
// kernel, are never slower in blocks, nor are the data gradients, but for bwd_in_blocks.)
static bool fwd_in_blocks(int cin, int cout, int B, int Z, int Y, int X)
{
    const long n = (long)B * Z * Y * X, tiles = conv_tiles(B, Z, Y, X);
    if (cout == 1) {
        const long wgs = few_workgroups(B, Z, Y, X);
        return few_planes(B, Z, Y, X) == 8 ? n > 200000 + 565 * wgs : n > 65000 + 200 * wgs;
    }
    return cin == 2 ? n + 26000 > 180 * tiles : n + 20000 > 115 * tiles;
}

// The data gradient of the 2 -> 16 layer: blocks except on long volumes of few voxels across
// (4000 x 3 x 3: 79 us with a thread per voxel, 93 in blocks; 130 x 130 x 3: 80 and 61).
static bool bwd_in_blocks(int B, int Z, int Y, int X)
{
    return (long)Y * X >= 25 || (few_planes(B, Z, Y, X) == 2 && few_workgroups(B, Z, Y, X) < 1600);
}

// input channels ci, output channels co of the pass (for the data gradient the
// layer's output and input channels); false: not one of the layers' shapes
template <bool BWD>
static bool train_conv(hipStream_t st, const float* in, int ci, const uint16_t* w, const float* bias, int co, ConvPost P,
                       int B, int Z, int Y, int X, float* out)
{
    if (!aligned16(in, out, P.act)) return false;
    const long tiles = conv_tiles(B, Z, Y, X);
    const long per = (tiles + kTrainBlocks - 1) / kTrainBlocks;
    const dim3 grid((unsigned)((tiles + per - 1) / per));
    // the small-channel kernel holds few weights: more, shorter ranges
    const long per1 = (tiles + 4 * kTrainBlocks - 1) / (4 * kTrainBlocks);
    const dim3 grid1((unsigned)((tiles + per1 - 1) / per1));
    const int zch = few_planes(B, Z, Y, X);
    const long few = few_workgroups(B, Z, Y, X);
    if (ci == 16 && co == 16)
        hipLaunchKernelGGL(k_conv16_mfma_f32<BWD>, grid, dim3(256), 0, st, in, w, bias, B, Z, Y, X, P, out, per);
    else if (ci == (BWD ? 1 : 2) && co == 16)
        hipLaunchKernelGGL((k_conv_few_to16_mfma_f32<BWD ? 1 : 2, BWD>), grid1, dim3(256), 0, st, in, w, bias, B, Z, Y, X,
                           P, out, per1);
    else if (ci == 16 && co == (BWD ? 2 : 1) && few < (1L << 31) && ((uintptr_t)w & 3) == 0 && (!BWD || bwd_in_blocks(B, Z, Y, X)))
        hipLaunchKernelGGL((k_conv16_to_few_f32<BWD ? 2 : 1, BWD>), dim3((unsigned)few), dim3(256), 0, st, in, w, bias, B,
                           Z, Y, X, P, out, zch);
    else
        return false;
    return true;
}

void net_conv_fwd_f32(hipStream_t st, const float* in, int cin, const uint16_t* w, const float* bias, int cout, int relu,
                      int B, int Z, int Y, int X, float* out)
{
    long nv = (long)B * Z * Y * X;
    if (fwd_in_blocks(cin, cout, B, Z, Y, X) &&
        train_conv<false>(st, in, cin, w, bias, cout, ConvPost{relu, 0, nullptr}, B, Z, Y, X, out))
        return;
    if (conv_fwd_fixed(st, in, cin, w, bias, cout, relu, B, Z, Y, X, out)) return;
    hipLaunchKernelGGL((k_conv_fwd<float, float>), dim3(cdiv(nv, kNB)), dim3(kNB), 0, st, in, cin, w, bias, cout, relu, B,
                       Z, Y, X, out);
}

void net_conv_fwd_bf16(hipStream_t st, const uint16_t* in, int cin, const uint16_t* w, const float* bias, int cout,
                       int relu, int B, int Z, int Y, int X, uint16_t* out)
{
    long nv = (long)B * Z * Y * X;
    if (conv_fwd_fixed(st, in, cin, w, bias, cout, relu, B, Z, Y, X, out)) return;
    hipLaunchKernelGGL((k_conv_fwd<uint16_t, uint16_t>), dim3(cdiv(nv, kNB)), dim3(kNB), 0, st, in, cin, w, bias, cout,
                       relu, B, Z, Y, X, out);
}

void net_conv_fwd_bf16_to_f32(hipStream_t st, const uint16_t* in, int cin, const uint16_t* w, const float* bias,
                              int cout, int relu, int B, int Z, int Y, int X, float* out)
{
    long nv = (long)B * Z * Y * X;
    if (conv_fwd_fixed(st, in, cin, w, bias, cout, relu, B, Z, Y, X, out)) return;
    hipLaunchKernelGGL((k_conv_fwd<uint16_t, float>), dim3(cdiv(nv, kNB)), dim3(kNB), 0, st, in, cin, w, bias, cout,
                       relu, B, Z, Y, X, out);
}

void net_conv_mfma(hipStream_t st, const uint16_t* in, int cin, const uint16_t* w, const float* bias, int cout, int relu,
                   int B, int Z, int Y, int X, void* out)
{
    // a row is one buffer, whose size and the offset that stands for "outside" (kCvOob) need
    // 31 bits: longer rows, of 2^26 voxels and more, go to the thread-per-voxel kernels
    if ((long)X * 16 * (long)sizeof(uint16_t) >= (long)kCvOob) {
        if (cout == 16) net_conv_fwd_bf16(st, in, cin, w, bias, cout, relu, B, Z, Y, X, (uint16_t*)out);
        else net_conv_fwd_bf16_to_f32(st, in, cin, w, bias, cout, relu, B, Z, Y, X, (float*)out);
        return;
    }
    const auto launch = [&](auto ci, auto co, auto rows, auto* o, int per_cu) {
        constexpr int R = decltype(rows)::value;
        const int ntx = cdiv(X, 16), nty = cdiv(Y, R * kCvWaves);
        // planes per workgroup: a range reads two more than its own, the ranges run in
        // rounds of per_cu workgroups per CU.  Each number of planes that equal ranges can have
        // is looked at once, 2 sqrt(Z) of them (over every number of ranges the host took
        // longer than the kernel for 4000 planes of 3 x 3 voxels: 15 us, now 7 to 10)
        const long cols = (long)ntx * nty * B, slots = 256L * per_cu;
        int kz = Z;
        long best = 0;
        for (int k = Z;; ) {
            const long cost = (cols * cdiv(Z, k) + slots - 1) / slots * (k + 2);
            if (k == Z || cost < best) {
                best = cost;
                kz = k;
            }
            if (k == 1) break;
            k = cdiv(Z, cdiv(Z, k - 1));  // the next smaller one
        }
        const int ntz = (Z + kz - 1) / kz;
        hipLaunchKernelGGL((k_conv_mfma<decltype(ci)::value, decltype(co)::value, R, std::remove_pointer_t<decltype(o)>>),
                           dim3((unsigned)(cols * ntz)), dim3(64 * kCvWaves), 0, st, in, w, bias, relu, Z, Y, X, o, ntx, nty,
                           ntz, kz);
    };
    const auto go = [&](auto ci, auto co, auto* o, int per_cu) {
        if constexpr (decltype(ci)::value == 16) {
            if ((long)B * Z * cdiv(X, 16) * cdiv(Y, 16) >= kCvLarge)
                return launch(ci, co, std::integral_constant<int, 4>{}, o, per_cu);
        }
        launch(ci, co, std::integral_constant<int, 2>{}, o, per_cu);
    };
    using C1 = std::integral_constant<int, 1>;
    using C2 = std::integral_constant<int, 2>;
    using C16 = std::integral_constant<int, 16>;
    if (cin == 16 && cout == 16) go(C16{}, C16{}, (uint16_t*)out, 2);
    else if (cin == 2 && cout == 16) go(C2{}, C16{}, (uint16_t*)out, 4);
    else if (cin == 16 && cout == 1) go(C16{}, C1{}, (float*)out, 2);
}

void net_conv_bwd_data(hipStream_t st, const float* gout, int cout, const uint16_t* w, int cin, int B, int Z, int Y,
                       int X, float* gin)
{
    long nv = (long)B * Z * Y * X;
    if (train_conv<true>(st, gout, cout, w, nullptr, cin, ConvPost{0, 0, nullptr}, B, Z, Y, X, gin)) return;
    hipLaunchKernelGGL(k_conv_bwd_data, dim3(cdiv(nv, kNB)), dim3(kNB), 0, st, gout, cout, w, cin, B, Z, Y, X, gin);
}

size_t net_bwd_weight_workspace(int cin, int cout) { return (size_t)kNetParts * (27 * cin * cout + cout) * sizeof(float); }

void net_conv_bwd_weight(hipStream_t st, const float* in, int cin, const float* gout, int cout, int B, int Z, int Y,
                         int X, float* gw, float* gb, float* part)
{
    const int ne = 27 * cin * cout + cout;
    const long tiles = conv_tiles(B, Z, Y, X);
    const long per = (tiles + kWgBlocks - 1) / kWgBlocks;
    const dim3 grid((unsigned)((tiles + per - 1) / per));
    int parts = (int)grid.x;
    const bool wide = aligned16(cin == 16 ? in : nullptr, cout == 16 ? gout : nullptr, nullptr);
    if (wide && cin == 16 && cout == 16)
        hipLaunchKernelGGL((k_conv_bwd_weight_mfma<16, 16>), grid, dim3(256), 0, st, in, gout, B, Z, Y, X, part, per);
    else if (wide && cin == 2 && cout == 16)
        hipLaunchKernelGGL((k_conv_bwd_weight_mfma<2, 16>), grid, dim3(256), 0, st, in, gout, B, Z, Y, X, part, per);
    else if (wide && cin == 16 && cout == 1)
        hipLaunchKernelGGL((k_conv_bwd_weight_mfma<16, 1>), grid, dim3(256), 0, st, in, gout, B, Z, Y, X, part, per);
    else {
        parts = kNetParts;
        hipLaunchKernelGGL(k_conv_bwd_weight_part, dim3(parts), dim3(kNB), 0, st, in, cin, gout, cout, B, Z, Y, X, part);
    }
    hipLaunchKernelGGL(k_sum_parts, dim3(cdiv(ne, 64)), dim3(64 * kSumGroups), 0, st, part, parts, ne, 27 * cin * cout, gw,
                       gb);
}

void net_relu_bwd(hipStream_t st, const float* act, float* g, long n)
{
    hipLaunchKernelGGL(k_relu_bwd, dim3(cdiv(n, kNB)), dim3(kNB), 0, st, act, g, n);
}

size_t net_mse_workspace(long n) { return (size_t)cdiv(n, kNB) * sizeof(float); }

void net_mse(hipStream_t st, const float* pred, const float* target, const float* mask, long n, float count,
             float* grad, float* part, float* loss)
{
    int nb = cdiv(n, kNB);
    hipLaunchKernelGGL(k_mse, dim3(nb), dim3(kNB), 0, st, pred, target, mask, n, 1.0f / count, grad, part);
    hipLaunchKernelGGL(k_sum, dim3(1), dim3(64), 0, st, part, nb, 1.0f / count, loss);
}

void net_adam(hipStream_t st, float* w, const float* g, float* m, float* v, long n, float lr, float b1, float b2,
              float eps, int step, uint16_t* wb)
{
    float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(cdiv(n, kNB)), dim3(kNB), 0, st, w, g, m, v, n, lr, b1, b2, eps, c1, c2, wb);
}

void net_to_bf16(hipStream_t st, const float* a, uint16_t* b, long n)
{
    hipLaunchKernelGGL(k_to_bf16, dim3(cdiv(n, kNB)), dim3(kNB), 0, st, a, b, n);
}

void net_features_bf16(hipStream_t st, SGrid g, const double* phi, const double* f, double inv_fnorm, double inv_h2,
                       uint16_t* x)
{
    const long nvox = (long)(g.nx - 2) * (g.ny - 2) * (g.nz - 2);
    hipLaunchKernelGGL((k_net_features<uint16_t>), dim3(cdiv(nvox, kNB)), dim3(kNB), 0, st, g, phi, f, inv_fnorm,
                       inv_h2, x);
}

void net_features_f32(hipStream_t st, SGrid g, const double* phi, const double* f, double inv_fnorm, double inv_h2,
                      float* x)
{
    const long nvox = (long)(g.nx - 2) * (g.ny - 2) * (g.nz - 2);
    hipLaunchKernelGGL((k_net_features<float>), dim3(cdiv(nvox, kNB)), dim3(kNB), 0, st, g, phi, f, inv_fnorm,
                       inv_h2, x);
}

void net_apply(hipStream_t st, SGrid g, double* phi, const float* out, double s)
{
    const long nvox = (long)(g.nx - 2) * (g.ny - 2) * (g.nz - 2);
    hipLaunchKernelGGL(k_net_apply, dim3(cdiv(nvox, kNB)), dim3(kNB), 0, st, g, phi, out, s);
}

void net_target(hipStream_t st, SGrid g, const double* pa, const double* pb, double inv_s, float* t)
{
    const long nvox = (long)(g.nx - 2) * (g.ny - 2) * (g.nz - 2);
    hipLaunchKernelGGL(k_net_target, dim3(cdiv(nvox, kNB)), dim3(kNB), 0, st, g, pa, pb, inv_s, t);
}

}  // namespace np

// ------------------------------------------------------------------ C ABI (include/nested_poisson.h)
using namespace np;

static bool net_ok(int cin, int cout) { return cin >= 1 && cin <= 16 && cout >= 1 && cout <= 16; }
static bool dims_ok(int b, int z, int y, int x) { return b >= 1 && z >= 1 && y >= 1 && x >= 1; }

extern "C" {

size_t np_net_workspace_bytes(int cin, int cout, long nvox)
{
    size_t a = net_ok(cin, cout) ? net_bwd_weight_workspace(cin, cout) : 0;
    size_t b = nvox > 0 ? net_mse_workspace(nvox) : 0;
    return a > b ? a : b;
}

int np_net_conv3d_fwd(const float* in, int cin, const unsigned short* w, const float* bias, int cout, int relu,
                      int batch, int nz, int ny, int nx, float* out, void* stream)
{
    if (!in || !w || !bias || !out || !net_ok(cin, cout) || !dims_ok(batch, nz, ny, nx)) return NP_EINVAL;
    net_conv_fwd_f32((hipStream_t)stream, in, cin, w, bias, cout, relu, batch, nz, ny, nx, out);
    return hipGetLastError() == hipSuccess ? NP_OK : NP_EHIP;
}

int np_net_conv3d_fwd_mfma(const unsigned short* in, int cin, const unsigned short* w, const float* bias, int cout,
                           int relu, int batch, int nz, int ny, int nx, void* out, void* stream)
{
    if (!in || !w || !bias || !out || !dims_ok(batch, nz, ny, nx)) return NP_EINVAL;
    if (!((cin == 2 && cout == 16) || (cin == 16 && cout == 16) || (cin == 16 && cout == 1))) return NP_EINVAL;
    if ((uintptr_t)in & (uintptr_t)(4 * cin - 1)) return NP_EINVAL;
    net_conv_mfma((hipStream_t)stream, in, cin, w, bias, cout, relu, batch, nz, ny, nx, out);
    return hipGetLastError() == hipSuccess ? NP_OK : NP_EHIP;
}

int np_net_conv3d_bwd_data(const float* gout, int cout, const unsigned short* w, int cin, int batch, int nz, int ny,
                           int nx, float* gin, void* stream)
{
    if (!gout || !w || !gin || !net_ok(cin, cout) || !dims_ok(batch, nz, ny, nx)) return NP_EINVAL;
    net_conv_bwd_data((hipStream_t)stream, gout, cout, w, cin, batch, nz, ny, nx, gin);
    return hipGetLastError() == hipSuccess ? NP_OK : NP_EHIP;
}

int np_net_conv3d_fwd_round(const float* in, int cin, const unsigned short* w, const float* bias, int cout, int batch,
                            int nz, int ny, int nx, float* out, void* stream)
{
    if (!in || !w || !bias || !out || !net_ok(cin, cout) || !dims_ok(batch, nz, ny, nx)) return NP_EINVAL;
    const hipStream_t st = (hipStream_t)stream;
    if (!train_conv<false>(st, in, cin, w, bias, cout, ConvPost{1, 1, nullptr}, batch, nz, ny, nx, out)) {
        const long n = (long)batch * nz * ny * nx * cout;
        net_conv_fwd_f32(st, in, cin, w, bias, cout, 1, batch, nz, ny, nx, out);
        hipLaunchKernelGGL(k_round_bf16, dim3(cdiv(n, kNB)), dim3(kNB), 0, st, out, n);
    }
    return hipGetLastError() == hipSuccess ? NP_OK : NP_EHIP;
}

int np_net_conv3d_bwd_data_relu(const float* gout, int cout, const unsigned short* w, int cin, int batch, int nz, int ny,
                                int nx, const float* act, float* gin, void* stream)
{
    if (!gout || !w || !act || !gin || !net_ok(cin, cout) || !dims_ok(batch, nz, ny, nx)) return NP_EINVAL;
    const hipStream_t st = (hipStream_t)stream;
    if (!train_conv<true>(st, gout, cout, w, nullptr, cin, ConvPost{0, 0, act}, batch, nz, ny, nx, gin)) {
        net_conv_bwd_data(st, gout, cout, w, cin, batch, nz, ny, nx, gin);
        net_relu_bwd(st, act, gin, (long)batch * nz * ny * nx * cin);
    }
    return hipGetLastError() == hipSuccess ? NP_OK : NP_EHIP;
}

int np_net_conv3d_bwd_weight(const float* in, int cin, const float* gout, int cout, int batch, int nz, int ny, int nx,
                             float* gw, float* gb, float* workspace, size_t workspace_bytes, void* stream)
{
    if (!in || !gout || !gw || !gb || !workspace || !net_ok(cin, cout) || !dims_ok(batch, nz, ny, nx)) return NP_EINVAL;
    if (workspace_bytes < net_bwd_weight_workspace(cin, cout)) return NP_EINVAL;
    net_conv_bwd_weight((hipStream_t)stream, in, cin, gout, cout, batch, nz, ny, nx, gw, gb, workspace);
    return hipGetLastError() == hipSuccess ? NP_OK : NP_EHIP;
}

int np_net_relu_bwd(const float* act, float* grad, long n, void* stream)
{
    if (!act || !grad || n < 0) return NP_EINVAL;
    if (n) net_relu_bwd((hipStream_t)stream, act, grad, n);
    return hipGetLastError() == hipSuccess ? NP_OK : NP_EHIP;
}

int np_net_mse(const float* pred, const float* target, const float* mask, long n, float count, float* grad,
               float* loss, float* workspace, size_t workspace_bytes, void* stream)
{
    if (!pred || !target || !grad || !loss || !workspace || n < 1 || !(count > 0)) return NP_EINVAL;
    if (workspace_bytes < net_mse_workspace(n)) return NP_EINVAL;
    net_mse((hipStream_t)stream, pred, target, mask, n, count, grad, workspace, loss);
    return hipGetLastError() == hipSuccess ? NP_OK : NP_EHIP;
}

// Partial sums of np_net_mse_noalloc: one file-scope device array, never
// allocated at run time.  Each device holds its own copy at its own address,
// looked up once per device (hipGetSymbolAddress) and kept in mse_scratch_dev;
// host code uses only those addresses, never the array's name.
static __device__ __align__(256) float scratch[NP_NET_MSE_NOALLOC_MAX / 256];
static float* mse_scratch_dev[64];
static std::mutex mse_scratch_mu;

static int mse_scratch(float** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        (void)hipGetLastError();
        set_last_error("np_net_mse_noalloc: no current HIP device (or device index >= 64)");
        return NP_ENODEV;
    }
    std::lock_guard<std::mutex> lock(mse_scratch_mu);
    if (!mse_scratch_dev[dev]) {
        float* p = nullptr;
        const hipError_t e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            char msg[160];
            snprintf(msg, sizeof msg, "np_net_mse_noalloc: hipGetSymbolAddress: %s", hipGetErrorString(e));
            set_last_error(msg);
            return NP_EHIP;
        }
        mse_scratch_dev[dev] = p;
    }
    *out = mse_scratch_dev[dev];
    return NP_OK;
}

int np_net_mse_noalloc(const float* pred, const float* target, const float* mask, long n, float count, float* grad,
                       float* loss, void* stream)
{
    if (!pred || !target || !grad || !loss || n < 1 || !(count > 0)) return NP_EINVAL;
    if (n > NP_NET_MSE_NOALLOC_MAX) {
        char msg[160];
        snprintf(msg, sizeof msg, "np_net_mse_noalloc: n = %ld exceeds the maximum %ld", n,
                 (long)NP_NET_MSE_NOALLOC_MAX);
        set_last_error(msg);
        return NP_EINVAL;
    }
    float* part = nullptr;
    const int rc = mse_scratch(&part);
    if (rc) return rc;
    // every partial k_sum reads (blocks 0 .. ceil(n/256) - 1) is written by k_mse
    // first, so nothing needs clearing between calls
    net_mse((hipStream_t)stream, pred, target, mask, n, count, grad, part, loss);
    return hipGetLastError() == hipSuccess ? NP_OK : NP_EHIP;
}

int np_net_adam(float* w, const float* g, float* m, float* v, long n, float lr, float beta1, float beta2, float eps,
                int step, unsigned short* w_bf16, void* stream)
{
    if (!w || !g || !m || !v || n < 0 || step < 1) return NP_EINVAL;
    if (n) net_adam((hipStream_t)stream, w, g, m, v, n, lr, beta1, beta2, eps, step, w_bf16);
    return hipGetLastError() == hipSuccess ? NP_OK : NP_EHIP;
}

int np_net_round_bf16(float* a, long n, void* stream)
{
    if (!a || n < 0) return NP_EINVAL;
    if (n) hipLaunchKernelGGL(k_round_bf16, dim3(cdiv(n, kNB)), dim3(kNB), 0, (hipStream_t)stream, a, n);
    return hipGetLastError() == hipSuccess ? NP_OK : NP_EHIP;
}

int np_net_lap7(const float* in, int batch, int nz, int ny, int nx, float* out, void* stream)
{
    if (!in || !out || in == out || !dims_ok(batch, nz, ny, nx)) return NP_EINVAL;
    const long nv = (long)batch * nz * ny * nx;
    hipLaunchKernelGGL(k_lap7, dim3(cdiv(nv, kNB)), dim3(kNB), 0, (hipStream_t)stream, in, batch, nz, ny, nx, out);
    return hipGetLastError() == hipSuccess ? NP_OK : NP_EHIP;
}

int np_net_to_bf16(const float* a, unsigned short* b, long n, void* stream)
{
    if (!a || !b || n < 0) return NP_EINVAL;
    if (n) net_to_bf16((hipStream_t)stream, a, b, n);
    return hipGetLastError() == hipSuccess ? NP_OK : NP_EHIP;
}

}  // extern "C"
