// Learned proposal network: downsampling to 64^3, four 3x3x3 stride-2
// convolutions (2 -> 16 -> 32 -> 64 -> 64 channels, zero padding 1, bias,
// ReLU), a linear head to 6 means and 6 log-variances, the Gaussian NLL of
// the filter's final weighted cloud, its backward pass and Adam.
//
// Convolutions are implicit GEMMs on v_mfma_f32_16x16x32_bf16 whose operands
// are 16-byte loads of eight consecutive K values: each of the three products
// of a layer reads its operands in the order in which its K is contiguous, and
// the kernel that produces a tensor writes it in the orders that its readers
// need (a second copy costs a write, a gather of 2-byte elements with index
// divisions cost more than the product itself).
//   forward  C[m = output voxel][n = c_out]  K = (tap, c_in)
//            activations channels last ("cl"), weights [c_out][tap][c_in]
//   dgrad    C[m = input voxel][n = c_in]    K = (tap, c_out)
//            dY channels last, weights [tap][c_in][c_out].  A stride-2 kernel
//            reaches an input voxel by one tap per axis where its coordinate is
//            even and by two where it is odd: a wave takes the voxels of one
//            (z, y) parity and both x parities, so no product is with zero
//   wgrad    C[m = c_out][n = (tap, c_in)]   K = output voxel
//            dY channels first ("cf"); X "split": [c][z][y][3][x / 2], the
//            planes holding x - 1 (odd), x (even) and x + 1 (odd) of an output
//            voxel's three taps, so that eight consecutive output voxels read
//            eight consecutive elements.  K is split over waves, whose partial
//            sums k_grads_finish adds in a fixed order (no floating-point
//            atomics: a training step is reproducible bit for bit)
// Weights, activations and the operands of all products are bfloat16 (round to
// nearest even), accumulation FP32, gradients FP32; dY is rounded once, after
// its bias gradient has been summed from the FP32 values.
//
// What it measured: a training step of 32 pairs (inputs, backward with the
// gradients read back, Adam) 5.72 ms with operands gathered element by element
// (dgrad 2.3, bias gradients 1.2, wgrad 1.1, forward 0.58), 0.68 ms so (dgrad
// 0.090, wgrad 0.134, forward 0.10, the 32 downsamplings 0.125); a proposal of
// one pair 94 -> 48 us.  Bound: latency -- 4 to 50 us kernels of a few thousand
// waves, launches, and the copy of the gradients to the host.
#include <hip/hip_fp16.h>

#include "internal.h"

namespace smc {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kBufferWord3 = 0x00020000;
constexpr uint32_t kOutside = 0xFFFFFFF0u;  // a buffer offset past any end: loads read zero

__device__ __forceinline__ uint16_t to_bf16(float f) {
    uint32_t b = __float_as_uint(f);
    b = b + 0x7FFFu + ((b >> 16) & 1u);
    return (uint16_t)(b >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ uint32_t pair_bf16(float lo, float hi) {
    return (uint32_t)to_bf16(lo) | ((uint32_t)to_bf16(hi) << 16);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, size_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)(uint32_t)bytes, kBufferWord3);
}
__device__ __forceinline__ bf16x8 load8(__amdgpu_buffer_rsrc_t rs, uint32_t byte_offset) {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, byte_offset, 0, 0));
}
__device__ __forceinline__ bf16x8 load8(const uint16_t *p) { return __builtin_bit_cast(bf16x8, *(const u32x4 *)p); }

// Lane l of a wave holds A[l % 16][8 (l / 16) + i] and B[8 (l / 16) + i][l % 16],
// i = 0..7, of v_mfma_f32_16x16x32_bf16, and C[4 (l / 16) + i][l % 16], i = 0..3.
__device__ __forceinline__ v4f mfma(bf16x8 a, bf16x8 b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

constexpr int kChan[5] = {2, 16, 32, 64, 64};
constexpr int kSide = 64;
constexpr int side_of(int L) { return kSide >> L; }  // input side of layer L
// K of a forward layer's packed weights: 27 c_in rounded up to 32; the first
// layer's rows (c_in, kz, ky) hold four x taps, the last of them zero.
constexpr int fwd_k(int L) { return L == 0 ? 96 : (27 * kChan[L] + 31) / 32 * 32; }

// ---- forward --------------------------------------------------------------------

// Activation (ReLU, bf16) of four consecutive output voxels m .. m + 3 (one
// row of side DO) of channel n: channels last, and for training the split form
// that the next layer's wgrad reads, or channels first for the head.
template <int CO, int DO, bool LAST>
__device__ __forceinline__ void store_act(const float v[4], int m, int n, uint16_t *ycl, uint16_t *yx) {
    constexpr int VOX = DO * DO * DO;
    if constexpr (LAST) {
        const int b = m / VOX, r = m - b * VOX;
        *(u32x2 *)(ycl + ((size_t)b * CO + n) * VOX + r) = u32x2{pair_bf16(v[0], v[1]), pair_bf16(v[2], v[3])};
    } else {
        uint16_t h[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h[i] = to_bf16(v[i]);
            ycl[(size_t)(m + i) * CO + n] = h[i];
        }
        if (yx) {
            const int b = m / VOX, r = m - b * VOX, x = r % DO;
            uint16_t *row = yx + (((size_t)b * CO + n) * (DO * DO) + r / DO) * (3 * (DO / 2)) + x / 2;
            *(uint32_t *)(row + DO / 2) = (uint32_t)h[0] | ((uint32_t)h[2] << 16);
            *(uint32_t *)(row + DO) = (uint32_t)h[1] | ((uint32_t)h[3] << 16);
            row[1] = h[1];  // (element 0 of the plane of x - 1 stays zero)
            if (x / 2 + 2 < DO / 2) row[2] = h[3];
        }
    }
}

// First layer: a workgroup takes four output rows of one slice; the input rows
// they read are staged in LDS as bf16, element x at x + 1, so that the four
// values from 2 ox - 1 on (three taps and one that is dropped) start at a
// 4-byte boundary.
constexpr int kL0Rows = 4, kL0Pitch = 68;
__global__ __launch_bounds__(256) void k_conv_first(const uint16_t *X, const uint16_t *W, const float *bias,
                                                    uint16_t *ycl, uint16_t *yx) {
    constexpr int DI = 64, DO = 32, NY = 2 * kL0Rows + 1;
    __shared__ __attribute__((aligned(16))) uint16_t slab[2 * 3 * NY * kL0Pitch];
    const int b = blockIdx.x / (DO * (DO / kL0Rows)), rem = blockIdx.x % (DO * (DO / kL0Rows));
    const int oz = rem / (DO / kL0Rows), oy0 = rem % (DO / kL0Rows) * kL0Rows;
    for (int q = threadIdx.x; q < 2 * 3 * NY * (DI / 4); q += 256) {
        const int x = 4 * (q % (DI / 4)), row = q / (DI / 4);
        const int yy = row % NY, zc = row / NY, kz = zc % 3, c = zc / 3;
        const int z = 2 * oz + kz - 1, y = 2 * oy0 + yy - 1;
        uint2 v = make_uint2(0u, 0u);
        if (z >= 0 && y >= 0) v = *(const uint2 *)(X + (((size_t)b * 2 + c) * DI + z) * (DI * DI) + y * DI + x);
        uint16_t *d = slab + row * kL0Pitch + x + 1;
        const uint32_t h[4] = {v.x & 0xFFFFu, v.x >> 16, v.y & 0xFFFFu, v.y >> 16};
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = to_bf16(__half2float(__ushort_as_half((uint16_t)h[e])));
        if (x == 0) d[-1] = 0;
    }
    __syncthreads();
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, r = lane % 16, g = lane / 16;
    bf16x8 w[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) w[s] = load8(W + r * 96 + 32 * s + 8 * g);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int ox = 16 * t + r;
        v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            u32x4 a = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int row = 8 * s + 2 * g + e;  // (c, kz, ky)
                if (row < 18) {
                    const int ky = row % 3, ck = row / 3;
                    const uint32_t *p = (const uint32_t *)(slab + (ck * NY + 2 * wave + ky) * kL0Pitch) + ox;
                    a[2 * e] = p[0];
                    a[2 * e + 1] = p[1] & 0xFFFFu;
                }
            }
            acc = mfma(__builtin_bit_cast(bf16x8, a), w[s], acc);
        }
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = fmaxf(acc[i] + bias[r], 0.0f);
        const int m = ((b * DO + oz) * DO + oy0 + wave) * DO + 16 * t + 4 * g;
        store_act<16, DO, false>(v, m, r, ycl, yx);
    }
}

// Layers 1 .. 3.  A wave computes MT x NT tiles of 16 output voxels x 16
// channels; KW = 1: four waves on their own voxels; KW > 1: KW waves share the
// tiles and K, adding their accumulators in LDS in wave order (the deep layers
// have few voxels).
template <int L, int MT, int NT, int KW>
__global__ __launch_bounds__(KW == 1 ? 256 : 64 * KW) void k_conv(const uint16_t *X, const uint16_t *W,
                                                                 const float *bias, uint16_t *ycl, uint16_t *yx,
                                                                 int B) {
    constexpr int CI = kChan[L], CO = kChan[L + 1], DI = side_of(L), DO = DI / 2, VOX = DO * DO * DO;
    constexpr int KP = fwd_k(L), STEPS = KP / 32;
    __shared__ v4f red[KW > 1 ? KW - 1 : 1][MT * NT][64];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, r = lane % 16, g = lane / 16;
    const int tile = (KW == 1 ? (int)blockIdx.x * 4 + wave : (int)blockIdx.x) * MT;
    const int n0 = blockIdx.y * NT * 16;
    if (KW == 1 && tile * 16 >= B * VOX) return;
    const __amdgpu_buffer_rsrc_t rs = buffer_of(X, (size_t)B * DI * DI * DI * CI * 2);
    int base[MT], edge[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const int m = (tile + t) * 16 + r, b = m / VOX, v = m % VOX;
        const int oz = v / (DO * DO), oy = v / DO % DO, ox = v % DO;
        base[t] = (((b * DI + 2 * oz - 1) * DI + 2 * oy - 1) * DI + 2 * ox - 1) * CI;
        // taps 0 read coordinate 2 o - 1: outside for o = 0
        edge[t] = (oz == 0 ? 4 : 0) | (oy == 0 ? 2 : 0) | (ox == 0 ? 1 : 0);
    }
    v4f acc[MT][NT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[t][n] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 3
    for (int s = KW == 1 ? 0 : wave; s < STEPS; s += KW) {
        const int tap = CI == 16 ? 2 * s + g / 2 : (CI == 32 ? s : s / 2);
        const int ch = CI == 16 ? 8 * (g % 2) : (CI == 32 ? 8 * g : 32 * (s % 2) + 8 * g);
        const int kz = tap / 9, ky = tap / 3 % 3, kx = tap % 3;
        const int off = (kz * DI * DI + ky * DI + kx) * CI + ch;
        const int low = (kz == 0 ? 4 : 0) | (ky == 0 ? 2 : 0) | (kx == 0 ? 1 : 0);
        bf16x8 a[MT], w[NT];
#pragma unroll
        for (int t = 0; t < MT; ++t)
            a[t] = load8(rs, tap < 27 && (low & edge[t]) == 0 ? 2u * (uint32_t)(base[t] + off) : kOutside);
#pragma unroll
        for (int n = 0; n < NT; ++n) w[n] = load8(W + (size_t)(n0 + 16 * n + r) * KP + 32 * s + 8 * g);
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int n = 0; n < NT; ++n) acc[t][n] = mfma(a[t], w[n], acc[t][n]);
    }
    if constexpr (KW > 1) {
        if (wave > 0)
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int n = 0; n < NT; ++n) red[wave - 1][t * NT + n][lane] = acc[t][n];
        __syncthreads();
        if (wave > 0) return;
        for (int k = 0; k < KW - 1; ++k)
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int n = 0; n < NT; ++n) acc[t][n] += red[k][t * NT + n][lane];
    }
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            const int c = n0 + 16 * n + r;
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = fmaxf(acc[t][n][i] + bias[c], 0.0f);
            store_act<CO, DO, L == 3>(v, (tile + t) * 16 + 4 * g, c, ycl, yx);
        }
}

// ---- backward -------------------------------------------------------------------

// The network input in the split form (bf16): eight x a thread.
__global__ __launch_bounds__(256) void k_split_input(const uint16_t *X, int64_t rows, uint16_t *out) {
    const int64_t q = blockIdx.x * 256ll + threadIdx.x;
    if (q >= rows * 8) return;
    const int64_t row = q / 8;
    const int j = 4 * (int)(q % 8);  // x / 2 of the first
    const u32x4 v = *(const u32x4 *)(X + row * 64 + 2 * j);
    uint16_t *o = out + row * 96 + j;
    uint16_t e[4], d[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        e[i] = to_bf16(__half2float(__ushort_as_half((uint16_t)(v[i] & 0xFFFFu))));
        d[i] = to_bf16(__half2float(__ushort_as_half((uint16_t)(v[i] >> 16))));
    }
    *(u32x2 *)(o + 32) = u32x2{(uint32_t)e[0] | ((uint32_t)e[1] << 16), (uint32_t)e[2] | ((uint32_t)e[3] << 16)};
    *(u32x2 *)(o + 64) = u32x2{(uint32_t)d[0] | ((uint32_t)d[1] << 16), (uint32_t)d[2] | ((uint32_t)d[3] << 16)};
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (j + i + 1 < 32) o[i + 1] = d[i];
}

// dL/dX of layer L masked by the ReLU that made X: the dY of layer L - 1.  A
// job is 16 pairs of input voxels (x = 2 mx, 2 mx + 1) of one slice and row
// parity; the lane's four pairs are eight consecutive x.  Workgroups take jobs
// in strides and keep the channels' sums, the bias gradient of layer L - 1.
template <int L, int NT>
__global__ __launch_bounds__(256) void k_dgrad(const uint16_t *dY, const uint16_t *W, const uint16_t *xs, uint16_t *dxf,
                                               uint16_t *dxl, float *bias_part, int B) {
    constexpr int CI = kChan[L], CO = kChan[L + 1], DI = side_of(L), H = DI / 2, RT = 16 / H;
    constexpr int JOBS = DI * 2 * (H / RT);  // per pair of volumes
    __shared__ float red[4][NT][16];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, r = lane % 16, g = lane / 16;
    const int n0 = blockIdx.y * NT * 16;
    const __amdgpu_buffer_rsrc_t rs = buffer_of(dY, (size_t)B * H * H * H * CO * 2);
    float bsum[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) bsum[n] = 0.0f;
    for (int job = blockIdx.x * 4 + wave; job < B * JOBS; job += gridDim.x * 4) {
        const int b = job / JOBS, q = job % JOBS;
        const int iz = q / (2 * (H / RT)), py = q / (H / RT) % 2, ty = q % (H / RT);
        const int pz = iz % 2, mz = iz / 2, mx = r % H, my = ty * RT + r / H;
        v4f acc[2][NT];
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int n = 0; n < NT; ++n) acc[p][n] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        // even coordinates: tap 1 of output m; odd: tap 0 of m + 1 and tap 2 of m
        for (int jz = 0; jz <= pz; ++jz) {
            const int kz = pz ? 2 * jz : 1, oz = mz + (pz && jz == 0 ? 1 : 0);
            if (oz >= H) continue;
            for (int jy = 0; jy <= py; ++jy) {
                const int ky = py ? 2 * jy : 1, oy = my + (py && jy == 0 ? 1 : 0);
                const int at = (((b * H + oz) * H + oy) * H + mx) * CO;
                const uint16_t *w = W + ((size_t)(kz * 9 + ky * 3) * CI + n0 + r) * CO + 8 * g;
#pragma unroll
                for (int c = 0; c < CO / 32; ++c) {
                    const uint32_t o = 2u * (uint32_t)(at + 32 * c + 8 * g);
                    const bf16x8 a0 = load8(rs, oy < H ? o : kOutside);
                    const bf16x8 a1 = load8(rs, oy < H && mx + 1 < H ? o + 2u * CO : kOutside);
#pragma unroll
                    for (int n = 0; n < NT; ++n) {
                        const uint16_t *wn = w + (size_t)16 * n * CO + 32 * c;
                        acc[0][n] = mfma(a0, load8(wn + (size_t)CI * CO), acc[0][n]);
                        acc[1][n] = mfma(a0, load8(wn + (size_t)2 * CI * CO), acc[1][n]);
                        acc[1][n] = mfma(a1, load8(wn), acc[1][n]);
                    }
                }
            }
        }
        // the lane's pairs: m = 4 g .. 4 g + 3
        const int x0 = 2 * ((4 * g) % H), iy = 2 * (ty * RT + 4 * g / H) + py;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            const int c = n0 + 16 * n + r;
            const uint16_t *xr = xs + ((((size_t)b * CI + c) * DI + iz) * DI + iy) * (3 * H) + x0 / 2;
            const u32x2 even = *(const u32x2 *)(xr + H), odd = *(const u32x2 *)(xr + 2 * H);
            float v[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[2 * i] = ((even[i / 2] >> (16 * (i % 2))) & 0xFFFFu) ? acc[0][n][i] : 0.0f;
                v[2 * i + 1] = ((odd[i / 2] >> (16 * (i % 2))) & 0xFFFFu) ? acc[1][n][i] : 0.0f;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) bsum[n] += v[i];
            const size_t row = (size_t)(iz * DI + iy) * DI + x0;
            *(u32x4 *)(dxf + ((size_t)b * CI + c) * (DI * DI * DI) + row) =
                u32x4{pair_bf16(v[0], v[1]), pair_bf16(v[2], v[3]), pair_bf16(v[4], v[5]), pair_bf16(v[6], v[7])};
            if (dxl)
#pragma unroll
                for (int i = 0; i < 8; ++i) dxl[((size_t)b * (DI * DI * DI) + row + i) * CI + c] = to_bf16(v[i]);
        }
    }
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        bsum[n] += __shfl_xor(bsum[n], 16);
        bsum[n] += __shfl_xor(bsum[n], 32);
        if (g == 0) red[wave][n][r] = bsum[n];
    }
    __syncthreads();
    if (threadIdx.x < NT * 16) {
        const int n = threadIdx.x / 16, c = threadIdx.x % 16;
        bias_part[(size_t)blockIdx.x * CI + n0 + threadIdx.x] =
            (red[0][n][c] + red[1][n][c]) + (red[2][n][c] + red[3][n][c]);
    }
}

// Weight gradient of layers 1 .. 3.  A wave: taps (kz, ky, 0 .. 2), 16 CT input
// channels, 32 output channels and K range [split KS, (split + 1) KS) of the
// output voxels; partial sums to part[split][c_out][c_in][27].
template <int L, int CT>
__global__ __launch_bounds__(256) void k_wgrad(const uint16_t *dY, const uint16_t *xs, float *part, int B, int KS,
                                               int splits) {
    constexpr int CI = kChan[L], CO = kChan[L + 1], DI = side_of(L), DO = DI / 2, VOX = DO * DO * DO;
    constexpr int MT = 2, CG = CI / (16 * CT), MG = CO / (16 * MT), JOBS = 9 * CG * MG;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, r = lane % 16, g = lane / 16;
    const int job = blockIdx.x * 4 + wave;
    if (job >= JOBS * splits) return;
    const int split = job / JOBS, q = job % JOBS;
    const int tap = q % 9, kz = tap / 3, ky = tap % 3, cg = q / 9 % CG, mg = q / (9 * CG);
    const int c0 = cg * 16 * CT, m0 = mg * 16 * MT;
    const __amdgpu_buffer_rsrc_t rx = buffer_of(xs, (size_t)B * CI * DI * DI * 3 * DO * 2);
    v4f acc[MT][3][CT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int x = 0; x < 3; ++x)
#pragma unroll
            for (int c = 0; c < CT; ++c) acc[t][x][c] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    const int k1 = min((split + 1) * KS, B * VOX);
#pragma unroll 2
    for (int k0 = split * KS; k0 < k1; k0 += 32) {
        const int v = k0 + 8 * g, b = v / VOX, o = v % VOX;
        const int oz = o / (DO * DO), oy = o / DO % DO, ox = o % DO;
        const int z = 2 * oz + kz - 1, y = 2 * oy + ky - 1;
        bf16x8 a[MT], w[3][CT];
#pragma unroll
        for (int t = 0; t < MT; ++t) a[t] = load8(dY + ((size_t)b * CO + m0 + 16 * t + r) * VOX + o);
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const uint32_t row = (uint32_t)(((b * CI + c0 + 16 * c + r) * DI + z) * DI + y) * (3 * DO) + (uint32_t)ox;
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                if constexpr (DO >= 8) {
                    w[x][c] = load8(rx, z >= 0 && y >= 0 ? 2u * (row + x * DO) : kOutside);
                } else {
                    // rows of four voxels: two output rows, input rows y and y + 2
                    const u32x2 lo = __builtin_amdgcn_raw_buffer_load_b64(
                        rx, z >= 0 && y >= 0 ? 2u * (row + x * DO) : kOutside, 0, 0);
                    const u32x2 hi = __builtin_amdgcn_raw_buffer_load_b64(
                        rx, z >= 0 ? 2u * (row + x * DO + 2 * 3 * DO) : kOutside, 0, 0);
                    w[x][c] = __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
                }
            }
        }
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int x = 0; x < 3; ++x)
#pragma unroll
                for (int c = 0; c < CT; ++c) acc[t][x][c] = mfma(a[t], w[x][c], acc[t][x][c]);
    }
    float *out = part + (size_t)split * CO * CI * 27;
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int x = 0; x < 3; ++x)
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    out[((size_t)(m0 + 16 * t + 4 * g + i) * CI + c0 + 16 * c + r) * 27 + 3 * tap + x] =
                        acc[t][x][c][i];
}

// Weight gradient of the first layer: a K step is one output row; the four
// waves of a workgroup take every gridDim.x * 4-th row and add their sums in
// LDS; part[workgroup][16][54].
__global__ __launch_bounds__(256) void k_wgrad_first(const uint16_t *dY, const uint16_t *xs, float *part, int B) {
    constexpr int DI = 64, DO = 32, VOX = DO * DO * DO;
    __shared__ v4f red[3][4][64];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, r = lane % 16, g = lane / 16;
    const __amdgpu_buffer_rsrc_t rx = buffer_of(xs, (size_t)B * 2 * DI * DI * 3 * DO * 2);
    int chan[4], kz[4], ky[4], kx[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int n = 16 * t + r, tap = n % 27;
        chan[t] = n < 54 ? n / 27 : -1;
        kz[t] = tap / 9;
        ky[t] = tap / 3 % 3;
        kx[t] = tap % 3;
    }
    v4f acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 2
    for (int row = blockIdx.x * 4 + wave; row < B * DO * DO; row += gridDim.x * 4) {
        const int b = row / (DO * DO), oz = row / DO % DO, oy = row % DO;
        const bf16x8 a = load8(dY + ((size_t)b * 16 + r) * VOX + (row % (DO * DO)) * DO + 8 * g);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int z = 2 * oz + kz[t] - 1, y = 2 * oy + ky[t] - 1;
            const bool ok = chan[t] >= 0 && z >= 0 && y >= 0;
            const uint32_t at = (uint32_t)((((b * 2 + chan[t]) * DI + z) * DI + y) * 3 + kx[t]) * DO + 8u * (uint32_t)g;
            acc[t] = mfma(a, load8(rx, ok ? 2u * at : kOutside), acc[t]);
        }
    }
    if (wave > 0)
#pragma unroll
        for (int t = 0; t < 4; ++t) red[wave - 1][t][lane] = acc[t];
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        acc[t] += red[0][t][lane];
        acc[t] += red[1][t][lane];
        acc[t] += red[2][t][lane];
        if (16 * t + r < 54)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                part[(size_t)blockIdx.x * 864 + (4 * g + i) * 54 + 16 * t + r] = acc[t][i];
    }
}

// Sums of the partial gradients, in order: weights one thread each, biases one
// wave each (lanes take every 64th partial, then a fixed tree).
struct FinishArgs {
    const float *wpart[4], *bpart[3];
    int wn[4], wsplits[4], bn[3], bsplits[3];  // elements, partials
    int woff[4], boff[3];                      // place in the flat gradients
};
__global__ __launch_bounds__(256) void k_grads_finish(const FinishArgs a, int wblocks, float *grads) {
    if ((int)blockIdx.x < wblocks) {
        int q = blockIdx.x * 256 + threadIdx.x;
        for (int L = 0; L < 4; ++L) {
            if (q < a.wn[L]) {
                float s = 0.0f;
                const float *p = a.wpart[L] + q;
#pragma unroll 8
                for (int k = 0; k < a.wsplits[L]; ++k) s += p[(size_t)k * a.wn[L]];
                grads[a.woff[L] + q] = s;
                return;
            }
            q -= a.wn[L];
        }
        return;
    }
    int q = ((int)blockIdx.x - wblocks) * 4 + (int)threadIdx.x / 64;
    const int lane = threadIdx.x % 64;
    for (int L = 0; L < 3; ++L) {
        if (q < a.bn[L]) {
            float s = 0.0f;
            for (int k = lane; k < a.bsplits[L]; k += 64) s += a.bpart[L][(size_t)k * a.bn[L] + q];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
            if (lane == 0) grads[a.boff[L] + q] = s;
            return;
        }
        q -= a.bn[L];
    }
}

// ---- small kernels -----------------------------------------------------------

// Trilinear resampling to side^3 at half-pixel centres, FP16 output; the
// source (blockIdx.y = 0) and the target volume of a slot in one launch.
struct DownArgs {
    const uint8_t *vol[2];
    int n[2][3];
    float scale;
    uint16_t *out;  // two consecutive grids
};
__global__ void k_downsample(const DownArgs d) {
    constexpr int side = kSide;
    const int q = blockIdx.x * blockDim.x + threadIdx.x, which = blockIdx.y;
    if (q >= side * side * side) return;
    const uint8_t *vol = d.vol[which];
    const int nx = d.n[which][0], ny = d.n[which][1], nz = d.n[which][2];
    const float scale = d.scale;
    const int a = q % side, bq = (q / side) % side, c = q / (side * side);
    const float px = fminf(fmaxf((a + 0.5f) * ((float)nx / side) - 0.5f, 0.0f), (float)(nx - 1));
    const float py = fminf(fmaxf((bq + 0.5f) * ((float)ny / side) - 0.5f, 0.0f), (float)(ny - 1));
    const float pz = fminf(fmaxf((c + 0.5f) * ((float)nz / side) - 0.5f, 0.0f), (float)(nz - 1));
    const int x0 = (int)floorf(px), y0 = (int)floorf(py), z0 = (int)floorf(pz);
    const int x1 = min(x0 + 1, nx - 1), y1 = min(y0 + 1, ny - 1), z1 = min(z0 + 1, nz - 1);
    const float fx = px - x0, fy = py - y0, fz = pz - z0;
    auto V = [&](int x, int y, int z) { return (float)vol[(size_t)x + (size_t)nx * ((size_t)y + (size_t)ny * z)]; };
    const float c00 = V(x0, y0, z0) * (1 - fx) + V(x1, y0, z0) * fx;
    const float c10 = V(x0, y1, z0) * (1 - fx) + V(x1, y1, z0) * fx;
    const float c01 = V(x0, y0, z1) * (1 - fx) + V(x1, y0, z1) * fx;
    const float c11 = V(x0, y1, z1) * (1 - fx) + V(x1, y1, z1) * fx;
    const float v = ((c00 * (1 - fy) + c10 * fy) * (1 - fz) + (c01 * (1 - fy) + c11 * fy) * fz) * scale;
    d.out[which * side * side * side + q] = __half_as_ushort(__float2half(v));
}

// Head: out[b][j] = sum_f h[b][f] Wh[j][f] + bh[j] (FP32), one workgroup per
// (b, j); a thread takes 2 x 8 consecutive f.
__global__ __launch_bounds__(256) void k_head_fwd(const uint16_t *h, const float *Wh, const float *bh, float *out,
                                                  int F) {
    const int b = blockIdx.y, j = blockIdx.x;
    float s = 0.0f;
    for (int f = 8 * (int)threadIdx.x; f < F; f += 8 * 256) {
        const u32x4 v = *(const u32x4 *)(h + (size_t)b * F + f);
        const v4f w0 = *(const v4f *)(Wh + (size_t)j * F + f), w1 = *(const v4f *)(Wh + (size_t)j * F + f + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float lo = __uint_as_float(v[e] << 16), hi = __uint_as_float(v[e] & 0xFFFF0000u);
            const v4f &w = e < 2 ? w0 : w1;
            s += lo * w[2 * (e % 2)];
            s += hi * w[2 * (e % 2) + 1];
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    __shared__ float red[4];
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = s;
    __syncthreads();
    if (threadIdx.x == 0) out[(size_t)b * 12 + j] = ((red[0] + red[1]) + (red[2] + red[3])) + bh[j];
}

// Gaussian NLL (batch mean) and its gradient w.r.t. the 12 outputs.
__global__ void k_nll(const float *out, const float *target, int B, float *dout, float *loss) {
    const int b = threadIdx.x;
    __shared__ float red[1024];
    float l = 0.0f;
    if (b < B) {
        for (int d = 0; d < 6; ++d) {
            const float mu = out[b * 12 + d], lv = out[b * 12 + 6 + d];
            const float xb = target[b * 12 + d], var = target[b * 12 + 6 + d];
            const float e = expf(-lv), dm = xb - mu;
            l += 0.5f * ((var + dm * dm) * e + lv);
            dout[b * 12 + d] = -dm * e / B;
            dout[b * 12 + 6 + d] = 0.5f * (1.0f - (var + dm * dm) * e) / B;
        }
    }
    red[b] = l;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if (b < o) red[b] += red[b + o];
        __syncthreads();
    }
    if (b == 0) *loss = red[0] / B;
}

// Head backward, one workgroup per channel c of the last activation (f = 64 c +
// voxel): dWh[j][f] = sum_b dout[b][j] h[b][f]; dh[b][f] = (sum_j dout[b][j]
// Wh[j][f]) masked by h > 0 (the dY of the last layer, in both forms), and its
// sum over b and voxels, the last layer's bias gradient.  Wave w takes every
// fourth b, a lane a voxel.  Workgroup 0 adds dbh[j] = sum_b dout[b][j].
__global__ __launch_bounds__(256) void k_head_bwd(const uint16_t *h, const float *Wh, const float *dout, int B,
                                                  float *dWh, float *dbh, uint16_t *dyf, uint16_t *dyl, float *db) {
    constexpr int F = 4096;
    __shared__ float red[4][12][64];
    __shared__ float bred[4];
    const int c = blockIdx.x, v = threadIdx.x % 64, wave = threadIdx.x / 64, f = 64 * c + v;
    float w[12], dw[12], bs = 0.0f;
#pragma unroll
    for (int j = 0; j < 12; ++j) {
        w[j] = Wh[(size_t)j * F + f];
        dw[j] = 0.0f;
    }
    for (int b = wave; b < B; b += 4) {
        const uint16_t hv = h[(size_t)b * F + f];
        const float hf = from_bf16(hv);
        float s = 0.0f;
#pragma unroll
        for (int j = 0; j < 12; ++j) {
            const float d = dout[b * 12 + j];
            dw[j] += d * hf;
            s += d * w[j];
        }
        s = hv != 0 ? s : 0.0f;
        bs += s;
        const uint16_t q = to_bf16(s);
        dyf[(size_t)b * F + f] = q;
        dyl[((size_t)b * 64 + v) * 64 + c] = q;
    }
#pragma unroll
    for (int j = 0; j < 12; ++j) red[wave][j][v] = dw[j];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) bs += __shfl_xor(bs, o);
    if (v == 0) bred[wave] = bs;
    __syncthreads();
    for (int q = threadIdx.x; q < 12 * 64; q += 256) {
        const int j = q / 64, e = q % 64;
        dWh[(size_t)j * F + 64 * c + e] = (red[0][j][e] + red[1][j][e]) + (red[2][j][e] + red[3][j][e]);
    }
    if (threadIdx.x == 0) db[c] = (bred[0] + bred[1]) + (bred[2] + bred[3]);
    if (c == 0 && threadIdx.x < 12) {
        float s = 0.0f;
        for (int b = 0; b < B; ++b) s += dout[b * 12 + threadIdx.x];
        dbh[threadIdx.x] = s;
    }
}

// The bfloat16 copies of convolution weight q of the flat parameters (value w):
// the forward's [c_out][tap][c_in] (first layer [c_out][(c_in, kz, ky)][4]) and
// the dgrad's [tap][c_in][c_out].
struct WeightForms {
    uint16_t *fwd[4], *dgrad[4];
    int first[4], count[4];  // place of a layer's weights in the flat parameters
};
__device__ __forceinline__ void put_weight(const WeightForms &f, int64_t q, float w) {
    constexpr int chan[5] = {2, 16, 32, 64, 64};
#pragma unroll
    for (int L = 0; L < 4; ++L) {
        const int e = (int)(q - f.first[L]);
        if (e < 0 || e >= f.count[L]) continue;
        const int t = e % 27, ci = e / 27 % chan[L], co = e / (27 * chan[L]);
        const uint16_t v = to_bf16(w);
        if (L == 0) {
            f.fwd[0][co * 96 + (ci * 9 + t / 3) * 4 + t % 3] = v;
        } else {
            f.fwd[L][co * fwd_k(L) + t * chan[L] + ci] = v;
            f.dgrad[L][(t * chan[L] + ci) * chan[L + 1] + co] = v;
        }
    }
}

// Adam on FP32 master weights; refreshes the bfloat16 copies of the
// convolution weights.
// One Adam step (Kingma & Ba): m and v are the decayed first and second
// moments of the gradient, c1 = 1 - b1^t and c2 = 1 - b2^t their bias
// corrections.  The coefficients come from the host rounded once from FP64
// (1 - b and 1 - b^t lose digits if formed from FP32 b).
__global__ void k_adam(float *p, const float *g, float *m, float *v, const WeightForms forms, int64_t n,
                       float lr, float b1, float omb1, float b2, float omb2, float c1, float c2, float eps) {
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x) {
        const float gq = g[q];
        const float mq = b1 * m[q] + omb1 * gq;
        const float vq = b2 * v[q] + omb2 * (gq * gq);
        m[q] = mq;
        v[q] = vq;
        const float w = p[q] - lr * (mq / c1) / (sqrtf(vq / c2) + eps);
        p[q] = w;
        put_weight(forms, q, w);
    }
}

__global__ void k_pack_weights(const float *src, const WeightForms forms, int64_t n) {
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
        put_weight(forms, q, src[q]);
}

__global__ void k_zero_u32(uint32_t *p, int64_t n) {
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
        p[q] = 0u;
}

unsigned blocks(int64_t n) { return (unsigned)std::min<int64_t>((n + 255) / 256, 65535); }

}  // namespace

// ---- host side ----------------------------------------------------------------

const int kCnnChannels[5] = {2, 16, 32, 64, 64};
const int kCnnSide = 64;
const int kCnnFlat = 64 * 4 * 4 * 4;

int64_t cnn_param_offset(int part) {
    // parts: W1 b1 W2 b2 W3 b3 W4 b4 Wh bh
    int64_t o = 0;
    for (int q = 0; q < part; ++q) {
        const int L = q / 2;
        if (q < 8) o += (q % 2 == 0) ? (int64_t)kCnnChannels[L + 1] * kCnnChannels[L] * 27 : kCnnChannels[L + 1];
        else o += (q == 8) ? 12 * kCnnFlat : 12;
    }
    return o;
}

namespace {

// K splits of a layer's weight gradient: about 600 waves (four or five per
// CU's SIMDs) of at least eight 32-voxel steps; a wave's step is a few loads
// and six MFMAs, and every split costs a copy of the gradient.
int wgrad_splits(int L, int B) {
    const int steps = B * (kSide >> (L + 1)) * (kSide >> (L + 1)) * (kSide >> (L + 1)) / 32;
    const int want = L == 1 ? 64 : (L == 2 ? 32 : 8);
    return std::max(1, std::min(want, steps / 8));
}
constexpr int kFirstGroups = 256;   // workgroups (and partials) of the first layer's weight gradient
constexpr int kDgradGroups = 1024;  // most workgroups of a data gradient (bias partials)

int dgrad_groups(int L, int B) {
    const int di = kSide >> L, h = di / 2, rt = 16 / h;
    return std::min(kDgradGroups, (B * di * 2 * (h / rt) + 3) / 4);
}

size_t fwd_weight_elems(int L) { return (size_t)kChan[L + 1] * (size_t)fwd_k(L); }

WeightForms forms_of(const CnnBuffers &c) {
    WeightForms f;
    for (int L = 0; L < 4; ++L) {
        f.fwd[L] = c.wf[L];
        f.dgrad[L] = c.wd[L];
        f.first[L] = (int)cnn_param_offset(2 * L);
        f.count[L] = kChan[L + 1] * kChan[L] * 27;
    }
    return f;
}

}  // namespace

CnnSizes cnn_sizes(int max_batch) {
    CnnSizes z;
    const size_t B = (size_t)max_batch;
    z.wpart = (size_t)kFirstGroups * 864;
    for (int L = 0; L < 4; ++L) {
        const size_t di = (size_t)(kSide >> L), d = di / 2, out = B * (size_t)kChan[L + 1] * d * d * d;
        z.wf[L] = fwd_weight_elems(L);
        z.wd[L] = L ? (size_t)kChan[L + 1] * kChan[L] * 27 : 0;
        z.act[L] = out;
        z.xs[L] = B * (size_t)kChan[L] * di * di * 3 * d;
        z.dyf[L] = out;
        z.dyl[L] = L ? out : 0;
        if (L) z.wpart += 64 * (size_t)kChan[L + 1] * kChan[L] * 27;  // (64: the most splits)
    }
    z.bpart = 3 * (size_t)kDgradGroups * 64;
    return z;
}

hipError_t cnn_prepare(const CnnBuffers &c, int max_batch, hipStream_t s) {
    // padding taps of the packed weights, and element 0 of the split form's
    // planes of x - 1, are zero for good
    const CnnSizes z = cnn_sizes(max_batch);
    for (int L = 0; L < 4; ++L) {
        hipLaunchKernelGGL(k_zero_u32, dim3(blocks((int64_t)z.wf[L] / 2)), dim3(256), 0, s, (uint32_t *)c.wf[L],
                           (int64_t)z.wf[L] / 2);
        hipLaunchKernelGGL(k_zero_u32, dim3(blocks((int64_t)z.xs[L] / 2)), dim3(256), 0, s, (uint32_t *)c.xs[L],
                           (int64_t)z.xs[L] / 2);
    }
    return cnn_refresh_bf16(c, s);
}

hipError_t cnn_downsample(const uint8_t *src, const int32_t sn[3], const uint8_t *tgt, const int32_t tn[3], float scale,
                          uint16_t *out, hipStream_t s) {
    DownArgs d;
    d.vol[0] = src;
    d.vol[1] = tgt;
    for (int e = 0; e < 3; ++e) {
        d.n[0][e] = sn[e];
        d.n[1][e] = tn[e];
    }
    d.scale = scale;
    d.out = out;
    hipLaunchKernelGGL(k_downsample, dim3(kSide * kSide * kSide / 256, 2), dim3(256), 0, s, d);
    return hipGetLastError();
}

namespace {

template <int L, int MT, int NT, int KW>
void run_conv(const uint16_t *x, const CnnBuffers &c, uint16_t *yx, int B, hipStream_t s) {
    constexpr int d = side_of(L) / 2;
    const int tiles = B * d * d * d / 16, per = KW == 1 ? 4 * MT : MT;
    hipLaunchKernelGGL((k_conv<L, MT, NT, KW>), dim3((tiles + per - 1) / per, kChan[L + 1] / (16 * NT)),
                       dim3(KW == 1 ? 256 : 64 * KW), 0, s, x, c.wf[L], c.params + cnn_param_offset(2 * L + 1),
                       c.act[L], yx, B);
}

}  // namespace

hipError_t cnn_forward(const CnnBuffers &c, const uint16_t *input, int B, float *out, bool train, hipStream_t s) {
    hipLaunchKernelGGL(k_conv_first, dim3(B * 32 * (32 / kL0Rows)), dim3(256), 0, s, input, c.wf[0],
                       c.params + cnn_param_offset(1), c.act[0], train ? c.xs[1] : nullptr);
    uint16_t *x2 = train ? c.xs[2] : nullptr, *x3 = train ? c.xs[3] : nullptr;
    // layer 1: from 16 pairs on, 64 voxels a wave (four times fewer weight
    // loads) still leave a wave per SIMD; below, K shared by four waves
    if (B >= 16) run_conv<1, 4, 2, 1>(c.act[0], c, x2, B, s);
    else run_conv<1, 1, 2, 4>(c.act[0], c, x2, B, s);
    if (B >= 8) run_conv<2, 1, 4, 4>(c.act[1], c, x3, B, s);
    else run_conv<2, 1, 1, 8>(c.act[1], c, x3, B, s);
    run_conv<3, 1, 1, 8>(c.act[2], c, nullptr, B, s);
    hipLaunchKernelGGL(k_head_fwd, dim3(12, B), dim3(256), 0, s, c.act[3], c.params + cnn_param_offset(8),
                       c.params + cnn_param_offset(9), out, kCnnFlat);
    return hipGetLastError();
}

hipError_t cnn_backward(const CnnBuffers &c, const uint16_t *input, int B, const float *out, const float *target,
                        float *loss_dev, hipStream_t s) {
    hipLaunchKernelGGL(k_nll, dim3(1), dim3(1024), 0, s, out, target, B, c.dout, loss_dev);
    hipLaunchKernelGGL(k_split_input, dim3(B * 2 * 64 * 64 * 8 / 256), dim3(256), 0, s, input,
                       (int64_t)B * 2 * 64 * 64, c.xs[0]);
    hipLaunchKernelGGL(k_head_bwd, dim3(64), dim3(256), 0, s, c.act[3], c.params + cnn_param_offset(8), c.dout, B,
                       c.grads + cnn_param_offset(8), c.grads + cnn_param_offset(9), c.dyf[3], c.dyl[3],
                       c.grads + cnn_param_offset(7));
    FinishArgs f;
    float *wp = c.wpart;
    for (int L = 0; L < 4; ++L) {
        f.wn[L] = kChan[L + 1] * kChan[L] * 27;
        f.wsplits[L] = L ? wgrad_splits(L, B) : kFirstGroups;
        f.woff[L] = (int)cnn_param_offset(2 * L);
        f.wpart[L] = wp;
        wp += (size_t)(L ? 64 : kFirstGroups) * f.wn[L];
        if (L < 3) {  // the bias gradient of layer L comes from the data gradient of layer L + 1
            f.bn[L] = kChan[L + 1];
            f.bsplits[L] = dgrad_groups(L + 1, B);
            f.boff[L] = (int)cnn_param_offset(2 * L + 1);
            f.bpart[L] = c.bpart + (size_t)L * kDgradGroups * 64;
        }
    }
    const auto wgrad = [&](auto kernel, int L, int jobs) {
        const int sp = f.wsplits[L], d = kSide >> (L + 1), steps = B * d * d * d / 32;
        const int ks = (steps + sp - 1) / sp * 32;
        hipLaunchKernelGGL(kernel, dim3((jobs * sp + 3) / 4), dim3(256), 0, s, c.dyf[L], c.xs[L],
                           const_cast<float *>(f.wpart[L]), B, ks, sp);
    };
    wgrad(k_wgrad<3, 1>, 3, 9 * 4 * 2);
    hipLaunchKernelGGL((k_dgrad<3, 1>), dim3(f.bsplits[2], 4), dim3(256), 0, s, c.dyl[3], c.wd[3], c.xs[3], c.dyf[2],
                       c.dyl[2], const_cast<float *>(f.bpart[2]), B);
    wgrad(k_wgrad<2, 2>, 2, 9 * 1 * 2);
    hipLaunchKernelGGL((k_dgrad<2, 2>), dim3(f.bsplits[1], 1), dim3(256), 0, s, c.dyl[2], c.wd[2], c.xs[2], c.dyf[1],
                       c.dyl[1], const_cast<float *>(f.bpart[1]), B);
    wgrad(k_wgrad<1, 1>, 1, 9);
    hipLaunchKernelGGL((k_dgrad<1, 1>), dim3(f.bsplits[0], 1), dim3(256), 0, s, c.dyl[1], c.wd[1], c.xs[1], c.dyf[0],
                       (uint16_t *)nullptr, const_cast<float *>(f.bpart[0]), B);
    hipLaunchKernelGGL(k_wgrad_first, dim3(kFirstGroups), dim3(256), 0, s, c.dyf[0], c.xs[0],
                       const_cast<float *>(f.wpart[0]), B);
    const int weights = f.wn[0] + f.wn[1] + f.wn[2] + f.wn[3], wblocks = (weights + 255) / 256;
    const int biases = f.bn[0] + f.bn[1] + f.bn[2];
    hipLaunchKernelGGL(k_grads_finish, dim3(wblocks + (biases + 3) / 4), dim3(256), 0, s, f, wblocks, c.grads);
    return hipGetLastError();
}

hipError_t cnn_adam(const CnnBuffers &c, float lr, int t, hipStream_t s) {
    const double b1 = 0.9, b2 = 0.999;
    const float c1 = (float)(1.0 - pow(b1, (double)t)), c2 = (float)(1.0 - pow(b2, (double)t));
    hipLaunchKernelGGL(k_adam, dim3(blocks(c.n_params)), dim3(256), 0, s, c.params, c.grads, c.adam_m, c.adam_v,
                       forms_of(c), (int64_t)c.n_params, lr, (float)b1, (float)(1.0 - b1), (float)b2,
                       (float)(1.0 - b2), c1, c2, 1e-8f);
    return hipGetLastError();
}

hipError_t cnn_refresh_bf16(const CnnBuffers &c, hipStream_t s) {
    const int64_t n = cnn_param_offset(8);
    hipLaunchKernelGGL(k_pack_weights, dim3(blocks(n)), dim3(256), 0, s, c.params, forms_of(c), n);
    return hipGetLastError();
}

}  // namespace smc
