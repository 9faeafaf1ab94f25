// Learned proposal network: downsampling to 64^3, four 3x3x3 stride-2
// convolutions (2 -> 16 -> 32 -> 64 -> 64 channels, zero padding 1, bias,
// ReLU), a linear head to 6 means and 6 log-variances, the Gaussian NLL of
// the filter's final weighted cloud, its backward pass and Adam.
//
// Convolutions are implicit GEMMs on v_mfma_f32_16x16x32_bf16.
//   forward  C[m = output voxel][n = c_out]  K = (c_in, kz, ky, kx)
//   dgrad    C[m = input voxel][n = c_in]    K = (c_out, kz, ky, kx).  A stride-2
//            kernel reaches an input voxel by one tap per axis where its
//            coordinate is even and by two where it is odd; a tile's rows have
//            one parity
//   wgrad    C[m = c_out][n = (tap, c_in)]   K = output voxel
// The order of the sums of the first two is fixed: 32 consecutive K an
// instruction at their places in it, and for the forward the chains of
// instructions and the order of their sums that fwd_split describes.  Activations
// and dY are rounded to bfloat16, where another order of FP32 sums turns some
// roundings and moves a training step's gradients by up to 1e-4.
// So their operand from the activations (dY) is gathered: a workgroup stages
// what its tiles read in LDS, where a lane's eight K are eight 2-byte reads at
// offsets from a table (forward) or four reads of two neighbouring x (dgrad:
// the three kx of a (c_out, kz, ky) need no more, for both parities of x);
// weights are 16-byte loads in K order.  wgrad, whose sums are rounded to no
// less than FP32, reads 16 bytes of consecutive K for both operands: dY channels
// first; X "split": [c][z][y][3][x / 2], the planes holding x - 1 (odd), x
// (even) and x + 1 (odd) of an output voxel's three taps.  Its K is split over
// waves, whose partial sums k_grads_finish adds in a fixed order (no
// floating-point atomics: a training step is reproducible bit for bit).
// Weights, activations and the operands of all products are bfloat16 (round to
// nearest even), accumulation FP32, gradients FP32; dY is rounded once, after
// its bias gradient has been summed from the FP32 values.
//
// What it measured: a training step of 32 pairs (inputs, backward with the
// gradients read back, Adam) 5.67 ms with every operand gathered element by
// element from memory (dgrad 2.3, bias gradients 1.2, wgrad 1.1, forward 0.58),
// 0.68 ms so (dgrad 0.076, wgrad 0.13, forward 0.098, the 32 downsamplings
// 0.122); a proposal of one pair 94 -> 47 us.  With K in the order (tap, channel),
// whose operands are 16-byte loads without LDS, the forward and the dgrad took
// as long (0.103 and 0.089 ms, a step 0.70).  Weights in rows of K made a wave's
// load touch sixteen lines: dgrad 0.097 ms, 0.076 in the order of weight_at.
// Bound: latency -- 4 to 45 us kernels of a few thousand waves, launches, and the
// copy of the gradients to the host.
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
// Place of weight (K k, column n) in the order in which waves load them: 1 KB
// for each 16 columns and 32 K, sixteen bytes a lane.
constexpr int kWeightBlock = 512;
__device__ __forceinline__ int weight_at(int k, int n, int steps) {
    return ((n / 16) * steps + k / 32) * kWeightBlock + (k % 32 / 8 * 16 + n % 16) * 8 + k % 8;
}

// Lane l of a wave holds A[l % 16][8 (l / 16) + i] and B[8 (l / 16) + i][l % 16],
// i = 0..7, of v_mfma_f32_16x16x32_bf16, and C[4 (l / 16) + i][l % 16], i = 0..3.
__device__ __forceinline__ v4f mfma(bf16x8 a, bf16x8 b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

constexpr int kChan[5] = {2, 16, 32, 64, 64};
constexpr int kSide = 64;
constexpr int side_of(int L) { return kSide >> L; }  // input side of layer L
// K of a forward layer's packed weights: 27 c_in rounded up to 32.
constexpr int fwd_k(int L) { return (27 * kChan[L] + 31) / 32 * 32; }

// ---- forward --------------------------------------------------------------------

// Activation (ReLU, bf16) of four consecutive output voxels m .. m + 3 (one
// row of side DO) of channel n: channels first, and for training the split form
// that the next layer's wgrad reads.
template <int CO, int DO>
__device__ __forceinline__ void store_act(const float v[4], int m, int n, uint16_t *y, uint16_t *yx) {
    constexpr int VOX = DO * DO * DO;
    const int b = m / VOX, r = m - b * VOX;
    uint16_t h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = to_bf16(v[i]);
    *(u32x2 *)(y + ((size_t)b * CO + n) * VOX + r) =
        u32x2{(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16)};
    if (yx) {
        const int x = r % DO;
        uint16_t *row = yx + (((size_t)b * CO + n) * (DO * DO) + r / DO) * (3 * (DO / 2)) + x / 2;
        *(uint32_t *)(row + DO / 2) = (uint32_t)h[0] | ((uint32_t)h[2] << 16);
        *(uint32_t *)(row + DO) = (uint32_t)h[1] | ((uint32_t)h[3] << 16);
        row[1] = h[1];  // (element 0 of the plane of x - 1 stays zero)
        if (x / 2 + 2 < DO / 2) row[2] = h[3];
    }
}

// The input rows that R output rows of one slice read, in LDS as bf16: row (c,
// kz, y) of NY, element x at x + 4 (x = -1 and rows outside are zero).  Past
// them zeros for the K that only fill the last instruction.
template <int L, int R>
struct Patch {
    static constexpr int CI = kChan[L], DI = side_of(L), DO = DI / 2, NY = 2 * R + 1, P = DI + 4, K = 27 * CI;
    static constexpr int ROWS = CI * 3 * NY, ZEROS = K % 32 ? 2 * (R - 1) * P + 2 * DO : 0;
    static constexpr int ELEMS = (ROWS * P + ZEROS + 7) / 8 * 8, KP = fwd_k(L);
    static_assert(2 * ELEMS < 65536, "byte offsets of 16 bits");
};

// Fill a patch and its offsets in K order (bytes from the place of tap 0 of an
// output voxel).
template <int L, int R, int THREADS>
__device__ __forceinline__ void stage_patch(const uint16_t *X, int b, int oz, int oy0, uint16_t *patch,
                                            uint16_t *koff) {
    using S = Patch<L, R>;
    constexpr int CHUNKS = S::DI / 8, N = (S::ROWS * CHUNKS + THREADS - 1) / THREADS, AHEAD = N < 3 ? N : 3;
    u32x4 v[AHEAD];
    const auto load = [&](int first) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const int q = (int)threadIdx.x + THREADS * (first + i), row = q / CHUNKS, x = 8 * (q % CHUNKS);
            const int z = 2 * oz + row / S::NY % 3 - 1, y = 2 * oy0 + row % S::NY - 1, c = row / (3 * S::NY);
            v[i] = u32x4{0u, 0u, 0u, 0u};
            if (row < S::ROWS && z >= 0 && y >= 0)
                v[i] = *(const u32x4 *)(X + (((size_t)b * S::CI + c) * S::DI + z) * (S::DI * S::DI) + y * S::DI + x);
        }
    };
    const auto store = [&](int first) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const int q = (int)threadIdx.x + THREADS * (first + i), row = q / CHUNKS, x = 8 * (q % CHUNKS);
            if (row >= S::ROWS) break;
            if (L == 0) {  // (the network's input is FP16)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    v[i][e] = pair_bf16(__half2float(__ushort_as_half((uint16_t)(v[i][e] & 0xFFFFu))),
                                        __half2float(__ushort_as_half((uint16_t)(v[i][e] >> 16))));
            }
            uint16_t *d = patch + row * S::P + x + 4;
            *(u32x2 *)d = u32x2{v[i].x, v[i].y};
            *(u32x2 *)(d + 4) = u32x2{v[i].z, v[i].w};
            if (x == 0) *(u32x2 *)(d - 4) = u32x2{0u, 0u};
        }
    };
    load(0);
    for (int k = (int)threadIdx.x; k < S::KP; k += THREADS) {
        const int c = k / 27, t = k % 27, kz = t / 9, ky = t / 3 % 3, kx = t % 3;
        koff[k] = (uint16_t)(2 * (k < S::K ? ((c * 3 + kz) * S::NY + ky) * S::P + 3 + kx : S::ROWS * S::P));
    }
    for (int q = S::ROWS * S::P + (int)threadIdx.x; q < S::ELEMS; q += THREADS) patch[q] = 0;
    store(0);
#pragma unroll 1
    for (int first = AHEAD; first < N; first += AHEAD) {
        load(first);
        store(first);
    }
}

// Eight K of an output voxel whose tap 0 lies at p; o: their offsets.
__device__ __forceinline__ bf16x8 gather8(const uint16_t *p, u32x4 o) {
    const uint8_t *b = (const uint8_t *)p;
    u32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        v[e] = (uint32_t) * (const uint16_t *)(b + (o[e] & 0xFFFFu)) |
               ((uint32_t) * (const uint16_t *)(b + (o[e] >> 16)) << 16);
    return __builtin_bit_cast(bf16x8, v);
}

// First layer: a workgroup takes four output rows of one slice, a wave one of
// them.  Its two instructions are two chains.
constexpr int kL0Rows = 4;
__global__ __launch_bounds__(256) void k_conv_first(const uint16_t *X, const uint16_t *W, const float *bias,
                                                    uint16_t *y, uint16_t *yx) {
    using S = Patch<0, kL0Rows>;
    constexpr int DO = S::DO;
    __shared__ __attribute__((aligned(16))) uint16_t patch[S::ELEMS];
    __shared__ __attribute__((aligned(16))) uint16_t koff[S::KP];
    const int b = blockIdx.x / (DO * (DO / kL0Rows)), rem = blockIdx.x % (DO * (DO / kL0Rows));
    const int oz = rem / (DO / kL0Rows), oy0 = rem % (DO / kL0Rows) * kL0Rows;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, r = lane % 16, g = lane / 16;
    bf16x8 w[2];
    u32x4 o[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) w[s] = load8(W + s * kWeightBlock + 8 * lane);
    const float bn = bias[r];
    stage_patch<0, kL0Rows, 256>(X, b, oz, oy0, patch, koff);
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 2; ++s) o[s] = *(const u32x4 *)(koff + 32 * s + 8 * g);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const uint16_t *p = patch + 2 * wave * S::P + 2 * (16 * t + r);
        const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
        const v4f acc = mfma(gather8(p, o[0]), w[0], zero) + mfma(gather8(p, o[1]), w[1], zero);
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = fmaxf(acc[i] + bn, 0.0f);
        const int m = ((b * DO + oz) * DO + oy0 + wave) * DO + 16 * t + 4 * g;
        store_act<16, DO>(v, m, r, y, yx);
    }
}

// Layers 1 .. 3: a workgroup takes R output rows of one slice (MT tiles of 16
// voxels) and NT tiles of 16 channels.  The K steps of 32 fall into `splits`
// ranges of `per` steps, and those of a range into four chains (every fourth
// step): wave q takes chains q, q + WAVES, .. (CH at most), and a tile's sum is
// the ranges' in order, each its four chains' in order.
template <int L, int R, int NT, int WAVES, int CH>
__global__ __launch_bounds__(64 * WAVES) void k_conv(const uint16_t *X, const uint16_t *W, const float *bias,
                                                    uint16_t *y, uint16_t *yx, int splits, int per) {
    using S = Patch<L, R>;
    constexpr int CO = kChan[L + 1], DO = S::DO, MT = R * DO / 16, STEPS = S::KP / 32, GROUPS = DO / R;
    constexpr int TILE = (16 / DO) * 2 * S::P;  // elements from a tile's rows to the next one's
    constexpr size_t STAGE = 2 * (S::ELEMS + S::KP), SUMS = (size_t)WAVES * CH * MT * NT * 64 * sizeof(v4f);
    __shared__ __attribute__((aligned(16))) uint8_t lds[STAGE > SUMS ? STAGE : SUMS];
    uint16_t *patch = (uint16_t *)lds, *koff = patch + S::ELEMS;
    v4f *sums = (v4f *)lds;  // (after the products: [chain][tile][lane])
    const int b = blockIdx.x / (DO * GROUPS), rem = blockIdx.x % (DO * GROUPS);
    const int oz = rem / GROUPS, oy0 = rem % GROUPS * R, n0 = blockIdx.y * NT * 16;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, r = lane % 16, g = lane / 16;
    const uint16_t *p = patch + 2 * (r / DO) * S::P + 2 * (r % DO);
    const uint16_t *w0 = W + (size_t)(n0 / 16) * STEPS * kWeightBlock + 8 * lane;
    // a chain's weights are loaded a step ahead, its first ones before the patch
    bf16x8 w[CH][NT];
    int begin[CH], end[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int chain = wave + WAVES * c, range = chain / 4;
        begin[c] = range * per + chain % 4;
        end[c] = range < splits ? min(STEPS, (range + 1) * per) : 0;
#pragma unroll
        for (int n = 0; n < NT; ++n) w[c][n] = load8(w0 + (n * STEPS + min(begin[c], STEPS - 1)) * kWeightBlock);
    }
    stage_patch<L, R, 64 * WAVES>(X, b, oz, oy0, patch, koff);
    __syncthreads();
    v4f acc[CH][MT][NT];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int n = 0; n < NT; ++n) acc[c][t][n] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 2
        for (int s = begin[c]; s < end[c]; s += 4) {
            const u32x4 o = *(const u32x4 *)(koff + 32 * s + 8 * g);
            bf16x8 a[MT], now[NT];
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                now[n] = w[c][n];
                w[c][n] = load8(w0 + (n * STEPS + min(s + 4, STEPS - 1)) * kWeightBlock);
            }
#pragma unroll
            for (int t = 0; t < MT; ++t) a[t] = gather8(p + t * TILE, o);
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int n = 0; n < NT; ++n) acc[c][t][n] = mfma(a[t], now[n], acc[c][t][n]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int n = 0; n < NT; ++n)
                sums[((wave + WAVES * c) * MT * NT + t * NT + n) * 64 + lane] = acc[c][t][n];
    __syncthreads();
    for (int q = wave; q < MT * NT; q += WAVES) {
        const v4f *from = sums + q * 64 + lane;
        v4f total = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
        for (int range = 0; range < splits; ++range) {
            v4f sum = from[(4 * range) * MT * NT * 64];
#pragma unroll
            for (int c = 1; c < 4; ++c) sum += from[(4 * range + c) * MT * NT * 64];
            total += sum;
        }
        const int t = q / NT, n = n0 + 16 * (q % NT) + r, at = 16 * t + 4 * g;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = fmaxf(total[i] + bias[n], 0.0f);
        store_act<CO, DO>(v, ((b * DO + oz) * DO + oy0) * DO + at, n, y, yx);
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

// What the data gradient of layer L stages in LDS: the dY rows that kDgradRows
// pairs of input rows in a pair of slices read, as dwords (v[x], v[x + 1]), row
// (c_out, dz, dy); past them zeros for taps that do not reach.
constexpr int kDgradRows = 4;
template <int L>
struct Reach {
    static constexpr int CO = kChan[L + 1], H = side_of(L) / 2, NY = kDgradRows + 1, ROWS = CO * 2 * NY;
    static constexpr int ZERO = ROWS * H, DWORDS = ZERO + kDgradRows * H, STEPS = 27 * CO / 32;
    static_assert(4 * DWORDS < 65536, "byte offsets of 16 bits");
};

// Offsets of the (c_out, kz, ky) that a lane's eight K belong to: four of 16
// bits at [(z parity, y parity)][step][lane / 16].
template <int L>
__global__ void k_reach(uint2 *out) {
    using S = Reach<L>;
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= 4 * S::STEPS * 4) return;
    const int g = q % 4, s = q / 4 % S::STEPS, pz = q / (8 * S::STEPS), py = q / (4 * S::STEPS) % 2;
    uint32_t o[4];
    for (int i = 0; i < 4; ++i) {
        const int t = (32 * s + 8 * g) / 3 + i, c = t / 9, kz = t / 3 % 3, ky = t % 3;
        // even coordinates: tap 1 of output m; odd: tap 0 of m + 1 and tap 2 of m
        const bool ok = c < S::CO && (kz == 1) != (pz == 1) && (ky == 1) != (py == 1);
        o[i] = 4u * (uint32_t)(ok ? ((c * 2 + (kz == 0 ? 1 : 0)) * S::NY + (ky == 0 ? 1 : 0)) * S::H : S::ZERO);
    }
    out[q] = make_uint2(o[0] | (o[1] << 16), o[2] | (o[3] << 16));
}

// Selector for v_perm_b32 (first: bytes 0 .. 3, second: 4 .. 7) of the K pair
// 2 d, 2 d + 1 of a lane whose K begin at kx = a: the elements of a triple (kx = 0,
// 1, 2) are (v[x + 1], 0, v[x]) at odd input x and (0, v[x], 0) at even; first
// is the triple of number from, second the next.
__device__ __forceinline__ uint32_t pair_selector(int a, int d, int from, bool odd) {
    uint32_t s = 0u;
    for (int e = 0; e < 2; ++e) {
        const int pos = a + 2 * d + e, kx = pos % 3, second = pos / 3 - from;
        const uint32_t bytes = odd ? (kx == 1 ? 0x0C0Cu : (kx == 0 ? 0x0302u : 0x0100u)) : (kx == 1 ? 0x0100u : 0x0C0Cu);
        s |= (bytes == 0x0C0Cu ? bytes : bytes + (second ? 0x0404u : 0u)) << (16 * e);
    }
    return s;
}

// dL/dX of layer L masked by the ReLU that made X: the dY of layer L - 1.  A
// unit is a pair of input slices and kDgradRows pairs of rows; a wave takes one
// parity of z and y, and 16 pairs of voxels (x = 2 mx, 2 mx + 1) a tile, of which
// a lane holds four: eight consecutive x.  Workgroups take units in strides and
// keep the channels' sums, the bias gradient of layer L - 1.
template <int L, int NT>
__global__ __launch_bounds__(256) void k_dgrad(const uint16_t *dY, const uint16_t *W, const uint2 *reach,
                                               const uint16_t *X, uint16_t *dx, float *bias_part, int B) {
    using S = Reach<L>;
    constexpr int CI = kChan[L], CO = S::CO, DI = side_of(L), H = S::H, RT = 16 / H, T = kDgradRows / RT;
    constexpr int CHUNK = H < 8 ? H : 8, CHUNKS = H / CHUNK, GROUPS = H / kDgradRows;
    __shared__ uint32_t patch[S::DWORDS];
    __shared__ float red[4][NT][16];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, r = lane % 16, g = lane / 16;
    const int n0 = blockIdx.y * NT * 16;
    // the selectors of three consecutive steps (a step of 32 moves a by 2)
    uint32_t sel[3][2][4];
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int d = 0; d < 4; ++d) sel[s][o][d] = pair_selector((2 * s + 2 * g) % 3, d, d < 2 ? 0 : d - 1, o != 0);
    for (int q = S::ZERO + (int)threadIdx.x; q < S::DWORDS; q += 256) patch[q] = 0u;
    const uint8_t *base = (const uint8_t *)(patch + (r / H) * H + r % H);
    const uint2 *offs = reach + (size_t)wave * S::STEPS * 4 + g;
    const uint16_t *w0 = W + (size_t)(n0 / 16) * S::STEPS * kWeightBlock + 8 * lane;
    const int pz = wave / 2, py = wave % 2;
    float bsum[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) bsum[n] = 0.0f;
    for (int unit = blockIdx.x; unit < B * H * GROUPS; unit += gridDim.x) {
        const int b = unit / (H * GROUPS), mz = unit / GROUPS % H, my0 = unit % GROUPS * kDgradRows;
        __syncthreads();  // the patch before has been read
        for (int q = (int)threadIdx.x; q < S::ROWS * CHUNKS; q += 256) {
            const int row = q / CHUNKS, x = CHUNK * (q % CHUNKS);
            const int oy = my0 + row % S::NY, oz = mz + row / S::NY % 2, c = row / (2 * S::NY);
            uint32_t v[CHUNK / 2], next = 0u;
#pragma unroll
            for (int e = 0; e < CHUNK / 2; ++e) v[e] = 0u;
            if (oy < H && oz < H) {
                const uint16_t *from = dY + (((size_t)b * CO + c) * H + oz) * (H * H) + oy * H + x;
                __builtin_memcpy(v, __builtin_assume_aligned(from, 2 * CHUNK), 2 * CHUNK);
                if (x + CHUNK < H) next = from[CHUNK];
            }
            uint32_t *to = patch + row * H + x;
#pragma unroll
            for (int e = 0; e < CHUNK / 2; ++e) {
                to[2 * e] = v[e];
                to[2 * e + 1] = (v[e] >> 16) | ((e + 1 < CHUNK / 2 ? v[e + 1 < CHUNK / 2 ? e + 1 : e] : next) << 16);
            }
        }
        __syncthreads();
        v4f acc[2][T][NT];
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int n = 0; n < NT; ++n) acc[o][t][n] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        // (offsets and weights of three steps are loaded while the three before run)
        uint2 o3[3];
        bf16x8 w3[3][NT];
        const auto load3 = [&](int s0) {
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const int s = min(s0 + p, S::STEPS - 1);
                o3[p] = offs[4 * s];
#pragma unroll
                for (int n = 0; n < NT; ++n) w3[p][n] = load8(w0 + (n * S::STEPS + s) * kWeightBlock);
            }
        };
        load3(0);
        for (int s0 = 0; s0 < S::STEPS; s0 += 3) {
            uint2 off[3];
            bf16x8 w[3][NT];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                off[p] = o3[p];
#pragma unroll
                for (int n = 0; n < NT; ++n) w[p][n] = w3[p][n];
            }
            load3(s0 + 3);
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const uint2 o = off[p];
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const uint8_t *at = base + 4 * t * RT * H;
                    const uint32_t q[4] = {*(const uint32_t *)(at + (o.x & 0xFFFFu)), *(const uint32_t *)(at + (o.x >> 16)),
                                           *(const uint32_t *)(at + (o.y & 0xFFFFu)), *(const uint32_t *)(at + (o.y >> 16))};
#pragma unroll
                    for (int odd = 0; odd < 2; ++odd) {
                        u32x4 a;
#pragma unroll
                        for (int d = 0; d < 4; ++d) {
                            const int from = d < 2 ? 0 : d - 1;
                            a[d] = __builtin_amdgcn_perm(q[from + 1], q[from], sel[p][odd][d]);
                        }
#pragma unroll
                        for (int n = 0; n < NT; ++n)
                            acc[odd][t][n] = mfma(__builtin_bit_cast(bf16x8, a), w[p][n], acc[odd][t][n]);
                    }
                }
            }
        }
        // the lane's pairs of a tile: m = 4 g .. 4 g + 3
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int x0 = 2 * ((4 * g) % H), iy = 2 * (my0 + t * RT + 4 * g / H) + py, iz = 2 * mz + pz;
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const int c = n0 + 16 * n + r;
                const size_t o = (((size_t)b * CI + c) * DI + iz) * (DI * DI) + iy * DI + x0;
                const u32x4 x = *(const u32x4 *)(X + o);
                float v[8];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[2 * i] = (x[i] & 0xFFFFu) ? acc[0][t][n][i] : 0.0f;
                    v[2 * i + 1] = (x[i] >> 16) ? acc[1][t][n][i] : 0.0f;
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) bsum[n] += v[i];
                *(u32x4 *)(dx + o) =
                    u32x4{pair_bf16(v[0], v[1]), pair_bf16(v[2], v[3]), pair_bf16(v[4], v[5]), pair_bf16(v[6], v[7])};
            }
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
// (b, j); a thread takes every 256th f, and the threads' sums meet in halves.
__global__ __launch_bounds__(256) void k_head_fwd(const uint16_t *h, const float *Wh, const float *bh, float *out,
                                                  int F) {
    const int b = blockIdx.y, j = blockIdx.x;
    float s = 0.0f;
#pragma unroll 16
    for (int f = threadIdx.x; f < F; f += 256) s += from_bf16(h[(size_t)b * F + f]) * Wh[(size_t)j * F + f];
    __shared__ float red[256];
    red[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const float *v = red + threadIdx.x;
    s = (v[0] + v[128]) + (v[64] + v[192]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (threadIdx.x == 0) out[(size_t)b * 12 + j] = s + bh[j];
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
// Wh[j][f]) masked by h > 0 (the dY of the last layer), and its sum over b and
// voxels, the last layer's bias gradient.  Wave w takes every
// fourth b, a lane a voxel.  Workgroup 0 adds dbh[j] = sum_b dout[b][j].
__global__ __launch_bounds__(256) void k_head_bwd(const uint16_t *h, const float *Wh, const float *dout, int B,
                                                  float *dWh, float *dbh, uint16_t *dy, float *db) {
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
        dy[(size_t)b * F + f] = to_bf16(s);
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
// the forward's K = (c_in, tap), n = c_out and the dgrad's K = (c_out, tap), n = c_in.
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
        f.fwd[L][weight_at(ci * 27 + t, co, fwd_k(L) / 32)] = v;
        if (L) f.dgrad[L][weight_at(co * 27 + t, ci, 27 * chan[L + 1] / 32)] = v;
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
    const int h = kSide >> (L + 1);
    return std::min(kDgradGroups, B * h * (h / kDgradRows));
}

// Ranges of a forward layer's K steps, and steps of a range: part of the order
// of its sums (about 512 workgroups of one tile and one range; whatever the
// workgroups of k_conv are, the sums stay those).
struct FwdSplit {
    int ranges, steps;
};
FwdSplit fwd_split(int L, int B) {
    const int d = kSide >> (L + 1), tiles = B * d * d * d / 16 * (kChan[L + 1] / 16), steps = fwd_k(L) / 32;
    const int want = std::max(1, std::min((512 + tiles - 1) / tiles, steps / 4));
    const int per = (steps + want - 1) / want;
    return {(steps + per - 1) / per, per};
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
        z.dy[L] = out;
        z.reach[L] = L ? 4 * 4 * (27 * (size_t)kChan[L + 1] / 32) : 0;
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
    const auto reach = [&](auto kernel, int L) {
        hipLaunchKernelGGL(kernel, dim3(blocks((int64_t)z.reach[L])), dim3(256), 0, s, (uint2 *)c.reach[L]);
    };
    reach(k_reach<1>, 1);
    reach(k_reach<2>, 2);
    reach(k_reach<3>, 3);
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

template <int L, int R, int NT, int WAVES, int CH>
void run_conv(const CnnBuffers &c, uint16_t *yx, int B, hipStream_t s) {
    constexpr int d = side_of(L) / 2;
    const FwdSplit f = fwd_split(L, B);
    hipLaunchKernelGGL((k_conv<L, R, NT, WAVES, CH>), dim3(B * d * (d / R), kChan[L + 1] / (16 * NT)), dim3(64 * WAVES),
                       0, s, c.act[L - 1], c.wf[L], c.params + cnn_param_offset(2 * L + 1), c.act[L], yx, f.ranges,
                       f.steps);
}

}  // namespace

hipError_t cnn_forward(const CnnBuffers &c, const uint16_t *input, int B, float *out, bool train, hipStream_t s) {
    hipLaunchKernelGGL(k_conv_first, dim3(B * 32 * (32 / kL0Rows)), dim3(256), 0, s, input, c.wf[0],
                       c.params + cnn_param_offset(1), c.act[0], train ? c.xs[1] : nullptr);
    uint16_t *x2 = train ? c.xs[2] : nullptr, *x3 = train ? c.xs[3] : nullptr;
    // four output rows a workgroup share their weights and most of their input
    // rows where that still leaves two workgroups a CU (layer 1) or one (layer 2)
    if (B >= 8) run_conv<1, 4, 2, 4, 1>(c, x2, B, s);
    else run_conv<1, 1, 2, 4, 1>(c, x2, B, s);
    // several ranges of K: up to 4 (16 chains) in layer 2, 11 (44) in layer 3
    if (fwd_split(2, B).ranges > 1) run_conv<2, 2, 1, 8, 2>(c, x3, B, s);
    else if (B >= 16) run_conv<2, 4, 4, 4, 1>(c, x3, B, s);
    else run_conv<2, 2, 2, 4, 1>(c, x3, B, s);
    if (fwd_split(3, B).ranges > 1) run_conv<3, 4, 1, 16, 3>(c, nullptr, B, s);
    else run_conv<3, 4, 1, 4, 1>(c, nullptr, B, s);
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
                       c.grads + cnn_param_offset(8), c.grads + cnn_param_offset(9), c.dy[3],
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
        hipLaunchKernelGGL(kernel, dim3((jobs * sp + 3) / 4), dim3(256), 0, s, c.dy[L], c.xs[L],
                           const_cast<float *>(f.wpart[L]), B, ks, sp);
    };
    wgrad(k_wgrad<3, 1>, 3, 9 * 4 * 2);
    const auto dgrad = [&](auto kernel, int L, int parts) {
        hipLaunchKernelGGL(kernel, dim3(f.bsplits[L - 1], parts), dim3(256), 0, s, c.dy[L], c.wd[L],
                           (const uint2 *)c.reach[L], c.act[L - 1], c.dy[L - 1], const_cast<float *>(f.bpart[L - 1]), B);
    };
    dgrad(k_dgrad<3, 1>, 3, 4);
    wgrad(k_wgrad<2, 2>, 2, 9 * 1 * 2);
    dgrad(k_dgrad<2, 2>, 2, 1);
    wgrad(k_wgrad<1, 1>, 1, 9);
    dgrad(k_dgrad<1, 1>, 1, 1);
    hipLaunchKernelGGL(k_wgrad_first, dim3(kFirstGroups), dim3(256), 0, s, c.dy[0], c.xs[0],
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
