// Once-per-pair preparation: packed mask / FOV bytes, the trilinear
// corner-validity mask of the source FOV, and exact per-volume sums
// (FOV voxel count, nonzero count, sum and sum of squares) from which the
// host derives |T| for Dice, the minimum overlap and the mean-0 / std-1
// normalisation statistics of Implementation Details.
#include <stdint.h>

#include <algorithm>

#include "internal.h"

namespace smc {
namespace {

// Voxel indices are 32 bits wide (a volume has fewer than 2^31 voxels; a grid
// stride past the last one stays below 2^32): a 64-bit division per voxel cost
// more than the memory traffic.
struct Cell {
    uint32_t i, j, k;
};
__device__ __forceinline__ Cell cell_of(uint32_t q, uint32_t nx, uint32_t ny) {
    const uint32_t row = q / nx, k = row / ny;
    return {q - row * nx, row - k * ny, k};
}

// Rows of the source, kRows at a time by a wave, lanes along x: the voxel bytes,
// and the bitmaps that the distance field starts from, made from ballots
// (bit 31 - x % 32 of dword y + ny (x / 32 + W z), pad bits zero).
//
// MASK: the prepared byte (bit 0: inside the FOV, no FOV = everywhere; bit 1:
// nonzero and inside), and the bitmap of bit 1.
// Otherwise: the corner-validity byte -- a trilinear sample with base corner
// (i, j, k) is valid iff all eight (edge-clamped) corners are inside the FOV --
// and the bitmaps of the cells a valid sample may lie in (ok) and must lie in
// to be certainly valid (those below the last index of every axis: at the last
// index only the exact coordinate is inside).
//
// One pass where bytes and bitmaps took two (8.2 M voxels, masks: 8 + 18 us;
// 4.1 M, validity: 20 + 11 us); now 15 and 16 us.
constexpr uint32_t kRows = 8;
template <bool MASK>
__global__ __launch_bounds__(256) void k_source_rows(const uint8_t *vol, const uint8_t *fov, uint32_t nx, uint32_t ny,
                                                     uint32_t nz, uint32_t W, uint8_t *out, uint32_t *may,
                                                     uint32_t *must) {
    const uint32_t rows = ny * nz, chunks = (nx + 63) / 64, lane = threadIdx.x % 64;
    const uint32_t n = (rows + kRows - 1) / kRows * chunks;
    for (uint32_t w = blockIdx.x * 4 + threadIdx.x / 64; w < n; w += gridDim.x * 4) {
        const uint32_t group = w / chunks, c = w - group * chunks;
        const uint32_t x = c * 64 + lane;
        uint64_t mine = 0ull, mine_must = 0ull;  // lane r: the ballots of row r
#pragma unroll
        for (uint32_t r = 0; r < kRows; ++r) {
            const uint32_t row = group * kRows + r;
            bool on = false, sure = false;
            if (row < rows && x < nx) {
                const uint32_t q = row * nx + x;
                if (MASK) {
                    const uint32_t in = fov ? (fov[q] != 0) : 1u;
                    on = in && vol[q] != 0;
                    out[q] = (uint8_t)(in | (on ? 2u : 0u));
                } else {
                    const uint32_t k = row / ny, j = row - k * ny;
                    const bool ex = x + 1 < nx, ey = j + 1 < ny, ez = k + 1 < nz;
                    const uint32_t dx = ex ? 1u : 0u, dy = ey ? nx : 0u, dz = ez ? nx * ny : 0u;
                    on = (fov[q] != 0) & (fov[q + dx] != 0) & (fov[q + dy] != 0) & (fov[q + dx + dy] != 0) &
                         (fov[q + dz] != 0) & (fov[q + dz + dx] != 0) & (fov[q + dz + dy] != 0) &
                         (fov[q + dz + dy + dx] != 0);
                    out[q] = on ? 1 : 0;
                    sure = on & ex & ey & ez;
                }
            }
            const uint64_t b = __ballot(on), m = MASK ? 0ull : __ballot(sure);
            if (lane == r) {
                mine = b;
                mine_must = m;
            }
        }
        const uint32_t row = group * kRows + lane;
        if (lane < kRows && row < rows) {
            const uint32_t z = row / ny, y = row - z * ny;
            for (uint32_t h = 0; h < 2 && 2 * c + h < W; ++h) {
                const uint32_t o = y + ny * (2 * c + h + W * z);
                may[o] = __brev((uint32_t)(mine >> (32 * h)));
                if (!MASK) must[o] = __brev((uint32_t)(mine_must >> (32 * h)));
            }
        }
    }
}

// Per volume (blockIdx.y): FOV voxels, nonzero ones, sum and sum of squares.
// Sixteen bytes a load at any address, few workgroups: every one ends in four
// atomics on the same words, and 4096 of them took 53 us for 4.1 MB, twice; 128
// take 9 us for both volumes.  (With a byte a load for volumes that are not 16-byte
// aligned, smc_init of 800^3 images at an odd address took 9.0 ms, 2.6 so.)
struct SumsOf {
    const uint8_t *vol[2], *fov[2];
    uint32_t n[2];
};
constexpr uint32_t kSumBlocks = 128;

__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t v) {  // 1 in each byte that is not zero
    return ((((v & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | v) >> 7) & 0x01010101u;
}

__global__ __launch_bounds__(256) void k_volume_sums(const SumsOf a, unsigned long long *out) {
    const uint8_t *vol = a.vol[blockIdx.y], *fov = a.fov[blockIdx.y];
    const uint32_t n = a.n[blockIdx.y], stride = gridDim.x * 256, t = blockIdx.x * 256 + threadIdx.x;
    const uint32_t n16 = n / 16;
    unsigned long long red4[4] = {0ull, 0ull, 0ull, 0ull};
    for (uint32_t q = t; q < n16; q += stride) {
        uint4 v4, f4 = make_uint4(~0u, ~0u, ~0u, ~0u);
        __builtin_memcpy(&v4, vol + 16 * (size_t)q, 16);
        if (fov) __builtin_memcpy(&f4, fov + 16 * (size_t)q, 16);
        const uint32_t v[4] = {v4.x, v4.y, v4.z, v4.w}, f[4] = {f4.x, f4.y, f4.z, f4.w};
        uint32_t c = 0u, o = 0u, s1 = 0u, s2 = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t in = nonzero_bytes(f[e]), x = v[e] & (in * 255u);
            c += (uint32_t)__popc(in);
            o += (uint32_t)__popc(nonzero_bytes(x));
            s1 = __builtin_amdgcn_udot4(x, 0x01010101u, s1, false);
            s2 = __builtin_amdgcn_udot4(x, x, s2, false);
        }
        red4[0] += c;
        red4[1] += o;
        red4[2] += s1;
        red4[3] += s2;
    }
    for (uint32_t q = 16 * n16 + t; q < n; q += stride) {
        if (fov && fov[q] == 0) continue;
        const uint32_t v = vol[q];
        red4[0] += 1;
        red4[1] += v != 0;
        red4[2] += v;
        red4[3] += v * v;
    }
    __shared__ unsigned long long red[4][4];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        for (int e = 0; e < 4; ++e) red4[e] += __shfl_xor(red4[e], off);
    if (threadIdx.x % 64 == 0)
        for (int e = 0; e < 4; ++e) red[threadIdx.x / 64][e] = red4[e];
    __syncthreads();
    if (threadIdx.x < 4) {
        const unsigned long long s =
            red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
        atomicAdd(out + 4 * blockIdx.y + threadIdx.x, s);
    }
}

// Trilinear source layouts: per base voxel the corner bytes the kernel needs,
// with corners past the last voxel repeating it (see score.hip).  The
// element of voxel q and its FOV validity (all voxels it covers inside):
//   pairx  (v[x], v[x+1]) of one row;  quadxy  the 2x2 of one slice;
//   oct    the 2x2x2 of the trilinear cell (lerp stores the same cell ready
//          for the x-lerps).
// A trilinear sample is inside the FOV iff every element it reads is, so an
// invalid element may hold a sentinel value that no valid element takes.
struct Elem {
    uint64_t value;
    bool valid;
};

__device__ __forceinline__ Elem element(const uint8_t *vol, const uint8_t *fov, int32_t nx, int32_t ny, int32_t nz,
                                        int layout, uint32_t q) {
    const Cell at = cell_of(q, (uint32_t)nx, (uint32_t)ny);
    const uint32_t dx = (int32_t)at.i + 1 < nx ? 1u : 0u;
    const uint32_t dy = (int32_t)at.j + 1 < ny ? (uint32_t)nx : 0u;
    const uint32_t dz = (int32_t)at.k + 1 < nz ? (uint32_t)nx * (uint32_t)ny : 0u;
    Elem e;
    if (layout == kLayoutPairX) {
        e.value = (uint64_t)vol[q] | ((uint64_t)vol[q + dx] << 8);
        e.valid = !fov || (fov[q] && fov[q + dx]);
        return e;
    }
    const uint32_t q0 = (uint32_t)vol[q] | ((uint32_t)vol[q + dx] << 8) | ((uint32_t)vol[q + dy] << 16) |
                        ((uint32_t)vol[q + dy + dx] << 24);
    const bool v0 = !fov || (fov[q] && fov[q + dx] && fov[q + dy] && fov[q + dy + dx]);
    if (layout == kLayoutQuadXY) {
        e.value = q0;
        e.valid = v0;
        return e;
    }
    const uint32_t r = q + dz;
    const uint32_t q1 = (uint32_t)vol[r] | ((uint32_t)vol[r + dx] << 8) | ((uint32_t)vol[r + dy] << 16) |
                        ((uint32_t)vol[r + dy + dx] << 24);
    const bool v1 = !fov || (fov[r] && fov[r + dx] && fov[r + dy] && fov[r + dy + dx]);
    e.value = (uint64_t)q0 | ((uint64_t)q1 << 32);
    e.valid = v0 && v1;
    return e;
}

// The layouts of one slice or row (pairx, quadxy).
__global__ __launch_bounds__(256) void k_pack_rows(const uint8_t *vol, const uint8_t *fov, int32_t nx, int32_t ny,
                                                   int32_t nz, int layout, uint64_t sentinel, void *out) {
    const uint32_t n = (uint32_t)nx * ny * nz;
    for (uint32_t q = blockIdx.x * 256u + threadIdx.x; q < n; q += gridDim.x * 256u) {
        const Elem e = element(vol, fov, nx, ny, nz, layout, q);
        const uint64_t v = e.valid ? e.value : sentinel;
        if (layout == kLayoutPairX)
            ((uint16_t *)out)[q] = (uint16_t)v;
        else
            ((uint32_t *)out)[q] = (uint32_t)v;
    }
}

// The layouts of whole cells: octets (or tiled octets) and the x-lerps, either
// or both in one pass (lerp and tiled octets of 160^3: two launches of 31 us
// each, 27 us together).  ok: corner validity, or nullptr; cells that are
// not valid hold the sentinel in `oct` and the NaN word in `lerp`.  hits counts
// the valid cells that equal the sentinel.
__global__ __launch_bounds__(256) void k_pack_cells(const uint8_t *vol, const uint8_t *ok, int32_t nx, int32_t ny,
                                                    int32_t nz, uint4 *lerp, uint2 *oct, bool tiled,
                                                    uint64_t sentinel, unsigned long long *hits) {
    const uint32_t n = (uint32_t)nx * ny * nz, tx = (uint32_t)(nx + 3) / 4, ty = (uint32_t)(ny + 3) / 4;
    for (uint32_t q = blockIdx.x * 256u + threadIdx.x; q < n; q += gridDim.x * 256u) {
        const Cell at = cell_of(q, (uint32_t)nx, (uint32_t)ny);
        const uint32_t dx = (int32_t)at.i + 1 < nx ? 1u : 0u;
        const uint32_t dy = (int32_t)at.j + 1 < ny ? (uint32_t)nx : 0u;
        const uint32_t dz = (int32_t)at.k + 1 < nz ? (uint32_t)nx * (uint32_t)ny : 0u;
        const bool valid = ok == nullptr || ok[q] != 0;
        uint32_t lo[4], hi[4];  // v(x, .) and v(x + 1, .) of the rows (y, z), (y + 1, z), (y, z + 1), (y + 1, z + 1)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t o = q + (r & 1 ? dy : 0u) + (r & 2 ? dz : 0u);
            lo[r] = vol[o];
            hi[r] = vol[o + dx];
        }
        if (oct) {
            uint32_t w0 = lo[0] | (hi[0] << 8) | (lo[1] << 16) | (hi[1] << 24);
            uint32_t w1 = lo[2] | (hi[2] << 8) | (lo[3] << 16) | (hi[3] << 24);
            if (!valid) {
                w0 = (uint32_t)sentinel;
                w1 = (uint32_t)(sentinel >> 32);
            } else if (hits && w0 == (uint32_t)sentinel && w1 == (uint32_t)(sentinel >> 32)) {
                atomicAdd(hits, 1ull);
            }
            // tiled: 4 x 4 tiles of one slice, 16 octets (128 bytes) each, x fastest
            // inside a tile, tiles x fastest, then y, then slices
            const uint64_t o = tiled ? (((uint64_t)at.k * ty + at.j / 4) * tx + at.i / 4) * 16 + (at.j % 4) * 4 + at.i % 4
                                     : (uint64_t)q;
            oct[o] = make_uint2(w0, w1);
        }
        if (lerp) {
            // the four x-lerp starts a = v(x, .) and steps d = v(x + 1, .) - v(x, .),
            // each times 256 in half precision (exact: |256 v| <= 65280 with at most
            // eight significant bits)
            uint32_t h[8];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const _Float16 a = (_Float16)(256.0f * (float)lo[r]),
                               d = (_Float16)(256.0f * (float)((int)hi[r] - (int)lo[r]));
                h[r] = __builtin_bit_cast(uint16_t, a);
                h[4 + r] = __builtin_bit_cast(uint16_t, d);
            }
            lerp[q] = valid ? make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16),
                                         h[6] | (h[7] << 16))
                            : make_uint4(kLerpSentinel, 0u, 0u, 0u);
        }
    }
}

__global__ void k_count_elements(const uint8_t *vol, const uint8_t *fov, int32_t nx, int32_t ny, int32_t nz,
                                 int layout, const uint64_t *cand, int n_cand, unsigned long long *counts) {
    const uint32_t n = (uint32_t)nx * ny * nz;
    const uint64_t mask = layout == kLayoutPairX ? 0xFFFFull : (layout == kLayoutQuadXY ? 0xFFFFFFFFull : ~0ull);
    for (uint32_t q = blockIdx.x * 256u + threadIdx.x; q < n; q += gridDim.x * 256u) {
        const Elem e = element(vol, fov, nx, ny, nz, layout, q);
        if (!e.valid) continue;
        if (n_cand == 0) {
            atomicAdd(counts + e.value, 1ull);
        } else {
            for (int c = 0; c < n_cand; ++c)
                if (e.value == (cand[c] & mask)) atomicAdd(counts + c, 1ull);
        }
    }
}

unsigned blocks_for(int64_t n) {
    int64_t b = (n + 255) / 256;
    return (unsigned)(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

}  // namespace

namespace {
template <bool MASK>
hipError_t source_rows(const uint8_t *vol, const uint8_t *fov, const int32_t n[3], uint8_t *out, uint32_t *may,
                       uint32_t *must, hipStream_t s) {
    const int64_t groups = ((int64_t)n[1] * n[2] + kRows - 1) / kRows * ((n[0] + 63) / 64);
    hipLaunchKernelGGL(k_source_rows<MASK>, dim3(blocks_for(64 * groups)), dim3(256), 0, s, vol, fov, (uint32_t)n[0],
                       (uint32_t)n[1], (uint32_t)n[2], (uint32_t)(n[0] + 31) / 32, out, may, must);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_mask_source(const uint8_t *vol, const uint8_t *fov, const int32_t n[3], uint8_t *out, uint32_t *bits,
                              hipStream_t s) {
    return source_rows<true>(vol, fov, n, out, bits, nullptr, s);
}

hipError_t launch_corner_valid(const uint8_t *fov, const int32_t n[3], uint8_t *out, uint32_t *may, uint32_t *must,
                               hipStream_t s) {
    return source_rows<false>(nullptr, fov, n, out, may, must, s);
}

size_t packed_bytes_per_voxel(int layout) {
    switch (layout) {
    case kLayoutPairX: return 2;
    case kLayoutQuadXY: return 4;
    case kLayoutOct: case kLayoutOctTile: return 8;
    case kLayoutLerp: return 16;
    default: return 1;
    }
}

uint64_t packed_bytes(int layout, const int32_t n[3]) {
    if (layout == kLayoutOctTile)
        return (uint64_t)((n[0] + 3) / 4) * (uint64_t)((n[1] + 3) / 4) * 128ull * (uint64_t)n[2];
    return (uint64_t)n[0] * n[1] * n[2] * packed_bytes_per_voxel(layout);
}

hipError_t launch_pack_rows(const uint8_t *vol, const uint8_t *fov, const int32_t n[3], int layout, uint64_t sentinel,
                            void *out, hipStream_t s) {
    const int64_t tot = (int64_t)n[0] * n[1] * n[2];
    hipLaunchKernelGGL(k_pack_rows, dim3(blocks_for(tot)), dim3(256), 0, s, vol, fov, n[0], n[1], n[2], layout,
                       sentinel, out);
    return hipGetLastError();
}

hipError_t launch_pack_cells(const uint8_t *vol, const uint8_t *ok, const int32_t n[3], void *lerp, void *oct,
                             bool tiled, uint64_t sentinel, unsigned long long *hits, hipStream_t s) {
    const int64_t tot = (int64_t)n[0] * n[1] * n[2];
    hipLaunchKernelGGL(k_pack_cells, dim3(blocks_for(tot)), dim3(256), 0, s, vol, ok, n[0], n[1], n[2], (uint4 *)lerp,
                       (uint2 *)oct, tiled, sentinel, hits);
    return hipGetLastError();
}

hipError_t launch_count_elements(const uint8_t *vol, const uint8_t *fov, const int32_t n[3], int layout,
                                 const uint64_t *cand, int n_cand, unsigned long long *counts, hipStream_t s) {
    const int64_t tot = (int64_t)n[0] * n[1] * n[2];
    hipLaunchKernelGGL(k_count_elements, dim3(blocks_for(tot)), dim3(256), 0, s, vol, fov, n[0], n[1], n[2], layout,
                       cand, n_cand, counts);
    return hipGetLastError();
}

hipError_t launch_volume_sums(const uint8_t *const vol[2], const uint8_t *const fov[2], const int64_t n[2],
                              unsigned long long *out, hipStream_t s) {
    SumsOf a;
    for (int v = 0; v < 2; ++v) {
        a.vol[v] = vol[v];
        a.fov[v] = fov[v];
        a.n[v] = (uint32_t)n[v];
    }
    const int64_t blocks = (std::max(n[0], n[1]) + 4095) / 4096;  // 16 bytes a thread
    hipLaunchKernelGGL(k_volume_sums, dim3((unsigned)std::min<int64_t>(blocks, kSumBlocks), 2), dim3(256), 0, s, a, out);
    return hipGetLastError();
}

}  // namespace smc
