// Mask warp-and-score of the filter's launches (Eq. 4 on LV masks): per
// particle the counts a (target voxels in the FOV whose nearest-neighbour
// sample of the source is on) and c (those that are on in the target too).
//
// Most of a mask is far from its surface, where every sample of a block of
// target voxels reads the same value.  A distance field of the source (one
// byte per voxel: its state and the distance from its box to the nearest box
// of a voxel of the other state) decides that for a whole block: the
// image of a cubic block under the recipe lies in a ball about the image of
// its centre, so when the field there exceeds the ball's radius the block adds
// nothing (off) or its precomputed target counts (on).  Blocks of 16^3 are
// tested first, the undecided ones are split into 8^3 and then 4^3, and only
// undecided 4^3 blocks are sampled -- the counts are exactly those of sampling
// every voxel.
//
// A wave takes one particle and up to 64 of the target's 16^3 blocks: one lane
// per block and test, survivors compacted through a per-wave LDS list, no
// workgroup barrier, no list in memory and no pre-pass.  Sampling gives a
// 4^3 block to a quarter-wave: 16 lanes are a 4 x 4 patch of a slice (the
// texture path serves a quarter together and a 4 x 4 patch's image touches few
// rows and slices), each walking four slices, eight gathers in flight a lane.
// The sampled bits of a lane's four slices form a nibble that is counted
// against the target's nibbles with two population counts.
//
// What it measured (224 x 208 x 176 filled LV masks, N = 4096, K = 40, a whole
// registration): 79.2 ms with every 32 x 8 x 16 tile of the occupied part
// sampled (13.6 % of the pairs, 1.50 ms a launch); 38.4 ms with blocks down to
// 4^3 by a field of 2^3-voxel cells and 19 VALU instructions a gather; 26.7 ms
// with the block list in floats, a byte of target bits a lane and eighths of a
// voxel (15); 24.0 ms with the field at voxels.  Bound: the texture path (TD 96 %,
// TA 94 % busy; 16 VALU instructions a wave's load, 0.89 a CU and clock); six to
// eight waves a SIMD (fewer registers) ran no faster than five.
//
// Every mask goes this way.  Off the usual, a registration of 128 x 120 x 110 masks
// (N = 1000, K = 8; ms, tiles culled by the mask's box and cells first): filled
// ellipsoids 3.0, 1.1; voxels at random, half of them on or one in fifty (nothing
// is ever decided) 6.3, 6.0; one in a thousand 6.8, 2.1; target voxels of 1.5, 2, 3
// and 6 times the source's (no block of 16^3 or 8^3 is decided from 1.2 and 2.6
// times on) 2.8, 2.0, 1.3, 1.0 and 1.0, 0.79, 0.62, 0.45; one slice of 512^2 2.9, 2.8.
#include <string.h>

#include <algorithm>

#include "internal.h"

namespace smc {
namespace {

constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kBufferWord3 = 0x00020000;
constexpr int kWindow = 16;  // voxels searched on either side
constexpr int kStrip = 16;   // voxels of a line a thread of the field's passes makes

#if defined(__HIP_DEVICE_COMPILE__)
#define SMC_CONSTANT_AS __attribute__((address_space(4)))
#else
#define SMC_CONSTANT_AS
#endif
template <typename T>
__device__ __forceinline__ const SMC_CONSTANT_AS T *as_const(const T *p) {
    return (const SMC_CONSTANT_AS T *)p;
}

typedef int v4i __attribute__((ext_vector_type(4)));
// 32-bit load at element `vindex` of a buffer with a record stride; records
// past the end read zero.
__device__ uint32_t struct_load_u32(v4i rsrc, int vindex, int voffset, int soffset,
                                    int aux) __asm("llvm.amdgcn.struct.buffer.load.i32");

struct Args {
    // source bitmap: dword y + ny (x / 32 + W z), bit 31 - x % 32.  A 4 x 4
    // patch's image spans about five rows and one or two slices: rows four
    // bytes apart put a slice's part of it in one cache line
    const uint32_t *bits;
    const uint8_t *field;  // source distance field, one byte per voxel
    // target 4^3 blocks, 16 bytes: byte l of the column (l % 4, l / 4), slice s
    // in bit 3 - s (FOV) and 7 - s (on)
    const uint4 *t4;
    uint32_t t4_bytes;
    const uint32_t *t8, *t16;  // target counts of 8^3 and 16^3 blocks: FOV | on << 16
    const float *words;
    unsigned long long *sums, *work;
    int32_t sn[3], tn[3];
    uint32_t ny, WH, bwords;  // bitmap strides (dwords) of 32 voxels in x and of a slice
    uint32_t fx, fxy, fbytes;
    uint32_t g4[3], g8[3], g16[3], n16;
    uint32_t p0, np;
    uint32_t blocks, parts;  // 16^3 blocks per wave, waves per particle
};

// A block of a list: x | y << 16, z, and in z's word the flag that the image
// of its 32 x 16 x 16 tile lies inside the source.
constexpr uint32_t kInner = 0x80000000u;

// A block to sample: the floats of its first voxel, then its index in t4 with
// the flag.
struct WaveLds {
    uint2 l16[64], l8[64];
    uint4 u[72];
};

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t rank_of(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// One particle over 16^3 blocks [part * blocks, (part + 1) * blocks).  PROBE:
// the same tests, coordinates and source loads, the loaded words XORed into
// the result instead of counted.
template <bool PROBE, typename A>
__device__ __forceinline__ uint32_t dice_wave(const A &a, uint32_t part, uint32_t p, WaveLds &q) {
    const uint32_t lane = threadIdx.x % 64u;
    const auto *wp = as_const(a.words) + 12 * (size_t)p;
    float w[12];
#pragma unroll
    for (int e = 0; e < 12; ++e) w[e] = wp[e];

    const float rho = ball_radius(w);
    const bool bounded = coords_bounded(w, a.tn);
    const uint32_t need16 = field_need(7.5f, rho, bounded), need8 = field_need(3.5f, rho, bounded),
                   need4 = field_need(1.5f, rho, bounded);
    // half extents of the image's box of a 32 x 16 x 16 tile
    float rt[3];
#pragma unroll
    for (int d = 0; d < 3; ++d)
        rt[d] = fmaf(15.5f, fabsf(w[4 * d]), fmaf(7.5f, fabsf(w[4 * d + 1]), 7.5f * fabsf(w[4 * d + 2]))) + kFieldMargin;

    const __amdgpu_buffer_rsrc_t rs_f =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.field), (short)0, (int)a.fbytes, kBufferWord3);
    const uint64_t bits_addr = (uint64_t)a.bits;
    const v4i rs_b = {(int)(uint32_t)bits_addr, (int)((uint32_t)(bits_addr >> 32) & 0xFFFFu) | (4 << 16), (int)a.bwords,
                      kBufferWord3};
    const float n0 = (float)a.sn[0], n1 = (float)a.sn[1], n2 = (float)a.sn[2];

    // field byte at the image u of a block centre (clipped into the source:
    // a point outside it is no nearer to an on voxel than its clipped point)
    const auto field_at = [&](float cx, float cy, float cz, float u[3]) {
        u[0] = fmaf(w[2], cz, fmaf(w[1], cy, fmaf(w[0], cx, w[3])));
        u[1] = fmaf(w[6], cz, fmaf(w[5], cy, fmaf(w[4], cx, w[7])));
        u[2] = fmaf(w[10], cz, fmaf(w[9], cy, fmaf(w[8], cx, w[11])));
        const uint32_t x = floor_u32(__builtin_amdgcn_fmed3f(u[0], 0.0f, n0 - 0.5f));
        const uint32_t y = floor_u32(__builtin_amdgcn_fmed3f(u[1], 0.0f, n1 - 0.5f));
        const uint32_t z = floor_u32(__builtin_amdgcn_fmed3f(u[2], 0.0f, n2 - 0.5f));
        const uint32_t o = mad_u24(z, a.fxy, mad_u24(y, a.fx, x));
        return (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rs_f, o, 0, 0);
    };

    uint32_t na = 0u, nc = 0u, chk = 0u;  // a, c of this lane
    uint32_t ev = 0u, evi = 0u;           // pairs sampled; those of interior blocks

    // this lane's column in a sampled block
    const uint32_t l16 = lane % 16u, quarter = lane / 16u;
    const float dx = (float)(l16 % 4u), dy = (float)(l16 / 4u);
    const __amdgpu_buffer_rsrc_t rs_t =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(a.t4), (short)0, (int)a.t4_bytes, kBufferWord3);

    // sample units base .. base + n - 1 (n <= 8) of the list
    const auto sample = [&](uint32_t base, uint32_t n) {
        float mx[2], my[2], mz[2], fk[2];
        uint32_t tb[2];
        bool inner = true;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const uint32_t i = 4u * g + quarter;
            const bool ok = i < n;
            const uint4 e = q.u[base + (ok ? i : 0u)];
            inner = inner && (e.w & kInner) != 0u;
            // (the shift drops the flag; a record past the end reads zero)
            if (!PROBE) tb[g] = __builtin_amdgcn_raw_buffer_load_b8(rs_t, ok ? (e.w << 4) | l16 : a.t4_bytes, 0, 0);
            const float fi = __uint_as_float(e.x) + dx, fj = __uint_as_float(e.y) + dy;
            fk[g] = __uint_as_float(e.z);
            mx[g] = fmaf(w[1], fj, fmaf(w[0], fi, w[3]));
            my[g] = fmaf(w[5], fj, fmaf(w[4], fi, w[7]));
            mz[g] = fmaf(w[9], fj, fmaf(w[8], fi, w[11]));
        }
        uint32_t ix[2][4], word[2][4];
        if (__all(inner)) {
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const float k = s ? fk[g] + (float)s : fk[g];
                    ix[g][s] = floor_u32(fmaf(w[2], k, mx[g]));
                    const uint32_t iy = floor_u32(fmaf(w[6], k, my[g])), iz = floor_u32(fmaf(w[10], k, mz[g]));
                    word[g][s] = struct_load_u32(rs_b, (int)mad_u24(iz, a.WH, mad_u24(ix[g][s] >> 5, a.ny, iy)), 0, 0, 0);
                }
        } else {
            // inside iff 0 <= u < n per axis, as unsigned compares of bit
            // patterns (coordinates are never -0); outside samples load past
            // the end: zero, no cache line touched
            const uint32_t b0 = __float_as_uint(n0), b1 = __float_as_uint(n1), b2 = __float_as_uint(n2);
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const float k = s ? fk[g] + (float)s : fk[g];
                    const float ux = fmaf(w[2], k, mx[g]), uy = fmaf(w[6], k, my[g]), uz = fmaf(w[10], k, mz[g]);
                    ix[g][s] = floor_u32(ux);
                    const bool in = (__float_as_uint(ux) < b0) & (__float_as_uint(uy) < b1) & (__float_as_uint(uz) < b2);
                    const uint32_t o = mad_u24(floor_u32(uz), a.WH, mad_u24(ix[g][s] >> 5, a.ny, floor_u32(uy)));
                    word[g][s] = struct_load_u32(rs_b, (int)(in ? o : a.bwords), 0, 0, 0);
                }
        }
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            uint32_t b = 0u;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (PROBE) chk ^= word[g][s];
                else b = __builtin_amdgcn_alignbit(b, word[g][s] << (ix[g][s] & 31u), 31u);
            }
            if (!PROBE) {
                const uint32_t t = tb[g] & (b | (b << 4));
                na += (uint32_t)__popc(t & 15u);
                nc += (uint32_t)__popc(t >> 4);
            }
        }
    };

    // 16^3 blocks, one a lane
    uint32_t n_l16;
    {
        const uint32_t id = part * a.blocks + lane;
        const bool valid = lane < a.blocks && id < a.n16;
        const uint32_t row = id / a.g16[0], bx = id - row * a.g16[0], bz = row / a.g16[1], by = row - bz * a.g16[1];
        float u[3];
        const uint32_t f = field_at(fmaf(16.0f, (float)bx, 7.5f), fmaf(16.0f, (float)by, 7.5f),
                                    fmaf(16.0f, (float)bz, 7.5f), u);
        const uint32_t t = valid ? a.t16[id] : 0u;
        const bool decided = (f & kFieldDist) >= need16;
        if (decided && (f & kFieldOn)) {
            na += t & 0xFFFFu;
            nc += t >> 16;
        }
        // (t = 0: no target voxel of the block is in the FOV)
        const bool open = !decided && t != 0u;
        const uint64_t m = __ballot(open);
        n_l16 = (uint32_t)__popcll(m);
        // every sample of the block's 32 x 16 x 16 tile lies inside the source:
        // the block's parts skip the inside test.  (u moves by half a tile from
        // the block's centre to the tile's.)
        const float e = bx & 1u ? -8.0f : 8.0f;
        bool inner = bounded;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float ut = fmaf(w[4 * d], e, u[d]);
            inner = inner && ut - rt[d] >= 0.0f && ut + rt[d] < (float)a.sn[d];
        }
        if (open) q.l16[rank_of(m)] = make_uint2(bx | (by << 16), bz | (inner ? kInner : 0u));
        wave_sync();
    }
    uint32_t n_u = 0u;
    for (uint32_t s16 = 0; s16 < n_l16; s16 += 8u) {
        // the eight 8^3 blocks of eight 16^3 blocks
        const uint32_t child = lane % 8u;
        uint32_t n_l8;
        {
            const uint32_t i = s16 + lane / 8u;
            const uint2 e = q.l16[min(i, n_l16 - 1u)];
            const uint32_t x = 2u * (e.x & 0xFFFFu) + (child & 1u), y = 2u * (e.x >> 16) + ((child >> 1) & 1u),
                           z = 2u * (e.y & ~kInner) + (child >> 2);
            const bool valid = i < n_l16 && x < a.g8[0] && y < a.g8[1] && z < a.g8[2];
            float u[3];
            const uint32_t f = field_at(fmaf(8.0f, (float)x, 3.5f), fmaf(8.0f, (float)y, 3.5f),
                                        fmaf(8.0f, (float)z, 3.5f), u);
            const uint32_t t = valid ? a.t8[x + a.g8[0] * (y + a.g8[1] * z)] : 0u;
            const bool decided = (f & kFieldDist) >= need8;
            if (decided && (f & kFieldOn)) {
                na += t & 0xFFFFu;
                nc += t >> 16;
            }
            const bool open = !decided && t != 0u;
            const uint64_t m = __ballot(open);
            n_l8 = (uint32_t)__popcll(m);
            wave_sync();  // the previous list of 8^3 blocks has been read
            if (open) q.l8[rank_of(m)] = make_uint2(x | (y << 16), z | (e.y & kInner));
            wave_sync();
        }
        for (uint32_t s8 = 0; s8 < n_l8; s8 += 8u) {
            const uint32_t i = s8 + lane / 8u;
            const uint2 e = q.l8[min(i, n_l8 - 1u)];
            const uint32_t x = 2u * (e.x & 0xFFFFu) + (child & 1u), y = 2u * (e.x >> 16) + ((child >> 1) & 1u),
                           z = 2u * (e.y & ~kInner) + (child >> 2);
            const bool valid = i < n_l8 && x < a.g4[0] && y < a.g4[1] && z < a.g4[2];
            float u[3];
            const uint32_t f = field_at(fmaf(4.0f, (float)x, 1.5f), fmaf(4.0f, (float)y, 1.5f),
                                        fmaf(4.0f, (float)z, 1.5f), u);
            const bool decided = (f & kFieldDist) >= need4;
            const uint32_t id = x + a.g4[0] * (y + a.g4[1] * z);
            if (!PROBE && valid && decided && (f & kFieldOn)) {
                const uint4 t = a.t4[id];
                const uint32_t all[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    na += (uint32_t)__popc(all[d] & 0x0F0F0F0Fu);
                    nc += (uint32_t)__popc(all[d] & 0xF0F0F0F0u);
                }
            }
            const bool open = valid && !decided;
            const uint64_t m = __ballot(open);
            if (open) {
                q.u[n_u + rank_of(m)] = make_uint4(__float_as_uint(4.0f * (float)x), __float_as_uint(4.0f * (float)y),
                                                   __float_as_uint(4.0f * (float)z), id | (e.y & kInner));
                const uint32_t pairs = min(4u, (uint32_t)a.tn[0] - 4u * x) * min(4u, (uint32_t)a.tn[1] - 4u * y) *
                                       min(4u, (uint32_t)a.tn[2] - 4u * z);
                ev += pairs;
                evi += (e.y & kInner) ? pairs : 0u;
            }
            n_u += (uint32_t)__popcll(m);
            wave_sync();
            while (n_u >= 8u) {
                n_u -= 8u;
                sample(n_u, 8u);
            }
            wave_sync();  // the sampled units have been read
        }
    }
    if (n_u) sample(0u, n_u);
    if (PROBE) return chk;

    if (__any((na | ev) != 0u)) {
        na = wave_sum(na);
        nc = wave_sum(nc);
        ev = wave_sum(ev);
        evi = wave_sum(evi);
        if (lane == 0u) {
            if (na) atomicAdd(a.sums + 6 * (size_t)p + 1, (unsigned long long)na);
            if (nc) atomicAdd(a.sums + 6 * (size_t)p + 2, (unsigned long long)nc);
            if (a.work && ev) {
                unsigned long long *slot =
                    a.work + kWorkSlotWords * ((blockIdx.x * kWaves + threadIdx.x / 64u) % kWorkSlots);
                atomicAdd(slot, (unsigned long long)ev);
                if (evi) atomicAdd(slot + 2, (unsigned long long)evi);
            }
        }
    }
    return 0u;
}

// Workgroup `block` of the launch: 16^3 blocks of part block / groups, a
// particle a wave, so the workgroups in flight share a part of the target and,
// the particles being clustered, a part of the source.
template <typename A>
__device__ __forceinline__ bool wave_unit(const A &a, uint32_t block, uint32_t &part, uint32_t &p) {
    const uint32_t groups = (a.np + kWaves - 1u) / kWaves;
    part = block / groups;
    const uint32_t i = (block - part * groups) * kWaves +
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64u));
    p = a.p0 + i;
    return i < a.np;
}

// (workgroups first .. of the launch)
__global__ __launch_bounds__(kThreads) void k_score_dice(const Args a, uint32_t first) {
    __shared__ WaveLds q[kWaves];
    uint32_t part, p;
    if (first + blockIdx.x == 0u && threadIdx.x == 0u && a.work)
        atomicAdd(a.work + 1, (unsigned long long)a.np * (unsigned long long)a.tn[0] * (unsigned long long)a.tn[1] *
                                  (unsigned long long)a.tn[2]);
    if (!wave_unit(a, first + blockIdx.x, part, p)) return;
    dice_wave<false>(a, part, p, q[threadIdx.x / 64u]);
}

__global__ __launch_bounds__(kThreads) void k_probe_dice(const Args a, uint32_t first, uint32_t key, uint32_t *out) {
    __shared__ WaveLds q[kWaves];
    uint32_t part, p;
    if (!wave_unit(a, first + blockIdx.x, part, p)) return;
    const uint32_t chk = dice_wave<true>(a, part, p, q[threadIdx.x / 64u]);
    if (chk == key) out[0] = chk;
}

// The mask pairs of a batch: pair d owns workgroups offs[d] .. offs[d + 1) - 1.
__global__ __launch_bounds__(kThreads) void k_batch_dice(const Args *pairs_g, const uint32_t *offs_g,
                                                         const uint32_t *kmax_g, uint32_t n_pairs, uint32_t k,
                                                         uint32_t first) {
    __shared__ WaveLds q[kWaves];
    const auto *offs = as_const(offs_g);
    const uint32_t block = first + blockIdx.x;
    uint32_t lo = 0, hi = n_pairs - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (offs[mid] <= block) lo = mid;
        else hi = mid - 1;
    }
    if (as_const(kmax_g)[lo] < k) return;  // pairs with fewer iterations are done
    const Args a = as_const(pairs_g)[lo];
    uint32_t part, p;
    if (!wave_unit(a, block - offs[lo], part, p)) return;
    dice_wave<false>(a, part, p, q[threadIdx.x / 64u]);
}

// ---------------------------------------------------------------- preparation

// The field, one axis at a time.  Gaps are whole voxels between two voxels'
// boxes, 0 where they touch; kWindow and more read as kWindow, and squared
// distances saturate at 255 (both lower bounds).  Voxels outside the source
// are off.  Of a voxel's distances to the nearest voxel that may be on and to
// that may be off one is 0, so a byte holds both: the distance, and in bit 7
// that it is the one to off.  Passes of 8.2 M voxels 15, 25 and 46 us; with two
// bytes a voxel 17, 26 and 29, and four times the memory between them, which each
// context then held or paid 80 us to give back.
constexpr uint32_t kToOff = 128u;

// The squared distances within a slice are sums of two squares: 97 values below
// 255.  Their numbers, and per byte the distances to on (low) and off (high).
struct SquareCodes {
    uint8_t number[256] = {};
    uint32_t pair[256] = {};
    constexpr SquareCodes() {
        uint32_t count = 0;
        for (uint32_t d = 0; d < 256; ++d) {
            bool sum = d == 255;  // (255 and more)
            for (uint32_t a = 0; a <= kWindow && !sum; ++a)
                for (uint32_t b = 0; b <= kWindow && !sum; ++b) sum = a * a + b * b == d;
            if (!sum) continue;
            number[d] = (uint8_t)count;
            pair[count] = d;
            pair[count | kToOff] = d << 16;
            ++count;
        }
    }
};
__device__ const SquareCodes kSquareCodes{};

// x: gaps along the rows, four voxels a thread.
__global__ __launch_bounds__(256) void k_field_x(const uint32_t *may, const uint32_t *must, int32_t nx, uint32_t ny,
                                                 uint32_t rows, uint32_t W, uint8_t *out) {
    const uint32_t quads = (uint32_t)(nx + 3) / 4, n = quads * rows;
    for (uint32_t q = blockIdx.x * 256u + threadIdx.x; q < n; q += gridDim.x * 256u) {
        const uint32_t row = q / quads, z = row / ny;
        const int32_t xa = 4 * (int32_t)(q - row * quads), x0 = xa - kWindow;  // first voxel of the window
        const int64_t r = (row - z * ny) + (int64_t)ny * W * z;
        const int32_t d = x0 >> 5, s = x0 & 31;
        const auto window = [&](const uint32_t *bits) {
            const auto word = [&](int32_t e) { return e >= 0 && e < (int32_t)W ? __brev(bits[r + (int64_t)ny * e]) : 0u; };
            uint64_t m = ((uint64_t)word(d) | ((uint64_t)word(d + 1) << 32)) >> s;
            if (s) m |= (uint64_t)word(d + 2) << (64 - s);
            return m;
        };
        const uint64_t on = window(may), off = ~window(must);
        // kWindow bits to the left of a voxel, its own, kWindow to the right
        const auto gap = [&](uint64_t b) -> uint32_t {
            if ((b >> kWindow) & 1u) return 0u;
            const uint32_t l = (uint32_t)b & ((1u << kWindow) - 1u),
                           rt = (uint32_t)(b >> (kWindow + 1)) & ((1u << kWindow) - 1u);
            const uint32_t gl = l ? (uint32_t)__clz(l) - (32u - kWindow) : (uint32_t)kWindow;
            const uint32_t gr = rt ? (uint32_t)__ffs(rt) - 1u : (uint32_t)kWindow;
            return min(gl, gr);
        };
        uint32_t v = 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t to_on = gap(on >> j);
            v |= (to_on ? to_on : gap(off >> j) | kToOff) << (8 * j);
        }
        uint8_t *o = out + row * (uint32_t)nx + xa;
        if (xa + 4 <= nx)
            __builtin_memcpy(o, &v, 4);
        else
            for (int j = 0; xa + j < nx; ++j) o[j] = (uint8_t)(v >> (8 * j));
    }
}

// Lower envelopes of a strip of kStrip voxels along a line: v holds, from
// kWindow before the strip on, the squared distances within the rows (planes)
// crossed so far, on in the low and off in the high half; a voxel t steps away
// adds the square of its gap.  Both halves move together in packed 16-bit
// arithmetic.
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 envelope(const u16x2 *v) {
    u16x2 m = v[kWindow];
#pragma unroll
    for (int t = -kWindow; t <= kWindow; ++t) {
        if (t == 0) continue;
        const int g = (t < 0 ? -t : t) - 1;
        m = __builtin_elementwise_min(m, (u16x2)(v[kWindow + t] + (uint16_t)(g * g)));
    }
    return m;
}

// y: squared distances within a slice.
__global__ __launch_bounds__(256) void k_field_y(const uint8_t *gx, int32_t nx, int32_t ny, int32_t nz,
                                                 uint8_t *out) {
    __shared__ uint8_t number[256];
    number[threadIdx.x] = kSquareCodes.number[threadIdx.x];
    __syncthreads();
    const uint32_t strips = (uint32_t)(ny + kStrip - 1) / kStrip, n = (uint32_t)nx * strips * (uint32_t)nz;
    for (uint32_t q = blockIdx.x * 256u + threadIdx.x; q < n; q += gridDim.x * 256u) {
        const uint32_t t = q / (uint32_t)nx, z = t / strips;
        const int32_t y0 = kStrip * (int32_t)(t - z * strips);
        const uint32_t line = (q - t * nx) + (uint32_t)nx * ((uint32_t)ny * z);
        u16x2 v[kStrip + 2 * kWindow];
#pragma unroll
        for (int e = 0; e < kStrip + 2 * kWindow; ++e) {
            const int32_t y = y0 + e - kWindow;
            const uint32_t g = y >= 0 && y < ny ? gx[line + (uint32_t)(nx * y)] : (uint32_t)kWindow;  // outside: off
            const uint16_t d = (uint16_t)((g & 127u) * (g & 127u));
            v[e] = g & kToOff ? u16x2{0, d} : u16x2{d, 0};
        }
#pragma unroll
        for (int j = 0; j < kStrip; ++j) {
            if (y0 + j >= ny) break;
            const u16x2 m = envelope(v + j);
            const uint32_t code = number[min((uint32_t)max(m.x, m.y), 255u)];
            out[line + (uint32_t)(nx * (y0 + j))] = (uint8_t)(m.x ? code : code | kToOff);
        }
    }
}

// z, and the field byte: 0 where a voxel of the other state touches (always
// sampled).
__global__ __launch_bounds__(256) void k_field_z(const uint8_t *gy, uint32_t plane, int32_t nz, uint8_t *out) {
    __shared__ uint32_t pair[256];
    pair[threadIdx.x] = kSquareCodes.pair[threadIdx.x];
    __syncthreads();
    const uint32_t strips = (uint32_t)(nz + kStrip - 1) / kStrip, n = plane * strips;
    for (uint32_t q = blockIdx.x * 256u + threadIdx.x; q < n; q += gridDim.x * 256u) {
        const uint32_t t = q / plane;
        const int32_t z0 = kStrip * (int32_t)t;
        const uint32_t line = q - t * plane;
        u16x2 v[kStrip + 2 * kWindow];
#pragma unroll
        for (int e = 0; e < kStrip + 2 * kWindow; ++e) {
            const int32_t z = z0 + e - kWindow;
            v[e] = u16x2{255, 0};  // outside: off
            if (z >= 0 && z < nz) v[e] = __builtin_bit_cast(u16x2, pair[gy[line + plane * (uint32_t)z]]);
        }
#pragma unroll
        for (int j = 0; j < kStrip; ++j) {
            if (z0 + j >= nz) break;
            const u16x2 m = envelope(v + j);
            // (one of the two is 0: the voxel's own state)
            const uint32_t d2 = min((uint32_t)max(m.x, m.y), 255u);
            const uint32_t dist = min(kFieldDist, (uint32_t)floorf(sqrtf((float)(64u * d2))));
            out[line + plane * (uint32_t)(z0 + j)] = (uint8_t)(dist | (m.x == 0 && m.y != 0 ? kFieldOn : 0u));
        }
    }
}

// Prepared bytes (bit 0: inside the FOV, no FOV = everywhere; bit 1: nonzero and
// inside) and 4^3 blocks (layout: Args::t4) of the target, a block a thread, a
// row of it a dword (bytes at the last columns and of an unaligned volume
// all the same: a dword load takes any address).  8.2 M voxels: 10 us; a byte
// a load and the bytes in a pass of their own 8 + 17.
__global__ __launch_bounds__(256) void k_target4(const uint8_t *vol, const uint8_t *fov, uint8_t *prep, int32_t nx,
                                                 int32_t ny, int32_t nz, uint32_t gx, uint32_t gy, uint32_t gz,
                                                 uint4 *out) {
    const uint32_t n = gx * gy * gz;
    for (uint32_t q = blockIdx.x * 256u + threadIdx.x; q < n; q += gridDim.x * 256u) {
        const uint32_t t = q / gx, tz = t / gy;
        const int32_t x0 = 4 * (int32_t)(q - t * gx), y0 = 4 * (int32_t)(t - tz * gy), z0 = 4 * (int32_t)tz;
        uint32_t v[4] = {0u, 0u, 0u, 0u};
        const int32_t wide = min(4, nx - x0);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                if (z0 + s >= nz || y0 + y >= ny) continue;
                const int64_t o = (int64_t)x0 + (int64_t)nx * ((y0 + y) + (int64_t)ny * (z0 + s));
                uint32_t a = 0u, f = 0x01010101u, keep = ~0u;
                if (wide == 4) {
                    __builtin_memcpy(&a, vol + o, 4);
                    if (fov) __builtin_memcpy(&f, fov + o, 4);
                } else {
                    keep = 0u;
                    for (int x = 0; x < wide; ++x) {
                        a |= (uint32_t)vol[o + x] << (8 * x);
                        if (fov) f = (f & ~(255u << (8 * x))) | ((uint32_t)fov[o + x] << (8 * x));
                        keep |= 255u << (8 * x);
                    }
                }
                const auto nonzero = [](uint32_t b) {  // 1 in each byte that is not zero
                    return ((((b & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | b) >> 7) & 0x01010101u;
                };
                const uint32_t in = nonzero(f) & keep, on = nonzero(a) & in, bytes = in | (on << 1);
                if (wide == 4)
                    __builtin_memcpy(prep + o, &bytes, 4);
                else
                    for (int x = 0; x < wide; ++x) prep[o + x] = (uint8_t)(bytes >> (8 * x));
                v[y] |= (in | (on << 4)) << (3 - s);
            }
        out[q] = make_uint4(v[0], v[1], v[2], v[3]);
    }
}

// Counts (FOV | on << 16) of the target blocks of side 8 and 16: a wave makes one
// of 16 from its 64 blocks of 4^3, a lane each (one thread over all 64 waited
// on a chain of loads: 4 + 14 us for both sides, 5 us so).
__global__ __launch_bounds__(256) void k_target_counts(const uint4 *t4, uint32_t g4x, uint32_t g4y, uint32_t g4z,
                                                       uint32_t g8x, uint32_t g8y, uint32_t g8z, uint32_t gx,
                                                       uint32_t gy, uint32_t gz, uint32_t *t8, uint32_t *t16) {
    const uint32_t n = gx * gy * gz, lane = threadIdx.x % 64;
    const uint32_t lx = lane & 3u, ly = (lane >> 2) & 3u, lz = lane >> 4;
    for (uint32_t w = blockIdx.x * 4 + threadIdx.x / 64; w < n; w += gridDim.x * 4) {
        const uint32_t t = w / gx, bz = t / gy, bx = w - t * gx, by = t - bz * gy;
        const uint32_t x = 4 * bx + lx, y = 4 * by + ly, z = 4 * bz + lz;
        uint32_t v = 0u;
        if (x < g4x && y < g4y && z < g4z) {
            const uint4 b = t4[x + (int64_t)g4x * (y + (int64_t)g4y * z)];
            v = (uint32_t)(__popc(b.x & 0x0F0F0F0Fu) + __popc(b.y & 0x0F0F0F0Fu) + __popc(b.z & 0x0F0F0F0Fu) +
                           __popc(b.w & 0x0F0F0F0Fu)) +
                ((uint32_t)(__popc(b.x & 0xF0F0F0F0u) + __popc(b.y & 0xF0F0F0F0u) + __popc(b.z & 0xF0F0F0F0u) +
                            __popc(b.w & 0xF0F0F0F0u))
                 << 16);
        }
        for (int o = 1; o < 64; o <<= 2) v += __shfl_xor(v, o);
        const uint32_t x8 = 2 * bx + lx / 2, y8 = 2 * by + ly / 2, z8 = 2 * bz + lz / 2;
        if ((lane & 21u) == 0u && x8 < g8x && y8 < g8y && z8 < g8z) t8[x8 + (int64_t)g8x * (y8 + (int64_t)g8y * z8)] = v;
        for (int o = 2; o < 64; o <<= 2) v += __shfl_xor(v, o);
        if (lane == 0) t16[w] = v;
    }
}

unsigned blocks_for(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 8192)); }

uint32_t cells(int32_t n, int32_t side) { return (uint32_t)((n + side - 1) / side); }

Args make_args(const ScoreLaunch &L) {
    Args a;
    a.bits = L.dice.bits;
    a.field = L.dice.field;
    a.t4 = (const uint4 *)L.dice.t4;
    a.t8 = L.dice.t8;
    a.t16 = L.dice.t16;
    a.words = L.words;
    a.sums = L.sums;
    a.work = L.work;
    for (int d = 0; d < 3; ++d) {
        a.sn[d] = L.sn[d];
        a.tn[d] = L.tn[d];
        a.g4[d] = cells(L.tn[d], 4);
        a.g8[d] = cells(L.tn[d], 8);
        a.g16[d] = cells(L.tn[d], 16);
    }
    a.n16 = a.g16[0] * a.g16[1] * a.g16[2];
    a.t4_bytes = 16u * a.g4[0] * a.g4[1] * a.g4[2];
    a.ny = (uint32_t)L.sn[1];
    a.WH = cells(L.sn[0], 32) * a.ny;
    a.bwords = a.WH * (uint32_t)L.sn[2];
    a.fx = (uint32_t)L.sn[0];
    a.fxy = a.fx * a.ny;
    a.fbytes = a.fxy * (uint32_t)L.sn[2];
    a.p0 = L.p0;
    a.np = L.np;
    // blocks per wave: as many as keep about 32k waves (16 per SIMD slot of
    // the 256 CUs), since a wave tests 64 blocks at the price of one; at least
    // two (a launch of 64^3 shells, N = 256: 17.4 us, 21.6 with four), and all
    // parts of one size, so that no wave is left with a few (180 x 170 x 160,
    // N = 2000: 256 us, 287 with a remainder; 224 x 208 x 176, N = 4096: 585, 612)
    const uint64_t want = (uint64_t)a.n16 * L.np / 32768u;
    a.blocks = (uint32_t)std::min<uint64_t>(64u, std::max<uint64_t>(2u, want));
    a.parts = (a.n16 + a.blocks - 1) / a.blocks;
    a.blocks = (a.n16 + a.parts - 1) / a.parts;
    return a;
}

uint64_t groups_of(const Args &a) { return (uint64_t)a.parts * ((a.np + kWaves - 1) / kWaves); }

}  // namespace

DiceSizes dice_sizes(const int32_t sn[3], const int32_t tn[3]) {
    DiceSizes s;
    const uint64_t n = (uint64_t)sn[0] * sn[1] * sn[2];
    s.bits = 4ull * cells(sn[0], 32) * (uint64_t)sn[1] * (uint64_t)sn[2];
    s.field = n;
    const auto grid = [&](int32_t side) {
        return (uint64_t)cells(tn[0], side) * cells(tn[1], side) * cells(tn[2], side);
    };
    s.t4 = 16ull * grid(4);
    s.t8 = 4ull * grid(8);
    s.t16 = 4ull * grid(16);
    return s;
}

hipError_t launch_field(const uint32_t *may, const uint32_t *must, const int32_t n[3], uint8_t *gaps, uint8_t *field,
                        hipStream_t s) {
    const int64_t rows = (int64_t)n[1] * n[2], plane = (int64_t)n[0] * n[1];
    hipLaunchKernelGGL(k_field_x, dim3(blocks_for((n[0] + 3) / 4 * rows)), dim3(256), 0, s, may, must, n[0],
                       (uint32_t)n[1], (uint32_t)rows, cells(n[0], 32), field);
    hipLaunchKernelGGL(k_field_y, dim3(blocks_for(((int64_t)n[1] + kStrip - 1) / kStrip * n[0] * n[2])), dim3(256), 0, s,
                       (const uint8_t *)field, n[0], n[1], n[2], gaps);
    hipLaunchKernelGGL(k_field_z, dim3(blocks_for(((int64_t)n[2] + kStrip - 1) / kStrip * plane)), dim3(256), 0, s,
                       (const uint8_t *)gaps, (uint32_t)plane, n[2], field);
    return hipGetLastError();
}

hipError_t launch_dice_target(const uint8_t *vol, const uint8_t *fov, const int32_t n[3], uint8_t *prep, void *t4,
                              uint32_t *t8, uint32_t *t16, hipStream_t s) {
    uint32_t g[3][3];
    for (int l = 0; l < 3; ++l)
        for (int d = 0; d < 3; ++d) g[l][d] = cells(n[d], 4 << l);
    const auto count = [&](int l) { return (int64_t)g[l][0] * g[l][1] * g[l][2]; };
    hipLaunchKernelGGL(k_target4, dim3(blocks_for(count(0))), dim3(256), 0, s, vol, fov, prep, n[0], n[1], n[2], g[0][0],
                       g[0][1], g[0][2], (uint4 *)t4);
    hipLaunchKernelGGL(k_target_counts, dim3(blocks_for(64 * count(2))), dim3(256), 0, s, (const uint4 *)t4, g[0][0],
                       g[0][1], g[0][2], g[1][0], g[1][1], g[1][2], g[2][0], g[2][1], g[2][2], t8, t16);
    return hipGetLastError();
}

size_t dice_args_bytes() { return sizeof(Args); }

uint64_t dice_args(const ScoreLaunch &L, void *out) {
    const Args a = make_args(L);
    memcpy(out, &a, sizeof a);
    return groups_of(a);
}

hipError_t launch_dice(const ScoreLaunch &L, hipStream_t s) {
    if (L.np == 0) return hipSuccess;
    const Args a = make_args(L);
    return launch_groups(groups_of(a), [&](uint32_t first, dim3 grid) {
        hipLaunchKernelGGL(k_score_dice, grid, dim3(kThreads), 0, s, a, first);
    });
}

hipError_t launch_dice_probe(const ScoreLaunch &L, uint32_t key, uint32_t *out, hipStream_t s) {
    if (L.np == 0) return hipSuccess;
    const Args a = make_args(L);
    return launch_groups(groups_of(a), [&](uint32_t first, dim3 grid) {
        hipLaunchKernelGGL(k_probe_dice, grid, dim3(kThreads), 0, s, a, first, key, out);
    });
}

hipError_t launch_batch_dice(const void *pairs, const uint32_t *offs, const uint32_t *kmax, uint32_t n_pairs,
                             uint32_t groups, uint32_t k, hipStream_t s) {
    if (n_pairs == 0) return hipSuccess;
    return launch_groups(groups, [&](uint32_t first, dim3 grid) {
        hipLaunchKernelGGL(k_batch_dice, grid, dim3(kThreads), 0, s, (const Args *)pairs, offs, kmax, n_pairs, k, first);
    });
}

}  // namespace smc
