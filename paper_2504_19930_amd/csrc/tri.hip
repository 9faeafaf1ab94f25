// Trilinear warp-and-score of a source with a FOV from the one-gather layouts
// (octets, tiled octets, lerp elements): the exact sums of NCC / SSD, or the joint histogram of the
// mutual information.
//
// A distance field of the source (one byte per voxel, as for masks) says of a
// whole block of target voxels whether every sample of it is valid (inside the
// source and its FOV) or none is: blocks of 16^3, then 8^3, then 4^3.  Blocks
// without a valid sample are skipped -- with an apical cone two fifths of the
// pairs; FOVs that leave little to skip go by tiles, see tri_pays -- and blocks with nothing but valid samples drop the per-sample tests:
// three compares, a select, the sentinel and the lane mask, and the sums n, t
// and t^2, which are the target block's own.
//
// A workgroup takes four particles (neighbours after resampling, so their
// gathers meet in the L1) and up to twelve blocks of 16^3.  A block that is
// valid throughout is sampled by its four waves together, a 16 x 4 strip each
// (quarters of a wave are 4 x 4 squares, which the texture path serves
// together), so that the cache lines at the strips' edges meet in the L1 as
// well; smaller ones go to a wave (8^3) or a quarter-wave (4^3).  Two slices and
// so eight gathers at a time.  The target's bytes are kept as dwords of four
// slices.
//
// Sums: s_fx - 2^15 of two slices are packed as 16-bit integers; one dot
// product instruction each forms s', s'^2 and s' t for both (s'^2 of a pair
// stays within 2^31 and goes to a 64-bit sum, the others stay in 32 bits for
// the at most 256 samples a lane takes), and the offset is put back exactly
// from n and t at the end: three instructions for two samples instead of six.
//
// What it measured (160^3 speckle images in a 60-degree cone, N = 2048, lerp
// elements, concentrated cloud): 5.98 ms a launch over whole tiles with every
// sample tested, 4.69 with blocks down to 8^3, 4.55 with each load issued as its
// offset is known, 4.37 with 4^3 blocks.  A whole registration 193 -> 141 ms; 16
// uneven pairs 33.6 -> 25.9 ms.  Bound: the texture path (TD 97 %, TA 90 % busy,
// about 28 clocks a wave's 16-byte gather, 30 cache accesses a wave's load) with VALU
// issue close behind (0.98 instructions a CU and clock, 30 a load).  More waves
// (one slice at a time, 95 registers, five waves a SIMD) ran 2 to 9 % slower:
// their gathers evict each other's lines.
#include <math.h>
#include <string.h>

#include <algorithm>

#include "internal.h"

namespace smc {
namespace {

constexpr int PT = 4;  // particles of a workgroup
constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kBufferWord3 = 0x00020000;
constexpr int kHB = kMiBins * kMiBins;
// 16^3 blocks of a workgroup: twelve are 192 samples a lane, and at most 16
// more where parts do not share out evenly (the 32-bit sums hold 257); a
// histogram takes more (its flush costs up to 4096 global atomics).
constexpr int kSumBlocks = 12, kHistBlocks = 48;
// Consecutive workgroups of a launch that one XCD takes (see tri_body): a
// single launch shares its work out evenly from 16 down (160^3 141.5 ms a
// registration, 150 x 60 x 50 0.088 ms a launch; 64: 142.4 and 0.126); a batch,
// whose pairs have few particle groups, gains from longer runs (16 pairs 26.8 ms
// with 16, 25.9 with 32, 26.2 with 64, 27.8 without).
constexpr uint32_t kRun = 16, kBatchRun = 32;
// Particles far apart (ScoreLaunch::apart): small parts and longer runs, since the
// image of a part under all the particles has to stay in the L2.  Rotations up to
// 180 degrees, 128 x 120 x 110 in a cone, N = 600, K = 6: 13.5 ms with twelve blocks
// and runs of 16, 9.6 with four and 32 (11.2 in tiles).
constexpr uint32_t kApartBlocks = 4, kApartRun = 32;

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
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short i16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
// Element `vindex` of a buffer with a record stride; records past the end
// read zero without touching memory.
__device__ u32x4 struct_load_u32x4(v4i rsrc, int vindex, int voffset, int soffset,
                                   int aux) __asm("llvm.amdgcn.struct.buffer.load.v4i32");
__device__ u32x2 struct_load_u32x2(v4i rsrc, int vindex, int voffset, int soffset,
                                   int aux) __asm("llvm.amdgcn.struct.buffer.load.v2i32");

struct Args {
    const void *src;       // packed source
    const uint8_t *src_ok; // corner validity (vmode 1)
    const uint8_t *field;  // distance field of the valid cells
    const uint32_t *tz;    // target: dword of slices 4 q .. 4 q + 3 at (x, y): ((q ny) + y) nx + x
    const uint32_t *fz;    // its FOV likewise (nonzero bytes inside), or nullptr
    const uint4 *t8, *t16; // blocks of 8^3 and 16^3: n, sum t, sum t^2 over the FOV
    const uint2 *t4;       // blocks of 4^3: n | sum t << 8, sum t^2
    const float *words;
    unsigned long long *sums;
    uint32_t *hist;
    uint64_t sentinel;
    int32_t sn[3], tn[3];
    uint32_t records;      // elements of the packed source
    uint32_t ysb, zsb;     // element strides (tiled octets: byte strides, see score.hip)
    uint32_t g4[3], g8[3], g16[3], n16;
    uint32_t p0, np, blocks, parts;  // 16^3 blocks per workgroup; workgroups per four particles
    uint32_t run;                    // consecutive workgroups of an XCD
};

__device__ __forceinline__ half2v as_half2(uint32_t u) {
    half2v h;
    __builtin_memcpy(&h, &u, sizeof h);
    return h;
}
__device__ __forceinline__ i16x2 as_i16x2(uint32_t u) { return __builtin_bit_cast(i16x2, u); }

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// The four x-lerps fma(fx, b - a, a) of a packed cell (see score.hip).
template <int LAYOUT>
__device__ __forceinline__ void x_lerps(const u32x4 w, float f, float &x00, float &x10, float &x01, float &x11) {
    if constexpr (LAYOUT == kLayoutLerp) {
        const half2v a0 = as_half2(w.x), a1 = as_half2(w.y), d0 = as_half2(w.z), d1 = as_half2(w.w);
        x00 = fmaf(f, (float)d0.x, (float)a0.x);
        x10 = fmaf(f, (float)d0.y, (float)a0.y);
        x01 = fmaf(f, (float)d1.x, (float)a1.x);
        x11 = fmaf(f, (float)d1.y, (float)a1.y);
    } else {
        constexpr uint32_t kMagic = 0x64646464u;
        const half2v a0 = as_half2(__builtin_amdgcn_perm(kMagic, w.x, 0x04020400u));
        const half2v b0 = as_half2(__builtin_amdgcn_perm(kMagic, w.x, 0x04030401u));
        const half2v a1 = as_half2(__builtin_amdgcn_perm(kMagic, w.y, 0x04020400u));
        const half2v b1 = as_half2(__builtin_amdgcn_perm(kMagic, w.y, 0x04030401u));
        const half2v k1024 = {(_Float16)1024.0f, (_Float16)1024.0f};
        const half2v d0 = b0 - a0, d1 = b1 - a1;
        const half2v v0 = a0 - k1024, v1 = a1 - k1024;
        x00 = fmaf(f, (float)d0.x, (float)v0.x);
        x10 = fmaf(f, (float)d0.y, (float)v0.y);
        x01 = fmaf(f, (float)d1.x, (float)v1.x);
        x11 = fmaf(f, (float)d1.y, (float)v1.y);
    }
}

// s_fx = floor(256 s + 0.5) of a cell at fractions f.
template <int LAYOUT>
__device__ __forceinline__ uint32_t sample_fx(const u32x4 w, float fx, float fy, float fz) {
    float x00, x10, x01, x11;
    x_lerps<LAYOUT>(w, fx, x00, x10, x01, x11);
    const float y0 = fmaf(fy, x10 - x00, x00);
    const float y1 = fmaf(fy, x11 - x01, x01);
    const float sv = fmaf(fz, y1 - y0, y0);
    return LAYOUT == kLayoutLerp ? (uint32_t)(sv + 0.5f) : (uint32_t)fmaf(sv, 256.0f, 0.5f);
}

// What a workgroup samples, valid throughout: 16^3 blocks (a wave takes a 16 x
// 4 strip), 8^3 blocks (a wave each) and 4^3 blocks (a quarter-wave each); to be
// tested sample by sample: 4^3 blocks.  16^3 and 8^3 blocks are first voxel x |
// y << 16 and z; 4^3 ones x, y, z (in blocks, two bits each) within a 16^3 block
// and its slot in base, the first voxels of the workgroup's blocks.
template <int BLOCKS>
struct Lists {
    uint32_t n16, n8, n4, nt4;
    uint2 base[BLOCKS], plain16[BLOCKS], plain8[8 * BLOCKS];
    uint16_t plain4[64 * BLOCKS], tested4[64 * BLOCKS];
};

__device__ __forceinline__ uint32_t rank_of(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// Place in a list of each lane for which `take` holds (lists grow by one
// LDS atomic a wave).
__device__ __forceinline__ uint32_t claim(uint32_t *count, bool take) {
    const uint64_t m = __ballot(take);
    uint32_t base = 0u;
    if (m != 0ull && threadIdx.x % 64u == 0u) base = atomicAdd(count, (uint32_t)__popcll(m));
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + rank_of(m);
}
// Bit 4 i of the result: all four bits 4 i .. 4 i + 3 of m.
__device__ __forceinline__ uint64_t all_four(uint64_t m) {
    m &= m >> 1;
    return m & (m >> 2) & 0x1111111111111111ull;
}

// The block tests: wave v of the workgroup takes a quarter of its 16^3 blocks.
// Lanes 4 i .. 4 i + 3 test a block for the four particles; it is skipped or
// plain if all four agree.  Lane 4 i adds the plain blocks' n, sum t and sum
// t^2.
template <int BLOCKS, typename A>
__device__ __forceinline__ void list_blocks(const A &a, uint32_t first, uint32_t wave, uint32_t pbase, uint32_t last,
                                            Lists<BLOCKS> &list, uint32_t sums[3]) {
    const uint32_t lane = threadIdx.x % 64u;
    float w[12];
    const float4 *wp = (const float4 *)(a.words + 12 * (size_t)min(pbase + lane % 4u, last));
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const float4 v = wp[e];
        w[4 * e] = v.x;
        w[4 * e + 1] = v.y;
        w[4 * e + 2] = v.z;
        w[4 * e + 3] = v.w;
    }
    const float radius = ball_radius(w);
    const bool bounded = coords_bounded(w, a.tn);
    const uint32_t need16 = field_need(7.5f, radius, bounded), need8 = field_need(3.5f, radius, bounded),
                   need4 = field_need(1.5f, radius, bounded);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t *>(a.field), (short)0, a.sn[0] * a.sn[1] * a.sn[2], kBufferWord3);
    const uint32_t fx = (uint32_t)a.sn[0], fxy = (uint32_t)a.sn[0] * (uint32_t)a.sn[1];
    const auto field_at = [&](float cx, float cy, float cz) {
        const float u0 = fmaf(w[2], cz, fmaf(w[1], cy, fmaf(w[0], cx, w[3])));
        const float u1 = fmaf(w[6], cz, fmaf(w[5], cy, fmaf(w[4], cx, w[7])));
        const float u2 = fmaf(w[10], cz, fmaf(w[9], cy, fmaf(w[8], cx, w[11])));
        const uint32_t x = floor_u32(__builtin_amdgcn_fmed3f(u0, 0.0f, (float)a.sn[0] - 0.5f));
        const uint32_t y = floor_u32(__builtin_amdgcn_fmed3f(u1, 0.0f, (float)a.sn[1] - 0.5f));
        const uint32_t z = floor_u32(__builtin_amdgcn_fmed3f(u2, 0.0f, (float)a.sn[2] - 0.5f));
        return (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rs, mad_u24(z, fxy, mad_u24(y, fx, x)), 0, 0);
    };
    const bool leader = lane % 4u == 0u;
    // 16^3 blocks
    const uint32_t quota = a.blocks / kWaves, slot0 = wave * quota + lane / 4u, id = first + slot0;
    const bool exists = lane / 4u < quota && id < a.n16;
    const uint32_t row = id / a.g16[0], bx = id - row * a.g16[0], bz = row / a.g16[1], by = row - bz * a.g16[1];
    uint64_t open;
    {
        const uint32_t f = field_at(fmaf(16.0f, (float)bx, 7.5f), fmaf(16.0f, (float)by, 7.5f),
                                    fmaf(16.0f, (float)bz, 7.5f));
        uint4 t = make_uint4(0u, 0u, 0u, 0u);
        if (exists) t = a.t16[id];
        const bool decided = (f & kFieldDist) >= need16;
        const uint64_t off = all_four(__ballot(decided && !(f & kFieldOn))),
                       on = all_four(__ballot(decided && (f & kFieldOn) != 0u));
        const uint64_t me = 1ull << (lane & ~3u);
        // (t.x: voxels of the block in the target and its FOV)
        const bool plain = leader && t.x == 4096u && (on & me) != 0ull;
        if (plain) {
            sums[0] += t.x;
            sums[1] += t.y;
            sums[2] += t.z;
        }
        const uint2 origin = make_uint2((16u * bx) | ((16u * by) << 16), 16u * bz);
        if (leader && exists) list.base[slot0] = origin;
        const uint32_t at = claim(&list.n16, plain);
        if (plain) list.plain16[at] = origin;
        open = __ballot(leader && t.x != 0u && !plain && (off & me) == 0ull);
    }
    // the 8^3 parts of the open ones, two blocks a turn
    while (open) {
        const uint32_t s0 = (uint32_t)__builtin_ctzll(open);
        open &= open - 1ull;
        const bool two = open != 0ull;
        const uint32_t s1 = two ? (uint32_t)__builtin_ctzll(open) : s0;
        if (two) open &= open - 1ull;
        const uint32_t src = lane < 32u ? s0 : s1, child = lane / 4u % 8u;
        const uint32_t x = 2u * (uint32_t)__shfl((int)bx, (int)src) + (child & 1u),
                       y = 2u * (uint32_t)__shfl((int)by, (int)src) + ((child >> 1) & 1u),
                       z = 2u * (uint32_t)__shfl((int)bz, (int)src) + (child >> 2);
        const bool ok = (lane < 32u || two) && x < a.g8[0] && y < a.g8[1] && z < a.g8[2];
        const uint32_t f = field_at(fmaf(8.0f, (float)x, 3.5f), fmaf(8.0f, (float)y, 3.5f), fmaf(8.0f, (float)z, 3.5f));
        uint4 t = make_uint4(0u, 0u, 0u, 0u);
        if (ok) t = a.t8[x + a.g8[0] * (y + a.g8[1] * z)];
        const bool decided = (f & kFieldDist) >= need8;
        const uint64_t off = all_four(__ballot(decided && !(f & kFieldOn))),
                       on = all_four(__ballot(decided && (f & kFieldOn) != 0u));
        const uint64_t me = 1ull << (lane & ~3u);
        const bool plain = leader && t.x == 512u && (on & me) != 0ull;
        if (plain) {
            sums[0] += t.x;
            sums[1] += t.y;
            sums[2] += t.z;
        }
        const uint32_t at = claim(&list.n8, plain);
        if (plain) list.plain8[at] = make_uint2((8u * x) | ((8u * y) << 16), 8u * z);
        // their 4^3 parts, two at a time
        uint64_t open8 = __ballot(leader && t.x != 0u && !plain && (off & me) == 0ull);
        while (open8) {
            const uint32_t r0 = (uint32_t)__builtin_ctzll(open8);
            open8 &= open8 - 1ull;
            const bool both = open8 != 0ull;
            const uint32_t r1 = both ? (uint32_t)__builtin_ctzll(open8) : r0;
            if (both) open8 &= open8 - 1ull;
            const uint32_t from = lane < 32u ? r0 : r1;
            const uint32_t x4 = 2u * (uint32_t)__shfl((int)x, (int)from) + (child & 1u),
                           y4 = 2u * (uint32_t)__shfl((int)y, (int)from) + ((child >> 1) & 1u),
                           z4 = 2u * (uint32_t)__shfl((int)z, (int)from) + (child >> 2);
            const bool ok4 = (lane < 32u || both) && x4 < a.g4[0] && y4 < a.g4[1] && z4 < a.g4[2];
            const uint32_t f4 =
                field_at(fmaf(4.0f, (float)x4, 1.5f), fmaf(4.0f, (float)y4, 1.5f), fmaf(4.0f, (float)z4, 1.5f));
            uint2 t4 = make_uint2(0u, 0u);
            if (ok4) t4 = a.t4[x4 + a.g4[0] * (y4 + a.g4[1] * z4)];
            const bool dec = (f4 & kFieldDist) >= need4;
            const uint64_t off4 = all_four(__ballot(dec && !(f4 & kFieldOn))),
                           on4 = all_four(__ballot(dec && (f4 & kFieldOn) != 0u));
            const uint32_t n4 = t4.x & 255u;
            const bool pl = leader && n4 == 64u && (on4 & me) != 0ull;
            const bool te = leader && n4 != 0u && !pl && (off4 & me) == 0ull;
            if (pl) {
                sums[0] += n4;
                sums[1] += t4.x >> 8;
                sums[2] += t4.y;
            }
            const uint32_t slot = wave * quota + (uint32_t)__shfl((int)src, (int)from) / 4u;
            const uint16_t e = (uint16_t)((x4 & 3u) | ((y4 & 3u) << 2) | ((z4 & 3u) << 4) | (slot << 6));
            const uint32_t pat = claim(&list.n4, pl), tat = claim(&list.nt4, te);
            if (pl) list.plain4[pat] = e;
            if (te) list.tested4[tat] = e;
        }
    }
}

// VMODE: source FOV validity of a sample: 1 src_ok gathered, 2 packed elements
// equal to the sentinel.  ACC: 0 moments, 1 histogram, 2 the gathers
// alone (loaded words XORed into the result).
template <int LAYOUT, int VMODE, int ACC, typename A>
__device__ __forceinline__ uint32_t tri_body(const A &a, uint32_t block) {
    constexpr bool HIST = ACC == 1, PROBE = ACC == 2;
    constexpr int BLOCKS = HIST ? kHistBlocks : kSumBlocks;
    __shared__ uint32_t lhist[HIST ? PT : 1][HIST ? kHB : 1];
    __shared__ unsigned long long red[HIST ? 1 : kWaves][PT][6];
    __shared__ Lists<BLOCKS> list;
    // The dispatcher hands workgroup b to XCD b % 8: each XCD takes runs of a.run
    // of the (part, particles) sequence, so the workgroups in flight on it share
    // a part or two, whose source its L2 holds, and all of them their share of
    // the parts that are mostly skipped (the last ones in order)
    const uint32_t all = 8u * a.run, groups = (a.np + PT - 1u) / PT, whole = groups * a.parts / all * all;
    const uint32_t seq = block < whole ? block / all * all + block % 8u * a.run + block / 8u % a.run : block;
    const uint32_t part = seq / groups, group = seq - part * groups;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64u));
    const uint32_t lane = threadIdx.x % 64u;
    const uint32_t pbase = a.p0 + group * PT, last = a.p0 + a.np - 1u;
    if (threadIdx.x == 0u) list.n16 = list.n8 = list.n4 = list.nt4 = 0u;
    if constexpr (HIST)
        for (uint32_t q = threadIdx.x; q < (uint32_t)(PT * kHB); q += kThreads) lhist[q / kHB][q % kHB] = 0u;
    __syncthreads();
    uint32_t bsum[3] = {0u, 0u, 0u};
    list_blocks<BLOCKS>(a, part * a.blocks, wave, pbase, last, list, bsum);
    __syncthreads();
    const uint32_t n16 = (uint32_t)__builtin_amdgcn_readfirstlane((int)list.n16),
                   n8 = (uint32_t)__builtin_amdgcn_readfirstlane((int)list.n8),
                   n4 = (uint32_t)__builtin_amdgcn_readfirstlane((int)list.n4),
                   nt4 = (uint32_t)__builtin_amdgcn_readfirstlane((int)list.nt4);

    // recipe words of the four particles (slots past the range repeat the
    // last particle; their sums are not stored)
    float w[PT][12];
#pragma unroll
    for (int p = 0; p < PT; ++p) {
        const auto *wp = as_const(a.words) + 12 * (size_t)min(pbase + (uint32_t)p, last);
#pragma unroll
        for (int e = 0; e < 12; ++e) w[p][e] = wp[e];
    }
    // source element of integer position (x, y, z)
    const uint64_t addr = (uint64_t)a.src;
    constexpr int kElem = LAYOUT == kLayoutLerp ? 16 : 8;
    const v4i rs = {(int)(uint32_t)addr, (int)((uint32_t)(addr >> 32) & 0xFFFFu) | (kElem << 16), (int)a.records,
                    kBufferWord3};
    const auto element_of = [&](uint32_t x, uint32_t y, uint32_t z) -> uint32_t {
        if constexpr (LAYOUT == kLayoutOctTile) {
            uint32_t o = __mul24((int)(x & 3u), -3) + (x << 2);
            o += __mul24((int)(y & 3u), 4 - (int)a.ysb);
            return o + __umul24(y, a.ysb) + __umul24(z, a.zsb);
        } else {
            return mad_u24(z, a.zsb, mad_u24(y, a.ysb, x));
        }
    };
    const auto load = [&](uint32_t e) -> u32x4 {
        if constexpr (LAYOUT == kLayoutLerp) return struct_load_u32x4(rs, (int)e, 0, 0, 0);
        const u32x2 v = struct_load_u32x2(rs, (int)e, 0, 0, 0);
        return u32x4{v.x, v.y, 0u, 0u};
    };
    const uint32_t trow = 4u * (uint32_t)a.tn[0] * (uint32_t)a.tn[1];  // bytes of four slices
    const uint32_t tbytes = trow * (uint32_t)((a.tn[2] + 3) / 4);
    const __amdgpu_buffer_rsrc_t rs_t =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.tz), (short)0, (int)tbytes, kBufferWord3);

    int32_t s1[PT], st[PT];
    unsigned long long s2[PT];
    uint32_t rbin[HIST ? PT : 1], rcnt[HIST ? PT : 1];  // histogram: the current run of samples in one bin
    uint32_t chk = 0u;
#pragma unroll
    for (int p = 0; p < PT; ++p) {
        s1[p] = st[p] = 0;
        s2[p] = 0ull;
        if (HIST) rbin[p] = rcnt[p] = 0u;
    }
    const auto count_bin = [&](int p, uint32_t sfx, uint32_t t3) {
        if constexpr (HIST) {
            const uint32_t bin = (sfx >> 11) * kMiBins + t3;
            if (bin != rbin[p]) {
                if (rcnt[p]) atomicAdd(&lhist[p][rbin[p]], rcnt[p]);
                rbin[p] = bin;
                rcnt[p] = 0u;
            }
            rcnt[p] += 1u;
        }
    };
    // quarters of a wave are 4 x 4 squares
    const uint32_t l16 = lane % 16u, quarter = lane / 16u;

    // Two slices fk, fk + 1 of a column of valid samples (t: their target
    // bytes in the low half); mask: 0 where the samples do not count.
    const auto two_slices = [&](const float mx[PT], const float my[PT], const float mz[PT], float fk, uint32_t t,
                                uint32_t mask) {
        float fx[2][PT], fy[2][PT], fz[2][PT];
        u32x4 v[2][PT];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float z = k ? fk + 1.0f : fk;
#pragma unroll
            for (int p = 0; p < PT; ++p) {
                const float ux = fmaf(w[p][2], z, mx[p]);
                const float uy = fmaf(w[p][6], z, my[p]);
                const float uz = fmaf(w[p][10], z, mz[p]);
                v[k][p] = load(element_of(floor_u32(ux), floor_u32(uy), floor_u32(uz)));
                fx[k][p] = __builtin_amdgcn_fractf(ux);
                fy[k][p] = __builtin_amdgcn_fractf(uy);
                fz[k][p] = __builtin_amdgcn_fractf(uz);
            }
        }
        const uint32_t t2 = __builtin_amdgcn_perm(0u, t, 0x0C010C00u);
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            if constexpr (PROBE) {
                chk ^= v[0][p].x ^ v[1][p].x;
                if (LAYOUT == kLayoutLerp) chk ^= v[0][p].w ^ v[1][p].w;
                continue;
            }
            const uint32_t a0 = sample_fx<LAYOUT>(v[0][p], fx[0][p], fy[0][p], fz[0][p]);
            const uint32_t a1 = sample_fx<LAYOUT>(v[1][p], fx[1][p], fy[1][p], fz[1][p]);
            if constexpr (HIST) {
                if (mask) {
                    count_bin(p, a0, (t2 & 0xFFu) >> 3);
                    count_bin(p, a1, t2 >> 19);
                }
            } else {
                const i16x2 s = as_i16x2((((a1 << 16) | a0) ^ 0x80008000u) & mask);
                s1[p] = __builtin_amdgcn_sdot2(s, i16x2{1, 1}, s1[p], false);
                s2[p] += (uint32_t)__builtin_amdgcn_sdot2(s, s, 0, false);
                st[p] = __builtin_amdgcn_sdot2(s, as_i16x2(t2), st[p], false);
            }
        }
    };

    const auto columns = [&](uint32_t i, uint32_t j, float mx[PT], float my[PT], float mz[PT]) {
        const float fi = (float)i, fj = (float)j;
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            mx[p] = fmaf(w[p][1], fj, fmaf(w[p][0], fi, w[p][3]));
            my[p] = fmaf(w[p][5], fj, fmaf(w[p][4], fi, w[p][7]));
            mz[p] = fmaf(w[p][9], fj, fmaf(w[p][8], fi, w[p][11]));
        }
    };
    // 16^3 blocks, a 16 x 4 strip a wave, then 8^3 blocks
#pragma unroll 1
    for (uint32_t u = 0; u < n16 + (n8 + kWaves - 1u) / kWaves; ++u) {
        const bool whole = u < n16;
        const uint32_t u8 = (u - n16) * kWaves + wave;
        if (!whole && u8 >= n8) break;
        const uint2 unit = whole ? list.plain16[u] : list.plain8[u8];
        const uint32_t xy = (uint32_t)__builtin_amdgcn_readfirstlane((int)unit.x),
                       z0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)unit.y);
        const uint32_t i = (xy & 0xFFFFu) + l16 % 4u + 4u * (whole ? quarter : quarter % 2u);
        const uint32_t j = (xy >> 16) + l16 / 4u + 4u * (whole ? wave : quarter / 2u);
        float mx[PT], my[PT], mz[PT];
        columns(i, j, mx, my, mz);
        const uint32_t tcol = 4u * ((uint32_t)a.tn[0] * j + i);
        const uint32_t zq1 = z0 / 4u + (whole ? 4u : 2u);
#pragma unroll 1
        for (uint32_t zq = z0 / 4u; zq < zq1; ++zq) {
            uint32_t t4 = 0u;
            if (!PROBE) t4 = __builtin_amdgcn_raw_buffer_load_b32(rs_t, tcol, zq * trow, 0);
#pragma unroll
            for (int h = 0; h < 2; ++h) two_slices(mx, my, mz, (float)(4u * zq + 2u * h), t4 >> (16 * h), 0xFFFFFFFFu);
        }
    }
    // 4^3 blocks, a quarter of a wave each (the quarters left over in the last
    // turn repeat the first block, masked out)
    const auto part_of = [&](const uint16_t *parts, uint32_t i, uint32_t &x, uint32_t &y, uint32_t &z) {
        const uint32_t e = parts[i];
        const uint2 b = list.base[e >> 6];
        x = (b.x & 0xFFFFu) + 4u * (e & 3u) + l16 % 4u;
        y = (b.x >> 16) + 4u * ((e >> 2) & 3u) + l16 / 4u;
        z = b.y + 4u * ((e >> 4) & 3u);
    };
#pragma unroll 1
    for (uint32_t u = 4u * wave; u < n4; u += 4u * kWaves) {
        const bool mine = u + quarter < n4;
        uint32_t i, j, z;
        part_of(list.plain4, mine ? u + quarter : 0u, i, j, z);
        float mx[PT], my[PT], mz[PT];
        columns(i, j, mx, my, mz);
        uint32_t t4 = 0u;
        if (!PROBE) t4 = __builtin_amdgcn_raw_buffer_load_b32(rs_t, 4u * ((uint32_t)a.tn[0] * j + i) + z / 4u * trow, 0, 0);
#pragma unroll
        for (int h = 0; h < 2; ++h)
            two_slices(mx, my, mz, (float)z + (float)(2 * h), t4 >> (16 * h), mine ? 0xFFFFFFFFu : 0u);
    }

    // blocks whose samples are tested one by one; n | t << 9 and t^2 of the
    // valid ones
    uint32_t nt[PT], tt[PT];
#pragma unroll
    for (int p = 0; p < PT; ++p) nt[p] = tt[p] = 0u;
    const __amdgpu_buffer_rsrc_t rs_tf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.fz), (short)0,
                                                                           a.fz ? (int)tbytes : 0, kBufferWord3);
    const uint32_t fx1 = (uint32_t)a.sn[0], fx2 = (uint32_t)a.sn[0] * (uint32_t)a.sn[1];
    const __amdgpu_buffer_rsrc_t rs_ok = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t *>(a.src_ok), (short)0, VMODE == 1 ? a.sn[0] * a.sn[1] * a.sn[2] : 0, kBufferWord3);
    const uint32_t ex = __float_as_uint((float)(a.sn[0] - 1)), ey = __float_as_uint((float)(a.sn[1] - 1)),
                   ez = __float_as_uint((float)(a.sn[2] - 1));
#pragma unroll 1
    for (uint32_t u = 4u * wave; u < nt4; u += 4u * kWaves) {
        const bool mine = u + quarter < nt4;
        uint32_t i, j, z0;
        part_of(list.tested4, mine ? u + quarter : 0u, i, j, z0);
        float mx[PT], my[PT], mz[PT];
        columns(i, j, mx, my, mz);
        const bool column = mine && i < (uint32_t)a.tn[0] && j < (uint32_t)a.tn[1];
        uint32_t t4 = 0u, f4 = 0xFFFFFFFFu;
        if constexpr (!PROBE) {
            const uint32_t o = column ? 4u * ((uint32_t)a.tn[0] * j + i) + z0 / 4u * trow : 0xFFFFFFF0u;
            t4 = __builtin_amdgcn_raw_buffer_load_b32(rs_t, o, 0, 0);
            if (a.fz) f4 = __builtin_amdgcn_raw_buffer_load_b32(rs_tf, o, 0, 0);
        }
#pragma unroll 1
        for (uint32_t k = 0; k < 4u; ++k) {
            const uint32_t z = z0 + k;
            const uint32_t t = t4 & 255u;
            const bool ton = column && z < (uint32_t)a.tn[2] && (f4 & 255u) != 0u;
            t4 >>= 8;
            f4 >>= 8;
            const float fk = (float)z;
            float fx[PT], fy[PT], fz[PT];
            uint32_t e[PT], ok[PT];
            bool in[PT];
            u32x4 v[PT];
#pragma unroll
            for (int p = 0; p < PT; ++p) {
                const float ux = fmaf(w[p][2], fk, mx[p]);
                const float uy = fmaf(w[p][6], fk, my[p]);
                const float uz = fmaf(w[p][10], fk, mz[p]);
                // 0 <= u <= n - 1 as unsigned compares of bit patterns (the
                // coordinates are never -0); outside samples load past the end
                in[p] = ton & (__float_as_uint(ux) <= ex) & (__float_as_uint(uy) <= ey) & (__float_as_uint(uz) <= ez);
                const uint32_t ix = floor_u32(ux), iy = floor_u32(uy), iz = floor_u32(uz);
                fx[p] = __builtin_amdgcn_fractf(ux);
                fy[p] = __builtin_amdgcn_fractf(uy);
                fz[p] = __builtin_amdgcn_fractf(uz);
                e[p] = in[p] ? element_of(ix, iy, iz) : a.records;
                ok[p] = 1u;
                if (VMODE == 1)
                    ok[p] = __builtin_amdgcn_raw_buffer_load_b8(
                        rs_ok, in[p] ? mad_u24(iz, fx2, mad_u24(iy, fx1, ix)) : 0xFFFFFFFFu, 0, 0);
            }
#pragma unroll
            for (int p = 0; p < PT; ++p) v[p] = load(e[p]);
#pragma unroll
            for (int p = 0; p < PT; ++p) {
                if constexpr (PROBE) {
                    chk ^= v[p].x;
                    if (LAYOUT == kLayoutLerp) chk ^= v[p].w;
                    continue;
                }
                bool valid = in[p] & (ok[p] != 0u);
                if (VMODE == 2)
                    valid = valid & (LAYOUT == kLayoutLerp ? v[p].x != kLerpSentinel
                                                           : (v[p].x != (uint32_t)a.sentinel) |
                                                                 (v[p].y != (uint32_t)(a.sentinel >> 32)));
                if (valid) {
                    const uint32_t sfx = sample_fx<LAYOUT>(v[p], fx[p], fy[p], fz[p]);
                    if constexpr (HIST) {
                        count_bin(p, sfx, t >> 3);
                    } else {
                        const i16x2 s = as_i16x2(sfx ^ 0x8000u);  // (high half zero)
                        nt[p] += 1u + (t << 9);
                        tt[p] += t * t;
                        s1[p] = __builtin_amdgcn_sdot2(s, i16x2{1, 0}, s1[p], false);
                        s2[p] += (uint32_t)__builtin_amdgcn_sdot2(s, s, 0, false);
                        st[p] = __builtin_amdgcn_sdot2(s, as_i16x2(t), st[p], false);
                    }
                }
            }
        }
    }
    if constexpr (PROBE) return chk;

    if constexpr (HIST) {
#pragma unroll
        for (int p = 0; p < PT; ++p)
            if (rcnt[p]) atomicAdd(&lhist[p][rbin[p]], rcnt[p]);
        __syncthreads();
        for (uint32_t q = threadIdx.x; q < (uint32_t)(PT * kHB); q += kThreads) {
            const uint32_t p = q / kHB, b = q % kHB, v = lhist[p][b];
            if (v != 0u && pbase + p <= last) atomicAdd(a.hist + (size_t)kHB * (pbase + p) + b, v);
        }
        return 0u;
    }

    if ((n16 | n8 | n4 | nt4) == 0u) return 0u;
    const unsigned long long bn = wave_sum(bsum[0]), bt = wave_sum(bsum[1]);
    const unsigned long long btt = wave_sum((unsigned long long)bsum[2]);
#pragma unroll
    for (int p = 0; p < PT; ++p) {
        const long long S1 = wave_sum(s1[p]), ST = wave_sum((long long)st[p]);
        const unsigned long long S2 = wave_sum(s2[p]);
        unsigned long long n = bn, t = bt, t2 = btt;
        if (nt4) {
            n += wave_sum(nt[p] & 511u);
            t += wave_sum(nt[p] >> 9);
            t2 += wave_sum(tt[p]);
        }
        if (lane == 0u) {
            red[wave][p][0] = n;
            red[wave][p][1] = (unsigned long long)S1;
            red[wave][p][2] = t;
            red[wave][p][3] = S2;
            red[wave][p][4] = t2;
            red[wave][p][5] = (unsigned long long)ST;
        }
    }
    __syncthreads();
    if (threadIdx.x < (unsigned)(PT * 6)) {
        const uint32_t p = threadIdx.x / 6u, m = threadIdx.x % 6u;
        const auto sum = [&](uint32_t q) { return (red[0][p][q] + red[1][p][q]) + (red[2][p][q] + red[3][p][q]); };
        // s = s' + 2^15 (two's complement throughout)
        unsigned long long v = sum(m);
        if (m == 1u) v += sum(0) << 15;
        if (m == 3u) v += (sum(1) << 16) + (sum(0) << 30);
        if (m == 5u) v += sum(2) << 15;
        if (pbase + p <= last && v) atomicAdd(a.sums + 6 * (size_t)(pbase + p) + m, v);
    }
    return 0u;
}

template <int LAYOUT, int VMODE, int ACC>
__global__ __launch_bounds__(kThreads) void k_score_tri(const Args a, uint32_t first) {
    tri_body<LAYOUT, VMODE, ACC>(a, first + blockIdx.x);
}

template <int LAYOUT>
__global__ __launch_bounds__(kThreads) void k_probe_tri(const Args a, uint32_t first, uint32_t key, uint32_t *out) {
    const uint32_t chk = tri_body<LAYOUT, 2, 2>(a, first + blockIdx.x);
    if (chk == key) out[0] = chk;
}

// The pairs of a batch's image class: pair d owns workgroups offs[d] ..
// offs[d + 1) - 1.
template <int LAYOUT, int VMODE>
__global__ __launch_bounds__(kThreads) void k_batch_tri(const Args *pairs_g, const uint32_t *offs_g,
                                                        const uint32_t *kmax_g, uint32_t n_pairs, uint32_t k,
                                                        uint32_t first) {
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
    tri_body<LAYOUT, VMODE, 0>(a, block - offs[lo]);
}

// ---------------------------------------------------------------- preparation

// Bytes of four slices as dwords (slices past the end zero); blockIdx.y 1: of
// the FOV.
__global__ __launch_bounds__(256) void k_slices4(const uint8_t *vol, const uint8_t *fov, uint32_t plane, int32_t nz,
                                                 uint32_t *tz, uint32_t *fz) {
    const uint8_t *in = blockIdx.y ? fov : vol;
    uint32_t *out = blockIdx.y ? fz : tz;
    const uint32_t n = plane * ((uint32_t)(nz + 3) / 4);
    for (uint32_t q = blockIdx.x * 256u + threadIdx.x; q < n; q += gridDim.x * 256u) {
        const uint32_t zq = q / plane, xy = q - zq * plane;
        uint32_t v = 0u;
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if ((int32_t)(4 * zq) + s < nz) v |= (uint32_t)in[xy + (int64_t)plane * (4 * zq + s)] << (8 * s);
        out[q] = v;
    }
}

// n | sum t << 8 and sum t^2 of the 4^3 blocks: four threads a block, a column
// of four dwords each.
__global__ __launch_bounds__(256) void k_blocks4(const uint32_t *tz, const uint32_t *fz, int32_t nx, int32_t ny,
                                                 int32_t nz, uint32_t gx, uint32_t gy, uint32_t gz, uint2 *out) {
    const uint32_t n = gx * gy * gz;
    for (uint32_t q = blockIdx.x * 256u + threadIdx.x; q < 4 * n; q += gridDim.x * 256u) {
        const uint32_t blk = q / 4, r = blk / gx, zb = r / gy;
        const int32_t x = 4 * (int32_t)(blk - r * gx) + (int32_t)(q % 4), y0 = 4 * (int32_t)(r - zb * gy), zq = (int32_t)zb;
        uint32_t c = 0u, s = 0u, s2 = 0u;
        for (int32_t y = y0; y < min(y0 + 4, ny) && x < nx; ++y) {
            const int64_t o = ((int64_t)zq * ny + y) * nx + x;
            const uint32_t t = tz[o], f = fz ? fz[o] : 0xFFFFFFFFu;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (4 * zq + k >= nz || ((f >> (8 * k)) & 255u) == 0u) continue;
                const uint32_t v = (t >> (8 * k)) & 255u;
                c += 1u;
                s += v;
                s2 += v * v;
            }
        }
#pragma unroll
        for (int o = 2; o > 0; o >>= 1) {
            c += __shfl_xor(c, o);
            s += __shfl_xor(s, o);
            s2 += __shfl_xor(s2, o);
        }
        if (q % 4 == 0) out[blk] = make_uint2(c | (s << 8), s2);
    }
}

// Sums over the blocks of side 8 and 16: a wave makes one of 16 from its 64
// blocks of 4^3, a lane each (one thread over all 64 waited on a chain of
// loads: 4 + 12 us for both sides, 4 us so).
__global__ __launch_bounds__(256) void k_blocks(const uint2 *t4, uint32_t g4x, uint32_t g4y, uint32_t g4z, uint32_t g8x,
                                                uint32_t g8y, uint32_t g8z, uint32_t gx, uint32_t gy, uint32_t gz,
                                                uint4 *t8, uint4 *t16) {
    const uint32_t n = gx * gy * gz, lane = threadIdx.x % 64;
    const uint32_t lx = lane & 3u, ly = (lane >> 2) & 3u, lz = lane >> 4;
    for (uint32_t w = blockIdx.x * 4 + threadIdx.x / 64; w < n; w += gridDim.x * 4) {
        const uint32_t t = w / gx, bz = t / gy, bx = w - t * gx, by = t - bz * gy;
        const uint32_t x = 4 * bx + lx, y = 4 * by + ly, z = 4 * bz + lz;
        uint32_t c = 0u, s = 0u, s2 = 0u;
        if (x < g4x && y < g4y && z < g4z) {
            const uint2 b = t4[x + (int64_t)g4x * (y + (int64_t)g4y * z)];
            c = b.x & 255u;
            s = b.x >> 8;
            s2 = b.y;
        }
        const auto add = [&](int o) {
            c += __shfl_xor(c, o);
            s += __shfl_xor(s, o);
            s2 += __shfl_xor(s2, o);
        };
        add(1);
        add(4);
        add(16);
        const uint32_t x8 = 2 * bx + lx / 2, y8 = 2 * by + ly / 2, z8 = 2 * bz + lz / 2;
        if ((lane & 21u) == 0u && x8 < g8x && y8 < g8y && z8 < g8z)
            t8[x8 + (int64_t)g8x * (y8 + (int64_t)g8y * z8)] = make_uint4(c, s, s2, 0u);
        add(2);
        add(8);
        add(32);
        if (lane == 0) t16[w] = make_uint4(c, s, s2, 0u);
    }
}

// Field bytes of state off at a distance of at least `need` (its bytes are 16-byte
// aligned).
__global__ __launch_bounds__(256) void k_count_off(const uint8_t *field, uint32_t n, uint32_t need,
                                                   unsigned long long *out) {
    const uint32_t stride = gridDim.x * 256u, t = blockIdx.x * 256u + threadIdx.x;
    uint32_t c = 0u;
    const auto off = [&](uint32_t b) { return b - need < 128u - need ? 1u : 0u; };
    for (uint32_t q = t; q < n / 16; q += stride) {
        const uint4 v = ((const uint4 *)field)[q];
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 16; ++e) c += off((w[e / 4] >> (8 * (e % 4))) & 255u);
    }
    for (uint32_t q = n / 16 * 16 + t; q < n; q += stride) c += off(field[q]);
    c = wave_sum(c);
    if (threadIdx.x % 64u == 0u && c) atomicAdd(out, (unsigned long long)c);
}

unsigned blocks_for(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 8192)); }
uint32_t cells(int32_t n, int32_t side) { return (uint32_t)((n + side - 1) / side); }

Args make_args(const ScoreLaunch &L, bool batch = false) {
    Args a;
    a.src = L.src_packed;
    a.src_ok = L.src_ok;
    a.field = L.tri.field;
    a.tz = L.tri.tz;
    a.fz = L.tri.fz;
    a.t8 = (const uint4 *)L.tri.t8;
    a.t16 = (const uint4 *)L.tri.t16;
    a.t4 = (const uint2 *)L.tri.t4;
    a.words = L.words;
    a.sums = L.sums;
    a.hist = L.hist;
    a.sentinel = L.sentinel;
    for (int d = 0; d < 3; ++d) {
        a.sn[d] = L.sn[d];
        a.tn[d] = L.tn[d];
        a.g4[d] = cells(L.tn[d], 4);
        a.g8[d] = cells(L.tn[d], 8);
        a.g16[d] = cells(L.tn[d], 16);
    }
    a.n16 = a.g16[0] * a.g16[1] * a.g16[2];
    const uint32_t eb = (uint32_t)packed_bytes_per_voxel(L.layout);
    a.records = (uint32_t)(packed_bytes(L.layout, L.sn) / eb);
    if (L.layout == kLayoutOctTile) {
        a.ysb = 4u * cells(L.sn[0], 4);  // a quarter of a row of tiles
        a.zsb = 16u * cells(L.sn[0], 4) * cells(L.sn[1], 4);
    } else {
        a.ysb = (uint32_t)L.sn[0];
        a.zsb = (uint32_t)L.sn[0] * (uint32_t)L.sn[1];
    }
    a.p0 = L.p0;
    a.np = L.np;
    // fewer blocks a workgroup while the launch would have under 2048 of them
    // (eight per CU)
    const uint64_t groups = (L.np + PT - 1) / PT, most = L.hist ? kHistBlocks : (L.apart ? (int)kApartBlocks : kSumBlocks);
    const uint64_t want = (uint64_t)a.n16 * groups / 2048u;
    a.blocks = kWaves * (uint32_t)std::min<uint64_t>(most / kWaves, std::max<uint64_t>(1u, want / kWaves));
    a.parts = (a.n16 + a.blocks - 1) / a.blocks;
    a.run = batch ? kBatchRun : (L.apart ? kApartRun : kRun);
    return a;
}

uint64_t groups_of(const Args &a) { return (uint64_t)a.parts * ((a.np + PT - 1) / PT); }

typedef void (*Kernel)(const Args, uint32_t);
typedef void (*BatchKernel)(const Args *, const uint32_t *, const uint32_t *, uint32_t, uint32_t, uint32_t);

template <int LAYOUT, int ACC>
Kernel pick(int vmode) {
    return vmode == 2 ? k_score_tri<LAYOUT, 2, ACC> : k_score_tri<LAYOUT, 1, ACC>;
}
template <int ACC>
Kernel pick(int layout, int vmode) {
    if (layout == kLayoutLerp) return pick<kLayoutLerp, ACC>(vmode);
    return layout == kLayoutOct ? pick<kLayoutOct, ACC>(vmode) : pick<kLayoutOctTile, ACC>(vmode);
}
template <int LAYOUT>
BatchKernel pick_batch(int vmode) {
    return vmode == 2 ? k_batch_tri<LAYOUT, 2> : k_batch_tri<LAYOUT, 1>;
}

}  // namespace

TriSizes tri_sizes(const int32_t sn[3], const int32_t tn[3]) {
    TriSizes s;
    const uint64_t n = (uint64_t)sn[0] * sn[1] * sn[2];
    s.bits = 4ull * cells(sn[0], 32) * (uint64_t)sn[1] * (uint64_t)sn[2];
    s.field = n;
    s.tz = 4ull * (uint64_t)tn[0] * tn[1] * cells(tn[2], 4);
    s.t4 = 8ull * cells(tn[0], 4) * cells(tn[1], 4) * cells(tn[2], 4);
    s.t8 = 16ull * cells(tn[0], 8) * cells(tn[1], 8) * cells(tn[2], 8);
    s.t16 = 16ull * cells(tn[0], 16) * cells(tn[1], 16) * cells(tn[2], 16);
    return s;
}

hipError_t launch_tri_target(const uint8_t *vol, const uint8_t *fov, const int32_t n[3], uint32_t *tz, uint32_t *fz,
                             void *t4, void *t8, void *t16, hipStream_t s) {
    const int64_t plane = (int64_t)n[0] * n[1];
    hipLaunchKernelGGL(k_slices4, dim3(blocks_for(plane * ((n[2] + 3) / 4)), fov ? 2 : 1), dim3(256), 0, s, vol, fov,
                       (uint32_t)plane, n[2], tz, fz);
    uint32_t g[3][3];
    for (int l = 0; l < 3; ++l)
        for (int d = 0; d < 3; ++d) g[l][d] = cells(n[d], 4 << l);
    const auto count = [&](int l) { return (int64_t)g[l][0] * g[l][1] * g[l][2]; };
    hipLaunchKernelGGL(k_blocks4, dim3(blocks_for(4 * count(0))), dim3(256), 0, s, (const uint32_t *)tz,
                       (const uint32_t *)(fov ? fz : nullptr), n[0], n[1], n[2], g[0][0], g[0][1], g[0][2], (uint2 *)t4);
    hipLaunchKernelGGL(k_blocks, dim3(blocks_for(64 * count(2))), dim3(256), 0, s, (const uint2 *)t4, g[0][0], g[0][1],
                       g[0][2], g[1][0], g[1][1], g[1][2], g[2][0], g[2][1], g[2][2], (uint4 *)t8, (uint4 *)t16);
    return hipGetLastError();
}

// With a source FOV only, and for moments only if it leaves enough to skip: with
// an apical cone two fifths of the pairs are skipped (4.37 against 5.98 ms on
// 160^3 images).  With little to skip both kernels run at the rate of the texture
// path, and the tiles of score.hip, whose 32-voxel rows share more cache lines,
// are ahead: without a FOV 2.63 against 2.69 ms (128 x 130 x 126, N = 1500), 2.02
// against 2.16 (60 x 150 x 90, N = 3000), histograms 3.69 against 3.96; with a FOV
// of the whole 128 x 120 x 110 (N = 600) 0.83 against 0.94 ms, 1.0 against 1.3 in
// the first iterations, whose particles lie far apart, and with holes a
// few voxels apart 1.0 against 1.6.  (Histograms with a FOV are faster by blocks
// throughout: full FOV 6.6 against 8.2 ms a registration.)
//
// The line: the share of source voxels from which a target block of 8^3 reaches
// no valid sample, against what both kernels took (128 x 120 x 110, N = 600;
// early, late iterations): 0.07 of them 1.25, 0.90 of the tiles' time; 0.16 1.1,
// 0.82; 0.25 0.95, 0.79; a cone 0.35 0.86; target voxels of twice the spacing in
// that cone 0.26 0.99, of four times 0.115 1.14.
constexpr double kOffShare = 0.12;
bool tri_pays(uint64_t off, const int32_t sn[3]) {
    return (double)off >= kOffShare * (double)sn[0] * (double)sn[1] * (double)sn[2];
}

hipError_t launch_tri_off(const uint8_t *field, const int32_t sn[3], const double ts[3], const double ss[3],
                          unsigned long long *out, hipStream_t s) {
    // ball radius of the unit block: exact for cubic source voxels
    const double radius = sqrt(ts[0] * ts[0] + ts[1] * ts[1] + ts[2] * ts[2]) / cbrt(ss[0] * ss[1] * ss[2]);
    const double need = ceil((double)kFieldUnit * (3.5 * radius + (double)kFieldMargin));
    if (!(need <= (double)kFieldDist)) return hipSuccess;  // no such block is ever decided
    const uint32_t n = (uint32_t)sn[0] * (uint32_t)sn[1] * (uint32_t)sn[2];
    hipLaunchKernelGGL(k_count_off, dim3(std::min(blocks_for(n / 16 + 1), 256u)), dim3(256), 0, s, field, n,
                       (uint32_t)need, out);
    return hipGetLastError();
}

bool tri_supported(const ScoreLaunch &L) {
    return L.mode == kModeImageTrilinear && L.tri.field != nullptr && L.src_ok != nullptr &&
           (L.layout == kLayoutOct || L.layout == kLayoutOctTile || L.layout == kLayoutLerp);
}

hipError_t launch_tri(const ScoreLaunch &L, hipStream_t s) {
    if (L.np == 0) return hipSuccess;
    const Args a = make_args(L);
    const int vmode = L.has_sentinel ? 2 : 1;
    const Kernel k = L.hist ? pick<1>(L.layout, vmode) : pick<0>(L.layout, vmode);
    return launch_groups(groups_of(a), [&](uint32_t first, dim3 grid) {
        hipLaunchKernelGGL(k, grid, dim3(kThreads), 0, s, a, first);
    });
}

hipError_t launch_tri_probe(const ScoreLaunch &L, uint32_t key, uint32_t *out, hipStream_t s) {
    if (L.np == 0) return hipSuccess;
    const Args a = make_args(L);
    auto *k = L.layout == kLayoutLerp ? k_probe_tri<kLayoutLerp>
                                      : (L.layout == kLayoutOct ? k_probe_tri<kLayoutOct> : k_probe_tri<kLayoutOctTile>);
    return launch_groups(groups_of(a), [&](uint32_t first, dim3 grid) {
        hipLaunchKernelGGL(k, grid, dim3(kThreads), 0, s, a, first, key, out);
    });
}

size_t tri_args_bytes() { return sizeof(Args); }

uint64_t tri_args(const ScoreLaunch &L, void *out) {
    const Args a = make_args(L, true);
    memcpy(out, &a, sizeof a);
    return groups_of(a);
}

hipError_t launch_batch_tri(int layout, int vmode, const void *pairs, const uint32_t *offs, const uint32_t *kmax,
                            uint32_t n_pairs, uint32_t groups, uint32_t k, hipStream_t s) {
    if (n_pairs == 0) return hipSuccess;
    const BatchKernel b = layout == kLayoutLerp
                              ? pick_batch<kLayoutLerp>(vmode)
                              : (layout == kLayoutOct ? pick_batch<kLayoutOct>(vmode) : pick_batch<kLayoutOctTile>(vmode));
    return launch_groups(groups, [&](uint32_t first, dim3 grid) {
        hipLaunchKernelGGL(b, grid, dim3(kThreads), 0, s, (const Args *)pairs, offs, kmax, n_pairs, k, first);
    });
}

}  // namespace smc
