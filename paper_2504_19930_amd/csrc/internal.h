// Internal launch interface between the C ABI (api.hip) and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace smc {

// floor and convert in one instruction (exact for the non-negative
// coordinates whose results are used)
__device__ __forceinline__ uint32_t floor_u32(float x) {
    int r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
    return (uint32_t)r;
}

// a * b + c on the low 24 bits of a and b, as one instruction (the compiler
// otherwise forms two multiplies and a three-way add); b is uniform across
// the wave (a stride) and is passed as a scalar operand.
__device__ __forceinline__ uint32_t mad_u24(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(b), "v"(c));
    return r;
}

// ---- block tests on a source's distance field (dice.hip, tri.hip)
//
// Field byte of a voxel: its state, and the distance (eighths of a voxel, below
// 16 voxels) from its box to the nearest box of a voxel of the other state; 0
// where that touches.  The image of a cubic block of target voxels under the
// recipe lies in a ball about the image of its centre, so a distance of at
// least the ball's radius decides the block.
constexpr uint32_t kFieldOn = 128u, kFieldDist = 127u;
constexpr float kFieldUnit = 8.0f;
// Bound on the partial sums of the recipe below which a sample's and a block
// centre's FP32 coordinates are each within 0.023 voxel of the exact map, so
// that the margin covers both; beyond it no block is decided.
constexpr float kFieldCoordLimit = 262144.0f, kFieldMargin = 0.0625f;

// Farthest image of a corner of the cube [-1, 1]^3 from its centre's, under
// recipe words w.
__device__ __forceinline__ float ball_radius(const float w[12]) {
    float r2 = 0.0f;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        float d2 = 0.0f;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float v = w[4 * d] + (s & 1 ? w[4 * d + 1] : -w[4 * d + 1]) + (s & 2 ? w[4 * d + 2] : -w[4 * d + 2]);
            d2 = fmaf(v, v, d2);
        }
        r2 = fmaxf(r2, d2);
    }
    return sqrtf(r2);
}
__device__ __forceinline__ bool coords_bounded(const float w[12], const int32_t tn[3]) {
    bool ok = true;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const float b = fabsf(w[4 * d]) * (float)(tn[0] + 16) + fabsf(w[4 * d + 1]) * (float)(tn[1] + 16) +
                        fabsf(w[4 * d + 2]) * (float)(tn[2] + 16) + fabsf(w[4 * d + 3]);
        ok = ok && b < kFieldCoordLimit;
    }
    return ok;
}
// Least field distance (in its units) that decides a block of half side `half`.
__device__ __forceinline__ uint32_t field_need(float half, float radius, bool bounded) {
    return bounded ? (uint32_t)fminf(ceilf(kFieldUnit * (half * radius + kFieldMargin)), 255.0f) : 255u;
}

// Warp-and-score launch: particle range [p0, p0 + np) of `words`, sums
// accumulated (atomically, exactly) into sums[6 * p].
enum ScoreMode : int { kModeMask = 0, kModeImageTrilinear = 1, kModeImageNearest = 2 };

// Source layouts for trilinear sampling (see score.hip): bytes per voxel
// 1, 2, 4, 8, 8, 16; eight, four, two or one gathers per sample.
enum SourceLayout : int {
    kLayoutRaw = 0,
    kLayoutPairX = 1,
    kLayoutQuadXY = 2,
    kLayoutOct = 3,
    kLayoutOctTile = 4,
    kLayoutLerp = 5
};
constexpr int kLayouts = 6;
// The lerp layout marks elements that touch a voxel outside the source FOV
// with a pair of half-precision NaNs in the first word; no valid element
// holds a NaN, so this sentinel always exists.
constexpr uint32_t kLerpSentinel = 0x7E007E00u;

struct ScoreLaunch {
    int mode;
    const uint8_t *src;       // mask: prepared bits; image: intensities
    const void *src_packed;   // trilinear: source in `layout` (nullptr = raw bytes)
    bool has_sentinel;        // packed elements equal to `sentinel` mark samples outside the source FOV
    uint64_t sentinel;
    int layout;               // SourceLayout
    int pt;                   // particles per workgroup: 4, 8 or 16
    int zchunk;               // target z-extent of a tile, less in launches of few items (0 = up to 256)
    // masks: only a and c are needed (the filter's launches), by blocks of the
    // target on the source's distance field (dice.hip); false: all four counts
    bool ac = false;
    struct Dice {
        const uint32_t *bits = nullptr;  // source bitmap
        const uint8_t *field = nullptr;  // source distance field
        const void *t4 = nullptr;        // target blocks of 4^3, 8^3 and 16^3 voxels
        const uint32_t *t8 = nullptr, *t16 = nullptr;
    } dice;
    // trilinear images with a source FOV in the one-gather layouts (tri.hip;
    // nullptr without a FOV or where tiles are faster): field of the valid
    // cells, target (and FOV) bytes of four slices as dwords, target blocks
    struct Tri {
        const uint8_t *field = nullptr;
        const uint32_t *tz = nullptr, *fz = nullptr;
        const void *t4 = nullptr, *t8 = nullptr, *t16 = nullptr;
    } tri;
    // images by blocks: the particles lie far apart for the source's voxels
    bool apart = false;
    // masks, ac launches (or nullptr): kWorkSlots counter triples,
    // kWorkSlotWords apart; summed over the slots, word 0 counts the particle x
    // voxel pairs sampled, word 1 the pairs covered (the decided ones
    // included), word 2 the sampled pairs of blocks inside the source
    unsigned long long *work = nullptr;
    const uint8_t *src_ok;    // image: corner-valid bytes (source FOV) or nullptr
    const uint8_t *tgt;       // mask: prepared bits; image: intensities
    const uint8_t *tgt_fov;   // image: target FOV or nullptr
    const float *words;       // 12 per particle
    unsigned long long *sums; // 6 per particle
    int32_t sn[3], tn[3];
    uint32_t p0, np;
    // mutual information: the launch adds into kMiBins^2 counts per particle
    // (indexed like words) instead of the moments
    uint32_t *hist = nullptr;
};
// Most work items (tiles x particle groups) one scoring launch takes: a grid
// dimension of signed 32-bit size.
constexpr uint64_t kMaxScoreItems = 0x7FFFFFFFull;
// Workgroups of one launch: a grid counts its threads in 32 bits.  launch(first,
// n) launches workgroups first .. first + n - 1 (first a multiple of 8, the XCDs).
constexpr uint64_t kMaxGridGroups = 1ull << 23;
template <typename F>
hipError_t launch_groups(uint64_t groups, F launch) {
    if (groups > kMaxScoreItems) return hipErrorInvalidConfiguration;
    hipError_t e = hipSuccess;
    for (uint64_t first = 0; first < groups && e == hipSuccess; first += kMaxGridGroups) {
        const uint64_t left = groups - first;
        launch((uint32_t)first, dim3((unsigned)(left < kMaxGridGroups ? left : kMaxGridGroups)));
        e = hipGetLastError();
    }
    return e;
}
// Items (tiles x particle groups) of a launch of L's shape with np particles.
uint64_t score_items_for(const ScoreLaunch &L);

hipError_t launch_score(const ScoreLaunch &L, hipStream_t s);
// Gather probe (measurement): the launch's grid, culling, coordinates and
// source loads without the rest of the kernel's work; see score.hip.
bool gather_probe_supported(const ScoreLaunch &L);
hipError_t launch_gather_probe(const ScoreLaunch &L, uint32_t key, uint32_t *out, hipStream_t s);
bool score_pt_supported(int pt);
// whether a packed trilinear layout can address a source of this shape
bool layout_fits(int layout, const int32_t sn[3]);
// Pack a source volume into the layouts pairx or quadxy (edge corners repeat the
// last voxel).  With fov, elements touching a voxel outside it hold `sentinel`
// instead.
hipError_t launch_pack_rows(const uint8_t *vol, const uint8_t *fov, const int32_t n[3], int layout, uint64_t sentinel,
                            void *out, hipStream_t s);
// The same into the x-lerps and the (tiled) octets, either of which may be
// nullptr; ok: corner validity or nullptr, hits: += valid octets that equal the
// sentinel, or nullptr.
hipError_t launch_pack_cells(const uint8_t *vol, const uint8_t *ok, const int32_t n[3], void *lerp, void *oct,
                             bool tiled, uint64_t sentinel, unsigned long long *hits, hipStream_t s);
// Over the elements of `layout` that lie inside the fov, count those equal to
// each candidate (truncated to the element width) -- or, for x-pairs with
// n_cand == 0, a 65536-bin histogram of all element values.
hipError_t launch_count_elements(const uint8_t *vol, const uint8_t *fov, const int32_t n[3], int layout,
                                 const uint64_t *cand, int n_cand, unsigned long long *counts, hipStream_t s);
size_t packed_bytes_per_voxel(int layout);
// bytes of a packed source of shape n (the tiled layout pads x and y to 4)
uint64_t packed_bytes(int layout, const int32_t n[3]);

// Batched warp-and-score: one persistent launch over the work items of many
// pairs of one class (masks, or trilinear images in one layout).
struct BatchPlan {
    int mode, layout, pt, vmode;  // vmode: source FOV validity (0 none, 1 gathered, 2 sentinel)
    const void *pairs;        // device array of per-pair kernel arguments (score_args)
    const uint32_t *offs;     // n_pairs + 1 item offsets
    const uint32_t *kmax;     // iterations per pair
    const uint32_t *lists;    // item ids grouped by XCD
    uint32_t list_off[9];
    uint32_t n_pairs;
    uint32_t grid;            // workgroups: persistent, or (blocks) offs[n_pairs]
    // masks and one-gather images: block kernels, pairs holds their arguments
    // and offs counts workgroups; no queues
    bool blocks = false;
    // item queues: 8 counters (one per XCD list) per iteration, zero before
    // the run; iteration k uses counters[8 (k - 1) .. 8 k)
    uint32_t *counters;
};
size_t score_args_bytes();
void score_args(const ScoreLaunch &L, void *out);
hipError_t launch_batch_score(const BatchPlan &P, uint32_t k, hipStream_t s);
const void *batch_kernel(const BatchPlan &P);
// resident workgroups per CU of the plan's kernel (the persistent grid size)
int batch_blocks_per_cu(const BatchPlan &P);
// source FOV validity mode of a launch: 0 none, 1 gathered mask, 2 sentinel
int score_vmode(const ScoreLaunch &L);

// Preparation of inputs.
// Bitmaps: dword y + ny (x / 32 + W z), bit 31 - x % 32.
// A mask source: prepared bytes and the bitmap of the nonzero voxels in the FOV.
hipError_t launch_mask_source(const uint8_t *vol, const uint8_t *fov, const int32_t n[3], uint8_t *out, uint32_t *bits,
                              hipStream_t s);
// A trilinear source's FOV: corner-validity bytes, bitmaps of the cells a valid
// sample may and must lie in.
hipError_t launch_corner_valid(const uint8_t *fov, const int32_t n[3], uint8_t *out, uint32_t *may, uint32_t *must,
                               hipStream_t s);
constexpr uint32_t kWorkSlots = 64, kWorkSlotWords = 16;
// Device bytes of the structures of the filter's mask launches (dice.hip).
struct DiceSizes {
    uint64_t bits, field, t4, t8, t16;
};
DiceSizes dice_sizes(const int32_t sn[3], const int32_t tn[3]);
// Distance field of a source from bitmaps of the voxels that may be on and that
// certainly are; gaps is scratch, a byte a voxel.
hipError_t launch_field(const uint32_t *may, const uint32_t *must, const int32_t n[3], uint8_t *gaps, uint8_t *field,
                        hipStream_t s);
hipError_t launch_dice_target(const uint8_t *vol, const uint8_t *fov, const int32_t n[3], uint8_t *prep, void *t4,
                              uint32_t *t8, uint32_t *t16, hipStream_t s);
hipError_t launch_dice(const ScoreLaunch &L, hipStream_t s);
hipError_t launch_dice_probe(const ScoreLaunch &L, uint32_t key, uint32_t *out, hipStream_t s);
// A batch's mask pairs: kernel arguments of a pair (its workgroups are
// returned), and one launch over the workgroups of all pairs (offs, prefix
// sums; pairs whose kmax is below k are done).
size_t dice_args_bytes();
uint64_t dice_args(const ScoreLaunch &L, void *out);
hipError_t launch_batch_dice(const void *pairs, const uint32_t *offs, const uint32_t *kmax, uint32_t n_pairs,
                             uint32_t groups, uint32_t k, hipStream_t s);
// The same for trilinear images with a source FOV (tri.hip); may, must
// (bits bytes each) are scratch.
struct TriSizes {
    uint64_t bits, field, tz, t4, t8, t16;
};
TriSizes tri_sizes(const int32_t sn[3], const int32_t tn[3]);
hipError_t launch_tri_target(const uint8_t *vol, const uint8_t *fov, const int32_t n[3], uint32_t *tz, uint32_t *fz,
                             void *t4, void *t8, void *t16, hipStream_t s);
bool tri_supported(const ScoreLaunch &L);
// out += voxels of a field without a valid sample within the reach of a target
// block of 8^3, and whether so many pay for the block launch of moments
// (spacings ts, ss in mm).
hipError_t launch_tri_off(const uint8_t *field, const int32_t sn[3], const double ts[3], const double ss[3],
                          unsigned long long *out, hipStream_t s);
bool tri_pays(uint64_t off, const int32_t sn[3]);
hipError_t launch_tri(const ScoreLaunch &L, hipStream_t s);
hipError_t launch_tri_probe(const ScoreLaunch &L, uint32_t key, uint32_t *out, hipStream_t s);
size_t tri_args_bytes();
uint64_t tri_args(const ScoreLaunch &L, void *out);
hipError_t launch_batch_tri(int layout, int vmode, const void *pairs, const uint32_t *offs, const uint32_t *kmax,
                            uint32_t n_pairs, uint32_t groups, uint32_t k, hipStream_t s);
// out[4 v + 0..3] += (fov count, nonzero count, sum, sum of squares) of volume v over its FOV
hipError_t launch_volume_sums(const uint8_t *const vol[2], const uint8_t *const fov[2], const int64_t n[2],
                              unsigned long long *out, hipStream_t s);

// Filter state of one registration pair.
struct FilterState {
    uint32_t n;               // particles
    uint32_t n_iters;         // K
    uint64_t seed;
    uint32_t pair;
    Geom geom;
    bool nearest;             // recipe words with the +0.5 shift
    ScoreConst sc;
    double x0[6], limit[6], lo[6], hi[6], sigma0[6], anneal;
    double *x;                // n x 6 current particles
    double *x_next;           // n x 6 scratch
    float *words;             // (n + 1) x 12, the last row is the ghost (estimate)
    unsigned long long *sums; // (n + 1) x 6
    double *lw;               // n log-weights of the last evaluation
    double *w;                // n scratch weights
    unsigned long long *cdf;  // n
    int32_t *anc;             // n
    double *est;              // 6 current estimate
    double *trace_score;      // K + 1
    double *trace_ess;        // K
    double *trace_est;        // 6 K
    // [0] degenerate weights seen, [1] at the latest iteration, [2] the current
    // particle set is a draw from the proposal (its first update adds lq)
    int32_t *flags;
    // learned proposal: the next prior draw comes from a Gaussian truncated to
    // the limits box; the draw records itself in flags[2], and the first update
    // of such a set adds log p - log q (p uniform)
    int32_t has_proposal;
    double prop_mu[6], prop_sigma[6];
    double *lq;               // n: -log q(x_i) + const of the proposal draw
    // wide rotations: quaternion-mean estimate; rotation axes with limit >= pi wrap
    int32_t wide;
};

hipError_t launch_init_particles(const FilterState &f, hipStream_t s);
// Batched filter: one workgroup per pair, states in device memory.
hipError_t launch_init_batch(const FilterState *states_dev, uint32_t n_pairs, uint32_t max_threads, hipStream_t s);
hipError_t launch_filter_batch(const FilterState *states_dev, uint32_t n_pairs, uint32_t k, hipStream_t s);
hipError_t launch_filter(const FilterState &f, uint32_t k, hipStream_t s);
hipError_t launch_ghost_final(const FilterState &f, hipStream_t s);
// Weighted mean (out[0..5]) and per-axis weighted variance (out[6..11]) of the
// particle set under the normalised weights of the last evaluation.
hipError_t launch_cloud_moments(const FilterState &f, double *out, hipStream_t s);
// recipe words of n device states; sums (or nullptr): 6 n words, cleared
hipError_t launch_words(const double *x, uint32_t n, const Geom &g, bool nearest, float *words,
                        unsigned long long *sums, hipStream_t s);
constexpr uint32_t kFewStates = 32;
hipError_t launch_words_few(const double *host, uint32_t n, const Geom &g, bool nearest, float *words,
                            unsigned long long *sums, hipStream_t s);
hipError_t launch_fill_u64(unsigned long long *p, uint64_t n, hipStream_t s);
// Mutual information: scores of particles p0 .. p0 + np - 1 from their joint
// histograms into their sums (overlap count, score bits), clearing the
// histograms for the next evaluation.
hipError_t launch_mi_finalize(uint32_t *hist, uint32_t p0, uint32_t np, unsigned long long *sums, hipStream_t s);
// Final scores of n particles from their sums.
hipError_t launch_scores_from_sums(const unsigned long long *sums, uint32_t n, const ScoreConst &sc, double *z,
                                   hipStream_t s);

// Learned proposal network (cnn.hip).
extern const int kCnnChannels[5];
extern const int kCnnSide;
extern const int kCnnFlat;
struct CnnBuffers {
    float *params;       // FP32 master weights (flat; layout in smc.h)
    float *grads, *adam_m, *adam_v;
    int64_t n_params;
    // bfloat16 copies of the convolution weights and tensors per layer, in the
    // orders that cnn.hip describes
    uint16_t *wf[4], *wd[4];    // weights of the forward and of the data gradient
    uint16_t *act[4];           // outputs after ReLU, channels first
    uint16_t *xs[4];            // inputs, split (training)
    uint16_t *dy[4];            // gradients of the pre-activations, channels first
    uint64_t *reach[4];         // offsets that the data gradient gathers by
    float *dout;                // B x 12
    float *wpart, *bpart;       // partial weight and bias gradients
};
// Elements of the buffers of a network of up to max_batch pairs.
struct CnnSizes {
    size_t wf[4], wd[4], act[4], xs[4], dy[4], reach[4], wpart, bpart;
};
CnnSizes cnn_sizes(int max_batch);
// Clear what stays zero, make the tables and pack the weights of params.
hipError_t cnn_prepare(const CnnBuffers &c, int max_batch, hipStream_t s);
int64_t cnn_param_offset(int part);
hipError_t cnn_downsample(const uint8_t *src, const int32_t sn[3], const uint8_t *tgt, const int32_t tn[3], float scale,
                          uint16_t *out, hipStream_t s);
// train: also keep what cnn_backward reads
hipError_t cnn_forward(const CnnBuffers &c, const uint16_t *input, int B, float *out, bool train, hipStream_t s);
hipError_t cnn_backward(const CnnBuffers &c, const uint16_t *input, int B, const float *out, const float *target,
                        float *loss_dev, hipStream_t s);
hipError_t cnn_adam(const CnnBuffers &c, float lr, int t, hipStream_t s);
hipError_t cnn_refresh_bf16(const CnnBuffers &c, hipStream_t s);

// Exhaustive search (exhaustive.hip).
hipError_t launch_grid_words(const double lo[6], const double step[6], const uint32_t count[6], uint64_t first,
                             uint32_t n, const Geom &g, bool nearest, double *x, float *words, hipStream_t s);
hipError_t launch_chunk_best(const unsigned long long *sums, uint32_t n, uint64_t first, const ScoreConst &sc,
                             double *scores, double *best_z, unsigned long long *best_i, hipStream_t s);

// warp_apply
hipError_t launch_warp_apply(const uint8_t *src, const int32_t sn[3], const float w[12], bool trilinear,
                             uint8_t *dst, const int32_t tn[3], uint32_t frames, int64_t src_stride,
                             int64_t dst_stride, hipStream_t s);

}  // namespace smc
