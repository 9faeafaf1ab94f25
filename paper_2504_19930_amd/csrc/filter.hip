// Particle-filter kernels (Fig. 1): prior draw, and the per-iteration update
// -> normalise / estimate -> systematic resampling -> prediction.
//
// Up to 512 particles one workgroup does all of it, a thread per particle, the
// workgroup no larger than the set (256 or 512 threads).  Larger sets take
// two launches: a workgroup of 1024 threads forms the weights, the estimate and
// the CDF, and one thread per particle, over the chip, resamples and predicts
// (the random walk's Philox draws and FP64 logarithms and sines kept one CU busy
// for most of the launch: 88 us for 4096 particles, 40.7 + 15.5 so; 22.7 us for
// 256, 16.5 with a workgroup of 256; 29 us for 512, 21.7 with one of 512).  A
// batch keeps one workgroup per pair; its pairs fill the chip.
//
// Determinism: log-weights come from exact integer sums; the resampling CDF
// is an exact 64-bit integer prefix sum of q_i = floor(w_i 2^48) and every
// pointer comparison is an exact 128-bit product, so the ancestors do not
// depend on reduction order.  Only the estimate and the ESS use FP64 tree
// sums, in one order whatever the workgroup (absent threads add zeros).
#include <string.h>

#include "internal.h"

namespace smc {
namespace {

constexpr int kFT = 1024;  // largest filter workgroup
constexpr int kFW = kFT / 64;
// Particles whose resampling CDF a workgroup keeps in LDS (32 KB); larger sets
// search the CDF in global memory.
constexpr uint32_t kCdfLds = 4096;

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
    for (int o = 32; o > 0; o >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, o));
    return v;
}

__device__ __forceinline__ double wave_add(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__global__ __launch_bounds__(256) void k_fill_u64(unsigned long long *p, uint64_t n) {
    for (uint64_t q = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; q < n; q += (uint64_t)gridDim.x * blockDim.x)
        p[q] = 0ull;
}

// Recipe words of n states; sums (or nullptr): the six of each, cleared.
__device__ __forceinline__ void words_of(const double *p, uint32_t i, const Geom &g, bool nearest, float *words,
                                         unsigned long long *sums) {
    particle_words(p, g, nearest, words + 12 * (size_t)i);
    if (sums)
        for (int d = 0; d < 6; ++d) sums[6 * (size_t)i + d] = 0ull;
}

__global__ __launch_bounds__(256) void k_words(const double *x, uint32_t n, Geom g, bool nearest, float *words,
                                               unsigned long long *sums) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double p[6];
    for (int d = 0; d < 6; ++d) p[d] = x[6 * (size_t)i + d];
    words_of(p, i, g, nearest, words, sums);
}

// The same for a few states on the host, which travel as the kernel's argument
// instead of by a copy of their own (with the sums cleared here and not by a
// launch of their own, 41 -> 36 us for 4 states on 64^3 masks).
struct FewStates {
    double x[6 * kFewStates];
};
__global__ __launch_bounds__(64) void k_words_few(const FewStates s, uint32_t n, Geom g, bool nearest, float *words,
                                                  unsigned long long *sums) {
    const uint32_t i = threadIdx.x;
    if (i >= n) return;
    double p[6];
    for (int d = 0; d < 6; ++d) p[d] = s.x[6 * i + d];
    words_of(p, i, g, nearest, words, sums);
}

// Prior: x_i = x0 + L (2u - 1), u from Philox (tag 0, three blocks).
constexpr uint32_t kProposalTries = 16;

// Six standard normals of try t for particle i from the proposal stream.
__device__ __forceinline__ void proposal_normals(const FilterState &f, uint32_t i, uint32_t t, double g[6]) {
    for (uint32_t b = 0; b < 3; ++b) {
        uint32_t r[4];
        draw4(f.seed, i, t, f.pair, kTagProposal, b, r);
        const double u1 = uniform53(r[0], r[1]), u2 = uniform53(r[2], r[3]);
        const double rad = sqrt(-2.0 * log(u1));
        const double th = 6.283185307179586 * u2;
        g[2 * b] = rad * cos(th);
        g[2 * b + 1] = rad * sin(th);
    }
}

__device__ __forceinline__ void init_body(const FilterState &f, uint32_t i, uint32_t stride) {
    if (i < f.n) {
        double p[6];
        if (f.has_proposal) {
            // per-axis rejection into the box (a product region), clamp after 16 tries
            bool done[6] = {false, false, false, false, false, false};
            for (int d = 0; d < 6; ++d) p[d] = fmin(fmax(f.prop_mu[d], f.lo[d]), f.hi[d]);
            for (uint32_t t = 0; t < kProposalTries; ++t) {
                double g[6];
                proposal_normals(f, i, t, g);
                for (int d = 0; d < 6; ++d) {
                    const double v = f.prop_mu[d] + f.prop_sigma[d] * g[d];
                    if (!done[d] && v >= f.lo[d] && v <= f.hi[d]) {
                        p[d] = v;
                        done[d] = true;
                    }
                }
            }
            double lq = 0.0;
            for (int d = 0; d < 6; ++d) {
                const double z = (p[d] - f.prop_mu[d]) / f.prop_sigma[d];
                lq += 0.5 * (z * z);
            }
            f.lq[i] = lq;
        } else {
            for (uint32_t b = 0; b < 3; ++b) {
                uint32_t r[4];
                draw4(f.seed, i, 0u, f.pair, kTagInit, b, r);
                const double ua = uniform53(r[0], r[1]), ub = uniform53(r[2], r[3]);
                const int d0 = 2 * b, d1 = 2 * b + 1;
                p[d0] = f.x0[d0] + f.limit[d0] * (2.0 * ua - 1.0);
                p[d1] = f.x0[d1] + f.limit[d1] * (2.0 * ub - 1.0);
            }
        }
        for (int d = 0; d < 6; ++d) f.x[6 * (size_t)i + d] = p[d];
        particle_words(p, f.geom, f.nearest, f.words + 12 * (size_t)i);
        f.lw[i] = 0.0;
        f.anc[i] = -1;
    }
    if (i == 0) {
        for (int d = 0; d < 6; ++d) f.est[d] = f.x0[d];
        particle_words(f.x0, f.geom, f.nearest, f.words + 12 * (size_t)f.n);
        f.flags[0] = 0;
        f.flags[1] = 0;
        f.flags[2] = f.has_proposal ? 1 : 0;
    }
    for (uint64_t q = i; q < 6ull * (f.n + 1ull); q += stride) f.sums[q] = 0ull;
    const uint32_t nt = f.n_iters + 1;
    for (uint32_t q = i; q < nt; q += stride) {
        f.trace_score[q] = __builtin_nan("");
        if (q < f.n_iters) {
            f.trace_ess[q] = __builtin_nan("");
            for (int d = 0; d < 6; ++d) f.trace_est[6 * q + d] = __builtin_nan("");
        }
    }
}

__global__ __launch_bounds__(256) void k_init(const FilterState f) {
    init_body(f, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

__global__ __launch_bounds__(256) void k_init_batch(const FilterState *fs) {
    const FilterState &f = fs[blockIdx.y];
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    init_body(f, i, gridDim.x * blockDim.x);
}

__device__ __forceinline__ bool pointer_passed(unsigned long long c, unsigned __int128 scale,
                                               unsigned __int128 rhs) {
    return (unsigned __int128)c * scale > rhs;
}

__device__ __forceinline__ unsigned long long wave_scan(unsigned long long v) {
    const int lane = threadIdx.x % 64;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long u = __shfl_up(v, o);
        v += lane >= o ? u : 0ull;
    }
    return v;
}

// The random walk of particle j: its ancestor's state (the first CDF entry past
// the systematic pointer) in `from` moved and reflected, written to out.
__device__ __forceinline__ void predict_one(const FilterState &f, const double *from, const uint32_t k,
                                            const uint32_t j, const unsigned long long *cdf, const unsigned long long Q,
                                            const uint32_t offset, const double sg[6], double out[6]) {
    const uint32_t n = f.n;
    const unsigned __int128 scale = (unsigned __int128)n << 32;
    const unsigned __int128 rhs = ((((unsigned __int128)j) << 32) + offset) * (unsigned __int128)Q;
    uint32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (pointer_passed(cdf[mid], scale, rhs)) hi = mid;
        else lo = mid + 1;
    }
    f.anc[j] = (int32_t)lo;
    // prediction: reflected annealed Gaussian random walk (Box-Muller)
    double g[6];
    for (uint32_t b = 0; b < 3; ++b) {
        uint32_t r[4];
        draw4(f.seed, j, k, f.pair, kTagPerturb, b, r);
        const double u1 = uniform53(r[0], r[1]), u2 = uniform53(r[2], r[3]);
        const double rad = sqrt(-2.0 * log(u1));
        const double th = 6.283185307179586 * u2;
        g[2 * b] = rad * cos(th);
        g[2 * b + 1] = rad * sin(th);
    }
    for (int d = 0; d < 6; ++d) {
        const double v = from[6 * (size_t)lo + d] + sg[d] * g[d];
        // wide rotations: an axis whose limit covers the circle wraps
        out[d] = f.wide && d < 3 && f.limit[d] >= 3.141592653589793 ? wrap_near(v, f.x0[d])
                                                                     : reflect_into(v, f.lo[d], f.hi[d]);
    }
}

// Random-walk widths of iteration k.
__device__ __forceinline__ void walk_widths(const FilterState &f, const uint32_t k, double sg[6]) {
    for (int d = 0; d < 6; ++d) {
        double v = f.sigma0[d];
        for (uint32_t m = 1; m < k; ++m) v = v * f.anneal;
        sg[d] = v;
    }
}

// Update, normalise, estimate and CDF by one workgroup of FT threads.  The CDF
// (cdf: LDS or global) is made for k < n_iters; Q, its total, is returned to
// every thread.  SNAPSHOT: the states are copied to f.x_next as they are read.
template <int FT, bool SNAPSHOT = false>
__device__ __forceinline__ unsigned long long weigh(const FilterState &f, const uint32_t k, unsigned long long *cdf) {
    constexpr int FW = FT / 64;
    __shared__ double red[FW][12];
    __shared__ double bcast[12];
    __shared__ uint32_t ref_idx[FW];
    __shared__ unsigned long long wtot[FW];
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
    const uint32_t n = f.n;

    // update: log-weights of the scores, and their maximum; a set drawn from
    // the proposal carries the importance correction in its first update
    const bool from_proposal = f.flags[2] != 0;
    double mx = -INFINITY;
    for (uint32_t i = tid; i < n; i += FT) {
        int64_t m[6];
        for (int q = 0; q < 6; ++q) m[q] = (int64_t)f.sums[6 * (size_t)i + q];
        double l = log_likelihood(score_from_sums(m, f.sc), f.sc);
        if (k == 1 && from_proposal) l = l + f.lq[i];
        f.lw[i] = l;
        mx = fmax(mx, l);
    }
    if (tid == FT - 1) {  // (the last thread: it has the fewest particles)
        int64_t m[6];
        for (int q = 0; q < 6; ++q) m[q] = (int64_t)f.sums[6 * (size_t)n + q];
        f.trace_score[k - 1] = score_from_sums(m, f.sc);
    }
    mx = wave_max(mx);
    if (lane == 0) red[wave][0] = mx;
    __syncthreads();
    double M = red[0][0];
    for (int w = 1; w < FW; ++w) M = fmax(M, red[w][0]);
    const bool degenerate = M == -INFINITY;

    // wide rotations: the reference hemisphere is that of the first particle
    // of largest log-weight (all of them when every weight is -inf)
    double qref[4] = {1.0, 0.0, 0.0, 0.0};
    if (f.wide) {
        uint32_t first = n;
        for (uint32_t i = tid; i < n; i += FT)
            if (f.lw[i] == M) {
                first = i;
                break;
            }
        first = wave_min_u32(first);
        if (lane == 0) ref_idx[wave] = first;
        __syncthreads();
        uint32_t r = ref_idx[0];
        for (int w = 1; w < FW; ++w) r = min(r, ref_idx[w]);
        rotation_quaternion(f.x + 6 * (size_t)(r < n ? r : 0u), qref);
    }

    // normalise and estimate: w_i = exp(lw_i - M), weighted mean, ESS, and
    // for wide rotations the weighted sum of hemisphere-aligned quaternions
    double s = 0.0, s2 = 0.0, sx[6] = {0, 0, 0, 0, 0, 0}, sq[4] = {0, 0, 0, 0};
    for (uint32_t i = tid; i < n; i += FT) {
        const double w = degenerate ? 1.0 : exp(f.lw[i] - M);
        f.w[i] = w;
        s += w;
        s2 += w * w;
        for (int d = 0; d < 6; ++d) {
            const double v = f.x[6 * (size_t)i + d];
            sx[d] += w * v;
            if (SNAPSHOT) f.x_next[6 * (size_t)i + d] = v;
        }
        if (f.wide) {
            double q[4];
            rotation_quaternion(f.x + 6 * (size_t)i, q);
            const double dot = q[0] * qref[0] + q[1] * qref[1] + q[2] * qref[2] + q[3] * qref[3];
            const double ws = dot < 0.0 ? -w : w;
            for (int c = 0; c < 4; ++c) sq[c] += ws * q[c];
        }
    }
    s = wave_add(s);
    s2 = wave_add(s2);
    for (int d = 0; d < 6; ++d) sx[d] = wave_add(sx[d]);
    if (f.wide)
        for (int c = 0; c < 4; ++c) sq[c] = wave_add(sq[c]);
    __syncthreads();
    if (lane == 0) {
        red[wave][0] = s;
        red[wave][1] = s2;
        for (int d = 0; d < 6; ++d) red[wave][2 + d] = sx[d];
        for (int c = 0; c < 4; ++c) red[wave][8 + c] = sq[c];
    }
    __syncthreads();
    if (tid < 12) {
        double v = 0.0;
        for (int w = 0; w < FW; ++w) v += red[w][tid];
        bcast[tid] = v;
    }

    // exact integer CDF: contiguous chunk per thread, block scan of chunk sums
    unsigned long long Q = 0ull;
    if (k < f.n_iters) {
        const uint32_t per = (n + FT - 1) / FT;
        const uint32_t b0 = min(n, tid * per), b1 = min(n, b0 + per);
        unsigned long long local = 0;
        for (uint32_t i = b0; i < b1; ++i) local += (unsigned long long)floor(f.w[i] * 0x1p48);
        const unsigned long long incl = wave_scan(local);
        if (lane == 63) wtot[wave] = incl;
        __syncthreads();
        unsigned long long run = incl - local;
        for (int w = 0; w < FW; ++w) {
            run += w < wave ? wtot[w] : 0ull;
            Q += wtot[w];
        }
        for (uint32_t i = b0; i < b1; ++i) {
            run += (unsigned long long)floor(f.w[i] * 0x1p48);
            cdf[i] = run;
        }
    }
    __syncthreads();
    // the estimate, by a wave whose threads end with the others
    if (tid == FT - 64) {
        double est[6];
        for (int d = 0; d < 6; ++d) est[d] = bcast[2 + d] / bcast[0];
        if (f.wide) {
            const double nq = sqrt(bcast[8] * bcast[8] + bcast[9] * bcast[9] + bcast[10] * bcast[10] +
                                   bcast[11] * bcast[11]);
            const double q[4] = {bcast[8] / nq, bcast[9] / nq, bcast[10] / nq, bcast[11] / nq};
            double e[3];
            quaternion_euler(q, e);
            for (int d = 0; d < 3; ++d) est[d] = wrap_near(e[d], f.x0[d]);
        }
        for (int d = 0; d < 6; ++d) {
            f.est[d] = est[d];
            f.trace_est[6 * (size_t)(k - 1) + d] = est[d];
        }
        f.trace_ess[k - 1] = (bcast[0] * bcast[0]) / bcast[1];
        if (degenerate) f.flags[0] = 1;
        f.flags[1] = degenerate ? 1 : 0;  // the latest iteration's weights were all -inf
        particle_words(est, f.geom, f.nearest, f.words + 12 * (size_t)n);
    }
    return Q;
}

// A whole iteration by one workgroup.
template <int FT>
__device__ __forceinline__ void filter_body(const FilterState &f, const uint32_t k) {
    __shared__ unsigned long long cdf_lds[FT < kFT ? FT : (int)kCdfLds];
    const uint32_t n = f.n, tid = threadIdx.x;
    // the binary searches read this CDF: each is a chain of dependent loads,
    // far shorter from LDS than from L2
    unsigned long long *const cdf = n <= sizeof cdf_lds / sizeof cdf_lds[0] ? cdf_lds : f.cdf;
    const unsigned long long Q = weigh<FT>(f, k, cdf);
    if (k < f.n_iters) {
        uint32_t rw[4];
        draw4(f.seed, 0u, k, f.pair, kTagResample, 0u, rw);
        double sg[6];
        walk_widths(f, k, sg);
        if (n <= FT) {
            // a thread per particle: the new states stay in registers until
            // every ancestor has been read
            double p[6];
            if (tid < n) predict_one(f, f.x, k, tid, cdf, Q, rw[0], sg, p);
            __syncthreads();
            if (tid < n) {
                for (int d = 0; d < 6; ++d) f.x[6 * (size_t)tid + d] = p[d];
                particle_words(p, f.geom, f.nearest, f.words + 12 * (size_t)tid);
            }
        } else {
            for (uint32_t j = tid; j < n; j += FT) {
                double p[6];
                predict_one(f, f.x, k, j, cdf, Q, rw[0], sg, p);
                for (int d = 0; d < 6; ++d) f.x_next[6 * (size_t)j + d] = p[d];
            }
            __syncthreads();
            for (uint32_t j = tid; j < n; j += FT) {
                double p[6];
                for (int d = 0; d < 6; ++d) {
                    p[d] = f.x_next[6 * (size_t)j + d];
                    f.x[6 * (size_t)j + d] = p[d];
                }
                particle_words(p, f.geom, f.nearest, f.words + 12 * (size_t)j);
            }
        }
    }
    // clear the sums for the next evaluation
    for (uint32_t q = tid; q < 6 * (n + 1); q += FT) f.sums[q] = 0ull;
}

template <int FT>
__global__ __launch_bounds__(FT) void k_filter(const FilterState f, const uint32_t k) {
    filter_body<FT>(f, k);
}

__global__ __launch_bounds__(kFT) void k_filter_batch(const FilterState *fs, const uint32_t k) {
    const FilterState &f = fs[blockIdx.x];
    if (k <= f.n_iters) filter_body<kFT>(f, k);
}

// Larger sets: the weights, the CDF (in f.cdf) and a copy of the states in
// f.x_next, then resampling and prediction, a thread per particle, from the
// copy into f.x.  In the last iteration the second launch only clears the sums.
__global__ __launch_bounds__(kFT) void k_weigh(const FilterState f, const uint32_t k) { weigh<kFT, true>(f, k, f.cdf); }

__global__ __launch_bounds__(256) void k_predict(const FilterState f, const uint32_t k) {
    __shared__ unsigned long long cdf_lds[kCdfLds];
    const uint32_t n = f.n, j = blockIdx.x * 256u + threadIdx.x;
    if (k < f.n_iters) {
        if (n <= kCdfLds) {
            for (uint32_t i = threadIdx.x; i < n; i += 256u) cdf_lds[i] = f.cdf[i];
            __syncthreads();
        }
        uint32_t rw[4];
        draw4(f.seed, 0u, k, f.pair, kTagResample, 0u, rw);
        double sg[6];
        walk_widths(f, k, sg);
        if (j < n) {
            double p[6];
            predict_one(f, f.x_next, k, j, n <= kCdfLds ? cdf_lds : f.cdf, f.cdf[n - 1], rw[0], sg, p);
            for (int d = 0; d < 6; ++d) f.x[6 * (size_t)j + d] = p[d];
            particle_words(p, f.geom, f.nearest, f.words + 12 * (size_t)j);
        }
    }
    for (uint32_t q = j; q < 6 * (n + 1); q += gridDim.x * 256u) f.sums[q] = 0ull;
}

// Weighted mean and per-axis weighted variance of the particle set under the
// normalised weights exp(lw_i - max lw) of the last evaluation (uniform when
// every log-weight is -inf): out[0..5] the mean, out[6..11] the variance,
// in the filter's units.  One workgroup; FP64 tree sums.
__global__ __launch_bounds__(kFT) void k_cloud_moments(const FilterState f, double *out) {
    __shared__ double red[kFW][7];
    __shared__ double bc[7];
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
    const uint32_t n = f.n;
    double mx = -INFINITY;
    for (uint32_t i = tid; i < n; i += kFT) mx = fmax(mx, f.lw[i]);
    mx = wave_max(mx);
    if (lane == 0) red[wave][0] = mx;
    __syncthreads();
    if (tid == 0) {
        double v = red[0][0];
        for (int w = 1; w < kFW; ++w) v = fmax(v, red[w][0]);
        bc[0] = v;
    }
    __syncthreads();
    const double M = bc[0];
    const bool flat = M == -INFINITY;
    // pass 1: total weight and weighted sums of the states
    double acc[7] = {0, 0, 0, 0, 0, 0, 0};
    for (uint32_t i = tid; i < n; i += kFT) {
        const double w = flat ? 1.0 : exp(f.lw[i] - M);
        acc[0] += w;
        for (int d = 0; d < 6; ++d) acc[1 + d] += w * f.x[6 * (size_t)i + d];
    }
    for (int q = 0; q < 7; ++q) acc[q] = wave_add(acc[q]);
    __syncthreads();
    if (lane == 0)
        for (int q = 0; q < 7; ++q) red[wave][q] = acc[q];
    __syncthreads();
    if (tid < 7) {
        double v = 0.0;
        for (int w = 0; w < kFW; ++w) v += red[w][tid];
        bc[tid] = v;
    }
    __syncthreads();
    const double total = bc[0];
    double mean[6];
    for (int d = 0; d < 6; ++d) mean[d] = bc[1 + d] / total;
    // pass 2: weighted squared deviations from the mean
    double dv[6] = {0, 0, 0, 0, 0, 0};
    for (uint32_t i = tid; i < n; i += kFT) {
        const double w = flat ? 1.0 : exp(f.lw[i] - M);
        for (int d = 0; d < 6; ++d) {
            const double e = f.x[6 * (size_t)i + d] - mean[d];
            dv[d] += w * (e * e);
        }
    }
    for (int d = 0; d < 6; ++d) dv[d] = wave_add(dv[d]);
    __syncthreads();
    if (lane == 0)
        for (int d = 0; d < 6; ++d) red[wave][d] = dv[d];
    __syncthreads();
    if (tid < 6) {
        double v = 0.0;
        for (int w = 0; w < kFW; ++w) v += red[w][tid];
        out[tid] = mean[tid];
        out[6 + tid] = v / total;
    }
}

__global__ void k_ghost_final(const FilterState f) {
    int64_t m[6];
    for (int q = 0; q < 6; ++q) m[q] = (int64_t)f.sums[6 * (size_t)f.n + q];
    f.trace_score[f.n_iters] = score_from_sums(m, f.sc);
    for (int q = 0; q < 6; ++q) f.sums[6 * (size_t)f.n + q] = 0ull;
}

// One workgroup per particle: the histogram and its marginals (exact integer
// counts) in LDS, the entropies' terms f ln f a thread each, and their sums in
// bin order by one lane of three waves (an FP64 sum's bits depend on the order,
// and the score is the same on every platform); 2 I / (H_s + H_t).  Terms of
// empty bins are zero and change no sum.  One lane taking the 1024 logarithms as
// well took 215 us for 513 particles.
__global__ __launch_bounds__(256) void k_mi_finalize(uint32_t *hist, uint32_t p0, unsigned long long *sums) {
    constexpr int kHB = kMiBins * kMiBins;
    __shared__ double term[kHB], mterm[2 * kMiBins], ent[3];
    __shared__ unsigned long long marg[2 * kMiBins], wtot[4];  // (frames pool: totals beyond 32 bits)
    const uint32_t i = p0 + blockIdx.x;
    uint32_t *hp = hist + (size_t)kHB * i;
    const int tid = threadIdx.x;
    if (tid < 2 * kMiBins) marg[tid] = 0ull;
    // four consecutive bins a thread: one source row, four target columns
    const uint4 v4 = *(const uint4 *)(hp + 4 * tid);
    *(uint4 *)(hp + 4 * tid) = make_uint4(0u, 0u, 0u, 0u);  // ready for the next evaluation
    const uint32_t v[4] = {v4.x, v4.y, v4.z, v4.w};
    const unsigned long long row = (unsigned long long)v[0] + v[1] + v[2] + v[3];
    unsigned long long mine = row;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o);
    if (tid % 64 == 0) wtot[tid / 64] = mine;
    __syncthreads();
    if (row) atomicAdd(&marg[tid / 8], row);
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (v[e]) atomicAdd(&marg[kMiBins + 4 * (tid % 8) + e], (unsigned long long)v[e]);
    const unsigned long long n = wtot[0] + wtot[1] + wtot[2] + wtot[3];
    const double N = (double)n;
    const auto entropy_term = [&](unsigned long long c) {
        if (c == 0ull) return 0.0;
        const double f = (double)c / N;
        return f * mi_log(f);
    };
#pragma unroll
    for (int e = 0; e < 4; ++e) term[4 * tid + e] = entropy_term(v[e]);
    __syncthreads();
    if (tid < 2 * kMiBins) mterm[tid] = entropy_term(marg[tid]);
    __syncthreads();
    if (tid % 64 == 0 && tid < 192) {
        // wave 0: the joint entropy; 1 and 2: the marginals'
        const double *t = tid == 0 ? term : mterm + (tid / 64 - 1) * kMiBins;
        const int count = tid == 0 ? kHB : kMiBins;
        double h = 0.0;
        for (int q = 0; q < count; q += 8) {
            double x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = t[q + e];
#pragma unroll
            for (int e = 0; e < 8; ++e) h = h - x[e];
        }
        ent[tid / 64] = h;
    }
    __syncthreads();
    if (tid != 0) return;
    double z = 0.0;
    if (n && ent[1] + ent[2] > 0.0) z = 2.0 * (ent[1] + ent[2] - ent[0]) / (ent[1] + ent[2]);
    unsigned long long bits;
    memcpy(&bits, &z, sizeof bits);
    unsigned long long *o = sums + 6 * (size_t)i;
    o[0] = n;
    o[1] = bits;
    o[2] = o[3] = o[4] = o[5] = 0ull;
}

__global__ __launch_bounds__(256) void k_scores_from_sums(const unsigned long long *sums, uint32_t n,
                                                          const ScoreConst sc, double *z) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int64_t m[6];
    for (int q = 0; q < 6; ++q) m[q] = (int64_t)sums[6 * (size_t)i + q];
    z[i] = score_from_sums(m, sc);
}

}  // namespace

hipError_t launch_mi_finalize(uint32_t *hist, uint32_t p0, uint32_t np, unsigned long long *sums, hipStream_t s) {
    if (np == 0) return hipSuccess;
    hipLaunchKernelGGL(k_mi_finalize, dim3(np), dim3(256), 0, s, hist, p0, sums);
    return hipGetLastError();
}

hipError_t launch_scores_from_sums(const unsigned long long *sums, uint32_t n, const ScoreConst &sc, double *z,
                                   hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_scores_from_sums, dim3((n + 255) / 256), dim3(256), 0, s, sums, n, sc, z);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long *p, uint64_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    uint64_t b = (n + 255) / 256;
    hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)(b < 2048 ? b : 2048)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_words(const double *x, uint32_t n, const Geom &g, bool nearest, float *words,
                        unsigned long long *sums, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_words, dim3((n + 255) / 256), dim3(256), 0, s, x, n, g, nearest, words, sums);
    return hipGetLastError();
}

hipError_t launch_words_few(const double *host, uint32_t n, const Geom &g, bool nearest, float *words,
                            unsigned long long *sums, hipStream_t s) {
    if (n == 0) return hipSuccess;
    if (n > kFewStates) return hipErrorInvalidValue;
    FewStates few = {};
    memcpy(few.x, host, 48ull * n);
    hipLaunchKernelGGL(k_words_few, dim3(1), dim3(64), 0, s, few, n, g, nearest, words, sums);
    return hipGetLastError();
}

hipError_t launch_init_particles(const FilterState &f, hipStream_t s) {
    const uint32_t n = f.n > f.n_iters + 1 ? f.n : f.n_iters + 1;
    hipLaunchKernelGGL(k_init, dim3((n + 255) / 256), dim3(256), 0, s, f);
    return hipGetLastError();
}

hipError_t launch_filter(const FilterState &f, uint32_t k, hipStream_t s) {
    if (f.n <= 256) {
        hipLaunchKernelGGL(k_filter<256>, dim3(1), dim3(256), 0, s, f, k);
    } else if (f.n <= 512) {
        hipLaunchKernelGGL(k_filter<512>, dim3(1), dim3(512), 0, s, f, k);
    } else {
        // two launches cost less from here on, gap included: 513 particles 26.4 us
        // (one workgroup of 1024 threads: 29.1), 1024 particles 31.2 us (36.8)
        hipLaunchKernelGGL(k_weigh, dim3(1), dim3(kFT), 0, s, f, k);
        hipLaunchKernelGGL(k_predict, dim3((f.n + 255) / 256), dim3(256), 0, s, f, k);
    }
    return hipGetLastError();
}

hipError_t launch_init_batch(const FilterState *fs, uint32_t n_pairs, uint32_t max_threads, hipStream_t s) {
    hipLaunchKernelGGL(k_init_batch, dim3((max_threads + 255) / 256, n_pairs), dim3(256), 0, s, fs);
    return hipGetLastError();
}

hipError_t launch_filter_batch(const FilterState *fs, uint32_t n_pairs, uint32_t k, hipStream_t s) {
    hipLaunchKernelGGL(k_filter_batch, dim3(n_pairs), dim3(kFT), 0, s, fs, k);
    return hipGetLastError();
}

hipError_t launch_cloud_moments(const FilterState &f, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_cloud_moments, dim3(1), dim3(kFT), 0, s, f, out);
    return hipGetLastError();
}

hipError_t launch_ghost_final(const FilterState &f, hipStream_t s) {
    hipLaunchKernelGGL(k_ghost_final, dim3(1), dim3(1), 0, s, f);
    return hipGetLastError();
}

}  // namespace smc
