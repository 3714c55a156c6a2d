// Map growth and scale regularisation of GS^3LAM (Sec. 3.3.1-3.3.2):
//
//   adaptive expansion: every pixel with M_unobs (mask bit 1, from the SLAM
//   loss) and an observed depth D* > 0 adds one Gaussian at the unprojection
//   of its centre at D*, with the pixel's observed colour, caller-drawn
//   random features, opacity 0.5, scale D*/fx and the identity rotation.
//   New Gaussians are appended in pixel order (views back to back, rows,
//   columns) after the current count, which lives on the device: a count
//   kernel per block of pixels, one block that scans the counts and updates
//   the device-side Gaussian count, then a write kernel that ranks its
//   block's candidates with a block scan.  No host round trip.
//
//   depth-adaptive scale regularisation (Eq. 12): over the 3n per-axis
//   scales s = exp(log s) (the decision-path exponential, bit-identical to
//   any implementation of the same operation sequence), their mean and
//   population standard deviation, the sets s > mu + 2 sigma and
//   s < mu - 2 sigma, L_big = mean of s over the first, L_small = mean of
//   -log s over the second, and the gradient with respect to log s with the
//   sets held.  Every sum is per block in double, then in a fixed order.
#include "growth.h"
#include "decision_exp.h"

namespace sgs {

namespace {

constexpr int kGrowThreads = 256;
constexpr int kExpandItems = 4;  // pixels per thread
constexpr int kExpandChunk = kGrowThreads * kExpandItems;

__device__ __forceinline__ bool expand_candidate(const uint8_t* masks, const float* depth_t, int64_t p) {
    return ((masks[p] >> 1) & 1) && depth_t[p] > 0.0f;
}

__global__ void __launch_bounds__(kGrowThreads) k_expand_count(const uint8_t* __restrict__ masks,
                                                               const float* __restrict__ depth_t, int64_t P,
                                                               uint32_t* __restrict__ block_counts) {
    __shared__ uint32_t s_tmp[kGrowThreads / kWave];
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < kExpandItems; ++k) {
        const int64_t p = (int64_t)blockIdx.x * kExpandChunk + k * kGrowThreads + threadIdx.x;
        if (p < P && expand_candidate(masks, depth_t, p)) ++c;
    }
    uint32_t total;
    block_exclusive<kGrowThreads>(c, s_tmp, &total);
    if (threadIdx.x == 0) block_counts[blockIdx.x] = total;
}

// One block: exclusive scan of the block counts in place, the number of
// candidates, and the Gaussian count n <- min(n + candidates, capacity)
// (n_before keeps the old count for the write kernel).
__global__ void __launch_bounds__(1024) k_expand_scan(uint32_t* __restrict__ block_counts, int nblk,
                                                      int64_t* __restrict__ n_dev, int64_t capacity,
                                                      int64_t* __restrict__ n_before,
                                                      int64_t* __restrict__ candidates) {
    __shared__ uint32_t s_tmp[1024 / kWave];
    const int per = (nblk + 1023) / 1024;
    const int b0 = threadIdx.x * per, b1 = min(b0 + per, nblk);
    uint32_t sum = 0;
    for (int b = b0; b < b1; ++b) sum += block_counts[b];
    uint32_t total;
    uint32_t run = block_exclusive<1024>(sum, s_tmp, &total);
    for (int b = b0; b < b1; ++b) {
        const uint32_t v = block_counts[b];
        block_counts[b] = run;
        run += v;
    }
    if (threadIdx.x == 0) {
        const int64_t n = *n_dev;
        *n_before = n;
        if (candidates != nullptr) *candidates = (int64_t)total;
        const int64_t m = n + (int64_t)total;
        *n_dev = m < capacity ? m : capacity;
    }
}

template <int F>
__global__ void __launch_bounds__(kGrowThreads) k_expand_write(const uint8_t* __restrict__ masks,
                                                               const float* __restrict__ rgb_t,
                                                               const float* __restrict__ depth_t,
                                                               const float* __restrict__ feat_init, int64_t P,
                                                               const gs_view* __restrict__ views, int n_views,
                                                               const uint32_t* __restrict__ block_offsets,
                                                               const int64_t* __restrict__ n_before, int64_t capacity,
                                                               gs_gaussian_grads g) {
    __shared__ uint32_t s_tmp[kGrowThreads / kWave];
    bool cand[kExpandItems];
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < kExpandItems; ++k) {
        const int64_t p = (int64_t)blockIdx.x * kExpandChunk + k * kGrowThreads + threadIdx.x;
        cand[k] = p < P && expand_candidate(masks, depth_t, p);
        c += cand[k] ? 1u : 0u;
    }
    // the block's candidates in pixel order: item k of thread t is pixel
    // k * 256 + t of the chunk, so rank item-major: first all k = 0, ...
    uint32_t rank0[kExpandItems];
    uint32_t base = 0;
#pragma unroll
    for (int k = 0; k < kExpandItems; ++k) {
        uint32_t tot;
        rank0[k] = base + block_exclusive<kGrowThreads>(cand[k] ? 1u : 0u, s_tmp, &tot);
        base += tot;
    }
    const int64_t first = *n_before + (int64_t)block_offsets[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kExpandItems; ++k) {
        if (!cand[k]) continue;
        const int64_t i = first + rank0[k];
        if (i >= capacity) continue;
        const int64_t p = (int64_t)blockIdx.x * kExpandChunk + k * kGrowThreads + threadIdx.x;
        int v = 0;
        while (v + 1 < n_views && views[v + 1].pixel_offset <= p) ++v;
        const gs_view& vw = views[v];
        const int64_t q = p - vw.pixel_offset;
        const int y = (int)(q / vw.width), x = (int)(q - (int64_t)y * vw.width);
        const float d = depth_t[p];
        const float xc0 = ((float)x + 0.5f - vw.cx) / vw.fx * d, xc1 = ((float)y + 0.5f - vw.cy) / vw.fy * d;
        const float r0 = xc0 - vw.Rt[3], r1 = xc1 - vw.Rt[7], r2 = d - vw.Rt[11];
        // mu = R^T (x_c - t)
        g.mu[i] = vw.Rt[0] * r0 + vw.Rt[4] * r1 + vw.Rt[8] * r2;
        g.mu[capacity + i] = vw.Rt[1] * r0 + vw.Rt[5] * r1 + vw.Rt[9] * r2;
        g.mu[2 * capacity + i] = vw.Rt[2] * r0 + vw.Rt[6] * r1 + vw.Rt[10] * r2;
        const float lsv = logf(d / vw.fx);
        g.log_scale[i] = lsv;
        g.log_scale[capacity + i] = lsv;
        g.log_scale[2 * capacity + i] = lsv;
        g.quat[i] = 1.0f;
        g.quat[capacity + i] = 0.0f;
        g.quat[2 * capacity + i] = 0.0f;
        g.quat[3 * capacity + i] = 0.0f;
        g.opacity_logit[i] = 0.0f;  // opacity 0.5
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) g.color[ch * capacity + i] = rgb_t[ch * P + p];
#pragma unroll
        for (int f = 0; f < F; ++f) g.feat[f * capacity + i] = feat_init[f * P + p];
    }
}

// ---------------------------------------------------------------------------
// DSR
// ---------------------------------------------------------------------------
constexpr int kDsrItems = 8;
constexpr int kDsrChunk = kGrowThreads * kDsrItems;
constexpr int kDsrBlocks = 1024;  // most blocks: each reads every block's numbers in the merges below

// Sums of N values over the block, to every thread, in a fixed order.
template <int N>
__device__ __forceinline__ void block_sums_d(double (&v)[N], double (*s_red)[kGrowThreads / kWave]) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        for (int d = kWave / 2; d > 0; d >>= 1) v[k] += __shfl_xor(v[k], d, kWave);
        if (lane == 0) s_red[k][wave] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N; ++k) {
        v[k] = 0.0;
        for (int w = 0; w < kGrowThreads / kWave; ++w) v[k] += s_red[k][w];
    }
    __syncthreads();
}

__host__ __device__ __forceinline__ int64_t dsr_chunks(int64_t m) { return (m + kDsrChunk - 1) / kDsrChunk; }

// Log scales of chunk c: item k of the thread is c * kDsrChunk +
// k * kGrowThreads + threadIdx.x (the last one where there is none).
__device__ __forceinline__ void dsr_load(const float* __restrict__ ls, int64_t m, int64_t c, float (&x)[kDsrItems]) {
    const int64_t j0 = c * kDsrChunk + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kDsrItems; ++k) {
        const int64_t j = j0 + k * kGrowThreads;
        x[k] = ls[j < m ? j : m - 1];
    }
}

// The block's chunks in turn: body(k-th scales, which of them are there,
// chunk).  x holds the first chunk; the next one is under way during a body.
template <typename Body>
__device__ __forceinline__ void dsr_each(const float* __restrict__ ls, int64_t m, float (&x)[kDsrItems], Body body) {
    for (int64_t c = blockIdx.x; c < dsr_chunks(m); c += gridDim.x) {
        double s[kDsrItems];
        bool live[kDsrItems];
        float y[kDsrItems];
        if (c + gridDim.x < dsr_chunks(m)) dsr_load(ls, m, c + gridDim.x, y);
#pragma unroll
        for (int k = 0; k < kDsrItems; ++k) {
            s[k] = (double)dec_exp(x[k]);
            live[k] = c * kDsrChunk + k * kGrowThreads + threadIdx.x < m;
        }
        body(s, live, c);
#pragma unroll
        for (int k = 0; k < kDsrItems; ++k) x[k] = y[k];
    }
}

// Three launches: the moments of every block's chunks, their two sets, the
// gradient.  The blocks of the second and third merge what the one before
// left for themselves (at most kDsrBlocks numbers of each kind), instead of a
// one-block launch after every pass: seven launches took 47 us for 1 M
// Gaussians and 35 us for 77 k, three take 30 and 17.

// Count, sum and squared deviations from the mean of the block's scales, chunks merged pairwise (no sum of squares, whose difference from
// the squared mean would cancel): mom[3 b ..].
__global__ void __launch_bounds__(kGrowThreads) k_dsr_moments(const float* __restrict__ ls, int64_t m,
                                                              double* __restrict__ mom) {
    __shared__ double s_red[1][kGrowThreads / kWave];
    float x[kDsrItems];
    dsr_load(ls, m, blockIdx.x, x);
    double n = 0.0, sum = 0.0, q = 0.0;
    dsr_each(ls, m, x, [&](const double(&s)[kDsrItems], const bool(&live)[kDsrItems], int64_t c) {
        double a[1] = {0.0}, e[1] = {0.0};
#pragma unroll
        for (int k = 0; k < kDsrItems; ++k) a[0] += live[k] ? s[k] : 0.0;
        block_sums_d(a, s_red);
        const int64_t left = m - c * kDsrChunk;
        const double nc = (double)(left < kDsrChunk ? left : kDsrChunk), mc = a[0] / nc;
#pragma unroll
        for (int k = 0; k < kDsrItems; ++k) e[0] += live[k] ? (s[k] - mc) * (s[k] - mc) : 0.0;
        block_sums_d(e, s_red);
        q += e[0];
        if (n > 0.0) {
            const double d = mc - sum / n;
            q += d * d * (n * nc / (n + nc));
        }
        n += nc;
        sum += a[0];
    });
    if (threadIdx.x == 0) {
        mom[3 * blockIdx.x] = n;
        mom[3 * blockIdx.x + 1] = sum;
        mom[3 * blockIdx.x + 2] = q;
    }
}

// Mean and population standard deviation from the blocks' moments, by the
// whole block, in a fixed order.
__device__ __forceinline__ void dsr_stats(const double* __restrict__ mom, int64_t m,
                                          double (*s_red)[kGrowThreads / kWave], double& mu, double& sd) {
    double a[1] = {0.0}, q[1] = {0.0};
    for (int b = threadIdx.x; b < (int)gridDim.x; b += kGrowThreads) a[0] += mom[3 * b + 1];
    block_sums_d(a, s_red);
    mu = a[0] / (double)m;
    for (int b = threadIdx.x; b < (int)gridDim.x; b += kGrowThreads) {
        const double d = mom[3 * b + 1] / mom[3 * b] - mu;
        q[0] += mom[3 * b + 2] + mom[3 * b] * d * d;
    }
    block_sums_d(q, s_red);
    sd = sqrt(q[0] / (double)m);
}

// Sums over the block's part of the big set (s > mu + 2 sigma) of s, its
// count, over that of the small set (s < mu - 2 sigma) of -log s, its count:
// sets[4 b ..].
__global__ void __launch_bounds__(kGrowThreads) k_dsr_sets(const float* __restrict__ ls, int64_t m,
                                                           const double* __restrict__ mom,
                                                           double* __restrict__ sets, double* __restrict__ out) {
    __shared__ double s_red[4][kGrowThreads / kWave];
    float x[kDsrItems];
    dsr_load(ls, m, blockIdx.x, x);
    double mu, sd, a[4] = {0.0, 0.0, 0.0, 0.0};
    dsr_stats(mom, m, s_red, mu, sd);
    const double big = mu + 2.0 * sd, small = mu - 2.0 * sd;
    dsr_each(ls, m, x, [&](const double(&s)[kDsrItems], const bool(&live)[kDsrItems], int64_t) {
#pragma unroll
        for (int k0 = 0; k0 < kDsrItems; k0 += 4) {
            // one logarithm for four scales: the product of four floats stays
            // far inside the doubles (2^-149 to the fourth is 2^-596)
            double prod = 1.0;
#pragma unroll
            for (int k = k0; k < k0 + 4; ++k) {
                const bool in_big = live[k] && s[k] > big, in_small = live[k] && s[k] < small;
                a[0] += in_big ? s[k] : 0.0;
                a[1] += in_big ? 1.0 : 0.0;
                prod *= in_small ? s[k] : 1.0;
                a[3] += in_small ? 1.0 : 0.0;
            }
            if (prod != 1.0) a[2] -= log(prod);
        }
    });
    block_sums_d(a, s_red);
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) sets[4 * blockIdx.x + k] = a[k];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        out[3] = mu;
        out[4] = sd;
    }
}

// grad_ls[j] += w_big s / n_big (big set), -w_small / n_small (small set);
// block 0 also writes the values.  nb: the blocks of k_dsr_sets.
__global__ void __launch_bounds__(kGrowThreads) k_dsr_grad(const float* __restrict__ ls, int64_t m,
                                                           const double* __restrict__ sets, int nb, float w_big,
                                                           float w_small, float* __restrict__ grad, double* out) {
    __shared__ double s_red[4][kGrowThreads / kWave];
    float x[kDsrItems];
    dsr_load(ls, m, blockIdx.x, x);
    double r[4] = {0.0, 0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < nb; b += kGrowThreads)
#pragma unroll
        for (int k = 0; k < 4; ++k) r[k] += sets[4 * b + k];
    block_sums_d(r, s_red);
    const double mu = out[3], sd = out[4];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const double Lb = r[1] > 0.0 ? r[0] / r[1] : 0.0, Ls = r[3] > 0.0 ? r[2] / r[3] : 0.0;
        out[0] = Lb;
        out[1] = Ls;
        out[2] = (double)w_big * Lb + (double)w_small * Ls;
        out[5] = r[1];
        out[6] = r[3];
    }
    if (grad == nullptr) return;
    const double big = mu + 2.0 * sd, small = mu - 2.0 * sd;
    const double g_big = (double)w_big / r[1], g_small = -(double)w_small / r[3];
    dsr_each(ls, m, x, [&](const double(&s)[kDsrItems], const bool(&live)[kDsrItems], int64_t c) {
#pragma unroll
        for (int k = 0; k < kDsrItems; ++k) {
            if (!live[k]) continue;
            double g = 0.0;
            if (s[k] > big) g += g_big * s[k];
            if (s[k] < small) g += g_small;
            if (g != 0.0) grad[c * kDsrChunk + k * kGrowThreads + threadIdx.x] += (float)g;
        }
    });
}

}  // namespace

size_t expand_workspace_bytes(int64_t P) {
    const int64_t nblk = (P + kExpandChunk - 1) / kExpandChunk;
    return ((size_t)nblk * 4 + 255) / 256 * 256 + 256;  // block offsets, then the old count
}

hipError_t launch_expand(const uint8_t* masks, const float* rgb_t, const float* depth_t, const float* feat_init,
                         int n_feat, int64_t P, const gs_view* views_dev, int n_views, int64_t* n_dev,
                         int64_t capacity, int64_t* candidates, const gs_gaussian_grads& g, void* ws, hipStream_t s) {
    const int nblk = (int)((P + kExpandChunk - 1) / kExpandChunk);
    uint32_t* counts = static_cast<uint32_t*>(ws);
    int64_t* n_before = reinterpret_cast<int64_t*>(static_cast<char*>(ws) + ((size_t)nblk * 4 + 255) / 256 * 256);
    hipLaunchKernelGGL(k_expand_count, dim3(nblk), dim3(kGrowThreads), 0, s, masks, depth_t, P, counts);
    hipLaunchKernelGGL(k_expand_scan, dim3(1), dim3(1024), 0, s, counts, nblk, n_dev, capacity, n_before, candidates);
    switch (n_feat) {
        case 0:
            hipLaunchKernelGGL(k_expand_write<0>, dim3(nblk), dim3(kGrowThreads), 0, s, masks, rgb_t, depth_t, feat_init,
                               P, views_dev, n_views, counts, n_before, capacity, g);
            break;
        case 8:
            hipLaunchKernelGGL(k_expand_write<8>, dim3(nblk), dim3(kGrowThreads), 0, s, masks, rgb_t, depth_t, feat_init,
                               P, views_dev, n_views, counts, n_before, capacity, g);
            break;
        case 32:
            hipLaunchKernelGGL(k_expand_write<32>, dim3(nblk), dim3(kGrowThreads), 0, s, masks, rgb_t, depth_t,
                               feat_init, P, views_dev, n_views, counts, n_before, capacity, g);
            break;
        default:
            hipLaunchKernelGGL(k_expand_write<16>, dim3(nblk), dim3(kGrowThreads), 0, s, masks, rgb_t, depth_t,
                               feat_init, P, views_dev, n_views, counts, n_before, capacity, g);
            break;
    }
    return hipGetLastError();
}

static int dsr_blocks(int64_t m) {
    const int64_t chunks = dsr_chunks(m), per = (chunks + kDsrBlocks - 1) / kDsrBlocks;
    return (int)((chunks + per - 1) / per);
}

size_t dsr_workspace_bytes(int64_t n) {
    if (n <= 0) return 0;
    // moments [nb][3], sets [nb][4]; all kDsrBlocks from there on, so that a
    // workspace sized for more Gaussians serves fewer
    const int64_t chunks = dsr_chunks(3 * n);
    return ((size_t)(chunks < kDsrBlocks ? chunks : kDsrBlocks) * 7 * 8 + 255) / 256 * 256;
}

hipError_t launch_dsr(const float* log_scale, int64_t n, float w_big, float w_small, float* grad_ls, double* out,
                      void* ws, hipStream_t s) {
    const int64_t m = 3 * n;
    const int nb = dsr_blocks(m);
    double* mom = static_cast<double*>(ws);
    double* sets = mom + 3 * (size_t)nb;
    hipLaunchKernelGGL(k_dsr_moments, dim3(nb), dim3(kGrowThreads), 0, s, log_scale, m, mom);
    hipLaunchKernelGGL(k_dsr_sets, dim3(nb), dim3(kGrowThreads), 0, s, log_scale, m, mom, sets, out);
    hipLaunchKernelGGL(k_dsr_grad, dim3(grad_ls != nullptr ? nb : 1), dim3(kGrowThreads), 0, s, log_scale, m, sets, nb,
                       w_big, w_small, grad_ls, out);
    return hipGetLastError();
}

}  // namespace sgs
