// SLAM losses of GS^3LAM with their masks (Sec. 3.3.1, Eq. 11; Sec. 3.3.4,
// Eq. 15-18; Sec. 3.4, Eq. 21), all on the device and graph-capturable:
//
//   1. median depth error per view: the lower median of the binary32
//      residuals r = |D - D*| over the pixels with D* > 0, found exactly by
//      a radix select over the residual bits (non-negative floats order as
//      their bit patterns): three passes of 11, 10 and 10 bits, each a
//      histogram of the digit among the residuals that match the prefix
//      selected so far (k_median).  Every block of the next pass locates the
//      bucket holding the wanted rank for itself.  Integer counts only, so
//      the result is the same every run.
//   2. one thread per pixel (k_slam_loss): the masks M_obs (Eq. 21) and
//      M_unobs (Eq. 11) from binary32 tests, then the L1
//      colour and depth terms and the semantic cross-entropy, each weighted
//      by M_obs when the tracking mask is on, with their gradients.  With the
//      decoder's own gradients, k_slam_loss_dec.
//   3. with lambda > 0, the SSIM part of Eq. (15)'s colour term: per colour
//      channel and 64x16 output tile, k_ssim_fwd filters x, y, x^2, y^2 and
//      xy with the separable 11-tap Gaussian (sigma 1.5) over the tile plus
//      a 5-pixel apron staged in LDS (zero outside the view), forms SSIM and
//      its partial derivatives with respect to the three windowed sums that
//      depend on x, and writes them, scaled, as three maps; k_ssim_bwd
//      filters the maps again (the window is symmetric, so the adjoint is the
//      same filter) and adds G*m_mu + 2 x G*m_xx + y G*m_xy to the colour
//      gradient.  Both walk the tiles persistently, loading the next tile
//      while the current one is filtered.  Where it takes less time (strip_rows),
//      k_ssim does both in one pass down strips of columns, and the maps never
//      leave the chip.
//   4. a fixed-order sum of the per-block partial losses (deterministic).
#include "loss_common.h"

namespace sgs {

namespace {

constexpr int kSlamThreads = 256;
constexpr int kMedItems = 16;  // pixels per thread in a histogram block
constexpr int kMedChunk = kSlamThreads * kMedItems;
constexpr int kSsimTX = 64, kSsimTY = 16, kSsimR = 5;  // output tile, window radius
constexpr int kSsimIX = kSsimTX + 2 * kSsimR, kSsimIY = kSsimTY + 2 * kSsimR;

struct SlamParams {
    float w0, w1, w2, lam;
    float tau_obs, tau_unobs, obs_factor, unobs_factor;
    int use_obs, bce;
};

struct SsimConst {
    float g[2 * kSsimR + 1];  // 1-D window; the 2-D window is g[a] g[b]
    float c1, c2, lam_w0;     // lambda * w_color
};

// First SSIM tile of each view (tiles of kSsimTX x kSsimTY, row-major per view).
struct SsimTiles {
    int first[GS_MAX_VIEWS + 1];
    int n_views;
};

// Strips of k_ssim: first workgroup of each view (x strip fastest, then
// channel, then y strip), output rows of a strip.
constexpr int kStripBW = 256, kStripR = 4;  // columns of a strip with its 10 on either side, rows of a step
constexpr int kSsimPad = 8;                 // columns of zeros left and right of a strip in LDS
// k_ssim filters x - 1/2 and y - 1/2 (-1/2 outside the view): variances and
// the covariance do not change with it, and the squares that round are at most
// a quarter instead of one.  Against 64 bits the colour gradient of the
// mapping loss is 1.9e-7 off instead of 1.0e-6 (eight 1200x680 views).
constexpr float kSsimMid = 0.5f;
struct SsimStrips {
    int first[GS_MAX_VIEWS + 1];
    int n_views, rows;
};

// View of pixel p of a workgroup whose pixels are consecutive, p0 (uniform) the
// first of them: found once, with scalar loads, where they are all of one
// view.
__device__ __forceinline__ int view_of_pixel(const gs_view* views, int n_views, int64_t p0, int64_t p) {
    int v = 0;
    while (v + 1 < n_views && views[v + 1].pixel_offset <= p0) ++v;
    if (v + 1 < n_views && views[v + 1].pixel_offset < p0 + kSlamThreads)  // uniform
        while (v + 1 < n_views && views[v + 1].pixel_offset <= p) ++v;
    return v;
}

// ---------------------------------------------------------------------------
// 1. median depth error
// ---------------------------------------------------------------------------
// Digits of the passes, from the top of the 31 bits of a residual.
template <int PASS>
struct MedDigit {
    static constexpr int bits = PASS == 0 ? 11 : 10;
    static constexpr int shift = PASS == 0 ? 20 : (PASS == 1 ? 10 : 0);
    static constexpr int bins = 1 << bits;
    static constexpr int first = PASS == 0 ? 0 : (PASS == 1 ? 2048 : 3072);  // of the view's histogram words
};
constexpr int kMedWords = 2048 + 2 * 1024;

// Per view, after the selection of a pass: the prefix selected so far, the
// rank still wanted within it, the number of valid pixels.
struct MedSel {
    uint32_t prefix, rank, count, pad;
};

// The transposed decoder [K][F], at most 64 rows of 32, then its bias.
constexpr int kWtBias = 32 * GS_SLAM_MAX_CLASSES, kWtFloats = kWtBias + GS_SLAM_MAX_CLASSES;

// Weight of each term per pixel of a view, in the precision it is applied in
// (a division each, eleven of binary32 and thirty of FP64 instructions, which
// every pixel would repeat).
struct ViewWeights {
    float gc, gd, gs, pad;  // gradients of the colour L1, depth and semantic term
    double d, s;            // values of the depth and semantic term
};

// Clears the histograms, transposes the decoder and forms the views' weights.
__global__ void __launch_bounds__(256) k_slam_prep(uint32_t* __restrict__ words, int n, const float* __restrict__ W,
                                                   const float* __restrict__ bias, int F, int K,
                                                   float* __restrict__ Wt, const gs_view* __restrict__ views,
                                                   int n_views, SlamParams sp, ViewWeights* __restrict__ vw) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n_views) {
        const float Pv = (float)((int64_t)views[i].width * views[i].height);
        vw[i] = {(1.0f - sp.lam) * sp.w0 / (3.0f * Pv), sp.w1 / Pv, sp.w2 / Pv, 0.0f,
                 (double)sp.w1 / (double)Pv, (double)sp.w2 / (double)Pv};
    }
    if (i < n) words[i] = 0;
    if (W != nullptr) {
        transpose_decoder(W, F, K, Wt, i);
        // k_slam_loss_dec takes the classes four at a time: zero rows and a
        // bias of -infinity up to a multiple of four, so that the classes
        // that are not there have logit -infinity and probability 0
        const int K4 = (K + 3) / 4 * 4;
        if (i >= F * K && i < F * K4) Wt[i] = 0.0f;
        if (i < K4) Wt[kWtBias + i] = i < K ? (bias != nullptr ? bias[i] : 0.0f) : -INFINITY;
    }
}

// Lanes of the wavefront with the same `bits`-bit digit among the valid ones.
template <int BITS>
__device__ __forceinline__ uint64_t match_bits(uint32_t d, bool valid) {
    uint64_t m = __builtin_amdgcn_ballot_w64(valid);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bb = __builtin_amdgcn_ballot_w64(bit);
        m &= bit ? bb : ~bb;
    }
    return m;
}

// Selection after pass PASS, by a whole block: the bin of its histogram that
// holds the wanted rank.  Returns the selection after it (all threads).
template <int PASS>
__device__ __forceinline__ MedSel median_select(const uint32_t* __restrict__ hist, const MedSel* __restrict__ sel,
                                                int v, uint32_t* s_tmp, MedSel* s_sel) {
    using D = MedDigit<PASS>;
    constexpr int PER = D::bins / kSlamThreads;
    const int tid = threadIdx.x;
    const uint32_t* hv = hist + (size_t)v * kMedWords + D::first + tid * PER;
    uint32_t c[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        c[q] = hv[q];
        sum += c[q];
    }
    MedSel m = {0, 0, 0, 0};
    if constexpr (PASS > 0) m = sel[2 * v + PASS - 1];
    uint32_t total;
    uint32_t excl = block_exclusive<kSlamThreads>(sum, s_tmp, &total);
    if constexpr (PASS == 0) {
        m.count = total;
        m.rank = total > 0 ? (total - 1) / 2 : 0;
    }
    if (tid == 0) *s_sel = m;  // of a view without a valid depth
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (m.count > 0 && excl <= m.rank && m.rank < excl + c[q])  // exactly one thread and bin
            *s_sel = {(m.prefix << D::bits) | (uint32_t)(tid * PER + q), m.rank - excl, m.count, 0};
        excl += c[q];
    }
    __syncthreads();
    return *s_sel;
}

// One pass over one view (blockIdx.y).  Bound by latency: a block streams
// 32 KB and waits for it once, while it selects the previous pass's bucket.
// (Four 8-bit passes with a selection launch after each were 9 launches,
// 52 us for one 1200x680 view, 31 in 5 now; eight views 88 and 69.  The view's last block
// doing the selection instead, behind a device-wide fence in every block,
// made a pass 18 us there and 140 us at eight views: each fence writes an L2
// back.)
template <int PASS>
__global__ void __launch_bounds__(kSlamThreads) k_median(const float* __restrict__ depth,
                                                         const float* __restrict__ depth_t,
                                                         const gs_view* __restrict__ views,
                                                         uint32_t* __restrict__ hist, MedSel* __restrict__ sel) {
    using D = MedDigit<PASS>;
    __shared__ uint32_t h[D::bins];
    __shared__ uint32_t s_tmp[kSlamThreads / kWave];
    __shared__ MedSel s_sel;
    const int v = blockIdx.y, tid = threadIdx.x, lane = tid & (kWave - 1);
    const int64_t off = views[v].pixel_offset;
    const int64_t Pv = (int64_t)views[v].width * views[v].height;
    const int64_t b0 = (int64_t)blockIdx.x * kMedChunk;
    if (b0 >= Pv) return;  // uniform over the block
    // every load first (index clamped into the view), then the decisions
    float dtv[kMedItems], dv[kMedItems];
#pragma unroll
    for (int k = 0; k < kMedItems; ++k) {
        const int64_t j = b0 + k * kSlamThreads + tid;
        const int64_t jc = j < Pv ? j : Pv - 1;
        dtv[k] = depth_t[off + jc];
        dv[k] = depth[off + jc];
    }
    for (int i = tid; i < D::bins; i += kSlamThreads) h[i] = 0;
    uint32_t prefix = 0;
    if constexpr (PASS > 0) {
        const MedSel m = median_select<PASS - 1>(hist, sel, v, s_tmp, &s_sel);
        if (blockIdx.x == 0 && tid == 0) sel[2 * v + PASS - 1] = m;  // for the next launch
        if (m.count == 0) return;  // uniform: no valid pixel in the view
        prefix = m.prefix;
    } else {
        __syncthreads();
    }
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
#pragma unroll
    for (int k = 0; k < kMedItems; ++k) {
        const int64_t j = b0 + k * kSlamThreads + tid;
        const uint32_t u = __float_as_uint(fabsf(dv[k] - dtv[k]));
        bool ok = j < Pv && dtv[k] > 0.0f;
        if constexpr (PASS > 0) ok = ok && (u >> (D::shift + D::bits)) == prefix;
        const uint32_t d = (u >> D::shift) & (uint32_t)(D::bins - 1);
        if constexpr (PASS == 0) {
            // one LDS add per distinct digit of the wavefront (the residuals
            // of a view mostly share a few top digits; the lower ones differ)
            const uint64_t peers = match_bits<D::bits>(d, ok);
            if (ok && (peers & below) == 0) atomicAdd(&h[d], (uint32_t)__popcll(peers));
        } else {
            if (ok) atomicAdd(&h[d], 1u);
        }
    }
    __syncthreads();
    uint32_t* hv = hist + (size_t)v * kMedWords + D::first;
    for (int i = tid; i < D::bins; i += kSlamThreads)
        if (h[i] != 0) atomicAdd(&hv[i], h[i]);
}

__global__ void __launch_bounds__(kSlamThreads) k_median_final(const uint32_t* __restrict__ hist,
                                                               const MedSel* __restrict__ sel,
                                                               float* __restrict__ med_ws,
                                                               float* __restrict__ med_out) {
    __shared__ uint32_t s_tmp[kSlamThreads / kWave];
    __shared__ MedSel s_sel;
    const int v = blockIdx.x;
    const MedSel m = median_select<2>(hist, sel, v, s_tmp, &s_sel);
    if (threadIdx.x == 0) {
        // the selected residual, whatever its bits; 0 without a valid depth
        const float r = m.count > 0 ? __uint_as_float(m.prefix) : 0.0f;
        med_ws[v] = r;
        if (med_out != nullptr) med_out[v] = r;
    }
}

// ---------------------------------------------------------------------------
// 2. per-pixel masks, L1 terms and cross-entropy
// ---------------------------------------------------------------------------
// Semantic term of one pixel through the decoder z = W^T f + b (a 1x1
// convolution standing in for F_cnn, Eq. 8), K <= KC classes, logits in
// registers: the BCE of Eq. (16), -sum_k [y_k log p_k + (1 - y_k) log(1 -
// p_k)], each log clamped at -100 (no gradient through a clamped log).
// Returns the term and leaves dz = dterm/dz in z: dz_j = p_j (dp_j - sum_k
// p_k dp_k) with dp_k the derivative in p_k.  (The cross-entropy -log p_lab,
// dz = p - y, is semantic_ce.)  A class row of Wt is wavefront-uniform:
// scalar loads feeding the FMAs.
template <int F, int KC>
__device__ __forceinline__ float sem_dz(const float (&fv)[F], const float* __restrict__ Wt,
                                        const float* __restrict__ bias, int K, int lab, float (&z)[KC]) {
    // z = W^T f + b, then in place z - max (the only per-class state kept,
    // so that the logits cost one register per class)
    float m = -INFINITY;
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        if (k < K) {
            const float* wr = Wt + k * F;
            float acc = bias != nullptr ? bias[k] : 0.0f;
#pragma unroll
            for (int f = 0; f < F; ++f) acc = fmaf(wr[f], fv[f], acc);
            z[k] = acc;
            m = fmaxf(m, acc);
        }
    }
    float se = 0.0f;
#pragma unroll
    for (int k = 0; k < KC; ++k)
        if (k < K) {
            z[k] -= m;
            se += __expf(z[k]);
        }
    const float inv = 1.0f / se, lse = __logf(se);
    float L = 0.0f;
    // p_k, log p_k = z_k - lse, log(1 - p_k) = log(se - e_k) - lse;
    // z keeps p_k and one bit per class whether the log that class's
    // gradient uses is above the clamp, so dp_k = -1/p_k (label) or
    // 1/(1 - p_k) (other classes, hardware reciprocals) is rebuilt in the
    // last pass without another exp or log
    float sdp = 0.0f;
    uint64_t live = 0;
#pragma unroll
    for (int k = 0; k < KC; ++k)
        if (k < K) {
            const bool y = k == lab;
            const float e = __expf(z[k]), pk = e * inv;
            const float lp = z[k] - lse;            // log p_k
            const float lq = __logf(se - e) - lse;  // log(1 - p_k)
            L -= y ? fmaxf(lp, -100.0f) : fmaxf(lq, -100.0f);
            const bool on = y ? lp > -100.0f : lq > -100.0f;
            const float dp = on ? (y ? -__builtin_amdgcn_rcpf(pk) : __builtin_amdgcn_rcpf(1.0f - pk)) : 0.0f;
            sdp = fmaf(pk, dp, sdp);
            z[k] = pk;
            live |= (uint64_t)on << k;
        }
#pragma unroll
    for (int k = 0; k < KC; ++k)
        if (k < K) {
            const float pk = z[k];
            const float dp = ((live >> k) & 1) ? (k == lab ? -__builtin_amdgcn_rcpf(pk)
                                                            : __builtin_amdgcn_rcpf(1.0f - pk))
                                               : 0.0f;
            z[k] = pk * (dp - sdp);  // dz
        }
    return L;
}

// The per-pixel terms without the semantic one: masks, L1 colour and depth
// and their gradients.  Returns whether the pixel counts; terms not yet
// divided by the pixels.
struct PixelTerms {
    double c, d;     // sums of |C - C*| and |D - D*|
    ViewWeights w;
};
// The pixel is p0 + i, p0 uniform over the workgroup: the planes' addresses
// are then scalar work.
__device__ __forceinline__ bool pixel_terms(const float* __restrict__ out, int64_t P, int64_t p0, int i,
                                            const float* __restrict__ rgb_t, const float* __restrict__ depth_t,
                                            const SlamParams& sp, const float* __restrict__ med,
                                            const ViewWeights* __restrict__ vws,
                                            const gs_view* __restrict__ views, int n_views,
                                            float* __restrict__ grad_out, uint8_t* __restrict__ masks,
                                            PixelTerms& t) {
    // every load first: one round trip to memory
    float x[3], y[3];
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        x[ch] = (out + ch * P + p0)[i];
        y[ch] = (rgb_t + ch * P + p0)[i];
    }
    const float d = (out + 3 * P + p0)[i], dt = (depth_t + p0)[i], o = (out + 4 * P + p0)[i];
    const int v = view_of_pixel(views, n_views, p0, p0 + i);
    t.w = vws[v];
    t.c = t.d = 0.0;
    // Eq. (21) / Eq. (11), binary32 tests
    const float r = fabsf(d - dt), m = med[v];
    const float lim_obs = sp.obs_factor * m, lim_unobs = sp.unobs_factor * m;
    const bool obs = (o > sp.tau_obs) && (r < lim_obs);
    const bool unobs = (o < sp.tau_unobs) || ((d > dt) && (r > lim_unobs));
    (masks + p0)[i] = (uint8_t)((obs ? 1 : 0) | (unobs ? 2 : 0));
    const bool on = !sp.use_obs || obs;
    if (on) {
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            const float rc = x[ch] - y[ch];
            t.c += (double)fabsf(rc);
            (grad_out + ch * P + p0)[i] = rc > 0.0f ? t.w.gc : (rc < 0.0f ? -t.w.gc : 0.0f);
        }
        const float rd = d - dt;
        t.d += (double)fabsf(rd);
        (grad_out + 3 * P + p0)[i] = rd > 0.0f ? t.w.gd : (rd < 0.0f ? -t.w.gd : 0.0f);
    } else {
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) (grad_out + ch * P + p0)[i] = 0.0f;
    }
    (grad_out + 4 * P + p0)[i] = 0.0f;
    return on;
}

// The workgroup's sums of the three terms into its partials (term-major).
__device__ __forceinline__ void store_partials(double lc, double ld, double ls,
                                               double (&s_red)[3][kSlamThreads / kWave],
                                               double* __restrict__ partials) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    for (int dd = kWave / 2; dd > 0; dd >>= 1) {
        lc += __shfl_xor(lc, dd, kWave);
        ld += __shfl_xor(ld, dd, kWave);
        ls += __shfl_xor(ls, dd, kWave);
    }
    if (lane == 0) {
        s_red[0][wave] = lc;
        s_red[1][wave] = ld;
        s_red[2][wave] = ls;
    }
    __syncthreads();
    if (tid < 3) {
        double a = 0;
        for (int w = 0; w < kSlamThreads / kWave; ++w) a += s_red[tid][w];
        partials[(size_t)tid * gridDim.x + blockIdx.x] = a;
    }
}

// BCE: the semantic term through dz (sem_dz), otherwise the fused
// cross-entropy (fewer registers).
template <int F, int KC, bool BCE>
__global__ void __launch_bounds__(kSlamThreads) k_slam_loss(const float* __restrict__ out, int64_t P,
                                                            const float* __restrict__ rgb_t,
                                                            const float* __restrict__ depth_t,
                                                            const int32_t* __restrict__ labels,
                                                            const float* __restrict__ Wt,
                                                            const float* __restrict__ bias, int K, SlamParams sp,
                                                            const float* __restrict__ med,
                                                            const ViewWeights* __restrict__ vws,
                                                            const gs_view* __restrict__ views, int n_views,
                                                            float* __restrict__ grad_out,
                                                            uint8_t* __restrict__ masks,
                                                            double* __restrict__ partials) {
    __shared__ double s_red[3][kSlamThreads / kWave];
    const int64_t p0 = (int64_t)blockIdx.x * kSlamThreads;
    const int i = threadIdx.x;
    double lc = 0.0, ld = 0.0, ls = 0.0;
    if (p0 + i < P) {
        PixelTerms t;
        const bool on = pixel_terms(out, P, p0, i, rgb_t, depth_t, sp, med, vws, views, n_views, grad_out, masks, t);
        double ps = 0.0;
        if constexpr (F > 0) {
            float fv[F], gf[F];
#pragma unroll
            for (int f = 0; f < F; ++f) gf[f] = 0.0f;
            if (on && K > 0 && sp.w2 != 0.0f) {
#pragma unroll
                for (int f = 0; f < F; ++f) fv[f] = (out + (5 + f) * P + p0)[i];
                if constexpr (!BCE) {
                    ps = (double)semantic_ce<F, KC>(fv, Wt, K, (labels + p0)[i], gf, bias);
                } else {
                    float dz[KC];
                    ps = (double)sem_dz<F, KC>(fv, Wt, bias, K, (labels + p0)[i], dz);
                    // dL/df = W dz
#pragma unroll
                    for (int k = 0; k < KC; ++k)
                        if (k < K) {
                            const float* wr = Wt + k * F;
#pragma unroll
                            for (int f = 0; f < F; ++f) gf[f] = fmaf(wr[f], dz[k], gf[f]);
                        }
                }
            }
#pragma unroll
            for (int f = 0; f < F; ++f) (grad_out + (5 + f) * P + p0)[i] = t.w.gs * gf[f];
        }
        lc = t.c * (double)t.w.gc;
        ld = t.d * t.w.d;
        ls = ps * t.w.s;
    }
    store_partials(lc, ld, ls, s_red, partials);
}

// The same with the decoder gradients dW = sum_p s_p f_p dz_p^T and db =
// sum_p s_p dz_p (s = w_sem M(p) / P_v).  Workgroups stay and take 256
// pixels in turn; the wavefronts share nothing until the end, so no barrier
// holds one between its pixels.
//
// A lane's logits live in a row of LDS and not in registers: the classes run
// in a loop of four at a time (four independent chains of F FMAs, the four
// rows of W in scalar registers), the passes over the classes -- logits and
// maximum, exponentials and sum, dz and W dz -- read and write the row, and
// what it holds at the end is the operand B of the contraction.  That runs on
// MFMA (16x16x4 f32, four pixels per step: A[m][k] = f of pixel k at row m,
// staged 32 pixels at a time, B[k][n] = scaled dz of pixel k at class n); B is
// also what the bias sums add up.  Rows are an odd number of floats apart, so
// that neither the lanes' accesses nor the operand loads share banks.  Each
// 64 pixels are summed in binary32 by the MFMAs, and those sums in FP64.
//
// Bound by issue (4 F K flops per pixel, 2 F K more in the MFMAs, which share
// the issue slots, and an exponential per class: 1317 instructions per 64
// pixels at F = 16 and K = 20, 32 of them MFMA of 33 cycles, about 260 of its
// 400 us), then by latency.  With the logits in
// registers, one pixel per thread and the workgroup's reduction after every
// 256 pixels it was held by latency at three or four wavefronts per SIMD:
// 549 us for eight 1200x680 views at F = 16, K = 20, 400 us now; a fifth
// wavefront per SIMD spills 26 registers and is slower.
__host__ __device__ constexpr int odd_stride(int n) { return n | 1; }
// Floats of a wavefront's slot: its rows, and room for the operand loads of
// the last ones, which run past them (rows m >= F of A and classes n >= K of
// B: what they hold only reaches entries of D that nobody reads).
__host__ __device__ constexpr int dec_slot(int F, int K) {
    return kWave * odd_stride((K + 3) / 4 * 4) + kWave / 2 * odd_stride(F) + 16;
}
inline size_t dec_lds_bytes(int F, int K) {
    const size_t slot = (size_t)dec_slot(F, K), tile = (size_t)F * K;
    return (kSlamThreads / kWave) * sizeof(float) * (slot > tile ? slot : tile);
}

template <int F, int NT, bool BCE>
__global__ void __launch_bounds__(kSlamThreads)
    __attribute__((amdgpu_waves_per_eu(F <= 16 && NT <= 2 ? 4 : 2, 8))) k_slam_loss_dec(const float* __restrict__ out, int64_t P,
                                                                const float* __restrict__ rgb_t,
                                                                const float* __restrict__ depth_t,
                                                                const int32_t* __restrict__ labels,
                                                                const float* __restrict__ Wt, int K, SlamParams sp,
                                                                const float* __restrict__ med,
                                                                const ViewWeights* __restrict__ vws,
                                                                const gs_view* __restrict__ views, int n_views,
                                                                float* __restrict__ grad_out,
                                                                uint8_t* __restrict__ masks,
                                                                double* __restrict__ partials,
                                                                float* __restrict__ dec_partials) {
    constexpr int NW = kSlamThreads / kWave, MT = (F + 15) / 16, ROWS = kWave / 2;
    constexpr int FS = odd_stride(F), U = F > 16 ? 2 : 4;  // rows of W at a time, 64 scalar registers
    constexpr int U2 = F > 8 ? 2 : 4;                 // half in the last pass, whose loop holds more
    extern __shared__ float s_dyn[];
    __shared__ double s_red[3][NW];
    __shared__ float s_db[NW][16 * NT];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int K4 = (K + 3) / 4 * 4, ZS = odd_stride(K4);
    const float* bias = Wt + kWtBias;
    float* const sZ = s_dyn + wave * dec_slot(F, K);  // [64][ZS]
    float* const sF = sZ + kWave * ZS;                          // [32][FS]
    float* const z = sZ + lane * ZS;
    const int col = lane & 15, kk = lane >> 4;
    // entry i of tile (mt, nt) is row 16 mt + 4 kk + i, class 16 nt + col; the
    // bias sums are of class 16 nt + col over the pixel rows kk, kk + 4, ...
    double lc = 0.0, ld = 0.0, ls = 0.0;
    using f4 = __attribute__((__vector_size__(4 * sizeof(float)))) float;
    double dws[MT][NT][4], dbs[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        dbs[nt] = 0.0;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i) dws[mt][nt][i] = 0.0;
    }
    for (int64_t p0 = (int64_t)blockIdx.x * kSlamThreads; p0 < P; p0 += (int64_t)gridDim.x * kSlamThreads) {
        bool on = false;
        float scale = 0.0f, fv[F];
        if (p0 + tid < P) {
            // with every other load of the pixel, before anything waits; no
            // class at all for a label outside [0, K), as without the decoder
            // gradients (the rows up to K4 are no classes either)
            int lab = (labels + p0)[tid];
            lab = lab < K ? lab : -1;
#pragma unroll
            for (int f = 0; f < F; ++f) fv[f] = (out + (5 + f) * P + p0)[tid];
            PixelTerms t;
            on = pixel_terms(out, P, p0, tid, rgb_t, depth_t, sp, med, vws, views, n_views, grad_out, masks, t);
            float gf[F];
#pragma unroll
            for (int f = 0; f < F; ++f) gf[f] = 0.0f;
            if (on) {
                scale = t.w.gs;
                // logits, their maximum, the label's
                float m = -INFINITY, zl = 0.0f;
                for (int k0 = 0; k0 < K4; k0 += U) {
                    float a[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) a[u] = bias[k0 + u];
#pragma unroll
                    for (int f = 0; f < F; ++f)
#pragma unroll
                        for (int u = 0; u < U; ++u) a[u] = fmaf(Wt[(k0 + u) * F + f], fv[f], a[u]);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        z[k0 + u] = a[u];
                        m = fmaxf(m, a[u]);
                        zl = k0 + u == lab ? a[u] : zl;
                    }
                }
                const bool has = lab >= 0;
                float se = 0.0f, term = 0.0f, sdp = 0.0f, inv;
                uint64_t live = 0;
                if constexpr (!BCE) {
#pragma unroll 4
                    for (int k = 0; k < K4; ++k) {
                        const float e = __expf(z[k] - m);
                        z[k] = e;
                        se += e;
                    }
                    inv = 1.0f / se;
                    term = has ? __logf(se) - (zl - m) : 0.0f;
                } else {
                    // p_k, log p_k = z_k - lse, log(1 - p_k) = log(se - e_k) -
                    // lse; the row keeps p_k and `live` whether the log that
                    // the class's gradient uses is above the clamp, so that
                    // dp_k = -1/p_k (label) or 1/(1 - p_k) (other classes,
                    // hardware reciprocals) is rebuilt in the last pass
#pragma unroll 4
                    for (int k = 0; k < K4; ++k) {
                        const float zk = z[k] - m;
                        z[k] = zk;
                        se += __expf(zk);
                    }
                    inv = 1.0f / se;
                    const float lse = __logf(se);
#pragma unroll 4
                    for (int k = 0; k < K4; ++k) {
                        const bool y = k == lab;
                        const float zk = z[k], e = __expf(zk), pk = e * inv;
                        const float lp = zk - lse, lq = __logf(se - e) - lse;
                        term -= y ? fmaxf(lp, -100.0f) : fmaxf(lq, -100.0f);
                        const bool w = y ? lp > -100.0f : lq > -100.0f;
                        const float dp =
                            w ? (y ? -__builtin_amdgcn_rcpf(pk) : __builtin_amdgcn_rcpf(1.0f - pk)) : 0.0f;
                        sdp = fmaf(pk, dp, sdp);
                        z[k] = pk;
                        live |= (uint64_t)w << k;
                    }
                    // the rows past K gave 0, but of a pixel that is not
                    // finite (every logarithm NaN) the clamp's 100 each
                    if (se != se) term -= 100.0f * (float)(K4 - K);
                }
                // dz and dL/df = W dz; the row ends as the scaled dz
                for (int k0 = 0; k0 < K4; k0 += U2) {
                    float dz[U2];
#pragma unroll
                    for (int u = 0; u < U2; ++u) {
                        const int k = k0 + u;
                        if constexpr (!BCE) {
                            dz[u] = z[k] * inv - (k == lab ? 1.0f : 0.0f);
                        } else {
                            const float pk = z[k];
                            const float dp = ((live >> k) & 1)
                                                 ? (k == lab ? -__builtin_amdgcn_rcpf(pk) : __builtin_amdgcn_rcpf(1.0f - pk))
                                                 : 0.0f;
                            dz[u] = pk * (dp - sdp);
                        }
                        z[k] = scale * dz[u];
                    }
#pragma unroll
                    for (int u = 0; u < U2; ++u)
#pragma unroll
                        for (int f = 0; f < F; ++f) gf[f] = fmaf(Wt[(k0 + u) * F + f], dz[u], gf[f]);
                }
                ls += (double)term * t.w.s;
            }
#pragma unroll
            for (int f = 0; f < F; ++f) (grad_out + (5 + f) * P + p0)[tid] = t.w.gs * gf[f];
            lc += t.c * (double)t.w.gc;
            ld += t.d * t.w.d;
        }
        if (__builtin_amdgcn_ballot_w64(!on) != 0 && !on) {  // no contribution
            for (int k = 0; k < K4; ++k) z[k] = 0.0f;
#pragma unroll
            for (int f = 0; f < F; ++f) fv[f] = 0.0f;
        }
        f4 acc[MT][NT];
        float db[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            db[nt] = 0.0f;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = f4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        for (int half = 0; half < 2; ++half) {
            if ((lane >> 5) == half) {
#pragma unroll
                for (int f = 0; f < F; ++f) sF[(lane & (ROWS - 1)) * FS + f] = fv[f];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 2
            for (int st = 0; st < ROWS / 4; ++st) {
                const int pr = 4 * st + kk;
                float a[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    a[mt] = sF[pr * FS + col + 16 * mt];
                }
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    if (16 * nt >= K) continue;  // uniform
                    const float b = sZ[(half * ROWS + pr) * ZS + col + 16 * nt];
                    db[nt] += b;
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[mt], b, acc[mt][nt], 0, 0, 0);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            dbs[nt] += (double)db[nt];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i) dws[mt][nt][i] += (double)acc[mt][nt][i];
        }
    }
    // the wavefronts' tiles and bias sums added in a fixed order: this
    // workgroup's partial, dW [F][K], then db [K]
    __syncthreads();  // every wavefront is done with its slot
    float* sD = s_dyn + wave * F * K;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int mm = 16 * mt + 4 * kk + i, nn = 16 * nt + col;
                if (mm < F && nn < K) sD[mm * K + nn] = (float)dws[mt][nt][i];
            }
        double t = dbs[nt];
        t += __shfl_xor(t, 16, kWave);
        t += __shfl_xor(t, 32, kWave);
        if (kk == 0) s_db[wave][16 * nt + col] = (float)t;
    }
    __syncthreads();
    float* dst = dec_partials + (size_t)blockIdx.x * (F * K + K);
    for (int e = tid; e < F * K; e += kSlamThreads) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) t += s_dyn[w * F * K + e];
        dst[e] = t;
    }
    if (tid < K) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) t += s_db[w][tid];
        dst[F * K + tid] = t;
    }
    store_partials(lc, ld, ls, s_red, partials);
}

// ---------------------------------------------------------------------------
// 3. SSIM term
// ---------------------------------------------------------------------------
struct TileIdx {
    int v, x0, y0, W, H;
};
__device__ __forceinline__ TileIdx ssim_tile(const SsimTiles& st, const gs_view* views, int t) {
    int v = 0;
    while (v + 1 < st.n_views && st.first[v + 1] <= t) ++v;
    TileIdx ti;
    ti.v = v;
    ti.W = views[v].width;
    ti.H = views[v].height;
    const int tx = ceil_div(ti.W, kSsimTX);
    const int lt = t - st.first[v];
    ti.x0 = (lt % tx) * kSsimTX;
    ti.y0 = (lt / tx) * kSsimTY;
    return ti;
}

// Staged input of one tile: rows of the output tile plus a kSsimR apron
// above and below, kSsimIX columns (the tile plus the apron left and right)
// padded to kSsimLD so that every row starts 16-byte aligned.
constexpr int kSsimLD = (kSsimIX + 3) / 4 * 4;
// horizontal pass: a thread slides the window over kSsimHX consecutive
// outputs of one staged row; vertical pass: over kSsimVY rows of one column
constexpr int kSsimHX = 8;
constexpr int kSsimVY = kSsimTY / (kSlamThreads / kSsimTX);
static_assert(kSsimTX % kSsimHX == 0 && kSsimIY * (kSsimTX / kSsimHX) <= kSlamThreads, "one horizontal item per thread");
static_assert(kSsimHX + 2 * kSsimR <= kSsimLD - kSsimHX * (kSsimTX / kSsimHX - 1), "horizontal window inside the row");

// n consecutive floats of an LDS row from a 16-byte aligned start
template <int N>
__device__ __forceinline__ void lds_row(const float* __restrict__ src, float (&v)[N]) {
    static_assert(N % 4 == 0, "whole float4");
#pragma unroll
    for (int k = 0; k < N / 4; ++k) {
        const float4 a = reinterpret_cast<const float4*>(src)[k];
        v[4 * k] = a.x;
        v[4 * k + 1] = a.y;
        v[4 * k + 2] = a.z;
        v[4 * k + 3] = a.w;
    }
}
constexpr int kSsimHN = (kSsimHX + 2 * kSsimR + 3) / 4 * 4;  // floats read per horizontal item (18 -> 20)

// Stages rows [y0 - R, y0 + TY + R) x columns [x0 - R, x0 + TX + R) of NP
// planes into LDS, zero outside the view (and in the row padding).
// Work items of the persistent SSIM kernels: (channel, tile) pairs, item =
// c * ntiles + t.  With a grid of 8k workgroups, XCD x (the workgroups whose
// linear id is x mod 8: the dispatcher places them round-robin) takes the
// x-th of eight contiguous chunks of items and its k workgroups stride
// through it, so the tiles in flight on one XCD are neighbours and share
// their aprons (and row-end cache lines) in its L2.  Other grid sizes stride
// over all items.
struct ItemWalk {
    int first, stride, end;
    __device__ explicit ItemWalk(int nitems) {
        const int G = gridDim.x, b = blockIdx.x;
        if (G >= 8 && (G & 7) == 0) {
            const int chunk = (nitems + 7) / 8, x = b & 7;
            first = x * chunk + (b >> 3);
            stride = G >> 3;
            end = min((x + 1) * chunk, nitems);
        } else {
            first = b;
            stride = G;
            end = nitems;
        }
    }
};

// Staging of one tile in two halves: ssim_load issues every global load of
// the thread into registers (one memory round trip, and in flight while the
// previous tile is filtered), ssim_store writes them to LDS.
constexpr int kSsimN = kSsimIY * kSsimLD, kSsimIT = (kSsimN + kSlamThreads - 1) / kSlamThreads;
template <int NP>
__device__ __forceinline__ void ssim_load(const float* const (&src)[NP], const TileIdx& ti, float (&v)[kSsimIT][NP]) {
#pragma unroll
    for (int it = 0; it < kSsimIT; ++it) {
        const int i = it * kSlamThreads + threadIdx.x;
        const int r = i / kSsimLD, q = i - r * kSsimLD;
        const int gy = ti.y0 - kSsimR + r, gx = ti.x0 - kSsimR + q;
        const bool in = i < kSsimN && q < kSsimIX && gx >= 0 && gx < ti.W && gy >= 0 && gy < ti.H;
        const int64_t o = in ? (int64_t)gy * ti.W + gx : 0;
#pragma unroll
        for (int k = 0; k < NP; ++k) v[it][k] = in ? src[k][o] : 0.0f;
    }
}
template <int NP>
__device__ __forceinline__ void ssim_store(const float (&v)[kSsimIT][NP], float (*dst)[kSsimIY][kSsimLD]) {
#pragma unroll
    for (int it = 0; it < kSsimIT; ++it) {
        const int i = it * kSlamThreads + threadIdx.x;
        if (i < kSsimN) {
            const int r = i / kSsimLD, q = i - r * kSsimLD;
#pragma unroll
            for (int k = 0; k < NP; ++k) dst[k][r][q] = v[it][k];
        }
    }
}

// maps: [3 channels][3 maps][P]: m_mu, m_xx, m_xy, each coef * M(p) * the
// partial derivative of SSIM(p) (coef = -lambda w0 / (3 P_v)).  Persistent:
// each workgroup walks (channel, tile) items (ItemWalk).
__global__ void __launch_bounds__(kSlamThreads) k_ssim_fwd(const float* __restrict__ out,
                                                           const float* __restrict__ rgb_t, int64_t P,
                                                           const gs_view* __restrict__ views, SsimTiles st,
                                                           SsimConst sc, const uint8_t* __restrict__ masks,
                                                           int use_obs, float* __restrict__ maps,
                                                           double* __restrict__ partials) {
    __shared__ __align__(16) float sxy[2][kSsimIY][kSsimLD];  // x, y
    __shared__ __align__(16) float hs[5][kSsimIY][kSsimTX];   // horizontal sums of x, y, xx, yy, xy
    __shared__ double s_red[kSlamThreads / kWave];
    const int tid = threadIdx.x;
    const int ntiles = st.first[st.n_views];
    const ItemWalk iw(3 * ntiles);
    double acc = 0.0;  // sum of lambda w0 / (3 P_v) M(p) (1 - s(p)) over this thread's outputs
    const int q = tid % kSsimTX, r0 = (tid / kSsimTX) * kSsimVY;  // vertical-pass outputs of the thread
    // one tile's global data: staged x, y and M(p) at the thread's outputs
    // (every load of a tile goes out together: the wait for any of them is
    // a wait for all, counts being in order)
    float pre[kSsimIT][2], mkn[kSsimVY];
    auto load_tile = [&](const TileIdx& tl, int ch) {
        const int64_t b = views[tl.v].pixel_offset;
        const float* const src[2] = {out + ch * P + b, rgb_t + ch * P + b};
        ssim_load<2>(src, tl, pre);
        const int gx = tl.x0 + q;
#pragma unroll
        for (int j = 0; j < kSsimVY; ++j) {
            const int gy = tl.y0 + r0 + j;
            // the mask plane is always written, so the load is unconditional
            const bool in = gx < tl.W && gy < tl.H;
            const uint8_t mb = masks[b + (in ? (int64_t)gy * tl.W + gx : 0)];
            mkn[j] = (!use_obs || (mb & 1)) ? 1.0f : 0.0f;
        }
    };
    int it = iw.first;
    int c = it < iw.end ? it / ntiles : 0;
    TileIdx ti = ssim_tile(st, views, it < iw.end ? it - c * ntiles : 0);
    if (it < iw.end) load_tile(ti, c);
    for (; it < iw.end; it += iw.stride) {
        const int64_t base = views[ti.v].pixel_offset;
        __syncthreads();  // the previous tile's readers of sxy and hs are done
        ssim_store<2>(pre, sxy);
        float mk[kSsimVY];
#pragma unroll
        for (int j = 0; j < kSsimVY; ++j) mk[j] = mkn[j];
        __syncthreads();
        // the next item's loads fly while this one is filtered
        const int itn = it + iw.stride;
        const int cn = itn < iw.end ? itn / ntiles : c;
        const TileIdx tin = ssim_tile(st, views, itn < iw.end ? itn - cn * ntiles : 0);
        if (itn < iw.end) load_tile(tin, cn);
        // horizontal: item (row r, outputs h0 .. h0 + HX - 1)
        if (tid < kSsimIY * (kSsimTX / kSsimHX)) {
            const int r = tid / (kSsimTX / kSsimHX), h0 = (tid - r * (kSsimTX / kSsimHX)) * kSsimHX;
            float xv[kSsimHN], yv[kSsimHN];
            lds_row<kSsimHN>(&sxy[0][r][h0], xv);
            lds_row<kSsimHN>(&sxy[1][r][h0], yv);
            float a[5][kSsimHX];
#pragma unroll
            for (int j = 0; j < kSsimHX; ++j)
#pragma unroll
                for (int k = 0; k < 5; ++k) a[k][j] = 0.0f;
#pragma unroll
            for (int i = 0; i < kSsimHX + 2 * kSsimR; ++i) {
                const float x = xv[i], y = yv[i], xx = x * x, yy = y * y, xy = x * y;
#pragma unroll
                for (int j = 0; j < kSsimHX; ++j) {
                    const int tp = i - j;  // tap of input i for output j
                    if (tp >= 0 && tp <= 2 * kSsimR) {
                        const float w = sc.g[tp];
                        a[0][j] = fmaf(w, x, a[0][j]);
                        a[1][j] = fmaf(w, y, a[1][j]);
                        a[2][j] = fmaf(w, xx, a[2][j]);
                        a[3][j] = fmaf(w, yy, a[3][j]);
                        a[4][j] = fmaf(w, xy, a[4][j]);
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < 5; ++k)
#pragma unroll
                for (int j = 0; j < kSsimHX; j += 4)
                    *reinterpret_cast<float4*>(&hs[k][r][h0 + j]) =
                        make_float4(a[k][j], a[k][j + 1], a[k][j + 2], a[k][j + 3]);
        }
        __syncthreads();
        // vertical: column q, output rows r0 .. r0 + VY - 1
        const int gx = ti.x0 + q;
        float m[5][kSsimVY];
#pragma unroll
        for (int j = 0; j < kSsimVY; ++j)
#pragma unroll
            for (int k = 0; k < 5; ++k) m[k][j] = 0.0f;
#pragma unroll
        for (int i = 0; i < kSsimVY + 2 * kSsimR; ++i) {
            float h[5];
#pragma unroll
            for (int k = 0; k < 5; ++k) h[k] = hs[k][r0 + i][q];
#pragma unroll
            for (int j = 0; j < kSsimVY; ++j) {
                const int tp = i - j;
                if (tp >= 0 && tp <= 2 * kSsimR) {
                    const float w = sc.g[tp];
#pragma unroll
                    for (int k = 0; k < 5; ++k) m[k][j] = fmaf(w, h[k], m[k][j]);
                }
            }
        }
        const float Pv = (float)((int64_t)ti.W * ti.H);
        const float coef = -sc.lam_w0 / (3.0f * Pv);
        float part = 0.0f;
#pragma unroll
        for (int j = 0; j < kSsimVY; ++j) {
            const int gy = ti.y0 + r0 + j;
            if (gx < ti.W && gy < ti.H) {
                const int64_t p = (int64_t)gy * ti.W + gx;
                const float mx = m[0][j], my = m[1][j];
                const float vx = m[2][j] - mx * mx, vy = m[3][j] - my * my, cxy = m[4][j] - mx * my;
                const float N1 = 2.0f * mx * my + sc.c1, N2 = 2.0f * cxy + sc.c2;
                const float D1 = mx * mx + my * my + sc.c1, D2 = vx + vy + sc.c2;
                // hardware reciprocals: ~1 ulp, far inside the loss tolerance
                const float iD1 = __builtin_amdgcn_rcpf(D1), iD2 = __builtin_amdgcn_rcpf(D2);
                const float iD12 = iD1 * iD2;
                const float s = N1 * N2 * iD12;
                const float k1 = coef * mk[j];
                // partials of s with the other two windowed sums fixed
                const float d_mu = 2.0f * my * (N2 - N1) * iD12 + 2.0f * mx * s * (iD2 - iD1);
                const float d_xx = -s * iD2;
                const float d_xy = 2.0f * N1 * iD12;
                float* mp = maps + (size_t)(3 * c) * P + base + p;
                mp[0] = k1 * d_mu;
                mp[P] = k1 * d_xx;
                mp[2 * P] = k1 * d_xy;
                part += mk[j] * (1.0f - s);
            }
        }
        acc += (double)part * ((double)sc.lam_w0 / (3.0 * (double)Pv));
        ti = tin;
        c = cn;
    }
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    for (int dd = kWave / 2; dd > 0; dd >>= 1) acc += __shfl_xor(acc, dd, kWave);
    if (lane == 0) s_red[wave] = acc;
    __syncthreads();
    if (tid == 0) {
        double a = 0;
        for (int w = 0; w < kSlamThreads / kWave; ++w) a += s_red[w];
        partials[blockIdx.x] = a;
    }
}

__global__ void __launch_bounds__(kSlamThreads) k_ssim_bwd(const float* __restrict__ out,
                                                           const float* __restrict__ rgb_t, int64_t P,
                                                           const gs_view* __restrict__ views, SsimTiles st,
                                                           SsimConst sc, const float* __restrict__ maps,
                                                           float* __restrict__ grad_out) {
    __shared__ __align__(16) float sm[3][kSsimIY][kSsimLD];
    __shared__ __align__(16) float hs[3][kSsimIY][kSsimTX];
    const int tid = threadIdx.x;
    const int ntiles = st.first[st.n_views];
    const ItemWalk iw(3 * ntiles);
    const int q = tid % kSsimTX, r0 = (tid / kSsimTX) * kSsimVY;  // vertical-pass outputs of the thread
    // one tile's global data: the staged maps, and x, y and the gradient so
    // far at the thread's outputs (loaded together, see k_ssim_fwd)
    float pre[kSsimIT][3], xn[kSsimVY], yn[kSsimVY], gn[kSsimVY];
    auto load_tile = [&](const TileIdx& tl, int ch) {
        const int64_t b = views[tl.v].pixel_offset;
        const float* M = maps + (size_t)(3 * ch) * P + b;
        const float* const src[3] = {M, M + P, M + 2 * P};
        ssim_load<3>(src, tl, pre);
        const int gx = tl.x0 + q;
#pragma unroll
        for (int j = 0; j < kSsimVY; ++j) {
            const int gy = tl.y0 + r0 + j;
            const bool in = gx < tl.W && gy < tl.H;
            const int64_t p = b + (in ? (int64_t)gy * tl.W + gx : 0);
            xn[j] = in ? out[ch * P + p] : 0.0f;
            yn[j] = in ? rgb_t[ch * P + p] : 0.0f;
            gn[j] = in ? grad_out[ch * P + p] : 0.0f;
        }
    };
    int it = iw.first;
    int c = it < iw.end ? it / ntiles : 0;
    TileIdx ti = ssim_tile(st, views, it < iw.end ? it - c * ntiles : 0);
    if (it < iw.end) load_tile(ti, c);
    for (; it < iw.end; it += iw.stride) {
        const int64_t base = views[ti.v].pixel_offset;
        __syncthreads();
        ssim_store<3>(pre, sm);
        float xv[kSsimVY], yv[kSsimVY], gv[kSsimVY];
#pragma unroll
        for (int j = 0; j < kSsimVY; ++j) {
            xv[j] = xn[j];
            yv[j] = yn[j];
            gv[j] = gn[j];
        }
        __syncthreads();
        const int itn = it + iw.stride;
        const int cn = itn < iw.end ? itn / ntiles : c;
        const TileIdx tin = ssim_tile(st, views, itn < iw.end ? itn - cn * ntiles : 0);
        if (itn < iw.end) load_tile(tin, cn);
        if (tid < kSsimIY * (kSsimTX / kSsimHX)) {
            const int r = tid / (kSsimTX / kSsimHX), h0 = (tid - r * (kSsimTX / kSsimHX)) * kSsimHX;
            float a[3][kSsimHX];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                float v[kSsimHN];
                lds_row<kSsimHN>(&sm[k][r][h0], v);
#pragma unroll
                for (int j = 0; j < kSsimHX; ++j) {
                    float acc = 0.0f;
#pragma unroll
                    for (int tp = 0; tp <= 2 * kSsimR; ++tp) acc = fmaf(sc.g[tp], v[j + tp], acc);
                    a[k][j] = acc;
                }
            }
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int j = 0; j < kSsimHX; j += 4)
                    *reinterpret_cast<float4*>(&hs[k][r][h0 + j]) =
                        make_float4(a[k][j], a[k][j + 1], a[k][j + 2], a[k][j + 3]);
        }
        __syncthreads();
        const int gx = ti.x0 + q;
        float b[3][kSsimVY];
#pragma unroll
        for (int j = 0; j < kSsimVY; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k) b[k][j] = 0.0f;
#pragma unroll
        for (int i = 0; i < kSsimVY + 2 * kSsimR; ++i) {
            float h[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) h[k] = hs[k][r0 + i][q];
#pragma unroll
            for (int j = 0; j < kSsimVY; ++j) {
                const int tp = i - j;
                if (tp >= 0 && tp <= 2 * kSsimR) {
#pragma unroll
                    for (int k = 0; k < 3; ++k) b[k][j] = fmaf(sc.g[tp], h[k], b[k][j]);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < kSsimVY; ++j) {
            const int gy = ti.y0 + r0 + j;
            if (gx < ti.W && gy < ti.H) {
                const int64_t p = base + (int64_t)gy * ti.W + gx;
                grad_out[c * P + p] = gv[j] + (b[0][j] + 2.0f * xv[j] * b[1][j] + yv[j] * b[2][j]);
            }
        }
        ti = tin;
        c = cn;
    }
}

// One row more of a vertical window: returns the window that ends with h,
// part[k] the sum of the one that ends k + 1 rows later.  (The shift is the
// FMA's own, no ring and no moves.)
__device__ __forceinline__ float window_row(const SsimConst& sc, float h, float (&part)[2 * kSsimR]) {
    const float done = fmaf(sc.g[2 * kSsimR], h, part[0]);
#pragma unroll
    for (int k = 0; k < 2 * kSsimR - 1; ++k) part[k] = fmaf(sc.g[2 * kSsimR - 1 - k], h, part[k + 1]);
    part[2 * kSsimR - 1] = sc.g[0] * h;
    return done;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kSsimK = 7;  // steps of four inputs that hold the 26 of 16 outputs

// Horizontal windows of Q planes, R rows and the wavefront's 64 columns:
// o[q][i] that of plane q, row i and the lane's column.  Per plane and four
// rows one 16x16 product with the banded matrix of the weights (`band`: tap
// 4 s + lane / 16 - lane % 16), whose 16 rows are the four of each 16 columns,
// so that a lane's four results are its own column's.  With rows 4 times an
// odd number of words apart the 64 lanes of a read are on the 64 banks.
// The zeros of the band would turn an infinity or a NaN into NaNs outside
// its window: with `finite` false the windows are summed tap by tap.
template <int Q, int R, int LD>
__device__ __forceinline__ void window_cols(const SsimConst& sc, const float (*s_f)[R][LD],
                                            const float (&band)[kSsimK], bool finite, float (&o)[Q][R]) {
    static_assert(LD % 8 == 4, "no bank conflicts");
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const float* src = &s_f[0][0][kSsimPad - kSsimR];
    if (finite) {
        const float* a = src + (lane & 3) * LD + wave * kWave + (lane & 12) * 4 + (lane >> 4);
        f32x4 d[Q][R / 4];
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int g = 0; g < R / 4; ++g) d[q][g] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < kSsimK; ++s)
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int g = 0; g < R / 4; ++g)
                    d[q][g] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[(q * R + 4 * g) * LD + 4 * s], band[s], d[q][g], 0,
                                                                   0, 0);
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int i = 0; i < R; ++i) o[q][i] = d[q][i / 4][i % 4];
    } else {
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int i = 0; i < R; ++i) o[q][i] = 0.0f;
#pragma unroll 1
        for (int tp = 0; tp <= 2 * kSsimR; ++tp)
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int i = 0; i < R; ++i)
                    o[q][i] = fmaf(sc.g[tp], src[(q * R + i) * LD + threadIdx.x + tp], o[q][i]);
    }
}

// SSIM of one strip of one channel: the loss and its gradient, added to
// grad_out.  A workgroup of BW threads takes BW columns, one a thread, of which
// the middle BW - 20 are its own, and walks down pl.rows output rows in steps
// of R input rows:
//   1. x, y, x^2 + y^2 and xy of the new rows, x and y less 1/2, through the
//      vertical window (partial sums in registers), to LDS;
//   2. their horizontal windows (MFMA), SSIM and its derivatives with respect
//      to the windowed sums x, x^2 + y^2 and xy, scaled by coef M(p) (coef =
//      -lambda w0 / (3 P_v)), to LDS;
//   3. the horizontal windows of those three maps, their vertical windows, and
//      grad += B_mu + 2 x B_xx + y B_xy (the window is symmetric, so the
//      adjoint is the same filter).
// Step t's new rows complete windows 5 rows up and gradients 10 rows up.
// Bound by instruction issue and, at three wavefronts a SIMD, the latency of a
// step's two barriers: 164 vector instructions a row of 64 columns, 11 of them
// MFMA and 77 the four vertical and three adjoint windows, which take 142 us to
// issue, and MFMA busy 34 % of the time; with the
// horizontal windows on the vector unit too it took 325 us for eight 1200x680
// views (register and LDS use left two wavefronts a SIMD), now 245, and the
// two tile kernels, which move 9 maps of every pixel through memory, 354.
template <int BW, int R>
__global__ void __launch_bounds__(BW) __attribute__((amdgpu_waves_per_eu(3)))
k_ssim(const float* __restrict__ out, const float* __restrict__ rgb_t, int64_t P, const gs_view* __restrict__ views,
       SsimStrips pl, SsimConst sc, const uint8_t* __restrict__ masks, int use_obs, float* __restrict__ grad_out,
       double* __restrict__ partials) {
    constexpr int LD = BW + 2 * kSsimPad + 4;  // column c at kSsimPad + c
    __shared__ float s_f[7][R][LD];
    __shared__ double s_red[BW / kWave];
    __shared__ int s_bad[2][2];  // [step's parity]: a sum, a map of the step is not finite
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    int v = 0;
    while (v + 1 < pl.n_views && pl.first[v + 1] <= (int)blockIdx.x) ++v;
    const int W = views[v].width, H = views[v].height;
    const int64_t base = views[v].pixel_offset;
    const int nx = ceil_div(W, BW - 4 * kSsimR);
    int lt = blockIdx.x - pl.first[v];
    const int x0 = lt % nx * (BW - 4 * kSsimR);
    lt /= nx;
    const int c = lt % 3, y0 = lt / 3 * pl.rows, y1 = min(y0 + pl.rows, H);
    const float* X = out + c * P + base;
    const float* Y = rgb_t + c * P + base;
    float* G = grad_out + c * P + base;
    const uint8_t* M = masks + base;
    const int gx = x0 - 2 * kSsimR + tid;
    const bool col_in = gx >= 0 && gx < W, col_own = col_in && tid >= 2 * kSsimR && tid < BW - 2 * kSsimR;
    const int gxc = col_in ? gx : 0;
    float band[kSsimK];
#pragma unroll
    for (int s = 0; s < kSsimK; ++s) {
        const int tp = 4 * s + (lane >> 4) - (lane & 15);
        band[s] = 0.0f;
#pragma unroll
        for (int k = 0; k <= 2 * kSsimR; ++k) band[s] = tp == k ? sc.g[k] : band[s];
    }
    for (int k = tid; k < 7 * R * 2 * kSsimPad; k += BW) {  // the columns outside the block: zeros
        const int e = k % (2 * kSsimPad);
        s_f[k / (2 * kSsimPad) / R][k / (2 * kSsimPad) % R][e < kSsimPad ? e : BW + e] = 0.0f;
    }
    if (tid < 4) s_bad[tid >> 1][tid & 1] = 0;
    __syncthreads();
    const float Pv = (float)((int64_t)W * H);
    const float coef = -sc.lam_w0 / (3.0f * Pv);
    const int steps = ceil_div(y1 - y0 + 4 * kSsimR, R);

    // the row's offset, rows outside the view at its edge (loaded, not used)
    auto row = [&](int r) { return (int64_t)(r < 0 ? 0 : (r < H ? r : H - 1)) * W; };
    float xn[R], yn[R];
    auto load_rows = [&](int t) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int64_t o = row(y0 - 2 * kSsimR + t * R + i);
            xn[i] = (X + o)[gxc];
            yn[i] = (Y + o)[gxc];
        }
    };
    load_rows(0);
    float va[4][2 * kSsimR], vb[3][2 * kSsimR];
#pragma unroll
    for (int k = 0; k < 2 * kSsimR; ++k) {
#pragma unroll
        for (int q = 0; q < 4; ++q) va[q][k] = 0.0f;
#pragma unroll
        for (int q = 0; q < 3; ++q) vb[q][k] = 0.0f;
    }
    double acc = 0.0;  // sum of M(p) (1 - s(p)) over the block's own pixels
    for (int t = 0; t < steps; ++t) {
        const int r0 = y0 - 2 * kSsimR + t * R;  // first of the new rows
        bool bad = false;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const bool in = col_in && r0 + i >= 0 && r0 + i < H;
            const float x = in ? xn[i] - kSsimMid : -kSsimMid, y = in ? yn[i] - kSsimMid : -kSsimMid;
            const float sq = window_row(sc, fmaf(x, x, y * y), va[2]);
            s_f[0][i][kSsimPad + tid] = window_row(sc, x, va[0]);
            s_f[1][i][kSsimPad + tid] = window_row(sc, y, va[1]);
            s_f[2][i][kSsimPad + tid] = sq;
            s_f[3][i][kSsimPad + tid] = window_row(sc, x * y, va[3]);
            bad |= !(sq < INFINITY);
        }
        if (t + 1 < steps) load_rows(t + 1);  // in flight while this step is filtered
        if ((t + 1) * R <= 2 * kSsimR) continue;  // windows that no gradient of the strip needs
        // x, y and the gradient so far at the rows that this step completes
        const bool done = (t + 1) * R > 4 * kSsimR;
        float xo[R], yo[R], go[R];
        if (done) {
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const int64_t o = row(r0 - 2 * kSsimR + i);
                xo[i] = (X + o)[gxc];
                yo[i] = (Y + o)[gxc];
                go[i] = (G + o)[gxc];
            }
        }
        int mn[R];
        if (use_obs) {
#pragma unroll
            for (int i = 0; i < R; ++i) mn[i] = (M + row(r0 - kSsimR + i))[gxc];
        }
        if (__any(bad)) s_bad[t & 1][0] = 1;
        __syncthreads();
        if (tid < 2) s_bad[(t + 1) & 1][tid] = 0;  // read before this barrier, written after the next one
        {
            const bool finite = s_bad[t & 1][0] == 0;
            float f[4][R], part = 0.0f;
            window_cols(sc, s_f, band, finite, f);
            bad = false;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const int m = r0 - kSsimR + i;
                const float ux = f[0][i], uy = f[1][i], mx = ux + kSsimMid, my = uy + kSsimMid;
                // differences of nearly equal numbers: the products unrounded
                const float vs = fmaf(-uy, uy, fmaf(-ux, ux, f[2][i])), cxy = fmaf(-ux, uy, f[3][i]);
                const float N1 = 2.0f * (mx * my) + sc.c1, N2 = 2.0f * cxy + sc.c2;
                const float D1 = (mx * mx + my * my) + sc.c1, D2 = vs + sc.c2;
                // hardware reciprocals: ~1 ulp, far inside the loss tolerance
                const float iD1 = __builtin_amdgcn_rcpf(D1), iD2 = __builtin_amdgcn_rcpf(D2);
                const float iD12 = iD1 * iD2;
                const float s = N1 * N2 * iD12;
                const float mk = !use_obs || (mn[i] & 1) ? 1.0f : 0.0f, k1 = coef * mk;
                const bool in = col_in && m >= 0 && m < H;
                // partials of s with the other windowed sums fixed
                const float d_mu = 2.0f * (my * N2 - uy * N1) * iD12 + 2.0f * s * (ux * iD2 - mx * iD1);
                const float d_xx = -s * iD2;
                const float d_xy = 2.0f * N1 * iD12;
                part += col_own && m >= y0 && m < y1 ? mk * (1.0f - s) : 0.0f;
                const float m0 = in ? k1 * d_mu : 0.0f, m1 = in ? k1 * d_xx : 0.0f, m2 = in ? k1 * d_xy : 0.0f;
                bad |= !(fabsf(m0) + fabsf(m1) + fabsf(m2) < INFINITY);
                s_f[4][i][kSsimPad + tid] = m0;
                s_f[5][i][kSsimPad + tid] = m1;
                s_f[6][i][kSsimPad + tid] = m2;
            }
            acc += (double)part;
            if (__any(bad)) s_bad[t & 1][1] = 1;
        }
        __syncthreads();
        {
            const bool finite = s_bad[t & 1][1] == 0;
            float b[3][R];
            window_cols(sc, s_f + 4, band, finite, b);
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int i = 0; i < R; ++i) b[k][i] = window_row(sc, b[k][i], vb[k]);
            if (done && col_own) {
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const int r = r0 - 2 * kSsimR + i;
                    if (r >= y0 && r < y1)
                        (G + (int64_t)r * W)[gx] = go[i] + (b[0][i] + 2.0f * (xo[i] - kSsimMid) * b[1][i] + (yo[i] - kSsimMid) * b[2][i]);
                }
            }
        }
    }
    acc *= (double)sc.lam_w0 / (3.0 * (double)Pv);
    for (int d = kWave / 2; d > 0; d >>= 1) acc += __shfl_xor(acc, d, kWave);
    if (lane == 0) s_red[wave] = acc;
    __syncthreads();
    if (tid == 0) {
        double a = 0;
        for (int w = 0; w < BW / kWave; ++w) a += s_red[w];
        partials[blockIdx.x] = a;
    }
}

// ---------------------------------------------------------------------------
// 4. fixed-order sum: loss = (colour L1, SSIM, depth, semantic, total)
// ---------------------------------------------------------------------------
// src: the pixel kernel's (colour, depth, semantic) partials, or their
// first-stage sums, term-major [3][n]; ssim: the SSIM kernel's per-block
// partials.  One block; every sum in a fixed order.
__global__ void __launch_bounds__(kSumLast) k_slam_loss_final(const double* __restrict__ src, int n,
                                                              const double* __restrict__ ssim, int nssim,
                                                              double* __restrict__ loss) {
    __shared__ double s[4][kSumLast / kWave];
    sum_last<3>(src, n, s);
    sum_last<1>(ssim, nssim, s + 3);
    __syncthreads();
    if (threadIdx.x == 0) {
        const double r[4] = {sum_last_total(s[0]), sum_last_total(s[3]), sum_last_total(s[1]), sum_last_total(s[2])};
#pragma unroll
        for (int k = 0; k < 4; ++k) loss[k] = r[k];
        loss[4] = ((r[0] + r[1]) + r[2]) + r[3];
    }
}

// ---------------------------------------------------------------------------
// workspace
// ---------------------------------------------------------------------------
size_t align256(size_t b) { return (b + 255) / 256 * 256; }

// Pixel-kernel grid: one thread per pixel.
unsigned slam_blocks(int64_t P) { return (unsigned)((P + kSlamThreads - 1) / kSlamThreads); }

struct SlamWs {
    size_t hist, sel, med, vws, part, spart, stage, wt, mask, maps, dpart, dstage, total;
};

int ssim_tiles(const gs_view* views, int n_views, SsimTiles* st) {
    int t = 0;
    for (int v = 0; v < n_views; ++v) {
        if (st) st->first[v] = t;
        t += ceil_div(views[v].width, kSsimTX) * ceil_div(views[v].height, kSsimTY);
    }
    if (st) {
        st->first[n_views] = t;
        st->n_views = n_views;
    }
    return t;
}

int strip_blocks(const gs_view* views, int n_views, int rows, SsimStrips* pl) {
    int t = 0;
    for (int v = 0; v < n_views; ++v) {
        if (pl) pl->first[v] = t;
        t += 3 * ceil_div(views[v].width, kStripBW - 4 * kSsimR) * ceil_div(views[v].height, rows);
    }
    if (pl) {
        pl->first[n_views] = t;
        pl->n_views = n_views;
        pl->rows = rows;
    }
    return t;
}

// Output rows of a strip, or 0: the tiles (k_ssim_fwd, k_ssim_bwd), whichever
// takes less time by their measured rates.  Tiles: 17.2 ns for each (channel,
// tile) item, 6 us besides.  Strips: rows + 20 rows are filtered in steps of
// four, whose time depends on the workgroups that share a CU (three at most):
// 3.05, 4.2 and 5.35 us; more workgroups than that follow at the same rate, the
// last of them 0.8 us a step late.  Against 129 measured shapes, 1 to 24 views
// of 30x3000 to 1920x1080, the choice takes 0.8 % longer than the best of tiles
// and strips of 24, 40, 56 and 72 rows, at most 13 % (by the number of strips
// alone 11 % and 2.2 times: views that are not nearly whole strips wide do
// strips' work for columns that are not there).  Both in us, SSIM of both
// directions, tiles/strips: 320x240 11/33, 1200x680 49/47 (estimated 48/58:
// tiles), four 640x480 70/59, eight 1200x680 335/248, 256x256 x 12 49/64,
// 30x3000 x 8 84/170.
int strip_rows(const gs_view* views, int n_views) {
    constexpr int CUS = 256;
    double best = 6.0 + 0.0172 * 3 * ssim_tiles(views, n_views, nullptr);
    int height = 0, choice = 0;
    for (int v = 0; v < n_views; ++v) height = views[v].height > height ? views[v].height : height;
    for (int rows = 24; rows <= 72; rows += 16) {
        const int n = strip_blocks(views, n_views, rows, nullptr);
        const int steps = ceil_div((rows < height ? rows : height) + 4 * kSsimR, kStripR);
        const double step = n <= CUS ? 3.05 : (n <= 2 * CUS ? 4.2 : (n <= 3 * CUS ? 5.35 : n * 5.35 / (3 * CUS) + 0.8));
        if (steps * step < best) {
            best = steps * step;
            choice = rows;
        }
    }
    return choice;
}

// Decoder-gradient reduction: the pixel kernel's block partials, block-major
// [nblk][T] floats (T = F K + K), are summed in fixed order by chunks of
// kRowChunk rows (k_rows_stage, doubles [nchunk][T]), then over the chunks
// (k_rows_final).
constexpr int kRowChunk = 512;
int row_chunks(int64_t nblk) { return (int)((nblk + kRowChunk - 1) / kRowChunk); }

SlamWs slam_layout(int64_t P, const gs_view* views, int n_views, bool ssim, int dec_terms) {
    SlamWs L;
    size_t o = 0;
    L.hist = o;
    o += (size_t)n_views * kMedWords * 4;  // a multiple of 256
    L.sel = o;
    o += align256((size_t)n_views * 2 * sizeof(MedSel));
    L.med = o;
    o += align256((size_t)n_views * 4);
    L.vws = o;
    o += align256((size_t)n_views * sizeof(ViewWeights));
    const int64_t nblk = slam_blocks(P);
    L.part = o;
    o += align256((size_t)nblk * 3 * 8);
    // one partial per SSIM workgroup: of tiles at most three times their number
    // rounded up to 8, of strips (larger than a tile either way) fewer; the
    // maps of the tiles also where a call takes strips, so that a workspace
    // sized for many views serves fewer
    const int nt = ssim ? ssim_tiles(views, n_views, nullptr) : 0;
    L.spart = o;
    o += align256((size_t)(3 * nt + 8) * 8);
    L.stage = o;
    o += align256((size_t)sum_stage_blocks(nblk) * 3 * 8);
    L.wt = o;
    o += align256((size_t)kWtFloats * 4);
    L.mask = o;
    o += align256((size_t)P);
    L.maps = o;
    if (ssim) o += align256((size_t)9 * P * 4);
    L.dpart = o;
    o += align256((size_t)nblk * dec_terms * 4);
    L.dstage = o;
    o += align256((size_t)row_chunks(nblk) * dec_terms * 8);
    L.total = o;
    return L;
}

// block (c, g): column t = 64 g + lane of rows [c kRowChunk, (c + 1) kRowChunk);
// wavefront w takes rows w, w + 4, ... of the chunk, the four sums added in
// order.
__global__ void __launch_bounds__(256) k_rows_stage(const float* __restrict__ src, int64_t nrows, int T,
                                                    double* __restrict__ dst) {
    __shared__ double s[4][kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int t = blockIdx.y * kWave + lane;
    const int64_t r0 = (int64_t)blockIdx.x * kRowChunk;
    double acc = 0.0;
    if (t < T) {
        constexpr int U = 16;
        for (int j0 = 0; j0 < kRowChunk / 4; j0 += U) {
            float x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t r = r0 + wave + 4 * (j0 + u);
                x[u] = src[(r < nrows ? r : nrows - 1) * T + t];
                x[u] = r < nrows ? x[u] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) acc += (double)x[u];
        }
    }
    s[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && t < T) dst[(size_t)blockIdx.x * T + t] = ((s[0][lane] + s[1][lane]) + s[2][lane]) + s[3][lane];
}

__global__ void __launch_bounds__(256) k_rows_final(const double* __restrict__ stage, int nchunk, int F, int K,
                                                    float* __restrict__ grad_w, float* __restrict__ grad_b) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int T = F * K + K;
    if (t >= T) return;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;  // four chains, fixed order
    int c = 0;
    for (; c + 3 < nchunk; c += 4) {
        a0 += stage[(size_t)c * T + t];
        a1 += stage[(size_t)(c + 1) * T + t];
        a2 += stage[(size_t)(c + 2) * T + t];
        a3 += stage[(size_t)(c + 3) * T + t];
    }
    for (; c < nchunk; ++c) a0 += stage[(size_t)c * T + t];
    const double a = (a0 + a1) + (a2 + a3);
    if (t < F * K) {
        if (grad_w != nullptr) grad_w[t] = (float)a;
    } else if (grad_b != nullptr) {
        grad_b[t - F * K] = (float)a;
    }
}

// Workgroups of kSlamThreads that are resident on the device at once.
unsigned resident_blocks(const void* kern, size_t lds) {
    int dev = 0, cus = 0, per_cu = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kSlamThreads, lds);
    return (unsigned)((cus > 1 ? cus : 1) * (per_cu > 1 ? per_cu : 1));
}

// Workgroups of a persistent SSIM launch: the resident ones, rounded down to
// a multiple of the 8 XCDs (ItemWalk), at least 8, at most the items rounded
// up to 8.
unsigned ssim_grid(const void* kern, int nitems) {
    int g = (int)resident_blocks(kern, 0) / 8 * 8;
    const int cap = (nitems + 7) / 8 * 8;
    if (g > cap) g = cap;
    return (unsigned)(g >= 8 ? g : 8);
}

template <int F, int KC>
void launch_slam_pixels(unsigned nblk, hipStream_t s, const float* out, int64_t P, const float* rgb_t,
                        const float* depth_t, const int32_t* labels, const float* Wt, const float* bias, int K,
                        const SlamParams& sp, const float* med, const ViewWeights* vws, const gs_view* views, int n_views,
                        float* grad_out, uint8_t* masks, double* partials) {
    auto kern = sp.bce ? k_slam_loss<F, KC, true> : k_slam_loss<F, KC, false>;
    hipLaunchKernelGGL(kern, dim3(nblk), dim3(kSlamThreads), 0, s, out, P, rgb_t, depth_t, labels, Wt, bias, K, sp,
                       med, vws, views, n_views, grad_out, masks, partials);
}

// With the decoder gradients: as many workgroups as are resident at once (at
// most one per 256 pixels, for which the partials have room).
template <int F, int NT>
unsigned launch_slam_pixels_dec(hipStream_t s, const float* out, int64_t P, const float* rgb_t, const float* depth_t,
                                const int32_t* labels, const float* Wt, int K, const SlamParams& sp, const float* med,
                                const ViewWeights* vws, const gs_view* views, int n_views, float* grad_out, uint8_t* masks, double* partials,
                                float* dec_partials) {
    auto kern = sp.bce ? k_slam_loss_dec<F, NT, true> : k_slam_loss_dec<F, NT, false>;
    const size_t lds = dec_lds_bytes(F, K);
    const unsigned fit = resident_blocks(reinterpret_cast<const void*>(kern), lds), most = slam_blocks(P);
    const unsigned nblk = fit < most ? fit : most;
    hipLaunchKernelGGL(kern, dim3(nblk), dim3(kSlamThreads), lds, s, out, P, rgb_t, depth_t, labels, Wt, K, sp,
                       med, vws, views, n_views, grad_out, masks, partials, dec_partials);
    return nblk;
}

int dec_terms_of(int F, const gs_decoder* dec) {
    if (dec == nullptr || F == 0 || dec->n_classes == 0) return 0;
    if (dec->grad_weight == nullptr && dec->grad_bias == nullptr) return 0;
    return F * dec->n_classes + dec->n_classes;
}

template <int F>
hipError_t launch_slam_t(const float* out, const float* rgb_t, const float* depth_t, const int32_t* labels,
                         const gs_decoder* dec, const gs_slam_loss_opts& o, const gs_view* views_host,
                         const gs_view* views_dev, int n_views, int64_t P, float* grad_out, double* loss,
                         float* median, uint8_t* masks, char* ws, hipStream_t s) {
    const bool ssim = o.ssim_lambda != 0.0f;
    const int dterms = dec_terms_of(F, dec);
    const SlamWs L = slam_layout(P, views_host, n_views, ssim, dterms);
    uint32_t* hist = reinterpret_cast<uint32_t*>(ws + L.hist);
    MedSel* sel = reinterpret_cast<MedSel*>(ws + L.sel);
    float* med = reinterpret_cast<float*>(ws + L.med);
    double* part = reinterpret_cast<double*>(ws + L.part);
    double* spart = reinterpret_cast<double*>(ws + L.spart);
    float* Wt = reinterpret_cast<float*>(ws + L.wt);
    ViewWeights* vws = reinterpret_cast<ViewWeights*>(ws + L.vws);
    uint8_t* mk = masks != nullptr ? masks : reinterpret_cast<uint8_t*>(ws + L.mask);
    float* maps = reinterpret_cast<float*>(ws + L.maps);
    float* dpart = dterms > 0 ? reinterpret_cast<float*>(ws + L.dpart) : nullptr;
    double* dstage = reinterpret_cast<double*>(ws + L.dstage);

    // 1. median depth error per view
    SlamParams sp;
    sp.w0 = o.w_color;
    sp.w1 = o.w_depth;
    sp.w2 = o.w_sem;
    sp.lam = o.ssim_lambda;
    sp.tau_obs = o.tau_obs;
    sp.tau_unobs = o.tau_unobs;
    sp.obs_factor = o.obs_factor;
    sp.unobs_factor = o.unobs_factor;
    sp.use_obs = (o.flags & GS_LOSS_OBS_MASK) != 0;
    sp.bce = (o.flags & GS_LOSS_BCE) != 0;
    const int K = dec != nullptr ? dec->n_classes : 0;
    const bool sem = F > 0 && K > 0 && o.w_sem != 0.0f;
    const int words = n_views * kMedWords;
    const int wt = F * ((K + 3) / 4 * 4), prep = sem && wt > words ? wt : words;
    hipLaunchKernelGGL(k_slam_prep, dim3((unsigned)ceil_div(prep, 256)), dim3(256), 0, s, hist, words,
                       sem ? dec->weight : nullptr, sem ? dec->bias : nullptr, F, K, Wt, views_dev, n_views, sp, vws);
    int64_t pmax = 0;
    for (int v = 0; v < n_views; ++v) {
        const int64_t pv = (int64_t)views_host[v].width * views_host[v].height;
        pmax = pv > pmax ? pv : pmax;
    }
    const dim3 hg((unsigned)((pmax + kMedChunk - 1) / kMedChunk), (unsigned)n_views);
    const float* dep = out + 3 * P;
    hipLaunchKernelGGL(k_median<0>, hg, dim3(kSlamThreads), 0, s, dep, depth_t, views_dev, hist, sel);
    hipLaunchKernelGGL(k_median<1>, hg, dim3(kSlamThreads), 0, s, dep, depth_t, views_dev, hist, sel);
    hipLaunchKernelGGL(k_median<2>, hg, dim3(kSlamThreads), 0, s, dep, depth_t, views_dev, hist, sel);
    hipLaunchKernelGGL(k_median_final, dim3(n_views), dim3(kSlamThreads), 0, s, hist, sel, med, median);

    // 2. masks, L1 and the semantic term (with the decoder gradients' block partials)
    unsigned nblk = slam_blocks(P);
    const int Ke = sem ? K : 0;
    const float* bias = sem ? dec->bias : nullptr;
    if constexpr (F > 0) {
        if (sem && dterms > 0) {
            auto go = Ke > 32 ? launch_slam_pixels_dec<F, 4>
                              : (Ke > 16 ? launch_slam_pixels_dec<F, 2> : launch_slam_pixels_dec<F, 1>);
            nblk = go(s, out, P, rgb_t, depth_t, labels, Wt, Ke, sp, med, vws, views_dev, n_views, grad_out, mk, part,
                      dpart);
        }
    }
    if (!(sem && dterms > 0)) {
        auto go = Ke > 32 ? launch_slam_pixels<F, 64> : launch_slam_pixels<F, 32>;
        go(nblk, s, out, P, rgb_t, depth_t, labels, Wt, bias, Ke, sp, med, vws, views_dev, n_views, grad_out, mk, part);
    }
    if (dterms > 0) {
        // dL/dW and dL/db (zero when the semantic term is off)
        if (!sem) {
            const hipError_t e = fill_u32(reinterpret_cast<uint32_t*>(dpart), 0u, (int64_t)nblk * dterms, s);
            if (e != hipSuccess) return e;
        }
        const int nch = row_chunks(nblk);
        hipLaunchKernelGGL(k_rows_stage, dim3((unsigned)nch, (unsigned)ceil_div(dterms, kWave)), dim3(256), 0, s,
                           dpart, (int64_t)nblk, dterms, dstage);
        hipLaunchKernelGGL(k_rows_final, dim3((unsigned)ceil_div(dterms, 256)), dim3(256), 0, s, dstage, nch, F,
                           dec->n_classes, dec->grad_weight, dec->grad_bias);
    }

    // 3. SSIM
    int nssim = 0;
    if (ssim) {
        SsimConst sc;
        double g[2 * kSsimR + 1], tot = 0.0;
        for (int t = 0; t <= 2 * kSsimR; ++t) {
            const double d = t - kSsimR;
            g[t] = exp(-d * d / (2.0 * 1.5 * 1.5));
            tot += g[t];
        }
        for (int t = 0; t <= 2 * kSsimR; ++t) sc.g[t] = (float)(g[t] / tot);
        sc.c1 = (float)(0.01 * 0.01);
        sc.c2 = (float)(0.03 * 0.03);
        sc.lam_w0 = o.ssim_lambda * o.w_color;
        const int rows = strip_rows(views_host, n_views);
        if (rows > 0) {
            SsimStrips pl;
            nssim = strip_blocks(views_host, n_views, rows, &pl);
            hipLaunchKernelGGL((k_ssim<kStripBW, kStripR>), dim3((unsigned)nssim), dim3(kStripBW), 0, s, out, rgb_t, P,
                               views_dev, pl, sc, mk, sp.use_obs, grad_out, spart);
        } else {
            SsimTiles st;
            const int nt = ssim_tiles(views_host, n_views, &st);
            // persistent grids walking the (channel, tile) items
            const unsigned gf = ssim_grid(reinterpret_cast<const void*>(&k_ssim_fwd), 3 * nt);
            const unsigned gb = ssim_grid(reinterpret_cast<const void*>(&k_ssim_bwd), 3 * nt);
            if (nt > 0) {
                hipLaunchKernelGGL(k_ssim_fwd, dim3(gf), dim3(kSlamThreads), 0, s, out, rgb_t, P, views_dev, st, sc,
                                   mk, sp.use_obs, maps, spart);
                hipLaunchKernelGGL(k_ssim_bwd, dim3(gb), dim3(kSlamThreads), 0, s, out, rgb_t, P, views_dev, st, sc,
                                   maps, grad_out);
            }
            nssim = nt > 0 ? (int)gf : 0;
        }
    }
    // 4. loss terms: the per-block partials summed in a fixed order, in two
    // stages where there are many
    const double* src = part;
    int nsrc = (int)nblk;
    if (nsrc > kSumOne) {
        double* stage = reinterpret_cast<double*>(ws + L.stage);
        nsrc = sum_stage_blocks(nblk);
        hipLaunchKernelGGL(k_sum_stage, dim3((unsigned)nsrc), dim3(kSumThreads), 0, s, part, (int)nblk, 3, stage);
        src = stage;
    }
    hipLaunchKernelGGL(k_slam_loss_final, dim3(1), dim3(kSumLast), 0, s, src, nsrc, spart, nssim, loss);
    return hipGetLastError();
}

}  // namespace

size_t slam_loss_workspace_bytes(int64_t P, const gs_view* views_host, int n_views, int n_feat,
                                 const gs_decoder* dec, const gs_slam_loss_opts& o) {
    return slam_layout(P, views_host, n_views, o.ssim_lambda != 0.0f, dec_terms_of(n_feat, dec)).total;
}

hipError_t launch_slam_loss(const float* out, int n_feat, const float* rgb_t, const float* depth_t,
                            const int32_t* labels, const gs_decoder* dec, const gs_slam_loss_opts& o,
                            const gs_view* views_host, const gs_view* views_dev, int n_views, int64_t P,
                            float* grad_out, double* loss, float* median, uint8_t* masks, void* ws, hipStream_t s) {
    char* w = static_cast<char*>(ws);
    switch (n_feat) {
        case 0:
            return launch_slam_t<0>(out, rgb_t, depth_t, labels, dec, o, views_host, views_dev, n_views, P, grad_out,
                                    loss, median, masks, w, s);
        case 8:
            return launch_slam_t<8>(out, rgb_t, depth_t, labels, dec, o, views_host, views_dev, n_views, P, grad_out,
                                    loss, median, masks, w, s);
        case 32:
            return launch_slam_t<32>(out, rgb_t, depth_t, labels, dec, o, views_host, views_dev, n_views, P, grad_out,
                                     loss, median, masks, w, s);
        default:
            return launch_slam_t<16>(out, rgb_t, depth_t, labels, dec, o, views_host, views_dev, n_views, P,
                                     grad_out, loss, median, masks, w, s);
    }
}

}  // namespace sgs
