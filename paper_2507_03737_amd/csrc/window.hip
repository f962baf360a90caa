// Window management and regularisation around the mapping iteration:
//   - the isotropic regulariser of Eq. 16 (Sec. 3.3.3) and its gradient;
//   - keyframe covisibility, IOU and overlap coefficient of the visible Gaussian sets
//     (supplementary Eq. S1-S2), from the contributing-record marks of a forward;
//   - the median positive depth of each view (the median pointmap depth of the keyframe
//     rule), by radix selection on the float bits.
#include <algorithm>

#include "gspm_common.h"

namespace gspm {

namespace {

constexpr int kIsoBlock = 256;

// Eq. 16 per Gaussian, in float64: s = exp(log_scale), m = mean(s),
// loss = sum_k |s_k - m|, d loss / d log s_k = (sgn(s_k - m) - sum_j sgn(s_j - m) / 3) s_k.
__global__ void __launch_bounds__(kIsoBlock)
k_iso_loss(const float *__restrict__ ls, int64_t n, double weight, double *__restrict__ part,
           float *__restrict__ grad) {
    __shared__ double lds[kIsoBlock / kWave];
    double acc = 0.0;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n; g += (int64_t)gridDim.x * blockDim.x) {
        const double s0 = exp((double)ls[g]), s1 = exp((double)ls[n + g]), s2 = exp((double)ls[2 * n + g]);
        const double m = (s0 + s1 + s2) / 3.0;
        const double r0 = s0 - m, r1 = s1 - m, r2 = s2 - m;
        const double g0 = (r0 > 0.0) - (r0 < 0.0), g1 = (r1 > 0.0) - (r1 < 0.0), g2 = (r2 > 0.0) - (r2 < 0.0);
        acc += fabs(r0) + fabs(r1) + fabs(r2);
        if (grad) {
            const double c = (g0 + g1 + g2) / 3.0;
            grad[g] += (float)(weight * (g0 - c) * s0);
            grad[n + g] += (float)(weight * (g1 - c) * s1);
            grad[2 * n + g] += (float)(weight * (g2 - c) * s2);
        }
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane_id() == 0) lds[threadIdx.x / kWave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kIsoBlock / kWave; ++w) t += lds[w];
        part[blockIdx.x] = t;
    }
}

__global__ void __launch_bounds__(256)
k_sum_parts(const double *__restrict__ part, int nb, double weight, float *__restrict__ out) {
    __shared__ double lds[4];
    double acc = 0.0;
    for (int b = threadIdx.x; b < nb; b += blockDim.x) acc += part[b];
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane_id() == 0) lds[threadIdx.x / kWave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = (float)(weight * (lds[0] + lds[1] + lds[2] + lds[3]));
}

// Pairwise counts |G_i and G_j| (i <= j) of the visible sets; the diagonal is |G_i|.
__global__ void __launch_bounds__(256)
k_covis_count(const uint8_t *__restrict__ visible, int64_t n, int V, unsigned long long *__restrict__ counts) {
    __shared__ uint32_t lds[kMaxViews * kMaxViews];
    for (int k = threadIdx.x; k < V * V; k += blockDim.x) lds[k] = 0u;
    __syncthreads();
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n; g += (int64_t)gridDim.x * blockDim.x) {
        uint32_t bits = 0u;
        for (int v = 0; v < V; ++v) bits |= visible[(int64_t)v * n + g] ? (1u << v) : 0u;
        for (uint32_t bi = bits; bi; bi &= bi - 1u) {
            const int i = __builtin_ctz(bi);
            for (uint32_t bj = bi; bj; bj &= bj - 1u) atomicAdd(&lds[i * V + __builtin_ctz(bj)], 1u);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < V * V; k += blockDim.x)
        if (lds[k]) atomicAdd(counts + k, (unsigned long long)lds[k]);
}

__global__ void k_covis_finalize(const unsigned long long *__restrict__ counts, int V,
                                 const FrameHeader *__restrict__ hdr, double *__restrict__ iou,
                                 double *__restrict__ oc, int64_t *__restrict__ count_out) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= V * V) return;
    const int i = k / V, j = k % V;
    if (hdr->visible == 0u) {  // the forward did not mark contributing records
        iou[k] = oc[k] = __builtin_nan("");
        if (j == 0 && count_out) count_out[i] = -1;
        return;
    }
    const double ci = (double)counts[i * V + i], cj = (double)counts[j * V + j];
    const double inter = (double)counts[min(i, j) * V + max(i, j)];
    const double uni = ci + cj - inter, lo = fmin(ci, cj);
    iou[k] = uni > 0.0 ? inter / uni : 0.0;
    oc[k] = lo > 0.0 ? inter / lo : 0.0;
    if (j == 0 && count_out) count_out[i] = (int64_t)ci;
}

// Radix selection of the lower median of the positive depths of each view, 11, 11 and 10 bits
// from the top: positive float bit patterns order like the floats.  Each round is one histogram
// over the pixels, and every workgroup of the next takes the previous round's choice from its
// histogram itself: launches of a few us bound this (2 x 960x640: four rounds of 8 bits with a
// launch for each choice 84 us, 35 us now).
struct MedianState {
    uint32_t prefix;  // bits selected so far
    uint32_t rank;    // rank of the median among the values that match the prefix
    uint32_t n;       // positive values of the view
    uint32_t pad;
};

constexpr int kMedianBits = 11, kMedianBins = 1 << kMedianBits, kMedianRounds = 3;
constexpr int kMedianBlock = 256, kMedianPer = kMedianBins / kMedianBlock, kLeaders = 2;
__host__ __device__ constexpr int median_shift(int round) { return round == 2 ? 0 : 32 - kMedianBits * (round + 1); }

// The state after round `round` from the one before it and the round's histogram, for every lane.
__device__ inline MedianState median_choose(int round, const MedianState *__restrict__ st,
                                            const uint32_t *__restrict__ hist) {
    __shared__ uint32_t waves[kMedianBlock / kWave];
    __shared__ MedianState chosen;
    uint32_t h[kMedianPer], sum = 0u;
#pragma unroll
    for (int k = 0; k < kMedianPer; ++k) {
        h[k] = hist[threadIdx.x * kMedianPer + k];
        sum += h[k];
    }
    const uint32_t inc = wave_inclusive_scan(sum);
    if (lane_id() == kWave - 1) waves[threadIdx.x / kWave] = inc;
    __syncthreads();
    uint32_t below = inc - sum, n = 0u;
#pragma unroll
    for (int w = 0; w < kMedianBlock / kWave; ++w) {
        below += w < (int)(threadIdx.x / kWave) ? waves[w] : 0u;
        n += waves[w];
    }
    MedianState s = {0u, n ? (n - 1u) / 2u : 0u, n, 0u};
    if (round > 0) s = *st;
    if (threadIdx.x == 0) chosen = s;
    __syncthreads();
    if (s.rank >= below && s.rank < below + sum) {  // one lane, if there is a value at all
        s.rank -= below;
        int b = 0;
        while (s.rank >= h[b]) s.rank -= h[b++];
        s.prefix = (s.prefix << (median_shift(round - 1) - median_shift(round))) | (uint32_t)(threadIdx.x * kMedianPer + b);
        chosen = s;
    }
    __syncthreads();
    return chosen;
}

// st, hist: [rounds][views]; the state after round r is written by round r + 1.
__global__ void __launch_bounds__(kMedianBlock)
k_median_hist(ViewTable vt, const float *__restrict__ depth, int round, MedianState *__restrict__ st,
              uint32_t *__restrict__ hist) {
    __shared__ uint32_t h[kMedianBins];
    const int v = blockIdx.y, V = vt.n_views;
    MedianState s = {};
    if (round > 0) {
        const int64_t before = (int64_t)(round - 1) * V + v;
        s = median_choose(round - 1, st + before - V, hist + before * kMedianBins);
        if (blockIdx.x == 0 && threadIdx.x == 0) st[before] = s;
        if (s.n == 0u) return;  // block-uniform
    }
    for (int b = threadIdx.x; b < kMedianBins; b += kMedianBlock) h[b] = 0u;
    __syncthreads();
    const int shift = median_shift(round);
    const uint32_t bins = (1u << (round ? median_shift(round - 1) - shift : kMedianBits)) - 1u;
    const int64_t np = (int64_t)vt.width[v] * vt.height[v];
    const float *d = depth + vt.pix_off[v];
    // Uniform trip count per wave, so the ballots below see every lane.
    const int lane = lane_id();
    for (int64_t e0 = (int64_t)blockIdx.x * blockDim.x; e0 < np; e0 += (int64_t)gridDim.x * blockDim.x) {
        const int64_t e = e0 + threadIdx.x;
        const float x = e < np ? d[e] : 0.0f;
        const uint32_t b = __float_as_uint(x);
        const bool valid = x > 0.0f && (round == 0 || (b >> median_shift(round - 1)) == s.prefix);
        const uint32_t bin = (b >> shift) & bins;
        // Equal bins of a wave would queue at one LDS counter: one atomic for each of the first
        // kLeaders bins met (depths cluster in few top bins; later rounds find one bin where
        // depths are equal), a lane's own for what is left (then spread over many).
        // (16 x 1920x1080: ordinary depths 164 us, one depth 150, 17 decades 152; with an atomic per
        // bin met in the first round and per lane in the others 238, 282 and 634.)
        uint64_t active = ballot(valid);
        for (int l = round ? 1 : kLeaders; l > 0 && active != 0ull; --l) {
            const int leader = (int)__builtin_ctzll(active);
            const uint32_t lb = (uint32_t)__builtin_amdgcn_readlane((int)bin, leader);
            const uint64_t same = ballot(bin == lb) & active;
            if (lane == leader) atomicAdd(&h[lb], (uint32_t)__popcll(same));
            active &= ~same;
        }
        if ((active >> lane) & 1ull) atomicAdd(&h[bin], 1u);
    }
    __syncthreads();
    uint32_t *out = hist + ((int64_t)round * V + v) * kMedianBins;
    for (int b = threadIdx.x; b < kMedianBins; b += kMedianBlock)
        if (h[b]) atomicAdd(out + b, h[b]);
}

__global__ void __launch_bounds__(kMedianBlock)
k_median_finish(const MedianState *__restrict__ st, const uint32_t *__restrict__ hist, float *__restrict__ out) {
    const int v = blockIdx.x, V = gridDim.x;
    const int64_t last = (int64_t)(kMedianRounds - 1) * V + v;
    const MedianState s = median_choose(kMedianRounds - 1, st + last - V, hist + last * kMedianBins);
    if (threadIdx.x == 0) out[v] = s.n ? __uint_as_float(s.prefix) : 0.0f;
}

}  // namespace

int64_t iso_partials() { return 1024; }

hipError_t launch_iso_loss(const float *log_scales, int64_t n, float weight, double *part, float *loss_out,
                           float *grad, hipStream_t s) {
    const int nb = (int)std::min<int64_t>(iso_partials(), std::max<int64_t>(1, (n + kIsoBlock - 1) / kIsoBlock));
    hipLaunchKernelGGL(k_iso_loss, dim3(nb), dim3(kIsoBlock), 0, s, log_scales, n, (double)weight, part, grad);
    hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(256), 0, s, part, nb, (double)weight, loss_out);
    return hipGetLastError();
}

hipError_t launch_covisibility(const uint8_t *visible, int64_t n, int V, const FrameHeader *hdr,
                               unsigned long long *counts, double *iou, double *oc, int64_t *count_out,
                               hipStream_t s) {
    hipError_t e = launch_fill_u32(reinterpret_cast<uint32_t *>(counts), 0u, 2 * (int64_t)V * V, s);
    if (e != hipSuccess) return e;
    if (n > 0) {
        const int64_t nb = std::min<int64_t>(1024, (n + 255) / 256);
        hipLaunchKernelGGL(k_covis_count, dim3((unsigned)nb), dim3(256), 0, s, visible, n, V, counts);
    }
    hipLaunchKernelGGL(k_covis_finalize, dim3((V * V + 255) / 256), dim3(256), 0, s, counts, V, hdr, iou, oc,
                       count_out);
    return hipGetLastError();
}

int64_t median_scratch_words(int V) { return (int64_t)V * kMedianRounds * (kMedianBins + 4); }

hipError_t launch_median_depth(const ViewTable &vt, const float *depth, uint32_t *scratch, float *out,
                               hipStream_t s) {
    const int V = vt.n_views;
    uint32_t *hist = scratch;
    MedianState *st = reinterpret_cast<MedianState *>(scratch + (int64_t)V * kMedianRounds * kMedianBins);
    hipError_t e = launch_fill_u32(hist, 0u, (int64_t)V * kMedianRounds * kMedianBins, s);
    if (e != hipSuccess) return e;
    int64_t maxp = 1;
    for (int v = 0; v < V; ++v) maxp = std::max<int64_t>(maxp, (int64_t)vt.width[v] * vt.height[v]);
    const unsigned bx = (unsigned)std::min<int64_t>(256, (maxp + kMedianBlock - 1) / kMedianBlock);
    for (int round = 0; round < kMedianRounds; ++round)
        hipLaunchKernelGGL(k_median_hist, dim3(bx, V), dim3(kMedianBlock), 0, s, vt, depth, round, st, hist);
    hipLaunchKernelGGL(k_median_finish, dim3(V), dim3(kMedianBlock), 0, s, st, hist, out);
    return hipGetLastError();
}

}  // namespace gspm
