// Patch-based pointmap scale alignment (supplementary Alg. 1, behind Sec. 3.3.1) and
// pointmap replacement (Sec. 3.3.2, Eq. 14).
//
// The per-pixel scalar of a pointmap is its norm |X(x)|.  Alg. 1 rescales the prior as
// X^p_iter = sigma' X^p between iterations; norms, patch means and patch standard
// deviations of X^p_iter are then sigma' times those of X^p, so the normalised values
// (|X| - mu) / sd, and with them the set of correct points of a patch, do not depend on
// sigma'.  Only the patch test (candidate or not) does.  The work therefore splits into:
//   k_align_stats   one pass over the pixels (HBM-bound): per patch the means and
//                   standard deviations of |X^r| and |X^p|, and over the pixels that pass
//                   the normalised test, the sums of |X^r| and |X^p| and their count;
//   k_align_iterate one workgroup per view runs the max_iter iterations over the patch
//                   records: candidates under the current sigma', pooled sums over their
//                   correct points, sigma' = sum|X^r| / sum|X^p| (means over the same set).
// Everything after the float32 loads is float64, in the same formulas as the definition,
// so every discrete decision is taken at float64 precision.
//
// Layout: one wave per strip of floor(64 / P) horizontally adjacent P x P patches (as the
// patch-loss kernel): lane l owns image column x0 + l and walks the strip's P rows.
#include <algorithm>

#include "gspm_common.h"

namespace gspm {

namespace {

constexpr int kAlignBlock = 256;
constexpr int kAlignWaves = kAlignBlock / kWave;

struct AlignStrips {
    int32_t n_views;
    int32_t patch, per_wave;
    int32_t npx[kMaxViews];
    int32_t strips_x[kMaxViews];
    int32_t patch_off[kMaxViews + 1];
    int32_t wave_off[kMaxViews + 1];
};

AlignStrips align_strips(const ViewTable &vt, int patch) {
    AlignStrips st;
    st.n_views = vt.n_views;
    st.patch = patch;
    st.per_wave = kWave / patch;
    st.patch_off[0] = 0;
    st.wave_off[0] = 0;
    for (int v = 0; v < vt.n_views; ++v) {
        const int npx = (vt.width[v] + patch - 1) / patch, npy = (vt.height[v] + patch - 1) / patch;
        st.npx[v] = npx;
        st.strips_x[v] = (npx + st.per_wave - 1) / st.per_wave;
        st.patch_off[v + 1] = st.patch_off[v] + npx * npy;
        st.wave_off[v + 1] = st.wave_off[v] + st.strips_x[v] * npy;
    }
    return st;
}

__device__ inline double norm3(const float *X, int64_t a, int64_t plane) {
    const double x = X[a], y = X[a + plane], z = X[a + 2 * plane];
    return sqrt(x * x + y * y + z * z);
}

// Makes a wave's LDS writes visible to its other lanes.
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Sum of the P column partials of each patch of the strip; lanes < per receive them.  lds is
// the wave's own.
__device__ inline double fold_patch(double x, double *lds, int lane, int P, int per) {
    wave_sync();
    lds[lane] = x;
    wave_sync();
    double t = 0.0;
    if (lane < per)
        for (int k = 0; k < P; ++k) t += lds[lane * P + k];
    return t;
}

// Patch statistics.  The means, the deviations and the normalised test follow one another, so
// every norm is used three times: a lane keeps those of its first 12 rows in registers (four
// waves per SIMD hold that many; taller patches read the rest again).  Reading the pointmaps
// once and taking each root once leaves loads and float64 divisions about equal: 8 views with
// 3.7M pixels, patch 10: 57 us with the rows read three times, 36 us now.
constexpr int kKeepRows = 12, kReadRows = 4;

__global__ void __launch_bounds__(kAlignBlock) __attribute__((amdgpu_waves_per_eu(4)))
k_align_stats(ViewTable vt, AlignStrips st, const float *__restrict__ Xr, const float *__restrict__ Xp,
              const float *__restrict__ mask, double eps_r, AlignPatch *__restrict__ out) {
    __shared__ double lds_all[kAlignWaves][kWave];
    __shared__ double mom_all[kAlignWaves][4][kWave];
    const int lane = lane_id(), wid = threadIdx.x / kWave;
    double *lds = lds_all[wid];
    double(*mom)[kWave] = mom_all[wid];
    const int64_t gw = (int64_t)blockIdx.x * kAlignWaves + wid;
    if (gw >= st.wave_off[st.n_views]) return;  // wave-uniform; no workgroup barrier below
    int v = 0;
    for (int k = 1; k < st.n_views; ++k)
        if (gw >= st.wave_off[k]) v = k;
    const int P = st.patch, per = st.per_wave;
    const int lw = (int)(gw - st.wave_off[v]);
    const int py = lw / st.strips_x[v], sx = lw % st.strips_x[v];
    const int W = vt.width[v], H = vt.height[v];
    const int g = lane / P;                       // patch within the strip
    const int x = sx * per * P + lane;            // image column of this lane
    const bool col = g < per && sx * per + g < st.npx[v] && x < W;
    const int y0 = py * P, rows = col ? min(H, y0 + P) - y0 : 0;
    const int64_t plane = (int64_t)W * H, e0 = (int64_t)y0 * W + x;
    const float *r0 = Xr + 3 * vt.pix_off[v] + e0, *p0 = Xp + 3 * vt.pix_off[v] + e0;
    const float *m0 = mask ? mask + vt.pix_off[v] + e0 : nullptr;

    double nr[kKeepRows], np[kKeepRows];
    uint32_t used = 0u;  // the kept rows that the mask selects
#pragma unroll
    for (int k = 0; k < kKeepRows; ++k) {
        nr[k] = np[k] = 0.0;
        if (k < rows && !(m0 && m0[(int64_t)k * W] == 0.f)) {
            nr[k] = norm3(r0, (int64_t)k * W, plane);
            np[k] = norm3(p0, (int64_t)k * W, plane);
            used |= 1u << k;
        }
    }
    // Calls f(|X^r|, |X^p|) for every selected pixel of the column, top to bottom.  The rows
    // that are not kept are read kReadRows at a time, without a branch around a load (rows past
    // the patch read its last one), so that their latencies overlap.
    auto each = [&](auto f) {
#pragma unroll
        for (int k = 0; k < kKeepRows; ++k)
            if ((used >> k) & 1u) f(nr[k], np[k]);
        for (int k = kKeepRows; k < rows; k += kReadRows) {
            float xr[kReadRows][3], xp[kReadRows][3], m[kReadRows];
#pragma unroll
            for (int q = 0; q < kReadRows; ++q) {
                const int64_t e = (int64_t)min(k + q, rows - 1) * W;
                m[q] = m0 ? m0[e] : 1.0f;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    xr[q][c] = r0[e + c * plane];
                    xp[q][c] = p0[e + c * plane];
                }
            }
#pragma unroll
            for (int q = 0; q < kReadRows; ++q)
                if (k + q < rows && m[q] != 0.f) f(norm3(xr[q], 0, 1), norm3(xp[q], 0, 1));
        }
    };

    // Counts and means.
    double cnt = 0.0, sr = 0.0, sp = 0.0;
    each([&](double a, double b) {
        sr += a;
        sp += b;
        cnt += 1.0;
    });
    const double pc = fold_patch(cnt, lds, lane, P, per);
    const double psr = fold_patch(sr, lds, lane, P, per);
    const double psp = fold_patch(sp, lds, lane, P, per);
    if (lane < per) {
        mom[0][lane] = pc > 0.0 ? psr / pc : 0.0;
        mom[1][lane] = pc > 0.0 ? psp / pc : 0.0;
    }
    wave_sync();
    const double mu_r = (g < per) ? mom[0][g] : 0.0, mu_p = (g < per) ? mom[1][g] : 0.0;

    // Population standard deviations.
    double vr = 0.0, vp = 0.0;
    each([&](double nra, double npb) {
        const double a = nra - mu_r, b = npb - mu_p;
        vr += a * a;
        vp += b * b;
    });
    const double pvr = fold_patch(vr, lds, lane, P, per);
    const double pvp = fold_patch(vp, lds, lane, P, per);
    if (lane < per) {
        mom[2][lane] = pc > 0.0 ? sqrt(pvr / pc) : 0.0;
        mom[3][lane] = pc > 0.0 ? sqrt(pvp / pc) : 0.0;
    }
    wave_sync();
    const double sd_r = (g < per) ? mom[2][g] : 0.0, sd_p = (g < per) ? mom[3][g] : 0.0;

    // The normalised test |(|X^r| - mu_r) / sd_r - (|X^p| - mu_p) / sd_p| < eps_r.
    double csr = 0.0, csp = 0.0, cc = 0.0;
    if (sd_r > 0.0 && sd_p > 0.0)
        each([&](double a, double b) {
            if (fabs((a - mu_r) / sd_r - (b - mu_p) / sd_p) < eps_r) {
                csr += a;
                csp += b;
                cc += 1.0;
            }
        });
    const double pcsr = fold_patch(csr, lds, lane, P, per);
    const double pcsp = fold_patch(csp, lds, lane, P, per);
    const double pcc = fold_patch(cc, lds, lane, P, per);
    if (lane < per && sx * per + lane < st.npx[v]) {
        const int64_t pid = st.patch_off[v] + (int64_t)py * st.npx[v] + sx * per + lane;
        AlignPatch a;
        a.mu_r = mom[0][lane];
        a.mu_p = mom[1][lane];
        a.sd_r = mom[2][lane];
        a.sd_p = mom[3][lane];
        a.cp_sr = pcsr;
        a.cp_sp = pcsp;
        a.n = (int32_t)pc;
        a.cp_n = (int32_t)pcc;
        out[pid] = a;
    }
}

// One workgroup per view: the max_iter iterations of Alg. 1 over the patch records.  What an
// iteration finds depends on sigma' alone, so once sigma' repeats the rest would repeat too
// and is not run.  Latency-bound: 1024 lanes hold 6 records each in registers (what fits
// 16 waves of one compute unit), only further ones are read again.  37 us for 6144
// patches per view with 256 lanes, every record read by every iteration; 14 us now.
constexpr int kIterBlock = 1024, kIterWaves = kIterBlock / kWave, kKeepPatches = 6;

__global__ void __launch_bounds__(kIterBlock)
k_align_iterate(AlignStrips st, const AlignPatch *__restrict__ patches, double delta_mu, double delta_sigma,
                int max_iter, double tau, gspm_align_result *__restrict__ result) {
    __shared__ double lds_a[2][kIterWaves], lds_b[2][kIterWaves];
    __shared__ int64_t lds_c[2][kIterWaves], lds_n[kIterWaves];
    const int v = blockIdx.x;
    const int lane = lane_id(), wid = threadIdx.x / kWave;
    const int p0 = st.patch_off[v] + (int)threadIdx.x, p1 = st.patch_off[v + 1];
    AlignPatch kept[kKeepPatches];
    int64_t n_valid = 0;
#pragma unroll
    for (int k = 0; k < kKeepPatches; ++k) {
        const int p = p0 + k * kIterBlock;
        kept[k].n = 0;
        if (p < p1) kept[k] = patches[p];
        n_valid += kept[k].n;
    }
    for (int p = p0 + kKeepPatches * kIterBlock; p < p1; p += kIterBlock) n_valid += patches[p].n;
    for (int off = 32; off > 0; off >>= 1) n_valid += __shfl_xor(n_valid, off, 64);
    if (lane == 0) lds_n[wid] = n_valid;
    double sigma = 1.0;
    int64_t cp_total = 0;
    for (int it = 0; it < max_iter; ++it) {
        double a = 0.0, b = 0.0;
        int64_t c = 0;
        auto take = [&](const AlignPatch &q) {
            // Statistics of X^p_iter = sigma' X^p.
            const double mu_p = sigma * q.mu_p, sd_p = sigma * q.sd_p;
            if (q.n > 0 && fabs(q.mu_r - mu_p) < delta_mu * mu_p && fabs(q.sd_r - sd_p) < delta_sigma * sd_p) {
                a += q.cp_sr;
                b += q.cp_sp;
                c += q.cp_n;
            }
        };
#pragma unroll
        for (int k = 0; k < kKeepPatches; ++k) take(kept[k]);
        for (int p = p0 + kKeepPatches * kIterBlock; p < p1; p += kIterBlock) take(patches[p]);
        for (int off = 32; off > 0; off >>= 1) {
            a += __shfl_xor(a, off, 64);
            b += __shfl_xor(b, off, 64);
            c += __shfl_xor(c, off, 64);
        }
        const int slot = it & 1;  // the other half may still be read
        if (lane == 0) {
            lds_a[slot][wid] = a;
            lds_b[slot][wid] = b;
            lds_c[slot][wid] = c;
        }
        __syncthreads();
        double A = 0.0, Bs = 0.0;
        int64_t C = 0;
        for (int w = 0; w < kIterWaves; ++w) {
            A += lds_a[slot][w];
            Bs += lds_b[slot][w];
            C += lds_c[slot][w];
        }
        cp_total = C;
        const double before = sigma;
        if (C > 0) sigma = A / Bs;  // mean |X^r[CP]| / mean |X^p[CP]| over the same CP
        if (sigma == before) break;  // the same for every lane
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t n_all = 0;
        for (int w = 0; w < kIterWaves; ++w) n_all += lds_n[w];
        gspm_align_result r;
        r.scale = sigma;
        r.cp = (int32_t)cp_total;
        r.n_valid = (int32_t)n_all;
        r.insufficient = (double)cp_total < tau * (double)r.n_valid ? 1 : 0;
        r.pad = 0;
        result[v] = r;
    }
}

// Eq. 14: keep X^r where |X^r - s X^p| <= eps_m |s X^p|, else take s X^p.  Bound by memory
// traffic (36 bytes per pixel), four pixels per lane and step where the planes allow 16-byte
// accesses (wide, and W H a multiple of 4).  Atomics on one cache line take 9 ns each
// whatever their number, so the grid is two workgroups per compute unit: 8 views with 3.7M
// pixels: 170 us with one update per 256 pixels, 23 us now (5.7 TB/s, some of it cached).  Large
// windows take more workgroups, a view's side by side (fewer streams at a time through the
// memory: 16 views of 1920x1080 251 us with 512, 227 with 4096), and beyond 12M pixels one pixel
// per lane, for the same reason (221 us).
constexpr int kReplaceBlock = 512, kReplaceBlocks = 512, kReplaceMost = 4096;
constexpr int64_t kReplacePixels = 8192, kReplaceWide = 12 << 20;

__global__ void __launch_bounds__(kReplaceBlock)
k_replace(ViewTable vt, const float *__restrict__ Xr, const float *__restrict__ Xp,
          const gspm_align_result *__restrict__ res, double eps_m, bool wide, float *__restrict__ out,
          uint32_t *__restrict__ replaced) {
    const int v = blockIdx.y;
    const int64_t plane = (int64_t)vt.width[v] * vt.height[v], o3 = 3 * vt.pix_off[v];
    const double s = res[v].scale;
    __shared__ uint32_t wave_cnt[kReplaceBlock / kWave];
    uint32_t cnt = 0u;
    auto pixel = [&](const float (&r)[3], const float (&p)[3], float (&o)[3]) {
        const double h0 = s * (double)p[0], h1 = s * (double)p[1], h2 = s * (double)p[2];
        const double d0 = (double)r[0] - h0, d1 = (double)r[1] - h1, d2 = (double)r[2] - h2;
        const double d = sqrt(d0 * d0 + d1 * d1 + d2 * d2), t = eps_m * sqrt(h0 * h0 + h1 * h1 + h2 * h2);
        const bool rep = !(d <= t);
        o[0] = rep ? (float)h0 : r[0];
        o[1] = rep ? (float)h1 : r[1];
        o[2] = rep ? (float)h2 : r[2];
        cnt += rep ? 1u : 0u;
    };
    const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    if (wide && plane % 4 == 0 && o3 % 4 == 0) {
        for (int64_t e = 4 * first; e < plane; e += 4 * step) {
            float4 r[3], p[3], o[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                r[c] = *reinterpret_cast<const float4 *>(Xr + o3 + c * plane + e);
                p[c] = *reinterpret_cast<const float4 *>(Xp + o3 + c * plane + e);
            }
            auto part = [&](float float4::*m) {
                const float ra[3] = {r[0].*m, r[1].*m, r[2].*m}, pa[3] = {p[0].*m, p[1].*m, p[2].*m};
                float oa[3];
                pixel(ra, pa, oa);
                o[0].*m = oa[0];
                o[1].*m = oa[1];
                o[2].*m = oa[2];
            };
            part(&float4::x);
            part(&float4::y);
            part(&float4::z);
            part(&float4::w);
#pragma unroll
            for (int c = 0; c < 3; ++c) *reinterpret_cast<float4 *>(out + o3 + c * plane + e) = o[c];
        }
    } else {
        for (int64_t e = first; e < plane; e += step) {
            const int64_t a = o3 + e;
            const float r[3] = {Xr[a], Xr[a + plane], Xr[a + 2 * plane]};
            const float p[3] = {Xp[a], Xp[a + plane], Xp[a + 2 * plane]};
            float o[3];
            pixel(r, p, o);
            out[a] = o[0];
            out[a + plane] = o[1];
            out[a + 2 * plane] = o[2];
        }
    }
    // One atomic per workgroup: the per-view counter sees few updates.
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, 64);
    if (lane_id() == 0) wave_cnt[threadIdx.x / kWave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0u;
        for (int w = 0; w < kReplaceBlock / kWave; ++w) t += wave_cnt[w];
        if (t) atomicAdd(replaced + v, t);
    }
}

}  // namespace

int64_t align_patches(const ViewTable &vt, int patch) { return align_strips(vt, patch).patch_off[vt.n_views]; }

hipError_t launch_align_scale(const ViewTable &vt, const float *Xr, const float *Xp, const float *mask,
                              const gspm_align_params &prm, AlignPatch *patches, gspm_align_result *result,
                              hipStream_t s) {
    const AlignStrips st = align_strips(vt, prm.patch);
    const int64_t waves = st.wave_off[vt.n_views];
    if (waves > 0)
        hipLaunchKernelGGL(k_align_stats, dim3((unsigned)((waves + kAlignWaves - 1) / kAlignWaves)),
                           dim3(kAlignBlock), 0, s, vt, st, Xr, Xp, mask, (double)prm.eps_r, patches);
    hipLaunchKernelGGL(k_align_iterate, dim3(vt.n_views), dim3(kIterBlock), 0, s, st, patches,
                       (double)prm.delta_mu, (double)prm.delta_sigma, prm.max_iter, (double)prm.tau, result);
    return hipGetLastError();
}

hipError_t launch_replace(const ViewTable &vt, const float *Xr, const float *Xp, const gspm_align_result *result,
                          float eps_m, float *out, uint32_t *replaced, hipStream_t s) {
    hipError_t e = launch_fill_u32(replaced, 0u, vt.n_views, s);
    if (e != hipSuccess) return e;
    int64_t maxp = 1;
    for (int v = 0; v < vt.n_views; ++v) maxp = std::max<int64_t>(maxp, (int64_t)vt.width[v] * vt.height[v]);
    const int64_t pixels = vt.pix_off[vt.n_views];
    const bool wide = (((uintptr_t)Xr | (uintptr_t)Xp | (uintptr_t)out) & 15u) == 0u && pixels <= kReplaceWide;
    const int64_t most = std::min<int64_t>(kReplaceMost, std::max<int64_t>(kReplaceBlocks, pixels / kReplacePixels));
    const int64_t bx = std::min<int64_t>((maxp + 4 * kReplaceBlock - 1) / (4 * kReplaceBlock),
                                         std::max<int64_t>(1, most / vt.n_views));
    hipLaunchKernelGGL(k_replace, dim3((unsigned)bx, (unsigned)vt.n_views), dim3(kReplaceBlock), 0, s, vt, Xr, Xp,
                       result, (double)eps_m, wide, out, replaced);
    return hipGetLastError();
}

}  // namespace gspm
