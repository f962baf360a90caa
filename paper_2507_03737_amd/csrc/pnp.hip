// Pose initialisation of the tracking front end (Sec. 3.2.1, Eq. 6-9): RANSAC over
// caller-drawn samples of 2D-3D correspondences, a linear six-point PnP per hypothesis,
// inlier scoring, and Gauss-Newton refinement of the best hypothesis on its inliers.
//
//   k_pnp_hyp     one wave per hypothesis: the 12 x 12 normal matrix of the normalised
//                 six-point system in LDS, cyclic Jacobi with six rotations at a time, the
//                 eigenvector of least eigenvalue, the normalisation undone, the sign fixed by
//                 det(M) > 0, and the nearest rotation as the orthogonal polar factor (Newton
//                 iteration on M), with lambda = trace(R^T M) / 3 (the mean singular value);
//   k_pnp_score   one workgroup per two hypotheses streams the correspondences (coalesced
//                 SoA) and counts those with positive depth and reprojection error < threshold;
//                 the best hypothesis (highest score, lowest index) is a maximum over keys;
//   k_pnp_step    per-workgroup FP64 partial sums of J^T J and J^T r over the inliers (marked by
//                 the first step of a round).  Before that, every workgroup takes the previous
//                 step's Gauss-Newton update from its partials: the fixed-order sum, the
//                 damped Cholesky solve and the left update T <- Exp(xi) T (skipped with fewer
//                 than 6 inliers);
//   k_pnp_finish  the last update, inlier mask and count of the final pose, and the results.
// Everything is float64; the inputs are float32.
#include <algorithm>
#include <type_traits>

#include "gspm_common.h"

namespace gspm {

namespace {

constexpr int kHypWaves = 4;       // hypotheses (waves) per workgroup of k_pnp_hyp
constexpr int kScoreBlock = 512, kScoreHyps = 2;
constexpr int kAccBlock = 256;
constexpr int kAccBlocks = 256;    // most workgroups of a Gauss-Newton step
constexpr int kPart = 32;          // doubles of a workgroup's partial sums (28 used)

struct Pose {
    double R[9];
    double t[3];
};

// Kept between the kernels of one call; cleared by its first.
struct PnpState {
    unsigned long long best;  // max of (score + 1) 2^32 + 2^32 - 1 - index over the hypotheses
    uint32_t arrived;         // workgroups of the running kernel that have ended
    int32_t inliers;          // of the final pose
};

// Whether this workgroup is the last of the grid to get here; all that the others' first waves
// wrote before is then visible to it (the release waits for the stores of its own wave).  Leaves
// the counter at zero for the next kernel.
__device__ inline bool last_block(PnpState *st) {
    __shared__ bool last;
    __syncthreads();
    if (threadIdx.x == 0) {
        last = __hip_atomic_fetch_add(&st->arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
        if (last) __hip_atomic_store(&st->arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return last;
}

__device__ inline void se3_exp(const double xi[6], double R[9], double t[3]) {
    const double px = xi[3], py = xi[4], pz = xi[5];
    const double th2 = px * px + py * py + pz * pz, th = sqrt(th2);
    double a, b, c;  // sin(th) / th, (1 - cos(th)) / th^2, (th - sin(th)) / th^3
    if (th2 < 0.25) {
        // Power series, each term the last times -th^2 over two factors: the first one left out
        // is below 2^-53 of the sum.  Steps are small: this is the usual case, and short.
        a = b = c = 1.0;
#pragma unroll
        for (int k = 8; k >= 1; --k) {
            a = fma(a, -th2 * (1.0 / ((2 * k) * (2 * k + 1))), 1.0);
            b = fma(b, -th2 * (1.0 / ((2 * k + 1) * (2 * k + 2))), 1.0);
            c = fma(c, -th2 * (1.0 / ((2 * k + 2) * (2 * k + 3))), 1.0);
        }
        b *= 0.5;
        c *= 1.0 / 6.0;
    } else {
        a = sin(th) / th;
        b = (1.0 - cos(th)) / th2;
        c = (th - sin(th)) / (th2 * th);
    }
    const double K[9] = {0.0, -pz, py, pz, 0.0, -px, -py, px, 0.0};
    double K2[9];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) K2[3 * i + j] = K[3 * i] * K[j] + K[3 * i + 1] * K[3 + j] + K[3 * i + 2] * K[6 + j];
    double V[9];
    for (int k = 0; k < 9; ++k) {
        const double I = (k % 4 == 0) ? 1.0 : 0.0;
        R[k] = I + a * K[k] + b * K2[k];
        V[k] = I + b * K[k] + c * K2[k];
    }
    for (int i = 0; i < 3; ++i) t[i] = V[3 * i] * xi[0] + V[3 * i + 1] * xi[1] + V[3 * i + 2] * xi[2];
}

// Orthogonal polar factor of a 3x3 matrix with positive determinant (Newton iteration
// X <- (X + X^-T) / 2, which converges quadratically to U V^T of the SVD).
__device__ inline void polar(const double M[9], double R[9]) {
    for (int k = 0; k < 9; ++k) R[k] = M[k];
    for (int it = 0; it < 30; ++it) {
        // cofactor matrix C = det(X) X^-T
        double C[9];
        C[0] = R[4] * R[8] - R[5] * R[7];
        C[1] = R[5] * R[6] - R[3] * R[8];
        C[2] = R[3] * R[7] - R[4] * R[6];
        C[3] = R[2] * R[7] - R[1] * R[8];
        C[4] = R[0] * R[8] - R[2] * R[6];
        C[5] = R[1] * R[6] - R[0] * R[7];
        C[6] = R[1] * R[5] - R[2] * R[4];
        C[7] = R[2] * R[3] - R[0] * R[5];
        C[8] = R[0] * R[4] - R[1] * R[3];
        const double det = R[0] * C[0] + R[1] * C[1] + R[2] * C[2];
        if (!(fabs(det) > 1e-300)) return;
        const double inv = 1.0 / det;
        double d = 0.0;
        for (int k = 0; k < 9; ++k) {
            const double nv = 0.5 * (R[k] + C[k] * inv);
            d = fmax(d, fabs(nv - R[k]));
            R[k] = nv;
        }
        if (d < 1e-15) return;
    }
}

__global__ void __launch_bounds__(kHypWaves * kWave)
k_pnp_hyp(const float *__restrict__ X, const float *__restrict__ uv, int64_t n, gspm_intrinsics K,
          const int32_t *__restrict__ samples, int H, Pose *__restrict__ poses, int32_t *__restrict__ valid,
          PnpState *__restrict__ st) {
    __shared__ double Sm[kHypWaves][144];  // symmetric matrix, full storage
    __shared__ double Em[kHypWaves][144];  // eigenvectors (columns)
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int h = blockIdx.x * kHypWaves + w;
    if (blockIdx.x == 0 && threadIdx.x == 0) *st = PnpState{0ull, 0u, 0};
    if (h >= H) return;  // wave-uniform
    double *A = Sm[w], *E = Em[w];
    // Every lane loads the sample (wave-uniform values).
    bool ok = true;
    int idx[6];
    for (int k = 0; k < 6; ++k) {
        idx[k] = samples[6 * (int64_t)h + k];
        ok = ok && idx[k] >= 0 && idx[k] < n;
    }
    if (!ok)
        for (int k = 0; k < 6; ++k) idx[k] = 0;
    double P3[6][3], x2[6][2], c[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 6; ++k) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            P3[k][a] = X[a * n + idx[k]];
            c[a] += P3[k][a] / 6.0;
        }
        x2[k][0] = ((double)uv[idx[k]] - K.cx) / K.fx;
        x2[k][1] = ((double)uv[n + idx[k]] - K.cy) / K.fy;
    }
    double dm = 0.0;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const double dx = P3[k][0] - c[0], dy = P3[k][1] - c[1], dz = P3[k][2] - c[2];
        dm += sqrt(dx * dx + dy * dy + dz * dz) / 6.0;
    }
    const double s = dm > 0.0 ? sqrt(3.0) / dm : 1.0;
    // Lane l < 144 computes entry (l / 12, l % 12) of A^T A for the rows [Xh 0 -x Xh], [0 Xh -y Xh].
    for (int l = lane; l < 144; l += kWave) {
        const int i = l / 12, j = l % 12;
        double acc = 0.0;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const double Xh[4] = {s * (P3[k][0] - c[0]), s * (P3[k][1] - c[1]), s * (P3[k][2] - c[2]), 1.0};
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const double ri = i < 8 ? ((i / 4 == r) ? Xh[i % 4] : 0.0) : -x2[k][r] * Xh[i - 8];
                const double rj = j < 8 ? ((j / 4 == r) ? Xh[j % 4] : 0.0) : -x2[k][r] * Xh[j - 8];
                acc += ri * rj;
            }
        }
        A[l] = acc;
        E[l] = i == j ? 1.0 : 0.0;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // Cyclic Jacobi in rounds of six disjoint rotations (a round-robin schedule: 11 rounds meet
    // every pair once): a serial chain of 11 angles a sweep instead of the 66 of single
    // rotations (1024 hypotheses: 253 us with those, 61 us now).  Lane l takes the angle of pair
    // l % 6; then lanes 0..14 turn the 2 x 2 block of two pairs, 15..20 that of one, and 21..56
    // two rows of E at one pair each.
    int bi = 0, bj = 0, row0 = 0;
    const bool pairs = lane < 15, diagonal = lane >= 15 && lane < 21, vec = lane >= 21 && lane < 57;
    if (pairs) {
        bj = lane;
        while (bj >= 5 - bi) bj -= 5 - bi++;
        bj += bi + 1;
    } else if (diagonal) {
        bi = bj = lane - 15;
    } else if (vec) {
        bi = bj = (lane - 21) % 6;
        row0 = (lane - 21) / 6;
    }
    double *const M0 = vec ? E : A;
    // Pair i of round r: (r, 11) for i = 0, else (r + i, r - i) mod 11, the smaller first.
    struct Pair {
        int x, y, step, lim;
        __device__ explicit Pair(int i) : x(i), y(i == 0 ? 11 : 11 - i), step(i == 0 ? 0 : 1), lim(i == 0 ? 12 : 11) {}
        __device__ void next() {
            x += 1;
            x -= x == 11 ? 11 : 0;
            y += step;
            y -= y == lim ? lim : 0;
        }
    };
    Pair al(lane % 6), ai(bi), aj(bj);
    for (int sweep = 0; sweep < 20; ++sweep) {
        double off = 0.0, diag = 0.0;
        for (int l = lane; l < 144; l += kWave) {
            const double a = A[l];
            if (l % 13 == 0) diag += a * a; else off += a * a;
        }
        for (int o = 32; o > 0; o >>= 1) {
            off += __shfl_xor(off, o, kWave);
            diag += __shfl_xor(diag, o, kWave);
        }
        if (off <= 2e-30 * diag) break;  // wave-uniform
        for (int r = 0; r < 11; ++r) {
            const int p = min(al.x, al.y), q = max(al.x, al.y);
            const int pi = min(ai.x, ai.y), qi = max(ai.x, ai.y), pj = min(aj.x, aj.y), qj = max(aj.x, aj.y);
            al.next();
            ai.next();
            aj.next();
            const double apq = A[p * 12 + q], app = A[p * 13], aqq = A[q * 13];
            const int r0 = 12 * (vec ? row0 : pi), r1 = 12 * (vec ? row0 + 6 : qi);
            const double a = M0[r0 + pj], b = M0[r0 + qj], c = M0[r1 + pj], d = M0[r1 + qj];
            // With d = aqq - app, b = 2 apq and 1/h = (d^2 + b^2)^(-1/2): cos^2 = (1 + |d|/h) / 2,
            // sin = +-b / (2 h cos), tan = sin / cos.  Two reciprocal roots; outside the range of the
            // squares tan comes from theta = d / b as 1 / (|theta| + (theta^2 + 1)^(1/2)).
            const double d_ = aqq - app, b_ = 2.0 * apq, hh = d_ * d_ + b_ * b_;
            double cs, sn, tt;
            if ((hh > 1e-280 && hh < 1e280) || apq == 0.0) {
                const double rh = rsqrt(hh), c2 = 0.5 + 0.5 * fabs(d_) * rh, rc = rsqrt(c2);
                cs = c2 * rc;
                sn = (d_ >= 0.0 ? 0.5 : -0.5) * b_ * rh * rc;
                tt = sn * rc;
            } else {
                const double theta = d_ / b_;
                tt = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
                cs = rsqrt(tt * tt + 1.0);
                sn = tt * cs;
            }
            if (apq == 0.0) {
                cs = 1.0;
                sn = tt = 0.0;
            }
            const double shift = __shfl(tt * apq, bj, kWave);
            const double cj = __shfl(cs, bj, kWave), sj = __shfl(sn, bj, kWave);
            double ci = __shfl(cs, bi, kWave), si = __shfl(sn, bi, kWave);
            if (vec) {
                ci = 1.0;
                si = 0.0;
            }
            const double l00 = ci * a - si * c, l10 = si * a + ci * c, l01 = ci * b - si * d, l11 = si * b + ci * d;
            double n00 = cj * l00 - sj * l01, n01 = sj * l00 + cj * l01;
            double n10 = cj * l10 - sj * l11, n11 = sj * l10 + cj * l11;
            if (diagonal) {
                n00 = a - shift;
                n11 = d + shift;
                n01 = n10 = 0.0;
            }
            __builtin_amdgcn_wave_barrier();
            if (lane < 57) {
                M0[r0 + pj] = n00;
                M0[r0 + qj] = n01;
                M0[r1 + pj] = n10;
                M0[r1 + qj] = n11;
            }
            if (pairs) {
                A[pj * 12 + pi] = n00;
                A[qj * 12 + pi] = n01;
                A[pj * 12 + qi] = n10;
                A[qj * 12 + qi] = n11;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    if (lane != 0) return;
    int m = 0;
    for (int i = 1; i < 12; ++i)
        if (A[i * 13] < A[m * 13]) m = i;
    double p[12];
    for (int i = 0; i < 12; ++i) p[i] = E[i * 12 + m];
    // Undo the normalisation: M = s Pn[:, :3], p4 = Pn[:, 3] - s Pn[:, :3] c.
    double M[9], p4[3];
    for (int r = 0; r < 3; ++r) {
        for (int a = 0; a < 3; ++a) M[3 * r + a] = s * p[4 * r + a];
        p4[r] = p[4 * r + 3] - (M[3 * r] * c[0] + M[3 * r + 1] * c[1] + M[3 * r + 2] * c[2]);
    }
    const double det = M[0] * (M[4] * M[8] - M[5] * M[7]) - M[1] * (M[3] * M[8] - M[5] * M[6]) +
                       M[2] * (M[3] * M[7] - M[4] * M[6]);
    if (det < 0.0) {
        for (int k = 0; k < 9; ++k) M[k] = -M[k];
        for (int k = 0; k < 3; ++k) p4[k] = -p4[k];
    }
    Pose P;
    polar(M, P.R);
    double tr = 0.0;  // trace(R^T M) = sum of the singular values
    for (int k = 0; k < 9; ++k) tr += P.R[k] * M[k];
    const double lam = tr / 3.0;
    ok = ok && det != 0.0 && lam > 0.0;
    for (int k = 0; k < 3; ++k) P.t[k] = ok ? p4[k] / lam : 0.0;
    poses[h] = P;
    valid[h] = ok ? 1 : 0;
}

__device__ inline bool inlier(const Pose &P, double x, double y, double z, double u0, double v0,
                              const gspm_intrinsics &K, double thr2, double r[2], double Y[3]) {
    Y[0] = P.R[0] * x + P.R[1] * y + P.R[2] * z + P.t[0];
    Y[1] = P.R[3] * x + P.R[4] * y + P.R[5] * z + P.t[1];
    Y[2] = P.R[6] * x + P.R[7] * y + P.R[8] * z + P.t[2];
    if (!(Y[2] > 0.0)) return false;
    const double iz = 1.0 / Y[2];
    r[0] = K.fx * Y[0] * iz + K.cx - u0;
    r[1] = K.fy * Y[1] * iz + K.cy - v0;
    return r[0] * r[0] + r[1] * r[1] < thr2;
}

// Float64 arithmetic binds this (about 30 instructions per match and hypothesis); a workgroup
// takes two hypotheses, so that the loads and conversions of a match serve both, and a point's
// one reciprocal serves both coordinates: 20000 matches, 1024 hypotheses: 54 us with one
// hypothesis per workgroup and two divisions, 38 us now (four hypotheses: 43 us).  Invalid
// hypotheses are not counted.
__global__ void __launch_bounds__(kScoreBlock)
k_pnp_score(const float *__restrict__ X, const float *__restrict__ uv, int64_t n, gspm_intrinsics K, double thr2,
            const Pose *__restrict__ poses, const int32_t *__restrict__ valid, int H, int32_t *__restrict__ scores,
            PnpState *__restrict__ st) {
    __shared__ int lds[kScoreHyps][kScoreBlock / kWave];
    const int h0 = blockIdx.x * kScoreHyps;
    static_assert(kScoreHyps == 2, "both, one or none");
    int cnt[kScoreHyps] = {0, 0};
    const bool first = valid[h0] != 0, second = h0 + 1 < H && valid[h0 + 1] != 0;
    auto count = [&](auto both, const Pose &P0, const Pose &P1, int &c0, int &c1) {
        for (int64_t k = threadIdx.x; k < n; k += blockDim.x) {
            const double x = X[k], y = X[n + k], z = X[2 * n + k], u0 = uv[k], v0 = uv[n + k];
            double r[2], Y[3];
            c0 += inlier(P0, x, y, z, u0, v0, K, thr2, r, Y) ? 1 : 0;
            if (decltype(both)::value) c1 += inlier(P1, x, y, z, u0, v0, K, thr2, r, Y) ? 1 : 0;
        }
    };
    if (first && second) {
        const Pose P0 = poses[h0], P1 = poses[h0 + 1];
        count(std::true_type{}, P0, P1, cnt[0], cnt[1]);
    } else if (first || second) {
        const Pose P0 = poses[first ? h0 : h0 + 1];
        int c = 0;
        count(std::false_type{}, P0, P0, c, c);
        cnt[0] = first ? c : 0;
        cnt[1] = first ? 0 : c;
    }
#pragma unroll
    for (int i = 0; i < kScoreHyps; ++i) {
        for (int off = 32; off > 0; off >>= 1) cnt[i] += __shfl_xor(cnt[i], off, 64);
        if (lane_id() == 0) lds[i][threadIdx.x / kWave] = cnt[i];
    }
    __syncthreads();
    const int h = h0 + (int)threadIdx.x;
    if (threadIdx.x < kScoreHyps && h < H) {
        int t = 0;
        for (int w = 0; w < kScoreBlock / kWave; ++w) t += lds[threadIdx.x][w];
        t = valid[h] ? t : -1;
        scores[h] = t;
        atomicMax(&st->best, ((unsigned long long)((long long)t + 1) << 32) + (4294967295ull - (unsigned long long)h));
    }
}

// One step from the summed partials (acc: 21 of J^T J, 6 of J^T r, the inliers), unless the
// inliers are < 6 or the system is not positive definite.
__device__ inline Pose gauss_newton(const double *acc, const Pose &P) {
    if (acc[27] < 6.0) return P;
    double A[6][6];
    int q = 0;
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = i; j < 6; ++j) A[j][i] = acc[q++];
    const double damp = 1e-9 * (A[0][0] + A[1][1] + A[2][2] + A[3][3] + A[4][4] + A[5][5]) / 6.0;
    double inv[6];  // 1 / L[i][i]; L overwrites A
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        double sum = A[j][j] + damp;
#pragma unroll
        for (int k = 0; k < j; ++k) sum -= A[j][k] * A[j][k];
        if (!(sum > 0.0)) return P;
        inv[j] = rsqrt(sum);
#pragma unroll
        for (int i = j + 1; i < 6; ++i) {
            double x = A[i][j];
#pragma unroll
            for (int k = 0; k < j; ++k) x -= A[i][k] * A[j][k];
            A[i][j] = x * inv[j];
        }
    }
    double w[6], xi[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        double sum = -acc[21 + i];
#pragma unroll
        for (int k = 0; k < i; ++k) sum -= A[i][k] * w[k];
        w[i] = sum * inv[i];
    }
#pragma unroll
    for (int i = 5; i >= 0; --i) {
        double sum = w[i];
#pragma unroll
        for (int k = i + 1; k < 6; ++k) sum -= A[k][i] * xi[k];
        xi[i] = sum * inv[i];
    }
    double dR[9], dt[3];
    se3_exp(xi, dR, dt);
    Pose Pn;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int j = 0; j < 3; ++j)
            Pn.R[3 * i + j] = dR[3 * i] * P.R[j] + dR[3 * i + 1] * P.R[3 + j] + dR[3 * i + 2] * P.R[6 + j];
        Pn.t[i] = dR[3 * i] * P.t[0] + dR[3 * i + 1] * P.t[1] + dR[3 * i + 2] * P.t[2] + dt[i];
    }
    return Pn;
}

// The pose that step number `step` of a call starts from, for all lanes of the workgroup: the
// best hypothesis for step 0, else the last step's pose and its update from that step's
// partials (nb workgroups'), summed in a fixed order, eight interleaved sums first.
__device__ inline Pose pose_at(int step, const Pose *poses, const Pose *cur, const double *part, int nb,
                               const PnpState *st, double (*lds)[kPart]) {
    __shared__ Pose P;
    if (step == 0) return poses[4294967295ull - (st->best & 4294967295ull)];
    const Pose *from = cur + ((step - 1) & 1);
    const double *sums = part + ((step - 1) & 1) * kPart * kAccBlocks;
    const int q = threadIdx.x % kPart, g = threadIdx.x / kPart;
    double t = 0.0;
    for (int b = g; b < nb; b += 8) t += sums[b * kPart + q];
    lds[g][q] = t;
    __syncthreads();
    if (threadIdx.x < kPart) {
        t = 0.0;
#pragma unroll
        for (int k = 0; k < 8; ++k) t += lds[k][q];
        lds[0][q] = t;  // column q is this lane's
    }
    __syncthreads();
    if (threadIdx.x == 0) P = gauss_newton(lds[0], *from);
    __syncthreads();
    return P;
}

// One Gauss-Newton step.  mark: the first step of a round, which also sets the inlier mask from
// the pose it starts from.
//
// Steps follow one another, so launches and latencies decide (20000 matches: 79 workgroups).
// That every workgroup repeats the last step's solve saves a kernel for it (14 us beside the 9
// of the sums; a solve in the workgroup that ends last: 10.5 us together, of which
// the hand-over takes 2).  Summing a wave's 28 values by halving the values as well as the
// lanes takes 32 exchanges instead of 168.  8.4 us at 20000 matches, 20 times in a call.
__global__ void __launch_bounds__(kAccBlock)
k_pnp_step(const float *__restrict__ X, const float *__restrict__ uv, int64_t n, gspm_intrinsics K, double thr2,
           const Pose *poses, Pose *cur, const PnpState *st, int step, bool mark, uint8_t *__restrict__ mask,
           double *part) {
    __shared__ double lds[8][kPart];
    const Pose P = pose_at(step, poses, cur, part, (int)gridDim.x, st, lds);
    if (blockIdx.x == 0 && threadIdx.x == 0) cur[step & 1] = P;
    double acc[kPart];
#pragma unroll
    for (int q = 0; q < kPart; ++q) acc[q] = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
        const double x = X[k], y = X[n + k], z = X[2 * n + k], u0 = uv[k], v0 = uv[n + k];
        if (mark) {
            double r[2], Y[3];
            const bool in = inlier(P, x, y, z, u0, v0, K, thr2, r, Y);
            mask[k] = in ? 1 : 0;
            if (!in) continue;
        } else if (!mask[k]) {
            continue;
        }
        acc[27] += 1.0;
        const double Y[3] = {P.R[0] * x + P.R[1] * y + P.R[2] * z + P.t[0], P.R[3] * x + P.R[4] * y + P.R[5] * z + P.t[1],
                             P.R[6] * x + P.R[7] * y + P.R[8] * z + P.t[2]};
        if (!(Y[2] > 0.0)) continue;  // cannot happen for small steps; keeps the sums finite
        const double iz = 1.0 / Y[2];
        const double r[2] = {K.fx * Y[0] * iz + K.cx - u0, K.fy * Y[1] * iz + K.cy - v0};
        const double Jp[2][3] = {{K.fx * iz, 0.0, -K.fx * Y[0] * iz * iz}, {0.0, K.fy * iz, -K.fy * Y[1] * iz * iz}};
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            // d Y / d xi = [I | -[Y]x]: the rotation block is Y x Jp.
            const double J[6] = {Jp[c][0], Jp[c][1], Jp[c][2], Y[1] * Jp[c][2] - Y[2] * Jp[c][1],
                                 Y[2] * Jp[c][0] - Y[0] * Jp[c][2], Y[0] * Jp[c][1] - Y[1] * Jp[c][0]};
            int q = 0;
#pragma unroll
            for (int i = 0; i < 6; ++i)
#pragma unroll
                for (int j = i; j < 6; ++j) acc[q++] += J[i] * J[j];
#pragma unroll
            for (int i = 0; i < 6; ++i) acc[21 + i] += J[i] * r[c];
        }
    }
    // Halve the values with the lanes: lanes 2 q and 2 q + 1 end with value q of the wave.
    const int wid = threadIdx.x / kWave, lane = lane_id();
#pragma unroll
    for (int h = 16; h > 0; h >>= 1) {
        const bool upper = (lane & (2 * h)) != 0;
#pragma unroll
        for (int k = 0; k < h; ++k) {
            const double send = upper ? acc[k] : acc[k + h], keep = upper ? acc[k + h] : acc[k];
            acc[k] = keep + __shfl_xor(send, 2 * h, kWave);
        }
    }
    const double sum = acc[0] + __shfl_xor(acc[0], 1, kWave);
    if ((lane & 1) == 0) lds[wid][lane >> 1] = sum;
    __syncthreads();
    if (threadIdx.x < kPart)
        part[((step & 1) * kAccBlocks + (int)blockIdx.x) * kPart + threadIdx.x] =
            lds[0][threadIdx.x] + lds[1][threadIdx.x] + lds[2][threadIdx.x] + lds[3][threadIdx.x];
}

// Inlier mask and count of the final pose; the workgroup that ends last writes the results.
__global__ void __launch_bounds__(kAccBlock)
k_pnp_finish(const float *__restrict__ X, const float *__restrict__ uv, int64_t n, gspm_intrinsics K, double thr2,
             const Pose *__restrict__ poses, const Pose *__restrict__ cur, const double *__restrict__ part,
             PnpState *st, int step, uint8_t *__restrict__ mask, double *__restrict__ T_out, int32_t *__restrict__ n_inliers,
             const float *__restrict__ T_ak, float *__restrict__ T_n) {
    __shared__ double sums[8][kPart];
    const Pose P = pose_at(step, poses, cur, part, (int)gridDim.x, st, sums);
    int cnt = 0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
        double r[2], Y[3];
        const bool in = inlier(P, X[k], X[n + k], X[2 * n + k], uv[k], uv[n + k], K, thr2, r, Y);
        mask[k] = in ? 1 : 0;
        cnt += in ? 1 : 0;
    }
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, 64);
    __shared__ int lds[kAccBlock / kWave];
    if (lane_id() == 0) lds[threadIdx.x / kWave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(&st->inliers, lds[0] + lds[1] + lds[2] + lds[3]);
    if (!last_block(st) || threadIdx.x >= 12) return;
    if (threadIdx.x == 0) *n_inliers = __hip_atomic_load(&st->inliers, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int i = threadIdx.x / 4, j = threadIdx.x % 4;
    double R[3], t = 0.0;  // row i of the pose
#pragma unroll
    for (int r = 0; r < 3; ++r)
        if (r == i) {
            for (int k = 0; k < 3; ++k) R[k] = P.R[3 * r + k];
            t = P.t[r];
        }
    T_out[threadIdx.x] = j == 3 ? t : j == 0 ? R[0] : j == 1 ? R[1] : R[2];
    if (T_n) {  // Eq. 9: T_n = T_rel T_ak
        double acc = j == 3 ? t : 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) acc += R[k] * (double)T_ak[4 * k + j];
        T_n[threadIdx.x] = (float)acc;
    }
}

}  // namespace

int64_t pnp_scratch_bytes(int H, int64_t n) {
    return (int64_t)H * ((int64_t)sizeof(Pose) + 8) + 2 * (int64_t)sizeof(Pose) + (int64_t)sizeof(PnpState) +
           2 * 8 * kPart * kAccBlocks + n + 1024;
}

hipError_t launch_pnp(const float *X, const float *uv, int64_t n, const gspm_intrinsics &K, const int32_t *samples,
                      int H, double thr, int iters, int rounds, void *scratch, double *T_out, int32_t *n_inliers,
                      uint8_t *mask, int32_t *scores_out, const float *T_ak, float *T_n_out, hipStream_t s) {
    char *base = static_cast<char *>(scratch);
    Pose *poses = reinterpret_cast<Pose *>(base);
    Pose *cur = poses + H;
    PnpState *st = reinterpret_cast<PnpState *>(cur + 2);
    int32_t *valid = reinterpret_cast<int32_t *>(st + 1);
    int32_t *scores = scores_out ? scores_out : valid + H;
    double *part = reinterpret_cast<double *>(base + (((char *)(valid + 2 * H) - base + 255) & ~(int64_t)255));
    uint8_t *round_mask = reinterpret_cast<uint8_t *>(part + 2 * kPart * kAccBlocks);
    const double thr2 = thr * thr;
    hipLaunchKernelGGL(k_pnp_hyp, dim3((H + kHypWaves - 1) / kHypWaves), dim3(kHypWaves * kWave), 0, s, X, uv, n, K,
                       samples, H, poses, valid, st);
    hipLaunchKernelGGL(k_pnp_score, dim3((H + kScoreHyps - 1) / kScoreHyps), dim3(kScoreBlock), 0, s, X, uv, n, K, thr2,
                       poses, valid, H, scores, st);
    const dim3 grid((unsigned)std::min<int64_t>((n + kAccBlock - 1) / kAccBlock, kAccBlocks));
    int step = 0;
    for (int round = 0; round < rounds; ++round)
        for (int it = 0; it < iters; ++it, ++step)
            hipLaunchKernelGGL(k_pnp_step, grid, dim3(kAccBlock), 0, s, X, uv, n, K, thr2, poses, cur, st, step, it == 0,
                               round_mask, part);
    hipLaunchKernelGGL(k_pnp_finish, grid, dim3(kAccBlock), 0, s, X, uv, n, K, thr2, poses, cur, part, st, step,
                       mask ? mask : round_mask, T_out, n_inliers, T_ak, T_n_out);
    return hipGetLastError();
}

}  // namespace gspm
