// Tile rasterizer: front-to-back compositing (Sec. 3.1, Eq. 2; Sec. 3.2.1, Eq. 3-5) and
// its backward.
//
// One workgroup per tile of T x T pixels (T = 8, 16 or 32) with T*T/PPT lanes.  Each wave
// owns a compact rectangle of the tile (8 x 8 pixels for PPT = 1, 8 x 16 for PPT = 2, ...)
// and each lane PPT vertically adjacent pixels of one of its columns.  The tile's
// depth-ordered record list is streamed through LDS in batches of one record per lane (a
// 64-byte record, converted to tile-local coordinates on load).  When a tile holds several
// waves, each wave of the forward first tests the whole batch against its own rectangle (one record per
// lane: the maximum of the concave base-2 exponent over the rectangle, against the
// record's threshold, with a rounding margin so that no record a pixel would accept is
// dropped) and then walks only the records that meet it, taken from the ballot mask with
// scalar bit scans.  Binning stays at tile granularity while the per-pixel work is that of
// 8-pixel-wide tiles.  A fragment is rejected on its base-2 exponent against a per-record
// threshold, so the exponential is only evaluated for pixels that composite it; the
// workgroup stops as soon as every pixel has reached the transmittance floor.
//
// Windows with few waves are composited by independent waves instead (k_raster_fwd_waves): the
// same expressions per pixel in the same order, so the same images.
//
// The forward also records, per wave, which list entries one of its live pixels accepted
// (one bit per entry and wave, kept in the frame state).  The backward walks only those
// entries, front to back: with one pixel per lane by independent waves that stage their own
// entries (k_raster_bwd_waves), otherwise by workgroups that stage batches of one record per
// lane (k_raster_bwd).  It recomputes alpha and transmittance with the same
// instructions as the forward, so no per-fragment state is stored: only the bits and the
// per-pixel count of list entries up to the last contributing fragment.  The suffix sums
// that the alpha derivative needs are carried as a remainder: it starts at the sum over
// all fragments (from the forward's outputs) and each walked fragment subtracts its share.
// Per record the wave needs up to 13 sums over its pixels: the moments of alpha dL/dalpha
// over the pixel offsets (from which the mean, conic and opacity gradients follow) and the
// colour, depth and point sums.  With one pixel per lane the matrix cores form them for 16
// records at a time; with several pixels per lane each lane
// adds its pixels' contributions and the wave adds them up with one reduce-scatter
// (cross-half lane swaps and DPP) of 8, 12 or 16 values.  Either way the atomics are paid
// once per wave and record.
#include <type_traits>

#include "gspm_common.h"

namespace gspm {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

struct TilePos {
    int gt;  // global tile index
    int v, W, H;
    int tx, ty;
    float x0, y0;     // tile origin
    int64_t plane;    // W * H of the view
    int64_t pix_off;  // packed offset of the view
};

// Workgroups run the tiles in the given order (heaviest first, so that the long lists do
// not start last and leave the chip idle behind them).
template <int TILE>
__device__ inline TilePos tile_pos(const ViewTable &vt, const uint32_t *order, uint32_t slot) {
    TilePos p;
    const int gt = order ? (int)order[slot] : (int)slot;
    p.gt = gt;
    p.v = find_view(vt, gt);
    const int lt = gt - vt.tile_off[p.v];
    p.tx = lt % vt.tiles_x[p.v];
    p.ty = lt / vt.tiles_x[p.v];
    p.W = vt.width[p.v];
    p.H = vt.height[p.v];
    p.x0 = (float)(p.tx * TILE);
    p.y0 = (float)(p.ty * TILE);
    p.plane = (int64_t)p.W * p.H;
    p.pix_off = vt.pix_off[p.v];
    return p;
}

// Stage record r into LDS slot q, in tile-local pixel coordinates, with the record's
// threshold -e_min (see accept_threshold): alpha >= alpha_min exactly when the base-2
// exponent e = -s >= e_min, i.e. s <= -e_min, so rejected pixels never evaluate the
// exponential.  own_min > 0: with the threshold for this alpha_min instead.
//   s0 = (u, v, a, b), s1 = (c, -e_min, opacity, record index), s2 = (colour, z), s3 = point
// with (a, b, c) the factored conic of the record.
// The acceptance test reads s0 and s1 only.
__device__ inline void stage(const float4 *__restrict__ rec, uint32_t r, float x0, float y0, float4 *s0, float4 *s1,
                             float4 *s2, float4 *s3, int q, float own_min = 0.0f) {
    const float4 *src = rec + 4 * (int64_t)r;
    const float4 a = src[0], b = src[1], c = src[2], d = src[3];
    const float ul = (a.x - x0) + a.z;
    const float vl = (a.y - y0) + a.w;
    s0[q] = make_float4(ul, vl, b.x, b.y);
    s1[q] = make_float4(b.z, own_min > 0.0f ? accept_threshold(own_min, b.w) : d.w, b.w, __uint_as_float(r));
    s2[q] = c;
    s3[q] = d;
}

// min(alpha_max, a) for a >= 0, as one median instruction (min would first quiet a
// signalling NaN in the kernel-argument operand, on every call).
__device__ inline float clamp_alpha(float a, float amax) { return __builtin_amdgcn_fmed3f(a, 0.0f, amax); }

// Negated base-2 exponent of a Gaussian at a pixel offset (dx, dy) from its mean, from
// the factored conic and the per-column term a dx: s = -e = (a dx + b dy)^2 + (c dy)^2.
// A NaN offset gives NaN, which fails every threshold test.
__device__ inline float quad_s(float adx, float b, float c, float dy) {
    const float q1 = fmaf(b, dy, adx), q2 = c * dy;
    return fmaf(q1, q1, q2 * q2);
}

// Lane layout of a (TILE, PPT) workgroup: wave w owns a WW x WH pixel rectangle.
template <int TILE, int PPT>
struct Layout {
    static constexpr int NT = TILE * TILE / PPT;  // lanes per workgroup = records per batch
    static constexpr int NW = NT / kWave;         // waves per workgroup
    static constexpr int WH = TILE < 8 * PPT ? TILE : 8 * PPT;
    static constexpr int WW = kWave * PPT / WH;
    static constexpr bool CULL = NW > 1;  // a single wave owns the whole tile: binning culled already
    static_assert(WW * WH == kWave * PPT && TILE % WW == 0 && TILE % WH == 0, "unsupported raster shape");
    int w;                       // wave index within the tile
    int lx, ly;                  // tile-local column and first row of this lane
    float rx0, rx1, ry0, ry1;    // this wave's rectangle of pixel centres, tile-local
    // Of a workgroup of all the tile's waves, this thread's.  The wave index is uniform: keep
    // it (and the rectangle) in scalar registers.
    __device__ Layout() : Layout(__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave))) {}
    __device__ explicit Layout(int wave) : w(wave) {
        const int lane = lane_id();
        const int wx = (w % (TILE / WW)) * WW, wy = (w / (TILE / WW)) * WH;
        lx = wx + lane % WW;
        ly = wy + (lane / WW) * PPT;
        rx0 = (float)wx;
        rx1 = (float)(wx + WW - 1);
        ry0 = (float)wy;
        ry1 = (float)(wy + WH - 1);
    }
};

// Largest value of P d^2 + Q d t + R t^2 (R < 0) over t in [lo, hi], for fixed d.
__device__ inline float edge_max(float P, float Q, float R, float d, float lo, float hi) {
    const float t = fminf(hi, fmaxf(lo, -0.5f * Q * d * __builtin_amdgcn_rcpf(R)));
    return fmaf(fmaf(R, t, Q * d), t, P * d * d);
}

// Whether a staged record (s0 = (u, v, a, b), s1 = (c, -e_min, ...)) can reach its threshold
// at a pixel centre of the rectangle [x0, x1] x [y0, y1].  The exponent is concave with its
// maximum 0 at the mean, so it increases along any segment towards the mean: its maximum
// over the rectangle lies on an edge that faces the mean (a point elsewhere could move
// towards the mean inside the rectangle), or at the mean if that lies inside.  Both are
// covered by two segments: the column x = clamp(u, x0, x1) over [y0, y1] and the row
// y = clamp(v, y0, y1) over [x0, x1], each a one-dimensional concave quadratic (when the
// mean's x lies in [x0, x1], the column passes through the rectangle and the facing row
// holds the maximum; likewise for y).  The margin exceeds the float rounding of this
// evaluation plus that of the per-pixel evaluation (a few units in the last place of the
// sum of the terms' magnitudes), so the test never drops a record that a pixel accepts; it
// may keep a few that none does.
__device__ inline bool meets_rect(const float4 a, const float4 b, float x0, float x1, float y0, float y1) {
    // Expanded coefficients e = A dx^2 + B dx dy + C dy^2 of the factored conic (their
    // rounding is far inside the margin below).
    const float A = -a.z * a.z, B = -2.0f * a.z * a.w, C = -fmaf(a.w, a.w, b.x * b.x);
    const float ax = x0 - a.x, bx = x1 - a.x, ay = y0 - a.y, by = y1 - a.y;
    // Offsets of the column and the row from the mean: 0 where the mean's coordinate lies
    // inside the range, else that of the nearer edge (ax <= bx, ay <= by).
    const float cx = __builtin_amdgcn_fmed3f(0.0f, ax, bx), cy = __builtin_amdgcn_fmed3f(0.0f, ay, by);
    const float m = fmaxf(edge_max(A, B, C, cx, ay, by), edge_max(C, B, A, cy, ax, bx));
    const float DX = fmaxf(fabsf(ax), fabsf(bx)), DY = fmaxf(fabsf(ay), fabsf(by));
    const float S = fmaf(fabsf(A) * DX, DX, fmaf(fabsf(B) * DX, DY, fabsf(C) * DY * DY));
    return m >= -b.y - fmaf(0x1p-16f, S, 0x1p-10f);
}

// Ballot mask of the batch entries [c, c + 64) that this wave must walk.
template <bool CULL>
__device__ inline uint64_t batch_mask(const float4 *s0, const float4 *s1, int c, int cnt, float x0, float x1,
                                      float y0, float y1) {
    const int n = cnt - c;
    if (!CULL) return n >= kWave ? ~0ull : ((1ull << n) - 1ull);
    const int q = c + lane_id();  // below NT: c < cnt <= NT, both multiples of 64 apart from cnt
    const float4 a = s0[q], b = s1[q];
    // Whole 16-byte reads of consecutive records: the parts the test uses, read alone at a
    // 16-byte stride, would meet bank conflicts.
    asm volatile("" ::"v"(a.x), "v"(a.y), "v"(a.z), "v"(a.w), "v"(b.x), "v"(b.y), "v"(b.z), "v"(b.w));
    return ballot(q < cnt && meets_rect(a, b, x0, x1, y0, y1));
}

// This lane's bit of a lane mask, as the predicate of a select (the mask itself serves as it).
__device__ inline bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Orders a wave's LDS accesses across lanes (a wave's LDS instructions complete in order).
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// FRAME is the pointmap frame (0 world, 1 camera, 2 from the depth, Eq. 5).  In the
// camera frame the depth is the composited point's z and is not accumulated twice; in
// frame 2 the point is not accumulated at all.  COUNT: also write each pixel's number of
// contributing fragments (work statistics).
template <int TILE, int PPT, int FRAME, bool COUNT>
__global__ void __launch_bounds__(TILE *TILE / PPT)
k_raster_fwd(ViewTable vt, RasterSettings rs, const uint2 *__restrict__ ranges, const uint32_t *__restrict__ vals,
             const float4 *__restrict__ rec, float *__restrict__ out_rgb, float *__restrict__ out_depth,
             float *__restrict__ out_alpha, float *__restrict__ out_pm, float *__restrict__ t_final,
             uint32_t *__restrict__ last, uint32_t *__restrict__ contrib, uint8_t *__restrict__ visible,
             const uint32_t *__restrict__ order, uint32_t *__restrict__ tile_work, uint64_t *__restrict__ wmask,
             int64_t wstride, FrameHeader *__restrict__ hdr) {
    using L = Layout<TILE, PPT>;
    constexpr int NT = L::NT;
    __shared__ float4 s0[NT], s1[NT], s2[NT], s3[NT];
    __shared__ uint32_t block_work;
    __shared__ uint32_t block_walk[2];  // COUNT: list entries walked and accepted by the waves
    const TilePos tp = tile_pos<TILE>(vt, order, blockIdx.x);
    const uint2 rg = ranges[tp.gt];
    const L lay;
    const int lx = lay.lx, ly = lay.ly;
    const float px = (float)lx;
    const float amax = rs.alpha_max, tmin = rs.t_min;
    const int i = tp.tx * TILE + lx;

    float T[PPT], C0[PPT], C1[PPT], C2[PPT], D[PPT], X0[PPT], X1[PPT], X2[PPT];
    // The pixel's tile-local row while it composites; NaN once it has stopped (or if it
    // lies outside the view), which makes the exponent NaN, so that the acceptance test
    // stays one comparison whose lane mask is the wave's ballot as it stands.
    float py[PPT];
    uint32_t n_last[PPT], n_contrib[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        T[k] = 1.0f;
        C0[k] = C1[k] = C2[k] = D[k] = X0[k] = X1[k] = X2[k] = 0.f;
        n_last[k] = n_contrib[k] = 0u;
        const int j = tp.ty * TILE + ly + k;
        py[k] = (i < tp.W && j < tp.H) ? (float)(ly + k) : __builtin_nanf("");
    }
    // Whether any pixel of this lane is still compositing.  Re-evaluated once per 64
    // entries: a wave whose pixels have all stopped walks at most the rest of one mask.
    auto lane_live = [&]() {
        bool l = false;
#pragma unroll
        for (int k = 0; k < PPT; ++k) l |= py[k] == py[k];
        return l;
    };
    uint64_t live = ballot(lane_live());  // lanes with a pixel still compositing
    bool wave_live = live != 0ull;
    // The rectangle of the wave's live pixels, which the chunks are culled against: once
    // pixels stop, the entries that only they would take are not walked.  Scalar bit work on
    // the live-lane mask (lane = column + WW x lane row, PPT pixel rows per lane row).
    float lrx0 = lay.rx0, lrx1 = lay.rx1, lry0 = lay.ry0, lry1 = lay.ry1;
    auto live_rect = [&]() {
        uint64_t cols = live;
#pragma unroll
        for (int sh = 32; sh >= L::WW; sh >>= 1) cols |= cols >> sh;
        cols &= (L::WW >= 64 ? ~0ull : (1ull << L::WW) - 1ull);
        const int c0 = (int)__builtin_ctzll(cols), c1 = 63 - (int)__builtin_clzll(cols);
        const int r0 = (int)__builtin_ctzll(live) / L::WW, r1 = (63 - (int)__builtin_clzll(live)) / L::WW;
        lrx0 = lay.rx0 + (float)c0;
        lrx1 = lay.rx0 + (float)c1;
        lry0 = lay.ry0 + (float)(r0 * PPT);
        lry1 = lay.ry0 + (float)(r1 * PPT + PPT - 1);
    };
    if (wave_live) live_rect();
    uint32_t n_walked = 0u, n_accepted = 0u;  // COUNT: this wave's walked and accepted entries
    // The next batch's record indices are loaded one batch ahead, so staging waits on one
    // global read (the record) rather than two dependent ones.
    uint32_t vnext = rg.x + threadIdx.x < rg.y ? vals[rg.x + threadIdx.x] : 0u;
    for (uint32_t base = rg.x; base < rg.y; base += NT) {
        const uint32_t kk = base + threadIdx.x;
        const uint32_t vcur = vnext;
        if (kk + NT < rg.y) vnext = vals[kk + NT];
        if (kk < rg.y) stage(rec, vcur, tp.x0, tp.y0, s0, s1, s2, s3, threadIdx.x);
        __syncthreads();
        const int cnt = (int)min((uint32_t)NT, rg.y - base);
        for (int c = 0; c < cnt && wave_live; c += kWave) {
            uint64_t m = batch_mask<L::CULL>(s0, s1, c, cnt, lrx0, lrx1, lry0, lry1);
            if (COUNT) n_walked += (uint32_t)__popcll(m);
            uint64_t composited = 0ull;  // entries of this chunk accepted by one of the wave's live pixels
            while (m != 0ull) {
                const int q = c + (int)__builtin_ctzll(m);
                m &= m - 1ull;
                // All four words of the entry at once, before the test: the colour and point
                // reads share the address register, and their latency passes during the test
                // (most walked entries are composited).
                const float4 a = s0[q];
                const float4 b = s1[q];
                const float4 cc = s2[q];
                const float4 d = s3[q];
                // One 16-byte read now rather than a second, split read after the test.
                asm volatile("" ::"v"(b.z), "v"(b.w));
                const float dx = px - a.x;
                const float adx = a.z * dx;
                float sq[PPT];
                bool ok[PPT];
                uint64_t pass = 0ull;
#pragma unroll
                for (int k = 0; k < PPT; ++k) {
                    sq[k] = quad_s(adx, a.w, b.x, py[k] - a.y);
                    ok[k] = sq[k] <= b.y;
                    pass |= ballot(ok[k]);
                }
                if (pass == 0ull) continue;  // wave-uniform: nothing composites this entry
                // Some live pixel accepts the entry: it is composited there or stops that pixel.
                // The backward walks these entries (a superset of those it finds a valid
                // pixel for; it skips the rest), scalar work only.
                composited |= 1ull << (q - c);
                // Whole 16-byte reads: a 12-byte read of one address for the whole wave keeps
                // the LDS busy twice as long as a 16-byte one.
                asm volatile("" ::"v"(cc.w), "v"(d.w));
                const uint32_t rel = base - rg.x + (uint32_t)q + 1u;
                bool added = false;
#pragma unroll
                for (int k = 0; k < PPT; ++k) {
                    const float al = fminf(amax, b.z * __builtin_amdgcn_exp2f(-sq[k]));
                    const float Tn = fmaf(-al, T[k], T[k]);  // T (1 - alpha), rounded once
                    const bool add = ok[k] && !(Tn < tmin);
                    const bool stop = ok[k] && !add;  // one comparison; the masks combine in scalar code
                    const float w = add ? __fmul_rn(al, T[k]) : 0.0f;
                    C0[k] = fmaf(w, cc.x, C0[k]);
                    C1[k] = fmaf(w, cc.y, C1[k]);
                    C2[k] = fmaf(w, cc.z, C2[k]);
                    if (FRAME != 1) D[k] = fmaf(w, cc.w, D[k]);
                    if (FRAME != 2) {
                        X0[k] = fmaf(w, d.x, X0[k]);
                        X1[k] = fmaf(w, d.y, X1[k]);
                        X2[k] = fmaf(w, d.z, X2[k]);
                    }
                    T[k] = add ? Tn : T[k];
                    n_last[k] = add ? rel : n_last[k];
                    if (COUNT) n_contrib[k] += add ? 1u : 0u;
                    py[k] = stop ? __builtin_nanf("") : py[k];
                    added |= add;
                }
                if (visible) {  // uniform: marking requested
                    if (ballot(added) != 0ull && lane_id() == 0) visible[__float_as_uint(b.w)] = 1;
                }
            }
            if (COUNT) n_accepted += (uint32_t)__popcll(composited);
            if (composited != 0ull && lane_id() == 0) {
                // Entry q sits at list position base + q; the chunk's bits straddle at most
                // two words of this wave's plane.
                const uint64_t pos = (uint64_t)base + (uint64_t)c;
                uint64_t *w = wmask + (int64_t)lay.w * wstride + (int64_t)(pos >> 6);
                const int sh = (int)(pos & 63u);
                atomicOr((unsigned long long *)w, (unsigned long long)(composited << sh));
                if (sh != 0) atomicOr((unsigned long long *)(w + 1), (unsigned long long)(composited >> (64 - sh)));
            }
            const uint64_t now = ballot(lane_live());
            if (now != live) {  // wave-uniform: some pixels stopped in this chunk
                live = now;
                wave_live = live != 0ull;
                if (wave_live) live_rect();
            }
        }
        if (!__syncthreads_or(lane_live() ? 1 : 0)) break;
    }
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int j = tp.ty * TILE + ly + k;
        if (!(i < tp.W && j < tp.H)) continue;
        const int64_t e = (int64_t)j * tp.W + i;
        const int64_t pix = tp.pix_off + e, o3 = 3 * tp.pix_off + e, plane = tp.plane;
        out_rgb[o3] = fmaf(T[k], rs.bg[0], C0[k]);
        out_rgb[o3 + plane] = fmaf(T[k], rs.bg[1], C1[k]);
        out_rgb[o3 + 2 * plane] = fmaf(T[k], rs.bg[2], C2[k]);
        const float depth = FRAME == 1 ? X2[k] : D[k];
        out_depth[pix] = depth;
        out_alpha[pix] = 1.0f - T[k];
        float x0 = X0[k], x1 = X1[k], x2 = X2[k];
        if (FRAME == 2) {
            const float rx = ((float)i - vt.cx[tp.v]) / vt.fx[tp.v];
            const float ry = ((float)j - vt.cy[tp.v]) / vt.fy[tp.v];
            x0 = depth * rx;
            x1 = depth * ry;
            x2 = depth;
        }
        out_pm[o3] = x0;
        out_pm[o3 + plane] = x1;
        out_pm[o3 + 2 * plane] = x2;
        t_final[pix] = T[k];
        last[pix] = n_last[k];
        if (COUNT) contrib[pix] = n_contrib[k];
    }
    if (COUNT) {  // the launch's walked and accepted (wave, entry) pairs, one atomic pair per workgroup
        if (threadIdx.x == 0) block_walk[0] = block_walk[1] = 0u;
        __syncthreads();
        if (lane_id() == 0) {
            atomicAdd(&block_walk[0], n_walked);
            atomicAdd(&block_walk[1], n_accepted);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            atomicAdd(reinterpret_cast<unsigned long long *>(&hdr->walked), (unsigned long long)block_walk[0]);
            atomicAdd(reinterpret_cast<unsigned long long *>(&hdr->accepted), (unsigned long long)block_walk[1]);
        }
    }
    {
        if (threadIdx.x == 0) block_work = 0u;
        __syncthreads();
        uint32_t m = 0u;
#pragma unroll
        for (int k = 0; k < PPT; ++k) m = max(m, n_last[k]);
        for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
        if (lane_id() == 0) atomicMax(&block_work, m);
        __syncthreads();
        if (threadIdx.x == 0) tile_work[tp.gt] = block_work;
    }
}

// Launch of independent waves, one to a workgroup: workgroup b -> (slot of the tile order,
// wave of the tile).  Workgroups go to the 8 XCDs in turn: the waves of a tile are 8 apart, so
// that they run on one XCD and share its L2.
template <int NW>
inline uint32_t wave_grid(int n_tiles) {
    return (uint32_t)((n_tiles + 7) / 8 * 8 * NW);
}
template <int NW>
__device__ inline void wave_place(uint32_t b, uint32_t &slot, int &w) {
    slot = b / (8 * NW) * 8 + (b & 7u);
    w = (int)(b / 8 % NW);
}

constexpr int kChunk = kWave;       // list entries staged at a time
constexpr int kPlane = kChunk + 2;  // words of a staging plane: quad-lane writes without bank conflicts
// A stopped pixel's row: a quiet NaN carrying the chunk slot of the entry that stopped it.
constexpr uint32_t kNan = 0x7fc00000u, kNanStop = 0x7fc00040u;

// Forward compositing by independent waves (one pixel per lane): a wave owns its rectangle of a
// tile and walks the tile's list on its own, with no barrier.  It is bound by the latency of
// the longest waves where the launch holds only a few rounds of them: the workgroup form above
// meets at two barriers per 256 entries, where the busiest wave walks 1.34-1.41 times the mean,
// and walks one entry at a time, waiting for its LDS reads and its exponent each.
//
// Per 64 entries: the records arrive four lanes per record (one 16-byte word each, loaded one
// chunk ahead: 16 lines per load instead of 64), go to four LDS planes, and lane q converts
// record q to tile-local coordinates and tests it against the rectangle of the wave's live
// pixels.  The survivors are walked in pairs, so that the LDS latency, the tests and the
// exponents of two entries overlap.
template <int TILE, int FRAME, bool MARK>
__global__ void __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(5)))
k_raster_fwd_waves(ViewTable vt, RasterSettings rs, const uint2 *__restrict__ ranges,
                   const uint32_t *__restrict__ vals, const float4 *__restrict__ rec, float *__restrict__ out_rgb,
                   float *__restrict__ out_depth, float *__restrict__ out_alpha, float *__restrict__ out_pm,
                   float *__restrict__ t_final, uint32_t *__restrict__ last, uint8_t *__restrict__ visible,
                   const uint32_t *__restrict__ order, uint32_t *__restrict__ tile_work,
                   uint64_t *__restrict__ wmask, int64_t wstride) {
    using L = Layout<TILE, 1>;
    __shared__ float4 st[4 * kPlane];
    uint32_t tslot;
    int wv;
    wave_place<L::NW>(blockIdx.x, tslot, wv);
    if (tslot >= (uint32_t)vt.tile_off[vt.n_views]) return;
    const TilePos tp = tile_pos<TILE>(vt, order, tslot);
    const uint2 rg = ranges[tp.gt];
    const L lay(wv);
    const int lane = lane_id();
    const float px = (float)lay.lx;
    const float amax = rs.alpha_max, tmin = rs.t_min;
    const int i = tp.tx * TILE + lay.lx, j = tp.ty * TILE + lay.ly;
    const bool inside = i < tp.W && j < tp.H;

    float T = 1.0f, C0 = 0.f, C1 = 0.f, C2 = 0.f, D = 0.f, X0 = 0.f, X1 = 0.f, X2 = 0.f;
    // The pixel's tile-local row while it composites; NaN once it has stopped (or if it
    // lies outside the view), which makes the exponent NaN, so that the acceptance test
    // stays one comparison whose lane mask is the wave's ballot as it stands.
    float py = inside ? (float)lay.ly : __uint_as_float(kNan);
    // A bound on the list entries that the backward considers: an entry before it contributes
    // to the pixel exactly when its alpha reaches alpha_min.  A stopped pixel's is the entry
    // that stopped it; otherwise the end of the last chunk in which it composited, which
    // shows in T, unless the settings admit an alpha that T (1 - alpha) rounds away: then the
    // end of the last chunk that it met.
    uint32_t n_last = 0u;
    const bool faint = !(rs.alpha_min >= 0x1p-23f && tmin >= 0x1p-100f);
    uint64_t live = ballot(py == py);  // lanes that still composite, re-evaluated once per chunk
    // The rectangle of the wave's live pixels, which the chunks are culled against: once
    // pixels stop, the entries that only they would take are not walked.  Scalar bit work on
    // the live-lane mask (lane = column + WW x row).
    float lrx0 = lay.rx0, lrx1 = lay.rx1, lry0 = lay.ry0, lry1 = lay.ry1;
    auto live_rect = [&]() {
        uint64_t cols = live;
#pragma unroll
        for (int sh = 32; sh >= L::WW; sh >>= 1) cols |= cols >> sh;
        cols &= (1ull << L::WW) - 1ull;
        const int c0 = (int)__builtin_ctzll(cols), c1 = 63 - (int)__builtin_clzll(cols);
        lrx0 = lay.rx0 + (float)c0;
        lrx1 = lay.rx0 + (float)c1;
        lry0 = lay.ry0 + (float)((int)__builtin_ctzll(live) / L::WW);
        lry1 = lay.ry0 + (float)((63 - (int)__builtin_clzll(live)) / L::WW);
    };
    if (live != 0ull) live_rect();

    // Lane 4 i + w holds word w of records 16 r + i (r = 0..3) of a chunk.  The records are
    // loaded one chunk ahead and their indices two, so that a step waits on no load it has
    // just issued.  Entries past the list's end stage its last one, which no mask holds.
    const uint32_t n = rg.y - rg.x;
    const uint32_t *list = vals + rg.x;
    uint32_t nidx[4];
    v4f raw[4];  // a plain vector: as an array of float4 it would live in scratch memory
    auto load_idx = [&](uint32_t c0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) nidx[r] = list[min(c0 + 16u * r + ((uint32_t)lane >> 2), n - 1u)];
    };
    auto load_raw = [&]() {
#pragma unroll
        for (int r = 0; r < 4; ++r) raw[r] = reinterpret_cast<const v4f *>(rec)[4 * (int64_t)nidx[r] + (lane & 3)];
    };
    if (live != 0ull && n != 0u) {
        load_idx(0u);
        load_raw();
        if (n > (uint32_t)kChunk) load_idx(kChunk);
    }
    for (uint32_t c0 = 0u; c0 < n && live != 0ull; c0 += kChunk) {
        wave_sync();  // the previous chunk has been read
        v4f *dst = reinterpret_cast<v4f *>(st) + (lane & 3) * kPlane + (lane >> 2);
#pragma unroll
        for (int r = 0; r < 4; ++r) dst[16 * r] = raw[r];
        wave_sync();
        if (c0 + kChunk < n) {
            load_raw();
            if (c0 + 2 * kChunk < n) load_idx(c0 + 2 * kChunk);
        }
        // (u, v, a, b), (c, threshold, opacity, NaN | q) of record q = this lane.
        const float4 r0 = st[lane], r1 = st[kPlane + lane], r3 = st[3 * kPlane + lane];
        asm volatile("" ::"v"(r3.x), "v"(r3.y), "v"(r3.z), "v"(r3.w));  // 16 bytes: no bank conflicts
        const float4 sa = make_float4((r0.x - tp.x0) + r0.z, (r0.y - tp.y0) + r0.w, r1.x, r1.y);
        const float4 sb = make_float4(r1.z, r3.w, r1.w, __uint_as_float(kNanStop | (uint32_t)lane));
        uint64_t m = ballot((!L::CULL || meets_rect(sa, sb, lrx0, lrx1, lry0, lry1)) && c0 + (uint32_t)lane < n);
        st[lane] = sa;
        st[kPlane + lane] = sb;
        wave_sync();
        const float T0 = T;
        uint64_t composited = 0ull;  // entries of this chunk accepted by one of the wave's live pixels
        uint64_t marked = 0ull;      // MARK: entries that contribute to a pixel
        // Reads entry q (its words at one address for the whole wave: 16-byte reads; a
        // 12-byte one keeps the LDS busy twice as long as a 16-byte one, an 8-byte one half
        // as long).  In the camera frame the point's z is the depth, the colour's fourth word.
        auto fetch = [&](int q, float4 &a, float4 &b, float4 &cc, float4 &d) {
            a = st[q];
            b = st[kPlane + q];
            cc = st[2 * kPlane + q];
            if (FRAME == 0) d = st[3 * kPlane + q];
            if (FRAME == 1) {
                const float2 xy = *reinterpret_cast<const float2 *>(&st[3 * kPlane + q]);
                d = make_float4(xy.x, xy.y, cc.w, 0.f);
            }
            if (FRAME == 2) d = make_float4(0.f, 0.f, 0.f, 0.f);
            asm volatile("" ::"v"(cc.w));  // whole 16-byte reads where three words are used
            if (FRAME == 0) asm volatile("" ::"v"(d.w));
        };
        auto exponent = [&](const float4 &a, const float4 &b) {
            const float dx = px - a.x;
            return quad_s(a.z * dx, a.w, b.x, py - a.y);
        };
        // One entry's share of the wave's pixels, which may stop some of them (ok: the lanes
        // that accept it; stopped lanes leave ok_next, the next entry's).  special: some opacity
        // of the chunk reaches alpha_max (otherwise o exp2(-s) <= o < alpha_max and the clamp is
        // the identity), or some colour or point is not finite: then an entry that no pixel
        // accepts is left out (its weight 0 times infinity would be NaN; otherwise it adds 0).
        auto composite = [&](auto special, int q, const float4 &b, const float4 &cc, const float4 &d, float sq,
                             uint64_t ok, uint64_t &ok_next) {
            // Some live pixel accepts the entry: it is composited there or stops that pixel.
            // The backward walks these entries (a superset of those it finds a valid pixel for;
            // it skips the rest), scalar work only.
            if (decltype(special)::value && ok == 0ull) return;  // wave-uniform
            composited |= ok != 0ull ? 1ull << q : 0ull;
            float al = b.z * __builtin_amdgcn_exp2f(-sq);
            if (decltype(special)::value) al = clamp_alpha(al, amax);
            const float Tn = fmaf(-al, T, T);  // T (1 - alpha), rounded once
            // One comparison; the lane masks combine in scalar code.
            const uint64_t over = ballot(!(Tn < tmin));
            const uint64_t add = ok & over, stop = ok & ~over;
            ok_next &= ~stop;
            if (MARK) marked |= add != 0ull ? 1ull << q : 0ull;
            const float w = in_mask(add) ? __fmul_rn(al, T) : 0.0f;
            C0 = fmaf(w, cc.x, C0);
            C1 = fmaf(w, cc.y, C1);
            C2 = fmaf(w, cc.z, C2);
            if (FRAME != 1) D = fmaf(w, cc.w, D);
            if (FRAME != 2) {
                X0 = fmaf(w, d.x, X0);
                X1 = fmaf(w, d.y, X1);
                X2 = fmaf(w, d.z, X2);
            }
            T = in_mask(add) ? Tn : T;
            py = in_mask(stop) ? b.w : py;  // NaN with the entry's slot
        };
        auto walk_pairs = [&](auto special) {
            for (int p = (int)__popcll(m) >> 1; p > 0; --p) {
                const int q0 = (int)__builtin_ctzll(m);
                m ^= 1ull << q0;
                const int q1 = (int)__builtin_ctzll(m);
                m ^= 1ull << q1;
                float4 a0, b0, e0, d0, a1, b1, e1, d1;
                fetch(q0, a0, b0, e0, d0);
                fetch(q1, a1, b1, e1, d1);
                asm volatile("" ::"v"(b0.w), "v"(b1.w));
                const float s0 = exponent(a0, b0), s1 = exponent(a1, b1);
                uint64_t ok0 = ballot(s0 <= b0.y), ok1 = ballot(s1 <= b1.y), none = 0ull;
                composite(special, q0, b0, e0, d0, s0, ok0, ok1);
                composite(special, q1, b1, e1, d1, s1, ok1, none);
            }
        };
        if ((ballot(sb.z >= amax || sb.x < 0.0f) & m) != 0ull) walk_pairs(std::true_type{});
        else walk_pairs(std::false_type{});
        if (m != 0ull) {  // the last of an odd number
            const int q = (int)__builtin_ctzll(m);
            float4 a, b, cc, d;
            fetch(q, a, b, cc, d);
            asm volatile("" ::"v"(b.w));
            const float sq = exponent(a, b);
            uint64_t none = 0ull;
            composite(std::true_type{}, q, b, cc, d, sq, ballot(sq <= b.y), none);
        }
        if (MARK) {
            if ((marked >> lane) & 1ull) visible[list[c0 + (uint32_t)lane]] = 1;
        }
        if (composited != 0ull && lane == 0) {
            // Entry q sits at list position rg.x + c0 + q; the chunk's bits straddle at most
            // two words of this wave's plane.
            const uint64_t pos = (uint64_t)rg.x + c0;
            uint64_t *w = wmask + (int64_t)wv * wstride + (int64_t)(pos >> 6);
            const int sh = (int)(pos & 63u);
            atomicOr((unsigned long long *)w, (unsigned long long)(composited << sh));
            if (sh != 0) atomicOr((unsigned long long *)(w + 1), (unsigned long long)(composited >> (64 - sh)));
        }
        n_last = T != T0 || (faint && py == py) ? min(c0 + (uint32_t)kChunk, n) : n_last;
        const uint64_t now = ballot(py == py);
        if (now != live) {  // wave-uniform: some pixels stopped in this chunk
            const uint32_t pb = __float_as_uint(py);
            if ((pb & ~63u) == kNanStop) {
                n_last = c0 + (pb & 63u);
                py = __uint_as_float(kNan);
            }
            live = now;
            if (live != 0ull) live_rect();
        }
    }
    if (inside) {
        const int64_t e = (int64_t)j * tp.W + i;
        const int64_t pix = tp.pix_off + e, o3 = 3 * tp.pix_off + e, plane = tp.plane;
        out_rgb[o3] = fmaf(T, rs.bg[0], C0);
        out_rgb[o3 + plane] = fmaf(T, rs.bg[1], C1);
        out_rgb[o3 + 2 * plane] = fmaf(T, rs.bg[2], C2);
        const float depth = FRAME == 1 ? X2 : D;
        out_depth[pix] = depth;
        out_alpha[pix] = 1.0f - T;
        if (FRAME == 2) {
            X0 = depth * (((float)i - vt.cx[tp.v]) / vt.fx[tp.v]);
            X1 = depth * (((float)j - vt.cy[tp.v]) / vt.fy[tp.v]);
            X2 = depth;
        }
        out_pm[o3] = X0;
        out_pm[o3 + plane] = X1;
        out_pm[o3 + 2 * plane] = X2;
        t_final[pix] = T;
        last[pix] = n_last;
    }
    uint32_t work = n_last;  // the tile's deepest entry: the largest over its waves (cleared before the launch)
    for (int off = 32; off > 0; off >>= 1) work = max(work, (uint32_t)__shfl_xor((int)work, off, 64));
    if (lane == 0 && work != 0u) atomicMax(tile_work + tp.gt, work);
}

__device__ inline float load_or0(const float *p, int64_t i) { return p ? p[i] : 0.0f; }

// Which per-record sums the backward forms, in value order, and the accumulator column
// of each: [sum g] [moments of g: 5] [colour: 3] [depth] [point: 3].  A pose-only pass
// (tracking) needs no opacity or colour gradient; the camera frame carries the depth
// gradient in the point's z, and frame 2 has no point term.
template <bool POSE_ONLY, int FRAME>
struct BwdValues {
    static constexpr bool kOpacity = !POSE_ONLY, kColour = !POSE_ONLY;
    static constexpr bool kDepth = FRAME != 1, kPoint = FRAME != 2;
    static constexpr int N = (kOpacity ? 1 : 0) + 5 + (kColour ? 3 : 0) + (kDepth ? 1 : 0) + (kPoint ? 3 : 0);
    static constexpr int NR = N <= 8 ? 8 : (N <= 12 ? 12 : 16);  // reduce-scatter width
    // Column of value k in bits [4k, 4k + 4).
    static constexpr uint64_t columns() {
        uint64_t c = 0;
        int k = 0;
        auto put = [&](int col) { c |= (uint64_t)col << (4 * k++); };
        if (kOpacity) put(0);
        for (int j = 1; j <= 5; ++j) put(j);
        if (kColour) { put(7); put(8); put(9); }
        if (kDepth) put(6);
        if (kPoint) { put(10); put(11); put(12); }
        return c;
    }
    static constexpr uint64_t kColumns = columns();
    // The per-pixel weighted sums (colour, depth, point: weight w times the pixel's upstream
    // gradient), their count and their columns, 4 bits each.
    static constexpr int NW = (kColour ? 3 : 0) + (kDepth ? 1 : 0) + (kPoint ? 3 : 0);
    static constexpr uint32_t kWColumns = (uint32_t)(kColumns >> (4 * (N - NW)));
};

// A backward with another alpha_min than its forward's: its own, for its own thresholds; else 0.
__device__ inline float own_alpha_min(const RasterSettings &rs, const FrameHeader *hdr) {
    return hdr->alpha_min == rs.alpha_min ? 0.0f : rs.alpha_min;
}

// The frame state's layout follows the views, Gaussian count and tile of the call: unless they
// (and the pointmap frame of the records) are the forward's, and the forward's lists are
// complete, a backward may read nothing of it.  The test is uniform over the launch; one lane
// records the refusal for gspm_frame_status.
__device__ inline bool frame_matches(const ViewTable &vt, FrameHeader *hdr, int tile, int frame, int64_t n_records) {
    if (hdr->magic != kFrameMagic || hdr->overflow != 0u || hdr->sort_stall != 0u || hdr->tile != (uint32_t)tile ||
        hdr->n_views != (uint32_t)vt.n_views || hdr->n_tiles != (uint32_t)vt.tile_off[vt.n_views] ||
        hdr->n_pixels != (uint64_t)vt.pix_off[vt.n_views] || hdr->n_records != (uint64_t)n_records ||
        hdr->frame != (uint32_t)frame) {
        if (blockIdx.x == 0 && threadIdx.x == 0) hdr->bwd_error = 1u;
        return false;
    }
    return true;
}

template <int TILE, int PPT, bool POSE_ONLY, int FRAME>
__global__ void __launch_bounds__(TILE *TILE / PPT)
k_raster_bwd(ViewTable vt, RasterSettings rs, const uint2 *__restrict__ ranges, const uint32_t *__restrict__ vals,
             const float4 *__restrict__ rec, const uint32_t *__restrict__ last, const float *__restrict__ t_final,
             gspm_const_images fwd, gspm_const_images up, float *__restrict__ grad2d,
             const uint32_t *__restrict__ order, FrameHeader *__restrict__ hdr, int64_t n_records) {
    if (!frame_matches(vt, hdr, TILE, FRAME, n_records)) return;
    using L = Layout<TILE, PPT>;
    using V = BwdValues<POSE_ONLY, FRAME>;
    constexpr int NT = L::NT;
    __shared__ float4 s0[NT], s1[NT], s2[NT], s3[NT];
    __shared__ uint32_t block_last;
    const TilePos tp = tile_pos<TILE>(vt, order, blockIdx.x);
    const uint2 rg = ranges[tp.gt];
    const L lay;
    const int lx = lay.lx, ly = lay.ly;
    const float px = (float)lx;
    const float amax = rs.alpha_max, own_min = own_alpha_min(rs, hdr);
    const int i = tp.tx * TILE + lx;
    // Per-pixel upstream gradient and, to start the walk's remainder Rem, the total
    // G = sum_k w_k (g . e_k) + T_final (g_C . bg) that the forward's outputs give.
    uint32_t my_last[PPT];
    float gC0[PPT], gC1[PPT], gC2[PPT], gD[PPT], gA[PPT], gX0[PPT], gX1[PPT], gX2[PPT], Rem[PPT], py[PPT];
    float T[PPT];
    uint32_t thread_last = 0;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        my_last[k] = 0;
        gC0[k] = gC1[k] = gC2[k] = gD[k] = gA[k] = gX0[k] = gX1[k] = gX2[k] = Rem[k] = 0.f;
        T[k] = 1.0f;
        py[k] = (float)(ly + k);
        const int j = tp.ty * TILE + ly + k;
        if (!(i < tp.W && j < tp.H)) continue;
        const int64_t e = (int64_t)j * tp.W + i;
        const int64_t pix = tp.pix_off + e, o3 = 3 * tp.pix_off + e, plane = tp.plane;
        my_last[k] = last[pix];
        gC0[k] = load_or0(up.rgb, o3);
        gC1[k] = load_or0(up.rgb, o3 + plane);
        gC2[k] = load_or0(up.rgb, o3 + 2 * plane);
        gD[k] = load_or0(up.depth, pix);
        gA[k] = load_or0(up.alpha, pix);
        gX0[k] = load_or0(up.pointmap, o3);
        gX1[k] = load_or0(up.pointmap, o3 + plane);
        gX2[k] = load_or0(up.pointmap, o3 + 2 * plane);
        const float Tf = t_final[pix];
        const bool none = gC0[k] == 0.f && gC1[k] == 0.f && gC2[k] == 0.f && gD[k] == 0.f && gA[k] == 0.f &&
                          gX0[k] == 0.f && gX1[k] == 0.f && gX2[k] == 0.f;
        // The rgb output holds sum_k w_k c_k + T_final bg, which is exactly what G needs.
        Rem[k] = gC0[k] * fwd.rgb[o3] + gC1[k] * fwd.rgb[o3 + plane] + gC2[k] * fwd.rgb[o3 + 2 * plane] +
                gD[k] * fwd.depth[pix] + gA[k] * (1.0f - Tf);
        if (FRAME == 2) {
            // Eq. 5: the pointmap is D K^-1 [i, j, 1]^T, a function of the depth only.
            const float rx = ((float)i - vt.cx[tp.v]) / vt.fx[tp.v];
            const float ry = ((float)j - vt.cy[tp.v]) / vt.fy[tp.v];
            const float gXD = gX0[k] * rx + gX1[k] * ry + gX2[k];
            Rem[k] += gXD * fwd.depth[pix];
            gD[k] += gXD;
            gX0[k] = gX1[k] = gX2[k] = 0.f;
        } else {
            Rem[k] += gX0[k] * fwd.pointmap[o3] + gX1[k] * fwd.pointmap[o3 + plane] +
                     gX2[k] * fwd.pointmap[o3 + 2 * plane];
        }
        if (FRAME == 1) {
            // The depth is the point's z: one gradient for both.
            gX2[k] += gD[k];
            gD[k] = 0.f;
        }
        if (none) my_last[k] = 0;  // nothing flows back from this pixel
        thread_last = max(thread_last, my_last[k]);
    }
    if (threadIdx.x == 0) block_last = 0;
    __syncthreads();
    uint32_t wave_last = thread_last;
    for (int off = 32; off > 0; off >>= 1) wave_last = max(wave_last, (uint32_t)__shfl_xor((int)wave_last, off, 64));
    wave_last = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_last);  // uniform: keep it scalar
    if (lane_id() == 0) atomicMax(&block_last, wave_last);
    __syncthreads();
    const uint32_t end = rg.x + block_last;

    // The entries that one of this wave's live pixels accepted in the forward (its bit plane
    // after the pair list): every entry with a valid pixel here, plus the few that only
    // stopped a pixel, so the walk needs no culling test and meets almost no entry without
    // a contribution.
    const int64_t cap = (int64_t)hdr->capacity;
    const uint64_t *plane = wmask_at(vals, cap) + (int64_t)lay.w * wmask_stride(cap);
    // A forward with another number of pixels per lane had other waves: cull instead.
    const bool use_bits = hdr->ppt == (uint32_t)PPT;
    auto wave_bits = [&](uint32_t pos) {  // the 64 bits of list positions pos .. pos + 63
        const uint64_t *wp = plane + (pos >> 6);
        const int sh = (int)(pos & 63u);
        uint64_t m = wp[0] >> sh;
        if (sh != 0) m |= wp[1] << (64 - sh);
        return m;
    };
    // One list entry (its staged record, and its position rel in the tile's list): the
    // per-pixel recomputation and this wave's sums for it.
    auto walk_record = [&](const float4 &a, const float4 &b, const float4 &cc, const float4 &d, uint32_t rel) {
        const float dx = px - a.x;
        const float adx = a.z * dx;
        float sq[PPT];
        bool valid[PPT];
        uint64_t any = 0ull;
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            sq[k] = quad_s(adx, a.w, b.x, py[k] - a.y);
            // Two comparisons whose lane masks are combined by a scalar AND.
            valid[k] = rel < my_last[k] && sq[k] <= b.y;
            any |= ballot(valid[k]);
        }
        if (any == 0ull) return;  // wave-uniform
        float v[V::NR];
#pragma unroll
        for (int t = V::N; t < V::NR; ++t) v[t] = 0.f;
        // The per-pixel terms, in two forms.  alpha = min(alpha_max, o exp2(-s)) can only be
        // clamped when the opacity o reaches alpha_max (rare), where a clamped alpha passes
        // no gradient; otherwise alpha is o exp2(-s) itself (o exp2(-s) <= o for s >= 0).
        auto pixel_terms = [&](auto may_clamp) {
            constexpr bool kClamp = decltype(may_clamp)::value;
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                // The first pixel assigns, later ones accumulate (x + 0 is not folded).
                auto add = [&](int t, float x) { v[t] = k == 0 ? x : v[t] + x; };
                auto mad = [&](int t, float x, float y) { v[t] = k == 0 ? x * y : fmaf(x, y, v[t]); };
                // Branch-free: an invalid pixel takes alpha = 0, so its weight and its alpha
                // gradient are 0 and T * (1 - 0) leaves T unchanged.
                const float dy = py[k] - a.y;
                const float ao = b.z * __builtin_amdgcn_exp2f(-sq[k]);
                const float al = valid[k] ? (kClamp ? clamp_alpha(ao, amax) : ao) : 0.0f;
                const float w = __fmul_rn(al, T[k]);
                float sv = fmaf(gC0[k], cc.x, fmaf(gC1[k], cc.y, fmaf(gC2[k], cc.z, gA[k])));
                if (V::kDepth) sv = fmaf(gD[k], cc.w, sv);
                if (V::kPoint) sv = fmaf(gX0[k], d.x, fmaf(gX1[k], d.y, fmaf(gX2[k], d.z, sv)));
                // Rem = G - sum of w s over this and earlier fragments: the later fragments'
                // share plus the background term.
                Rem[k] = fmaf(-w, sv, Rem[k]);
                const float one_m = __fsub_rn(1.0f, al);
                const float dLda = T[k] * sv - Rem[k] * __builtin_amdgcn_rcpf(one_m);
                const float g = kClamp && al >= amax ? 0.0f : dLda * al;
                T[k] = fmaf(-al, T[k], T[k]);  // as in the forward
                const float gdx = g * dx, gdy = g * dy;
                int t = 0;
                if (V::kOpacity) add(t++, g);
                add(t++, gdx);
                add(t++, gdy);
                mad(t++, gdx, dx);
                mad(t++, gdy, dx);
                mad(t++, gdy, dy);
                if (V::kColour) {
                    mad(t++, w, gC0[k]);
                    mad(t++, w, gC1[k]);
                    mad(t++, w, gC2[k]);
                }
                if (V::kDepth) mad(t++, w, gD[k]);
                if (V::kPoint) {
                    mad(t++, w, gX0[k]);
                    mad(t++, w, gX1[k]);
                    mad(t++, w, gX2[k]);
                }
            }
        };
        // The opacity is wave-uniform; both are positive, so their bit patterns order as they do.
        if (__builtin_amdgcn_readfirstlane(__float_as_int(b.z)) >= __float_as_int(amax)) {
            pixel_terms(std::true_type{});
        } else {
            pixel_terms(std::false_type{});
        }
        int idx;
        const float tot = wave_reduce_scatter(v, idx);
        if (idx >= 0 && idx < V::N && tot != 0.f) {
            // The record index is wave-uniform: a scalar row base plus the lane's column.
            const uint32_t r = (uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(b.w));
            const uint32_t col = (uint32_t)((V::kColumns >> (4 * idx)) & 15u);
            unsafeAtomicAdd(grad2d + (int64_t)r * kG2 + col, tot);
        }
    };
    // The next batch's record indices are loaded one batch ahead, so staging waits on one
    // global read (the record) rather than two dependent ones.
    uint32_t vnext = (rg.x + threadIdx.x < end) ? vals[rg.x + threadIdx.x] : 0u;
    for (uint32_t base = rg.x; base < end; base += NT) {
        const uint32_t kk = base + threadIdx.x;
        const uint32_t vcur = vnext;
        if (kk + NT < end) vnext = vals[kk + NT];
        const uint64_t bits0 = use_bits ? wave_bits(base) : 0ull;  // read while the batch is staged
        if (kk < end) stage(rec, vcur, tp.x0, tp.y0, s0, s1, s2, s3, threadIdx.x, own_min);
        __syncthreads();
        const int cnt = (int)min((uint32_t)NT, end - base);
        const uint32_t rel0 = base - rg.x;
        for (int c = 0; c < cnt && rel0 + (uint32_t)c < wave_last; c += kWave) {
            uint64_t m;
            if (use_bits) {
                m = c == 0 ? bits0 : wave_bits(base + (uint32_t)c);
                if (cnt - c < kWave) m &= (1ull << (cnt - c)) - 1ull;  // the next tile's entries
            } else {
                m = batch_mask<L::CULL>(s0, s1, c, cnt, lay.rx0, lay.rx1, lay.ry0, lay.ry1);
            }
            // Entries at or past the wave's last contributing one are not walked.
            const uint32_t lim = wave_last - (rel0 + (uint32_t)c);
            if (lim < (uint32_t)kWave) m &= (1ull << lim) - 1ull;
            while (m != 0ull) {
                const int q = c + (int)__builtin_ctzll(m);
                m &= m - 1ull;
                const uint32_t rel = rel0 + (uint32_t)q;
                const float4 a = s0[q];
                const float4 b = s1[q];
                const float4 cc = s2[q];
                const float4 d = s3[q];
                // One 16-byte read now rather than a second, split read after the test.
                asm volatile("" ::"v"(b.z), "v"(b.w));
                walk_record(a, b, cc, d, rel);
            }
        }
        __syncthreads();
    }
}

constexpr int kBatch = 16;  // entries staged, walked and summed at a time: four lanes load one record
constexpr int kBatchPlane = kBatch + 2;  // words of a staging plane: quad-lane writes without bank conflicts
constexpr uint32_t kQueue = 80;          // ring of entries waiting to be staged: at most 15 + 64
constexpr int kSumPitch = 33;            // words of an entry's g and w: 16 entries' words in 16 different bank groups
constexpr int kOutPitch = 20;            // floats of an entry's sums: 16-byte writes without bank conflicts

// Backward compositing, one pixel per lane, by independent waves.
//
// A wave stages the entries its bits mark 16 at a time (loaded one batch ahead) and walks them
// four at a time, so that their LDS reads, exponents and reciprocals overlap; only the
// transmittance and the remainder pass from one entry to the next.
//
// Per entry the wave needs up to 13 sums over its 64 pixels: Out[f] = sum_p F_f(p) H(p), where
// the six moments take F = 1, x, y, x^2, xy, y^2 (pixel offsets from the wave rectangle's
// centre) and H = g = alpha dL/dalpha, and the colour, depth and point sums take F = the
// pixel's upstream gradient and H = w = alpha T.  The 16 entries' g and w pass through LDS to the
// matrix cores, 4 x 4 x 1 products in 16 blocks: four rows f by four entries each, one pixel per
// instruction.  Each sum is thus one chain of fused multiply-adds over the pixels 0 .. 63 in this
// order.  The order is part of the result: the parameter pass multiplies the moments by the
// conic twice, which for a near-degenerate Gaussian magnifies their last bits until a few of these
// carry the norm of the gradients of means, quats and log_scales.  (Sums by rows of pixels on the
// vector units, with one reciprocal for four entries, took 1.10 ms and 192 us where this takes
// 1.17 ms and 207 us, but their gradients lay 2 to 4 times further from these than two runs of one
// form from each other.)
//
// Vector issue (38 instructions per entry and wave), the matrix cores (32 cycles) and the LDS (26
// cycles, 57% of its time) bind it together.  8 views with 1M Gaussians: 1.40 ms before
// (workgroups, entries one by one, 16x16x4 products: 64 cycles per entry), 1.17 ms now; pose-only
// at 960x640 with 500k: 274 and 207 us.  Four waves per SIMD fit the LDS.  (Moments accumulated in
// float64 rows, which would take the order of the atomics out of the gradients: 1.95 ms.)
template <int TILE, bool POSE_ONLY, int FRAME>
__global__ void __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(4)))
k_raster_bwd_waves(ViewTable vt, RasterSettings rs, const uint2 *__restrict__ ranges,
                   const uint32_t *__restrict__ vals, const float4 *__restrict__ rec,
                   const uint32_t *__restrict__ last, const float *__restrict__ t_final, gspm_const_images fwd,
                   gspm_const_images up, float *__restrict__ grad2d, const uint32_t *__restrict__ order,
                   FrameHeader *__restrict__ hdr, int64_t n_records) {
    if (!frame_matches(vt, hdr, TILE, FRAME, n_records)) return;
    using L = Layout<TILE, 1>;
    using V = BwdValues<POSE_ONLY, FRAME>;
    static_assert(L::WW == 8 && L::WH == 8, "8 x 8 wave rectangles");
    // Staged entries: (u, v, a, b), (c, threshold, opacity, list position), colour and z, point
    // and record index.
    __shared__ float4 st[4 * kBatchPlane];
    __shared__ uint2 queue[kQueue];  // (record, list position) of the marked entries
    // Entry e's g, pixels 0 .. 63, then its w; over the same words afterwards its sums.
    __shared__ float4 gw[kSumPitch * kBatch];
    uint32_t tslot;
    int wv;
    wave_place<L::NW>(blockIdx.x, tslot, wv);
    if (tslot >= (uint32_t)vt.tile_off[vt.n_views]) return;
    const TilePos tp = tile_pos<TILE>(vt, order, tslot);
    const uint2 rg = ranges[tp.gt];
    const L lay(wv);
    const int lane = lane_id();
    const float px = (float)lay.lx, py = (float)lay.ly, amax = rs.alpha_max, own_min = own_alpha_min(rs, hdr);
    const int i = tp.tx * TILE + lay.lx, j = tp.ty * TILE + lay.ly;
    // The pixel's upstream gradient and, to start the walk's remainder Rem, the total
    // G = sum_k w_k (g . e_k) + T_final (g_C . bg) that the forward's outputs give.
    uint32_t my_last = 0u;
    float gC0 = 0.f, gC1 = 0.f, gC2 = 0.f, gD = 0.f, gA = 0.f, gX0 = 0.f, gX1 = 0.f, gX2 = 0.f, Rem = 0.f, T = 1.0f;
    if (i < tp.W && j < tp.H) {
        const int64_t e = (int64_t)j * tp.W + i;
        const int64_t pix = tp.pix_off + e, o3 = 3 * tp.pix_off + e, plane = tp.plane;
        my_last = last[pix];
        gC0 = load_or0(up.rgb, o3);
        gC1 = load_or0(up.rgb, o3 + plane);
        gC2 = load_or0(up.rgb, o3 + 2 * plane);
        gD = load_or0(up.depth, pix);
        gA = load_or0(up.alpha, pix);
        gX0 = load_or0(up.pointmap, o3);
        gX1 = load_or0(up.pointmap, o3 + plane);
        gX2 = load_or0(up.pointmap, o3 + 2 * plane);
        const float Tf = t_final[pix];
        const bool none = gC0 == 0.f && gC1 == 0.f && gC2 == 0.f && gD == 0.f && gA == 0.f && gX0 == 0.f &&
                          gX1 == 0.f && gX2 == 0.f;
        // The rgb output holds sum_k w_k c_k + T_final bg, which is exactly what G needs.
        Rem = gC0 * fwd.rgb[o3] + gC1 * fwd.rgb[o3 + plane] + gC2 * fwd.rgb[o3 + 2 * plane] + gD * fwd.depth[pix] +
              gA * (1.0f - Tf);
        if (FRAME == 2) {
            // Eq. 5: the pointmap is D K^-1 [i, j, 1]^T, a function of the depth only.
            const float rx = ((float)i - vt.cx[tp.v]) / vt.fx[tp.v];
            const float ry = ((float)j - vt.cy[tp.v]) / vt.fy[tp.v];
            const float gXD = gX0 * rx + gX1 * ry + gX2;
            Rem += gXD * fwd.depth[pix];
            gD += gXD;
            gX0 = gX1 = gX2 = 0.f;
        } else {
            Rem += gX0 * fwd.pointmap[o3] + gX1 * fwd.pointmap[o3 + plane] + gX2 * fwd.pointmap[o3 + 2 * plane];
        }
        if (FRAME == 1) {
            // The depth is the point's z: one gradient for both.
            gX2 += gD;
            gD = 0.f;
        }
        if (none) my_last = 0u;  // nothing flows back from this pixel
    }
    uint32_t wave_last = my_last;
    for (int off = 32; off > 0; off >>= 1) wave_last = max(wave_last, (uint32_t)__shfl_xor((int)wave_last, off, 64));
    wave_last = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_last);  // uniform: keep it scalar
    if (wave_last == 0u) return;

    float *gwf = reinterpret_cast<float *>(gw);
    // The products' left operand, rows f: 0 .. 5 the moments, 8 + m the m-th weighted sum.  Lane
    // 16 t + 4 b + i holds row 4 t + i of pixel 4 k + b in F[k]; instruction 4 k + b takes it
    // from the lanes of b for the four blocks of t.
    const int row = 4 * (lane >> 4) + (lane & 3);
    float F[16];
    {
        float wg[7];
        int m = 0;
        if (V::kColour) { wg[m++] = gC0; wg[m++] = gC1; wg[m++] = gC2; }
        if (V::kDepth) wg[m++] = gD;
        if (V::kPoint) { wg[m++] = gX0; wg[m++] = gX1; wg[m++] = gX2; }
#pragma unroll
        for (int t = 0; t < V::NW; ++t) gwf[64 * t + lane] = wg[t];
        wave_sync();
        const int b = (lane >> 2) & 3;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const float x = (float)(4 * (k & 1) + b) - 3.5f, y = (float)(k >> 1) - 3.5f;
            float f = row == 0 ? 1.0f : row == 1 ? x : row == 2 ? y : row == 3 ? x * x : row == 4 ? x * y : row == 5 ? y * y : 0.0f;
            if (row >= 8 && row < 8 + V::NW) f = gwf[64 * (row - 8) + 4 * k + b];
            F[k] = f;
        }
        wave_sync();  // read before the walk overwrites the buffer
    }
    // What each lane adds after that: column col of entry lane / 16 (+ 4 h), from the product's row
    // out_row, and the constants of its recentring.
    const int col = lane & 15;
    int out_row = col <= 5 && (col > 0 || V::kOpacity) ? col : -1;
#pragma unroll
    for (int m = 0; m < V::NW; ++m) out_row = (int)((V::kWColumns >> (4 * m)) & 15u) == col ? 8 + m : out_row;
    const bool has = out_row >= 0;
    const int out_at = has ? out_row : 0;
    const float kx = col == 1 || col == 3 || col == 4 ? 1.0f : 0.0f, ky = col == 2 || col == 5 ? 1.0f : 0.0f;
    const float lx = col == 3 ? 1.0f : 0.0f, ly = col == 4 || col == 5 ? 1.0f : 0.0f;
    const float l1 = col == 1 || col == 2 ? -1.0f : 0.0f;
    const float bx = col == 3 ? -2.0f : 0.0f, by = col == 4 ? -1.0f : 0.0f;
    const float gx = col == 4 ? -1.0f : 0.0f, gy = col == 5 ? -2.0f : 0.0f;
    const float cxw = lay.rx0 + 3.5f, cyw = lay.ry0 + 3.5f;
    // Adds the sums of those of the batch's n entries that adds marks.
    auto flush = [&](uint32_t n, uint32_t adds) {
        wave_sync();
        // Lane 16 t + e supplies entry e (g for the moments' rows, w for the others) and
        // receives rows 4 t .. 4 t + 3 of it.
        const float4 *src = gw + kSumPitch * (lane & 15) + (lane >= 32 ? 16 : 0);
        v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const float4 h = src[k];
            acc = __builtin_amdgcn_mfma_f32_4x4x1f32(F[k], h.x, acc, 2, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_4x4x1f32(F[k], h.y, acc, 2, 1, 0);
            acc = __builtin_amdgcn_mfma_f32_4x4x1f32(F[k], h.z, acc, 2, 2, 0);
            acc = __builtin_amdgcn_mfma_f32_4x4x1f32(F[k], h.w, acc, 2, 3, 0);
        }
        wave_sync();  // g and w have been read
        *reinterpret_cast<v4f *>(gwf + kOutPitch * (lane & 15) + 4 * (lane >> 4)) = acc;
        wave_sync();
        for (uint32_t e0 = 0u; e0 < n; e0 += 4u) {
            const uint32_t e = e0 + ((uint32_t)lane >> 4);  // entry of this lane: 16 adjacent lanes hold one row
            const float4 sm = *reinterpret_cast<const float4 *>(gwf + kOutPitch * e);  // S0, Sx, Sy
            const float val = gwf[kOutPitch * e + out_at];
            const float2 mean = *reinterpret_cast<const float2 *>(&st[e]);
            const uint32_t rid = __float_as_uint(st[3 * kBatchPlane + e].w);
            asm volatile("" ::"v"(rid), "v"(sm.w));  // read before the branch
            // Moments about the wave centre -> about the record's mean (dx = x - ux):
            // R_x = S_x - ux S0, R_xx = S_xx - 2 ux S_x + ux^2 S0, R_xy = S_xy - uy S_x -
            // ux S_y + ux uy S0, and likewise in y, with each column's coefficients picked by
            // products with lane constants (exact: 0, +-1, -2).
            const float ux = mean.x - cxw, uy = mean.y - cyw;
            const float al = fmaf(kx, ux, ky * uy) * fmaf(lx, ux, fmaf(ly, uy, l1));
            const float be = fmaf(bx, ux, by * uy), ga = fmaf(gx, ux, gy * uy);
            const float out = fmaf(ga, sm.z, fmaf(be, sm.y, fmaf(al, sm.x, val)));
            if (((adds >> e) & 1u) != 0u && has && out != 0.f) unsafeAtomicAdd(grad2d + (int64_t)rid * kG2 + col, out);
        }
        wave_sync();  // read before the next entries overwrite the buffer
    };

    // The entries that one of this wave's live pixels accepted in the forward (its bit plane
    // after the pair list): every entry with a valid pixel here, plus the few that only
    // stopped a pixel, so the walk needs no culling test.
    const int64_t cap = (int64_t)hdr->capacity;
    const uint64_t *plane = wmask_at(vals, cap) + (int64_t)wv * wmask_stride(cap);
    // A forward with another number of pixels per lane had other waves: every entry is tested.
    const bool use_bits = hdr->ppt == 1u;
    auto wave_bits = [&](uint32_t pos) {  // the 64 bits of list positions pos .. pos + 63
        const uint64_t *wp = plane + (pos >> 6);
        const int sh = (int)(pos & 63u);
        uint64_t m = wp[0] >> sh;
        if (sh != 0) m |= wp[1] << (64 - sh);
        return m;
    };
    // The next 64 positions' bits and record indices are loaded one step ahead.
    const uint32_t wend = rg.x + wave_last;
    uint32_t pos = rg.x, head = 0u, waiting = 0u;  // the ring's first entry (below kQueue) and how many wait
    uint64_t m_next = 0ull;
    uint32_t rec_next = 0u;
    auto load_step = [&]() {
        m_next = use_bits ? wave_bits(pos) : ~0ull;
        if (wend - pos < (uint32_t)kWave) m_next &= (1ull << (wend - pos)) - 1ull;
        rec_next = pos + (uint32_t)lane < wend ? vals[pos + (uint32_t)lane] : 0u;
    };
    load_step();
    // Queues marked entries until a batch is complete or the list ends.
    auto fill = [&]() {
        while (waiting < (uint32_t)kBatch && pos < wend) {
            const uint64_t m = m_next;
            const uint32_t r = rec_next, rel = pos - rg.x + (uint32_t)lane;
            pos += kWave;
            if (pos < wend) load_step();
            if ((m >> lane) & 1ull) {
                const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                const uint32_t q = head + waiting + rank;  // below 2 kQueue
                queue[q < kQueue ? q : q - kQueue] = make_uint2(r, rel);
            }
            waiting += (uint32_t)__popcll(m);
        }
        wave_sync();
    };
    // Lane 4 e + w loads word w of the batch's entry e.
    uint32_t cnt = 0u;
    uint2 mine;
    v4f word;
    auto load_batch = [&]() {
        cnt = min((uint32_t)kBatch, waiting);
        const uint32_t q = head + min((uint32_t)lane >> 2, cnt - 1u);
        mine = queue[q < kQueue ? q : q - kQueue];
        word = reinterpret_cast<const v4f *>(rec)[4 * (int64_t)mine.x + (lane & 3)];
        waiting -= cnt;
        head += cnt;
        head -= head >= kQueue ? kQueue : 0u;
    };
    // Whether some upstream gradient, image, colour or point is not finite: 0 times it is NaN, so an
    // entry without a valid pixel is left out (otherwise it adds 0).
    bool odd = ballot(!(fabsf(Rem) < __builtin_inff())) != 0ull;
    fill();
    if (waiting != 0u) load_batch();
    while (cnt != 0u) {
        // Stage the batch: word 0 takes the conic's (a, b) from its quad neighbour, word 1 the
        // threshold of word 3; slots past the batch's end accept nothing.
        const uint32_t n = cnt;
        bool special;
        {
            const int w = lane & 3;
            const bool dead = (uint32_t)lane >> 2 >= n;
            float4 o = make_float4(word.x, word.y, word.z, word.w);
            const float ca = GSPM_DPP_MOV(o.x, 0x55), cb = GSPM_DPP_MOV(o.y, 0x55);  // lane 1 of the quad
            float thr = GSPM_DPP_MOV(o.w, 0xff);                                     // lane 3
            if (own_min > 0.0f) thr = accept_threshold(own_min, word.w);             // used by lane 1
            if (w == 0) o = make_float4((word.x - tp.x0) + word.z, (word.y - tp.y0) + word.w, ca, cb);
            if (w == 1) o = make_float4(word.z, dead ? -__builtin_inff() : thr, word.w, __uint_as_float(mine.y));
            if (w == 3) o.w = __uint_as_float(mine.x);
            odd = odd || ballot(w == 1 && word.z < 0.0f) != 0ull;
            special = odd || ballot(w == 1 && word.w >= amax) != 0ull;
            wave_sync();  // the previous batch has been read
            st[w * kBatchPlane + (lane >> 2)] = o;
        }
        fill();
        cnt = 0u;
        if (waiting != 0u) load_batch();
        auto walk = [&](auto special) {
            constexpr bool kClamp = decltype(special)::value, kSkip = kClamp;
            uint32_t adds = kSkip ? 0u : (1u << n) - 1u;  // the batch's entries that add anything
            for (uint32_t g = 0u; g < n; g += 4u) {
                float al[4], sv[4], inv[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float4 a = st[g + t], b = st[kBatchPlane + g + t], c = st[2 * kBatchPlane + g + t];
                    // Whole 16-byte reads where three words are used (a 12-byte read keeps the
                    // LDS busy twice as long, an 8-byte one half as long).  In the camera
                    // frame the point's z is the depth, the colour's fourth word.
                    asm volatile("" ::"v"(c.w));
                    sv[t] = fmaf(gC0, c.x, fmaf(gC1, c.y, fmaf(gC2, c.z, gA)));
                    if (V::kDepth) sv[t] = fmaf(gD, c.w, sv[t]);
                    if (FRAME == 1) {
                        const float2 d = *reinterpret_cast<const float2 *>(&st[3 * kBatchPlane + g + t]);
                        sv[t] = fmaf(gX0, d.x, fmaf(gX1, d.y, fmaf(gX2, c.w, sv[t])));
                    }
                    if (FRAME == 0) {
                        const float4 d = st[3 * kBatchPlane + g + t];
                        asm volatile("" ::"v"(d.w));
                        sv[t] = fmaf(gX0, d.x, fmaf(gX1, d.y, fmaf(gX2, d.z, sv[t])));
                    }
                    const float dx = px - a.x;
                    const float sq = quad_s(a.z * dx, a.w, b.x, py - a.y);
                    const uint64_t valid = ballot(sq <= b.y) & ballot(__float_as_uint(b.w) < my_last);
                    float ao = b.z * __builtin_amdgcn_exp2f(-sq);
                    if (kClamp) ao = clamp_alpha(ao, amax);
                    // An invalid pixel takes alpha = 0: no weight, no gradient, T unchanged.
                    al[t] = in_mask(valid) ? ao : 0.0f;
                    if (kSkip) {
                        sv[t] = valid != 0ull ? sv[t] : 0.0f;
                        adds |= (valid != 0ull ? 1u : 0u) << (g + t);
                    }
                    inv[t] = __builtin_amdgcn_rcpf(__fsub_rn(1.0f, al[t]));
                }
                // Front to back: Rem = G - sum of w s over this and earlier fragments, the later
                // fragments' share plus the background term.
                float *dst = gwf + 4 * kSumPitch * g + lane;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float w = __fmul_rn(al[t], T);
                    Rem = fmaf(-w, sv[t], Rem);
                    const float dLda = fmaf(T, sv[t], -__fmul_rn(Rem, inv[t]));
                    // A clamped alpha passes no gradient.
                    dst[4 * kSumPitch * t] = kClamp && al[t] >= amax ? 0.0f : dLda * al[t];
                    dst[4 * kSumPitch * t + 64] = w;
                    T = fmaf(-al[t], T, T);  // as in the forward
                }
            }
            flush(n, adds);
        };
        if (special) walk(std::true_type{});
        else walk(std::false_type{});
    }
}

}  // namespace

// Launch configurations: (tile, pixels per lane).
#define GSPM_RASTER_CONFIGS(X) X(8, 1) X(16, 1) X(16, 2) X(16, 4) X(32, 1) X(32, 2) X(32, 4)

bool raster_config_supported(int tile, int ppt) {
#define GSPM_CHECK(T_, P_) \
    if (tile == T_ && ppt == P_) return true;
    GSPM_RASTER_CONFIGS(GSPM_CHECK)
#undef GSPM_CHECK
    return false;
}

// Windows of at most this many waves (at one pixel per lane) are composited by independent
// waves, larger ones by workgroups that share their staging.  The chip holds 5120 of these
// waves at once; up to about ten rounds of them the longest waves' latency decides (16 x 16 tiles,
// 960x640 with 500k Gaussians, 9.6k waves: 118 against 194 us; 1216x352 with 300k, 6.7k waves: 63
// against 103 us), at 58k waves (8 keyframes, 1M Gaussians) the two take the same time (645 and
// 655 us: vector issue binds both).  Beyond, the second reading of each record by every wave costs
// more the more waves there are (views of 1920x1080, waves against workgroups): 65k 0.527 and
// 0.523 ms, 98k 0.828 and 0.810, 131k 1.07 and 1.05, 261k 2.16 and 2.12, 522k 4.38 and 4.18.
// (Other tiles cross later: 32 x 32 at 98k 0.87 and 0.97 ms, 196k 1.74 and 1.89; 8 x 8 at 97k
// 0.83 and 0.86.)
constexpr int64_t kIndependentWaves = 65536;

hipError_t launch_raster_forward(const ViewTable &vt, const RasterSettings &rs, const uint2 *ranges,
                                 const uint32_t *pair_vals, const float *records, float *rgb, float *depth,
                                 float *alpha, float *pointmap, float *t_final, uint32_t *last, uint32_t *contrib,
                                 uint8_t *visible, const uint32_t *order, uint32_t *tile_work, uint64_t *wmask,
                                 int64_t wstride, FrameHeader *hdr, hipStream_t s) {
    const int n_tiles = vt.tile_off[vt.n_views];
    const float4 *rec = reinterpret_cast<const float4 *>(records);
    if (rs.frame < 0 || rs.frame > 2) return hipErrorInvalidValue;
    // The work counts come from the workgroup form only.
    const bool waves = vt.ppt == 1 && !rs.count_work &&
                       (int64_t)n_tiles * (vt.tile * vt.tile / kWave) <= kIndependentWaves;
#define GSPM_FWDW(T_, F_, M_)                                                                                  \
    hipLaunchKernelGGL((k_raster_fwd_waves<T_, F_, M_>), dim3(wave_grid<Layout<T_, 1>::NW>(n_tiles)), dim3(kWave), \
                       0, s, vt, rs, ranges, pair_vals, rec, rgb, depth, alpha, pointmap, t_final, last, visible,    \
                       order, tile_work, wmask, wstride)
#define GSPM_FWDW1(T_, F_)                        \
    do {                                          \
        if (visible) GSPM_FWDW(T_, F_, true);     \
        else GSPM_FWDW(T_, F_, false);            \
    } while (0)
#define GSPM_FWD2(T_, P_, F_, C_)                                                                        \
    hipLaunchKernelGGL((k_raster_fwd<T_, P_, F_, C_>), dim3(n_tiles), dim3(T_ * T_ / P_), 0, s, vt, rs, \
                       ranges, pair_vals, rec, rgb, depth, alpha, pointmap, t_final, last, contrib, visible,   \
                       order, tile_work, wmask, wstride, hdr)
#define GSPM_FWD1(T_, P_, F_)                                                                  \
    do {                                                                                       \
        if (P_ == 1 && waves) GSPM_FWDW1(T_, F_);                                              \
        else if (rs.count_work) GSPM_FWD2(T_, P_, F_, true);                                   \
        else GSPM_FWD2(T_, P_, F_, false);                                                     \
    } while (0)
#define GSPM_FWD(T_, P_)                                      \
    if (vt.tile == T_ && vt.ppt == P_) {                      \
        if (rs.frame == 0) GSPM_FWD1(T_, P_, 0);              \
        else if (rs.frame == 1) GSPM_FWD1(T_, P_, 1);         \
        else GSPM_FWD1(T_, P_, 2);                            \
        return hipGetLastError();                             \
    }
    GSPM_RASTER_CONFIGS(GSPM_FWD)
#undef GSPM_FWD
#undef GSPM_FWD2
#undef GSPM_FWD1
#undef GSPM_FWDW1
#undef GSPM_FWDW
    return hipErrorInvalidValue;
}

hipError_t launch_raster_backward(const ViewTable &vt, const RasterSettings &rs, const uint2 *ranges,
                                  const uint32_t *pair_vals, const float *records, const uint32_t *last,
                                  const float *t_final, const gspm_const_images &fwd, const gspm_const_images &up,
                                  float *grad2d, bool pose_only, const uint32_t *order, FrameHeader *hdr,
                                  int64_t n_records, hipStream_t s) {
    const int n_tiles = vt.tile_off[vt.n_views];
    const float4 *rec = reinterpret_cast<const float4 *>(records);
    if (rs.frame < 0 || rs.frame > 2) return hipErrorInvalidValue;
#define GSPM_BWD1(T_, P_, PO_, F_)                                                                          \
    do {                                                                                                    \
        if (P_ == 1 && !rs.bwd_lane_reduce)                                                                 \
            hipLaunchKernelGGL((k_raster_bwd_waves<T_, PO_, F_>), dim3(wave_grid<Layout<T_, 1>::NW>(n_tiles)),  \
                               dim3(kWave), 0, s, vt, rs, ranges, pair_vals, rec, last, t_final, fwd, up,    \
                               grad2d, order, hdr, n_records);                                              \
        else                                                                                                \
            hipLaunchKernelGGL((k_raster_bwd<T_, P_, PO_, F_>), dim3(n_tiles), dim3(T_ * T_ / P_), 0, s, vt, rs, \
                               ranges, pair_vals, rec, last, t_final, fwd, up, grad2d, order, hdr, n_records);  \
    } while (0)
#define GSPM_BWD2(T_, P_, PO_)                        \
    if (rs.frame == 0) GSPM_BWD1(T_, P_, PO_, 0);     \
    else if (rs.frame == 1) GSPM_BWD1(T_, P_, PO_, 1);\
    else GSPM_BWD1(T_, P_, PO_, 2);
#define GSPM_BWD(T_, P_)                                  \
    if (vt.tile == T_ && vt.ppt == P_) {                  \
        if (pose_only) {                                  \
            GSPM_BWD2(T_, P_, true)                       \
        } else {                                          \
            GSPM_BWD2(T_, P_, false)                      \
        }                                                 \
        return hipGetLastError();                         \
    }
    GSPM_RASTER_CONFIGS(GSPM_BWD)
#undef GSPM_BWD
#undef GSPM_BWD2
#undef GSPM_BWD1
    return hipErrorInvalidValue;
}

}  // namespace gspm
