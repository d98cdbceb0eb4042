// Projective SDF fusion (Dong et al., Sec. 4.2, Eq. (8)-(10)) into a dense
// grid of 16^3-voxel blocks on gfx950.
//
// One workgroup of 256 threads owns one block; thread (x, y) takes the 16
// voxels (x, y, 0..15) of its column layer by layer (four at a time in small
// launches, see kFewFrames), reading each voxel's state once and writing it
// once per launch whatever the number of scans fused into it (up to
// kSdfFrames).  Per scan and voxel: the sensor-frame
// position R x + t (three FMAs from per-block constants built in FP64), the
// projection of Eq. (3)-(4) at the finest level, one gather of the scan's
// range, the signed distance of Eq. (9) and the running mean of Eq. (10).  A
// block whose every voxel lies beyond the range clip plus the truncation band
// of a scan (plus the receiver radius) is not visited for that scan, and
// neither is a z-layer that no pixel of the scan can update (below); a layer
// no scan of the launch can update is neither read nor written.
//
// Which layers a scan can update.  Evaluating every voxel for every scan within
// reach the kernel was bound by VALU issue (97% busy), and of those evaluations
// only about 5% change a voxel: most voxels lie behind the surface their pixel sees, project to a pixel without
// a return or fall outside the field of view.  So before any evaluation each
// lane bounds, for one layer of the block and one scan, the pixel rectangle
// the layer projects to and the smallest range of its voxels, looks up the
// largest usable return (<= clip) of the rectangle in a table of tile maxima
// (k_range_tiles, made once per launch), and drops the layer if that is below
// the smallest range minus the truncation band: the test an evaluation would
// fail for every voxel, with margins far above the FP32 rounding of the
// projection, so the result does not change by a bit.  Why layers: of the
// 100-scan outdoor sequence's evaluations (128x2048, 0.1 m, 57x71x6 blocks)
// 5.6% change a voxel, and 32% lie in a block, 13% in a quarter of a block's
// height and about 8% in a layer that holds one that does.  Measured on that
// sequence: 4.85 ms without, 2.0 ms with rectangles read pixel by pixel for
// four slabs a block, 1.53 ms with an early exit and 32 scans a launch
// instead of 16, 1.07 ms with tile maxima for 16 layers (399 million vector
// instructions a launch of 16 scans before, 104 million a launch of 32 now).
// Now the vector units are 58% busy over a launch; the rest waits for the
// layer tests' look-ups, a chain each, and for the gathers.
#include <type_traits>

#include "rir_ops.h"

namespace rir {

namespace {

// Per-scan constants of one block in LDS: columns c0, c1, c2 of voxel * R and
// the sensor-frame position tb of the block's voxel (0, 0, 0), as 12 floats
// c0x c0y c0z c1x | c1y c1z c2x c2y | c2z tbx tby tbz (three 16-byte reads).
constexpr int kFrameWords = 16;
// Consecutive blocks one XCD takes at a time.
constexpr int kSdfXcdRun = 8;
// A layer's rectangle is looked up in at most this many tiles, fine ones or
// else coarse ones; one that spans more (a layer next to the sensor) is
// evaluated unseen.
constexpr int kMaxTiles = 64;
// Without tile maxima (few block-scans, a stream under capture, no free slot)
// launches of up to kFewFrames scans, or into up to kFewBlocks blocks, or of a
// sensor with a receiver offset take a column's voxels four at a time for each
// scan instead of a layer's scans four at a time: a layer after the other is a
// chain of 16 projections and gathers, which only many scans and blocks hide.
// 64 x 1024 scans, us a call, layers against columns: 1 scan into 16 x 16 x 4
// blocks 17.8 and 12.2, 12 scans 76.9 and 73.8; into 40 x 40 x 6 blocks 3 scans
// 139 and 118, 4 scans 150 and 150, 12 scans 393 and 410; 64 x 1000 with an
// offset, 12 scans into 40 x 40 x 6 blocks 1397 and 1359.
constexpr int kFewFrames = 3, kFewBlocks = 2048;

// Bounds of layer z (voxels (0..15, 0..15, z)) of a block in one scan, from
// the block's constants fr (s_fr).  The layer's four corners go through the
// affine map; with n the horizontal unit vector towards its centre and m the
// unit vector towards the centre, every point p of the layer has |p| >= p . m,
// horizontal distance h >= p . n, and azimuth (relative to n) and z / (p . n)
// between those of the corners (ratios of linear functions, p . n > 0).  The
// elevation follows from z / h = z / (p . n) cos(relative azimuth).  A
// receiver radius r0 moves a point's horizontal distance and its azimuth by
// at most r0 and about r0 / h.  Out: the smallest range, the tangents of the
// elevations, the azimuths.  Reciprocals and roots are the approximate ones
// (1 ulp): the margins are far larger.  false: no bound (the layer reaches
// the sensor's axis, or comes so near that rounding would matter).  A layer
// whose centre lies on the axis is sent back before n is formed: n would not
// be a number, and minima and maxima of floats skip those.
__device__ __forceinline__ bool layer_bound(const float *fr, float z, float r0, float &rmin, float &tlo, float &thi,
                                            float &alo, float &ahi)
{
    const float e = (float)(kSdfEdge - 1), mid = 0.5f * e;
    auto at = [&](float x, float y) -> V3<float> {
        return {fr[9] + x * fr[0] + y * fr[3] + z * fr[6], fr[10] + x * fr[1] + y * fr[4] + z * fr[7],
                fr[11] + x * fr[2] + y * fr[5] + z * fr[8]};
    };
    const V3<float> c = at(mid, mid);
    const float h2 = c.x * c.x + c.y * c.y, r2 = h2 + c.z * c.z;
    if (!(h2 > 1e-30f))
        return false;
    const float ih = d_rsqrt(h2), ir = d_rsqrt(r2);
    const float nx = c.x * ih, ny = c.y * ih, mx = c.x * ir, my = c.y * ir, mz = c.z * ir;
    float along = INFINITY, qlo = INFINITY, qhi = -INFINITY, slo = INFINITY, shi = -INFINITY;
    rmin = INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const V3<float> p = at(i & 1 ? e : 0.f, i & 2 ? e : 0.f);
        const float a = p.x * nx + p.y * ny, ia = d_rcp(a);
        const float q = p.z * ia, s = (p.y * nx - p.x * ny) * ia;
        along = fminf(along, a);
        rmin = fminf(rmin, p.x * mx + p.y * my + p.z * mz);
        qlo = fminf(qlo, q);
        qhi = fmaxf(qhi, q);
        slo = fminf(slo, s);
        shi = fmaxf(shi, s);
    }
    rmin -= r0;
    const float ext = e * (fabsf(fr[0]) + fabsf(fr[1]) + fabsf(fr[2]) + fabsf(fr[3]) + fabsf(fr[4]) + fabsf(fr[5]));
    // (an overflow leaves an infinite or NaN bound: also false)
    if (!(along > 8.0f * r0 + 0.02f * (r2 * ir + ext)))
        return false;
    const float smax = fmaxf(fabsf(slo), fabsf(shi)), cmin = d_rsqrt(1.0f + smax * smax);
    const float up = along * d_rcp(along - r0), dn = cmin * along * d_rcp(along + r0);
    thi = qhi > 0.0f ? qhi * up : qhi * dn;
    tlo = qlo < 0.0f ? qlo * up : qlo * dn;
    const float base = azimuth_mod(c.y, c.x), wid = 2.0f * r0 * d_rcp(along) + 5e-5f;
    alo = base + azimuth_mod(slo, 1.0f) - wid;
    ahi = base + azimuth_mod(shi, 1.0f) + wid;
    return true;
}

// Whether some usable return of scan f can update a voxel of layer z of the
// block (s_fr constants fr): its tile maxima reach the layer's smallest range
// minus the truncation band.
template <bool R0>
__device__ __forceinline__ bool layer_seen(const SdfArgs &a, const LevelView<float> &V, const float *fr, int f,
                                           float z)
{
    float rmin, tlo, thi, alo, ahi;
    if (!layer_bound(fr, z, R0 ? V.r0 : 0.f, rmin, tlo, thi, alo, ahi))
        return true;
    const int H = V.Hl, W = V.Wl;
    const float eps = 5e-5f;
    const float slo = tlo * d_rsqrt(1.f + tlo * tlo) - eps, shi = thi * d_rsqrt(1.f + thi * thi) + eps;
    if (slo > V.s_hi || shi < V.s_lo)
        return false;  // outside the field of view
    const float need = rmin - a.trunc - (1e-4f + 1e-4f * fabsf(rmin));
    const uint32_t nb = need > 0.f ? max(1u, __float_as_uint(need)) : 1u;
    // rows go down with sin(phi)
    float uo;
    int lo = elev_row(V.ebin, V.bin_lo, V.bin_scale, V.bin_max, shi, uo);
    int hi = elev_row(V.ebin, V.bin_lo, V.bin_scale, V.bin_max, slo, uo);
    // columns: azimuth in pixels minus the rows' offsets, which in the general
    // model may be those of a neighbouring row (twice the span)
    const float uo_lo = cload(&a.tab->uo_lo), uo_hi = cload(&a.tab->uo_hi), span = uo_hi - uo_lo;
    const float c0 = alo * V.kW - uo_hi - span - 1.5f, c1 = ahi * V.kW - uo_lo + span + 1.5f;
    int u0 = 0, u1 = W - 1;  // first and last column, u1 < u0: through column W - 1 and 0
    if (c1 - c0 < (float)(W - 3)) {
        // span < W / 2 here, so both lie in (-2 W, 3 W)
        u0 = (int)floorf(c0);
        u1 = (int)floorf(c1) + 1;
        auto wrap = [&](int u) {
            u += u < 0 ? W : 0;
            u += u < 0 ? W : 0;
            u -= u >= W ? W : 0;
            return u >= W ? u - W : u;
        };
        u0 = wrap(u0);
        u1 = wrap(u1);
    }
    const uint32_t *tile = a.tiles;
    int nt = (W + kTileCols - 1) / kTileCols, t0 = u0 / kTileCols, t1 = u1 / kTileCols;
    int rows = H;
    auto across = [&]() { return u1 >= u0 ? t1 - t0 + 1 : min(nt - t0 + t1 + 1, nt); };
    int n = across();
    if ((hi - lo + 1) * n > kMaxTiles) {
        tile += (size_t)a.n_frames * H * nt;
        nt = (W + kTileCols * kTileMerge - 1) / (kTileCols * kTileMerge);
        rows = (H + kTileMerge - 1) / kTileMerge;
        t0 /= kTileMerge;
        t1 /= kTileMerge;
        lo /= kTileMerge;
        hi /= kTileMerge;
        n = across();
        if ((hi - lo + 1) * n > kMaxTiles)
            return true;
    }
    uint32_t top = 0;
    for (int v = lo; v <= hi; ++v) {
        const uint32_t *r = tile + ((size_t)f * rows + v) * nt;
        for (int k = 0, t = t0; k < n; ++k) {
            top = max(top, r[t]);
            t = t + 1 == nt ? 0 : t + 1;
        }
    }
    return top >= nb;
}

// Voxel (x, y, z) of the block in scan f (s_fr constants s_f): its range r there
// and the return om of the pixel it projects to; false: it does not project.
template <bool R0, bool POW2>
__device__ __forceinline__ bool sample(const SdfArgs &a, const LevelView<float> &V, rsrc_t img, const float *s_f,
                                       int f, float x, float y, float z, float &om, float &r)
{
    const float4 *fr = reinterpret_cast<const float4 *>(s_f);
    const float4 q0 = fr[0], q1 = fr[1], q2 = fr[2];
    // tb + x c0 + y c1, then + z c2
    const float px = fmaf(y, q0.w, fmaf(x, q0.x, q2.y));
    const float py = fmaf(y, q1.x, fmaf(x, q0.y, q2.z));
    const float pz = fmaf(y, q1.y, fmaf(x, q0.z, q2.w));
    const float xs = fmaf(z, q1.z, px), ys = fmaf(z, q1.w, py), zs = fmaf(z, q2.x, pz);
    const uint32_t H = (uint32_t)V.Hl, W = (uint32_t)V.Wl;
    int u, v;
    const bool ok = project<float, R0, POW2>(V, xs, ys, zs, u, v, r);
    // u, v are in range even when ok is false: the gather is unconditional
    om = __uint_as_float(bld_u32s(img, ((uint32_t)v * W + (uint32_t)u) * 4u, (uint32_t)f * H * W * 4u));
    return ok;
}

// Eq. (9)-(10) for one voxel and one scan.
__device__ __forceinline__ void update(const SdfArgs &a, bool ok, float om, float r, float &sd, float &wt, bool &chg)
{
    float d = om - r;
    const bool use = ok && range_ok(om) && om <= a.clip && d >= -a.trunc;
    d = fminf(d, a.trunc);
    const float wn = wt + 1.0f;
    const float sn = fmaf(d - sd, d_rcp(wn), sd);
    sd = use ? sn : sd;
    wt = use ? wn : wt;
    chg = chg || use;
}

}  // namespace

// Tile maxima of n_frames scans: the bit pattern of the largest return of at
// most `clip` (positive floats order like their bits; 0: none) in every
// 1 x kTileCols tile of pixels, then in every kTileMerge x kTileMerge tiles
// of those.  One wavefront per kTileMerge rows and 64 columns; bound by the
// one read of the images (100 scans of 128 x 2048: 105 MB).
__global__ __launch_bounds__(256) void k_range_tiles(const float *ranges, int n_frames, int H, int W, float clip,
                                                     uint32_t *tiles)
{
    static_assert(kTileCols == 16 && kTileMerge == 4, "a tile is one DPP row, a wavefront's columns one coarse tile");
    const int nt = (W + kTileCols - 1) / kTileCols, ntc = (W + 63) / 64, rc = (H + kTileMerge - 1) / kTileMerge;
    const int lane = threadIdx.x & 63;
    const int item = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (item >= n_frames * rc * ntc)
        return;
    const int c = item % ntc, fr = item / ntc, f = fr / rc, v0 = (fr - f * rc) * kTileMerge;
    const int u = c * 64 + lane;
    const uint32_t cb = __float_as_uint(fminf(clip, 3.402823466e38f));
    uint32_t all = 0, om[kTileMerge];
#pragma unroll
    for (int j = 0; j < kTileMerge; ++j)
        om[j] = u < W && v0 + j < H ? __float_as_uint(ranges[((size_t)f * H + v0 + j) * W + u]) : 0u;
#pragma unroll
    for (int j = 0; j < kTileMerge; ++j) {
        uint32_t m = om[j] <= cb ? om[j] : 0u;
        // maximum over each 16 lanes (rotations within a DPP row)
        m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x128, 0xf, 0xf, false));
        m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x124, 0xf, 0xf, false));
        m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x122, 0xf, 0xf, false));
        m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x121, 0xf, 0xf, false));
        all = max(all, m);
        const int t = u / kTileCols;
        if ((lane & (kTileCols - 1)) == 0 && t < nt && v0 + j < H)
            tiles[((size_t)f * H + v0 + j) * nt + t] = m;
    }
    all = max(all, (uint32_t)__shfl_xor((int)all, 16, 64));
    all = max(all, (uint32_t)__shfl_xor((int)all, 32, 64));
    if (lane == 0)
        tiles[(size_t)n_frames * H * nt + (size_t)fr * ntc + c] = all;
}

// FEW: see kFewFrames.
template <bool R0, bool POW2, bool HASHED, bool FEW>
__global__ __launch_bounds__(256) void k_sdf_fuse(const SdfArgs a)
{
    __shared__ __align__(16) float s_fr[kSdfFrames][kFrameWords];
    __shared__ uint32_t s_reach, s_mask[kSdfEdge];  // scans within reach; per layer, scans that may update it
    __shared__ int s_list[kSdfFrames];              // the scans within reach, in order

    const int nblk = HASHED ? a.n_blocks : a.nbx * a.nby * a.nbz;
    int b = blockIdx.x;
    // XCD-aware order: workgroups go to the 8 XCDs round robin by id; give
    // each XCD runs of kSdfXcdRun consecutive blocks (neighbouring blocks read
    // neighbouring pixels, which then share that XCD's L2), the runs dealt to
    // the XCDs in turn, so that every XCD gets its share of the blocks the
    // scans reach (one contiguous slab per XCD would leave most XCDs idle:
    // the reachable blocks follow the sensor's path).  The grid is a
    // multiple of 8 runs; ids past the last block exit.
    if (a.xcd_remap) {
        const int j = b >> 3;
        b = (j / kSdfXcdRun) * (8 * kSdfXcdRun) + (b & 7) * kSdfXcdRun + j % kSdfXcdRun;
        if (b >= nblk)
            return;
    }
    int bx, by, bz, first = 0;
    if constexpr (HASHED) {
        const int *B = reinterpret_cast<const int *>(a.blocks + b);
        bx = cload(B);
        by = cload(B + 1);
        bz = cload(B + 2);
        first = cload(a.act + cload(B + 3)) - a.frame0;  // the launch's first scan that may update it
    } else {
        bx = b % a.nbx;
        const int byz = b / a.nbx;
        by = byz % a.nby;
        bz = byz / a.nby;
    }
    const int tid = threadIdx.x;

    if (tid < 64) {
        bool act = false;
        if (tid < a.n_frames && (!HASHED || tid >= first)) {
            const SdfFrame &F = a.f[tid];
            const double s = a.voxel;
            const double o[3] = {a.origin[0] + (double)(kSdfEdge * bx) * s, a.origin[1] + (double)(kSdfEdge * by) * s,
                                 a.origin[2] + (double)(kSdfEdge * bz) * s};
            double p[3];
            for (int i = 0; i < 3; ++i)
                p[i] = F.R[3 * i] * o[0] + F.R[3 * i + 1] * o[1] + F.R[3 * i + 2] * o[2] + F.t[i];
            float *dst = s_fr[tid];
            for (int k = 0; k < 3; ++k) {          // column k of s R
                dst[3 * k] = (float)(s * F.R[k]);
                dst[3 * k + 1] = (float)(s * F.R[3 + k]);
                dst[3 * k + 2] = (float)(s * F.R[6 + k]);
            }
            dst[9] = (float)p[0];
            dst[10] = (float)p[1];
            dst[11] = (float)p[2];
            if (a.cull > 0.0) {
                // distance from the sensor to the block centre, minus the
                // block's half diagonal
                const double h = 0.5 * (double)(kSdfEdge - 1) * s;
                double c2 = 0.0;
                for (int i = 0; i < 3; ++i) {
                    const double ci = p[i] + h * (F.R[3 * i] + F.R[3 * i + 1] + F.R[3 * i + 2]);
                    c2 += ci * ci;
                }
                act = sqrt(c2) - h * 1.7320508075688772 <= a.cull;
            } else {
                act = true;
            }
        }
        const uint64_t bal = __ballot(act);
        if (act)
            s_list[__builtin_popcountll(bal & ((1ull << tid) - 1ull))] = tid;
        if (tid == 0)
            s_reach = (uint32_t)bal;
        if (tid < kSdfEdge)
            s_mask[tid] = a.tiles ? 0u : (uint32_t)bal;
    }
    __syncthreads();
    const uint32_t reach = __builtin_amdgcn_readfirstlane(s_reach);
    if (reach == 0)
        return;

    const LevelView<float> V = level_view(a.tab, 0);
    const int H = V.Hl, W = V.Wl;
    const rsrc_t img = make_rsrc(a.ranges, (uint32_t)a.n_frames * (uint32_t)H * (uint32_t)W * 4u);
    const int lane = tid & 63;
    const float x = (float)(tid & (kSdfEdge - 1)), y = (float)(tid >> 4);
    float2 *vb = reinterpret_cast<float2 *>(a.vox) + (size_t)b * (kSdfEdge * kSdfEdge * kSdfEdge) + tid;

    if constexpr (FEW) {
        constexpr int kVox = 4, kStep = kSdfEdge / kVox;
        for (int z0 = 0; z0 < kStep; ++z0) {
            float sd[kVox], wt[kVox];
            bool chg[kVox];
#pragma unroll
            for (int k = 0; k < kVox; ++k) {
                const float2 st = vb[(z0 + k * kStep) * kSdfEdge * kSdfEdge];
                sd[k] = st.x;
                wt[k] = st.y;
                chg[k] = false;
            }
            for (uint32_t m = reach; m != 0; m &= m - 1) {
                const int f = __builtin_ctz(m);
                float om[kVox], r[kVox];
                bool ok[kVox];
#pragma unroll
                for (int k = 0; k < kVox; ++k)
                    ok[k] = sample<R0, POW2>(a, V, img, s_fr[f], f, x, y, (float)(z0 + k * kStep), om[k], r[k]);
#pragma unroll
                for (int k = 0; k < kVox; ++k)
                    update(a, ok[k], om[k], r[k], sd[k], wt[k], chg[k]);
            }
#pragma unroll
            for (int k = 0; k < kVox; ++k)
                if (chg[k])
                    vb[(z0 + k * kStep) * kSdfEdge * kSdfEdge] = make_float2(sd[k], wt[k]);
        }
        return;
    }

    // ---- which layers each scan can update: a wavefront takes four scans at
    // a time, 16 lanes (layers) each
    if (a.tiles) {
        const int n = __builtin_popcount(reach), layer = lane & (kSdfEdge - 1);
        for (int j = tid >> 4; j < n; j += 16) {
            const int f = s_list[j];
            if (layer_seen<R0>(a, V, s_fr[f], f, (float)layer))
                atomicOr(&s_mask[layer], 1u << f);
        }
        __syncthreads();
    }
    uint32_t layers = (uint32_t)__builtin_amdgcn_ballot_w64(lane < kSdfEdge && s_mask[lane & (kSdfEdge - 1)] != 0);
    if (layers == 0)
        return;

    // ---- evaluation, layer by layer; the next layer's state is on its way
    // while this one's scans are fused
    int z = __builtin_ctz(layers);
    float2 next = vb[z * kSdfEdge * kSdfEdge];
    while (layers != 0) {
        const float2 st = next;
        const int zc = z;
        layers &= layers - 1;
        if (layers != 0) {
            z = __builtin_ctz(layers);
            next = vb[z * kSdfEdge * kSdfEdge];
        }
        const float zf = (float)zc;
        float sd = st.x, wt = st.y;
        bool chg = false;
        // N scans at a time: their projections and gathers are independent
        // and overlap, the running mean takes them in order
        auto fuse = [&](auto count, uint32_t &m) {
            constexpr int N = decltype(count)::value;
            float om[N], r[N];
            bool ok[N];
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const int f = __builtin_ctz(m);
                m &= m - 1;
                const float4 *fr = reinterpret_cast<const float4 *>(s_fr[f]);
                const float4 q0 = fr[0], q1 = fr[1], q2 = fr[2];
                // tb + x c0 + y c1, then + z c2
                const float px = fmaf(y, q0.w, fmaf(x, q0.x, q2.y));
                const float py = fmaf(y, q1.x, fmaf(x, q0.y, q2.z));
                const float pz = fmaf(y, q1.y, fmaf(x, q0.z, q2.w));
                const float xs = fmaf(zf, q1.z, px), ys = fmaf(zf, q1.w, py), zs = fmaf(zf, q2.x, pz);
                int u, v;
                ok[k] = project<float, R0, POW2>(V, xs, ys, zs, u, v, r[k]);
                // u, v are in range even when ok is false: the gather is unconditional
                om[k] = __uint_as_float(bld_u32s(img, ((uint32_t)v * (uint32_t)W + (uint32_t)u) * 4u,
                                                 (uint32_t)f * (uint32_t)H * (uint32_t)W * 4u));
            }
#pragma unroll
            for (int k = 0; k < N; ++k) {
                float d = om[k] - r[k];
                const bool use = ok[k] && range_ok(om[k]) && om[k] <= a.clip && d >= -a.trunc;
                d = fminf(d, a.trunc);
                const float wn = wt + 1.0f;
                const float sn = fmaf(d - sd, d_rcp(wn), sd);
                sd = use ? sn : sd;
                wt = use ? wn : wt;
                chg = chg || use;
            }
        };
        uint32_t m = __builtin_amdgcn_readfirstlane(s_mask[zc]);
        for (int c = __builtin_popcount(m); c >= 4; c -= 4)
            fuse(std::integral_constant<int, 4>{}, m);
        if (__builtin_popcount(m) >= 2)
            fuse(std::integral_constant<int, 2>{}, m);
        if (m != 0)
            fuse(std::integral_constant<int, 1>{}, m);
        if (chg)
            vb[zc * kSdfEdge * kSdfEdge] = make_float2(sd, wt);
    }
}

hipError_t launch_range_tiles(const float *ranges, int n_frames, int H, int W, float clip, uint32_t *tiles,
                              hipStream_t stream)
{
    const int64_t items = (int64_t)n_frames * ((H + kTileMerge - 1) / kTileMerge) * ((W + 63) / 64);
    hipLaunchKernelGGL(k_range_tiles, dim3((unsigned)((items + 3) / 4)), dim3(256), 0, stream, ranges, n_frames, H, W,
                       clip, tiles);
    return hipGetLastError();
}

template <bool HASHED, bool FEW>
static void launch_sdf_fuse_h(const SdfArgs &a, bool r0, bool pow2, int nblk, hipStream_t stream)
{
    if (r0)
        hipLaunchKernelGGL((k_sdf_fuse<true, false, HASHED, FEW>), dim3(nblk), dim3(256), 0, stream, a);
    else if (pow2)
        hipLaunchKernelGGL((k_sdf_fuse<false, true, HASHED, FEW>), dim3(nblk), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL((k_sdf_fuse<false, false, HASHED, FEW>), dim3(nblk), dim3(256), 0, stream, a);
}

hipError_t launch_sdf_fuse(const SdfArgs &a, bool r0, bool pow2, bool hashed, hipStream_t stream)
{
    const int n = hashed ? a.n_blocks : a.nbx * a.nby * a.nbz, run = 8 * kSdfXcdRun;
    if (n <= 0)
        return hipSuccess;
    const int nblk = a.xcd_remap ? (n + run - 1) / run * run : n;
    const bool few = !a.tiles && (r0 || a.n_frames <= kFewFrames || n <= kFewBlocks);
    if (hashed) {
        if (few)
            launch_sdf_fuse_h<true, true>(a, r0, pow2, nblk, stream);
        else
            launch_sdf_fuse_h<true, false>(a, r0, pow2, nblk, stream);
    } else {
        if (few)
            launch_sdf_fuse_h<false, true>(a, r0, pow2, nblk, stream);
        else
            launch_sdf_fuse_h<false, false>(a, r0, pow2, nblk, stream);
    }
    return hipGetLastError();
}

}  // namespace rir
