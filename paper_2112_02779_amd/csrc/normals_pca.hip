// Target normals by principal component analysis of a pixel window (the
// eigen-decomposition estimator that Dong et al. name in Sec. 4.1 next to the
// neighbour cross product), for batches of range images on gfx950.
//
// The window's points are unprojected (Eq. (1)) from the FP64 sensor tables
// (once per point and tile, into shared memory) and accumulated relative to
// the centre point in FP64: the covariance of a planar patch has a smallest
// eigenvalue many orders of magnitude below the largest, which FP32 sums could
// not resolve.  The smallest eigenvalue is the smallest root of the
// characteristic cubic: the trigonometric form evaluated from an FP32 angle,
// then two Newton steps in FP64; its vector the largest cross product of two
// rows of A - lambda I.  The kernels are bound by this arithmetic, not by HBM
// (100 scans of 128x2048, 3x3: 446 MB, 86 us at the copy rate), so everything
// that does not have to be FP64 is not: the window's range test (decided in
// FP64 only where FP32 could round the other way), the angle, and the test for
// points on a line unless it is close.  Measured on those scans: 350 -> 237 us,
// 5x5 451 -> 323, 7x7 600 -> 455
// (FP64 library acos and cos, an integer division per tile point, FP64 range
// tests before).
#include "rir_ops.h"

namespace rir {

namespace {

// The unit eigenvector n of the smallest eigenvalue of the symmetric matrix
// [[a00 a01 a02] [a01 a11 a12] [a02 a12 a22]], if its middle eigenvalue exceeds
// 1e-6 times the largest (else the points lie on a line) and it has two
// eigenvalues at all.
//
// With q the mean eigenvalue, 6 p^2 the sum of squares of A - q I and
// r = det(A - q I) / (2 p^3) = cos(3 phi), the eigenvalues are q + p b with b
// the roots of b^3 - 3 b = 2 r; the smallest is 2 cos(phi + 2 pi / 3) = -1 - d
// with d = sqrt(3) sin phi - 2 sin^2(phi / 2) in [0, 1], the root of
// d^2 (3 + d) = 2 (1 - r), and it lies 2 sqrt(3) sin phi > 2 d below the middle
// one.  d comes from an FP32 arctangent and is off by 5e-6 of itself at most;
// each Newton step squares such a relative error, so two leave the rounding
// of r, the condition of the root.
__device__ __forceinline__ bool smallest_eigenvector(double a00, double a01, double a02, double a11, double a12,
                                                     double a22, double n[3])
{
    const double q = (a00 + a11 + a22) * (1.0 / 3.0);
    const double b00 = a00 - q, b11 = a11 - q, b22 = a22 - q;
    const double s01 = a01 * a01, s02 = a02 * a02, s12 = a12 * a12;
    const double p2 = b00 * b00 + b11 * b11 + b22 * b22 + 2.0 * (s01 + s02 + s12);
    if (!(p2 > 0.0))
        return false;
    const double h = p2 * (1.0 / 6.0), ip = d_rsqrt(h), p = h * ip;
    const double det = b00 * (b11 * b22 - s12) - a01 * (a01 * b22 - a12 * a02) + a02 * (a01 * a12 - b11 * a02);
    double r = 0.5 * det * ip * ip * ip;
    r = r < -1.0 ? -1.0 : (r > 1.0 ? 1.0 : r);
    const double w = 2.0 * (1.0 - r);
    const float f = atan2_abs(__builtin_amdgcn_sqrtf((float)(0.5 * w * (1.0 + r))), (float)r) * (1.0f / 3.0f);
    const float sh = __sinf(0.5f * f), ch = __cosf(0.5f * f);
    float df = 2.0f * sh * (1.73205081f * ch - sh);
    df = fmaxf(df, 1e-18f);  // r = 1: the step below stays finite
    double d = (double)df;
#pragma unroll
    for (int k = 0; k < 2; ++k)
        d -= fma(d * d, 3.0 + d, -w) * __builtin_amdgcn_rcp(3.0 * d * (2.0 + d));
    // the line test: the other roots (1 + d) / 2 -+ sqrt(3 (3 + d) (1 - d)) / 2
    {
        const float dd = (float)d, qf = (float)(q * ip) + 0.5f * (1.0f + dd);  // in units of p
        const float e = 0.5f * __builtin_amdgcn_sqrtf(fmaxf(3.0f * (3.0f + dd) * (1.0f - dd), 0.f)), m1 = qf - e, m2 = qf + e;
        if (!(m1 > 1e-4f * m2)) {  // close to the test, or not finite: in FP64
            const double disc = 3.0 * (3.0 + d) * (1.0 - d), ee = 0.5 * sqrt(disc > 0.0 ? disc : 0.0);
            const double l1 = q + p * (0.5 * (1.0 + d) - ee), l2 = q + p * (0.5 * (1.0 + d) + ee);
            if (!(l1 > 1e-6 * l2))
                return false;
        }
    }
    // the adjugate of A - l0 I is a positive multiple of n n^T: its column with
    // the largest diagonal entry
    const double l0 = q - fma(p, d, p);
    const double m00 = a00 - l0, m11 = a11 - l0, m22 = a22 - l0;
    const double d0 = m11 * m22 - s12, d1 = m00 * m22 - s02, d2 = m00 * m11 - s01;
    const double e01 = a02 * a12 - a01 * m22, e02 = a01 * a12 - a02 * m11, e12 = a01 * a02 - a12 * m00;
    const bool first = d1 > d0;
    double v0 = first ? e01 : d0, v1 = first ? d1 : e01, v2 = first ? e12 : e02;
    const bool last = d2 > (first ? d1 : d0);
    v0 = last ? e02 : v0;
    v1 = last ? e12 : v1;
    v2 = last ? d2 : v2;
    const double ss = v0 * v0 + v1 * v1 + v2 * v2;
    if (!(ss > 0.0))
        return false;
    // (tiny sums would leave the estimate's range)
    const double inv = ss > 1e-290 ? d_rsqrt(ss) : 1.0 / sqrt(ss);
    n[0] = v0 * inv;
    n[1] = v1 * inv;
    n[2] = v2 * inv;
    return true;
}

}  // namespace

// The normal from the window sums about the centre point (sx.. = sums of
// q = p - pc, sxx.. of its products, cnt points): covariance about the mean,
// smallest eigenpair, the middle-eigenvalue test (a line has no normal), the
// normal turned to face the sensor.  Returns false (n untouched) if none.
// (px, py, pz): the centre point without the receiver's offset, along its ray.
template <int HALF>
__device__ __forceinline__ bool pca_from_sums(double px, double py, double pz, int cnt, double sx, double sy, double sz,
                                              double sxx, double sxy, double sxz, double syy, double syz, double szz,
                                              double n[3])
{
    constexpr int K = 2 * HALF + 1;
    constexpr int kMinPts = (K * K + 1) / 2;
    if (cnt < kMinPts)
        return false;
    // 1 / cnt: the FP32 estimate and two Newton steps
    const double c = (double)cnt;
    double ic = (double)d_rcp((float)cnt);
    ic = ic * fma(-c, ic, 2.0);
    ic = ic * fma(-c, ic, 2.0);
    const double mx = sx * ic, my = sy * ic, mz = sz * ic;
    double m[3];
    if (!smallest_eigenvector(sxx * ic - mx * mx, sxy * ic - mx * my, sxz * ic - mx * mz, syy * ic - my * my,
                              syz * ic - my * mz, szz * ic - mz * mz, m))
        return false;
    // towards the sensor: against the ray
    const bool away = m[0] * px + m[1] * py + m[2] * pz > 0.0;
    n[0] = away ? -m[0] : m[0];
    n[1] = away ? -m[1] : m[1];
    n[2] = away ? -m[2] : m[2];
    return true;
}

// PCA normals of a tile of 32 columns x 8 rows of one H x W image by a
// workgroup of 256 threads, one pixel each: the covariance of the window
// points (2 HALF + 1 square, u wrapping, rows clipped) that have a return
// within edge_rel of the centre range, about their mean, in FP64; at least
// half the window must take part, the middle eigenvalue must exceed 1e-6 times
// the largest (a line has no normal); the normal faces the sensor.  The tile's
// points and a HALF-pixel halo are unprojected once into shared memory, so
// each point is formed once instead of once per window it falls in; a point
// without a return has range NaN there and so fails every test.  Returns
// whether this thread's pixel has a normal, which is then in n, and the
// pixel's range in rc.
constexpr int kPcaTileW = 32, kPcaTileH = 8;

template <int HALF>
__device__ __forceinline__ bool pca_tile(const SensorTab<double> &S, const float *rg, int H, int W, int u0, int v0,
                                         double edge_rel, double n[3], float &rc)
{
    constexpr int PW = kPcaTileW + 2 * HALF, PH = kPcaTileH + 2 * HALF;
    __shared__ double s_x[PH * PW], s_y[PH * PW], s_z[PH * PW];
    __shared__ float s_r[PH * PW];
    const double r0 = S.r0;
    for (int k = threadIdx.x; k < PH * PW; k += blockDim.x) {
        const int r = k / PW, c = k - r * PW;  // (division by a constant)
        const int vv = v0 - HALF + r;
        int uu = u0 - HALF + c;
        uu += uu < 0 ? W : 0;
        while (uu >= W)  // more than once only where a tile is wider than the image
            uu -= W;
        float rf = quiet_nan<float>();
        double x = 0.0, y = 0.0, z = 0.0;
        if (vv >= 0 && vv < H) {
            const float t = rg[(int64_t)vv * W + uu];
            if (range_ok(t)) {
                const V3<double> p = unproject(S.row, S.col, r0, uu, vv, (double)t);
                rf = t;
                x = p.x;
                y = p.y;
                z = p.z;
            }
        }
        s_r[k] = rf;
        s_x[k] = x;
        s_y[k] = y;
        s_z[k] = z;
    }
    __syncthreads();
    const int tx = (int)threadIdx.x % kPcaTileW, ty = (int)threadIdx.x / kPcaTileW;
    const int u = u0 + tx, v = v0 + ty;
    const int ci = (ty + HALF) * PW + tx + HALF;
    rc = s_r[ci];
    if (u >= W || v >= H || !(rc == rc))
        return false;
    // |r - rc| <= edge_rel rc: the FP32 difference is within 2^-24 of the true
    // one, so it decides outside a band of 4e-7 around the limit; a wavefront
    // with a window point in that band (one in thousands) sums again by the
    // FP64 test.  (Less one subnormal step, which a limit among the subnormal
    // floats could be rounded up by; rounding keeps the order for the upper end)
    const double rcd = (double)rc, lim = edge_rel * rcd;
    const float sure = (float)fma(lim, 1.0 - 4e-7, -0x1p-149), never = (float)(lim * (1.0 + 4e-7));
    const double pcx = s_x[ci], pcy = s_y[ci], pcz = s_z[ci];
    // r d = p - r0 (cos a, sin a, 0)
    double ca = 0.0, sa = 0.0;
    if (r0 > 0.0)
        ld2(S.col + 2 * u, ca, sa);
    double sx = 0, sy = 0, sz = 0, sxx = 0, sxy = 0, sxz = 0, syy = 0, syz = 0, szz = 0;
    int cnt = 1;  // the centre itself
    auto add = [&](int k) {
        const double qx = s_x[k] - pcx, qy = s_y[k] - pcy, qz = s_z[k] - pcz;
        sx += qx;
        sy += qy;
        sz += qz;
        sxx += qx * qx;
        sxy += qx * qy;
        sxz += qx * qz;
        syy += qy * qy;
        syz += qy * qz;
        szz += qz * qz;
        ++cnt;
    };
    uint64_t band = 0;
#pragma unroll
    for (int dv = -HALF; dv <= HALF; ++dv) {
#pragma unroll
        for (int du = -HALF; du <= HALF; ++du) {
            if (du == 0 && dv == 0)
                continue;
            const int k = ci + dv * PW + du;
            const float d = fabsf(s_r[k] - rc);
            const bool in = d <= sure;
            band |= __builtin_amdgcn_ballot_w64(d <= never) & ~__builtin_amdgcn_ballot_w64(in);
            asm volatile("" : "+s"(band));  // or the compiler keeps the masks of all points
            if (in)
                add(k);
        }
    }
    if (band != 0) {
        sx = sy = sz = sxx = sxy = sxz = syy = syz = szz = 0.0;
        cnt = 1;
#pragma unroll 1
        for (int dv = -HALF; dv <= HALF; ++dv)
#pragma unroll 1
            for (int du = -HALF; du <= HALF; ++du) {
                const int k = ci + dv * PW + du;
                if (k != ci && fabs((double)s_r[k] - rcd) <= lim)
                    add(k);
            }
    }
    return pca_from_sums<HALF>(pcx - r0 * ca, pcy - r0 * sa, pcz, cnt, sx, sy, sz, sxx, sxy, sxz, syy, syz, szz, n);
}

template <int HALF>
__global__ __launch_bounds__(256) void k_normals_pca(SensorTab<double> S, const float *range, double edge_rel,
                                                     float *nrm, uint8_t *valid)
{
    const int H = S.H, W = S.W;
    const int64_t img = blockIdx.z;
    const int u0 = blockIdx.x * kPcaTileW, v0 = blockIdx.y * kPcaTileH;
    double n[3] = {0.0, 0.0, 0.0};
    float rc;
    const bool ok = pca_tile<HALF>(S, range + img * H * W, H, W, u0, v0, edge_rel, n, rc);
    const int u = u0 + (int)threadIdx.x % kPcaTileW, v = v0 + (int)threadIdx.x / kPcaTileW;
    if (u >= W || v >= H)
        return;
    const int64_t i = (img * H + v) * W + u;
    nrm[3 * i] = ok ? (float)n[0] : 0.f;
    nrm[3 * i + 1] = ok ? (float)n[1] : 0.f;
    nrm[3 * i + 2] = ok ? (float)n[2] : 0.f;
    valid[i] = ok ? 1 : 0;
}

// Level-0 target records of the registration from PCA normals (the
// alternative estimator of Sec. 4.1): record (n, n . q) with n the FP64 PCA
// normal rounded to T and q the target point from the T tables (as the
// cross-product prepass forms it); (0, 0, 0, NaN) where there is no normal.
// Grid: (tiles of the largest image, pair).
template <typename T, int HALF>
__global__ __launch_bounds__(256) void k_pca_records(PrepArgs a)
{
    const PairDesc<T> *P = reinterpret_cast<const PairDesc<T> *>(a.pairs) + a.pair_base + blockIdx.y;
    const int H = cload(&P->H), W = cload(&P->W);
    const int across = (W + kPcaTileW - 1) / kPcaTileW, v0 = (int)blockIdx.x / across * kPcaTileH;
    const int u0 = ((int)blockIdx.x % across) * kPcaTileW;
    if (v0 >= H)
        return;  // a smaller image than the largest
    const SensorTab<T> *S = cload(&P->tab);
    double n[3] = {0.0, 0.0, 0.0};
    float rng;
    const bool ok = pca_tile<HALF>(*cload(&P->tabd), cload(&P->dstr[0]), H, W, u0, v0, a.edge_rel, n, rng);
    const int u = u0 + (int)threadIdx.x % kPcaTileW, v = v0 + (int)threadIdx.x / kPcaTileW;
    if (u >= W || v >= H)
        return;
    V4<T> rec = {(T)0, (T)0, (T)0, quiet_nan<T>()};
    if (ok) {
        const T r0 = cload(&S->r0);
        const V4<T> rw = ld4(cload(&S->row) + 4 * v);
        T ca, sa;
        ld2(cload(&S->col) + 2 * u, ca, sa);
        const V3<T> d = ray_dir(rw, ca, sa);
        const T rc = (T)rng;
        const T q0 = rc * d.x + r0 * ca, q1 = rc * d.y + r0 * sa, q2 = rc * d.z;
        const T n0 = (T)n[0], n1 = (T)n[1], n2 = (T)n[2];
        rec = V4<T>{n0, n1, n2, n0 * q0 + n1 * q1 + n2 * q2};
    }
    st4(cload(&P->dst4[0]) + 4 * ((size_t)v * W + u), rec);
}

template <typename T>
static hipError_t launch_pca_records_t(const PrepArgs &a, int half, int n_pairs, int max_tiles, hipStream_t stream)
{
    const dim3 grid((unsigned)max_tiles, (unsigned)n_pairs);
    switch (half) {
    case 1:
        hipLaunchKernelGGL((k_pca_records<T, 1>), grid, dim3(256), 0, stream, a);
        break;
    case 2:
        hipLaunchKernelGGL((k_pca_records<T, 2>), grid, dim3(256), 0, stream, a);
        break;
    case 3:
        hipLaunchKernelGGL((k_pca_records<T, 3>), grid, dim3(256), 0, stream, a);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int pca_tiles(int H, int W)
{
    return ((W + kPcaTileW - 1) / kPcaTileW) * ((H + kPcaTileH - 1) / kPcaTileH);
}

hipError_t launch_pca_records(bool fp64, const PrepArgs &a, int half, int n_pairs, int max_tiles, hipStream_t stream)
{
    return fp64 ? launch_pca_records_t<double>(a, half, n_pairs, max_tiles, stream)
                : launch_pca_records_t<float>(a, half, n_pairs, max_tiles, stream);
}

hipError_t launch_normals_pca(const SensorTab<double> &S, const float *range, int n_images, int half, double edge_rel,
                              float *nrm, uint8_t *valid, hipStream_t stream)
{
    if (half < 1 || half > 3)
        return hipErrorInvalidValue;
    const int64_t hw = (int64_t)S.H * S.W;
    const dim3 block(kPcaTileW * kPcaTileH);
    // images in launches of at most 65535 (the grid's third dimension)
    for (int k0 = 0; k0 < n_images; k0 += 65535) {
        const int nb = n_images - k0 < 65535 ? n_images - k0 : 65535;
        const dim3 grid((unsigned)((S.W + kPcaTileW - 1) / kPcaTileW),
                        (unsigned)((S.H + kPcaTileH - 1) / kPcaTileH), (unsigned)nb);
        const float *r = range + hw * k0;
        float *nm = nrm + 3 * hw * k0;
        uint8_t *vd = valid + hw * k0;
        if (half == 1)
            hipLaunchKernelGGL(k_normals_pca<1>, grid, block, 0, stream, S, r, edge_rel, nm, vd);
        else if (half == 2)
            hipLaunchKernelGGL(k_normals_pca<2>, grid, block, 0, stream, S, r, edge_rel, nm, vd);
        else
            hipLaunchKernelGGL(k_normals_pca<3>, grid, block, 0, stream, S, r, edge_rel, nm, vd);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

}  // namespace rir
