// Re-projection of range images under per-column poses on gfx950: the
// non-rigid model of Dong et al.'s outlook (Sec. 6), with consecutive poses
// assigned to each column as in LOAM.  Column u is captured at sweep time
// s_u = (u + 1/2) / W - 1/2; under a constant twist xi per sweep its pose in
// the mid-sweep frame is Exp(s_u xi).  Every return is unprojected (Eq. (1)),
// moved by its column's pose and projected again (Eq. (3)-(4)); the output
// pixel keeps the nearest range (an atomic minimum on the FP32 bit pattern,
// which orders like the value for positive floats).
//
// All in FP64 (the pose, the point and the projection with the FP64 sensor
// tables), so the output differs from an FP64 reference only where a
// projection lies on a rounding boundary.
#include "rir_ops.h"

namespace rir {

namespace {

constexpr uint32_t kInfBits = 0x7f800000u;

// Coefficients of Rodrigues' formula for an angle a, by a^2: A = sin a / a,
// B = (1 - cos a) / a^2, C = (a - sin a) / a^3.  Up to one radian their series
// (ten terms leave 2e-19), a column's rotation in a sweep in all ordinary use;
// the library's functions cost several times that.
__device__ __forceinline__ void rodrigues(double a2, double &A, double &B, double &C)
{
    if (a2 <= 1.0) {
        A = B = C = 0.0;
        // sum over k of (-a2)^k / (2 k + 1)!, / (2 k + 2)!, / (2 k + 3)!
#pragma unroll
        for (int k = 9; k >= 0; --k) {
            double f = 1.0;  // (2 k + 1)!
            for (int m = 2; m <= 2 * k + 1; ++m)
                f *= (double)m;
            A = fma(A, -a2, 1.0 / f);
            B = fma(B, -a2, 1.0 / (f * (double)(2 * k + 2)));
            C = fma(C, -a2, 1.0 / (f * (double)((2 * k + 2) * (2 * k + 3))));
        }
    } else {
        double sn, cs;
        const double a = sqrt(a2);
        sincos(a, &sn, &cs);
        A = sn / a;
        B = (1.0 - cs) / a2;
        C = (a - sn) / (a2 * a);
    }
}

// SE(3) exponential of xi = (omega, tau): R = I + A K + B K^2,
// t = (I + B K + C K^2) tau with K = [omega]x.
__device__ __forceinline__ void exp_twist(const double xi[6], double R[9], double t[3])
{
    const double wx = xi[0], wy = xi[1], wz = xi[2];
    double A, B, C;
    rodrigues(wx * wx + wy * wy + wz * wz, A, B, C);
    const double K[9] = {0.0, -wz, wy, wz, 0.0, -wx, -wy, wx, 0.0};
    double K2[9];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j)
            K2[3 * i + j] = K[3 * i] * K[j] + K[3 * i + 1] * K[3 + j] + K[3 * i + 2] * K[6 + j];
    double V[9];
    for (int i = 0; i < 9; ++i) {
        const double I = (i % 4 == 0) ? 1.0 : 0.0;
        R[i] = I + A * K[i] + B * K2[i];
        V[i] = I + B * K[i] + C * K2[i];
    }
    for (int i = 0; i < 3; ++i)
        t[i] = V[3 * i] * xi[3] + V[3 * i + 1] * xi[4] + V[3 * i + 2] * xi[5];
}

// Twists of up to kDeskewBatch scans, passed as kernel arguments (3 KB of 4).
constexpr int kDeskewBatch = 64;
struct Twists {
    double xi[kDeskewBatch][6];
};

}  // namespace

__global__ void k_fill_bits(uint32_t *p, int64_t n, uint32_t bits)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = bits;
}

// Columns of a workgroup of k_deskew, its wavefronts, the rows that a wavefront
// takes at a time, and the most rows of a workgroup.
constexpr int kDeskewCols = 64, kDeskewWaves = 4, kDeskewChunk = 2, kDeskewRows = 32;

// A workgroup re-projects `rows` rows of 64 columns of one scan (grid: column
// blocks x row blocks x scans).  Its first wavefront forms the columns' poses
// Exp(s_u xi) into shared memory, turned by the column's azimuth: a row's ray
// d = (A, B, s) with A = cos phi cos theta, B = cos phi sin theta, s = sin phi
// then moves to A g1 + B g2 + s g3; then each lane has one column, and each
// wavefront takes kDeskewChunk rows at a time, whose loads, FP64 chains and
// atomics are in flight together: the chain of one return is thousands of
// cycles long, and with one row at a time the kernel waited for it (VALU 37%
// busy).  The output starts as zeros (no return): a pixel's first return goes
// in by compare-and-swap, any other by an atomic minimum; the swap's answer
// is looked at one chunk later.  100 scans of 128 x 2048: 258 -> 138 us with
// the fill, 4 rows at a time 150 (fewer wavefronts); the floor of reading and
// writing once is 40 us, the FP64 instructions (VALU 66% busy) take 79.
template <bool R0, bool POW2>
__global__ __launch_bounds__(256, R0 ? 4 : 5) void k_deskew(const SensorTab<double> *tab, const float *in,
                                                            uint32_t *out, int rows, Twists tw)
{
    constexpr int N = kDeskewChunk;
    __shared__ double s_pose[12][kDeskewCols];
    const LevelView<double> V = level_view(tab, 0);
    const int H = V.Hl, W = V.Wl;
    const double r0 = R0 ? V.r0 : 0.0;
    const int img = blockIdx.z, c = (int)threadIdx.x % kDeskewCols;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kDeskewCols);
    const int u = blockIdx.x * kDeskewCols + c;
    const bool live = u < W;
    if (wave == 0) {
        const double su = ((double)u + 0.5) / (double)W - 0.5;
        double xs[6], R[9], t[3];
        for (int k = 0; k < 6; ++k)
            xs[k] = su * tw.xi[img][k];
        exp_twist(xs, R, t);
        double ca = 0.0, sa = 0.0;
        if (live)
            ld2(cload(&tab->col) + 2 * u, ca, sa);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double g = R[3 * k] * ca + R[3 * k + 1] * sa;
            s_pose[k][c] = g;
            s_pose[3 + k][c] = R[3 * k + 1] * ca - R[3 * k] * sa;
            s_pose[6 + k][c] = R[3 * k + 2];
            s_pose[9 + k][c] = r0 * g + t[k];
        }
    }
    const int64_t hw = (int64_t)H * W;
    const float *src = in + (size_t)img * hw;
    uint32_t *dst = out + (size_t)img * hw;
    const int vb = (int)blockIdx.y * rows, ve = min(H, vb + rows);
    __syncthreads();
    double G[9], t[3];
#pragma unroll
    for (int k = 0; k < 9; ++k)
        G[k] = s_pose[k][c];
#pragma unroll
    for (int k = 0; k < 3; ++k)
        t[k] = s_pose[9 + k][c];
    uint32_t old[N], bits[N];  // of the previous chunk's swaps
    uint32_t *at[N];
#pragma unroll
    for (int j = 0; j < N; ++j)
        old[j] = bits[j] = 0u, at[j] = dst;
    auto settle = [&]() {
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (old[j] > bits[j])  // taken (not 0) by a farther return
                atomicMin(at[j], bits[j]);
    };
    for (int v0 = vb + wave * N; v0 < ve; v0 += kDeskewWaves * N) {
        float rf[N];
#pragma unroll
        for (int j = 0; j < N; ++j)
            rf[j] = live && v0 + j < ve ? src[(size_t)(v0 + j) * W + u] : 0.f;
        double x[N], y[N], z[N], r2[N];
        int u2[N], v2[N];
        bool ok[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const V4<double> rw = sld4(V.rowp, min(v0 + j, H - 1));
            const double fa = rw.x * rw.z, fb = rw.x * rw.w, fs = rw.y;
            const bool has = range_ok(rf[j]);
            const double r = has ? (double)rf[j] : 1.0;
            x[j] = fma(r, fma(fa, G[0], fma(fb, G[3], fs * G[6])), t[0]);
            y[j] = fma(r, fma(fa, G[1], fma(fb, G[4], fs * G[7])), t[1]);
            z[j] = fma(r, fma(fa, G[2], fma(fb, G[5], fs * G[8])), t[2]);
            ok[j] = has;
        }
        project_n<double, R0, POW2, N>(V, x, y, z, u2, v2, r2, ok);
        settle();
#pragma unroll
        for (int j = 0; j < N; ++j) {
            bits[j] = __float_as_uint((float)r2[j]);
            at[j] = dst + ((size_t)v2[j] * W + u2[j]);
            old[j] = 0u;
            if (ok[j] && bits[j] < kInfBits)
                old[j] = atomicCAS(at[j], 0u, bits[j]);
        }
    }
    settle();
}

hipError_t launch_deskew(const SensorTab<double> *tab, int H, int W, bool r0, int n_images, const float *in,
                         const double *twists, float *out, hipStream_t stream)
{
    const int64_t hw = (int64_t)H * W, n = hw * n_images;
    uint32_t *ob = reinterpret_cast<uint32_t *>(out);
    const int gfill = (int)std::min<int64_t>((n + 255) / 256, 65536);
    hipLaunchKernelGGL(k_fill_bits, dim3(gfill), dim3(256), 0, stream, ob, n, 0u);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    const bool pow2 = (W & (W - 1)) == 0;
    const int per = n_images / ((n_images + kDeskewBatch - 1) / kDeskewBatch) + 1;  // launches of about one size
    for (int k0 = 0; k0 < n_images; k0 += std::min(per, kDeskewBatch)) {
        const int nb = std::min(std::min(per, kDeskewBatch), n_images - k0);
        Twists tw;
        for (int k = 0; k < nb; ++k)
            for (int j = 0; j < 6; ++j)
                tw.xi[k][j] = twists[6 * (k0 + k) + j];
        const float *src = in + hw * k0;
        uint32_t *dst = ob + hw * k0;
        // fewer rows a workgroup where the launch would not give each of the
        // 256 CUs four: one chunk of every wavefront at least
        const int nc = (W + kDeskewCols - 1) / kDeskewCols;
        int rows = kDeskewRows;
        while (rows > kDeskewWaves * kDeskewChunk && (int64_t)nc * nb * ((H + rows - 1) / rows) < 1024)
            rows /= 2;
        const dim3 g((unsigned)nc, (unsigned)((H + rows - 1) / rows), (unsigned)nb);
        const dim3 b(kDeskewCols * kDeskewWaves);
        if (r0)
            hipLaunchKernelGGL((k_deskew<true, false>), g, b, 0, stream, tab, src, dst, rows, tw);
        else if (pow2)
            hipLaunchKernelGGL((k_deskew<false, true>), g, b, 0, stream, tab, src, dst, rows, tw);
        else
            hipLaunchKernelGGL((k_deskew<false, false>), g, b, 0, stream, tab, src, dst, rows, tw);
        e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

}  // namespace rir
