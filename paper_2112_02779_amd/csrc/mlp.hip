// Learned per-pixel robust weight: standalone forward, training gradient and
// Adam update on gfx950.  Every product runs on the matrix cores
// (v_mfma_f32_16x16x16_bf16, FP32 accumulation) with these bfloat16 rounding
// points, shared with the FP64 test oracle:
//   forward  inputs f, hidden activations h1 = relu(a1), h2 = relu(a2);
//   backward dz = (sigmoid(z) - y) / B, g2 = relu'(a2) W3 dz and
//            g1 = relu'(a1) W2^T g2 (relu'(0) = 0); bias gradients are sums
//            of these rounded deltas.
// Gradients are reduced without atomics: every wavefront writes one record,
// and the update kernel sums the records in a fixed order.
#include <mutex>

#include "rir_internal.h"
#include "rir_mlp_device.h"

namespace rir {

constexpr int kMlpGradWaves = 4;  // wavefronts per workgroup of the gradient kernel

__global__ __launch_bounds__(256) void k_mlp_forward(MlpDev m, const float *feats, int64_t B, float *w_out)
{
    __shared__ uint32_t stage[4][64 * 8];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    MlpInfer F;
    mlp_infer_load(m, F);
    const int64_t stride = (int64_t)gridDim.x * 4 * 64;
    for (int64_t base = ((int64_t)blockIdx.x * 4 + wave) * 64; base < B; base += stride) {
        const int64_t i = base + lane;
        float f[14];
#pragma unroll
        for (int k = 0; k < 14; ++k)
            f[k] = i < B ? feats[14 * i + k] : 0.f;
        uint32_t fp[8];
        pack_features(f, fp);
        const float z = mlp_wave(F, fp, stage[wave]);
        if (i < B)
            w_out[i] = 1.f / (1.f + __expf(-z));
    }
}

__device__ __forceinline__ bf16x4_t lds_bf4(const uint16_t *p)
{
    const uint2 v = *reinterpret_cast<const uint2 *>(p);
    return bf4(v.x, v.y);
}

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sum over the 16 lanes of a DPP row (every lane gets it).
__device__ __forceinline__ float row_sum16(float v)
{
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xf, 0xf, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xf, 0xf, false));
    return v;
}

// Gradient of the summed loss over this wavefront's samples: `per` (16, 32 or
// 64) at a time.  Record layout: W1[64][14], b1[64], W2[64][64], b2[64],
// W3[64], b3, loss.
//
// Bound by latency: the matrix products of a training batch of 8192 take well
// under a microsecond of the chip, so the batch is cut into as many
// wavefronts as the record limit allows (mlp_grad_per) and each one's chain
// is kept short: W2 goes through shared memory once per workgroup (its
// transposed fragments are 64 two-byte reads a lane, slow from memory), the
// other fragments are 8- and 16-byte loads, each lane loads its own
// operand's features, and row sums are DPP rotations.  Batch of 8192 on an
// MI355X: 31 -> 14.6 us (64 samples a wavefront, two-byte weight loads before).
__global__ __launch_bounds__(256) void k_mlp_grad(MlpDev m, const float *feats, const float *labels, int64_t B,
                                                  int per, float *gpart)
{
    __shared__ __align__(16) uint16_t s_w2[64 * 64];                    // [h2][h1]
    __shared__ __align__(16) uint16_t s_f[kMlpGradWaves][16 * 16];      // [sample][input]
    __shared__ __align__(16) uint16_t s_g2[kMlpGradWaves][64 * 16];     // [h2][sample]
    __shared__ __align__(16) uint16_t s_h1[kMlpGradWaves][64 * 16];     // [h1][sample]
    __shared__ __align__(16) uint16_t s_g1[kMlpGradWaves][64 * 16];     // [h1][sample]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
    const int64_t stride = (int64_t)gridDim.x * kMlpGradWaves * per;
    const int64_t base0 = ((int64_t)blockIdx.x * kMlpGradWaves + wave) * per;
    // features 4 g .. 4 g + 3 of sample s (two zero inputs make 16) and its label
    auto load_sample = [&](int64_t s, float (&f)[4], float &y) {
        const bool ok = s < B;
        const float *p = feats + 14 * s + 4 * g;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            f[j] = ok && (j < 2 || g < 3) ? p[j] : 0.f;
        y = ok ? labels[s] : 0.f;
    };
    float fx[4], yx;
    load_sample(base0 + r, fx, yx);
    {
        const uint4 *src = reinterpret_cast<const uint4 *>(m.w + kMlpW2);
        uint4 *dst = reinterpret_cast<uint4 *>(s_w2);
        dst[threadIdx.x] = src[threadIdx.x];
        dst[threadIdx.x + 256] = src[threadIdx.x + 256];
    }
    bf16x4_t a1[4], a2[4][4], a2t[4][4];
    f32x4_t b1v[4], b2v[4];
    float w3[4][4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        // W1 rows mt * 16 + r, inputs 4 g ..: 28-byte rows, so 4-byte loads
        const uint32_t *p1 = reinterpret_cast<const uint32_t *>(m.w + kMlpW1 + (mt * 16 + r) * 14 + 4 * g);
        const uint2 p3 = *reinterpret_cast<const uint2 *>(m.w + kMlpW3 + mt * 16 + 4 * g);
        a1[mt] = bf4(p1[0], g < 3 ? p1[1] : 0u);
        b1v[mt] = *reinterpret_cast<const f32x4_t *>(m.b + kMlpB1 + mt * 16 + 4 * g);
        b2v[mt] = *reinterpret_cast<const f32x4_t *>(m.b + kMlpB2 + mt * 16 + 4 * g);
        w3[mt][0] = bf2f(p3.x & 0xffffu);
        w3[mt][1] = bf2f(p3.x >> 16);
        w3[mt][2] = bf2f(p3.y & 0xffffu);
        w3[mt][3] = bf2f(p3.y >> 16);
    }
    const float b3 = m.b[kMlpB3];
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
            a2[mt][kt] = lds_bf4(s_w2 + (mt * 16 + r) * 64 + kt * 16 + 4 * g);
            // W2^T: rows h1 = mt * 16 + r, inputs h2 = kt * 16 + 4 g + j
#pragma unroll
            for (int j = 0; j < 4; ++j)
                a2t[mt][kt][j] = (short)s_w2[(kt * 16 + 4 * g + j) * 64 + mt * 16 + r];
        }
    f32x4_t dW2[4][4], dW1[4];
    float dW3[4][4], db2[4][4], db1[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        dW1[a] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            dW2[a][b] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
            dW3[a][b] = db2[a][b] = db1[a][b] = 0.f;
        }
    }
    float db3 = 0.f, loss = 0.f;
    const float invB = 1.f / (float)B;
    uint16_t *sf = s_f[wave], *sg2 = s_g2[wave], *sh1 = s_h1[wave], *sg1 = s_g1[wave];
    for (int64_t base = base0; base < B; base += stride) {
#pragma unroll 1
        for (int t = 0; t < per; t += 16) {
            const int64_t smp = base + t + r;  // sample of this lane's column
            const bool ok = smp < B;
            const float y = yx;
            const uint32_t f01 = pack_bf2(fx[0], fx[1]), f23 = pack_bf2(fx[2], fx[3]);
            const bf16x4_t Bf = bf4(f01, f23);
            *reinterpret_cast<uint2 *>(sf + r * 16 + 4 * g) = make_uint2(f01, f23);
            // the next tile's sample
            load_sample(t + 16 < per ? smp + 16 : base + stride + r, fx, yx);
            // ---- forward
            bf16x4_t hb[4];
            bool m1[4][4];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const f32x4_t c = mfma16(a1[mt], Bf, b1v[mt]);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    m1[mt][j] = c[j] > 0.f;
                hb[mt] = bf4(pack_bf2(fmaxf(c[0], 0.f), fmaxf(c[1], 0.f)), pack_bf2(fmaxf(c[2], 0.f), fmaxf(c[3], 0.f)));
            }
            float h2[4][4];
            bool m2[4][4];
            float part = 0.f;
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                f32x4_t c = b2v[mt];
#pragma unroll
                for (int kt = 0; kt < 4; ++kt)
                    c = mfma16(a2[mt][kt], hb[kt], c);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    m2[mt][j] = c[j] > 0.f;
                    h2[mt][j] = round_bf(fmaxf(c[j], 0.f));
                    part += w3[mt][j] * h2[mt][j];
                }
            }
            part += __shfl_xor(part, 16, 64);
            part += __shfl_xor(part, 32, 64);
            const float z = part + b3;
            // ---- loss and output delta
            const float sp = z > 0.f ? z + log1pf(__expf(-z)) : log1pf(__expf(z));
            if (ok && g == 0)
                loss += sp - y * z;
            const float dz = ok ? round_bf((1.f / (1.f + __expf(-z)) - y) * invB) : 0.f;
            if (g == 0)
                db3 += dz;
            // ---- layer 3 and hidden-2 deltas (accumulator layout)
            bf16x4_t g2b[4];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    dW3[mt][j] += dz * h2[mt][j];
                    const uint32_t d2 = f2bf(m2[mt][j] ? w3[mt][j] * dz : 0.f);
                    db2[mt][j] += bf2f(d2);
                    g2b[mt][j] = (short)d2;
                    sg2[(mt * 16 + 4 * g + j) * 16 + r] = (uint16_t)d2;
                    sh1[(mt * 16 + 4 * g + j) * 16 + r] = (uint16_t)hb[mt][j];
                }
            // ---- hidden-1 deltas: W2^T g2
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                f32x4_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kt = 0; kt < 4; ++kt)
                    c = mfma16(a2t[mt][kt], g2b[kt], c);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t d1 = f2bf(m1[mt][j] ? c[j] : 0.f);
                    db1[mt][j] += bf2f(d1);
                    sg1[(mt * 16 + 4 * g + j) * 16 + r] = (uint16_t)d1;
                }
            }
            wave_lds_sync();
            // ---- weight gradients, contracting over the 16 samples of the tile
            bf16x4_t Bx, H1[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                Bx[j] = (short)sf[(4 * g + j) * 16 + r];
#pragma unroll
            for (int n = 0; n < 4; ++n)
                H1[n] = lds_bf4(sh1 + (n * 16 + r) * 16 + 4 * g);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const bf16x4_t A2 = lds_bf4(sg2 + (mt * 16 + r) * 16 + 4 * g);
#pragma unroll
                for (int n = 0; n < 4; ++n)
                    dW2[mt][n] = mfma16(A2, H1[n], dW2[mt][n]);
                const bf16x4_t A1 = lds_bf4(sg1 + (mt * 16 + r) * 16 + 4 * g);
                dW1[mt] = mfma16(A1, Bx, dW1[mt]);
            }
            wave_lds_sync();
        }
    }
    // ---- write this wavefront's record
    float *rec = gpart + ((size_t)blockIdx.x * kMlpGradWaves + wave) * kMlpGradRecord;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int h = mt * 16 + 4 * g + j;
#pragma unroll
            for (int n = 0; n < 4; ++n)
                rec[960 + h * 64 + n * 16 + r] = dW2[mt][n][j];
            if (r < 14)
                rec[h * 14 + r] = dW1[mt][j];
            const float a = row_sum16(dW3[mt][j]), b2 = row_sum16(db2[mt][j]), b1 = row_sum16(db1[mt][j]);
            if (r == 0) {
                rec[5120 + h] = a;
                rec[5056 + h] = b2;
                rec[896 + h] = b1;
            }
        }
    // lanes 0..15 hold the sums over samples of b3 and the loss (g = 0)
    db3 = row_sum16(db3);
    loss = row_sum16(loss);
    if (lane == 0) {
        rec[5184] = db3;
        rec[5185] = loss;
    }
}

// Sums the gradient records in a fixed order (FP64) and applies one Adam step
// (beta1 0.9, beta2 0.999, eps 1e-8, bias-corrected) to the FP32 master
// weights and the biases; the bf16 weights are re-rounded from the masters.
// Bound by the one read of the records (a batch of 8192: 512 records, 10.6
// MB): a workgroup takes 64 parameters, its 16 wavefronts every 16th record
// each (all those loads in flight together), and adds their sums in wavefront
// order.  One thread per parameter walking all records one after the other
// took 40 us for 128 records; now 4.8 us for 512.
constexpr int kAdamParams = 64, kAdamGroups = 16;

__global__ __launch_bounds__(kAdamParams *kAdamGroups) void k_mlp_adam(const float *gpart, int nrec, int64_t B,
                                                                       float lr, int step, float *master, float *bias,
                                                                       float *m1, float *m2, uint16_t *wbf,
                                                                       float *loss_out, float *grads_out)
{
    __shared__ double s_sum[kAdamGroups][kAdamParams];
    const int p = threadIdx.x & (kAdamParams - 1), grp = threadIdx.x / kAdamParams;
    const int j = blockIdx.x * kAdamParams + p;
    {
        double s = 0.0;
        if (j < kMlpGradRecord) {
            const float *q = gpart + j;
            int k = grp;
            for (; k + 7 * kAdamGroups < nrec; k += 8 * kAdamGroups) {
                float v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    v[i] = q[(size_t)(k + i * kAdamGroups) * kMlpGradRecord];
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    s += (double)v[i];
            }
            for (; k < nrec; k += kAdamGroups)
                s += (double)q[(size_t)k * kMlpGradRecord];
        }
        s_sum[grp][p] = s;
    }
    __syncthreads();
    if (grp != 0 || j >= kMlpGradRecord)
        return;
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kAdamGroups; ++w)
        s += s_sum[w][p];
    if (j == 5185) {
        if (loss_out)
            loss_out[0] = (float)(s / (double)B);
        return;
    }
    const float gj = (float)s;
    if (grads_out)
        grads_out[j] = gj;
    const float b1 = 0.9f, b2 = 0.999f;
    const float mm = b1 * m1[j] + (1.f - b1) * gj;
    const float vv = b2 * m2[j] + (1.f - b2) * gj * gj;
    m1[j] = mm;
    m2[j] = vv;
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    const float upd = lr * (mm / c1) / (sqrtf(vv / c2) + 1e-8f);
    // parameter j of the record layout -> weight or bias slot
    int wi = -1, bi = -1;
    if (j < 896)
        wi = kMlpW1 + j;
    else if (j < 960)
        bi = kMlpB1 + (j - 896);
    else if (j < 5056)
        wi = kMlpW2 + (j - 960);
    else if (j < 5120)
        bi = kMlpB2 + (j - 5056);
    else if (j < 5184)
        wi = kMlpW3 + (j - 5120);
    else
        bi = kMlpB3;
    if (wi >= 0) {
        const float nw = master[wi] - upd;
        master[wi] = nw;
        wbf[wi] = (uint16_t)f2bf(nw);
    } else {
        bias[bi] -= upd;
    }
}

// Gradient records of the allocation-free training step: a fixed device array
// of kMlpScratchRecords records (10.1 MiB), one copy per GPU for the life of
// the process.  Host code never uses the array's name as an address: the
// device address comes from hipGetSymbolAddress, once per device, with that
// device current.
static __device__ __align__(256) float scratch[(size_t)kMlpScratchRecords * kMlpGradRecord];
static std::mutex g_scratch_mu;
static float *g_scratch_ptr[kMlpMaxDevices] = {};

hipError_t mlp_scratch(int device, float **out)
{
    *out = nullptr;
    if (device < 0 || device >= kMlpMaxDevices)
        return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess)
            return e;
        g_scratch_ptr[device] = static_cast<float *>(p);
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}

// Samples a wavefront of the gradient kernel takes at a time: the fewest that
// keep a batch within 512 records (the allocation-free step's array; a record
// costs 20.7 KB of writes and reads), else 64.
static int mlp_grad_per(int64_t B) { return B <= 512 * 16 ? 16 : (B <= 512 * 32 ? 32 : 64); }

int mlp_grad_blocks(int64_t B)
{
    const int64_t per = (int64_t)mlp_grad_per(B) * kMlpGradWaves, nb = (B + per - 1) / per;
    return (int)(nb < 1 ? 1 : (nb > 512 ? 512 : nb)) * kMlpGradWaves;
}

// Each step of mlp_grad_per halves the records, so the most lie at B or at the
// last batch of a step before it.
int mlp_grad_blocks_upto(int64_t B)
{
    const int64_t a = B < 512 * 16 ? B : 512 * 16, b = B < 512 * 32 ? B : 512 * 32;
    const int na = mlp_grad_blocks(a), nb = mlp_grad_blocks(b), n = mlp_grad_blocks(B);
    return na > nb ? (na > n ? na : n) : (nb > n ? nb : n);
}

hipError_t launch_mlp_forward(const MlpDev &m, const float *feats, int64_t B, float *w_out, hipStream_t stream)
{
    int64_t nb = (B + 255) / 256;
    nb = nb < 1 ? 1 : (nb > 4096 ? 4096 : nb);
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)nb), dim3(256), 0, stream, m, feats, B, w_out);
    return hipGetLastError();
}

hipError_t launch_mlp_grad(const MlpDev &m, const float *feats, const float *labels, int64_t B, float *gpart,
                           int nrec, hipStream_t stream)
{
    hipLaunchKernelGGL(k_mlp_grad, dim3(nrec / kMlpGradWaves), dim3(64 * kMlpGradWaves), 0, stream, m, feats, labels,
                       B, mlp_grad_per(B), gpart);
    return hipGetLastError();
}

hipError_t launch_mlp_adam(const float *gpart, int nrec, int64_t B, float lr, int step, float *master, float *bias,
                           float *m1, float *m2, uint16_t *wbf, float *loss_out, float *grads_out, hipStream_t stream)
{
    hipLaunchKernelGGL(k_mlp_adam, dim3((kMlpGradRecord + kAdamParams - 1) / kAdamParams),
                       dim3(kAdamParams * kAdamGroups), 0, stream, gpart, nrec, B, lr, step, master,
                       bias, m1, m2, wbf, loss_out, grads_out);
    return hipGetLastError();
}

}  // namespace rir
