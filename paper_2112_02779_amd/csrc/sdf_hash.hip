// Sparse voxel-block volume of Sec. 4.2 on gfx950: the 16^3-voxel blocks near
// the returns of each scan are activated in an open-addressing hash table
// keyed by block coordinates, and only activated blocks are fused (the
// fusion and extraction kernels of sdf.hip / sdf_extract.hip, run over the
// table's block list).
//
// Activation: one thread per return.  The return is unprojected in FP64
// (Eq. (1)) and moved to the world frame, x = R^T (x_s - t); every block whose
// cell o + [E b, E (b + 1)) (o: the volume origin) meets the cube
// [x - radius, x + radius] is looked up
// and, if absent, inserted (64-bit compare-and-swap on the key, then a slot of
// the block pool from a counter).  Each table entry keeps the first scan that
// activated it (atomic minimum), so that fusion can apply a scan only to the
// blocks that scan or an earlier one activated, as if every scan were
// activated and then fused in turn.  Neighbouring returns mostly produce the
// same cube: a return whose block range equals that of the lane below it or of
// the row before leaves the inserts to that one.
#include "sdf_extract.h"
#include "sdf_hash.h"

namespace rir {

__device__ __forceinline__ uint64_t bvol_key(int bx, int by, int bz)
{
    return ((uint64_t)(uint32_t)(bx + kBvolBias) << 42) | ((uint64_t)(uint32_t)(by + kBvolBias) << 21) |
           (uint64_t)(uint32_t)(bz + kBvolBias);
}

// SplitMix64 finaliser (Steele, Lea and Flood, 2014): a bijective 64-bit mix.
__device__ __forceinline__ uint32_t bvol_hash(uint64_t k)
{
    k = (k ^ (k >> 30)) * 0xbf58476d1ce4e5b9ull;
    k = (k ^ (k >> 27)) * 0x94d049bb133111ebull;
    return (uint32_t)(k ^ (k >> 31));
}

__device__ __forceinline__ bool bvol_in_range(int b) { return b > -kBvolBias && b < kBvolBias; }

// Finds or inserts block (bx, by, bz) and lowers its entry's first scan to
// `frame`.  Once the pool is full no key is added (the call then fails and
// the volume must be reset), so the table stays below about half full and
// every probe sequence ends at a free entry.
__device__ __forceinline__ void bvol_insert(const BvolDev &t, int bx, int by, int bz, int frame)
{
    const unsigned long long key = bvol_key(bx, by, bz);
    uint32_t h = bvol_hash(key) & t.mask;
    for (uint32_t probe = 0; probe <= t.mask; ++probe) {
        unsigned long long k = __hip_atomic_load(t.keys + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (k == kBvolEmpty) {
            if (__hip_atomic_load(t.count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= t.max_blocks) {
                atomicOr(t.flags, kBvolFull);
                return;
            }
            k = atomicCAS(t.keys + h, kBvolEmpty, key);
            if (k == kBvolEmpty) {
                const int slot = atomicAdd(t.count, 1);
                if (slot < t.max_blocks) {
                    t.blocks[slot] = make_int4(bx, by, bz, (int)h);
                    t.vals[h] = slot;
                } else {
                    atomicOr(t.flags, kBvolFull);
                }
                atomicMin(t.act + h, frame);
                return;
            }
        }
        if (k == key) {
            if (__hip_atomic_load(t.act + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > frame)
                atomicMin(t.act + h, frame);
            return;
        }
        h = (h + 1) & t.mask;
    }
    atomicOr(t.flags, kBvolFull);
}

// Whether block (bx, by, bz) is in the table with a scan up to `frame`, by
// cached loads, the first key and scan at once (a quarter of the blocks is
// further on).  True is certain: during the launch a key only goes from free to
// its value and a first scan only down, and the caches hold nothing from
// before the launch.
__device__ __forceinline__ bool bvol_present(const BvolDev &t, int bx, int by, int bz, int frame)
{
    const unsigned long long key = bvol_key(bx, by, bz);
    uint32_t h = bvol_hash(key) & t.mask;
    for (int probe = 0; probe < 16; ++probe) {
        const unsigned long long k = __hip_atomic_load(t.keys + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const int f = __hip_atomic_load(t.act + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (k == key)
            return f <= frame;
        if (k == kBvolEmpty)
            return false;
        h = (h + 1) & t.mask;
    }
    return false;
}

__device__ __forceinline__ int bvol_find(const BvolDev &t, int bx, int by, int bz)
{
    if (!bvol_in_range(bx) || !bvol_in_range(by) || !bvol_in_range(bz))
        return -1;
    const unsigned long long key = bvol_key(bx, by, bz);
    uint32_t h = bvol_hash(key) & t.mask;
    for (uint32_t probe = 0; probe <= t.mask; ++probe) {
        const unsigned long long k = t.keys[h];
        if (k == key)
            return t.vals[h];
        if (k == kBvolEmpty)
            return -1;
        h = (h + 1) & t.mask;
    }
    return -1;
}

// floor(x / edge) by the reciprocal, and by the division where that could
// round to the other side (|x / edge| < 2^20 for every block of the table, so
// the product is within 4e-10 of the quotient).
__device__ __forceinline__ double block_of(double x, double edge, double inv)
{
    const double q = x * inv, l = floor(q), f = q - l;
    return f > 1e-9 && f < 1.0 - 1e-9 ? l : floor(x / edge);
}

// Grid: (64 columns, 4 ROWS rows, scan); each wavefront takes ROWS rows, one
// lane per column.  The cubes that are left to insert are queued in
// shared memory, and eight lanes look up the (mostly one to eight) blocks of
// one.  The kernel waits for its chain of dependent accesses (sensor tables,
// ranges, table entries; VALU 32% busy), so that many short wavefronts beat
// longer ones: 32 scans of 128 x 2048: 170 -> 56 us with 4 rows, 60 with 8, 82
// with 16 (before: a 64-bit division per return for its place, six FP64
// divisions, every cube inserted by one lane, through the XCDs' caches).
template <int ROWS>
__global__ __launch_bounds__(256) void k_bvol_activate(const BvolActArgs a)
{
    __shared__ int s_lo[4][64 * ROWS][3], s_hi[4][64 * ROWS][3];
    const int H = cload(&a.tab->H), W = cload(&a.tab->W);
    const double *row = cload(&a.tab->row), *col = cload(&a.tab->col);
    const double r0 = cload(&a.tab->r0), inv = 1.0 / a.edge;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int f = blockIdx.z, frame = a.frame0 + f;
    const SdfFrame &F = a.f[f];
    const float *rng = a.ranges + (int64_t)f * H * W;
    const int u = blockIdx.x * 64 + lane, v0 = ((int)blockIdx.y * 4 + wave) * ROWS;
    double ca = 0.0, sa = 0.0;
    if (u < W)
        ld2(col + 2 * u, ca, sa);
    float rf[ROWS];
#pragma unroll
    for (int k = 0; k < ROWS; ++k)
        rf[k] = u < W && v0 + k < H ? rng[(int64_t)(v0 + k) * W + u] : 0.f;
    int plo[3] = {0, 0, 0}, phi[3] = {0, 0, 0};  // the row before
    bool pon = false;
    int queued = 0;
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        int lo[3] = {0, 0, 0}, hi[3] = {-1, -1, -1};
        bool on = range_ok(rf[k]) && !(a.clip > 0.0 && (double)rf[k] > a.clip);
        if (on) {
            const V3<double> d0 = ray_dir(sld4(row, min(v0 + k, H - 1)), ca, sa);
            const double r = (double)rf[k];
            const double d[3] = {r * d0.x + r0 * ca - F.t[0], r * d0.y + r0 * sa - F.t[1], r * d0.z - F.t[2]};
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const double x = F.R[j] * d[0] + F.R[3 + j] * d[1] + F.R[6 + j] * d[2] - a.origin[j];
                const double l = block_of(x - a.radius, a.edge, inv), h = block_of(x + a.radius, a.edge, inv);
                // outside the table's coordinate range
                on = on && l > (double)-kBvolBias && h < (double)kBvolBias;
                lo[j] = (int)l;
                hi[j] = (int)h;
            }
            if (!on)
                atomicOr(a.t.flags, kBvolRange);
        }
        const bool above = pon && plo[0] == lo[0] && plo[1] == lo[1] && plo[2] == lo[2] && phi[0] == hi[0] &&
                           phi[1] == hi[1] && phi[2] == hi[2];
        const int q0 = __shfl_up(lo[0], 1), q1 = __shfl_up(lo[1], 1), q2 = __shfl_up(lo[2], 1);
        const int p0 = __shfl_up(hi[0], 1), p1 = __shfl_up(hi[1], 1), p2 = __shfl_up(hi[2], 1);
        const bool qon = __shfl_up(on ? 1 : 0, 1) != 0;
        const bool left = lane > 0 && qon && q0 == lo[0] && q1 == lo[1] && q2 == lo[2] && p0 == hi[0] &&
                          p1 == hi[1] && p2 == hi[2];
        const bool lead = on && !left && !above;
        const unsigned long long m = __builtin_amdgcn_ballot_w64(lead);
        if (lead) {
            const int at = queued + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                s_lo[wave][at][j] = lo[j];
                s_hi[wave][at][j] = hi[j];
            }
        }
        queued += __builtin_popcountll(m);
        pon = on;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            plo[j] = lo[j];
            phi[j] = hi[j];
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // lane bits 0..2: the block's offset in the cube (cubes of up to two
    // blocks a side; larger ones go on in steps of two)
    for (int e = lane >> 3; e < queued; e += 8) {
        const int x0 = s_lo[wave][e][0], y0 = s_lo[wave][e][1], z0 = s_lo[wave][e][2];
        const int x1 = s_hi[wave][e][0], y1 = s_hi[wave][e][1], z1 = s_hi[wave][e][2];
        for (int z = z0 + (lane >> 2 & 1); z <= z1; z += 2)
            for (int y = y0 + (lane >> 1 & 1); y <= y1; y += 2)
                for (int x = x0 + (lane & 1); x <= x1; x += 2)
                    if (!bvol_present(a.t, x, y, z, frame))
                        bvol_insert(a.t, x, y, z, frame);
    }
}

// Slots of the +x, +y, +z, +x+y, +x+z, +y+z and +x+y+z neighbours of every
// block (-1: not active).
__global__ __launch_bounds__(256) void k_bvol_neighbors(const BvolDev t, int n_blocks, int *nbr)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kNbrPerBlock * n_blocks)
        return;
    const int b = i / kNbrPerBlock, d = i - kNbrPerBlock * b;
    constexpr int kDx[kNbrPerBlock] = {1, 0, 0, 1, 1, 0, 1}, kDy[kNbrPerBlock] = {0, 1, 0, 1, 0, 1, 1},
                  kDz[kNbrPerBlock] = {0, 0, 1, 0, 1, 1, 1};
    const int4 B = t.blocks[b];
    nbr[i] = bvol_find(t, B.x + kDx[d], B.y + kDy[d], B.z + kDz[d]);
}

// Block coordinates and activation scans of the pool, in slot order.
__global__ __launch_bounds__(256) void k_bvol_export(const BvolDev t, int n_blocks, int4 *out)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_blocks)
        return;
    const int4 B = t.blocks[b];
    out[b] = make_int4(B.x, B.y, B.z, t.act[B.w]);
}

hipError_t launch_bvol_activate(const BvolActArgs &a, hipStream_t stream)
{
    // fewer rows a wavefront where the launch would not give each of the 256
    // CUs four workgroups: the inserts of a wavefront's cubes are its chain
    // (one scan of 16 x 256 into an empty table 36.2 us with 4 rows, 18.9 with
    // 1; a call with one scan of 128 x 2048 127 and 122)
    const unsigned nc = (unsigned)(a.W + 63) / 64u, nf = (unsigned)a.n_frames;
    auto rows = [&](unsigned r) { return ((unsigned)a.H + 4u * r - 1u) / (4u * r); };
    if ((int64_t)nc * rows(4) * nf >= 1024)
        hipLaunchKernelGGL(k_bvol_activate<4>, dim3(nc, rows(4), nf), dim3(256), 0, stream, a);
    else if ((int64_t)nc * rows(2) * nf >= 1024)
        hipLaunchKernelGGL(k_bvol_activate<2>, dim3(nc, rows(2), nf), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL(k_bvol_activate<1>, dim3(nc, rows(1), nf), dim3(256), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_bvol_neighbors(const BvolDev &t, int n_blocks, int *nbr, hipStream_t stream)
{
    if (n_blocks <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_bvol_neighbors, dim3((kNbrPerBlock * n_blocks + 255) / 256), dim3(256), 0, stream, t,
                       n_blocks, nbr);
    return hipGetLastError();
}

hipError_t launch_bvol_export(const BvolDev &t, int n_blocks, int4 *out, hipStream_t stream)
{
    if (n_blocks <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_bvol_export, dim3((n_blocks + 255) / 256), dim3(256), 0, stream, t, n_blocks, out);
    return hipGetLastError();
}

}  // namespace rir
