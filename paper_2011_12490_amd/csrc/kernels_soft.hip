// The soft decomposition on gfx950 (Sec. 3.2 Eq. 4-6 with the soft Voronoi
// weights of Sec. 3.3 Eq. 8): every head evaluates every sample (the grouped
// MLP with one all-samples bucket per head), then each sample's outputs are
// blended by
//   w_k(x) = exp(-beta |x - phi_k|) / sum_j exp(-beta |x - phi_j|)
// and the ray is composited front to back.  The per-ray head contributions
// of Eq. 6 come out of the same pass.
//
// Sample positions use the same explicit fused multiply-adds as the
// nearest-site path (no other contraction).
#pragma clang fp contract(off)

#include "derf_device.h"
#include "derf_internal.h"

namespace derf {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

// bucket[i] = i for every sample, totals[k] = S for every head, and the MLP's
// tile counters cleared: every head's rows are all the samples.
__global__ __launch_bounds__(kThreads) void soft_setup_kernel(unsigned S, int num_sites,
                                                              unsigned *__restrict__ bucket,
                                                              unsigned *__restrict__ totals,
                                                              unsigned *__restrict__ queue)
{
    const unsigned i0 = blockIdx.x * kThreads + threadIdx.x;
    if (i0 < (unsigned)num_sites)
        totals[i0] = S;
    if (i0 < (unsigned)(kMlpQueues * kMaxHeadGroups))
        queue[i0] = 0;
    for (unsigned i = i0; i < S; i += gridDim.x * kThreads)
        bucket[i] = i;
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        v += __shfl_xor(v, o);
    return v;
}

// product of v over lanes 0 .. lane
__device__ __forceinline__ float wave_inclusive_product(float v, int lane)
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float u = __shfl_up(v, o);
        if (lane >= o)
            v *= u;
    }
    return v;
}

__device__ __forceinline__ float site_distance(const float4 &p, float x, float y, float z)
{
    const float ex = x - p.x, ey = y - p.y, ez = z - p.z;
    return sqrtf(fmaf(ez, ez, fmaf(ey, ey, ex * ex)));
}

// Heads up to which the blend's distances and weights stay in LDS (STAGE): a
// row of 64 samples per head and wave, padded by one word, 67 KB per workgroup
// at 64 heads.
constexpr int kStageHeads = 64;
constexpr int kRow = 65;
// the static arrays' bytes at most (sites, positions or one row of them, coefficients)
constexpr size_t kStaticLds = kMaxSites * sizeof(float4) + 64 * sizeof(float4) + kWaves * 64 * sizeof(float);
// sr loads in flight per lane
constexpr int kBatch = 8;

// One wave per ray, 64 samples at a time (one per lane).  sr holds head k's
// (sigma, r, g, b) of sample s at k * S + s.  The blend is normalised by its
// own sum, and the weights are shifted by the nearest site's distance so that
// the largest is exp(0) = 1 and none overflows.  Compositing uses the
// midpoint intervals of the nearest-site path; the running transmittance
// passes from chunk to chunk, colour and depth add up per lane and are summed
// over the wave once per ray.
//
// What bounds it is the latency of the sr loads (a batch of training rays,
// 512 or so, leaves half the SIMDs without a wave) and their bandwidth on
// whole frames, so kBatch heads' loads are in flight, the first ones before
// the distances are computed.  STAGE: the distances go to LDS, the weights
// replace them, and the contributions (CONTRIB) are sums over that table: lane
// (part, k) adds head k's shares of every parts-th sample, and the parts meet
// once per ray.  Without STAGE, lane k computes head k's weight of every
// sample again (heads k, k + 64, ..).  512 rays of 128 samples, 16 heads, with
// contributions: 41 us before (one load at a time, every weight computed
// again by 16 of the 64 lanes), 13 us.
template <bool CONTRIB, bool STAGE>
__global__ __launch_bounds__(kThreads) void soft_composite_kernel(
    RenderGeometry g, const float4 *__restrict__ sites, int num_sites, HeadMask empty, float beta,
    const float *__restrict__ t, const float4 *__restrict__ sr, float *__restrict__ rgb,
    float *__restrict__ depth, float *__restrict__ opacity, float *__restrict__ contrib)
{
    extern __shared__ float s_table[];  // STAGE: [waves][num_sites][kRow]
    __shared__ float4 s_sites[kMaxSites];
    __shared__ float4 s_x[CONTRIB && !STAGE ? kWaves : 1][64];  // position, nearest distance
    __shared__ float s_coef[CONTRIB ? kWaves : 1][64];          // rendering weight / normaliser
    for (int k = threadIdx.x; k < num_sites; k += kThreads)
        s_sites[k] = sites[k];
    __syncthreads();
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const unsigned r = blockIdx.x * kWaves + wv;
    if (r >= g.num_rays)
        return;
    const unsigned n = g.n;
    const size_t S = g.num_samples;
    const float ox = g.rays_o[3 * (size_t)r], oy = g.rays_o[3 * (size_t)r + 1], oz = g.rays_o[3 * (size_t)r + 2];
    const float dx = g.rays_d[3 * (size_t)r], dy = g.rays_d[3 * (size_t)r + 1], dz = g.rays_d[3 * (size_t)r + 2];
    float *const table = s_table + (size_t)wv * num_sites * kRow;
    // LDS written by some lanes of the wave and read by others
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // STAGE: the wave's lanes as (part, head): heads padded to a power of two
    const int kbits = num_sites > 1 ? 32 - __builtin_clz((unsigned)num_sites - 1) : 0;
    const int part_k = lane & ((1 << kbits) - 1);

    float C0 = 0.0f, C1 = 0.0f, C2 = 0.0f, D = 0.0f, T = 1.0f;
    float W[CONTRIB && !STAGE ? kMaxSites / 64 : 1] = {};
    for (unsigned c0 = 0; c0 < n; c0 += 64) {
        const unsigned i = c0 + lane;
        const bool ok = i < n;
        const size_t si = (size_t)r * n + (ok ? i : n - 1);
        // a 0-capacity head contributes no density and no colour
        float4 v[kBatch];
        auto load = [&](int k0) {
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
                v[j] = k0 + j < num_sites && !empty.test(k0 + j)
                           ? sr[(size_t)(k0 + j) * S + si]
                           : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        };
        load(0);
        const float ti = t[si];
        // midpoint interval of sample i (Sec. 3.1 Eq. 1-2)
        const float tp = si > 0 ? t[si - 1] : 0.0f;
        const float tn = si + 1 < S ? t[si + 1] : 0.0f;
        const float lo = i == 0 ? g.near_t : 0.5f * (tp + ti);
        const float hi = i + 1 >= n ? g.far_t : 0.5f * (ti + tn);
        const float delta = ok ? hi - lo : 0.0f;
        const float x = fmaf(ti, dx, ox), y = fmaf(ti, dy, oy), z = fmaf(ti, dz, oz);
        float dmin = INFINITY, Z = 0.0f, sig = 0.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f;
        for (int k = 0; k < num_sites; ++k) {
            const float dk = site_distance(s_sites[k], x, y, z);
            if constexpr (STAGE)
                table[k * kRow + lane] = dk;
            dmin = fminf(dmin, dk);
        }
        for (int k0 = 0; k0 < num_sites; k0 += kBatch) {
            float4 u[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
                u[j] = v[j];
            if (k0 + kBatch < num_sites)
                load(k0 + kBatch);
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int k = k0 + j;
                if (k < num_sites) {
                    const float dk = STAGE ? table[k * kRow + lane] : site_distance(s_sites[k], x, y, z);
                    const float wk = __expf(-beta * (dk - dmin));
                    if constexpr (STAGE && CONTRIB)
                        table[k * kRow + lane] = wk;
                    Z += wk;
                    sig = fmaf(wk, u[j].x, sig);
                    cr = fmaf(wk, u[j].y, cr);
                    cg = fmaf(wk, u[j].z, cg);
                    cb = fmaf(wk, u[j].w, cb);
                }
            }
        }
        const float iz = 1.0f / Z;
        const float tau = ok ? __expf(-sig * iz * delta) : 1.0f;
        const float alpha = 1.0f - tau;
        const float incl = wave_inclusive_product(tau, lane);
        float excl = __shfl_up(incl, 1);
        if (lane == 0)
            excl = 1.0f;
        const float w = ok ? T * excl * alpha : 0.0f;  // rendering weight T_i alpha_i
        C0 = fmaf(w, cr * iz, C0);
        C1 = fmaf(w, cg * iz, C1);
        C2 = fmaf(w, cb * iz, C2);
        D = fmaf(w, ti, D);
        T *= __shfl(incl, 63);
        if constexpr (CONTRIB) {
            const unsigned cnt = n - c0 < 64u ? n - c0 : 64u;
            s_coef[wv][lane] = ok ? w / Z : 0.0f;
            if constexpr (STAGE) {
                wave_sync();
                if (part_k < num_sites)
                    for (unsigned j = (unsigned)lane >> kbits; j < cnt; j += 64u >> kbits)
                        W[0] = fmaf(s_coef[wv][j], table[part_k * kRow + j], W[0]);
                wave_sync();  // the next chunk rewrites the table
            } else {
                s_x[wv][lane] = make_float4(x, y, z, dmin);
                wave_sync();
                for (unsigned j = 0; j < cnt; ++j) {
                    const float4 q = s_x[wv][j];
                    const float cf = s_coef[wv][j];
#pragma unroll
                    for (int m = 0; m < kMaxSites / 64; ++m) {
                        const int k = lane + 64 * m;
                        if (k < num_sites)
                            W[m] = fmaf(cf, __expf(-beta * (site_distance(s_sites[k], q.x, q.y, q.z) - q.w)),
                                        W[m]);
                    }
                }
                wave_sync();
            }
        }
    }
    C0 = wave_sum(C0);
    C1 = wave_sum(C1);
    C2 = wave_sum(C2);
    D = wave_sum(D);
    if (lane == 0) {
        rgb[3 * (size_t)r] = C0;
        rgb[3 * (size_t)r + 1] = C1;
        rgb[3 * (size_t)r + 2] = C2;
        depth[r] = D;
        opacity[r] = 1.0f - T;
    }
    if constexpr (CONTRIB && STAGE) {
        for (int o = 1 << kbits; o < 64; o <<= 1)
            W[0] += __shfl_xor(W[0], o);
        if (lane < num_sites)
            contrib[(size_t)r * num_sites + lane] = W[0];
    } else if constexpr (CONTRIB) {
#pragma unroll
        for (int m = 0; m < kMaxSites / 64; ++m) {
            const int k = lane + 64 * m;
            if (k < num_sites)
                contrib[(size_t)r * num_sites + k] = W[m];
        }
    }
}

}  // namespace

hipError_t launch_soft_setup(unsigned S, int num_sites, unsigned *bucket, unsigned *totals,
                             unsigned *queue, hipStream_t s)
{
    const unsigned blocks = (S + kThreads - 1) / kThreads;
    soft_setup_kernel<<<blocks < 4096u ? (blocks ? blocks : 1u) : 4096u, kThreads, 0, s>>>(
        S, num_sites, bucket, totals, queue);
    return hipGetLastError();
}

hipError_t launch_soft_composite(const RenderGeometry &g, const float4 *sites, int num_sites,
                                 const HeadMask &empty, float beta, const float *t,
                                 const float4 *sr, float *rgb, float *depth, float *opacity,
                                 float *contrib, hipStream_t s)
{
    const unsigned blocks = (g.num_rays + kWaves - 1) / kWaves;
    const bool stage = num_sites <= kStageHeads;
    const size_t lds = stage ? (size_t)kWaves * num_sites * kRow * sizeof(float) : 0;
    auto go = [&](auto kernel) {
        // more than 64 KB of LDS (58 heads on, with the 6 KB of the static
        // arrays) has to be allowed, where the runtime keeps that limit; the
        // launch reports any real problem
        if (lds + kStaticLds > 0x10000 && hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                                (int)lds) != hipSuccess)
            (void)hipGetLastError();
        kernel<<<blocks, kThreads, lds, s>>>(g, sites, num_sites, empty, beta, t, sr, rgb, depth,
                                             opacity, contrib);
    };
    if (contrib)
        stage ? go(soft_composite_kernel<true, true>) : go(soft_composite_kernel<true, false>);
    else
        stage ? go(soft_composite_kernel<false, true>) : go(soft_composite_kernel<false, false>);
    return hipGetLastError();
}

}  // namespace derf
