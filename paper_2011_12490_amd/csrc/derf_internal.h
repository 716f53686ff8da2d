// Internal interfaces between the host API (derf_api.cpp) and the HIP kernel
// sources.  Nothing here is part of the public C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace derf {

// Samples covered by one bucketing block: the counting pass and the scatter
// pass must agree on this partition of the sample range.
constexpr int kBucketBlock = 4096;
// The same for frames of at most kSmallFrame samples: a block of 4096 leaves
// most of the chip idle there (1,024 rays of 192 samples are 48 blocks), and
// each block takes four rounds one after another.  Above, 4096 keeps the
// counts (and their scan) a quarter as long.  196,608 samples of 16 heads:
// assignment, scan and scatter 15.2 + 4.8 + 9.4 us in blocks of 4096; 6.0 and,
// the scan in the scatter, 5.6 us in blocks of 1024.  Whole renders through
// 4x64 bf16 heads, us in blocks of 4096 and of 1024:
//   samples   1 head        16 heads      64 heads      256 heads
//   131,072   29.6,  23.5   37.6,  26.7   82.0,  67.0   177.8, 161.3
//   1 << 20   124.0, 122.0  131.0, 124.0  177.0, 163.8  301.7, 288.4
//   1 << 21   176.2, 178.8  184.5, 178.4  230.0, 217.4  364.2, 353.9
//   1 << 22   285.7, 310.8  299.0, 290.3  339.9, 332.4  486.0, 480.0
// so the line lies where 1024 is the faster one for every number of heads.
// (The culled render keeps 4096 at every size: its level kernels are built for
// that partition alone, and the smaller one has not been measured there.)
constexpr int kSmallBlock = 1024;
constexpr unsigned kSmallFrame = 1u << 20;
inline unsigned bucket_block(unsigned num_samples)
{
    return num_samples <= kSmallFrame ? (unsigned)kSmallBlock : (unsigned)kBucketBlock;
}
// (head, block) counts up to which the scatter scans them itself, each of its
// blocks reading all (20 KB); above, a launch of its own is faster.  us per
// render, scan launched and in the scatter: 128 counts 27.1, 25.1; 3,072 30.1,
// 28.7; 4,688 146.7, 143.9; 5,008 35.5, 35.4; 8,192 120.8, 124.3; 32,768 151, 161.
constexpr unsigned long long kScanInScatter = 5120;
// Padded length of the per-ray direction feature vector gamma(d / |d|).
constexpr int kDirPad = 32;
constexpr int kMaxSites = 256;
// Tile counters of the MLP's work queues (one per XCD), for each of at most
// kMaxHeadGroups MLP launches of a render (one per head architecture).
constexpr int kMlpQueues = 8;
constexpr int kMaxHeadGroups = 4;

// Heads marked 0-capacity (empty space: no density anywhere), one bit each.
struct HeadMask {
    unsigned w[kMaxSites / 32];
    __host__ __device__ bool test(int k) const { return (w[k >> 5] >> (k & 31)) & 1u; }
};

// Per-ray cell walk (see ray_walk_kernel): at most kMaxSeg segments per ray,
// each with at most kMaxCand candidate sites.
constexpr int kMaxSeg = 32;
constexpr int kMaxCand = 11;
struct alignas(16) SegRec {
    float t_end;             // the segment covers depths up to t_end
    // low four bits: candidate sites; high four bits, if not 0: no site comes
    // near the segment's own between 2^-high of its length from either end
    unsigned char ncand_safe;
    unsigned char cand[kMaxCand];  // the segment's own site, then the others, ascending
};
// Heads from which the assignment uses the walk instead of all sites (below,
// the search over all sites costs less than the walk and its table lookups).
constexpr int kWalkSites = 17;
struct WalkTable {
    const SegRec *seg;           // [R][kMaxSeg]
    const unsigned char *nseg;   // [R]; 0: the ray takes the search over all sites
};

struct RenderGeometry {
    const float *rays_o;
    const float *rays_d;
    unsigned num_rays;
    unsigned n;          // samples per ray
    unsigned num_samples;
    double inv_n;        // 1.0 / n, for the sample -> (ray, index) split
    float near_t, far_t, step;
    uint64_t seed;
    uint64_t ray_offset;
    int perturb;
};

// ---- MLP gating (kernels_gate.hip) ---------------------------------------
// Gating networks with a compiled kernel: gamma_L(x) with L = 6 or 10 as
// input, one ReLU layer of 16, 32 or 64 units, K logits.
bool gate_shape_supported(int pos_freqs, int hidden);
// Bytes of a gate's weights and biases laid out for the kernel, and the
// layout itself from the packed fp32 order of derf.h (host side).
size_t gate_packed_bytes(int pos_freqs, int hidden, int num_sites);
void gate_pack(int pos_freqs, int hidden, int num_sites, const float *w, unsigned char *out);
// t[s] = the stratified depth of sample s (as the single pass draws it), and
// cell[s] = argmax of the gating logits there; also to out_cell (int32 [S])
// when not null.  packed: gate_pack's layout on the device; cus: compute
// units (the kernel's workgroups are persistent).
hipError_t launch_gate(const RenderGeometry &g, const unsigned char *packed, int pos_freqs,
                       int hidden, int num_sites, float *t, uint8_t *cell, int *out_cell, int cus,
                       hipStream_t s);

// ---- sampling, assignment and bucketing (kernels_sample.hip) -------------
// p[0 .. count) = v (a kernel: no memset node in a captured stream)
hipError_t launch_fill_u32(unsigned *p, unsigned count, unsigned v, hipStream_t s);
hipError_t launch_ray_encode(const RenderGeometry &g, void *dirbuf, bool bf16, hipStream_t s);
// Where launch_sample_assign also writes the rays' direction features (as
// launch_ray_encode does, by blocks of its own beside the assignment's): one
// launch instead of two.
struct DirOut {
    void *buf;  // null: not here
    bool bf16;
};
// Walk every ray of g through the cells on [near, far] (one lane per ray).
hipError_t launch_ray_walk(const RenderGeometry &g, const float4 *sites, int num_sites,
                           SegRec *seg, unsigned char *nseg, hipStream_t s);
// walk: the table of launch_ray_walk for the same rays, or {nullptr, nullptr}
// block: samples per block of the counts (kBucketBlock or kSmallBlock)
hipError_t launch_sample_assign(const RenderGeometry &g, const float4 *sites, int num_sites,
                                const WalkTable &walk, float *t, uint8_t *cell,
                                unsigned *counts, unsigned num_blocks, unsigned block,
                                const DirOut &dir, hipStream_t s);
// same, for given depths t (read only): no sampling
hipError_t launch_assign_given(const RenderGeometry &g, const float4 *sites, int num_sites,
                               const WalkTable &walk, const float *t,
                               uint8_t *cell, unsigned *counts, unsigned num_blocks,
                               unsigned block, hipStream_t s);
// The counts of given cells (the layout of the assignment's).
hipError_t launch_cell_count(const RenderGeometry &g, const uint8_t *cell, int num_sites,
                             unsigned *counts, unsigned num_blocks, unsigned block, hipStream_t s);
// also clears the kMlpQueues tile counters of the MLP launch that follows
hipError_t launch_bucket_scan(unsigned *counts, unsigned num_blocks, int num_sites,
                              unsigned *totals, unsigned *mlp_queue, hipStream_t s);
// Samples of 0-capacity heads also get sr = 0 here (the MLP skips those heads).
hipError_t launch_bucket_scatter(const uint8_t *cell, const unsigned *counts,
                                 const unsigned *totals, unsigned num_samples,
                                 unsigned num_blocks, unsigned block, int num_sites,
                                 const HeadMask &empty, unsigned *bucket, float4 *sr,
                                 hipStream_t s);
// launch_bucket_scan and launch_bucket_scatter in one launch, for at most
// kScanInScatter counts (which stay as they are).
hipError_t launch_bucket_scan_scatter(const uint8_t *cell, const unsigned *counts,
                                      unsigned *totals, unsigned *mlp_queue,
                                      unsigned num_samples, unsigned num_blocks, unsigned block,
                                      int num_sites, const HeadMask &empty, unsigned *bucket,
                                      float4 *sr, hipStream_t s);
// Soft decomposition: bucket[i] = i (i < S), totals[k] = S, queue cleared.
hipError_t launch_soft_setup(unsigned S, int num_sites, unsigned *bucket, unsigned *totals,
                             unsigned *queue, hipStream_t s);
// Blend every head's outputs sr[k * S + i] by the soft Voronoi weights and
// composite; contrib (nullable) receives the per-ray head contributions.
hipError_t launch_soft_composite(const RenderGeometry &g, const float4 *sites, int num_sites,
                                 const HeadMask &empty, float beta, const float *t,
                                 const float4 *sr, float *rgb, float *depth, float *opacity,
                                 float *contrib, hipStream_t s);
hipError_t launch_composite(const RenderGeometry &g, const float *t, const uint8_t *cell,
                            const float4 *sr, float *rgb, float *depth, float *opacity,
                            hipStream_t s);
hipError_t launch_debug_expand(unsigned num_samples, const float *t, const uint8_t *cell,
                               const float4 *sr, int *dcell, float *dt, float *dsigma,
                               float *drgb, hipStream_t s);

// ---- hierarchical sampling (kernels_fine.hip) -----------------------------
// g describes the coarse pass (n = n_coarse).  tf [R][n_fine] receives the
// sorted inverse-CDF depths drawn from the coarse outputs src.
hipError_t launch_fine_sample(const RenderGeometry &g, const float *tc, const float4 *src,
                              unsigned n_fine, float *tf, hipStream_t s);
// Composite of the depth-ordered merge of the coarse (tc, cc, sc) and fine
// (tf, cf, sf) samples; the optional debug arrays receive the merged fields.
hipError_t launch_merge_composite(const RenderGeometry &g, const float *tc, const uint8_t *cc,
                                  const float4 *sc, unsigned n_fine, const float *tf,
                                  const uint8_t *cf, const float4 *sf, float *rgb, float *depth,
                                  float *opacity, int *dcell, float *dt, float *dsigma,
                                  float *drgb, hipStream_t s);

// ---- grouped per-head MLP (mlp_kernel.h, mlp_*.hip) ----------------------
struct HeadArch {
    int pos_freqs, dir_freqs, depth, width, skip_layer, rgb_hidden;
};

struct MlpVariant {
    // bytes of one head's fragment stream and of its resident block
    size_t stream_bytes;
    size_t block_bytes;
    int tile;            // samples per tile
    // Lay out one head's fp32 weights (packed order of derf.h) for the kernel.
    void (*pack)(const float *w, unsigned char *stream, float *block);
    // queue: kMlpQueues tile counters, zero at launch.  soft: every head
    // takes every sample (bucket = 0 .. S-1, totals[k] = S) and writes its
    // outputs to sr[k * S + sample]; otherwise sr[sample].  offsets: null
    // (head k's entries follow head k - 1's), or where each head's totals[k]
    // entries start in bucket (not soft).  gxtab: null, or for the
    // stored-encoding form (which needs it, and takes no soft launch) the
    // table its encode wrote for the same samples.
    hipError_t (*launch)(const unsigned *bucket, const unsigned *totals, const unsigned *offsets,
                         int num_sites,
                         const RenderGeometry &g, const float *t, const void *dirbuf,
                         const void *gxtab, const unsigned char *streams, const float *blocks,
                         float4 *sr, unsigned *queue, int grid, bool soft, const HeadMask &empty,
                         hipStream_t s);
    // The stored-encoding form of this architecture (same packed weights;
    // gamma(x) read from a table instead of encoded per tile), or null.
    const MlpVariant *stored;
    // stored-encoding form only: table bytes per sample, the number of
    // position frequencies, and the kernel that fills the table from the
    // depths t of g's samples (one row per sample)
    size_t gx_bytes;
    int pos_freqs;
    hipError_t (*encode)(const RenderGeometry &g, const float *t, void *gxtab, int cus,
                         hipStream_t s);
    // a form for some weights only: whether a head's fit, and the form for
    // the others (null: every head's fit)
    const MlpVariant *plain;
    bool (*fits)(const float *w);
};

// Returns nullptr when no kernel is compiled for this architecture/precision.
const MlpVariant *find_mlp_variant(const HeadArch &a, bool bf16);
// the variants of each supported head architecture (one translation unit each;
// nullptr where a precision is not built)
const MlpVariant *mlp_variant_4x64(bool bf16);
const MlpVariant *mlp_variant_6x64(bool bf16);
const MlpVariant *mlp_variant_8x128(bool bf16);
const MlpVariant *mlp_variant_8x256(bool bf16);
// float32 heads: the form on the fp16 matrix units (split operands), and the
// form on the fp32 units that it names for weights that do not fit
const MlpVariant *mlp_split_4x64();
const MlpVariant *mlp_split_6x64();
const MlpVariant *mlp_split_8x128();
const MlpVariant *mlp_f32_4x64();
const MlpVariant *mlp_f32_6x64();
const MlpVariant *mlp_f32_8x128();

}  // namespace derf
