// Grouped per-head MLP on gfx950 matrix cores: the kernel template and its
// host-side launch and weight packing.  Included by one translation unit
// per head architecture (mlp_*.hip), which instantiates its variants.
//
// Every ray sample is evaluated by the single head that owns it (Sec. 3.2:
// the decomposition weights are one-hot, so only that head contributes).
// After bucketing, the samples of head k are one contiguous range, so the
// head network becomes a chain of dense products with M = (samples of k).
//
// Work split.  A workgroup of 4 waves (one per SIMD) takes a tile of one
// head's samples, NB x 32 per wave, and runs it through the whole network
// with the activations held in registers.  Two workgroups share a CU (one for
// width 256, three for width 64 but on the fp32 units); they do not synchronise with each
// other, so one's barriers and gathers are covered by another's matrix work.
// Workgroups are persistent and take tiles from per-XCD queues, each over a
// contiguous stretch of tiles (so an XCD's L2 sees few heads), stealing from
// the other stretches when their own runs out.
//
// Operand layout (v_mfma_f32_32x32x16_bf16 / _f16 / v_mfma_f32_32x32x2_f32;
// float32 heads as split fp16 operands, see Split, or on the fp32 units):
// weights are the A operand (32 output rows x k), samples the B operand
// (k x 32 samples).  Lane l = n + 32 g holds sample n; a 32x32 result leaves
// in lane l the 16 rows 8 (i / 4) + 4 g + (i % 4), i = 0..15, and the next
// layer consumes those registers directly as its B operand.  The k-order this
// implies is folded into the weight layout at creation time, so layers chain
// with no data movement.
//
// Weight streaming.  A head's weights are cut into stages -- one 32-row
// output tile and at most UMAX KB of its input chunks -- laid out as 1 KB units
// that are exactly one wave's A-operand registers.  Stages stream
// global -> LDS (global_load_lds_dwordx4, issued as asm so the compiler's
// LDS wait bookkeeping stays exact) through an 8-slot ring, six stages ahead
// (across tile boundaries too).  Stages are consumed in groups of two: before
// a group, each wave waits with a counted vmcnt for exactly the loads that
// group needs (the count is simulated at compile time from the issue order)
// and one fence-free barrier makes every wave's loads visible and orders
// slot reuse.  The per-step schedule is explicit: A fragments are read from
// LDS a few steps ahead (a window continuous across stages), and a tile's
// bias, ReLU and bf16 rounding are spread over the next tile's MFMAs.
// Density and colour come out of one extra 32-row output tile (row 0
// density, rows 1-3 colour logits), so the network tail needs no cross-lane
// reduction.
#pragma once
#include <math.h>
#include <string.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "derf_internal.h"

namespace derf {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short i16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

template <int N>
using ic = std::integral_constant<int, N>;

template <int B, int E, class F>
__host__ __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (B < E) {
        f(ic<B>{});
        static_for<B + 1, E>(f);
    }
}

// Row of a 32-row output tile held by lane group g in accumulator register i.
__host__ __device__ constexpr int c_row(int g, int i) { return 8 * (i / 4) + 4 * g + (i % 4); }

// ---------------------------------------------------------------------------
// Compile-time description of one head architecture / precision.
//
// Output tiles, in order: hidden layer l, tile mt (l * MT + mt); the colour
// hidden layer's tiles; the output tile.  Each tile's input is cut into
// stages of at most UMAX units.
enum { K_HID = 0, K_RGBH = 1, K_OUT = 2 };

// Arithmetic of a configuration: fp32 products on the fp32 matrix units, bf16
// operands, or fp32 operands split into two fp16 values (see Split below).
enum { P_F32 = 0, P_BF16 = 1, P_SPLIT = 2 };

// GX_: the stored-encoding form, which reads each sample's gamma(x) entries
// from a table in HBM (gx_encode_kernel) instead of encoding them in the
// tile prologue; kept to measure what the fusion saves.
template <int PREC_, int W_, int D_, int SKIP_, int RH_, int LP_, bool GX_ = false>
struct Cfg {
    static constexpr int PREC = PREC_;
    static constexpr bool BF16 = PREC == P_BF16, SPLIT = PREC == P_SPLIT;
    static constexpr int W = W_, D = D_, SKIP = SKIP_, RH = RH_, LP = LP_;
    static constexpr bool GX = GX_;
    static constexpr int E = PREC == P_F32 ? 1 : 8;    // k-entries per lane per MFMA
    static constexpr int CPU = PREC == P_F32 ? 4 : 1;  // MFMA k-chunks per 1 KB unit
    static constexpr int UPC = SPLIT ? 2 : 1;  // units per k-chunk (split: low half, high half)
    // A-fragment reads kept in flight ahead of the MFMA that uses them: during
    // step F (the F-th fragment of a tile) the wave reads fragment F + PF.
    static constexpr int PF = SPLIT ? 4 : 3;
    static constexpr int NB = BF16 ? 2 : 1;    // 32-sample column blocks per wave
    static constexpr int WAVES = 4;
    static constexpr int THREADS = WAVES * 64;
    // 64-wide heads but on the fp32 units: three workgroups per CU (4 KB ring
    // slots, at most 168 VGPRs), so that more waves hide the per-tile gathers
    // and encoding (split, 16.8 M samples of 6x64: 3.04 -> 2.92 ms)
    static constexpr int WG_PER_CU = W >= 256 ? 1 : (PREC != P_F32 && W == 64 ? 3 : 2);
    static constexpr int TILE = WAVES * NB * 32;
    static constexpr int P = 3 + 6 * LP;       // gamma(x) length
    static constexpr int DD = 27;              // gamma(d) length (4 frequencies)
    static constexpr int P0 = 3 * LP / 2;      // sin/cos pairs held by lane group 0
    static constexpr int EX = ((2 + 2 * P0) + 7) / 8 * 8;  // gamma(x) entries per lane
    static constexpr int EH = W / 2;           // hidden entries per lane
    static constexpr int ED = 16;              // direction entries per lane
    static constexpr int MT = W / 32;          // output tiles per hidden layer
    static constexpr int MTR = (RH + 31) / 32; // output tiles of the colour hidden layer
    static constexpr int ERH = MTR * 16;       // colour-hidden entries per lane
    static constexpr int EXC = EX / E, EHC = EH / E, EDC = ED / E, ERHC = ERH / E;
    static constexpr int UMAX = PREC != P_F32 && W == 64 ? 4 : 8;  // units per stage
    static constexpr int CMAX = UMAX * CPU / UPC;  // chunks per stage
    static constexpr int NBUF = 8;             // LDS ring slots (power of two)
    static constexpr int G = 2;                // stages per barrier
    static constexpr int LA = 6;               // weight loads issued this many stages ahead
    static constexpr int NT = D * MT + MTR + 1;
    static_assert(LP % 2 == 0, "pos_freqs must be even");
    static_assert(!GX || SKIP < 0, "the stored encoding has no skip-layer re-encode");
    static_assert(W % 64 == 0, "width");

    static constexpr int t_kind(int T) { return T < D * MT ? K_HID : (T < D * MT + MTR ? K_RGBH : K_OUT); }
    static constexpr int t_layer(int T) { return T < D * MT ? T / MT : -1; }
    static constexpr int t_mt(int T) { return T < D * MT ? T % MT : (T < D * MT + MTR ? T - D * MT : 0); }
    static constexpr int t_entries(int T)
    {
        return t_kind(T) == K_RGBH ? EH + ED
               : t_kind(T) == K_OUT ? EH + (RH > 0 ? ERH : ED)
               : t_layer(T) == 0    ? EX
               : t_layer(T) == SKIP ? EX + EH
                                    : EH;
    }
    static constexpr int t_chunks(int T) { return t_entries(T) / E; }
    static constexpr int t_splits(int T) { return (t_chunks(T) + CMAX - 1) / CMAX; }

    static constexpr int count_stages()
    {
        int n = 0;
        for (int T = 0; T < NT; ++T)
            n += t_splits(T);
        return n;
    }
    static constexpr int NS = count_stages();

    // per-stage table, built once at compile time
    struct StageTab {
        int tile[NS], split[NS], c0[NS], c1[NS], units[NS], lpw[NS], off[NS + 1], foff[NS + 1];
    };
    static constexpr StageTab make_tab()
    {
        StageTab t{};
        int s = 0;
        for (int T = 0; T < NT; ++T)
            for (int k = 0; k < t_splits(T); ++k, ++s) {
                t.tile[s] = T;
                t.split[s] = k;
                t.c0[s] = k * CMAX;
                t.c1[s] = (k + 1) * CMAX < t_chunks(T) ? (k + 1) * CMAX : t_chunks(T);
                t.units[s] = (t.c1[s] - t.c0[s]) * UPC / CPU;
                t.lpw[s] = (t.units[s] + WAVES - 1) / WAVES;
            }
        t.off[0] = 0;
        t.foff[0] = 0;
        for (int q = 0; q < NS; ++q) {
            t.off[q + 1] = t.off[q] + t.lpw[q] * WAVES;
            t.foff[q + 1] = t.foff[q] + t.units[q];
        }
        return t;
    }
    static constexpr StageTab TAB = make_tab();

    static constexpr int st_tile(int s) { return TAB.tile[s]; }
    static constexpr int st_split(int s) { return TAB.split[s]; }
    static constexpr int st_c0(int s) { return TAB.c0[s]; }
    static constexpr int st_c1(int s) { return TAB.c1[s]; }
    static constexpr bool st_first(int s) { return TAB.split[s] == 0; }
    static constexpr int st_units(int s) { return TAB.units[s]; }
    static constexpr int st_lpw(int s) { return TAB.lpw[s]; }  // loads per wave
    static constexpr int st_units_pad(int s) { return TAB.lpw[s] * WAVES; }
    static constexpr int st_offset(int s) { return TAB.off[s]; }  // in units
    static constexpr int STREAM_UNITS = TAB.off[NS];

    // A fragments of a tile's stages, numbered consecutively: stage s's
    // fragment j is number foff(s) + j.  The register window holds fragment
    // F in slot F % PF.
    static constexpr int foff(int s) { return TAB.foff[s]; }
    static constexpr int FTOTAL = TAB.foff[NS];
    static constexpr int f_stage(int F)
    {
        int q = 0;
        while (q + 1 < NS && TAB.foff[q + 1] <= F)
            ++q;
        return q;
    }
    static constexpr int f_index(int F) { return F - TAB.foff[f_stage(F)]; }

    static constexpr int first_stage_of_tile(int T)
    {
        int s = 0;
        for (int q = 0; q < T; ++q)
            s += t_splits(q);
        return s;
    }
    // first stage of the skip layer (gamma(x) is re-encoded one stage
    // earlier), first stage reading gamma(d), stage issuing the gamma(d) loads
    static constexpr int S_SKIP = SKIP >= 0 ? first_stage_of_tile(SKIP * MT) : -1;
    static constexpr int S_GDUSE = first_stage_of_tile(RH > 0 ? D * MT : D * MT + MTR);
    static constexpr int S_GD = S_GDUSE >= 4 ? (S_GDUSE - 4) / G * G : 0;  // a group start
    static constexpr int NGD = NB * (BF16 ? 2 : 4);  // gamma(d) load instructions per wave
    // The next tile's sample records are prefetched into LDS during this one:
    // its bucket ids at group start S_PA (NPA loads per wave), then, once the
    // group wait of S_PB has covered those, its depths and ray origins and
    // directions (NPB loads per wave; none in the stored-encoding form, whose
    // gamma(x) rows are read at the tile start).  The last tile re-reads its
    // own, so that the wait counts do not depend on whether a next tile exists.
    static constexpr int S_PA = 0, S_PB = LA;
    static constexpr int NPA = 1, NPB = GX ? 0 : 7;

    // Barrier groups: stages [a, a + G) of a tile share one barrier.  At a
    // group start a the wave issues the weight loads of stages a + LA ..
    // (the next tile's stages past the end), then the gamma(d) loads if a ==
    // S_GD.  Before the barrier of group a, the units of stage need(a) -- the
    // last stage the group's fragment reads reach: PF fragments past
    // its last step, which is beyond the next stage when that one is shorter
    // (the 2-unit stages of the 8x256 colour layer) -- must have landed;
    // vm_allowed(a) counts this wave's memory operations issued
    // after those loads (every operation before them has landed too: they
    // complete in issue order).  -1: nothing to wait for (the tile prologue
    // drained everything issued before stage LA's loads).
    static_assert(NS >= LA + G, "pipeline deeper than the stage list");
    static_assert(NBUF >= LA + G, "ring too small for the lookahead");
    static constexpr int grp_end(int a) { return a + G - 1 < NS ? a + G - 1 : NS - 1; }
    static constexpr int need(int a)
    {
        const int next = grp_end(a) + 1 < NS ? grp_end(a) + 1 : grp_end(a);
        const int fe = TAB.foff[grp_end(a) + 1] - 1 + PF;  // furthest fragment read
        const int reach = f_stage(fe < FTOTAL ? fe : FTOTAL - 1);
        return reach > next ? reach : next;
    }
    // every fragment a group reads lies in a stage its wait covers
    static constexpr bool waits_cover_reads()
    {
        for (int a = 0; a < NS; a += G) {
            const int fe = TAB.foff[grp_end(a) + 1] - 1 + PF;
            if ((fe < FTOTAL ? fe : FTOTAL - 1) >= TAB.foff[need(a) + 1])
                return false;
        }
        return true;
    }
    // the loads of need(a) were issued before group a (or drained by the tile
    // prologue), so the wait before its barrier can cover them
    static constexpr bool needs_issued_earlier()
    {
        for (int a = 0; a < NS; a += G)
            if (need(a) >= LA && (need(a) - LA) / G * G >= a)
                return false;
        return true;
    }
    static constexpr int vm_allowed(int a, bool has_next)
    {
        const int xn = need(a);
        if (xn < LA)
            return -1;
        const int gn = (xn - LA) / G * G;
        int cnt = 0;
        for (int g = gn; g < a; g += G) {
            for (int x = g + LA; x <= grp_end(g) + LA; ++x) {
                if (g == gn && x <= xn)
                    continue;
                if (x < NS)
                    cnt += st_lpw(x);
                else if (has_next)
                    cnt += st_lpw(x - NS);
            }
            if (g == S_GD)
                cnt += NGD;
            if (g == S_PA)
                cnt += NPA;
            if (g == S_PB)
                cnt += NPB;
        }
        return cnt;
    }
    // weight loads of a wave in stages 0 .. LA - 1 (at least: the head block's
    // share differs by wave)
    static constexpr int first_loads()
    {
        int cnt = 0;
        for (int x = 0; x < LA; ++x)
            cnt += st_lpw(x);
        return cnt < 63 ? cnt : 63;
    }
    // loads this wave issues after the S_PB prefetch until the next tile
    // starts (it has one: its records were prefetched)
    static constexpr int loads_after_pb()
    {
        int cnt = 0;
        for (int g = S_PB + G; g < NS; g += G)
            for (int x = g + LA; x <= grp_end(g) + LA; ++x)
                cnt += x < NS ? st_lpw(x) : st_lpw(x - NS);
        return cnt + (S_GD > S_PB ? NGD : 0);
    }
    static_assert(waits_cover_reads(), "a fragment read runs ahead of the group wait");
    static_assert(needs_issued_earlier(), "a group waits for weight loads issued after it");
    static_assert(S_PA % G == 0 && S_PB % G == 0 && S_PB < NS, "prefetch at group starts");
    // the group wait at S_PB covers the S_PA loads: the loads it waits for
    // were issued at a later group start
    static_assert((need(S_PB) - LA) / G * G > S_PA, "prefetch phases too close");

    // per-head resident block: bias of every output tile in accumulator layout;
    // split: then per hidden layer (the colour hidden layer last) the largest
    // row sum of |W|, the largest |b| and the inverse of the power of two that
    // its weights are stored with, in 16 bytes, then the output rows' factors
    static constexpr int SC_OFF = NT * 32, SC_OUT = SC_OFF + 4 * (D + 1);
    static constexpr int BLOCK_FLOATS = ((SPLIT ? SC_OUT + 4 : NT * 32) + 255) / 256 * 256;
    // the split form's re-encode at the skip layer takes the scale fixed
    // during the layer's second tile
    static_assert(!SPLIT || SKIP < 0 || MT >= 4, "skip re-encode before its scale is known");
    static constexpr int BLOCK_UNITS = BLOCK_FLOATS / 256;

    // LDS: ring | head block | per wave: the next tile's sample records
    // (bucket id, depth, origin xyz, direction xyz; 64 dwords each)
    static constexpr int SLOT_BYTES = UMAX * 1024;
    static constexpr int HB_OFF = NBUF * SLOT_BYTES;
    static constexpr int PF_OFF = HB_OFF + BLOCK_FLOATS * 4;
    static constexpr int PF_WAVE = 8 * 64 * 4;
    static constexpr int LDS_BYTES = PF_OFF + WAVES * PF_WAVE;
    static_assert(WG_PER_CU * (LDS_BYTES + 3 * 1024) <= 160 * 1024, "LDS budget");
    // a stage's loads cover its units padded to a multiple of WAVES
    static constexpr int max_units_pad()
    {
        int m = 0;
        for (int q = 0; q < NS; ++q)
            m = TAB.lpw[q] * WAVES > m ? TAB.lpw[q] * WAVES : m;
        return m;
    }
    static_assert(max_units_pad() * 1024 <= SLOT_BYTES, "a stage overflows its ring slot");
};

// Input column (in the packed layer's input order) of lane-entry e of lane
// group g, or -1 for a zero pad.  Layer inputs per lane group are lists:
// gamma(x): entry 0 = x | z, entry 1 = y | pad, then sin/cos pairs
// p = q + g P0 (level p / 3, coordinate p % 3) at entries 2 + 2q, 3 + 2q;
// hidden: entry e = 16 mt + i is row 32 mt + c_row(g, i) of the previous
// layer; direction: entries 0..7 are f[8 g + j], 8..15 are f[16 + 8 g + j].
template <class C>
constexpr int x_col(int g, int e)
{
    if (e == 0)
        return g ? 2 : 0;
    if (e == 1)
        return g ? -1 : 1;
    const int q = (e - 2) / 2;
    if (q >= C::P0)
        return -1;
    const int p = q + g * C::P0;
    const int l = p / 3, c = p % 3;
    return 3 + 6 * l + ((e - 2) % 2 ? 3 : 0) + c;
}
constexpr int h_col(int g, int e) { return 32 * (e / 16) + c_row(g, e % 16); }
constexpr int d_col(int g, int e) { return e < 8 ? 8 * g + e : 16 + 8 * g + (e - 8); }

// ---------------------------------------------------------------------------
// Host-side packing of one head (fp32 packed order of derf.h -> kernel layout).
template <class C>
struct Split;

template <class C>
struct Packer {
    struct View {
        const float *W;
        const float *b;
        int out, in;
    };

    static void views(const float *w, std::vector<View> &v)
    {
        const float *p = w;
        for (int l = 0; l < C::D; ++l) {
            const int in = l == 0 ? C::P : (l == C::SKIP ? C::P + C::W : C::W);
            v.push_back(View{p, p + C::W * in, C::W, in});
            p += C::W * in + C::W;
        }
        v.push_back(View{p, p + C::W, 1, C::W});  // density
        p += C::W + 1;
        if (C::RH > 0) {
            v.push_back(View{p, p + C::RH * (C::W + C::DD), C::RH, C::W + C::DD});
            p += C::RH * (C::W + C::DD) + C::RH;
            v.push_back(View{p, p + 3 * C::RH, 3, C::RH});
        } else {
            v.push_back(View{p, p + 3 * (C::W + C::DD), 3, C::W + C::DD});
        }
    }

    // Row m (0..31) of output tile T: its weights, or null for a row of zeros.
    // The output tile's row 0 is the density, rows 1..3 the colour logits.
    static const float *tile_row(const std::vector<View> &v, int T, int m)
    {
        const int kind = C::t_kind(T);
        const View &L = kind == K_HID    ? v[C::t_layer(T)]
                        : kind == K_RGBH ? v[C::D + 1]
                        : m == 0         ? v[C::D]
                                         : v.back();
        const int row = kind == K_OUT ? (m == 0 ? 0 : m - 1) : 32 * C::t_mt(T) + m;
        return row < L.out ? L.W + (size_t)row * L.in : nullptr;
    }
    // The column of that row which entry e of lane group g multiplies, or -1.
    static int tile_col(int T, int m, int g, int e)
    {
        const int kind = C::t_kind(T);
        auto dir = [&](int q) { return d_col(g, q) < C::DD ? C::W + d_col(g, q) : -1; };
        if (kind == K_HID) {
            if (C::t_layer(T) == 0)
                return x_col<C>(g, e);
            if (C::t_layer(T) == C::SKIP)
                return e < C::EX ? x_col<C>(g, e) : C::P + h_col(g, e - C::EX);
            return h_col(g, e);
        }
        if (kind == K_RGBH)
            return e < C::EH ? h_col(g, e) : dir(e - C::EH);
        if (m == 0)
            return e < C::EH ? h_col(g, e) : -1;
        if (C::RH == 0)
            return e < C::EH ? h_col(g, e) : dir(e - C::EH);
        return e < C::EH || h_col(g, e - C::EH) >= C::RH ? -1 : h_col(g, e - C::EH);
    }
    // The weights that entries [e, e + n) of every lane multiply in tile T:
    // out[lane][j].  (Columns do not depend on the row, but for row 0 of the
    // output tile, so they are looked up once and not for every weight.)
    template <int n>
    static void gather(const std::vector<View> &v, int T, int e, float (&out)[64][n])
    {
        for (int g = 0; g < 2; ++g) {
            int cols[2][n];
            for (int j = 0; j < n; ++j) {
                cols[0][j] = tile_col(T, 0, g, e + j);
                cols[1][j] = tile_col(T, 1, g, e + j);
            }
            for (int m = 0; m < 32; ++m) {
                const float *row = tile_row(v, T, m);
                const int *col = cols[m > 0];
                for (int j = 0; j < n; ++j)
                    out[m + 32 * g][j] = row && col[j] >= 0 ? row[col[j]] : 0.0f;
            }
        }
    }

    static float bval(const std::vector<View> &v, int T, int row)
    {
        const int kind = C::t_kind(T);
        if (kind == K_HID)
            return v[C::t_layer(T)].b[32 * C::t_mt(T) + row];
        if (kind == K_RGBH) {
            const int r = 32 * C::t_mt(T) + row;
            return r < C::RH ? v[C::D + 1].b[r] : 0.0f;
        }
        if (row == 0)
            return v[C::D].b[0];
        return row <= 3 ? v.back().b[row - 1] : 0.0f;
    }

    static void pack(const float *w, unsigned char *stream, float *block)
    {
        std::vector<View> v;
        views(w, v);
        if constexpr (C::SPLIT) {
            Split<C> sp(w, v);
            sp.pack(stream, block);
            return;
        }
        for (int s = 0; s < C::NS; ++s) {
            const int T = C::st_tile(s), c0 = C::st_c0(s);
            unsigned char *base = stream + (size_t)C::st_offset(s) * 1024;
            for (int u = 0; u < C::st_units_pad(s); ++u) {
                unsigned char *unit = base + (size_t)u * 1024;
                // bf16: 8 k-entries of chunk c0 + u; fp32: one each of chunks
                // c0 + 4 u .. + 3
                constexpr int n = C::BF16 ? 8 : 4;
                if (u >= C::st_units(s)) {
                    memset(unit, 0, 1024);
                    continue;
                }
                float x[64][n];
                gather(v, T, C::BF16 ? 8 * (c0 + u) : c0 + 4 * u, x);
                if constexpr (C::BF16) {
                    __bf16 y[64][n];
                    for (int i = 0; i < 64 * n; ++i)
                        y[i / n][i % n] = (__bf16)x[i / n][i % n];
                    memcpy(unit, y, sizeof(y));
                } else {
                    memcpy(unit, x, sizeof(x));
                }
            }
        }
        for (int i = 0; i < C::BLOCK_FLOATS; ++i)
            block[i] = 0.0f;
        for (int T = 0; T < C::NT; ++T)
            for (int g = 0; g < 2; ++g)
                for (int i = 0; i < 16; ++i)
                    block[(T * 2 + g) * 16 + i] = bval(v, T, c_row(g, i));
    }
};

// The split form: fp32 heads on the fp16 matrix units.
//
// Every fp32 operand a is carried as a_hi = fp16(a) and a_lo = fp16(a - a_hi)
// (nearest even, 23 significant bits together), every product as a_lo b_hi +
// a_hi b_lo + a_hi b_hi, accumulated in fp32: three MFMAs of 32x32x16 in 96
// cycles where the fp32 units take 512.  fp16's exponents are not fp32's, so
// both operands are kept in its range by powers of two (exact):
// - weights, here: each hidden unit's row and bias are scaled so that the
//   row's largest |weight| has the exponent of its layer's median row, and
//   the next layers' column of that unit by the inverse (a ReLU network is
//   unchanged by that); the layer's weights are stored times one power of
//   two more that takes them to [2^14, 2^15), undone on the accumulators.
//   (Units brought to [1, 2) each would grow from layer to layer, about 8
//   times in a Glorot-uniform head of width 64, and leave gamma(x) and
//   gamma(d), which share their scale, too few bits: 6x64 heads' colours were
//   off by 1.6e-7 rms, up to 9e-7 for rays of 40 units, with the fp32 units'
//   at 4.5e-8 and 6.7e-8.)  An output row (density, colour) is scaled alone,
//   its factor kept in the block.
// - activations, in the kernel: per sample and layer, by 2^(15 - e), where
//   2^e exceeds (largest row sum of |W|) (largest |input|) + largest |b|, so
//   that none exceeds 2^15.  What is lost then is below 2^-40 of that bound.
// Heads whose rows or biases do not fit this (fits()) take the fp32 units.
//
// What bounds it: with 8x128 heads the matrix pipe, 77 % busy at a
// power-limited 1.64 GHz beside 4.95 VALU instructions per MFMA (7 per output
// value); with 6x64 heads the VALU, 80 % active at 10.2 per MFMA.  One accumulator per tile (two, for the small and
// the large products, would cost the 8x128 heads their second wave per SIMD).
// 9.1 M samples of 8x128 heads: 18.2 ms on the fp32 units (142 TFLOP/s),
// 6.0 ms here; pixels off the float64 render by 6.9e-6 before, 6.8e-6 now
// (2.3e-7 and 2.0e-7 for opaque rays): the encoding's rounding, not the
// products', is what is left.
template <class C>
struct Split {
    typedef Packer<C> Pk;
    std::vector<float> w;
    std::vector<typename Pk::View> v;
    float factor[4];       // output rows: true = stored * factor
    int shift[C::D + 1];   // hidden layers (the colour hidden layer last): stored = scaled * 2^shift

    const float *base;
    const bool check;  // whether ok is wanted
    bool ok = true;

    // 2^e
    static float pow2(int e) { return ldexpf(1.0f, e); }
    // The exponent e of the power of two that takes a row's largest |weight| to
    // [1, 2) (kZeroRow for a row of zeros); e outside [-40, 40] does not fit
    // (powers of two cost no precision at any size: the limit keeps what the
    // scales and their inverses multiply inside float32's range).
    // Nor does a row most of whose sum can come from weights far below its
    // largest (read from a unit that is silent, say), which hold fewer bits
    // than float32: more than a quarter of its weights, but zeros, below 2^-12
    // of the largest (Glorot-uniform rows reach 2^-4).  One column 2^8 above
    // the others, which fits: colours of a float32 chain off by 2.4e-7, here
    // by 1.9e-7 (8x128, the worst of the three); 2^12 2.4e-7 and 2.9e-7, 2^16
    // 2.4e-7 and 8.6e-7, 2^20 2.4e-7 and 1.1e-5.
    static constexpr int kZeroRow = 1000;
    int row_exp(const float *p, int n)
    {
        // (magnitudes compare as integers, which the compiler vectorises)
        unsigned bits = 0;
        for (int i = 0; i < n; ++i) {
            unsigned u;
            memcpy(&u, p + i, 4);
            u &= 0x7FFFFFFFu;
            bits = u > bits ? u : bits;
        }
        float m;
        memcpy(&m, &bits, 4);
        if (m == 0.0f)
            return kZeroRow;
        if (bits >= 0x7F800000u) {  // the unit scales took a weight out of float32's range
            ok = false;
            return 0;
        }
        if (check) {
            unsigned least;
            const float floor = 0x1p-12f * m;
            memcpy(&least, &floor, 4);
            int small = 0, some = 0;
            for (int i = 0; i < n; ++i) {
                unsigned u;
                memcpy(&u, p + i, 4);
                small += (u & 0x7FFFFFFFu) - 1u < least - 1u;  // (zeros are none)
            }
            for (int i = 0; small > 0 && i < n; ++i)
                some += p[i] != 0.0f;
            if (4 * small > some)
                ok = false;
        }
        int x;
        (void)frexpf(m, &x);
        if (x < -39 || x > 41) {
            ok = false;
            return 0;
        }
        return 1 - x;
    }
    float *at(const float *p) { return w.data() + (p - base); }
    // columns [c0, c0 + col.size()) of a matrix times col, by rows
    static void scale_columns(float *p, int out, int in, int c0, const std::vector<float> &col)
    {
        for (int r = 0; r < out; ++r)
            for (size_t i = 0; i < col.size(); ++i)
                p[(size_t)r * in + c0 + i] *= col[i];
    }

    Split(const float *src, const std::vector<typename Pk::View> &views, bool check_fits = false)
        : w(src, views.back().b + views.back().out), v(views), base(src), check(check_fits)
    {
        std::vector<float> col;  // what the unit scales leave for the next layer's columns
        std::vector<int> exps, sorted;
        std::vector<float> mag;  // |biases|
        float typical = 1.0f;    // about the size of a layer's inputs
        // layer l's rows to their median's size; col: the inverse scales
        auto rows = [&](const typename Pk::View &L, int l) {
            col.assign(L.out, 1.0f);
            mag.resize(L.out);
            exps.resize(L.out);
            sorted.clear();
            for (int r = 0; r < L.out; ++r) {
                exps[r] = row_exp(at(L.W) + (size_t)r * L.in, L.in);
                if (exps[r] != kZeroRow)
                    sorted.push_back(exps[r]);
            }
            int median = 0;
            if (!sorted.empty()) {
                std::nth_element(sorted.begin(), sorted.begin() + sorted.size() / 2, sorted.end());
                median = sorted[sorted.size() / 2];
            }
            shift[l] = 14 + median;
            float sq = 0.0f;
            for (int r = 0; r < L.out; ++r) {
                float *p = at(L.W) + (size_t)r * L.in, *b = at(L.b) + r;
                const float f = exps[r] == kZeroRow ? 1.0f : pow2(exps[r] - median);
                *b *= f;
                mag[r] = fabsf(*b);
                float part[8] = {};
                for (int i = 0; i < L.in; ++i)
                    p[i] *= f;
                for (int i = 0; i + 8 <= L.in; i += 8)
                    for (int j = 0; j < 8; ++j)
                        part[j] += p[i + j] * p[i + j];
                for (float q : part)
                    sq += q;
                col[r] = 1.0f / f;
            }
            // one unit must not dwarf the others (all share a sample's scale):
            // no bias above 2^12 times what the layer's units reach.  An unread
            // one in every layer, worst colour's error over a float32 chain's:
            // 2^12 times 0.9 to 1.0, 2^14 0.8 to 1.2, 2^16 1.2 to 2.8.
            const float top = *std::max_element(mag.begin(), mag.end());
            std::nth_element(mag.begin(), mag.begin() + L.out / 2, mag.end());
            typical = 0.5f * sqrtf(sq / L.out) * typical + mag[L.out / 2];
            if (!(top <= 4096.0f * typical) || !(typical < 0x1p100f))
                ok = false;
        };
        for (int l = 0; l < C::D; ++l) {
            if (l > 0)
                scale_columns(at(v[l].W), v[l].out, v[l].in, l == C::SKIP ? C::P : 0, col);
            rows(v[l], l);
        }
        scale_columns(at(v[C::D].W), 1, v[C::D].in, 0, col);
        scale_columns(at(v[C::D + 1].W), v[C::D + 1].out, v[C::D + 1].in, 0, col);
        if (C::RH > 0) {
            rows(v[C::D + 1], C::D);
            scale_columns(at(v.back().W), 3, v.back().in, 0, col);
        }
        for (int j = 0; j < 4; ++j) {  // density, colour
            const typename Pk::View &L = j ? v.back() : v[C::D];
            float *p = at(L.W) + (size_t)(j ? j - 1 : 0) * L.in;
            const int x = row_exp(p, L.in);
            const float f = x == kZeroRow ? 1.0f : pow2(x);
            for (int i = 0; i < L.in; ++i)
                p[i] *= f;
            factor[j] = 1.0f / f;
        }
        for (typename Pk::View &L : v) {
            L.W = at(L.W);
            L.b = at(L.b);
        }
    }

    // whether a head's weights can take the split form
    static bool fits(const float *src)
    {
        std::vector<typename Pk::View> v;
        Pk::views(src, v);
        return Split(src, v, true).ok;
    }

    // x (|x| < 65504) to fp16, nearest even, and what is left of it.  In
    // integers and without a branch, so that the compiler vectorises it: a
    // host without a conversion instruction calls a routine for each.
    static inline unsigned short to_f16(float x, float &rest)
    {
        unsigned u;
        memcpy(&u, &x, 4);
        const unsigned sign = u & 0x80000000u, a = u ^ sign;
        // normal: drop 13 bits
        const unsigned h1 = (a + 0xFFFu + ((a >> 13) & 1u) - 0x38000000u) >> 13;
        const unsigned b1 = (h1 << 13) + 0x38000000u;
        // below 2^-14: multiples of 2^-24, the spacing of [0.5, 1)
        float f;
        memcpy(&f, &a, 4);
        const float r = f + 0.5f, q = r - 0.5f;
        unsigned h2, b2;
        memcpy(&h2, &r, 4);
        h2 -= 0x3F000000u;
        memcpy(&b2, &q, 4);
        const unsigned pick = (int)a >= 0x38800000 ? 0xFFFFFFFFu : 0u;
        const unsigned h = (h1 & pick) | (h2 & ~pick);
        const unsigned back = (b1 & pick) | (b2 & ~pick) | sign;
        float b;
        memcpy(&b, &back, 4);
        rest = x - b;
        return (unsigned short)(h | (sign >> 16));
    }

    void pack(unsigned char *stream, float *block)
    {
        for (int s = 0; s < C::NS; ++s) {
            const int T = C::st_tile(s), c0 = C::st_c0(s), nu = C::st_units_pad(s);
            const int kind = C::t_kind(T);
            const float up = pow2(kind == K_OUT ? 14 : shift[kind == K_HID ? C::t_layer(T) : C::D]);
            unsigned char *out = stream + (size_t)C::st_offset(s) * 1024;
            for (int u = 0; u < nu; u += 2) {  // units u (low halves), u + 1 (high halves)
                if (u >= C::st_units(s)) {
                    memset(out + (size_t)u * 1024, 0, 2048);
                    continue;
                }
                float x[64][8], y[512], rest[512];
                Pk::gather(v, T, 8 * (c0 + u / 2), x);
                memcpy(y, x, sizeof(y));
                unsigned short h[2][512];
                for (int i = 0; i < 512; ++i)
                    h[1][i] = to_f16(up * y[i], rest[i]);
                for (int i = 0; i < 512; ++i) {
                    float none;
                    h[0][i] = to_f16(rest[i], none);
                }
                memcpy(out + (size_t)u * 1024, h, sizeof(h));
            }
        }
        for (int i = 0; i < C::BLOCK_FLOATS; ++i)
            block[i] = 0.0f;
        for (int T = 0; T < C::NT; ++T)
            for (int g = 0; g < 2; ++g)
                for (int i = 0; i < 16; ++i)
                    block[(T * 2 + g) * 16 + i] = Pk::bval(v, T, c_row(g, i));
        for (int l = 0; l <= C::D; ++l) {
            if (l == C::D && C::RH == 0)
                continue;
            const typename Pk::View &L = v[l == C::D ? C::D + 1 : l];
            float n1 = 0.0f, b1 = 0.0f;
            for (int r = 0; r < L.out; ++r) {
                const float *p = L.W + (size_t)r * L.in;
                float part[8] = {}, sum = 0.0f;
                int i = 0;
                for (; i + 8 <= L.in; i += 8)
                    for (int j = 0; j < 8; ++j)
                        part[j] += fabsf(p[i + j]);
                for (; i < L.in; ++i)
                    sum += fabsf(p[i]);
                for (float q : part)
                    sum += q;
                n1 = sum > n1 ? sum : n1;
                b1 = fabsf(L.b[r]) > b1 ? fabsf(L.b[r]) : b1;
            }
            // (a little above, for the kernel's own rounding of the bound)
            block[C::SC_OFF + 4 * l] = 1.001f * n1;
            block[C::SC_OFF + 4 * l + 1] = 1.001f * b1;
            block[C::SC_OFF + 4 * l + 2] = pow2(-shift[l]);
        }
        for (int j = 0; j < 4; ++j)
            block[C::SC_OUT + j] = factor[j];
    }
};

// ---------------------------------------------------------------------------
// Device helpers
__device__ __forceinline__ f32x16 mfma(const f16x8 &a, const f16x8 &b, const f32x16 &c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma(const bf16x8 &a, const bf16x8 &b, const f32x16 &c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma(float a, float b, const f32x16 &c)
{
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// One wave copies 64 x 16 bytes global -> LDS: lane l reads base + voff and
// the data lands at lds_base + 16 l (base and lds_base are wave-uniform).
// Issued as asm so that the compiler does not track it: its completion is
// awaited explicitly with vmcnt (where it is counted), and the compiler's own
// LDS wait bookkeeping stays exact for the ds_reads around it (it would
// otherwise wait for every outstanding LDS read whenever one of these is in
// flight).  M0 carries the LDS address; nothing else in these kernels uses M0.
__device__ __forceinline__ void load_lds16(const unsigned char *base, unsigned voff,
                                           unsigned char *lds_base)
{
    const unsigned l = (unsigned)(unsigned long)(__attribute__((address_space(3))) unsigned char *)lds_base;
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(__builtin_amdgcn_readfirstlane(l)), "v"(voff), "s"(base)
                 : "memory");
}

// One wave gathers 64 dwords global -> LDS: lane l reads *p and the dword
// lands at lds_base + 4 l (lds_base wave-uniform).  Asm for the same reasons
// as load_lds16.
__device__ __forceinline__ void load_lds4(const void *p, unsigned char *lds_base)
{
    const unsigned l = (unsigned)(unsigned long)(__attribute__((address_space(3))) unsigned char *)lds_base;
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off"
                 :: "s"(__builtin_amdgcn_readfirstlane(l)), "v"(p)
                 : "memory");
}

// Round 8 floats to bf16 (nearest even) into one B chunk.
__device__ __forceinline__ bf16x8 to_bf16x8(const float *f)
{
    unsigned w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        w[j] = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{f[2 * j], f[2 * j + 1]}, bf16x2));
    return __builtin_bit_cast(bf16x8, w);
}

// ReLU then round to bf16: accumulator registers 8h .. 8h+7 -> one B chunk.
// A negative bf16 is a negative int16, so the ReLU is a packed int16 max with 0.
__device__ __forceinline__ bf16x8 relu_bf16(const f32x16 &a, int h)
{
    i16x2 p[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const bf16x2 v = __builtin_convertvector(f32x2{a[8 * h + 2 * j], a[8 * h + 2 * j + 1]}, bf16x2);
        p[j] = __builtin_elementwise_max(__builtin_bit_cast(i16x2, v), i16x2{0, 0});
    }
    return __builtin_bit_cast(bf16x8, p);
}

__device__ __forceinline__ float sigmoid(float x) { return __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }

// sin(pi 2^l p), cos(pi 2^l p): v_sin/v_cos take revolutions; 2^(l-1) p is
// exact and its fractional part is an exact reduction.
__device__ __forceinline__ void sincos_pi_pow2(float p, int l, float &s, float &c)
{
    const float u = __builtin_amdgcn_fractf(ldexpf(p, l - 1));
    s = __builtin_amdgcn_sinf(u);
    c = __builtin_amdgcn_cosf(u);
}

// This lane group's gamma(x) entries (see x_col): the lowest level of the
// group is evaluated directly, each higher level by the double-angle
// identities sin 2a = 2 sin a cos a, cos 2a = 1 - 2 sin^2 a.  The rounding
// error at most doubles per level (about 2^-19 after four doublings), far
// below the tolerance of either precision.
template <class C>
__device__ __forceinline__ void encode_x(const float x[3], int g, float *f)
{
    constexpr int LV = C::P0 / 3;  // levels per lane group
    f[0] = g ? x[2] : x[0];
    f[1] = g ? 0.0f : x[1];
    float s[3], c[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
        sincos_pi_pow2(x[k], g * LV, s[k], c[k]);
#pragma unroll
    for (int lv = 0; lv < LV; ++lv) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            f[2 + 2 * (3 * lv + k)] = s[k];
            f[3 + 2 * (3 * lv + k)] = c[k];
            if (lv + 1 < LV) {
                const float t = s[k] * c[k];
                c[k] = fmaf(-(s[k] + s[k]), s[k], 1.0f);
                s[k] = t + t;
            }
        }
    }
#pragma unroll
    for (int e = 2 + 2 * C::P0; e < C::EX; ++e)
        f[e] = 0.0f;
}

// Wait until at most N vector-memory operations of this wave are in flight.
// Written as asm with a memory clobber so that the compiler cannot move a
// memory access across it (the count relies on the issue order).
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_all() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }

// Workgroup barrier without the memory fences of __syncthreads(): the waits
// that make LDS data visible are explicit, so in-flight weight loads for
// later stages are not drained at every stage.  The memory clobber keeps the
// compiler from moving LDS accesses across it.
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }

// One k-chunk of B: a lane's E entries of a sample's layer input.
struct SplitChunk {
    f16x8 hi, lo;
};
template <class C>
using Chunk = std::conditional_t<C::SPLIT, SplitChunk, std::conditional_t<C::BF16, bf16x8, float>>;
// an entry of the stored encoding's table
template <class C>
using TabEntry = std::conditional_t<C::BF16, bf16x8, float>;

// Entries 2 p, 2 p + 1 of a split chunk: v_cvt_pk_f16_f32 for the high halves
// (nearest even), one fused multiply-add each for the remainders.
__device__ __forceinline__ void split_pair(SplitChunk &c, int p, float a, float b)
{
    const f16x2 h = __builtin_convertvector(f32x2{a, b}, f16x2);
    const f16x2 l = __builtin_convertvector(
        f32x2{fmaf((float)h[0], -1.0f, a), fmaf((float)h[1], -1.0f, b)}, f16x2);
    c.hi[2 * p] = h[0];
    c.hi[2 * p + 1] = h[1];
    c.lo[2 * p] = l[0];
    c.lo[2 * p + 1] = l[1];
}

// The value is computed by this point (and not moved past a wait that follows).
__device__ __forceinline__ void pin(bf16x8 &x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void pin(float &x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void pin(SplitChunk &x) { asm volatile("" : "+v"(x.hi), "+v"(x.lo)); }

// larger of x here and in the other lane group (lane ^ 32)
__device__ __forceinline__ float half_max(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// "no tile left" from the work queues
constexpr unsigned kNoTile = 0xFFFFFFFFu;

// SOFT: every head takes every sample (see MlpVariant::launch).  OFFS: each
// head's entries start at offsets[k] (not SOFT).
// gxtab (stored-encoding form only): gamma(x) rows of gx_encode_kernel.
template <class C, bool SOFT, bool OFFS>
__global__ __launch_bounds__(C::THREADS, C::WG_PER_CU) void mlp_kernel(
    const unsigned *__restrict__ bucket, const unsigned *__restrict__ totals,
    const unsigned *__restrict__ offsets, int num_sites, RenderGeometry geo,
    const float *__restrict__ tbuf, const void *__restrict__ dirbuf,
    const TabEntry<C> *__restrict__ gxtab,
    const unsigned char *__restrict__ streams, const float *__restrict__ blocks,
    float4 *__restrict__ sr, unsigned *__restrict__ queue, HeadMask empty)
{
    constexpr bool soft = SOFT;
    using CT = Chunk<C>;
    // one LDS unit per lane
    using AT = std::conditional_t<C::SPLIT, f16x8, std::conditional_t<C::BF16, bf16x8, f32x4>>;
    constexpr int NB = C::NB, NS = C::NS;
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    float *hb = reinterpret_cast<float *>(lds + C::HB_OFF);
    __shared__ unsigned s_off[kMaxSites + 1];   // bucket offset of each head
    __shared__ unsigned s_tile[kMaxSites + 1];  // first tile of each head
    __shared__ unsigned s_q[2];                 // tile indices handed out by the queues
    // queued tiles of each stretch: the first one and how many
    __shared__ unsigned s_qfirst[kMlpQueues], s_qcount[kMlpQueues];

    const int tid = threadIdx.x, lane = tid & 63;
    // wave-uniform by construction; saying so keeps LDS-destination pointers scalar
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, g = lane >> 5;

    // bucket offset and first tile of each head: exclusive scans of the
    // totals (or the given offsets, where the heads' entries need not be
    // adjacent) and of their tile counts, by wave 0 with 4 heads per lane
    if (tid < 64) {
        unsigned tot[4], nt[4], so = 0, st = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 4 * tid + j;
            tot[j] = k < num_sites ? totals[k] : 0u;
            // a 0-capacity head keeps its rows but gets no tiles
            nt[j] = k < num_sites && empty.test(k) ? 0u : tot[j] / C::TILE + (tot[j] % C::TILE != 0);
            so += tot[j];
            st += nt[j];
        }
        unsigned io = so, it = st;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned yo = __shfl_up(io, o), yt = __shfl_up(it, o);
            if (tid >= o) {
                io += yo;
                it += yt;
            }
        }
        unsigned off = io - so, tl = it - st;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 4 * tid + j;
            if (k < num_sites) {
                s_off[k] = OFFS ? offsets[k] : off;
                s_tile[k] = tl;
            }
            off += tot[j];
            tl += nt[j];
        }
        if (tid == 63) {
            s_off[num_sites] = off;
            s_tile[num_sites] = tl;
        }
    }
    __syncthreads();
    const unsigned total_tiles = s_tile[num_sites];

    // Tiles are handed out dynamically.  The tile range is cut into 8
    // contiguous stretches, one per XCD (each XCD has its own L2, and a
    // stretch covers few heads).  Workgroup b's first two tiles are fixed: of
    // stretch b % 8 (workgroups go to the XCDs in turn) the (b / 8)-th and, n
    // workgroups sharing the stretch, the (n + b / 8)-th, so that no
    // workgroup's start waits for the others' atomics.
    // queue[x] counts the tiles taken from stretch x after those; a workgroup
    // takes from its own XCD's stretch, then from the others.  The two
    // workgroups sharing a CU do not get equal shares of its matrix pipe, so
    // static ranges would leave one finishing long after the other.  The
    // counters are zero at launch (the bucket scan clears them).
    //
    // An atomic on these counters (one cache line, all XCDs) is served in
    // about 10 ns and the takes of a launch are served one after another, so
    // a stretch that has run out is found from the counters' values (8 loads
    // in flight at once), and a workgroup with nothing left asks no more.
    // With an atomic on every stretch for each failing take, 512 workgroups
    // spent about 90 us per launch on them, whatever its size: 32,768 samples
    // of 4x64 fp32 heads 117 -> 26 us, a level of 0.3 M samples of 8x128 heads
    // in the culled render 115 -> 38 us.  The stretches' first queued tile and
    // count are kept in LDS: the kernel has no scalar registers to spare (in
    // registers they cost the 6x64 heads 1 %).
    const unsigned xcc = (unsigned)__builtin_amdgcn_s_getreg(20 | (31 << 11)) & 7u;  // XCC_ID
    // take a tile of any stretch, from the own one on, or kNoTile: a failed
    // atomic means that the stretch's counter has passed its end, so the next
    // look skips it
    auto steal = [&]() -> unsigned {
        unsigned queued = 0;
#pragma unroll
        for (unsigned x = 0; x < (unsigned)kMlpQueues; ++x)
            queued |= s_qcount[x];
        if (queued == 0)
            return kNoTile;  // no tiles but the fixed ones
        for (;;) {
            unsigned cnt[kMlpQueues];
#pragma unroll
            for (unsigned x = 0; x < (unsigned)kMlpQueues; ++x)
                cnt[x] = __hip_atomic_load(queue + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            unsigned pick = kNoTile;
#pragma unroll
            for (unsigned x = 0; x < (unsigned)kMlpQueues; ++x)
                if (cnt[x] < s_qcount[x] && (pick == kNoTile || ((x - xcc) & 7u) < ((pick - xcc) & 7u)))
                    pick = x;
            if (pick == kNoTile)
                return kNoTile;
            const unsigned u = atomicAdd(queue + pick, 1u);
            if (u < s_qcount[pick])
                return s_qfirst[pick] + u;
        }
    };
    // the own stretch's queued tiles, 0 once it has run out, and their first
    // (thread 0's, in registers: a take that waited for an LDS read held up
    // its workgroup at every tile)
    unsigned own = 0, own_first = 0;
    // finish a take: the own stretch's atomic returned u (not asked when own == 0)
    auto take_rest = [&](unsigned u) -> unsigned {
        if (u < own)
            return own_first + u;
        own = 0;
        return steal();
    };
    auto q_base = [&](unsigned x) { return (unsigned)(((unsigned long long)total_tiles * x) / 8); };
    if (tid < kMlpQueues) {
        const unsigned x = (unsigned)tid, base = q_base(x), len = q_base(x + 1) - base;
        const unsigned share = (gridDim.x + 7u - x) >> 3, j = blockIdx.x >> 3;
        s_qfirst[x] = base + 2 * share;
        s_qcount[x] = len > 2 * share ? len - 2 * share : 0u;
        if (x == (blockIdx.x & 7u)) {
            s_q[0] = j < len ? base + j : kNoTile;
            s_q[1] = share + j < len ? base + share + j : kNoTile;
        }
    }
    __syncthreads();
    if (tid == 0) {
        own = s_qcount[xcc];
        own_first = s_qfirst[xcc];
        // stretches differ by a tile, so one may have more than its fixed ones
        // where another has none for this workgroup
        if (s_q[0] == kNoTile)
            s_q[0] = steal();
        else if (s_q[1] == kNoTile)
            s_q[1] = steal();
    }
    __syncthreads();
    unsigned tile = __builtin_amdgcn_readfirstlane(s_q[0]);
    unsigned next = __builtin_amdgcn_readfirstlane(s_q[1]);
    if (tile == kNoTile)
        return;

    // head owning a tile: the last h with s_tile[h] <= tile (empty heads
    // have s_tile[h] == s_tile[h + 1] and are skipped)
    auto head_of = [&](unsigned t) {
        int lo = 0, hi = num_sites;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (s_tile[mid] <= t)
                lo = mid;
            else
                hi = mid;
        }
        return __builtin_amdgcn_readfirstlane(lo);
    };
    // This wave's first unit of head h's stream.  The base is made opaque so
    // that each unit's address is formed from it with a compile-time offset,
    // instead of the compiler hoisting one wave-dependent offset per unit out
    // of the tile loop (more scalar registers than there are).
    auto stream_of = [&](int h) {
        const unsigned char *p = streams + ((size_t)h * C::STREAM_UNITS + wave) * 1024;
        asm volatile("" : "+s"(p));
        return p;
    };
    auto slot = [&](unsigned k) { return lds + (k & (C::NBUF - 1)) * C::SLOT_BYTES; };
    unsigned char *const lds_wave = lds + wave * 1024;
    // this wave's records of the next tile: [0] bucket id, [1] depth,
    // [2..4] origin, [5..7] direction, slot q = sample nb * 32 + n
    unsigned char *const pf_wave = lds + C::PF_OFF + wave * C::PF_WAVE;
    const unsigned *const pf = reinterpret_cast<const unsigned *>(pf_wave);
    // issue this wave's share of stage s's units into ring slot k
    auto issue = [&](auto sc, const unsigned char *src, unsigned k) {
        constexpr int s = decltype(sc)::value;
        constexpr int lpw = C::st_lpw(s), off = C::st_offset(s);
        unsigned char *dst = lds_wave + (k & (C::NBUF - 1)) * C::SLOT_BYTES;
#pragma unroll
        for (int q = 0; q < lpw; ++q)
            load_lds16(src + (size_t)(off + q * C::WAVES) * 1024, lane * 16, dst + q * C::WAVES * 1024);
        // keep the issue order the wait counts assume
        asm volatile("" ::: "memory");
    };

    // rows end at the sample count; with soft, each head's rows are all the
    // samples again (head k's at k S, read through bucket[row - k S])
    const unsigned row_cap = soft ? s_off[num_sites] : geo.num_samples;
    // end of head h's entries (with offsets, from memory: scalar loads)
    auto head_end = [&](int h) -> unsigned {
        if constexpr (OFFS)
            return offsets[h] + totals[h];
        else
            return s_off[h + 1];
    };
    // the two prefetch phases for the tile whose rows are [r0, r_end) and
    // whose bucket entries start at row base
    auto prefetch_ids = [&](unsigned r0, unsigned r_end, unsigned base) {
        // bucket ids (rows past the head's end read row 0's); offsets from r0,
        // so that a tile padded past 2^32 - 1 does not wrap into range
        const unsigned off = wave * (NB * 32) + lane % (NB * 32);
        const unsigned row = off < r_end - r0 ? r0 + off : r0;
        load_lds4(bucket + min(row - base, geo.num_samples - 1), pf_wave);
    };
    auto prefetch_rays = [&]() {
        if constexpr (C::GX)
            return;
        // depths, ray origins and directions of the ids in LDS
        const unsigned sn = min(pf[lane], geo.num_samples - 1);
        unsigned r = (unsigned)((double)sn * geo.inv_n);
        if (sn - r * geo.n >= geo.n)
            ++r;
        load_lds4(tbuf + sn, pf_wave + 256);
        const float *o = geo.rays_o + 3 * (size_t)r, *d = geo.rays_d + 3 * (size_t)r;
#pragma unroll
        for (int c = 0; c < 3; ++c)
            load_lds4(o + c, pf_wave + 256 * (2 + c));
#pragma unroll
        for (int c = 0; c < 3; ++c)
            load_lds4(d + c, pf_wave + 256 * (5 + c));
    };

    int head = head_of(tile);
    const unsigned char *stream = stream_of(head);
    // the first tile's head block and weights go out beside its sample ids, and
    // its rays' records once the ids are here
    auto load_block = [&](int h) {
        const unsigned char *src = reinterpret_cast<const unsigned char *>(blocks + (size_t)h * C::BLOCK_FLOATS);
        for (int u = wave; u < C::BLOCK_UNITS; u += C::WAVES)
            load_lds16(src + u * 1024, lane * 16, reinterpret_cast<unsigned char *>(hb) + u * 1024);
    };
    prefetch_ids(__builtin_amdgcn_readfirstlane(s_off[head] + (tile - s_tile[head]) * C::TILE),
                 __builtin_amdgcn_readfirstlane(min(head_end(head), row_cap)),
                 soft ? s_off[head] : 0u);
    load_block(head);
    unsigned ring = 0;  // ring slot of stage 0 of the current tile (mod NBUF)
    static_for<0, C::LA>([&](auto sc) { issue(sc, stream, ring + decltype(sc)::value); });
    wait_vmcnt<C::first_loads()>();  // the ids, issued before the weights
    prefetch_rays();
    wait_vmcnt<0>();
    int loaded_head = head;

    while (tile != kNoTile) {
        const bool has_next = next != kNoTile;
        const int nhead = has_next ? head_of(next) : head;
        const unsigned char *nstream = stream_of(nhead);
        const unsigned row0 = __builtin_amdgcn_readfirstlane(s_off[head] + (tile - s_tile[head]) * C::TILE);
        // rows never pass the sample count when the bucket counts are
        // consistent; the clamps keep every access in bounds regardless
        const unsigned row_end = __builtin_amdgcn_readfirstlane(min(head_end(head), row_cap));
        // rows of the tile whose records are prefetched (this one's if last)
        const unsigned pf_tile = has_next ? next : tile;
        const unsigned nrow0 = __builtin_amdgcn_readfirstlane(s_off[nhead] + (pf_tile - s_tile[nhead]) * C::TILE);
        const unsigned nrow_end = __builtin_amdgcn_readfirstlane(min(head_end(nhead), row_cap));

        wg_barrier();  // previous tile is done with the head block and the staging
        // this tile's records have landed (at most that many loads were issued
        // after them)
        wait_vmcnt<(C::loads_after_pb() < 63 ? C::loads_after_pb() : 63)>();
        // take the tile after next: the attempt on the own stretch is issued
        // here and completes under the prologue's full wait below, so it
        // never disturbs the counted waits of the weight stream
        // (the address goes through a vector register: for a uniform one the
        // compiler combines the lanes' atomics and waits for the result, and
        // for every load in flight, right here)
        unsigned q_first = 0, q_own = xcc;
        asm("" : "+v"(q_own));
        if (tid == 0 && has_next && own)
            q_first = atomicAdd(queue + q_own, 1u);
        if (head != loaded_head) {
            load_block(head);
            loaded_head = head;
        }

        // ---- gather the wave's samples and encode them ------------------------
        CT gx[NB][C::EXC];
        float xs[NB][3];  // sample positions, kept to re-encode for the skip layer
        unsigned sid[NB], ray[NB];
        bool valid[NB];
        // split: the layer inputs at hand are the true ones times 2^(15 - ex);
        // in_max bounds |gamma(x)|, top is the largest of a layer's scaled
        // outputs so far, mul and add the factors of the layer's accumulators
        // and biases (see Split)
        int ex = 0, ex_h = 0;
        float in_max = 1.0f, top = 0.0f, mul = 0.0f, add = 0.0f;
        // fp32 entries -> split chunks, scaled
        auto split_entries = [&](const float *f, auto &out) {
#pragma unroll
            for (int e = 0; e < C::EX; e += 2)
                split_pair(out[e / 8], e % 8 / 2, f[e] * add, f[e + 1] * add);
        };
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            valid[nb] = (wave * NB + nb) * 32 + n < row_end - row0;
            const unsigned q = nb * 32 + n;
            sid[nb] = min(pf[q], geo.num_samples - 1);
            unsigned r = (unsigned)((double)sid[nb] * geo.inv_n);
            if (sid[nb] - r * geo.n >= geo.n)
                ++r;
            ray[nb] = r;
            if constexpr (C::GX) {
                // this lane group's entries of the sample's row, as stored
                const TabEntry<C> *src = gxtab + ((size_t)sid[nb] * 2 + g) * (C::BF16 ? C::EXC : C::EX);
                if constexpr (C::SPLIT) {
                    float f[C::EX];
#pragma unroll
                    for (int e = 0; e < C::EX; e += 4) {
                        const f32x4 v = *reinterpret_cast<const f32x4 *>(src + e);
                        f[e] = v[0]; f[e + 1] = v[1]; f[e + 2] = v[2]; f[e + 3] = v[3];
                    }
                    in_max = half_max(fmaxf(1.0f, fmaxf(fabsf(f[0]), fabsf(f[1]))));
                    ex = __builtin_amdgcn_frexp_expf(in_max);
                    add = ldexpf(1.0f, 15 - ex);
                    split_entries(f, gx[nb]);
                } else if constexpr (C::BF16) {
#pragma unroll
                    for (int ch = 0; ch < C::EXC; ++ch)
                        gx[nb][ch] = src[ch];
                } else {
#pragma unroll
                    for (int e = 0; e < C::EX; e += 4) {
                        const f32x4 v = *reinterpret_cast<const f32x4 *>(src + e);
                        gx[nb][e] = v[0]; gx[nb][e + 1] = v[1]; gx[nb][e + 2] = v[2]; gx[nb][e + 3] = v[3];
                    }
                }
                continue;
            }
            const float t = __uint_as_float(pf[64 + q]);
            float x[3];
#pragma unroll
            for (int c = 0; c < 3; ++c)
                x[c] = fmaf(t, __uint_as_float(pf[64 * (5 + c) + q]), __uint_as_float(pf[64 * (2 + c) + q]));
            xs[nb][0] = x[0];
            xs[nb][1] = x[1];
            xs[nb][2] = x[2];
            float f[C::EX];
            encode_x<C>(x, g, f);
            if constexpr (C::SPLIT) {
                in_max = fmaxf(fmaxf(1.0f, fabsf(x[0])), fmaxf(fabsf(x[1]), fabsf(x[2])));
                ex = __builtin_amdgcn_frexp_expf(in_max);
                add = ldexpf(1.0f, 15 - ex);
                split_entries(f, gx[nb]);
            } else if constexpr (C::BF16) {
#pragma unroll
                for (int ch = 0; ch < C::EXC; ++ch)
                    gx[nb][ch] = to_bf16x8(f + 8 * ch);
            } else {
#pragma unroll
                for (int e = 0; e < C::EX; ++e)
                    gx[nb][e] = f[e];
            }
        }
        // encoded here, under the latency of what the wait below is for: left
        // to itself the compiler moves the encoding past the wait (6x64 heads,
        // 67 M samples: 3.27 -> 3.23 ms)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int ch = 0; ch < C::EXC; ++ch)
                pin(gx[nb][ch]);
        wait_all();  // the first LA weight stages and the head block have landed
        if (tid == 0)
            s_q[0] = has_next ? take_rest(q_first) : kNoTile;
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // the store above
        wg_barrier();

        CT hbuf[2][NB][C::EHC];                    // hidden outputs, by layer parity
        CT gbuf[NB][C::ERHC > 0 ? C::ERHC : 1];    // colour hidden outputs
        CT gxs[NB][C::EXC];                        // gamma(x) again, for the skip layer
        CT gd[NB][C::EDC];                         // gamma(d)
        float gdf[C::SPLIT ? C::ED : 1];           // the same as loaded
        f32x16 acc[2][NB];                         // by output-tile parity
        f32x16 bv;                                 // split: the finished tile's biases
        AT fr[C::PF];

        auto frag = [&](auto sc, int j) -> AT {
            constexpr int s = decltype(sc)::value;
            return *reinterpret_cast<const AT *>(slot(ring + s) + (j * 64 + lane) * 16);
        };
        auto load_bias = [&](auto tc) {
            // split: into bv, for tile T's epilogue; else as the accumulators of T
            constexpr int T = decltype(tc)::value;
            const float *b = hb + (T * 2 + g) * 16;
            f32x16 v;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4 q = *reinterpret_cast<const f32x4 *>(b + 4 * j);
                v[4 * j] = q[0]; v[4 * j + 1] = q[1]; v[4 * j + 2] = q[2]; v[4 * j + 3] = q[3];
            }
            if constexpr (C::SPLIT) {
                bv = v;
                return;
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                acc[T % 2][nb] = v;
        };
        // split: the scales of the outputs of layer l (C::D: the colour hidden
        // layer), whose inputs are complete
        auto next_scale = [&](auto lc) {
            constexpr int l = decltype(lc)::value;
            const f32x4 sc = *reinterpret_cast<const f32x4 *>(hb + C::SC_OFF + 4 * l);
            const float n1 = sc[0], b1 = sc[1];
            float m = l == 0 ? in_max : ldexpf(half_max(top), ex - 15);
            if constexpr (l > 0 && l == C::SKIP)
                m = fmaxf(m, in_max);
            if constexpr (l == C::D) {
                m = fmaxf(m, 1.0f);
                ex_h = ex;
            }
            float bound = fmaf(n1, m, b1);
            if constexpr (C::SKIP >= 0 && l + 1 == C::SKIP)
                bound = fmaxf(bound, in_max);  // the skip layer's gamma(x) takes the same scale
            if constexpr (l + 1 == C::D)
                bound = fmaxf(bound, 1.0f);  // and so does gamma(d)
            // Both factors stay finite: an infinite one times an accumulator or
            // bias of zero would be NaN.  (Below 2^-101 the layer's inputs are
            // all zero and its biases as small; the bound and mul saturate only
            // where every product is zero or rounds to it.)
            const int e = __builtin_amdgcn_frexp_expf(__builtin_amdgcn_fmed3f(bound, 0x1p-101f, 0x1p126f));
            mul = fminf(ldexpf(sc[2], ex - e), 0x1p126f);
            add = ldexpf(1.0f, 15 - e);
            ex = e;
            top = 0.0f;
        };
        // ReLU + conversion of output tile T into the next layer's input chunks,
        // in pieces so that it can be spread over the next tile's MFMAs:
        // bf16 piece p converts half p / NB of column block p % NB, fp32 piece
        // p a quarter of it
        auto epilogue_piece = [&](auto tc, auto pc) {
            constexpr int T = decltype(tc)::value, p = decltype(pc)::value;
            constexpr int kind = C::t_kind(T), mt = C::t_mt(T), par = C::t_layer(T) % 2;
            constexpr int nb = p % NB, h = p / NB;
            const f32x16 &a = acc[T % 2][nb];
            if constexpr (C::SPLIT) {
                // values 2 p and 2 p + 1: 7 VALU operations each
                if constexpr (mt == 0 && p == 0)
                    next_scale(ic<kind == K_HID ? C::t_layer(T) : C::D>{});
                const float v0 = fmaxf(fmaf(a[2 * p], mul, bv[2 * p] * add), 0.0f);
                const float v1 = fmaxf(fmaf(a[2 * p + 1], mul, bv[2 * p + 1] * add), 0.0f);
                top = fmaxf(top, fmaxf(v0, v1));
                if constexpr (kind == K_HID)
                    split_pair(hbuf[par][0][2 * mt + p / 4], p % 4, v0, v1);
                else
                    split_pair(gbuf[0][2 * mt + p / 4], p % 4, v0, v1);
            } else if constexpr (kind != K_OUT) {
                if constexpr (C::BF16) {
                    if constexpr (kind == K_HID)
                        hbuf[par][nb][2 * mt + h] = relu_bf16(a, h);
                    else
                        gbuf[nb][2 * mt + h] = relu_bf16(a, h);
                } else {
#pragma unroll
                    for (int i = 4 * h; i < 4 * h + 4; ++i) {
                        if constexpr (kind == K_HID)
                            hbuf[par][nb][16 * mt + i] = fmaxf(a[i], 0.0f);
                        else
                            gbuf[nb][16 * mt + i] = fmaxf(a[i], 0.0f);
                    }
                }
            }
        };
        constexpr int NPIECE = C::SPLIT ? 8 : C::BF16 ? 2 * NB : 4 * NB;

        // stage 0's bias and the first fragments of the window
        if constexpr (!C::SPLIT)
            load_bias(ic<0>{});
        static_for<0, (C::PF < C::FTOTAL ? C::PF : C::FTOTAL)>([&](auto fc) {
            constexpr int F = decltype(fc)::value;
            constexpr int fs = C::f_stage(F), fi = C::f_index(F);
            fr[F % C::PF] = frag(ic<fs>{}, fi);
        });

        // ---- stages ------------------------------------------------------------
        static_for<0, NS>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            constexpr int T = C::st_tile(s), kind = C::t_kind(T), layer = C::t_layer(T);
            constexpr int c0 = C::st_c0(s), NF = C::st_units(s);
            constexpr bool first = C::st_first(s);
            constexpr bool next_first = s + 1 < NS ? C::st_first(s + 1) : false;
            constexpr int next_tile = s + 1 < NS ? C::st_tile(s + 1) : 0;

            if constexpr (s % C::G == 0) {
                // group start: wait for the units the group needs, then one barrier
                constexpr int wa = C::vm_allowed(s, true), wb = C::vm_allowed(s, false);
                if constexpr (s > 0) {
                    if constexpr (wa >= 0 && wa == wb) {
                        wait_vmcnt<wa>();
                    } else if constexpr (wa >= 0) {
                        if (has_next)
                            wait_vmcnt<wa>();
                        else
                            wait_vmcnt<(wb >= 0 ? wb : 0)>();
                    }
                    wg_barrier();
                }
                // weights LA stages ahead (the next tile's past the end)
                static_for<s + C::LA, C::grp_end(s) + C::LA + 1>([&](auto xc) {
                    constexpr int x = decltype(xc)::value;
                    if constexpr (x < NS)
                        issue(ic<x>{}, stream, ring + x);
                    else if (has_next)
                        issue(ic<x - NS>{}, nstream, ring + x);
                });
            }
            if constexpr (s == C::S_GD) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const unsigned char *dp = reinterpret_cast<const unsigned char *>(dirbuf) +
                                              (size_t)ray[nb] * (kDirPad * (C::BF16 ? 2 : 4));
                    if constexpr (C::BF16) {
                        gd[nb][0] = *reinterpret_cast<const bf16x8 *>(dp + g * 16);
                        gd[nb][1] = *reinterpret_cast<const bf16x8 *>(dp + 32 + g * 16);
                    } else {
                        const f32x4 a0 = *reinterpret_cast<const f32x4 *>(dp + g * 32);
                        const f32x4 a1 = *reinterpret_cast<const f32x4 *>(dp + g * 32 + 16);
                        const f32x4 b0 = *reinterpret_cast<const f32x4 *>(dp + 64 + g * 32);
                        const f32x4 b1 = *reinterpret_cast<const f32x4 *>(dp + 64 + g * 32 + 16);
                        static_for<0, 4>([&](auto kc) {
                            constexpr int k = decltype(kc)::value;
                            if constexpr (C::SPLIT) {
                                gdf[k] = a0[k];
                                gdf[4 + k] = a1[k];
                                gdf[8 + k] = b0[k];
                                gdf[12 + k] = b1[k];
                            } else {
                                gd[nb][k] = a0[k];
                                gd[nb][4 + k] = a1[k];
                                gd[nb][8 + k] = b0[k];
                                gd[nb][12 + k] = b1[k];
                            }
                        });
                    }
                }
            }
            if constexpr (s == C::S_PA)
                prefetch_ids(nrow0, nrow_end, soft ? s_off[nhead] : 0u);
            if constexpr (s == C::S_PB)
                prefetch_rays();  // the group wait above covered the ids
            if constexpr (s + 1 == C::S_SKIP) {
                // gamma(x) again for the skip layer, overlapping this stage's MFMAs
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    float f[C::EX];
                    encode_x<C>(xs[nb], g, f);
                    if constexpr (C::SPLIT) {
                        split_entries(f, gxs[nb]);
                    } else if constexpr (C::BF16) {
#pragma unroll
                        for (int ch = 0; ch < C::EXC; ++ch)
                            gxs[nb][ch] = to_bf16x8(f + 8 * ch);
                    } else {
#pragma unroll
                        for (int e = 0; e < C::EX; ++e)
                            gxs[nb][e] = f[e];
                    }
                }
            }

            if constexpr (C::SPLIT) {
                if constexpr (s == C::S_GDUSE) {
#pragma unroll
                    for (int e = 0; e < C::ED; e += 2)
                        split_pair(gd[0][e / 8], e % 8 / 2, gdf[e] * add, gdf[e + 1] * add);
                }
            }

            // B operand chunk c of this tile's input for column block nb
            auto in_chunk = [&](auto cc, int nb) -> CT {
                constexpr int c = decltype(cc)::value;
                if constexpr (kind == K_HID) {
                    if constexpr (layer == 0) {
                        return gx[nb][c];
                    } else if constexpr (layer == C::SKIP) {
                        if constexpr (c < C::EXC) return gxs[nb][c];
                        else return hbuf[(layer - 1) % 2][nb][c - C::EXC];
                    } else {
                        return hbuf[(layer - 1) % 2][nb][c];
                    }
                } else if constexpr (kind == K_RGBH) {
                    if constexpr (c < C::EHC) return hbuf[(C::D - 1) % 2][nb][c];
                    else return gd[nb][c - C::EHC];
                } else {
                    if constexpr (c < C::EHC) return hbuf[(C::D - 1) % 2][nb][c];
                    else if constexpr (C::RH > 0) return gbuf[nb][c - C::EHC];
                    else return gd[nb][c - C::EHC];
                }
            };

            // Schedule of one step j: a piece of the previous tile's epilogue
            // (first stage of a tile), the read of the fragment PF
            // ahead (possibly the next stage's), the next tile's bias (late in
            // its last stage), then this step's MFMAs; sched_barrier keeps the
            // order, so LDS latency hides behind the MFMAs in between.
            constexpr bool EPI = first && T > 0;
            // (split: done before the step that reads the last chunk they fill:
            // the eighth unit of a tile at the earliest, two per chunk)
            constexpr int EMAX = C::SPLIT && NPIECE > 6 ? 6 : NPIECE;
            constexpr int ESTEPS = EPI ? (NF < EMAX ? NF : EMAX) : 0;
            static_assert(!C::SPLIT || !EPI || kind != K_HID || C::t_mt(T) > 0 ||
                              2 * (C::EHC - 2 + (layer == C::SKIP ? C::EXC : 0)) + 2 >= ESTEPS,
                          "a chunk is read before its epilogue");
            constexpr int JB0 = NF >= 2 ? NF - 2 : 0;
            constexpr int JB = next_first ? (JB0 > ESTEPS ? JB0 : ESTEPS) : NF;  // bias step
            constexpr int bias_tile = C::SPLIT ? T : next_tile;
            static_for<0, NF>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                constexpr int F = C::foff(s) + j;
                if constexpr (EPI && j < ESTEPS) {
                    // pieces p with p * ESTEPS / NPIECE == j
                    static_for<0, NPIECE>([&](auto pc) {
                        constexpr int pp = decltype(pc)::value;
                        if constexpr (pp * ESTEPS / NPIECE == j)
                            epilogue_piece(ic<T - 1>{}, pc);
                    });
                }
                const AT a = fr[F % C::PF];
                if constexpr (F + C::PF < C::FTOTAL) {
                    constexpr int fs = C::f_stage(F + C::PF), fi = C::f_index(F + C::PF);
                    fr[F % C::PF] = frag(ic<fs>{}, fi);
                }
                if constexpr (j == JB && next_first)
                    load_bias(ic<bias_tile>{});
                if constexpr (C::SPLIT) {
                    const SplitChunk x = in_chunk(ic<c0 + j / 2>{}, 0);
                    if constexpr (j % 2 == 0) {  // the weights' low halves
                        if constexpr (first && j == 0)
                            acc[T % 2][0] = mfma(a, x.hi, f32x16{});
                        else
                            acc[T % 2][0] = mfma(a, x.hi, acc[T % 2][0]);
                    } else {
                        acc[T % 2][0] = mfma(a, x.lo, acc[T % 2][0]);
                        acc[T % 2][0] = mfma(a, x.hi, acc[T % 2][0]);
                    }
                } else if constexpr (C::BF16) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        acc[T % 2][nb] = mfma(a, in_chunk(ic<c0 + j>{}, nb), acc[T % 2][nb]);
                } else {
                    static_for<0, 4>([&](auto qc) {
                        constexpr int q = decltype(qc)::value;
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            acc[T % 2][nb] = mfma(a[q], in_chunk(ic<c0 + 4 * j + q>{}, nb), acc[T % 2][nb]);
                    });
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (JB >= NF && next_first)
                load_bias(ic<bias_tile>{});
        });

        // ---- density and colour: rows 0..3 of the output tile, lanes g = 0 ----
        constexpr int TO = C::NT - 1;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            f32x16 a = acc[TO % 2][nb];
            if constexpr (C::SPLIT) {
                // the rows' biases and factors; the colours read the colour
                // hidden layer's outputs, where there is one
                const float sh = ldexpf(1.0f, (C::RH > 0 ? ex_h : ex) - 29);
                const float sc = ldexpf(1.0f, ex - 29);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    a[j] = fmaf(a[j] * (j ? sc : sh), hb[C::SC_OUT + j], hb[TO * 32 + j]);
            }
            if (g == 0 && valid[nb])
                sr[soft ? row0 + (wave * NB + nb) * 32 + n : sid[nb]] =
                    make_float4(fmaxf(a[0], 0.0f), sigmoid(a[1]), sigmoid(a[2]), sigmoid(a[3]));
        }
        ring += NS;
        head = nhead;
        stream = nstream;
        tile = next;
        next = __builtin_amdgcn_readfirstlane(s_q[0]);
    }
    // the last tile's prefetch re-read its own records: no LDS write may be
    // in flight when the workgroup's LDS is released
    wait_vmcnt<0>();
}

// gamma(x) of every sample into the table the stored-encoding form reads:
// row s holds lane group 0's EX entries, then lane group 1's, exactly as the
// tile prologue would hold them (the same encode_x and rounding), so both
// forms give the same outputs bit for bit.  One lane per (sample, group)
// encodes its entries into LDS; the block then writes its 256 rows out as
// one contiguous stretch, each store 16 contiguous bytes per lane.
template <class C>
__global__ __launch_bounds__(256) void gx_encode_kernel(RenderGeometry geo,
                                                        const float *__restrict__ tbuf,
                                                        TabEntry<C> *__restrict__ out)
{
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    constexpr int U = C::EX * (C::BF16 ? 2 : 4) / 16;  // 16-byte units per row
    __shared__ u32x4 stage[256 * U];
    const unsigned long long rows = 2ull * geo.num_samples;
    u32x4 *const dst_all = reinterpret_cast<u32x4 *>(out);
    for (unsigned long long base = (unsigned long long)blockIdx.x * 256; base < rows;
         base += (unsigned long long)gridDim.x * 256) {
        const unsigned long long i = base + threadIdx.x;
        if (i < rows) {
            const unsigned sn = (unsigned)(i >> 1);
            const int g = (int)(i & 1);
            unsigned r = (unsigned)((double)sn * geo.inv_n);
            if (sn - r * geo.n >= geo.n)
                ++r;
            const float t = tbuf[sn];
            float x[3];
#pragma unroll
            for (int c = 0; c < 3; ++c)
                x[c] = fmaf(t, geo.rays_d[3 * (size_t)r + c], geo.rays_o[3 * (size_t)r + c]);
            float f[C::EX];
            encode_x<C>(x, g, f);
            u32x4 *mine = stage + threadIdx.x * U;
            if constexpr (C::BF16) {
#pragma unroll
                for (int ch = 0; ch < C::EXC; ++ch)
                    mine[ch] = __builtin_bit_cast(u32x4, to_bf16x8(f + 8 * ch));
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    mine[u] = u32x4{__float_as_uint(f[4 * u]), __float_as_uint(f[4 * u + 1]),
                                    __float_as_uint(f[4 * u + 2]), __float_as_uint(f[4 * u + 3])};
            }
        }
        __syncthreads();
        const unsigned long long left = rows - base;
        const unsigned units = (unsigned)(left < 256 ? left : 256) * U;
        u32x4 *dst = dst_all + base * U;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const unsigned idx = k * 256 + threadIdx.x;
            if (idx < units)
                dst[idx] = stage[idx];
        }
        __syncthreads();  // the stage is rewritten by the next stretch
    }
}

template <class C>
hipError_t launch_gx_encode(const RenderGeometry &g, const float *t, void *gxtab, int cus,
                            hipStream_t s)
{
    if (g.num_samples == 0)
        return hipSuccess;
    const unsigned long long lanes = 2ull * g.num_samples;
    const unsigned long long want = (lanes + 255) / 256, cap = (unsigned long long)cus * 64;
    gx_encode_kernel<C><<<(unsigned)(want < cap ? want : cap), 256, 0, s>>>(
        g, t, reinterpret_cast<TabEntry<C> *>(gxtab));
    return hipGetLastError();
}

template <class C>
hipError_t launch_mlp(const unsigned *bucket, const unsigned *totals, const unsigned *offsets,
                      int num_sites,
                      const RenderGeometry &g, const float *t, const void *dirbuf,
                      const void *gxtab, const unsigned char *streams, const float *blocks,
                      float4 *sr, unsigned *queue, int cus, bool soft, const HeadMask &empty,
                      hipStream_t s)
{
    if (C::GX ? (soft || !gxtab) : gxtab != nullptr)
        return hipErrorInvalidValue;
    // raises the dynamic LDS limit where the runtime keeps one, once per
    // variant (thread-safe); a runtime without the limit may refuse the
    // call, and the launch below reports any real problem
    static const bool raised = [] {
        for (const void *k : {(const void *)mlp_kernel<C, false, false>,
                              (const void *)mlp_kernel<C, !C::GX, false>,
                              (const void *)mlp_kernel<C, false, true>})
            if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES) !=
                hipSuccess)
                (void)hipGetLastError();
        return true;
    }();
    (void)raised;
    const TabEntry<C> *gx = reinterpret_cast<const TabEntry<C> *>(gxtab);
    // as many persistent workgroups as fit, but no more than there can be
    // tiles (each head's last one may be partial)
    const unsigned long long heads_rows = soft ? num_sites : 1;
    const unsigned long long tiles =
        heads_rows * ((g.num_samples + (unsigned long long)C::TILE - 1) / C::TILE) + num_sites;
    const unsigned long long fit = (unsigned long long)cus * C::WG_PER_CU;
    const dim3 grid((unsigned)(tiles < fit ? tiles : fit)), block(C::THREADS);
    if constexpr (!C::GX) {
        if (soft) {
            mlp_kernel<C, true, false><<<grid, block, C::LDS_BYTES, s>>>(
                bucket, totals, nullptr, num_sites, g, t, dirbuf, gx, streams, blocks, sr, queue,
                empty);
            return hipGetLastError();
        }
    }
    if (offsets)
        mlp_kernel<C, false, true><<<grid, block, C::LDS_BYTES, s>>>(
            bucket, totals, offsets, num_sites, g, t, dirbuf, gx, streams, blocks, sr, queue, empty);
    else
        mlp_kernel<C, false, false><<<grid, block, C::LDS_BYTES, s>>>(
            bucket, totals, nullptr, num_sites, g, t, dirbuf, gx, streams, blocks, sr, queue, empty);
    return hipGetLastError();
}

// The stored-encoding form of an architecture without a skip layer.
template <class C>
using StoredForm = Cfg<C::PREC, C::W, C::D, C::SKIP, C::RH, C::LP, true>;

template <class C>
constexpr auto split_fits() -> bool (*)(const float *)
{
    if constexpr (C::SPLIT && !C::GX)
        return &Split<C>::fits;
    else
        return nullptr;
}

// plain: the form for weights that do not fit this one (split only)
template <class C>
const MlpVariant *variant(const MlpVariant *plain = nullptr)
{
    const MlpVariant *stored = nullptr;
    if constexpr (C::SKIP < 0 && !C::GX) {
        static_assert(StoredForm<C>::STREAM_UNITS == C::STREAM_UNITS &&
                          StoredForm<C>::BLOCK_FLOATS == C::BLOCK_FLOATS,
                      "both forms take the same packed weights");
        stored = variant<StoredForm<C>>();
    }
    static const MlpVariant v = {(size_t)C::STREAM_UNITS * 1024,
                                 (size_t)C::BLOCK_FLOATS * 4,
                                 C::TILE,
                                 &Packer<C>::pack,
                                 &launch_mlp<C>,
                                 stored,
                                 C::GX ? (size_t)2 * C::EX * (C::BF16 ? 2 : 4) : 0,
                                 C::LP,
                                 C::GX ? &launch_gx_encode<C> : nullptr,
                                 plain,
                                 split_fits<C>()};
    return &v;
}

}  // namespace derf
