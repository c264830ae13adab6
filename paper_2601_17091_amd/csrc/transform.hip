// ROCKET transform on CDNA4 (gfx950): the fp32 kernels (fused MFMA, Toeplitz,
// series-lane, MINIROCKET, plain direct) and the HIP-facing half of the C ABI.
// Most kernels of a univariate set run as split items instead (split.hip); the
// fp32 items here and in tiles.h run what those leave over, multivariate sets,
// and the sets that split items do not take or would not speed up.
//
// Fused kernel (one workgroup = a few series x one split of the work items
// of one code variant):
//   1. the series are staged HBM -> LDS with coalesced loads, with zero
//      margins on both sides that stand in for the zero padding (Sec. 2.1);
//   2. each wavefront takes work items from an LDS counter; an item holds 4
//      or 8 kernels of one (length, dilation, padding) bucket, which share
//      their outputs' positions and the series values under every tap;
//   3. outputs are computed in tiles of 64 consecutive positions, lane l
//      taking position 64k + l of tile k; for tap j the 64 lanes read 64
//      consecutive series values (index 64k - p + j*d + l): one
//      conflict-free ds_read_addtid_b32 per tile and tap, addressed by a
//      scalar register;
//   4. the dot products of a tile are an outer-product contraction over the
//      taps: v_mfma_f32_4x4x1_16b_f32 multiplies the 4 kernels' weights (A,
//      one kernel per block row) by the 64 lanes' series values (B), one tap
//      per instruction, accumulating onto the bias;
//   5. MAX is a per-lane running max reduced across the wavefront at the end
//      of a series; the positive count is a ballot of y > 0 popcounted on
//      the scalar unit; no dot product is written to memory (Sec. 3.2 keeps
//      only the two counters per pair as well);
//   6. PPV = count / O and MAX are written to F in the original kernel order.
//
// MINIROCKET kernel (the variant Sec. 5 names): the same staging and tiles;
// the dot products of its 42 kernels of one (dilation, padding) come from
// the 9 shared tap values and their sum on the vector unit, and each is
// compared with the item's biases of its kernel; PPV = count / O per
// (kernel, bias).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>

#include "rocket_internal.h"
#include "split_launch.h"
#include "tiles.h"

namespace {

constexpr int kBlock = 256;       // 4 wavefronts per workgroup
constexpr int kBigBlock = 1024;   // 16 wavefronts share one large staged row
constexpr int64_t kBigLds = 40 * 1024;  // staged rows above this use kBigBlock
constexpr int64_t kRowsLdsBudget = 30 * 1024;  // LDS for the series of one workgroup (5 per CU)

// Workgroup = (variant, row group, split); each workgroup stages its row
// group in LDS and runs the items of one variant over it.
template <int BLOCK, bool CLAMP, bool MPV, bool MC>
__global__ __launch_bounds__(BLOCK) void rocket_fused_kernel(FusedArgs a) {
    extern __shared__ __align__(16) float smem[];
    __shared__ int next_item;
    GroupWork w;
    if (!stage_group<BLOCK>(a, blockIdx.x, smem, &next_item, w)) return;
    const int lane = threadIdx.x & (rocket::kWave - 1);
    float *F0 = a.F + w.grow * (int64_t)a.nf * a.K;
    const float *rows0 = smem + a.halo_lo;
    const int beg = w.beg, cnt = w.cnt_items, nr = w.nrows;
    if constexpr (MC) {
        // multichannel plans hold 4-kernel items only (variants 0, 2, 4)
        switch (w.variant) {
            case 0: run_items<7, 1, CLAMP, MPV, MC>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
            case 2: run_items<9, 1, CLAMP, MPV, MC>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
            default: run_items<11, 1, CLAMP, MPV, MC>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        }
    } else {
        run_variant<CLAMP, MPV>(&next_item, w, a, rows0, F0, lane);
    }
}

// Toeplitz items (univariate long-series plans) in a kernel of their own,
// launched over the same row groups on a stream of the plan, beside the
// fused kernel (the two write disjoint features): in the fused kernel's code
// their extra tap counts raise the scalar-register pressure of every
// variant's loop.
template <int BLOCK, bool CLAMP, bool MPV>
__global__ __launch_bounds__(BLOCK) void rocket_toeplitz_kernel(FusedArgs a) {
    extern __shared__ __align__(16) float smem[];
    __shared__ int next_item;
    GroupWork w;
    if (!stage_group<BLOCK>(a, blockIdx.x, smem, &next_item, w)) return;
    const int lane = threadIdx.x & (rocket::kWave - 1);
    float *F0 = a.F + w.grow * (int64_t)a.nf * a.K;
    const float *rows0 = smem + a.halo_lo;
    const int beg = w.beg, cnt = w.cnt_items, nr = w.nrows;
    switch (w.variant) {
        case 12: run_toep_items<7, 1, CLAMP, MPV>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 13: run_toep_items<7, 2, CLAMP, MPV>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 14: run_toep_items<9, 1, CLAMP, MPV>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 15: run_toep_items<9, 2, CLAMP, MPV>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 16: run_toep_items<11, 1, CLAMP, MPV>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        default: run_toep_items<11, 2, CLAMP, MPV>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
    }
}

// ---------------------------------------------------------------------------
// Series-lane layout (short univariate series).  The 64 lanes of a
// wavefront take 64 series, and LDS holds the workgroup's 64 series
// position-major: the values of all 64 series at one position are 64
// consecutive floats, so a tap's read is again one ds_read_addtid_b32 per
// position.  One MFMA then computes one output position for 4 kernels x 64
// series, and a block runs NT consecutive positions.  Every lane keeps the
// count, the max (and the MPV sum) of its own series, so no cross-lane
// reduction is needed: for short series the per-series reductions and
// writes of the position-tiled layout cost more than the dot products.
// ---------------------------------------------------------------------------

constexpr int kSeriesLanes = rocket::kWave;              // series per workgroup
constexpr int kSeriesMargin = rocket::kMaxTilesPerBlock;  // zero positions on each side
using rocket::kSeriesMaxL;                                 // longest series it takes
constexpr int64_t kSeriesMinRows = 4096;  // fewer series per call: too few workgroups, use tiles

// Stages the group's series: position m of series r at
// smem[(m + kSeriesMargin) * 64 + r], with zeros in the margins and in the
// lanes past the group's last series.  Consecutive threads write
// consecutive LDS words (no bank conflicts); their global reads are a
// series apart and hit the same cache lines across the loop.
template <int BLOCK>
__device__ __forceinline__ bool stage_series(const FusedArgs &a, float *smem, int *next_item,
                                             GroupWork &w) {
    if (!group_work(a, blockIdx.x, w)) return false;
    const int total = (a.L + 2 * kSeriesMargin) * kSeriesLanes;
    const float *x = a.X + w.grow * (int64_t)a.L;
    for (int e = threadIdx.x; e < total; e += BLOCK) {
        const int r = e & (kSeriesLanes - 1);
        const int m = e / kSeriesLanes - kSeriesMargin;
        smem[e] = (r < w.nrows && m >= 0 && m < a.L) ? x[(int64_t)r * a.L + m] : 0.0f;
    }
    set_check_bounds(smem, total, a.S, a.S + a.s_floats);
    if (threadIdx.x == 0) *next_item = 0;
    __syncthreads();
    return true;
}

// Series-lane reads.  pos0 is the LDS byte address of position 0 (its 64
// series); the position of the block's first output under tap j is clamped
// into [-kSeriesMargin, L] on the scalar unit, as for ClampedTiles: a block
// whose positions all lie outside the series reads zeros from a margin, a
// block that overlaps it is not moved.
struct SeriesTiles {
    uint32_t pos0;
    int b0;  // position under tap 0 of the block's first output
    int d;
    int L;
    __device__ __forceinline__ uint32_t m0(int j) const {
        const int b = min(max(b0 + j * d, -kSeriesMargin), L);
        return pos0 + 256u * (uint32_t)b;
    }
};

template <>
struct PipelinedReads<SeriesTiles> {
    static constexpr bool value = true;
};

// Per-lane (per-series) accumulators of one work item.
template <int G>
struct SeriesAcc {
    v4f mx[G];
    uint32_t cnt[G][4];
    v4f ps[G];
};

// [y > 0] as 0 or 1.  For a float that is not a NaN the bits read as a
// signed integer are positive exactly when y > 0 (+0 reads 0; -0 and the
// negative values read negative), so med3(bits, 0, 1) is the indicator.
__device__ __forceinline__ uint32_t positive01(float y) {
    uint32_t r;
    asm("v_med3_i32 %0, %1, 0, 1" : "=v"(r) : "v"(y));
    return r;
}

// Fold NT positions of finished dot products into the lanes' accumulators:
// the counts add the indicators two at a time, MAX folds pairs with v_max3.
template <int G, int NT, bool MPV>
__device__ __forceinline__ void series_reduce(const v4f (&acc)[NT][G], SeriesAcc<G> &sa) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            uint32_t c = sa.cnt[g][v];
#pragma unroll
            for (int u = 0; u < NT; u += 2) {
                if (u + 1 < NT)
                    c += positive01(acc[u][g][v]) + positive01(acc[u + 1][g][v]);
                else
                    c += positive01(acc[u][g][v]);
            }
            sa.cnt[g][v] = c;
        }
    if (MPV) {
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int v = 0; v < 4; ++v) sa.ps[g][v] += fmaxf(acc[u][g][v], 0.0f);
    }
#pragma unroll
    for (int u = 0; u + 1 < NT; u += 2)
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                sa.mx[g][v] = fmaxf(fmaxf(sa.mx[g][v], acc[u][g][v]), acc[u + 1][g][v]);
    if (NT % 2 == 1) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int v = 0; v < 4; ++v) sa.mx[g][v] = fmaxf(sa.mx[g][v], acc[NT - 1][g][v]);
    }
}

// NT consecutive output positions of one item for the 64 series.
template <int ELL, int G, int NT, bool MPV>
__device__ __forceinline__ void series_block(const SeriesTiles &src, const float (&wa)[G][ELL],
                                             const v4f (&binit)[G], SeriesAcc<G> &sa) {
    v4f acc[NT][G];
    tile_mfma<ELL, G, NT, false, true>(src, wa, binit, binit, acc);
    __builtin_amdgcn_sched_barrier(0);
    // raised wave priority while the fold runs, as in the fused kernel
    __builtin_amdgcn_s_setprio(1);
    series_reduce<G, NT, MPV>(acc, sa);
    __builtin_amdgcn_s_setprio(0);
}

// The last positions of an item, nv (1..N) of them: a code copy per count.
template <int ELL, int G, int N, bool MPV>
struct SeriesTail {
    __device__ __forceinline__ static void run(int nv, const SeriesTiles &src, const float (&wa)[G][ELL],
                                               const v4f (&binit)[G], SeriesAcc<G> &sa) {
        if (nv == N)
            series_block<ELL, G, N, MPV>(src, wa, binit, sa);
        else
            SeriesTail<ELL, G, N - 1, MPV>::run(nv, src, wa, binit, sa);
    }
};
template <int ELL, int G, bool MPV>
struct SeriesTail<ELL, G, 0, MPV> {
    __device__ __forceinline__ static void run(int, const SeriesTiles &, const float (&)[G][ELL],
                                               const v4f (&)[G], SeriesAcc<G> &) {}
};

// One work item over the group's 64 series: all O positions in blocks of
// NT, then each lane writes the features of its series for the item's
// kernels.
template <int ELL, int G, bool MPV>
__device__ __forceinline__ void run_series_item(const ItemDesc &it, uint32_t pos0, int nrows,
                                                const FusedArgs &a, int64_t srow0, int lane) {
    constexpr int NT = rocket::kTilesPerBlock[G - 1];
    float wa[G][ELL];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int j = 0; j < ELL; ++j) wa[g][j] = a.wpk[it.w_off + (g * ELL + j) * 4 + (lane & 3)];
    // C operand of the first tap: the bias of block row v (kernel slot v),
    // the same on every lane (series)
    v4f binit[G];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float b = as_const(a.bias)[it.k_off + 4 * g + v];
            float bv;
            asm volatile("v_mov_b32 %0, %1" : "=v"(bv) : "s"(b));
            binit[g][v] = bv;
        }
    SeriesAcc<G> sa;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        v2f lo, hi;
        asm volatile("v_mov_b64 %0, %2\n\tv_mov_b64 %1, %2" : "=v"(lo), "=v"(hi) : "s"(kNegInfPair));
        sa.mx[g] = v4f{lo[0], lo[1], hi[0], hi[1]};
        if (MPV) sa.ps[g] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int v = 0; v < 4; ++v) sa.cnt[g][v] = 0;
    }
    const int nfull = it.O / NT;          // full blocks
    const int nv = it.O - nfull * NT;     // positions in the last block, 0..NT-1
    for (int blk = 0; blk < nfull; ++blk)
        series_block<ELL, G, NT, MPV>(SeriesTiles{pos0, blk * NT - it.p, it.d, a.L}, wa, binit, sa);
    if (nv > 0)
        SeriesTail<ELL, G, NT - 1, MPV>::run(nv, SeriesTiles{pos0, nfull * NT - it.p, it.d, a.L}, wa,
                                             binit, sa);
    // features into the slot-ordered buffer: slot s of series r (of this
    // launch) at S[(s * s_rows + r) * nf], so the 64 lanes of a slot write
    // 64 * nf consecutive floats
    if (lane < nrows) {
        float *Srow = a.S + (srow0 + lane) * (int64_t)a.nf;
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int slot = it.k_off + 4 * g + v;
                if (as_const(a.kid)[slot] >= 0)
                    write_features<MPV>(sa.cnt[g][v], sa.mx[g][v], sa.ps[g][v], 0, it.inv_O,
                                        Srow + slot * a.s_rows * (int64_t)a.nf);
            }
    }
}

template <int ELL, int G, bool MPV>
__device__ __forceinline__ void run_series_items(int *next_item, int beg, int cnt_items, uint32_t pos0,
                                                 int nrows, const FusedArgs &a, int64_t srow0, int lane) {
    while (true) {
        int idx = 0;
        if (lane == 0) idx = atomicAdd(next_item, 1);
        idx = __builtin_amdgcn_readfirstlane(__shfl(idx, 0, 64));
        if (idx >= cnt_items) break;
        const ItemDesc it = load_item(as_const(a.items) + as_const(a.order)[beg + idx]);
        run_series_item<ELL, G, MPV>(it, pos0, nrows, a, srow0, lane);
    }
}

// Workgroup = (variant, group of 64 series, split), mapped as for the fused
// kernel; each wavefront takes items from the workgroup's counter.
template <bool MPV>
__global__ __launch_bounds__(kBlock) void rocket_series_kernel(FusedArgs a) {
    extern __shared__ float smem[];
    __shared__ int next_item;
    GroupWork w;
    if (!stage_series<kBlock>(a, smem, &next_item, w)) return;
    const int lane = threadIdx.x & (rocket::kWave - 1);
    const int64_t F0 = w.grow - a.row0;  // first series of the group in S
    uint32_t pos0 = lds_addr(smem + kSeriesMargin * kSeriesLanes);
    asm volatile("" : "+s"(pos0));  // computed once (not again in every block)
    const int beg = w.beg, cnt = w.cnt_items, nr = w.nrows;
    switch (w.variant) {
        case 0: run_series_items<7, 1, MPV>(&next_item, beg, cnt, pos0, nr, a, F0, lane); break;
        case 1: run_series_items<7, 2, MPV>(&next_item, beg, cnt, pos0, nr, a, F0, lane); break;
        case 2: run_series_items<9, 1, MPV>(&next_item, beg, cnt, pos0, nr, a, F0, lane); break;
        case 3: run_series_items<9, 2, MPV>(&next_item, beg, cnt, pos0, nr, a, F0, lane); break;
        case 4: run_series_items<11, 1, MPV>(&next_item, beg, cnt, pos0, nr, a, F0, lane); break;
        default: run_series_items<11, 2, MPV>(&next_item, beg, cnt, pos0, nr, a, F0, lane); break;
    }
}

// F rows in the original kernel order from the slot-ordered buffer: a tile
// is 64 kernels x 64 series, and the workgroups (4 wavefronts) stride over
// the tiles; wavefront w takes the tile's series 16w .. 16w + 15.  Lane l
// moves kernel k0 + l: it reads the 16 series' features from its slot column
// as whole 16-byte vectors (16 * NF consecutive floats, 128 or 192 bytes),
// then writes them series by series, so each series' 64 kernels go out as
// 64 * NF consecutive floats.  Columns hold s_rows series, a multiple of 64,
// so the reads of a partial last tile stay inside the column; only the
// writes check the series count.  No LDS: the kernel runs beside the series
// kernel, which fills the LDS.
template <int NF>
__global__ __launch_bounds__(kBlock) void rocket_slot_permute_kernel(const float *S, int64_t s_rows,
                                                                     const int32_t *slot_of, int32_t K,
                                                                     int64_t n_rows, float *F,
                                                                     int32_t n_slots) {
    constexpr int kRows = 16;
    constexpr int kVec = kRows * NF / 4;  // float4 per lane
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t k_tiles = ((int64_t)K + 63) / 64;
    const int64_t n_tiles = k_tiles * ((n_rows + 63) / 64);
    for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        const int64_t k = (t % k_tiles) * 64 + lane;
        const int64_t r0 = (t / k_tiles) * 64 + wave * kRows;
        if (k >= K || r0 >= n_rows) continue;
#if ROCKET_CHECKED
        // the slot column this lane reads must be one of the buffer's n_slots
        if (slot_of[k] < 0 || slot_of[k] >= n_slots) {
            check_failed(kCheckSlotRead);
            continue;
        }
#endif
        const float4 *src = reinterpret_cast<const float4 *>(S + ((int64_t)slot_of[k] * s_rows + r0) * NF);
        float v[kVec * 4];
#pragma unroll
        for (int i = 0; i < kVec; ++i) {
            const float4 q = src[i];
            v[4 * i] = q.x;
            v[4 * i + 1] = q.y;
            v[4 * i + 2] = q.z;
            v[4 * i + 3] = q.w;
        }
        const int nr = (int)min<int64_t>(kRows, n_rows - r0);
        float *b = F + r0 * (int64_t)K * NF + k * NF;
#pragma unroll
        for (int rr = 0; rr < kRows; ++rr) {
            if (rr < nr) {
                if constexpr (NF == 2) {
                    *reinterpret_cast<float2 *>(b) = make_float2(v[2 * rr], v[2 * rr + 1]);
                } else {
#pragma unroll
                    for (int f = 0; f < NF; ++f) b[f] = v[NF * rr + f];
                }
            }
            b += (int64_t)K * NF;
        }
    }
}

// ---------------------------------------------------------------------------
// MINIROCKET (Dempster, Schmidt and Webb, KDD 2021; Sec. 5 names it as a
// variant the same principle carries over to).  Its 84 kernels have 9 taps,
// weight 2 on a choice of 3 taps (a, b, c) and -1 on the other six, so a dot
// product is
//     C = 3 (x_a + x_b + x_c) - (x_0 + ... + x_8).
// An item holds the 42 kernels of one parity at one (dilation, padding)
// (the pair (dilation i, kernel k) is padded when i + k is even) and NQ (4 or
// 8) of each kernel's biases.  For each tile of 64 output positions the nine
// tap values are read from LDS once and their sum S is formed once, by a
// pairwise tree, for all 42 kernels; a kernel then costs two adds and one
// fma on the vector unit,
//     C = fma(3, (x_a + x_b) + x_c, -S),
// instead of nine multiply-adds.  Rounding: |C - C_exact| <= 3 gamma_2
// sum_chosen |x| + gamma_4 sum_all |x| + u |C|, about 12u sum_chosen |x| +
// 5u sum_others |x| (u = 2^-24), inside the gamma_9 sum_j |w_j x_j| = 18u
// sum_chosen |x| + 9u sum_others |x| that bounds any 9-term fp32 evaluation
// (additions of subnormals are exact, so no underflow term is added).
// Feature (kernel, bias b) counts C > b: one compare per tile, a ballot
// popcounted on the scalar unit.
// ---------------------------------------------------------------------------

using rocket::kMrKappa;
constexpr int kMrTiles = 4;  // tiles per block (the last 0..3 tiles run one at a time)

// Tap `which` (0, 1, 2 for a < b < c) of MINIROCKET kernel k: the k-th choice
// of 3 of the 9 taps in lexicographic order.
constexpr int mr_tap(int k, int which) {
    int n = 0;
    for (int a = 0; a < 9; ++a)
        for (int b = a + 1; b < 9; ++b)
            for (int c = b + 1; c < 9; ++c) {
                if (n == k) return which == 0 ? a : (which == 1 ? b : c);
                ++n;
            }
    return -1;
}
static_assert(mr_tap(0, 0) == 0 && mr_tap(0, 2) == 2 && mr_tap(83, 0) == 6 && mr_tap(83, 2) == 8,
              "84 lexicographic choices of 3 of 9 taps");

// Count registers of an item: feature g = kappa * NQ + q (kernel 2 kappa +
// parity, bias q) lives in lane g % 64 of register g / 64.
template <int NQ>
constexpr int mr_regs() { return (kMrKappa * NQ + 63) / 64; }

// The count of feature G over the block's NT tiles (a ballot popcount per
// tile, summed on the scalar unit) into its lane of the block's partial
// counts.
template <int G, int NT>
__device__ __forceinline__ void mr_count(const float (&C)[NT], float b, uint32_t &part) {
    uint32_t s = 0;
#pragma unroll
    for (int u = 0; u < NT; ++u) s += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(C[u] > b));
    asm volatile("v_writelane_b32 %0, %1, %2" : "+v"(part) : "s"(s), "i"(G % 64));
}

template <int KAPPA, int Q, int NQ, int NT, int R>
struct MrCounts {
    __device__ __forceinline__ static void run(const float (&C)[NT], const float (&b)[NQ], uint32_t (&part)[R]) {
        constexpr int G = KAPPA * NQ + Q;
        mr_count<G, NT>(C, b[Q], part[G / 64]);
        MrCounts<KAPPA, Q + 1, NQ, NT, R>::run(C, b, part);
    }
};
template <int KAPPA, int NQ, int NT, int R>
struct MrCounts<KAPPA, NQ, NQ, NT, R> {
    __device__ __forceinline__ static void run(const float (&)[NT], const float (&)[NQ], uint32_t (&)[R]) {}
};

// Kernels 2 KAPPA + PAR, KAPPA = KAPPA0 .. 41, over the block's NT tiles: the
// dot products from the shared tap values and sum, then the compares.  Each
// kernel's section is closed by a scheduling barrier and loads the next
// kernel's biases (scalar loads) while its own compares run, so only two
// kernels' biases are live in scalar registers.
template <int PAR, int KAPPA, int NQ, int NT, int R>
struct MrKernels {
    __device__ __forceinline__ static void run(const float (&x)[9][NT], const float (&S)[NT],
                                               ConstPtr<float> thr, const float (&b)[NQ], uint32_t (&part)[R]) {
        constexpr int k = 2 * KAPPA + PAR;
        constexpr int ta = mr_tap(k, 0), tb = mr_tap(k, 1), tc = mr_tap(k, 2);
        float bn[NQ];
        if constexpr (KAPPA + 1 < kMrKappa) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) bn[q] = thr[(KAPPA + 1) * NQ + q];
        }
        float C[NT];
#pragma unroll
        for (int u = 0; u < NT; ++u) C[u] = fmaf(3.0f, (x[ta][u] + x[tb][u]) + x[tc][u], -S[u]);
        MrCounts<KAPPA, 0, NQ, NT, R>::run(C, b, part);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (KAPPA + 1 < kMrKappa) MrKernels<PAR, KAPPA + 1, NQ, NT, R>::run(x, S, thr, bn, part);
    }
};

// One block of NT tiles of an item over one series.  rem = outputs of the
// block's last tile (64 unless it is the series' last tile): lanes past it
// get S = +inf, so C = -inf there and no bias is exceeded.
template <int PAR, int NQ, int NT, typename Src>
__device__ __forceinline__ void mr_block(const Src &src, ConstPtr<float> thr, int rem, int lane,
                                         uint32_t (&part)[mr_regs<NQ>()], uint32_t (&cnt)[mr_regs<NQ>()]) {
    float x[9][NT];
#pragma unroll
    for (int j = 0; j < 9; ++j) lds_tiles<NT>(src.m0(j), x[j]);
    float S[NT];
#pragma unroll
    for (int u = 0; u < NT; ++u)
        S[u] = (((x[0][u] + x[1][u]) + (x[2][u] + x[3][u])) + ((x[4][u] + x[5][u]) + (x[6][u] + x[7][u]))) +
               x[8][u];
    S[NT - 1] = lane < rem ? S[NT - 1] : INFINITY;
    // a fresh copy of the bias pointer per block keeps the bias loads inside
    // the block (hoisted out of the row loop, 42 * NQ biases would not fit
    // the scalar registers)
    uint64_t tp = (uint64_t)(__UINTPTR_TYPE__)thr;
    asm volatile("" : "+s"(tp));
    const ConstPtr<float> tb = (ConstPtr<float>)(__UINTPTR_TYPE__)tp;
    float b0[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) b0[q] = tb[q];
    MrKernels<PAR, 0, NQ, NT, mr_regs<NQ>()>::run(x, S, tb, b0, part);
#pragma unroll
    for (int r = 0; r < mr_regs<NQ>(); ++r) cnt[r] += part[r];
}

template <int PAR, int NQ, bool CLAMP>
__device__ __forceinline__ void run_mr_item(const ItemDesc &it, const float *rows0, int nrows,
                                            const FusedArgs &a, float *F0, int lane) {
    constexpr int NT = kMrTiles;
    constexpr int R = mr_regs<NQ>();
    const ConstPtr<float> thr = as_const(a.thr) + it.t_off;
    // the feature each lane writes from each count register (-1: none)
    int64_t fidx[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int g = 64 * r + lane;
        const int kappa = g / NQ, q = g % NQ;
        fidx[r] = (kappa < kMrKappa && it.k_off + q < it.n_ch)
                      ? (int64_t)it.w_off + (int64_t)(2 * kappa + PAR) * it.n_ch + it.k_off + q
                      : -1;
    }
    uint32_t part[R], cnt[R];
#pragma unroll
    for (int r = 0; r < R; ++r) part[r] = cnt[r] = 0;  // lanes past 42 * NQ stay 0
    const int rem = it.O - (it.n_tiles - 1) * kTile;  // outputs in the last tile, 1..64
    const int nfull = it.n_tiles / NT;                // blocks of NT tiles
    const int ntail = it.n_tiles - nfull * NT;        // then 0..NT-1 single tiles
    const int row_pitch = a.row_stride;
    const int64_t f_stride = (int64_t)a.nf * a.K;
    for (int r = 0; r < nrows; ++r) {
        const uint32_t row = lds_addr(rows0 + r * row_pitch);
        for (int blk = 0; blk < nfull; ++blk) {
            const int b0 = blk * (NT * kTile) - it.p;
            const int rb = (ntail == 0 && blk == nfull - 1) ? rem : kTile;
            if constexpr (CLAMP)
                mr_block<PAR, NQ, NT>(ClampedTiles{row, b0, it.d, a.L}, thr, rb, lane, part, cnt);
            else
                mr_block<PAR, NQ, NT>(PaddedTiles{row + 4u * (uint32_t)b0, it.d}, thr, rb, lane, part, cnt);
        }
        for (int t = 0; t < ntail; ++t) {
            const int b0 = (nfull * NT + t) * kTile - it.p;
            const int rb = t == ntail - 1 ? rem : kTile;
            if constexpr (CLAMP)
                mr_block<PAR, NQ, 1>(ClampedTiles{row, b0, it.d, a.L}, thr, rb, lane, part, cnt);
            else
                mr_block<PAR, NQ, 1>(PaddedTiles{row + 4u * (uint32_t)b0, it.d}, thr, rb, lane, part, cnt);
        }
        // PPV = count / O, correctly rounded as in write_features
#pragma unroll
        for (int rr = 0; rr < R; ++rr) {
            if (fidx[rr] >= 0 && store_checked(F0 + r * f_stride + fidx[rr], 1))
                F0[r * f_stride + fidx[rr]] = (float)((double)cnt[rr] * it.inv_O);
            cnt[rr] = 0;
        }
    }
}

template <int PAR, int NQ, bool CLAMP>
__device__ __forceinline__ void run_mr_items(int *next_item, int beg, int cnt_items, const float *rows0,
                                             int nrows, const FusedArgs &a, float *F0, int lane) {
    while (true) {
        int idx = 0;
        if (lane == 0) idx = atomicAdd(next_item, 1);
        idx = __builtin_amdgcn_readfirstlane(__shfl(idx, 0, 64));
        if (idx >= cnt_items) break;
        const ItemDesc it = load_item(as_const(a.items) + as_const(a.order)[beg + idx]);
        run_mr_item<PAR, NQ, CLAMP>(it, rows0, nrows, a, F0, lane);
    }
}

// MINIROCKET workgroup: as rocket_fused_kernel; variant = mr_variant(parity, NQ).
template <int BLOCK, bool CLAMP>
__global__ __launch_bounds__(BLOCK) void rocket_minirocket_kernel(FusedArgs a) {
    extern __shared__ __align__(16) float smem[];
    __shared__ int next_item;
    GroupWork w;
    if (!stage_group<BLOCK>(a, blockIdx.x, smem, &next_item, w)) return;
    const int lane = threadIdx.x & (rocket::kWave - 1);
    float *F0 = a.F + w.grow * (int64_t)a.nf * a.K;
    const float *rows0 = smem + a.halo_lo;
    const int beg = w.beg, cnt = w.cnt_items, nr = w.nrows;
    switch (w.variant) {
        case 0: run_mr_items<0, rocket::kMrQSmall, CLAMP>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 1: run_mr_items<0, rocket::kMrQLarge, CLAMP>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 2: run_mr_items<0, rocket::kMrQTiny, CLAMP>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 3: run_mr_items<1, rocket::kMrQSmall, CLAMP>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 4: run_mr_items<1, rocket::kMrQLarge, CLAMP>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        default: run_mr_items<1, rocket::kMrQTiny, CLAMP>(&next_item, beg, cnt, rows0, nr, a, F0, lane); break;
    }
}

// Plain kernel: one wavefront per (series, kernel) pair, lanes over output
// positions, taps read straight from global memory with the zero padding
// applied by bounds checks.
__global__ __launch_bounds__(kBlock) void rocket_direct_kernel(
    const float *__restrict__ X, int64_t row0, int32_t L, int32_t K, int32_t k0,
    const int32_t *__restrict__ len, const int32_t *__restrict__ dil,
    const int32_t *__restrict__ pad, const float *__restrict__ bias,
    const float *__restrict__ w, int32_t max_len, int32_t nf, int32_t C,
    const int32_t *__restrict__ ccount, const int32_t *__restrict__ cindex,
    float *__restrict__ F) {
    const int64_t row = row0 + blockIdx.x;
    const int k = k0 + (int)blockIdx.y * (kBlock / 64) + (int)(threadIdx.x >> 6);
    if (k >= K) return;
    const int lane = threadIdx.x & 63;
    const int ell = len[k], d = dil[k], p = pad[k];
    const int nch = C > 1 ? ccount[k] : 1;
    const float b = bias[k];
    const int64_t O = (int64_t)L + 2 * (int64_t)p - (int64_t)(ell - 1) * d;
    float mx = -INFINITY, ps = 0.0f;
    uint32_t c = 0;
    for (int64_t t = lane; t < O; t += 64) {
        float acc = b;
        for (int s = 0; s < nch; ++s) {
            const int ch = C > 1 ? cindex[(int64_t)k * C + s] : 0;
            const float *x = X + (row * C + ch) * (int64_t)L;
            const float *wk = w + ((int64_t)k * C + s) * max_len;
            for (int j = 0; j < ell; ++j) {
                const int64_t m = t - p + (int64_t)j * d;
                const float xv = (m >= 0 && m < L) ? x[m] : 0.0f;
                acc = fmaf(wk[j], xv, acc);
            }
        }
        c += acc > 0.0f ? 1u : 0u;
        ps += acc > 0.0f ? acc : 0.0f;
        mx = fmaxf(mx, acc);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        mx = fmaxf(mx, __shfl_xor(mx, off, 64));
        c += __shfl_xor(c, off, 64);
        ps += __shfl_xor(ps, off, 64);
    }
    if (lane == 0) {
        float *f = F + row * (int64_t)nf * K + (int64_t)nf * k;
        f[0] = (float)c / (float)O;
        f[1] = mx;
        if (nf == 3) f[2] = c > 0 ? ps / (float)c : 0.0f;
    }
}

template <typename T>
hipError_t upload(const std::vector<T> &h, T **d) {
    *d = nullptr;
    if (h.empty()) return hipSuccess;
    hipError_t e = hipMalloc((void **)d, h.size() * sizeof(T));
    if (e != hipSuccess) return e;
    return hipMemcpy(*d, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice);
}

template <typename T>
hipError_t upload_raw(const T *h, size_t n, T **d) {
    *d = nullptr;
    hipError_t e = hipMalloc((void **)d, n * sizeof(T));
    if (e != hipSuccess) return e;
    return hipMemcpy(*d, h, n * sizeof(T), hipMemcpyHostToDevice);
}

}  // namespace

// The fused kernel's instances: bit 0 the 1024-thread block (rows above
// kBigLds), bit 1 clamped indices, bit 2 MPV, bit 3 multichannel items.
constexpr int kFusedInstances = 16;
static const void *fused_fn(int sel) {
    static const void *const fns[kFusedInstances] = {
        (const void *)rocket_fused_kernel<kBlock, false, false, false>,
        (const void *)rocket_fused_kernel<kBigBlock, false, false, false>,
        (const void *)rocket_fused_kernel<kBlock, true, false, false>,
        (const void *)rocket_fused_kernel<kBigBlock, true, false, false>,
        (const void *)rocket_fused_kernel<kBlock, false, true, false>,
        (const void *)rocket_fused_kernel<kBigBlock, false, true, false>,
        (const void *)rocket_fused_kernel<kBlock, true, true, false>,
        (const void *)rocket_fused_kernel<kBigBlock, true, true, false>,
        (const void *)rocket_fused_kernel<kBlock, false, false, true>,
        (const void *)rocket_fused_kernel<kBigBlock, false, false, true>,
        (const void *)rocket_fused_kernel<kBlock, true, false, true>,
        (const void *)rocket_fused_kernel<kBigBlock, true, false, true>,
        (const void *)rocket_fused_kernel<kBlock, false, true, true>,
        (const void *)rocket_fused_kernel<kBigBlock, false, true, true>,
        (const void *)rocket_fused_kernel<kBlock, true, true, true>,
        (const void *)rocket_fused_kernel<kBigBlock, true, true, true>,
    };
    return fns[sel];
}

// The MINIROCKET kernel's instances: bit 0 the 1024-thread block, bit 1
// clamped indices.
constexpr int kMrInstances = 4;
static const void *mr_fn(int sel) {
    static const void *const fns[kMrInstances] = {
        (const void *)rocket_minirocket_kernel<kBlock, false>,
        (const void *)rocket_minirocket_kernel<kBigBlock, false>,
        (const void *)rocket_minirocket_kernel<kBlock, true>,
        (const void *)rocket_minirocket_kernel<kBigBlock, true>,
    };
    return fns[sel];
}

// The Toeplitz kernel's instances: bit 0 the 1024-thread block, bit 1
// clamped indices, bit 2 MPV.
constexpr int kToepInstances = 8;
static const void *toep_fn(int sel) {
    static const void *const fns[kToepInstances] = {
        (const void *)rocket_toeplitz_kernel<kBlock, false, false>,
        (const void *)rocket_toeplitz_kernel<kBigBlock, false, false>,
        (const void *)rocket_toeplitz_kernel<kBlock, true, false>,
        (const void *)rocket_toeplitz_kernel<kBigBlock, true, false>,
        (const void *)rocket_toeplitz_kernel<kBlock, false, true>,
        (const void *)rocket_toeplitz_kernel<kBigBlock, false, true>,
        (const void *)rocket_toeplitz_kernel<kBlock, true, true>,
        (const void *)rocket_toeplitz_kernel<kBigBlock, true, true>,
    };
    return fns[sel];
}

constexpr int64_t kNoAllocHalfBytes = (int64_t)32 << 20;  // half of the static scratch (below)

static const void *series_fn(bool mpv) {
    return mpv ? (const void *)rocket_series_kernel<true> : (const void *)rocket_series_kernel<false>;
}

struct rocket_plan {
    rocket::HostPlan host;  // fp32 items: of every kernel, or of those split items leave over
    // split items (univariate plans, see split_eligible and split_pays): most
    // kernels run there, for series longer than kSeriesMaxL the rest in fp32
    // items of the same launch or one beside it (Toeplitz items in their own)
    rocket::SplitDevice *split = nullptr;
    bool split_rest = false;  // some kernels are left to fp32 items
    int64_t fp32_slots = 0;   // slots of the fp32 items of the whole set (0: few)
    // code variants in launch order: by total item cost, largest first
    int32_t variant_order[rocket::kNumVariants] = {};
    int device = 0;
    int n_cu = 0;
    bool direct = false;
    bool clamp = false;      // rows staged with kClampMargin zeros on each side, tap offsets clamped
    bool series = false;     // series-lane layout available (short univariate series)
    int64_t series_min_rows = 0;  // calls with at least this many series use it
    int64_t series_lds = 0;       // its LDS per workgroup
    int32_t *d_slot_of = nullptr;  // series-lane layout: the slot of each kernel
    // series-lane layout: the slot-ordered feature buffer (two halves),
    // allocated on first use and grown as needed; transforms on different
    // streams take turns on it (each waits for the previous user's event).
    // The permutation of one chunk runs on the plan's own stream while the
    // next chunk's series kernel runs on the caller's.
    mutable std::mutex scratch_mu;
    mutable float *d_scratch = nullptr;
    mutable size_t scratch_bytes = 0;
    mutable hipEvent_t scratch_done = nullptr;
    hipStream_t aux = nullptr;
    // the series kernels of odd chunks run on this stream (even ones on the
    // caller's), so that consecutive chunks overlap instead of draining the
    // GPU between them
    hipStream_t odd = nullptr;
    hipEvent_t half_full[2] = {nullptr, nullptr};
    hipEvent_t half_free[2] = {nullptr, nullptr};
    hipEvent_t aux_done = nullptr;
    hipEvent_t call_start = nullptr;  // the caller's stream at the start of a call (odd waits on it)
    hipEvent_t odd_done = nullptr;    // the odd stream's last chunk of a call
    // plans with Toeplitz items: their kernel runs on this stream, beside the
    // fused kernel on the caller's (they write disjoint features)
    mutable std::mutex side_mu;
    hipStream_t side = nullptr;
    hipEvent_t side_start = nullptr;
    hipEvent_t side_done = nullptr;
    bool mpv = false;        // third feature per kernel: mean of positive values
    bool minirocket = false; // MINIROCKET plan: F [n, n_features], PPV only
    int64_t f_cols = 0;      // columns of F
    int32_t C = 1;           // channels per series
    int32_t halo_lo = 0;     // staged layout actually used (floats)
    int32_t row_stride = 0;
    int32_t tail_pad = 0;
    int rows_per_block = 1;  // series staged per workgroup
    int64_t lds_bytes = 0;   // per workgroup: the rows plus the tail pad
    ItemDesc *d_items = nullptr;
    float *d_wpk = nullptr;
    float *d_bias = nullptr;
    int32_t *d_kid = nullptr;
    int32_t *d_order = nullptr;
    int32_t *d_split_begin = nullptr;
    float *d_thr = nullptr;
    // the kernel set as given, for the direct kernel
    int32_t max_len = 0;
    int32_t *d_cc = nullptr;  // channel counts and indices (multichannel sets)
    int32_t *d_ci = nullptr;
    int32_t *d_len = nullptr;
    int32_t *d_dil = nullptr;
    int32_t *d_pad = nullptr;
    float *d_b = nullptr;
    float *d_w = nullptr;
};

static void plan_free_device(rocket_plan *p) {
    rocket::split_destroy(p->split);
    if (p->scratch_done) (void)hipEventDestroy(p->scratch_done);
    for (hipEvent_t ev : {p->half_full[0], p->half_full[1], p->half_free[0], p->half_free[1], p->aux_done,
                          p->call_start, p->odd_done, p->side_start, p->side_done})
        if (ev) (void)hipEventDestroy(ev);
    if (p->aux) (void)hipStreamDestroy(p->aux);
    if (p->odd) (void)hipStreamDestroy(p->odd);
    if (p->side) (void)hipStreamDestroy(p->side);
    void *ptrs[] = {p->d_scratch, p->d_slot_of, p->d_items, p->d_wpk, p->d_bias, p->d_kid, p->d_order,
                    p->d_split_begin, p->d_thr, p->d_len, p->d_dil, p->d_pad, p->d_b,
                    p->d_w, p->d_cc, p->d_ci};
    for (void *q : ptrs)
        if (q) (void)hipFree(q);
}

static rocket_status map_hip(hipError_t e) {
    if (e == hipSuccess) return ROCKET_OK;
    if (e == hipErrorOutOfMemory) return ROCKET_ERR_OOM;
    return ROCKET_ERR_HIP;
}

// Staged layout: rows with zero margins wide enough for every tap of every
// real output if that fits one workgroup's LDS (and clamped is not asked
// for), else rows with kClampMargin zeros on each side and clamped tap
// offsets.  Rows per workgroup: as many as fit the LDS budget (at least
// one).  Returns false when neither layout fits; *lds is the workgroup's LDS.
static bool choose_layout(rocket_plan *p, bool clamped, const hipDeviceProp_t &prop, int64_t *lds) {
    const int64_t limit = (int64_t)prop.sharedMemPerBlock;
    const int64_t L = p->host.L;
    auto layout = [&](int64_t stride, int64_t pad, int *rows) {
        const int64_t row_bytes = stride * p->C * (int64_t)sizeof(float);  // every channel
        const int64_t pad_bytes = pad * (int64_t)sizeof(float);
        *rows = (int)std::max<int64_t>(
            1, std::min<int64_t>(kMaxRowsPerBlock, (kRowsLdsBudget - pad_bytes) / row_bytes));
        return *rows * row_bytes + pad_bytes;
    };
    if (!clamped && p->host.row_stride > 0 &&
        (*lds = layout(p->host.row_stride, p->host.tail_pad, &p->rows_per_block)) <= limit) {
        p->halo_lo = p->host.halo_lo;
        p->row_stride = p->host.row_stride;
        p->tail_pad = p->host.tail_pad;
        return true;
    }
    // the clamped layout: each row keeps both of its margins; zeros after
    // the last row cover the reads of lanes past O
    if ((*lds = layout(L + 2 * rocket::kClampMargin, rocket::kTile, &p->rows_per_block)) <= limit) {
        p->clamp = true;
        p->halo_lo = rocket::kClampMargin;
        p->row_stride = (int32_t)(L + 2 * rocket::kClampMargin);
        p->tail_pad = rocket::kTile;
        return true;
    }
    return false;
}

// Dynamic-LDS limits already granted to the workgroup kernels, per device.
// The limit is a process-wide attribute of each kernel function, shared by
// every plan, so it is only ever raised: a later plan with a smaller
// footprint above 64 KB must not lower it below what an earlier plan
// launches with.
constexpr int kMaxDevices = 64;
static std::mutex g_lds_attr_mu;
static int g_lds_attr[kMaxDevices][kFusedInstances + kMrInstances + kToepInstances];

static hipError_t allow_lds(int device, int64_t lds) {
    if (lds <= 64 * 1024) return hipSuccess;
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_lds_attr_mu);
    hipError_t e = hipSuccess;
    for (int sel = 0; sel < kFusedInstances + kMrInstances + kToepInstances && e == hipSuccess; ++sel) {
        int &granted = g_lds_attr[device][sel];
        if (granted >= lds) continue;
        const void *fn = sel < kFusedInstances ? fused_fn(sel)
                         : sel < kFusedInstances + kMrInstances ? mr_fn(sel - kFusedInstances)
                                                                 : toep_fn(sel - kFusedInstances - kMrInstances);
        e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e == hipSuccess) granted = (int)lds;
    }
    return e;
}

// Upload the work tables and allow the kernels the workgroup's LDS.
static hipError_t upload_tables(rocket_plan *p, int64_t lds) {
    // A launch runs the workgroups of one variant after another (per XCD),
    // and a variant's workgroups each hold 1/nsplit of its items, so the
    // variants with the most work per workgroup go first: the launch then
    // ends on the short workgroups of the light variants rather than on a
    // late start of the longest ones.
    const int nv = p->host.n_variants;
    int64_t cost[rocket::kNumVariants] = {};
    for (const ItemDesc &it : p->host.items) cost[it.variant] += it.cost;
    for (int v = 0; v < nv; ++v) p->variant_order[v] = v;
    std::stable_sort(p->variant_order, p->variant_order + nv,
                     [&](int32_t x, int32_t y) { return cost[x] > cost[y]; });
    hipError_t e = upload(p->host.items, &p->d_items);
    if (e == hipSuccess) e = upload(p->host.wpk, &p->d_wpk);
    if (e == hipSuccess) e = upload(p->host.bias, &p->d_bias);
    if (e == hipSuccess) e = upload(p->host.kid, &p->d_kid);
    if (e == hipSuccess) e = upload(p->host.order, &p->d_order);
    if (e == hipSuccess) e = upload(p->host.split_begin, &p->d_split_begin);
    if (e == hipSuccess) e = upload(p->host.thr, &p->d_thr);
    if (e == hipSuccess) e = allow_lds(p->device, lds);
    return e;
}

static void item_facts(const rocket::HostPlan &host, bool series, bool minirocket, rocket_plan_facts *f) {
    f->n_items = (int64_t)host.items.size();
    f->n_buckets = host.n_buckets;
    // series-lane plans: one MFMA serves 64 series, so a series costs
    // (positions x taps x groups) / 64 of them
    f->mfma_per_row = series ? (host.series_mfma_64 + kSeriesLanes / 2) / kSeriesLanes : host.mfma_per_row;
    f->valu_fma_per_row = host.valu_fma_per_row;
    f->toeplitz_items = 0;
    if (!minirocket)
        for (const rocket::ItemDesc &it : host.items)
            if (it.variant >= rocket::kToepVariant0) ++f->toeplitz_items;
}

// The fp32 plan of the kernels `rest` of a set (their ids as in the set), beside
// split items of split_cost issue cycles (8.7 to an fp32 MFMA) per series.
static rocket_status build_rest_plan(const rocket_kernels *k, int32_t L, const std::vector<int32_t> &rest,
                                     double split_cost, rocket::HostPlan *out) {
    try {
        rocket::HostPlan P;
        P.L = L;
        P.n_kernels = k->n_kernels;
        if (!rest.empty()) {
            std::vector<int32_t> len, dil, pad;
            std::vector<float> bias, w;
            for (int32_t i : rest) {
                len.push_back(k->length[i]);
                dil.push_back(k->dilation[i]);
                pad.push_back(k->padding[i]);
                bias.push_back(k->bias[i]);
                w.insert(w.end(), k->weights + (int64_t)i * k->max_len, k->weights + (int64_t)(i + 1) * k->max_len);
            }
            rocket_kernels sub = *k;
            sub.n_kernels = (int32_t)rest.size();
            sub.length = len.data();
            sub.dilation = dil.data();
            sub.padding = pad.data();
            sub.bias = bias.data();
            sub.weights = w.data();
            const rocket_status st = rocket::build_host_plan(&sub, L, &P, split_cost / 8.7);
            if (st != ROCKET_OK) return st;
            for (int32_t &q : P.kid)
                if (q >= 0) q = rest[(size_t)q];
            P.n_kernels = k->n_kernels;
        }
        *out = std::move(P);
        return ROCKET_OK;
    } catch (const std::bad_alloc &) {
        return ROCKET_ERR_OOM;
    }
}

extern "C" rocket_status rocket_plan_create_ex(const rocket_kernels *k, int32_t L, uint32_t flags,
                                               rocket_plan **out) {
    if (!out) return ROCKET_ERR_INVALID_ARG;
    *out = nullptr;
    if ((flags & ~(ROCKET_PLAN_DIRECT | ROCKET_PLAN_CLAMPED | ROCKET_PLAN_MPV | ROCKET_PLAN_TILED |
                   ROCKET_PLAN_SERIES)) ||
        ((flags & ROCKET_PLAN_DIRECT) && (flags & (ROCKET_PLAN_CLAMPED | ROCKET_PLAN_TILED))) ||
        ((flags & ROCKET_PLAN_SERIES) &&
         (flags & (ROCKET_PLAN_DIRECT | ROCKET_PLAN_CLAMPED | ROCKET_PLAN_TILED))))
        return ROCKET_ERR_INVALID_ARG;
    rocket_status st = rocket::validate_kernels(k, L);
    if (st != ROCKET_OK) return st;
    rocket_plan *p = new (std::nothrow) rocket_plan();
    if (!p) return ROCKET_ERR_OOM;
    hipError_t e = hipGetDevice(&p->device);
    hipDeviceProp_t prop;
    if (e == hipSuccess) e = hipGetDeviceProperties(&prop, p->device);
    if (e != hipSuccess) {
        delete p;
        return ROCKET_ERR_HIP;
    }
    p->n_cu = prop.multiProcessorCount;
    p->mpv = (flags & ROCKET_PLAN_MPV) != 0;
    p->C = k->n_channels < 1 ? 1 : k->n_channels;
    p->f_cols = (int64_t)(p->mpv ? 3 : 2) * k->n_kernels;
    int64_t lds = 0;
    p->direct = (flags & ROCKET_PLAN_DIRECT) != 0;
    // short univariate series: the series-lane layout for calls with many
    // series (ROCKET_PLAN_SERIES: for every call), unless a position-tiled
    // layout is asked for; the position-tiled layout serves the rest
    const bool want_series = (flags & ROCKET_PLAN_SERIES) != 0;
    if (!p->direct && !(flags & (ROCKET_PLAN_CLAMPED | ROCKET_PLAN_TILED)) && p->C == 1 && L <= kSeriesMaxL) {
        p->series_lds = (int64_t)(L + 2 * kSeriesMargin) * kSeriesLanes * (int64_t)sizeof(float);
        if (p->series_lds <= (int64_t)prop.sharedMemPerBlock) {
            p->series = true;
            p->series_min_rows = want_series ? 0 : kSeriesMinRows;
        }
    }
    if (want_series && !p->series) {
        delete p;
        return ROCKET_ERR_INVALID_ARG;
    }
    if (!p->direct && rocket::split_eligible(k, L) && rocket::split_fits(L, (int64_t)prop.sharedMemPerBlock)) {
        rocket::SplitPlan sp;
        rocket::HostPlan rest;
        st = rocket::build_split_plan(k, L, &sp);
        const bool pays = st == ROCKET_OK && rocket::split_pays(sp, p->mpv);
        if (pays) st = build_rest_plan(k, L, sp.rest, sp.cost, &rest);
        if (st == ROCKET_OK && pays) {
            // split items clamp their reads themselves: the flag chooses the
            // layout of the fp32 items beside them
            p->clamp = (flags & ROCKET_PLAN_CLAMPED) != 0;
            p->split_rest = !rest.items.empty();
            p->host = std::move(rest);
            // short series: the slots of the whole set's fp32 items bound what
            // the no-allocation entry takes (at most four per kernel: small
            // sets always fit)
            if (L <= kSeriesMaxL && 4 * p->f_cols * (int64_t)sizeof(float) * kSeriesLanes > kNoAllocHalfBytes) {
                rocket::HostPlan whole;
                st = rocket::build_host_plan(k, L, &whole);
                p->fp32_slots = (int64_t)whole.kid.size();
            }
            if (st == ROCKET_OK)
                e = rocket::split_create(std::move(sp), p->device, p->n_cu, (int64_t)prop.sharedMemPerBlock, p->mpv,
                                     &p->split);
        }
        if (st != ROCKET_OK || e != hipSuccess) {
            plan_free_device(p);
            delete p;
            return st != ROCKET_OK ? st : map_hip(e);
        }
    }
    if (!p->split && (st = rocket::build_host_plan(k, L, &p->host)) != ROCKET_OK) {
        plan_free_device(p);
        delete p;
        return st;
    }
    const bool fp32_items = !p->split || p->split_rest;
    if (!p->direct && fp32_items && !choose_layout(p, (flags & ROCKET_PLAN_CLAMPED) != 0, prop, &lds))
        p->direct = true;
    p->lds_bytes = p->direct ? 0 : lds;
    if (p->series) {
        std::vector<int32_t> slot_of((size_t)k->n_kernels, -1);
        const std::vector<int32_t> &kid = p->split ? rocket::split_slot_kernels(p->split) : p->host.kid;
        for (size_t q = 0; q < kid.size(); ++q)
            if (kid[q] >= 0) slot_of[(size_t)kid[q]] = (int32_t)q;
        if (std::find(slot_of.begin(), slot_of.end(), -1) != slot_of.end()) {  // every kernel has a slot
            plan_free_device(p);
            delete p;
            return ROCKET_ERR_INTERNAL;
        }
        e = upload(slot_of, &p->d_slot_of);
        for (hipEvent_t *ev : {&p->scratch_done, &p->half_full[0], &p->half_full[1], &p->half_free[0],
                               &p->half_free[1], &p->aux_done, &p->call_start, &p->odd_done})
            if (e == hipSuccess) e = hipEventCreateWithFlags(ev, hipEventDisableTiming);
        if (e == hipSuccess) e = hipStreamCreateWithFlags(&p->aux, hipStreamNonBlocking);
        if (e == hipSuccess) e = hipStreamCreateWithFlags(&p->odd, hipStreamNonBlocking);
    }
    if (!p->direct && !p->minirocket &&
        (p->split_rest ||
         (!p->split && std::any_of(p->host.items.begin(), p->host.items.end(),
                                   [](const rocket::ItemDesc &it) { return it.variant >= rocket::kToepVariant0; })))) {
        for (hipEvent_t *ev : {&p->side_start, &p->side_done})
            if (e == hipSuccess) e = hipEventCreateWithFlags(ev, hipEventDisableTiming);
        if (e == hipSuccess) e = hipStreamCreateWithFlags(&p->side, hipStreamNonBlocking);
    }
    const int32_t K = k->n_kernels;
    p->max_len = k->max_len;
    if (p->direct) {  // only its kernel reads the set as given
        if (e == hipSuccess) e = upload_raw(k->length, (size_t)K, &p->d_len);
        if (e == hipSuccess) e = upload_raw(k->dilation, (size_t)K, &p->d_dil);
        if (e == hipSuccess) e = upload_raw(k->padding, (size_t)K, &p->d_pad);
        if (e == hipSuccess) e = upload_raw(k->bias, (size_t)K, &p->d_b);
        if (e == hipSuccess) e = upload_raw(k->weights, (size_t)K * p->C * k->max_len, &p->d_w);
        if (e == hipSuccess && p->C > 1) e = upload_raw(k->channel_count, (size_t)K, &p->d_cc);
        if (e == hipSuccess && p->C > 1) e = upload_raw(k->channel_index, (size_t)K * p->C, &p->d_ci);
    }
    if (!p->direct && fp32_items && e == hipSuccess) e = upload_tables(p, lds);
    if (e != hipSuccess) {
        plan_free_device(p);
        delete p;
        return map_hip(e);
    }
    *out = p;
    return ROCKET_OK;
}

extern "C" rocket_status rocket_minirocket_plan_create(const rocket_minirocket_params *m, uint32_t flags,
                                                       rocket_plan **out) {
    if (!out) return ROCKET_ERR_INVALID_ARG;
    *out = nullptr;
    if (flags & ~ROCKET_PLAN_CLAMPED) return ROCKET_ERR_INVALID_ARG;
    rocket_status st = rocket::validate_minirocket(m);
    if (st != ROCKET_OK) return st;
    rocket_plan *p = new (std::nothrow) rocket_plan();
    if (!p) return ROCKET_ERR_OOM;
    st = rocket::build_minirocket_plan(m, &p->host);
    if (st != ROCKET_OK) {
        delete p;
        return st;
    }
    hipError_t e = hipGetDevice(&p->device);
    hipDeviceProp_t prop;
    if (e == hipSuccess) e = hipGetDeviceProperties(&prop, p->device);
    if (e != hipSuccess) {
        delete p;
        return ROCKET_ERR_HIP;
    }
    p->n_cu = prop.multiProcessorCount;
    p->minirocket = true;
    p->C = 1;
    p->f_cols = p->host.n_features;
    int64_t lds = 0;
    if (!choose_layout(p, (flags & ROCKET_PLAN_CLAMPED) != 0, prop, &lds)) {
        // a series too long for one workgroup's LDS even with 512-zero margins
        delete p;
        return ROCKET_ERR_LENGTH;
    }
    p->lds_bytes = lds;
    e = upload_tables(p, lds);
    if (e != hipSuccess) {
        plan_free_device(p);
        delete p;
        return map_hip(e);
    }
    *out = p;
    return ROCKET_OK;
}

extern "C" rocket_status rocket_plan_create(const rocket_kernels *k, int32_t L, rocket_plan **out) {
    return rocket_plan_create_ex(k, L, ROCKET_PLAN_DEFAULT, out);
}

extern "C" void rocket_plan_destroy(rocket_plan *p) {
    if (!p) return;
    plan_free_device(p);
    delete p;
}

extern "C" int32_t rocket_checked_build(void) { return ROCKET_CHECKED ? 1 : 0; }

extern "C" rocket_status rocket_check_flags(uint32_t *flags) {
    if (!flags) return ROCKET_ERR_INVALID_ARG;
    *flags = 0;
#if ROCKET_CHECKED
    // the variable's own symbol, not its host-side name: the runtime resolves
    // the current device's copy
    if (hipDeviceSynchronize() != hipSuccess) return ROCKET_ERR_HIP;
    unsigned int v = 0;
    const unsigned int zero = 0;
    if (hipMemcpyFromSymbol(&v, HIP_SYMBOL(g_rocket_checks), sizeof(v)) != hipSuccess ||
        hipMemcpyToSymbol(HIP_SYMBOL(g_rocket_checks), &zero, sizeof(zero)) != hipSuccess)
        return ROCKET_ERR_HIP;
    *flags = v;
    if (rocket::split_check_flags(flags) != ROCKET_OK) return ROCKET_ERR_HIP;
#endif
    return ROCKET_OK;
}

extern "C" rocket_status rocket_plan_info(const rocket_plan *p, rocket_plan_facts *out) {
    if (!p || !out) return ROCKET_ERR_INVALID_ARG;
    std::memset(out, 0, sizeof(*out));
    item_facts(p->host, p->series, p->minirocket, out);
    if (p->split) {
        // the plan's fp32 items are what split items leave over
        out->n_items += rocket::split_n_items(p->split);
        out->n_buckets = rocket::split_n_buckets(p->split);
    }
    if (p->split)
        out->lds_bytes = p->series ? rocket::split_series_lds(p->host.L) : rocket::split_lds_bytes(p->split);
    else
        out->lds_bytes = p->series ? p->series_lds : p->lds_bytes;
    out->direct = p->direct ? 1 : 0;
    out->clamped = p->clamp ? 1 : 0;
    out->features_per_kernel = p->minirocket ? 0 : (p->mpv ? 3 : 2);
    out->n_features = p->f_cols;
    out->minirocket = p->minirocket ? 1 : 0;
    out->series_lane = p->series ? 1 : 0;
    out->rows_per_block = p->direct   ? 0
                          : p->series ? kSeriesLanes
                          : p->split  ? rocket::split_rows_per_block(p->split)
                                      : p->rows_per_block;
    return ROCKET_OK;
}

extern "C" rocket_status rocket_plan_split_counts(const rocket_plan *p, int64_t *items, int64_t *kernels) {
    if (!p || !items || !kernels) return ROCKET_ERR_INVALID_ARG;
    *items = *kernels = 0;
    if (p->split) {
        *items = rocket::split_n_items(p->split);
        *kernels = p->host.n_kernels - rocket::split_n_rest(p->split);
    }
    return ROCKET_OK;
}

static rocket_status launch_direct(const rocket_plan *p, const float *X, int64_t n, float *F,
                                   hipStream_t s) {
    const int32_t K = p->host.n_kernels;
    const int per_block = kBlock / 64;
    const int64_t max_y = 65535;
    const int64_t max_x = INT_MAX;
    for (int64_t r0 = 0; r0 < n; r0 += max_x) {
        const int64_t nr = std::min<int64_t>(max_x, n - r0);
        for (int64_t k0 = 0; k0 < K; k0 += max_y * per_block) {
            const int64_t nk = std::min<int64_t>(max_y * per_block, K - k0);
            dim3 grid((unsigned)nr, (unsigned)((nk + per_block - 1) / per_block));
            hipLaunchKernelGGL(rocket_direct_kernel, grid, dim3(kBlock), 0, s, X, r0, p->host.L, K,
                               (int32_t)k0, p->d_len, p->d_dil, p->d_pad, p->d_b, p->d_w,
                               p->max_len, p->mpv ? 3 : 2, p->C, p->d_cc, p->d_ci, F);
            if (hipGetLastError() != hipSuccess) return ROCKET_ERR_HIP;
        }
    }
    return ROCKET_OK;
}

// The workgroup kernels (split, fused, MINIROCKET, series-lane) over n rows: F
// receives the features, or, for the series-lane kernel, S (s_rows rows per
// slot column).
static rocket_status launch_groups(const rocket_plan *p, bool series, const float *X, int64_t n, float *F,
                                   float *S, int64_t s_rows, hipStream_t s) {
    if (p->split && !p->split_rest)
        return rocket::split_launch(p->split, X, n, p->host.n_kernels, F, nullptr, 0, s);
    // enough workgroups to fill the chip several times over: split the work
    // items of a series across workgroups when there are few series
    const int64_t target = 8 * (int64_t)std::max(p->n_cu, 1);
    const int64_t row_bytes = (int64_t)p->row_stride * (int64_t)sizeof(float);  // one channel
    const int R = series ? kSeriesLanes : p->rows_per_block;
    const int64_t groups = (n + R - 1) / R;
    int li = 0;
    // ... but once there are 2 workgroups per CU, keep a few items per
    // wavefront of a workgroup in each split (on average over the variants
    // present): 2 for 4-wavefront workgroups, 4 for the 16-wavefront ones of
    // long rows (with fewer, wavefronts wait idle at the end of a workgroup
    // while others finish)
    const bool big_group = !series && row_bytes * p->C > kBigLds;
    const int min_items = big_group ? 4 * (kBigBlock / 64) : 2 * (kBlock / 64);
    const int n_var = p->host.n_variants;
    int64_t n_present = 0;
    for (int v = 0; v < n_var; ++v)
        if (p->host.split_begin[v + 1] > p->host.split_begin[v]) ++n_present;
    n_present = std::max<int64_t>(n_present, 1);
    const int64_t per_variant = (int64_t)p->host.items.size() / n_present;
    const int64_t few_groups = 2 * (int64_t)std::max(p->n_cu, 1);
    if (series) {
        // a series-lane chunk's workgroups are few and short: split them only
        // as far as about 4 workgroups per CU, so that the whole grid is
        // resident at once and no partial second round of workgroups trails
        // each chunk
        while (li + 1 < rocket::kNumSplitLayouts &&
               groups * rocket::kSplitCounts[li + 1] <= 4 * (int64_t)std::max(p->n_cu, 1) &&
               per_variant / rocket::kSplitCounts[li + 1] >= min_items)
            ++li;
    } else {
        while (li + 1 < rocket::kNumSplitLayouts && groups * rocket::kSplitCounts[li] < target &&
               (per_variant / rocket::kSplitCounts[li + 1] >= min_items ||
                groups * n_present * rocket::kSplitCounts[li] < few_groups))
            ++li;
    }
    const int nsplit = rocket::kSplitCounts[li];
    FusedArgs a;
    a.X = X;
    a.F = F;
    a.L = p->host.L;
    // F rows hold nf * K floats: per kernel (PPV, MAX[, MPV]); a MINIROCKET
    // plan's rows hold its n_features PPVs (nf = 1)
    a.K = p->minirocket ? (int32_t)p->f_cols : p->host.n_kernels;
    a.nf = p->minirocket ? 1 : (p->mpv ? 3 : 2);
    a.thr = p->d_thr;
    a.C = p->C;
    a.items = p->d_items;
    a.wpk = p->d_wpk;
    a.bias = p->d_bias;
    a.kid = p->d_kid;
    a.order = p->d_order;
    a.split_begin = p->d_split_begin + p->host.layout_off[li];
    a.nsplit = nsplit;
    a.n_variants = 0;
    // The cost order (variant_order) pays where a launch is a few rounds
    // of workgroups per CU, so that its end is a visible share of it (1,000
    // series: 2.5-3.5 % faster).  Launches of many rounds keep the index
    // order, which measured 0.2 % faster on 100,000 series; series-lane
    // chunks keep it too (their launches overlap the next chunk's on a
    // second stream, and the cost order measured 1.6 % slower there).
    const bool cost_order = !series && groups * nsplit * n_present < 128 * (int64_t)std::max(p->n_cu, 1);
    for (int i = 0; i < n_var; ++i) {
        const int v = cost_order ? p->variant_order[i] : i;
        const int32_t *sb = p->host.split_begin.data() + p->host.layout_off[li];
        if (sb[(v + 1) * nsplit] > sb[v * nsplit]) a.variants[a.n_variants++] = v;
    }
    a.halo_lo = p->halo_lo;
    a.row_stride = p->row_stride;
    a.tail_pad = p->tail_pad;
    a.rows_per_block = R;
    a.vec4 = (a.L % 4 == 0 && a.halo_lo % 4 == 0 && a.row_stride % 4 == 0 && a.tail_pad % 4 == 0 &&
              ((uintptr_t)X % 16) == 0)
                 ? 1
                 : 0;
    a.S = S;
    a.s_rows = s_rows;
    a.s_floats = series ? (int64_t)p->host.kid.size() * s_rows * a.nf : 0;
    const size_t lds = (size_t)(series ? p->series_lds : p->lds_bytes);
    const bool big = big_group;
    const int sel = (big ? 1 : 0) | (p->clamp ? 2 : 0) | (p->mpv ? 4 : 0) | (p->C > 1 ? 8 : 0);
    // ROCKET plans: the Toeplitz items' variants go to a kernel of their
    // own
    FusedArgs parts[2] = {a, a};
    const void *fns[2] = {nullptr, nullptr};
    int nparts = 0, toep_part = -1;
    if (series || p->minirocket) {
        fns[nparts++] = series ? series_fn(p->mpv) : mr_fn(sel & 3);
    } else {
        parts[0].n_variants = parts[1].n_variants = 0;
        for (int i = 0; i < a.n_variants; ++i) {
            FusedArgs &q = parts[a.variants[i] >= rocket::kToepVariant0 ? 1 : 0];
            q.variants[q.n_variants++] = a.variants[i];
        }
        if (parts[0].n_variants > 0) {
            parts[nparts] = parts[0];
            fns[nparts++] = fused_fn(sel);
        }
        if (parts[1].n_variants > 0) {
            toep_part = nparts;
            parts[nparts] = parts[1];
            fns[nparts++] = toep_fn(sel & 7);
        }
    }
    // Split plans: the MFMA and VALU items run in the split items' launch
    // while that costs less than a launch of their own on the side stream and
    // its events (about 30 us): in that kernel they run 3 wavefronts per SIMD
    // instead of 5, about a quarter slower.  The bounds are 100 us of the whole
    // chip (2.4 GHz, 4 SIMDs of 256 CUs), and 400 us for rows above 40 KB,
    // which run one workgroup per CU.  One launch against two, us: 400 x 1,000
    // samples, 1,000 kernels (1.3e8 cycles) 114 and 119; 2,000 x 1,000, 300
    // (3.2e8) 268 and 229; 400 x 5,000, 5,000 (1e9) 2,054 and 1,943; 100,000 x
    // 1,000, 10,000 (4e10) 126,200 and 123,500; 16 x 16,000, 10,000 (7.5e8) 502
    // and 594; 400 x 16,000, 1,000 (2.4e9) 2,171 and 2,085.
    const double rest_cycles = p->split ? rocket::split_rest_cost(p->split) * (double)n : 0.0;
    const bool joined = p->split && !p->clamp && rest_cycles < (rocket::split_one_per_cu(p->split) ? 1e9 : 2.5e8) &&
                        p->lds_bytes <= rocket::split_lds_room(p->split);
    // Toeplitz items, and the fp32 items of a split plan's long calls, run on
    // the plan's side stream, concurrently with the other part: they start
    // after the caller's earlier work and the call ends on the caller's
    // stream after all of them
    const bool fp32_part = nparts > (toep_part >= 0 ? 1 : 0);
    bool side = p->side != nullptr && (toep_part >= 0 ? (fp32_part || p->split) : (p->split && !joined));
    // a call under capture stays on the caller's stream: the side stream would
    // belong to the capture until it ends, calls of other threads on this plan
    // would fail meanwhile, and destroying the plan would release a stream and
    // events that take part in it
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (side && s != nullptr) {
        if (hipStreamIsCapturing(s, &capture) != hipSuccess) return ROCKET_ERR_HIP;
        side = capture == hipStreamCaptureStatusNone;
    }
    std::unique_lock<std::mutex> side_lock(p->side_mu, std::defer_lock);
    if (side) {
        side_lock.lock();
        if (hipEventRecord(p->side_start, s) != hipSuccess || hipStreamWaitEvent(p->side, p->side_start, 0) != hipSuccess)
            return ROCKET_ERR_HIP;
    }
    rocket_status st = ROCKET_OK;
    if (p->split) {
        st = rocket::split_launch(p->split, X, n, p->host.n_kernels, F, joined && fp32_part ? &parts[0] : nullptr,
                                  p->lds_bytes, s);
    }
    for (int part = nparts - 1; part >= 0 && st == ROCKET_OK; --part) {
        FusedArgs &q = parts[part];
        if (joined && part != toep_part) continue;
        hipStream_t sq = (side && (part == toep_part || p->split)) ? p->side : s;
        const int64_t max_rows =
            ((int64_t)INT_MAX / (nsplit * std::max(q.n_variants, 1)) / kXcds - 1) * kXcds * R;
        for (int64_t r0 = 0; r0 < n; r0 += max_rows) {
            q.row0 = r0;
            q.n_rows = std::min<int64_t>(max_rows, n - r0);
            const int64_t groups_now = (q.n_rows + R - 1) / R;
            q.xcd_shift = series ? kXcdShift : xcd_shift(groups_now);
            q.groups_per_xcd = (groups_now + (1 << q.xcd_shift) - 1) >> q.xcd_shift;
            const unsigned nb = (unsigned)((q.groups_per_xcd << q.xcd_shift) * nsplit * q.n_variants);
            void *args[] = {&q};
            if (hipLaunchKernel(fns[part], dim3(nb), dim3(big ? kBigBlock : kBlock), args, lds, sq) != hipSuccess ||
                hipGetLastError() != hipSuccess) {
                st = ROCKET_ERR_HIP;
                break;
            }
        }
    }
    // also after a failure part-way: the caller's stream waits for whatever
    // the side stream holds
    if (side && (hipEventRecord(p->side_done, p->side) != hipSuccess ||
                 hipStreamWaitEvent(s, p->side_done, 0) != hipSuccess))
        return ROCKET_ERR_HIP;
    return st;
}

// Series-lane layout: the rows go in chunks; for each chunk the series
// kernel writes the features in slot order into one half of a feature
// buffer (each slot's features of 64 consecutive series are contiguous), and
// the permutation kernel writes the chunk's F rows in the original kernel
// order, 64 kernels (64 * nf floats) at a time.  The scatter of single
// features over F rows would otherwise cost more than the dot products of
// short series.  The permutation (memory-bound) runs on the plan's own
// stream, beside the next chunk's series kernel (compute-bound) on the
// caller's; chunk i uses half i % 2, which it takes once the permutation of
// chunk i - 2 is done with it.  The call ends on the caller's stream after
// the last permutation.

// Floats of one series' slot-ordered features.
static int64_t series_slots(const rocket_plan *p) {
    return (int64_t)(p->split ? rocket::split_slot_kernels(p->split).size() : p->host.kid.size());
}
static int64_t series_slot_row_floats(const rocket_plan *p) { return series_slots(p) * (p->mpv ? 3 : 2); }

// Rows per chunk for halves of at most half_bytes (a multiple of 64, at
// most 8,192 and no more than the call needs); 0 when not even 64 series fit.
static int64_t series_chunk_rows(const rocket_plan *p, int64_t n, size_t half_bytes) {
    const int64_t row_bytes = std::max<int64_t>(series_slot_row_floats(p), 1) * (int64_t)sizeof(float);
    int64_t chunk = (int64_t)(half_bytes / (size_t)row_bytes) / kSeriesLanes * kSeriesLanes;
    if (chunk < kSeriesLanes) return 0;
    chunk = std::min<int64_t>(8192, chunk);
    return std::min(chunk, (n + kSeriesLanes - 1) / kSeriesLanes * kSeriesLanes);
}

// The chunk loop over a two-half buffer of `chunk` rows per half.  Chunk i
// runs its series kernel on the caller's stream (i even) or on the plan's
// odd-chunk stream (i odd), so each stream only ever uses its own half, and
// consecutive chunks overlap; the permutations run in chunk order on the
// plan's permutation stream.  The caller holds p->scratch_mu (the plan's
// streams and events are shared by every transform of the plan).
static rocket_status enqueue_series(const rocket_plan *p, const float *X, int64_t n, float *F,
                                    hipStream_t s, float *buf, int64_t chunk) {
    const int64_t K = p->host.n_kernels;
    const int nf = p->mpv ? 3 : 2;
    const int64_t half = chunk * series_slot_row_floats(p);  // floats
    const void *pf = nf == 3 ? (const void *)rocket_slot_permute_kernel<3>
                             : (const void *)rocket_slot_permute_kernel<2>;
    // a failure part-way still ends with the tail below, so that the next
    // transform of this plan waits for whatever this one enqueued
    rocket_status st = ROCKET_OK;
    // the odd-chunk stream starts after the caller's earlier work (X ready,
    // the previous user of the buffer done)
    if (hipEventRecord(p->call_start, s) != hipSuccess || hipStreamWaitEvent(p->odd, p->call_start, 0) != hipSuccess)
        st = ROCKET_ERR_HIP;
    int i = 0;
    for (int64_t r0 = 0; r0 < n && st == ROCKET_OK; r0 += chunk, ++i) {
        const int h = i & 1;
        hipStream_t sh = h ? p->odd : s;
        const int64_t m = std::min(chunk, n - r0);
        float *Sh = buf + h * half;
        if (i >= 2 && hipStreamWaitEvent(sh, p->half_free[h], 0) != hipSuccess) {
            st = ROCKET_ERR_HIP;
            break;
        }
        st = p->split ? rocket::split_launch_series(p->split, X + r0 * p->host.L, m, p->host.n_kernels, Sh, chunk, sh)
                      : launch_groups(p, true, X + r0 * p->host.L, m, nullptr, Sh, chunk, sh);
        if (st != ROCKET_OK) break;
        if (hipEventRecord(p->half_full[h], sh) != hipSuccess ||
            hipStreamWaitEvent(p->aux, p->half_full[h], 0) != hipSuccess) {
            st = ROCKET_ERR_HIP;
            break;
        }
        const int64_t tiles = ((K + 63) / 64) * ((m + 63) / 64);
        // one workgroup per CU, striding over the tiles: the permutation then
        // moves its bytes at a modest rate over the whole of the next chunk's
        // series kernel (a full grid moves them in a burst that stalls it)
        const dim3 grid((unsigned)std::min<int64_t>(tiles, std::max(p->n_cu, 1)));
        const float *S = Sh;
        const int32_t *slot_of = p->d_slot_of;
        int32_t K32 = (int32_t)K;
        int64_t s_rows = chunk;
        float *Fc = F + r0 * K * nf;
        int64_t mm = m;
        int32_t n_slots = (int32_t)series_slots(p);
        void *args[] = {(void *)&S, &s_rows, (void *)&slot_of, &K32, (void *)&mm, &Fc, &n_slots};
        if (hipLaunchKernel(pf, grid, dim3(kBlock), args, 0, p->aux) != hipSuccess ||
            hipGetLastError() != hipSuccess || hipEventRecord(p->half_free[h], p->aux) != hipSuccess) {
            st = ROCKET_ERR_HIP;
            break;
        }
    }
    const bool tail_ok = hipEventRecord(p->aux_done, p->aux) == hipSuccess &&
                         hipStreamWaitEvent(s, p->aux_done, 0) == hipSuccess &&
                         hipEventRecord(p->odd_done, p->odd) == hipSuccess &&
                         hipStreamWaitEvent(s, p->odd_done, 0) == hipSuccess;
    if (st != ROCKET_OK) return st;
    return tail_ok ? ROCKET_OK : ROCKET_ERR_HIP;
}

// The plan's own feature buffer: at most 1 GiB (halves of up to 8,192 rows),
// allocated on first use and grown as needed; transforms on different
// streams take turns on it (each waits for the previous user's event).
static rocket_status launch_series(const rocket_plan *p, const float *X, int64_t n, float *F,
                                   hipStream_t s) {
    const int64_t chunk = std::max<int64_t>(kSeriesLanes, series_chunk_rows(p, n, (size_t)1 << 29));
    const size_t need = (size_t)(2 * chunk * series_slot_row_floats(p)) * sizeof(float);
    std::lock_guard<std::mutex> lock(p->scratch_mu);
    if (p->scratch_bytes < need) {
        // hipFree waits for the work that still uses the old buffer
        if (p->d_scratch && hipFree(p->d_scratch) != hipSuccess) return ROCKET_ERR_HIP;
        p->d_scratch = nullptr;
        p->scratch_bytes = 0;
        if (hipMalloc(&p->d_scratch, need) != hipSuccess) return ROCKET_ERR_OOM;
        p->scratch_bytes = need;
    }
    // the previous transform of this plan (on any stream) is done with it
    if (hipStreamWaitEvent(s, p->scratch_done, 0) != hipSuccess) return ROCKET_ERR_HIP;
    const rocket_status st = enqueue_series(p, X, n, F, s, p->d_scratch, chunk);
    // recorded after the tail, also after a failure part-way
    const bool rec_ok = hipEventRecord(p->scratch_done, s) == hipSuccess;
    if (st != ROCKET_OK) return st;
    return rec_ok ? ROCKET_OK : ROCKET_ERR_HIP;
}

// ---------------------------------------------------------------------------
// Static scratch of rocket_transform_plan_noalloc: the series-lane feature
// buffer of callers that cannot allocate device memory.  Every GPU the
// library runs on holds its own copy of the array (from the first use of the
// library's code there until the process ends).  Host code uses the device
// address that hipGetSymbolAddress returns for the current device, never the
// array's name (a host-side stand-in).
// ---------------------------------------------------------------------------
constexpr size_t kNoAllocScratchBytes = 2 * (size_t)kNoAllocHalfBytes;  // ROCKET_NOALLOC_SCRATCH_BYTES
static_assert(kNoAllocScratchBytes == (size_t)ROCKET_NOALLOC_SCRATCH_BYTES, "header and library agree");
static __device__ __align__(256) float scratch[kNoAllocScratchBytes / sizeof(float)];

static std::mutex g_scratch_mu;
static float *g_scratch_ptr[kMaxDevices];

// The device address of `scratch` on `device` (which must be current),
// looked up once per device.
static rocket_status noalloc_scratch(int device, float **out) {
    if (device < 0 || device >= kMaxDevices) return ROCKET_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return ROCKET_ERR_HIP;
        g_scratch_ptr[device] = (float *)ptr;
    }
    *out = g_scratch_ptr[device];
    return ROCKET_OK;
}

// The series-lane chunk loop over the static scratch (two halves of 32 MiB).
static rocket_status launch_series_noalloc(const rocket_plan *p, const float *X, int64_t n, float *F,
                                           hipStream_t s, float *buf) {
    // what fits is decided by the fp32 items' slots; a split plan that needs a
    // few more runs its tiled layout instead (the same features)
    const int64_t slots = p->split ? p->fp32_slots : series_slots(p);
    if (slots * (p->mpv ? 3 : 2) * (int64_t)sizeof(float) * kSeriesLanes > kNoAllocHalfBytes) return ROCKET_ERR_SCRATCH;
    const int64_t chunk = series_chunk_rows(p, n, kNoAllocScratchBytes / 2);
    if (chunk == 0) return launch_groups(p, false, X, n, F, nullptr, 0, s);
    std::lock_guard<std::mutex> lock(p->scratch_mu);
    return enqueue_series(p, X, n, F, s, buf, chunk);
}

static rocket_status launch_fused(const rocket_plan *p, const float *X, int64_t n, float *F,
                                  hipStream_t s) {
    return (p->series && n >= p->series_min_rows) ? launch_series(p, X, n, F, s)
                                                  : launch_groups(p, false, X, n, F, nullptr, 0, s);
}

// The plan's streams, events and tables live on the device it was created
// on: that device must be the current one.
static rocket_status check_plan_device(const rocket_plan *p) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return ROCKET_ERR_HIP;
    return dev == p->device ? ROCKET_OK : ROCKET_ERR_INVALID_ARG;
}

extern "C" rocket_status rocket_transform_plan(const rocket_plan *p, const float *X_dev, int64_t n,
                                               float *F_dev, void *hip_stream) {
    if (!p || n < 0) return ROCKET_ERR_INVALID_ARG;
    const rocket_status dst = check_plan_device(p);
    if (dst != ROCKET_OK) return dst;
    if (n == 0) return ROCKET_OK;
    if (!X_dev || !F_dev) return ROCKET_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)hip_stream;
    return p->direct ? launch_direct(p, X_dev, n, F_dev, s) : launch_fused(p, X_dev, n, F_dev, s);
}

extern "C" rocket_status rocket_transform_plan_noalloc(const rocket_plan *p, const float *X_dev, int64_t n,
                                                       float *F_dev, void *hip_stream) {
    if (!p || n < 0) return ROCKET_ERR_INVALID_ARG;
    const rocket_status dst = check_plan_device(p);
    if (dst != ROCKET_OK) return dst;
    const int dev = p->device;
    float *buf = nullptr;
    const rocket_status st = noalloc_scratch(dev, &buf);
    if (st != ROCKET_OK) return st;
    if (n == 0) return ROCKET_OK;
    if (!X_dev || !F_dev) return ROCKET_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)hip_stream;
    if (p->direct) return launch_direct(p, X_dev, n, F_dev, s);
    if (p->series && n >= p->series_min_rows) return launch_series_noalloc(p, X_dev, n, F_dev, s, buf);
    return launch_groups(p, false, X_dev, n, F_dev, nullptr, 0, s);
}

// Host-to-host transform with copies overlapped against the transform:
// batch i uses X and F staging buffer i % 2.  Its copy in waits until the
// transform of batch i-2 (the last reader of that X buffer) is done; its
// transform waits for its copy in and for the copy out of batch i-2 (the
// last reader of that F buffer); its copy out waits for its transform.
extern "C" rocket_status rocket_transform_host(const rocket_plan *p, const float *X_host, int64_t n,
                                               float *F_host, int64_t batch_rows,
                                               void *hip_stream) {
    if (!p || n < 0 || batch_rows < 0) return ROCKET_ERR_INVALID_ARG;
    const rocket_status dst = check_plan_device(p);
    if (dst != ROCKET_OK) return dst;
    if (n == 0) return ROCKET_OK;
    if (!X_host || !F_host) return ROCKET_ERR_INVALID_ARG;
    const int64_t L = (int64_t)p->host.L * p->C;  // floats per series (every channel)
    const int64_t K2 = p->f_cols;  // floats per feature row
    int64_t B = batch_rows;
    // default: about 8 batches, so copies have neighbours to overlap with,
    // each within 256 MiB of staging.  Few long rows of split plans (eighths
    // of under a row per CU) take 3: a row computes for longer than its
    // features are copied (both grow with the kernels, only the first with L).  Times of one shape vary by a third
    // with the hardware queues that the call's copy streams come to share with
    // the transform's (a process has four), more than the number of batches
    // moves them; lowest seen, ms: 1,000 x 2,000 samples, 10,000 kernels 3.5 in
    // 3 and in 8; 200 x 8,000, 5,000 kernels 2.5 in 3, 3.3 in 8; 1,000 x 1,600
    // 4.0 and 4.5; 1,000 x 1,280 3.5 and 4.0; 1,000 x 1,000 2.1 and 3.9; 2,000
    // x 500 4.9 and 4.7; 3,000 x 300, 8,000 kernels 5.8 and 4.8; 5,000 x
    // 1,400, 2,000 kernels 4.0 and 3.6; 91,340 x 1,612, 296 kernels 24 and 18.
    const int64_t parts = p->split && L >= 1280 && n < 8 * (int64_t)p->n_cu ? 3 : 8;
    if (B == 0)
        B = std::max<int64_t>(1, std::min<int64_t>((n + parts - 1) / parts, (int64_t)(256 << 20) / ((L + K2) * 4)));
    B = std::min(B, n);
    const int64_t nb = (n + B - 1) / B;
    hipStream_t sc = (hipStream_t)hip_stream;
    hipStream_t s_in = nullptr, s_out = nullptr;
    float *dX[2] = {nullptr, nullptr}, *dF[2] = {nullptr, nullptr};
    hipEvent_t ev_in[2] = {}, ev_tr[2] = {}, ev_out[2] = {};
    rocket_status st = ROCKET_OK;
    hipError_t e = hipStreamCreateWithFlags(&s_in, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&s_out, hipStreamNonBlocking);
    for (int j = 0; j < 2 && e == hipSuccess; ++j) {
        e = hipMalloc((void **)&dX[j], (size_t)(B * L * 4));
        if (e == hipSuccess) e = hipMalloc((void **)&dF[j], (size_t)(B * K2 * 4));
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ev_in[j], hipEventDisableTiming);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ev_tr[j], hipEventDisableTiming);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ev_out[j], hipEventDisableTiming);
    }
    for (int64_t i = 0; i < nb && e == hipSuccess && st == ROCKET_OK; ++i) {
        const int j = (int)(i & 1);
        const int64_t r0 = i * B, m = std::min(B, n - r0);
        if (i >= 2) e = hipStreamWaitEvent(s_in, ev_tr[j], 0);
        if (e == hipSuccess)
            e = hipMemcpyAsync(dX[j], X_host + r0 * L, (size_t)(m * L * 4), hipMemcpyHostToDevice, s_in);
        if (e == hipSuccess) e = hipEventRecord(ev_in[j], s_in);
        if (e == hipSuccess) e = hipStreamWaitEvent(sc, ev_in[j], 0);
        if (e == hipSuccess && i >= 2) e = hipStreamWaitEvent(sc, ev_out[j], 0);
        if (e == hipSuccess) st = rocket_transform_plan(p, dX[j], m, dF[j], sc);
        if (e == hipSuccess && st == ROCKET_OK) e = hipEventRecord(ev_tr[j], sc);
        if (e == hipSuccess && st == ROCKET_OK) e = hipStreamWaitEvent(s_out, ev_tr[j], 0);
        if (e == hipSuccess && st == ROCKET_OK)
            e = hipMemcpyAsync(F_host + r0 * K2, dF[j], (size_t)(m * K2 * 4), hipMemcpyDeviceToHost, s_out);
        if (e == hipSuccess && st == ROCKET_OK) e = hipEventRecord(ev_out[j], s_out);
    }
    // drain every stream before the staging buffers go away
    const hipError_t e1 = s_in ? hipStreamSynchronize(s_in) : hipSuccess;
    const hipError_t e2 = hipStreamSynchronize(sc);
    const hipError_t e3 = s_out ? hipStreamSynchronize(s_out) : hipSuccess;
    for (int j = 0; j < 2; ++j) {
        if (dX[j]) (void)hipFree(dX[j]);
        if (dF[j]) (void)hipFree(dF[j]);
        if (ev_in[j]) (void)hipEventDestroy(ev_in[j]);
        if (ev_tr[j]) (void)hipEventDestroy(ev_tr[j]);
        if (ev_out[j]) (void)hipEventDestroy(ev_out[j]);
    }
    if (s_in) (void)hipStreamDestroy(s_in);
    if (s_out) (void)hipStreamDestroy(s_out);
    if (st != ROCKET_OK) return st;
    if (e != hipSuccess) return map_hip(e);
    if (e1 != hipSuccess || e2 != hipSuccess || e3 != hipSuccess) return ROCKET_ERR_HIP;
    return ROCKET_OK;
}

extern "C" rocket_status rocket_transform(const float *X_dev, int64_t n, int32_t L,
                                          const rocket_kernels *k, float *F_dev, void *hip_stream) {
    if (n < 0) return ROCKET_ERR_INVALID_ARG;
    if (n > 0 && (!X_dev || !F_dev)) return ROCKET_ERR_INVALID_ARG;
    rocket_status st = rocket::validate_kernels(k, L);
    if (st != ROCKET_OK) return st;
    if (n == 0) return ROCKET_OK;
    rocket_plan *p = nullptr;
    st = rocket_plan_create(k, L, &p);
    if (st != ROCKET_OK) return st;
    st = rocket_transform_plan(p, X_dev, n, F_dev, hip_stream);
    const hipError_t e = hipStreamSynchronize((hipStream_t)hip_stream);
    rocket_plan_destroy(p);
    if (st != ROCKET_OK) return st;
    return e == hipSuccess ? ROCKET_OK : ROCKET_ERR_HIP;
}
