// Internal layout shared by the host planner (plan.cpp) and the gfx950
// kernels (transform.hip).  Not part of the public ABI.
#pragma once

#include <cstdint>
#include <vector>

#include "rocket.h"

namespace rocket {

// The fused MFMA path keeps the three kernel lengths ROCKET draws
// (Sec. 2.1: 7, 9, 11).  A hand-built kernel of another length is run as the
// next supported length with zero weights on the extra taps.
constexpr int kNumEll = 3;
constexpr int kEllValues[kNumEll] = {7, 9, 11};

inline int ell_index_for(int length) { return length <= 7 ? 0 : (length <= 9 ? 1 : 2); }

// Wavefront size on CDNA4 and the number of kernel slots one
// v_mfma_f32_4x4x1_16b_f32 block holds (its 4 A-matrix rows).
constexpr int kWave = 64;
constexpr int kSlotsPerGroup = 4;
constexpr int kMaxGroups = 2;  // a work item holds 4 or 8 kernels of one bucket

// Outputs are computed in tiles of 64 consecutive positions: lane l of a
// wavefront computes output 64*k + l of tile k for every kernel slot of the
// item.  A block runs kTilesPerBlock[G-1] tiles at once (the independent
// MFMA accumulation chains of a wavefront: tiles x groups = 8).
constexpr int kTile = kWave;
constexpr int kTilesPerBlock[kMaxGroups] = {8, 4};
constexpr int kMaxTilesPerBlock = 8;

// Clamped row layout (long series): each staged row carries this many zeros
// on each side; the series index of a block's first lane is clamped into
// [-kClampMargin, L] on the scalar unit, so a block whose 64*NT positions all
// fall outside the series reads zeros from a margin.
constexpr int kClampMargin = kTile * kMaxTilesPerBlock;

// The fused kernel runs multichannel items over a 64-bit channel mask.
static_assert(ROCKET_MAX_CHANNELS <= 64, "channel masks are 64 bits");

// Every output of an item is computed by exactly one lane of one tile; lanes
// of the last tile past O start from -inf and change no feature.
constexpr int64_t kMaxOutputs = (int64_t)1 << 24;  // O must stay below 2^24

// One work item: up to 4*G kernels that share (length, dilation, padding),
// so every slot has the same O outputs and reads the same series values.
// MINIROCKET items use d, p, O, n_tiles, cost, t_off, nq and inv_O as named,
// and three fields for their feature numbering: w_off = the first feature of
// the item's dilation, k_off = the item's first bias (of each kernel), n_ch =
// the dilation's features per kernel; variant = mr_variant(parity, nq).
struct alignas(16) ItemDesc {
    int32_t variant;   // ell_index * 2 + (G - 1)
    int32_t d;         // dilation
    int32_t p;         // padding
    int32_t O;         // number of dot products (outputs)
    int32_t n_tiles;   // ceil(O / 64); Toeplitz items: chunks per super-tile, ceil(d / 64)
    int32_t w_off;     // first packed weight: [n_ch][G][ell][4] floats
    int32_t k_off;     // first slot entry: kernel ids and biases, [4G]
    int32_t cost;      // MFMA instructions per series (scheduling weight)
    int32_t n_ch;      // channels the item's kernels read (their union; 1 if univariate)
    int32_t ch_off;    // first entry of the item's channel list
    int32_t t_off;     // MINIROCKET: first threshold, [kMrKappa][nq] floats
    int32_t nq;        // MINIROCKET: thresholds per kernel in this item (kMrQTiny, kMrQSmall or kMrQLarge)
    uint32_t ch_mask[2];  // multichannel: the item's channels as a bit mask (lo, hi words)
    double inv_O;      // 1 / O rounded to double (exact PPV, see transform.hip)
};
static_assert(sizeof(ItemDesc) == 64, "ItemDesc must stay 64 bytes");
constexpr int kItemWords = (int)(sizeof(ItemDesc) / sizeof(int32_t));

// Item orders for a few split counts.  Within a layout with `nsplit` splits
// the items are grouped by variant, so that every workgroup runs one code
// variant: the items of variant v in split s are
// order[split_begin[v*nsplit + s] .. split_begin[v*nsplit + s + 1]).
// Variants 0..5 are MFMA items, 2 * ell_index + (G - 1).  Variants 6..11 are
// VALU items: the one or two leftover kernels of a bucket (nk of them), run
// with plain fp32 FMA instead of a 4-slot MFMA group that would be mostly
// empty, 6 + 2 * ell_index + (nk - 1); their weights keep the 4-slot packing
// of a one-group item.
constexpr int kNumMfmaVariants = 2 * kNumEll;
constexpr int kNumVariants = 6 * kNumEll;
constexpr int kValuVariant0 = kNumMfmaVariants;

// Variants 12..17 are Toeplitz items: the one or two kernels left over in a
// bucket at a large dilation d, 12 + 2 * ell_index + (nk - 1).  The 4 slots
// of one MFMA group hold the same kernel shifted by sigma = 4 / nk taps:
// slot s is kernel s / sigma at shift h = s % sigma, whose weight at tap m is
// w[m - h], over ell + sigma - 1 taps; lane l of chunk c of super-tile st
// then computes, in slot s, the output at position
//     st * sigma * d + 64 c + l + h * d,
// valid when 64 c + l < d (the chunks of a super-tile cover d positions per
// shift) and the position is below O.  A super-tile covers sigma * d
// consecutive outputs per kernel in ceil(d / 64) chunks; each chunk is one
// tile of 64 consecutive series reads per tap, as in an MFMA item.
constexpr int kToepVariant0 = 4 * kNumEll;

// Series of at most this length can run in the series-lane layout, which
// takes MFMA items only; VALU items are made for longer series.
constexpr int kSeriesMaxL = 128;
constexpr int kNumSplitLayouts = 6;  // 1, 2, 4, 8, 16, 32 splits
constexpr int kSplitCounts[kNumSplitLayouts] = {1, 2, 4, 8, 16, 32};

// MINIROCKET (Sec. 5 names it): 84 kernels of 9 taps.  Pair (dilation i,
// kernel k) is padded when i + k is even, so at one (dilation, padding) the
// kernels are those of one parity of k: an item holds those 42 kernels and
// kMrQTiny, kMrQSmall or kMrQLarge of each kernel's biases (dummy biases of
// +inf fill the last chunk; C > +inf never holds).  Variant = 3 * parity +
// bias class (0: kMrQSmall, 1: kMrQLarge, 2: kMrQTiny).
constexpr int kMrKernels = 84;
constexpr int kMrTaps = 9;
constexpr int kMrKappa = kMrKernels / 2;
constexpr int kMrQTiny = 3;
constexpr int kMrQSmall = 4;
constexpr int kMrQLarge = 8;
constexpr int kMrNumVariants = 6;  // parity x {kMrQSmall, kMrQLarge, kMrQTiny}
constexpr int mr_variant(int parity, int nq) {
    return 3 * parity + (nq == kMrQLarge ? 1 : (nq == kMrQTiny ? 2 : 0));
}

struct HostPlan {
    bool minirocket = false;
    int64_t n_features = 0;  // columns of F
    int32_t n_kernels = 0;
    int32_t L = 0;
    int32_t halo_lo = 0;     // padded layout: zeros staged before the series
    int32_t halo_hi = 0;     // padded layout: zeros staged after the series
    int32_t row_stride = 0;  // padded layout: floats per staged row (0: does not fit 32 bits)
    int32_t tail_pad = 0;    // zeros staged after the last row (reads of lanes past O)
    int32_t n_channels = 1;  // channels per series
    int64_t n_buckets = 0;
    int64_t mfma_per_row = 0;
    int64_t series_mfma_64 = 0;  // MFMAs for 64 series in the series-lane layout (O x taps x G)
    int64_t valu_fma_per_row = 0;  // VALU items: fp32 FMA instructions (64 lanes) per series
    std::vector<ItemDesc> items;
    std::vector<float> wpk;       // packed A-operand weights
    std::vector<float> bias;      // per slot
    std::vector<int32_t> kid;     // per slot, -1 = empty
    std::vector<int32_t> chan;    // per item, its channel list (ascending)
    std::vector<float> thr;       // MINIROCKET: per item [nq][4] thresholds
    std::vector<int32_t> order;   // kNumSplitLayouts concatenated item orders
    int32_t n_variants = kNumVariants;  // code variants of the plan's kernel (kMrNumVariants for MINIROCKET)
    std::vector<int32_t> split_begin;  // per layout: n_variants*nsplit + 1 offsets into order
    std::vector<int32_t> layout_off;   // per layout: offset into split_begin
};

// Validate a kernel set for series length L (host only, no device calls).
rocket_status validate_kernels(const rocket_kernels *k, int32_t L);

// Build the host-side tables of a plan.  Assumes validate_kernels passed.
// beside: what else a call runs per series, in MFMAs (split items, which
// decide whether Toeplitz items pay their launch).
rocket_status build_host_plan(const rocket_kernels *k, int32_t L, HostPlan *out, double beside = 0.0);

// MINIROCKET parameters: validation and the plan's host tables.
rocket_status validate_minirocket(const rocket_minirocket_params *m);
rocket_status build_minirocket_plan(const rocket_minirocket_params *m, HostPlan *out);

// Item orders: per variant (0 .. n_variants - 1), longest-processing-time
// split of the items into every layout's split count (fills order,
// split_begin, layout_off).
void build_item_orders(HostPlan &P);

// ---------------------------------------------------------------------------
// Split items (univariate plans): the dot products on v_mfma_f32_32x32x16_bf16, with every fp32 weight and series
// value split into three bf16 parts (8 + 8 + 8 significant bits, so the three
// parts hold all 24).  Of the nine part products the six largest are summed
// (dropped: x2 w3 and x3 w2, each at most 2^-24 of the product and about 2^-27
// in the mean, and x3 w3, below 2^-31).  An item holds up to
// 32 kernels of one dilation: the rows of the MFMA.  Its columns are 32
// consecutive positions, its contraction index the taps and their parts.
//
// Kernels of any padding, and of shorter lengths, share an item: kernel k of
// length len sits in a frame of `frame` taps (7, 9 or 11) at frame tap
// f = (frame - len) / 2, and column c stands for the outputs whose frame tap 0
// reads series index s0 + c.  The valid columns of every row are then centred
// on the same point (series length minus frame span, halved), a row with O
// outputs being valid where |2 c + 1 - n_cols| < O, with n_cols the largest O.
// (Kernels of even and odd length have centres half a dilation apart and do
// not share items.)
//
// LDS holds each staged row twice as 32-bit words, one per position: word 0 =
// (x1, x2), word 1 = (x3, x1) (low half first), kSplitMargin zeros around.
// ---------------------------------------------------------------------------
constexpr int kSplitRows = 32;             // kernels per item
constexpr int kSplitTile = 32;             // columns per MFMA
constexpr int kSplitBlock = 64;            // columns per block: two tiles
constexpr int kSplitMargin = kSplitBlock;  // zeros on each side of a staged row
constexpr int kSplitSeriesMargin = 8;      // series-lane layout: zero positions on each side
constexpr int kSplitVariants = 3;          // by frame: 7, 9, 11 taps
constexpr int kSplitFrame[kSplitVariants] = {7, 9, 11};
constexpr int kSplitFrags[kSplitVariants] = {3, 4, 5};  // MFMAs (A fragments) per tile
constexpr int64_t kSplitMaxOutputs = 65535;  // counts are kept in 16-bit halves

// Rows of an item have at most kSplitWidths[variant] different O.  Columns
// outside a row's range are masked by the MFMA itself: each variant has a word
// slot per lane half that no tap uses (the eighth tap of a 7-tap frame; the
// tail's last word otherwise), whose weights are kSplitMask in the 16-bit half
// of the row's width (halves: widths 0, 1 in lane half 0, 2, 3 in half 1; the
// 7-tap frame has half 1 only, widths 0, 1).  Where the kernel puts kSplitMask
// into that half of the word the product overflows to +infinity, elsewhere the
// word is zero and adds nothing.
constexpr int kSplitWidths[kSplitVariants] = {2, 4, 4};
constexpr uint32_t kSplitMask = 0x7180u;  // 2^100 as bf16

struct alignas(16) SplitItem {
    int32_t variant;
    int32_t d;         // dilation
    int32_t s0;        // series index of frame tap 0 at column 0
    int32_t n_cols;    // columns: the largest O of the item's kernels
    int32_t clean_lo;  // blocks [clean_lo, clean_hi) need neither a mask nor a clamp:
    int32_t clean_hi;  //   every row valid, every read within the margins
    int32_t a_off;     // first A fragment, in 16-byte words: [frags][64 lanes]
    int32_t r_off;     // first row entry (32 per item)
    int32_t reach;     // last frame tap that holds a weight
    int32_t cost;      // issue cycles per series (scheduling weight)
    int32_t n_rows;    // kernels
    int32_t width[4];  // the O that a mask half stands for
    int32_t series_lo; // as clean_lo and clean_hi, in blocks of two positions of the
    int32_t series_hi; //   series-lane layout (kSplitSeriesMargin zero positions)
};
static_assert(sizeof(SplitItem) == 80, "SplitItem is 16-byte words");

// The result register i (0..15) and lane half h (0, 1) of v_mfma_f32_32x32
// hold matrix row 8 (i / 4) + 4 h + i % 4; rows are numbered q = 2 i + h here.
constexpr int split_matrix_row(int q) { return 8 * (q / 8) + 4 * (q & 1) + (q / 2) % 4; }

struct SplitPlan {
    int32_t L = 0;
    std::vector<SplitItem> items;
    std::vector<uint32_t> a;      // A fragments, bf16 pairs: [item][frag][lane][4]
    std::vector<float> cinit;     // per item [half][reg]: -bias
    std::vector<int32_t> kid;     // per item [row q]: kernel id, -1 = empty
    std::vector<double> inv_O;    // per item [row q]
    std::vector<float> div_O;     // per item [half][reg]: O and 1 / O as floats (series-lane layout)
    std::vector<int32_t> order;   // as HostPlan
    std::vector<int32_t> split_begin;
    std::vector<int32_t> layout_off;
    std::vector<int32_t> rest;    // kernels left to the fp32 items (ascending)
    int64_t n_buckets = 0;        // distinct (length, dilation, padding) of the set
    double cost = 0.0;            // issue cycles per series of the items
    double rest_cost = 0.0;       // and of the rest as fp32 items
    double fp32_cost = 0.0;       // and of all kernels as fp32 items
};

// Whether a kernel set can run as split items on series of length L.
bool split_eligible(const rocket_kernels *k, int32_t L);
// Groups the kernels into split items; those that fp32 items run faster are
// left in `rest` when together they carry a real share of the work.
rocket_status build_split_plan(const rocket_kernels *k, int32_t L, SplitPlan *out);
// Whether a plan with split items beats the fp32 plan of the whole set.
bool split_pays(const SplitPlan &P, bool mpv);

// Item orders of items given by variant and cost (see build_item_orders).
void order_items(const std::vector<int32_t> &variant, const std::vector<int32_t> &cost, int n_variants,
                 std::vector<int32_t> &order, std::vector<int32_t> &split_begin, std::vector<int32_t> &layout_off);

// Element `index` of the SplitMix64 sequence started at `seed`.
uint64_t splitmix64_at(uint64_t seed, uint64_t index);

}  // namespace rocket
