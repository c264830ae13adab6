// Host-side planning of split items: kernels grouped by dilation into items
// of up to 32 rows, their weights split into bf16 parts and packed as MFMA A
// fragments.  Pure host code; no HIP calls.
#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>
#include <new>
#include <utility>
#include <vector>

#include "rocket_internal.h"

namespace rocket {

// What a 32-column tile costs by variant, an edge tile more, and an item's
// reductions and stores per series.  The split kernel runs at the card's power
// limit (its clock falls to 1.6-1.9 GHz), so these are time at the limit in
// 2.4 GHz cycles per SIMD: a 32x32x16 MFMA on random data 43, a vector
// instruction 1.9, an LDS read 4.6 (each measured in a loop on all CUs).
// Sweeps of the three rates by 10 % and of the edge and item terms from 0 to
// twice moved passes over 30,000 x 1,000, 1,000 x 500 and 1,000 x 16,384
// samples by less than 1 %.
static constexpr double kTileCycles[kSplitVariants] = {185.0, 228.0, 272.0};
static constexpr double kEdgeCycles = 50.0;
static constexpr double kItemRowCycles = 400.0;
static constexpr double kSeriesRowCycles = 1000.0;  // series-lane: an item's stores per 32 series

// Weights whose parts would leave the normal range of bf16 stay on the fp32
// items.
static constexpr float kMinWeight = 0x1p-64f, kMaxWeight = 0x1p64f;

// The kernels scale a tap's series index to bytes (by 4, in the series-lane
// layout by 256) before they clamp it.  With at most 65,535 outputs and
// dilations up to here an index stays below 2^21 in magnitude, its bytes
// below 2^29; kernels beyond stay on the fp32 items, which clamp first.
static constexpr int32_t kMaxDilation = 1 << 16;

static uint16_t bf16_rn(float x) {
    uint32_t u;
    std::memcpy(&u, &x, 4);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
static float bf16_value(uint16_t b) {
    const uint32_t u = (uint32_t)b << 16;
    float x;
    std::memcpy(&x, &u, 4);
    return x;
}
// x = p[0] + p[1] + p[2] exactly (each remainder is exact in fp32)
static void split3(float x, uint16_t p[3]) {
    p[0] = bf16_rn(x);
    const float r = x - bf16_value(p[0]);
    p[1] = bf16_rn(r);
    p[2] = bf16_rn(r - bf16_value(p[1]));
}

// Samples below 2^-110 lose bits in the split (the third part's last bits
// fall below 2^-133, the smallest bf16), at most 2^-134 each; a sum of such
// products alone rounds at 2^-149 several times.  Neither shows beside a bias
// of at least 2^-100 of the weights' sum, whose own rounding is 2^9 times
// larger; kernels with smaller biases (zero among them) stay on fp32 items.
static bool bias_carries(const rocket_kernels *k, int32_t i) {
    float sum = 0.0f;
    for (int32_t j = 0; j < k->length[i]; ++j) sum += std::fabs(k->weights[(int64_t)i * k->max_len + j]);
    return std::fabs(k->bias[i]) >= 0x1p-100f * std::max(1.0f, sum);
}

static int64_t outputs(const rocket_kernels *k, int32_t i, int64_t L) {
    return L + 2 * (int64_t)k->padding[i] - (int64_t)(k->length[i] - 1) * k->dilation[i];
}

bool split_eligible(const rocket_kernels *k, int32_t L) {
    if (k->n_channels > 1) return false;
    for (int32_t i = 0; i < k->n_kernels; ++i) {
        if (outputs(k, i, L) > kSplitMaxOutputs || k->dilation[i] > kMaxDilation) return false;
        for (int32_t j = 0; j < k->length[i]; ++j) {
            const float w = std::fabs(k->weights[(int64_t)i * k->max_len + j]);
            if (w != 0.0f && !(w >= kMinWeight && w <= kMaxWeight)) return false;
        }
    }
    return true;
}

namespace {

struct Row {
    int32_t k;
    int32_t v;  // variant of its own length
    int32_t O;  // at most kSplitMaxOutputs
    float bias;
};

struct Group {
    int variant = 0;
    std::vector<int32_t> slot;    // kernel ids, at most kSplitRows
    int64_t widths[4] = {};       // the different O of its kernels
    int n_widths = 0;
    int64_t n_cols = 0, o_min = 0;
    double cost = 0.0;
};

// The blocks of `block` columns whose rows are all valid and whose reads stay
// within `margin` zeros around the series.
void group_bounds(const Group &g, int32_t L, int32_t d, bool even, int32_t reach, int margin, int block, int64_t *s0,
                  int64_t *lo, int64_t *hi) {
    const int frame = kSplitFrame[g.variant];
    // lo + hi of every row's range of frame-tap-0 indices
    *s0 = ((int64_t)L - (int64_t)(even ? frame - 2 : frame - 1) * d - g.n_cols) / 2;
    const int64_t in_lo = (g.n_cols - g.o_min) / 2, in_hi = in_lo + g.o_min;
    const int64_t first = std::max<int64_t>(in_lo, -(int64_t)margin - *s0);
    const int64_t last = std::min<int64_t>(in_hi - 1, (int64_t)L + margin - 1 - *s0 - (int64_t)reach * d);
    const int64_t n_blocks = (g.n_cols + block - 1) / block;
    *lo = std::min(n_blocks, first <= 0 ? 0 : (first + block - 1) / block);
    *hi = last < block - 1 ? 0 : (last + 1) / block;
    if (*hi <= *lo) *lo = *hi = n_blocks;
}

// Cut rows (in the given order) into groups of at most 32 rows and as many
// widths as the group's variant can mask.
// (out null: only their cost).
void cut(const Row *rows, size_t n, int32_t L, int32_t d, bool even, std::vector<Group> *out, double &cost) {
    Group g;
    size_t first = 0;  // the group's rows are first .. i - 1
    auto flush = [&](size_t end) {
        if (first == end) return;
        int64_t s0, lo, hi;
        if (L <= kSeriesMaxL) {
            // series-lane: a tile is one position of 32 series
            group_bounds(g, L, d, even, kSplitFrame[g.variant] - 1, kSplitSeriesMargin, 2, &s0, &lo, &hi);
            g.cost = ((double)g.n_cols * kTileCycles[g.variant] + (double)(g.n_cols - 2 * (hi - lo)) * kEdgeCycles +
                      kSeriesRowCycles) / kSplitTile;
        } else {
            group_bounds(g, L, d, even, kSplitFrame[g.variant] - 1, kSplitMargin, kSplitBlock, &s0, &lo, &hi);
            const int64_t tiles = (g.n_cols + kSplitTile - 1) / kSplitTile;
            const int64_t clean = 2 * (hi - lo);
            g.cost = (double)tiles * kTileCycles[g.variant] + (double)(tiles - std::min(tiles, clean)) * kEdgeCycles +
                     kItemRowCycles;
        }
        cost += g.cost;
        if (out) {
            for (size_t i = first; i < end; ++i) g.slot.push_back(rows[i].k);
            out->push_back(std::move(g));
            g.slot = std::vector<int32_t>();
        }
        g.variant = g.n_widths = 0;
        first = end;
    };
    for (size_t i = 0; i < n; ++i) {
        const Row &r = rows[i];
        // (rows of one width mostly follow each other)
        int64_t *end = g.widths + g.n_widths;
        bool known = g.n_widths > 0 && (end[-1] == r.O || std::find(g.widths, end, r.O) != end);
        if (i - first == (size_t)kSplitRows || (!known && g.n_widths == kSplitWidths[std::max(g.variant, r.v)])) {
            flush(i);
            known = false;
        }
        if (first == i) g.n_cols = g.o_min = r.O;
        if (!known) {
            g.widths[g.n_widths++] = r.O;
            g.n_cols = std::max<int64_t>(g.n_cols, r.O);
            g.o_min = std::min<int64_t>(g.o_min, r.O);
        }
        g.variant = std::max(g.variant, r.v);
    }
    flush(n);
}

// The same of a group's kernels as fp32 items: 4-kernel MFMA groups and VALU
// items for the rest, per (length class, O).  kFp32Factor: measured time over
// these issue cycles, relative to the split items' (1.3-1.5 times; passes are
// 2.5 % faster with it and flat from 1.15 to 1.5).
constexpr double kFp32Factor = 1.3;

double fp32_cycles(const Group &g, const rocket_kernels *k, int64_t L) {
    int n[kSplitVariants][4] = {};
    for (int32_t i : g.slot)
        ++n[ell_index_for(k->length[i])][std::find(g.widths, g.widths + g.n_widths, outputs(k, i, L)) - g.widths];
    double c = 0.0;
    for (int e = 0; e < kSplitVariants * 4; ++e) {
        const int count = n[e / 4][e % 4];
        const double ell = kEllValues[e / 4];
        const int full = count / 4, rest = count % 4;
        if (L <= kSeriesMaxL) {
            // series-lane MFMA items: 2 vector instructions to fold a register
            c += (double)((count + 3) / 4 * g.widths[e % 4]) / kTile * (ell * 8.7 + 36.0);
            continue;
        }
        const double tiles = (double)((g.widths[e % 4] + kTile - 1) / kTile);
        double t = full * (ell * 8.7 + 27.0);
        if (rest == 3) t += ell * 8.7 + 27.0;
        if (rest == 1 || rest == 2) t += rest * (ell * 4.5 + 6.75);
        c += tiles * t + 25.0 * count;
    }
    return kFp32Factor * c;
}

}  // namespace

// The kernels of one dilation and length parity, grouped in the cheapest of a
// few ways: lengths apart or together (a short kernel in a longer frame), rows
// of all widths together or apart.  Small dilations have many kernels of
// nearly the same O and run best with lengths apart; at large ones an item is
// filled only by everything the dilation has.
static std::vector<Group> best_groups(const std::vector<Row> &rows, int32_t L, int32_t d, bool even) {
    // which variants run together (bit masks): {7}{9}{11}, {7,9,11}, {7}{9,11}, {7,9}{11}
    static const int kParts[4][kSplitVariants] = {{1, 2, 4}, {7, 0, 0}, {1, 6, 0}, {3, 4, 0}};
    // longest frame first, or widest first
    if (rows.empty()) return {};
    std::vector<Row> order[2] = {rows, rows}, sel;
    std::stable_sort(order[0].begin(), order[0].end(),
                     [](const Row &a, const Row &b) { return a.v != b.v ? a.v > b.v : a.O > b.O; });
    std::stable_sort(order[1].begin(), order[1].end(),
                     [](const Row &a, const Row &b) { return a.O != b.O ? a.O > b.O : a.v > b.v; });
    // how 2: widest first, a group boundary wherever O changes
    auto run = [&](int mask, int how, std::vector<Group> *out) {
        double cost = 0.0;
        const std::vector<Row> &all = order[how == 0 ? 0 : 1];
        const Row *r = all.data();
        size_t n = all.size();
        if (mask != 7) {
            sel.clear();
            for (const Row &x : all)
                if ((mask >> x.v) & 1) sel.push_back(x);
            r = sel.data();
            n = sel.size();
        }
        for (size_t i = 0; i < n;) {
            size_t j = how == 2 ? i : n;
            while (j < n && r[j].O == r[i].O) ++j;
            cut(r + i, j - i, L, d, even, out, cost);
            i = j;
        }
        return cost;
    };
    int best_part = 1, best_how = 0;
    // (a handful of kernels makes one group or none)
    if (rows.size() > 6) {
        double best = -1.0, known[3][8];
        std::fill(&known[0][0], &known[0][0] + 24, -1.0);
        for (int part = 0; part < 4; ++part)
            for (int how = 0; how < 3; ++how) {
                double c = 0.0;
                for (int mask : kParts[part]) {
                    if (mask == 0) continue;
                    // one variant: both orders are the same
                    double &k = known[how == 1 && (mask & (mask - 1)) == 0 ? 0 : how][mask];
                    if (k < 0.0) k = run(mask, how, nullptr);
                    c += k;
                }
                if (best < 0.0 || c < best) {
                    best = c;
                    best_part = part;
                    best_how = how;
                }
            }
    }
    std::vector<Group> out;
    for (int mask : kParts[best_part])
        if (mask) run(mask, best_how, &out);
    return out;
}

// The bf16 pair of (plane word, weight part) slots: word 0 = (x1, x2) and
// word 1 = (x3, x1).
static uint32_t pair16(uint32_t lo, uint32_t hi) { return lo | (hi << 16); }

// The fragment whose dword 3 is the mask slot.
static constexpr int kSplitMaskFrag[kSplitVariants] = {0, 2, 1};

static void add_item(SplitPlan &P, const Group &g, const rocket_kernels *k, int32_t L, int32_t d, bool even) {
    const int frame = kSplitFrame[g.variant], nf = kSplitFrags[g.variant];
    SplitItem it;
    std::memset(&it, 0, sizeof(it));
    it.variant = g.variant;
    it.d = d;
    it.n_cols = (int32_t)g.n_cols;
    it.n_rows = (int32_t)g.slot.size();
    it.a_off = (int32_t)(P.a.size() / 4);
    it.r_off = (int32_t)P.kid.size();
    // negated weights (the accumulators hold -y, see the kernel), split, by
    // matrix row and frame tap
    uint16_t w[kSplitRows][12][3] = {};
    std::vector<float> cinit(kSplitRows, 0.0f);  // [half][reg]
    std::array<int, kSplitRows> cls{};           // the row's width, by matrix row; -1 = empty
    cls.fill(-1);
    for (int i = 0; i < g.n_widths; ++i) it.width[i] = (int32_t)g.widths[i];
    std::vector<float> div_O(2 * kSplitRows);
    for (int q = 0; q < kSplitRows; ++q) {
        const int32_t kk = q < (int)g.slot.size() ? g.slot[q] : -1;
        P.kid.push_back(kk);
        const int64_t O = kk >= 0 ? outputs(k, kk, L) : 1;
        P.inv_O.push_back(1.0 / (double)O);
        div_O[(q & 1) * kSplitRows + q / 2 * 2] = (float)O;
        div_O[(q & 1) * kSplitRows + q / 2 * 2 + 1] = 1.0f / (float)O;
        if (kk < 0) continue;
        const int len = k->length[kk], f = (frame - len) / 2;
        for (int j = 0; j < len; ++j) {
            uint16_t p[3];
            split3(-k->weights[(int64_t)kk * k->max_len + j], p);
            std::copy(p, p + 3, w[split_matrix_row(q)][f + j]);
            it.reach = std::max(it.reach, f + j);
        }
        cinit[(q & 1) * (kSplitRows / 2) + q / 2] = -k->bias[kk];
        cls[split_matrix_row(q)] = (int)(std::find(g.widths, g.widths + g.n_widths, outputs(k, kk, L)) - g.widths);
    }
    int64_t s0, lo, hi;
    group_bounds(g, L, d, even, it.reach, kSplitMargin, kSplitBlock, &s0, &lo, &hi);
    it.s0 = (int32_t)s0;
    it.clean_lo = (int32_t)lo;
    it.clean_hi = (int32_t)hi;
    group_bounds(g, L, d, even, it.reach, kSplitSeriesMargin, 2, &s0, &lo, &hi);
    it.series_lo = (int32_t)lo;
    it.series_hi = (int32_t)hi;
    it.cost = (int32_t)std::min(g.cost, 1e9);
    // fragments in the order of the kernel's MFMAs, dword i of lane (matrix
    // row m, half h).  The main words' taps are 4 h + i; the tail is taps 8 up.
    enum Kind { kZero, kW13, kW22, kW11, kMask };  // x3 w1 + x1 w3, (x1 + x2) w2, (x1 + x2) w1
    P.a.resize(P.a.size() + (size_t)nf * kWave * 4);
    uint32_t *dst = P.a.data() + P.a.size() - (size_t)nf * kWave * 4;
    for (int fr = 0; fr < nf; ++fr)
        for (int h = 0; h < 2; ++h) {
            // the parts of each dword (frame tap 11 holds zeros)
            int taps[4], lo[4], hi[4];
            bool masked = false;
            for (int i = 0; i < 4; ++i) {
                Kind kind = kZero;
                int tap = 4 * h + i;
                if (fr == kSplitMaskFrag[g.variant] && i == 3 && (g.variant > 0 || h == 1)) {
                    kind = kMask;
                } else if (fr == 0) {
                    kind = kW13;
                } else if (fr == nf - 1) {
                    kind = kW11;
                } else if (fr == (g.variant == 2 ? 2 : 1)) {
                    kind = kW22;
                } else if (g.variant == 1) {
                    // tail: half 0 word 0 of tap 8 by w2, word 1; half 1 word 0 by w1
                    if (i == 0) kind = h == 0 ? kW22 : kW11;
                    if (i == 2 && h == 0) kind = kW13;
                    tap = 8;
                } else {
                    // tail: taps 8 + i, half 0 word 0 (by w2, then w1), half 1 word 1
                    if (fr == 1) kind = h == 0 ? kW22 : kW13;
                    if (fr == 3 && h == 0) kind = kW11;
                    tap = 8 + i;
                }
                masked = masked || kind == kMask;
                taps[i] = kind == kZero || kind == kMask ? 11 : tap;
                lo[i] = kind == kW22 ? 1 : 0;
                hi[i] = kind == kW13 ? 2 : lo[i];
            }
            const int c0 = g.variant > 0 ? 2 * h : 0;  // the mask slot's first width
            uint32_t *out = dst + ((size_t)fr * kWave + 32 * h) * 4;
            for (int m = 0; m < kSplitRows; ++m, out += 4) {
                for (int i = 0; i < 4; ++i) out[i] = pair16(w[m][taps[i]][lo[i]], w[m][taps[i]][hi[i]]);
                if (masked) out[3] = pair16(cls[m] == c0 ? kSplitMask : 0u, cls[m] == c0 + 1 ? kSplitMask : 0u);
            }
        }
    P.cinit.insert(P.cinit.end(), cinit.begin(), cinit.end());
    P.div_O.insert(P.div_O.end(), div_O.begin(), div_O.end());
    P.items.push_back(it);
    P.cost += g.cost;
}

// Kernels that fp32 items run faster are left to them only where that saves
// this share of the pass (they stage the series again, in workgroups or a
// launch of their own).
static constexpr double kRestMinGain = 0.02;
// Short series take split items below this share of the fp32 items' cost: 300
// kernels x 100 samples (0.8) run 5,000 to 100,000 series at 0.79 to 0.91 of
// the fp32 items' speed but 1,000 (tiled) at 1.6, 500 x 128 (0.69) 1.07 to 1.24.
static constexpr double kShortGain = 0.85;
// Sets of few kernels leave the wavefronts of a split workgroup without items
// (it stages its series for each of three variants), and their rest is most of
// the work.  Speed against the fp32 plan of the whole set at 100,000 / 1,000 /
// 100 / 16 series, by model gain: 100 kernels x 2,000 samples (1.03) 1.00 / 0.74
// / 1.07 / 1.06, 100 x 300 (1.06) 1.10 / 0.84 / 0.98 / 1.12, 150 x 500 (1.07)
// 1.12 / 0.89 / 1.14 / 1.29, 200 x 300 (1.16) 1.12 / 0.80 / 1.16 / 1.20, 300 x
// 1,000 (1.11) 1.12 / 0.81 / 1.33 / 1.41, 500 x 500 (1.26) 1.19 / 1.03 / 1.12 /
// 1.19: the line lies where many series break even; about 1,000 series of the
// smallest sets stay slower, as their fp32 items run beside split workgroups
// that are too few to fill the chip.  With MPV (two wavefronts per SIMD) more is
// needed, and 20 items: 300 x 500 (6 items, 1.16) 0.91 / 0.68 / 0.90, 500 x 500
// (13, 1.26) 1.03 / 0.79 / 0.89, 1,000 x 2,000 (22, 1.22) 1.04 / 1.02 / 0.81,
// 1,000 x 500 (27, 1.42) 1.12 / 0.96 / 0.98, 2,000 x 5,000 (1.27) 1.08 / 1.06 /
// 1.02.  Above 10,000 samples any split items pay with many series (150 kernels
// 1.07, 1,000 kernels 1.05 at 16,000 samples; 200 x 12,000 1.27).
static constexpr double kSplitMinGain = 1.04, kSplitMinGainMpv = 1.25;
static constexpr size_t kSplitMinItemsMpv = 20;

bool split_pays(const SplitPlan &P, bool mpv) {
    if (P.items.empty()) return false;
    if (P.L <= kSeriesMaxL || P.L > 10000) return true;
    return P.items.size() >= (mpv ? kSplitMinItemsMpv : 1) &&
           P.fp32_cost >= (mpv ? kSplitMinGainMpv : kSplitMinGain) * (P.cost + P.rest_cost);
}

rocket_status build_split_plan(const rocket_kernels *k, int32_t L, SplitPlan *out) {
    try {
        SplitPlan P;
        P.L = L;
        // the kernels of a dilation and length parity, those that split items
        // take apart from the others (dilations are at most kMaxDilation)
        struct Dil {
            int32_t d;
            bool even;
            std::vector<Row> rows, fp32_only;
        };
        int32_t d_max = 0;
        for (int32_t i = 0; i < k->n_kernels; ++i) d_max = std::max(d_max, k->dilation[i]);
        std::vector<int32_t> n_of(2 * ((size_t)d_max + 1), 0), at(n_of.size(), -1);
        for (int32_t i = 0; i < k->n_kernels; ++i) ++n_of[2 * k->dilation[i] + (k->length[i] % 2 == 0)];
        std::vector<Dil> dils;
        for (size_t c = 0; c < n_of.size(); ++c) {
            if (n_of[c] == 0) continue;
            at[c] = (int32_t)dils.size();
            dils.push_back(Dil{(int32_t)(c / 2), c % 2 != 0, {}, {}});
            dils.back().rows.reserve(n_of[c]);
        }
        for (int32_t i = 0; i < k->n_kernels; ++i) {
            Dil &e = dils[at[2 * k->dilation[i] + (k->length[i] % 2 == 0)]];
            (bias_carries(k, i) ? e.rows : e.fp32_only)
                .push_back(Row{i, ell_index_for(k->length[i]), (int32_t)outputs(k, i, L), k->bias[i]});
        }
        // by their own numbers (a total order but for equal kernels), so that a
        // kernel's item, and with it the rounding of its dot products, does not
        // depend on the set's order
        auto before = [&](const Row &x, const Row &y) {
            if (x.bias != y.bias) return x.bias < y.bias;
            if (k->length[x.k] != k->length[y.k]) return k->length[x.k] < k->length[y.k];
            if (x.O != y.O) return x.O < y.O;
            const float *wx = k->weights + (int64_t)x.k * k->max_len, *wy = k->weights + (int64_t)y.k * k->max_len;
            const auto d = std::mismatch(wx, wx + k->length[x.k], wy);
            return d.first != wx + k->length[x.k] ? *d.first < *d.second : x.k < y.k;
        };
        std::vector<int64_t> buckets;
        for (Dil &e : dils) {
            buckets.clear();
            for (const auto *rows : {&e.rows, &e.fp32_only})
                for (const Row &r : *rows) buckets.push_back((int64_t)r.O * 16 + k->length[r.k]);  // these give the padding
            std::sort(buckets.begin(), buckets.end());
            P.n_buckets += std::unique(buckets.begin(), buckets.end()) - buckets.begin();
            std::sort(e.rows.begin(), e.rows.end(), before);
        }
        struct Choice {
            int32_t d;
            bool even;
            Group g;
            double fp32;
        };
        std::vector<Choice> all;
        double total = 0.0, gain = 0.0;
        for (const Dil &e : dils) {
            for (Group &g : best_groups(e.rows, L, e.d, e.even)) {
                const double c = fp32_cycles(g, k, L);
                total += std::min(g.cost, c);
                P.fp32_cost += c;
                gain += std::max(0.0, g.cost - c);
                all.push_back(Choice{e.d, e.even, std::move(g), c});
            }
            for (const Group &g : best_groups(e.fp32_only, L, e.d, e.even)) {
                P.rest.insert(P.rest.end(), g.slot.begin(), g.slot.end());
                const double c = fp32_cycles(g, k, L);
                P.rest_cost += c;
                P.fp32_cost += c;
            }
        }
        // short series: all kernels or none (the series-lane layout runs one
        // kind of item), by the total
        if (L <= kSeriesMaxL && !P.rest.empty()) all.clear();
        if (L <= kSeriesMaxL) {
            double split = 0.0, fp32 = 0.0;
            for (const Choice &c : all) {
                split += c.g.cost;
                fp32 += c.fp32;
            }
            if (split > kShortGain * fp32) all.clear();
        }
        const bool leave = L > kSeriesMaxL && gain > kRestMinGain * total;
        size_t words = 0;
        for (const Choice &c : all) words += (size_t)kSplitFrags[c.g.variant] * kWave * 4;
        P.a.reserve(words);
        for (const Choice &c : all) {
            if (leave && c.fp32 < c.g.cost) {
                P.rest.insert(P.rest.end(), c.g.slot.begin(), c.g.slot.end());
                P.rest_cost += c.fp32;
            } else {
                add_item(P, c.g, k, L, c.d, c.even);
            }
        }
        std::sort(P.rest.begin(), P.rest.end());
        std::vector<int32_t> variant, cost;
        for (const SplitItem &it : P.items) {
            variant.push_back(it.variant);
            cost.push_back(it.cost);
        }
        order_items(variant, cost, kSplitVariants, P.order, P.split_begin, P.layout_off);
        *out = std::move(P);
        return ROCKET_OK;
    } catch (const std::bad_alloc &) {
        return ROCKET_ERR_OOM;
    } catch (...) {
        return ROCKET_ERR_INTERNAL;
    }
}

}  // namespace rocket
