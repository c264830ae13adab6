// Host replay of a split plan: its items walked as the kernels walk them, in
// 64 bits, against direct dot products.
#include <cmath>
#include <cstring>
#include <limits>
#include <set>
#include <vector>

#include "rocket_internal.h"

using namespace rocket;

static float bf(uint32_t h) {
    const uint32_t u = h << 16;
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}
static uint32_t rn(float x) {
    uint32_t u;
    std::memcpy(&u, &x, 4);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
static double dot2(uint32_t a, uint32_t b) {
    return (double)bf(a & 0xffffu) * bf(b & 0xffffu) + (double)bf(a >> 16) * bf(b >> 16);
}

// 0: everything agrees; otherwise the number of the check that failed, with
// the kernel in *where.  series: the series-lane layout's blocks and margins.
// *forms: bit 0 an item of three or more widths, bit 1 of several lengths, bit
// 2 of even lengths, bit 3 with a kernel of at most two outputs.
extern "C" int split_replay(const rocket_kernels *k, int32_t L, const float *x, int32_t series, int32_t *where,
                            int32_t *n_items, int32_t *forms) {
    *where = -1;
    *n_items = *forms = 0;
    if (!split_eligible(k, L)) return 1;
    SplitPlan P;
    if (build_split_plan(k, L, &P) != ROCKET_OK) return 2;
    *n_items = (int32_t)P.items.size();
    std::vector<int> seen(k->n_kernels, 0);
    for (int32_t i : P.rest) ++seen[i];
    for (int32_t i : P.kid)
        if (i >= 0) ++seen[i];
    for (int32_t i = 0; i < k->n_kernels && *n_items > 0; ++i)
        if (seen[*where = i] != 1) return 3;
    // biases that could not hide what the split loses of tiny samples
    for (int32_t i : P.kid)
        if (i >= 0 && !(std::fabs(k->bias[*where = i]) >= 0x1p-100f)) return 11;
    // every layout of the orders holds every item once, under its own variant
    for (int li = 0; li < kNumSplitLayouts; ++li) {
        const int32_t *sb = P.split_begin.data() + P.layout_off[li];
        std::vector<int> used(P.items.size(), 0);
        for (int v = 0; v < kSplitVariants; ++v)
            for (int32_t j = sb[v * kSplitCounts[li]]; j < sb[(v + 1) * kSplitCounts[li]]; ++j)
                if (P.items[P.order[j]].variant != v || used[P.order[j]]++) return 4;
        for (int u : used)
            if (u != 1) return 4;
    }
    std::vector<uint32_t> word[2];
    for (int32_t t = 0; t < L; ++t) {
        const uint32_t p1 = rn(x[t]), p2 = rn(x[t] - bf(p1)), p3 = rn(x[t] - bf(p1) - bf(p2));
        if (bf(p1) + (double)bf(p2) + bf(p3) != x[t]) return 5;
        word[0].push_back(p1 | p2 << 16);
        word[1].push_back(p3 | p1 << 16);
    }
    const int tile = series ? 1 : kSplitTile, block = 2 * tile, margin = series ? kSplitSeriesMargin : kSplitMargin;
    for (const SplitItem &it : P.items) {
        std::set<int64_t> widths, lengths;
        for (int q = 0; q < it.n_rows; ++q) {
            const int32_t kk = P.kid[it.r_off + q], len = k->length[kk];
            const int64_t O = (int64_t)L + 2 * (int64_t)k->padding[kk] - (int64_t)(len - 1) * k->dilation[kk];
            widths.insert(O);
            lengths.insert(len);
            *forms |= (len % 2 == 0 ? 4 : 0) | (O <= 2 ? 8 : 0);
        }
        *forms |= (widths.size() >= 3 ? 1 : 0) | (lengths.size() >= 2 ? 2 : 0);
        const int v = it.variant, nf = kSplitFrags[v];
        const int lo = series ? it.series_lo : it.clean_lo, hi = series ? it.series_hi : it.clean_hi;
        const int n_blocks = (it.n_cols + block - 1) / block;
        if (lo < 0 || hi > n_blocks || lo > hi) return 6;
        std::vector<double> mn(kSplitRows, std::numeric_limits<double>::infinity());
        std::vector<int64_t> cnt(kSplitRows, 0);
        for (int b = 0; b < n_blocks; ++b)
            for (int u = 0; u < (it.n_cols - b * block > tile ? 2 : 1); ++u)
                for (int n = 0; n < tile; ++n) {
                    const bool edge = b < lo || b >= hi;
                    bool outside = false;
                    auto at = [&](int plane, int tap) -> uint32_t {
                        // bytes in the kernel's 32 bits, as it scales and clamps them
                        const int scale = 4 * (series ? kWave : 1);
                        int32_t a = (int32_t)((uint32_t)scale * ((uint32_t)it.s0 + (uint32_t)n +
                                                                 (uint32_t)std::min(tap, it.reach) * (uint32_t)it.d));
                        a = (int32_t)((uint32_t)a + (uint32_t)(b * block * scale));
                        if (edge) a = std::min(std::max(a, -margin * scale), L * scale);
                        const int64_t i = a / scale + u * tile;
                        outside |= i < -margin || i >= (int64_t)L + margin;
                        return i < 0 || i >= L ? 0u : word[plane][i];
                    };
                    uint32_t fr[5][2][4];  // the words under each fragment
                    for (int h = 0; h < 2; ++h) {
                        const int64_t off = 2 * ((int64_t)b * block + u * tile + n) + 1 - it.n_cols;
                        const int64_t dist = std::max(off, -off);
                        const int w = v > 0 && h ? 2 : 0;
                        const uint32_t mask = !edge ? 0u : (dist < it.width[w] ? 0u : kSplitMask) |
                                                               (dist < it.width[w + 1] ? 0u : kSplitMask << 16);
                        uint32_t b0[4], b1[4], bt[4] = {};
                        for (int i = 0; i < 4; ++i) {
                            const bool idle = v == 0 && h == 1 && i == 3;
                            b0[i] = idle ? 0u : at(0, 4 * h + i);
                            b1[i] = idle ? mask : at(1, 4 * h + i);
                        }
                        if (v == 1) {
                            bt[0] = at(0, 8);
                            bt[2] = at(1, 8);
                        }
                        for (int i = 0; i < 3 && v == 2; ++i) bt[i] = at(h, 8 + i);
                        if (v > 0) bt[3] = mask;
                        const uint32_t *use[3][5] = {{b1, b0, b0}, {b1, b0, bt, b0}, {b1, bt, b0, bt, b0}};
                        for (int f = 0; f < nf; ++f) std::memcpy(fr[f][h], use[v][f], sizeof(b0));
                    }
                    if (outside) return 7;
                    for (int q = 0; q < it.n_rows; ++q) {
                        const int m = split_matrix_row(q);
                        double z = P.cinit[it.r_off + (q & 1) * 16 + q / 2];
                        for (int f = 0; f < nf; ++f)
                            for (int h = 0; h < 2; ++h)
                                for (int i = 0; i < 4; ++i)
                                    z += dot2(P.a[4 * ((size_t)it.a_off + f * kWave + 32 * h + m) + i], fr[f][h][i]);
                        if (z > 1e50) continue;  // masked (2^200 here, infinity in 32 bits)
                        mn[q] = std::min(mn[q], z);
                        cnt[q] += z < 0.0;
                    }
                }
        for (int q = 0; q < it.n_rows; ++q) {
            const int32_t kk = *where = P.kid[it.r_off + q];
            const int len = k->length[kk], d = k->dilation[kk], p = k->padding[kk];
            const int64_t O = (int64_t)L + 2 * p - (int64_t)(len - 1) * d;
            int64_t least = 0, most = 0;
            double mx = -std::numeric_limits<double>::infinity(), slack = 0.0;
            for (int64_t t = 0; t < O; ++t) {
                double y = k->bias[kk], mag = 0.0;
                for (int j = 0; j < len; ++j) {
                    const int64_t i = t - p + (int64_t)j * d;
                    if (i < 0 || i >= L) continue;
                    const double w = k->weights[(int64_t)kk * k->max_len + j];
                    y += w * x[i];
                    mag += std::fabs(w * x[i]);
                }
                // the part products left out: x2 w3 and x3 w2 are at most 2^-24
                // of the product each, x3 w3 2^-32
                const double e = mag * 0x1p-22;
                least += y > e;
                most += y > -e;
                mx = std::max(mx, y);
                slack = std::max(slack, e);
            }
            if (cnt[q] < least || cnt[q] > most) return 8;
            if (!(std::fabs(-mn[q] - mx) <= slack)) return 9;
            if (P.inv_O[it.r_off + q] != 1.0 / (double)O) return 10;
        }
    }
    return 0;
}

// The slot of every kernel (-1: left to fp32 items).
extern "C" int split_places(const rocket_kernels *k, int32_t L, int32_t *place) {
    SplitPlan P;
    if (build_split_plan(k, L, &P) != ROCKET_OK) return 2;
    for (int32_t i = 0; i < k->n_kernels; ++i) place[i] = -1;
    for (size_t q = 0; q < P.kid.size(); ++q)
        if (P.kid[q] >= 0) place[P.kid[q]] = (int32_t)q;
    return 0;
}
