// Split items of the ROCKET transform on CDNA4 (gfx950): fp32 dot products on
// the bf16 matrix instruction, each fp32 factor split into three bf16 parts.
//
// One workgroup = a few series x one split of the items of one code variant
// (as the fused fp32 kernel).  The series are staged into LDS as two 32-bit
// words per position, (x1, x2) and (x3, x1), the bf16 parts of x.  An item is
// up to 32 kernels of one dilation (the 32 matrix rows; see SplitItem); a
// wavefront runs it over blocks of two tiles of 32 consecutive positions (the
// 32 matrix columns).  The contraction index of v_mfma_f32_32x32x16_bf16 has
// two halves of 8: a lane half holds 4 words, so one instruction sums, for 8
// (tap, word) pairs, both 16-bit halves of each word times its pair of weight
// parts: (x1 + x2) w1, (x1 + x2) w2 or x3 w1 + x1 w3.
//
// Why: an fp32 MFMA does 256 multiply-adds in 8.7 cycles and no vector
// instruction of its SIMD runs beside it; this one does 16,384 in 32 cycles,
// of which about 22 are left to vector instructions of other wavefronts
// (measured: 6 v_max3 beside each, 34.9 cycles).  With 24 of the 32 products
// of a word pair used, a dot product costs 96 (7 taps) to 160 (11 taps) cycles
// per 1,024 outputs against 280 to 383, and the fold of the results (20 vector
// instructions per 1,024 outputs) runs under it.
//
// Rounding: the instruction adds the 8 products of a lane half and the
// accumulator exactly up to 2^-24 of the largest product and rounds once, so
// the small parts go first (rounded at the bias's magnitude) and the x w1
// products last, 8 taps in two steps: fewer roundings of the full sum than an
// fp32 chain's one per tap (rms error against 64 bits 0.79 to 0.85 of the
// chain's at 11 and 9 taps).
//
// The accumulators hold -y (the packed weights and biases are negated), so a
// positive y is a set sign bit: one v_perm collects the signs of two rows as
// 16-bit masks and one v_add3 counts two of those, 0.75 instructions per
// result register, and MAX is a running minimum (v_min3, half an
// instruction).  No result is -0: no bias is zero, and a sum that cancels
// gives +0.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <mutex>
#include <new>

#include "split_launch.h"
#include "tiles.h"

using rocket::SplitItem;

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const volatile uint32_t lds_word;
typedef __attribute__((address_space(3))) uint32_t lds_out;

namespace {

constexpr int kRegs = 16;       // result registers of a tile
constexpr int kMargin = rocket::kSplitMargin;
constexpr int kEndZeros = 2 * rocket::kSplitBlock;  // zeros after the last row: its margin, and the mask slot's reads
constexpr uint32_t kSignPair = 0x0b0b0909u;  // v_perm: sign of S1 twice, sign of S0 twice

struct SplitArgs {
    const float *X;
    float *F;
    int64_t row0, n_rows;
    int32_t L, K;
    const SplitItem *items;
    const uint32_t *a;
    const float *cinit;
    const int32_t *kid;
    const double *inv_O;
    const float *div_O;
    const int32_t *order;
    const int32_t *split_begin;
    int32_t nsplit, n_variants;
    int32_t variants[rocket::kSplitVariants];
    int32_t part_cap, part_even;  // see part_shift
    int32_t xcd_shift;  // as in FusedArgs
    int64_t groups_per_xcd;
    uint32_t blocks;      // workgroups of split items
    int32_t rows_per_block;
    int32_t pitch;        // words between staged rows: L + kMargin
    int32_t plane_words;  // words per plane
    int32_t vec4;         // rows are read 4 floats at a time (L a multiple of 4, X 16-byte aligned)
    float *S;             // series-lane layout: features in slot order, s_rows series per slot column
    int64_t s_rows;
    int64_t s_floats;     // floats of S (bounds of checked builds)
};

struct CheckBounds {
    uint32_t lds_hi;  // staged bytes from the start of the workgroup's LDS
    float *out_lo, *out_hi;
};

// The staged word at LDS byte address a.
__device__ __forceinline__ uint32_t lds_load(uint32_t a, const CheckBounds &cb) {
#if ROCKET_CHECKED
    if (a + 4 > cb.lds_hi) {
        atomicOr(&g_rocket_checks, kCheckLdsRead);
        a = 0;
    }
#endif
    (void)cb;
    return *(lds_word *)(__UINTPTR_TYPE__)a;
}

// bf16 parts of x, round to nearest even, as the two staged words.  Values
// that would round to an infinity are cut to the largest bf16 first.
__device__ __forceinline__ void split_words(float x, uint32_t &w0, uint32_t &w1) {
    constexpr float kBf16Max = 0x1.fep127f;
    const float c = __builtin_amdgcn_fmed3f(x, -kBf16Max, kBf16Max);
    const __bf16 x1 = (__bf16)c;
    const float r = x - (float)x1;
    const __bf16 x2 = (__bf16)r;
    const __bf16 x3 = (__bf16)(r - (float)x2);
    const uint32_t u1 = __builtin_bit_cast(uint16_t, x1), u2 = __builtin_bit_cast(uint16_t, x2),
                   u3 = __builtin_bit_cast(uint16_t, x3);
    w0 = u1 | (u2 << 16);
    w1 = u3 | (u1 << 16);
}

// Per-row accumulators of an item, per lane.
template <int MPV>
struct Acc {
    float mn[kRegs];            // running minimum of -y
    uint32_t cnt[kRegs / 2];    // sums of sign masks of rows (2 j, 2 j + 1) in the halves
    // sums of positive y in MPV chains, two of them one per tile of a block:
    // chains of O / 64 additions, as in the fp32 items (one chain of O / 32 had
    // up to 7 % more rounding error, at 16,384 samples; up to 128 samples it
    // has no more than the fp32 items, and two cost 5 to 9 % of a call)
    float ps[MPV == 2 ? 2 : 1][MPV ? kRegs : 1];
    // the sum of both chains
    __device__ __forceinline__ float sum(int i) const { return MPV == 2 ? ps[0][i] + ps[MPV == 2 ? 1 : 0][i] : ps[0][i]; }
};

// The word addresses of one block: LDS bytes of the lane's column in tile 0
// under its main taps (plane 0) and its tail taps.  (7-tap frames: main[3] of
// lane half 1 is the mask slot and points to zeros.)
template <int V>
struct Addr {
    uint32_t main[4];
    uint32_t tail[V == 2 ? 3 : 1];
};
constexpr int tail_addrs(int v) { return v == 0 ? 0 : (v == 1 ? 1 : 3); }

__device__ __forceinline__ v16f mfma(const v4u &a, const v4u &b, const v16f &c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0,
                                                   0);
}

// One block of NT tiles, FIRST blocks after the one the addresses stand for:
// the words, the MFMAs (small parts first) and the fold.  plane: bytes from
// plane 0 to plane 1; mask(u): the mask word of tile u (EDGE blocks; others
// have zeros in its slot).  STRIDE: bytes from one tile's words to the next's.
template <int V, int NT, int MPV, bool EDGE, int FIRST, int STRIDE, typename Mask>
__device__ __forceinline__ void block(const Addr<V> &ad, uint32_t plane, const v4u (&fa)[rocket::kSplitFrags[V]],
                                      const v16f &cinit, const Mask &mask, int h, Acc<MPV> &ac,
                                      const CheckBounds &cb) {
    v16f z[NT];
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        const uint32_t off = (uint32_t)STRIDE * (2u * FIRST + u);
        v4u b0, b1, bt = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            b0[i] = lds_load(ad.main[i] + off, cb);
            b1[i] = lds_load(ad.main[i] + plane + off, cb);
        }
        if constexpr (V == 1) {
            bt[0] = lds_load(ad.tail[0] + off, cb);
            bt[2] = lds_load(ad.tail[0] + plane + off, cb);
        }
        if constexpr (V == 2) {
#pragma unroll
            for (int i = 0; i < 3; ++i) bt[i] = lds_load(ad.tail[i] + off, cb);
        }
        if constexpr (V > 0 && EDGE) bt[3] = mask(u);
        if constexpr (V == 0 && EDGE) b1[3] = h ? mask(u) : b1[3];
        z[u] = mfma(fa[0], b1, cinit);
        if constexpr (V == 0) {
            z[u] = mfma(fa[1], b0, z[u]);
            z[u] = mfma(fa[2], b0, z[u]);
        } else if constexpr (V == 1) {
            z[u] = mfma(fa[1], b0, z[u]);
            z[u] = mfma(fa[2], bt, z[u]);
            z[u] = mfma(fa[3], b0, z[u]);
        } else {
            z[u] = mfma(fa[1], bt, z[u]);
            z[u] = mfma(fa[2], b0, z[u]);
            z[u] = mfma(fa[3], bt, z[u]);
            z[u] = mfma(fa[4], b0, z[u]);
        }
    }
#pragma unroll
    for (int j = 0; j < kRegs / 2; ++j) {
        uint32_t s[NT];
#pragma unroll
        for (int u = 0; u < NT; ++u)
            s[u] = __builtin_amdgcn_perm(__float_as_uint(z[u][2 * j + 1]), __float_as_uint(z[u][2 * j]), kSignPair);
        ac.cnt[j] += NT == 2 ? s[0] + s[NT - 1] : s[0];
    }
#pragma unroll
    for (int i = 0; i < kRegs; ++i) {
        ac.mn[i] = NT == 2 ? fminf(fminf(ac.mn[i], z[0][i]), z[NT - 1][i]) : fminf(ac.mn[i], z[0][i]);
        if constexpr (MPV > 0) {
#pragma unroll
            for (int u = 0; u < NT; ++u) ac.ps[u % MPV][i] += fmaxf(-z[u][i], 0.0f);
        }
    }
}

// Combining operations of the lane reductions.
struct OpMin {
    __device__ __forceinline__ static uint32_t f(uint32_t a, uint32_t b) {
        return __float_as_uint(fminf(__uint_as_float(a), __uint_as_float(b)));
    }
};
struct OpAdd {
    __device__ __forceinline__ static uint32_t f(uint32_t a, uint32_t b) { return a + b; }
};
struct OpFadd {
    __device__ __forceinline__ static uint32_t f(uint32_t a, uint32_t b) {
        return __float_as_uint(__uint_as_float(a) + __uint_as_float(b));
    }
};
template <typename Op, int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
    return Op::f(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true));
}
// 16-lane rows 0 and 2 of the result combine a over row pairs, rows 1 and 3 b.
template <typename Op>
__device__ __forceinline__ uint32_t fold_rows(uint32_t a, uint32_t b) {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    return Op::f(r[0], r[1]);
}
// Reduce N registers over each half's 32 lanes, halving registers and lanes
// together: afterwards lane bits 4, 3, 2, (1) select the register, most
// significant register bit first, and the other lane bits hold copies.
template <typename Op, int N>
__device__ __forceinline__ uint32_t tree(uint32_t (&v)[N], int lane) {
    static_assert(N == 16 || N == 8, "one bit of the register number per lane bit");
#pragma unroll
    for (int i = 0; i < N / 2; ++i) v[i] = fold_rows<Op>(v[i], v[i + N / 2]);
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        const uint32_t a = dpp<Op, kDppRowRor8>(v[i]), b = dpp<Op, kDppRowRor8>(v[i + N / 4]);
        v[i] = (lane & 8) ? b : a;
    }
#pragma unroll
    for (int i = 0; i < N / 8; ++i) {
        const uint32_t a = dpp<Op, kDppRowHalfMirror>(v[i]), b = dpp<Op, kDppRowHalfMirror>(v[i + N / 8]);
        v[i] = (lane & 4) ? b : a;
    }
    if constexpr (N == 16) {
        const uint32_t a = dpp<Op, kDppQuadSwap2>(v[0]), b = dpp<Op, kDppQuadSwap2>(v[1]);
        v[0] = (lane & 2) ? b : a;
    } else {
        v[0] = dpp<Op, kDppQuadSwap2>(v[0]);
    }
    return dpp<Op, kDppQuadSwap1>(v[0]);
}

// An item's A fragments and start values.
template <int V>
__device__ __forceinline__ void load_fragments(const SplitItem &it, const SplitArgs &a, int lane,
                                               v4u (&fa)[rocket::kSplitFrags[V]], v16f &cinit) {
#pragma unroll
    for (int f = 0; f < rocket::kSplitFrags[V]; ++f)
        fa[f] = reinterpret_cast<const v4u *>(a.a)[it.a_off + f * rocket::kWave + lane];
    const float4 *c4 = reinterpret_cast<const float4 *>(a.cinit + it.r_off + (lane >> 5) * kRegs);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float4 c = c4[i];
        cinit[4 * i] = c.x;
        cinit[4 * i + 1] = c.y;
        cinit[4 * i + 2] = c.z;
        cinit[4 * i + 3] = c.w;
    }
}

constexpr int kTileBytes = 4 * rocket::kSplitTile;

// One item over the staged series r0, r0 + r_step, ...
template <int V, int MPV>
__device__ __forceinline__ void run_split_item(const SplitItem &it, const SplitArgs &a, uint32_t lds0, uint32_t plane,
                                               int r0, int r_step, int nrows, float *F0, int lane,
                                               const CheckBounds &cb) {
    const int n = lane & 31, h = lane >> 5;
    v4u fa[rocket::kSplitFrags[V]];
    v16f cinit;
    load_fragments<V>(it, a, lane, fa, cinit);
    // the row this lane writes after the reductions (even lanes): register
    // bits 3..0 = lane bits 4..1
    const int reg = (((lane >> 4) & 1) << 3) | (((lane >> 3) & 1) << 2) | (((lane >> 2) & 1) << 1) | ((lane >> 1) & 1);
    const int okid = (lane & 1) ? -1 : a.kid[it.r_off + 2 * reg + h];
    const double inv_O = a.inv_O[it.r_off + 2 * reg + h];
    const int n_blocks = (it.n_cols + rocket::kSplitBlock - 1) / rocket::kSplitBlock;
    // series index of the lane's column under its taps, in bytes; the word
    // slots no tap uses (and those past the last weight, whose weights are
    // zero) repeat the last tap's words, or read zeros (the mask slot)
    int main0[4], tail0[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) main0[i] = 4 * (it.s0 + n + min(4 * h + i, it.reach) * it.d);
#pragma unroll
    for (int i = 0; i < 3; ++i) tail0[i] = 4 * (it.s0 + n + min(8 + i, it.reach) * it.d);
    constexpr int kUnroll = MPV ? 1 : 2;
    constexpr uint32_t kBlockBytes = 4u * rocket::kSplitBlock;
    constexpr uint32_t step = kUnroll * kBlockBytes;
    const bool idle = V == 0 && h == 1;  // main[3] is the mask slot: zeros, not advanced
    const uint32_t step3 = idle ? 0u : step;
    const int wa = (V > 0 && h) ? it.width[2] : it.width[0], wb = (V > 0 && h) ? it.width[3] : it.width[1];
    const int64_t f_stride = (int64_t)(MPV ? 3 : 2) * a.K;
    const uint32_t zero = lds0 + 4u * (uint32_t)(nrows * a.pitch + n);
    for (int r = r0; r < nrows; r += r_step) {
        const uint32_t row = lds0 + 4u * (uint32_t)(kMargin + r * a.pitch);  // series index 0
        const uint32_t row_tail = row + (V == 2 ? (uint32_t)h * plane : 0u);
        Acc<MPV> ac;
#pragma unroll
        for (int i = 0; i < kRegs; ++i) {
            ac.mn[i] = INFINITY;
            if (MPV) ac.ps[0][i] = 0.0f;
            if constexpr (MPV == 2) ac.ps[1][i] = 0.0f;
        }
#pragma unroll
        for (int j = 0; j < kRegs / 2; ++j) ac.cnt[j] = 0u;
        // blocks whose rows are not all valid, or whose reads leave the
        // margins: clamped addresses and masks
        auto edge = [&](int b) {
            const int c0 = b * rocket::kSplitBlock;
            auto clamped = [&](int i0) { return (uint32_t)min(max(i0 + 4 * c0, -4 * kMargin), 4 * a.L); };
            Addr<V> ad;
#pragma unroll
            for (int i = 0; i < 4; ++i) ad.main[i] = row + clamped(main0[i]);
            if (idle) ad.main[3] = zero;
#pragma unroll
            for (int i = 0; i < tail_addrs(V); ++i) ad.tail[i] = row_tail + clamped(tail0[i]);
            auto mask = [&](int u) {
                const int off = 2 * (c0 + rocket::kSplitTile * u + n) + 1 - it.n_cols;
                const int dist = max(off, -off);
                return (dist < wa ? 0u : rocket::kSplitMask) | (dist < wb ? 0u : rocket::kSplitMask << 16);
            };
            if (it.n_cols - c0 > rocket::kSplitTile)
                block<V, 2, MPV, true, 0, kTileBytes>(ad, plane, fa, cinit, mask, h, ac, cb);
            else
                block<V, 1, MPV, true, 0, kTileBytes>(ad, plane, fa, cinit, mask, h, ac, cb);
        };
        for (int b = 0; b < it.clean_lo; ++b) edge(b);
        Addr<V> ad;
#pragma unroll
        for (int i = 0; i < 4; ++i) ad.main[i] = row + (uint32_t)main0[i] + (uint32_t)it.clean_lo * kBlockBytes;
        if (idle) ad.main[3] = zero;
#pragma unroll
        for (int i = 0; i < tail_addrs(V); ++i) ad.tail[i] = row_tail + (uint32_t)tail0[i] + (uint32_t)it.clean_lo * kBlockBytes;
        // opaque, so that the loop advances the sums and not their terms
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(ad.main[i]));
#pragma unroll
        for (int i = 0; i < tail_addrs(V); ++i) asm volatile("" : "+v"(ad.tail[i]));
        auto none = [](int) { return 0u; };
        const int n_clean = it.clean_hi - it.clean_lo;
        // kUnroll blocks per address update (one with MPV, whose registers are
        // short: two measured 3.6 % slower)
        for (int b = 0; b + kUnroll <= n_clean; b += kUnroll) {
            block<V, 2, MPV, false, 0, kTileBytes>(ad, plane, fa, cinit, none, h, ac, cb);
            if constexpr (kUnroll == 2) block<V, 2, MPV, false, 1, kTileBytes>(ad, plane, fa, cinit, none, h, ac, cb);
#pragma unroll
            for (int i = 0; i < 4; ++i) ad.main[i] += i == 3 ? step3 : step;
#pragma unroll
            for (int i = 0; i < tail_addrs(V); ++i) ad.tail[i] += step;
        }
        if (n_clean % kUnroll) block<V, 2, MPV, false, 0, kTileBytes>(ad, plane, fa, cinit, none, h, ac, cb);
        for (int b = it.clean_hi; b < n_blocks; ++b) edge(b);

        // reductions over the 32 columns, then one store per row
        uint32_t mn[kRegs];
#pragma unroll
        for (int i = 0; i < kRegs; ++i) mn[i] = __float_as_uint(ac.mn[i]);
        // MAX = -min; +0 where the minimum is zero
        const float m = 0.0f - __uint_as_float(tree<OpMin>(mn, lane));
        // a mask adds 65,535 to its half and carries into the upper one: with
        // counts lo and hi below 65,536 the word is 65,536 (lo - hi) - lo
        const uint32_t packed = tree<OpAdd>(ac.cnt, lane);
        const uint32_t lo = (0u - packed) & 0xffffu;
        const uint32_t hi = (lo - ((packed + lo) >> 16)) & 0xffffu;
        const uint32_t c = (lane & 2) ? hi : lo;
        float ps = 0.0f;
        if constexpr (MPV > 0) {
            uint32_t p[kRegs];
#pragma unroll
            for (int i = 0; i < kRegs; ++i) p[i] = __float_as_uint(ac.sum(i));
            ps = __uint_as_float(tree<OpFadd>(p, lane));
        }
        if (okid >= 0) {
            // (float)c / (float)O correctly rounded: the double product is
            // within 2^-52 of the quotient, which lies 2^-49 or more (relative)
            // from a midpoint of floats
            const float ppv = (float)((double)c * inv_O);
            float *f = F0 + r * f_stride + (MPV ? 3 : 2) * (int64_t)okid;
#if ROCKET_CHECKED
            if (f < cb.out_lo || f + (MPV ? 3 : 2) > cb.out_hi) {
                atomicOr(&g_rocket_checks, kCheckStore);
                continue;
            }
#endif
            if (MPV) {
                f[0] = ppv;
                f[1] = m;
                f[2] = c > 0 ? ps / (float)c : 0.0f;
            } else {
                *reinterpret_cast<float2 *>(f) = make_float2(ppv, m);
            }
        }
    }
}

__device__ __forceinline__ SplitItem load_split_item(ConstPtr<SplitItem> p) {
    SplitItem it;
    it.variant = p->variant;
    it.d = p->d;
    it.s0 = p->s0;
    it.n_cols = p->n_cols;
    it.clean_lo = p->clean_lo;
    it.clean_hi = p->clean_hi;
    it.a_off = p->a_off;
    it.r_off = p->r_off;
    it.reach = p->reach;
    it.cost = p->cost;
    it.n_rows = p->n_rows;
#pragma unroll
    for (int i = 0; i < 4; ++i) it.width[i] = p->width[i];
    it.series_lo = p->series_lo;
    it.series_hi = p->series_hi;
    return it;
}

// A workgroup of few items deals each of them to its wavefronts in 2^sh parts
// of its series (rows do not interact): so that no wavefront goes without, and,
// for parts of at least kPartWork samples (part_even), to even out two rounds
// of tasks (a part costs its item's weights again: 931 x 28 samples, 289
// kernels, 4 items and 3 series a workgroup, 11.2 us whole and 13.4 in parts).
constexpr int64_t kPartWork = 1024;
__device__ __forceinline__ int part_shift(int n_items, const SplitArgs &a, int n_waves) {
    if (a.part_cap == 0) return 0;
    const int few = a.part_even ? 2 * n_waves : n_waves;
    return n_items >= few ? 0 : (2 * n_items >= few ? 1 : a.part_cap);
}

// The tasks (item, part) of one variant: a wavefront's first is its own
// number's (it, read by the caller while the series were staged), the others
// come from the workgroup's counter.
template <int V, int MPV>
__device__ __forceinline__ void run_split_items(int *next_item, int idx, SplitItem it, int beg, int n_items, int sh,
                                                const SplitArgs &a, uint32_t lds0, uint32_t plane, int nrows, float *F0,
                                                int lane, const CheckBounds &cb) {
    const int n_tasks = n_items << sh, parts = 1 << sh;
    while (idx < n_tasks) {
        run_split_item<V, MPV>(it, a, lds0, plane, idx & (parts - 1), parts, nrows, F0, lane, cb);
        int nx = 0;
        if (lane == 0) nx = atomicAdd(next_item, 1);
        idx = __builtin_amdgcn_readfirstlane(__shfl(nx, 0, 64));
        if (idx < n_tasks) it = load_split_item(as_const(a.items) + as_const(a.order)[beg + (idx >> sh)]);
    }
}

// Stage nrows rows: both words of every position, kMargin zeros before each
// row and kEndZeros after the last.
template <int BLOCK>
__device__ __forceinline__ void stage_rows(const SplitArgs &a, const float *X, int nrows, uint32_t *w0, uint32_t *w1) {
    for (int r = 0; r < nrows; ++r) {
        const float *x = X + (int64_t)r * a.L;
        uint32_t *d0 = w0 + r * a.pitch, *d1 = w1 + r * a.pitch;
        if (threadIdx.x < kMargin) d0[threadIdx.x] = d1[threadIdx.x] = 0u;
        if (a.vec4) {
            for (int e = threadIdx.x; e < a.L / 4; e += BLOCK) {
                const float4 v = reinterpret_cast<const float4 *>(x)[e];
                v4u p, q;
                uint32_t s0, s1;
                split_words(v.x, s0, s1);
                p[0] = s0;
                q[0] = s1;
                split_words(v.y, s0, s1);
                p[1] = s0;
                q[1] = s1;
                split_words(v.z, s0, s1);
                p[2] = s0;
                q[2] = s1;
                split_words(v.w, s0, s1);
                p[3] = s0;
                q[3] = s1;
                // pitch and margin are multiples of 4 words here
                reinterpret_cast<v4u *>(d0 + kMargin)[e] = p;
                reinterpret_cast<v4u *>(d1 + kMargin)[e] = q;
            }
        } else {
            for (int e = threadIdx.x; e < a.L; e += BLOCK) split_words(x[e], d0[kMargin + e], d1[kMargin + e]);
        }
    }
    if (threadIdx.x < kEndZeros) w0[nrows * a.pitch + threadIdx.x] = w1[nrows * a.pitch + threadIdx.x] = 0u;
}

// Workgroups 0 .. a.blocks - 1 run split items, the rest of the launch the
// fp32 items of q.  BLOCK threads; PLANE: bytes of a plane where fixed (an
// immediate offset of the LDS reads), 0 where given at run time (rows above
// 40 KB).
template <int BLOCK, int PLANE, int MPV>
__global__ __launch_bounds__(BLOCK, MPV ? 2 : 3) void rocket_split_kernel(SplitArgs a, FusedArgs q) {
    extern __shared__ __align__(16) uint32_t smem[];
    __shared__ int next_item;
    const int lane = threadIdx.x & (rocket::kWave - 1);
    if (blockIdx.x >= a.blocks) {
        GroupWork w;
        float *rows = reinterpret_cast<float *>(smem);
        if (!stage_group<BLOCK>(q, blockIdx.x - a.blocks, rows, &next_item, w)) return;
        run_variant<false, (MPV > 0)>(&next_item, w, q, rows + q.halo_lo, q.F + w.grow * (int64_t)q.nf * q.K, lane);
        return;
    }
    // workgroup b runs on XCD b % 8; every XCD takes its own share of the row
    // groups and walks them variant by variant
    const int64_t b = blockIdx.x;
    const int xcd = (int)b & ((1 << a.xcd_shift) - 1);
    const int64_t local = b >> a.xcd_shift;
    const int64_t per_variant = a.groups_per_xcd * a.nsplit;
    const int vi = (int)(local / per_variant);
    const int variant = a.variants[vi];
    const int64_t rest = local % per_variant;
    int64_t group;
    const int split = group_split(xcd, a.xcd_shift, a.groups_per_xcd, a.nsplit, vi, rest, group);
    const int beg = as_const(a.split_begin)[variant * a.nsplit + split];
    const int n_items = as_const(a.split_begin)[variant * a.nsplit + split + 1] - beg;
    const int64_t first = group * a.rows_per_block;
    if (n_items == 0 || first >= a.n_rows) return;
    const int nrows = (int)min((int64_t)a.rows_per_block, a.n_rows - first);
    const int64_t grow = a.row0 + first;
    const uint32_t plane = PLANE ? (uint32_t)PLANE : 4u * (uint32_t)a.plane_words;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / rocket::kWave);
    const int sh = part_shift(n_items, a, BLOCK / rocket::kWave);
    const SplitItem it0 =
        load_split_item(as_const(a.items) + as_const(a.order)[beg + min(wave >> sh, n_items - 1)]);
    stage_rows<BLOCK>(a, a.X + grow * a.L, nrows, smem, smem + plane / 4);
    if (threadIdx.x == 0) next_item = BLOCK / rocket::kWave;
    __syncthreads();
    const uint32_t lds0 = (uint32_t)(__UINTPTR_TYPE__)(lds_out *)smem;
    const int64_t f_row = (int64_t)(MPV ? 3 : 2) * a.K;
    CheckBounds cb{lds0 + plane + 4u * (uint32_t)(nrows * a.pitch + kEndZeros), a.F + a.row0 * f_row,
                   a.F + (a.row0 + a.n_rows) * f_row};
    float *F0 = a.F + grow * f_row;
    switch (variant) {
        case 0: run_split_items<0, MPV>(&next_item, wave, it0, beg, n_items, sh, a, lds0, plane, nrows, F0, lane, cb); break;
        case 1: run_split_items<1, MPV>(&next_item, wave, it0, beg, n_items, sh, a, lds0, plane, nrows, F0, lane, cb); break;
        default: run_split_items<2, MPV>(&next_item, wave, it0, beg, n_items, sh, a, lds0, plane, nrows, F0, lane, cb); break;
    }
}

// ---------------------------------------------------------------------------
// Series-lane layout (series of at most kSeriesMaxL samples, calls of many).
// LDS holds 64 series position-major, 64 consecutive words per position and
// plane: the 32 columns of a tile are 32 series at one position, a block is two
// positions, and every lane keeps the counts and minima of its own series, so
// nothing is reduced across lanes.  The same MFMAs in the same order as the
// tiled layout, so PPV and MAX are bit for bit the same.  The features go to a
// slot-ordered buffer, which rocket_slot_permute_kernel turns into F rows.
// ---------------------------------------------------------------------------
constexpr int kPosBytes = 4 * rocket::kWave;  // one position of a plane
constexpr int kSM = rocket::kSplitSeriesMargin;

template <int V, int MPV>
__device__ __forceinline__ void run_series_item(const SplitItem &it, const SplitArgs &a, uint32_t lds0, uint32_t plane,
                                                int64_t series0, int first, int n_series, int lane,
                                                const CheckBounds &cb) {
    const int n = lane & 31, h = lane >> 5;
    v4u fa[rocket::kSplitFrags[V]];
    v16f cinit;
    load_fragments<V>(it, a, lane, fa, cinit);
    const int n_blocks = (it.n_cols + 1) / 2;
    const bool idle = V == 0 && h == 1;
    const int wa = (V > 0 && h) ? it.width[2] : it.width[0], wb = (V > 0 && h) ? it.width[3] : it.width[1];
    constexpr int kUnroll = MPV ? 1 : 2;
    constexpr uint32_t step = kUnroll * 2 * kPosBytes;
    const uint32_t step3 = idle ? 0u : step;
    for (int s0 = first; s0 < n_series; s0 += rocket::kSplitTile) {
        const int base = (int)lds0 + kSM * kPosBytes + 4 * (s0 + n);  // position 0
        const uint32_t zero = (uint32_t)(base - kSM * kPosBytes);
        int main0[4], tail0[3];
#pragma unroll
        for (int i = 0; i < 4; ++i) main0[i] = base + kPosBytes * (it.s0 + min(4 * h + i, it.reach) * it.d);
#pragma unroll
        for (int i = 0; i < 3; ++i) tail0[i] = base + kPosBytes * (it.s0 + min(8 + i, it.reach) * it.d);
        const uint32_t tail_plane = V == 2 ? (uint32_t)h * plane : 0u;
        Acc<MPV> ac;
#pragma unroll
        for (int i = 0; i < kRegs; ++i) {
            ac.mn[i] = INFINITY;
            if (MPV) ac.ps[0][i] = 0.0f;
            if constexpr (MPV == 2) ac.ps[1][i] = 0.0f;
        }
#pragma unroll
        for (int j = 0; j < kRegs / 2; ++j) ac.cnt[j] = 0u;
        const int lo = base - kSM * kPosBytes, hi = base + a.L * kPosBytes;
        auto edge = [&](int b) {
            const int c0 = 2 * b;
            auto clamped = [&](int m) { return (uint32_t)min(max(m + c0 * kPosBytes, lo), hi); };
            Addr<V> ad;
#pragma unroll
            for (int i = 0; i < 4; ++i) ad.main[i] = clamped(main0[i]);
            if (idle) ad.main[3] = zero;
#pragma unroll
            for (int i = 0; i < tail_addrs(V); ++i) ad.tail[i] = clamped(tail0[i]) + tail_plane;
            auto mask = [&](int u) {
                const int off = 2 * (c0 + u) + 1 - it.n_cols;
                const int dist = max(off, -off);
                return (dist < wa ? 0u : rocket::kSplitMask) | (dist < wb ? 0u : rocket::kSplitMask << 16);
            };
            if (it.n_cols - c0 > 1)
                block<V, 2, MPV, true, 0, kPosBytes>(ad, plane, fa, cinit, mask, h, ac, cb);
            else
                block<V, 1, MPV, true, 0, kPosBytes>(ad, plane, fa, cinit, mask, h, ac, cb);
        };
        for (int b = 0; b < it.series_lo; ++b) edge(b);
        Addr<V> ad;
        const uint32_t start = (uint32_t)it.series_lo * 2 * kPosBytes;
#pragma unroll
        for (int i = 0; i < 4; ++i) ad.main[i] = (uint32_t)main0[i] + start;
        if (idle) ad.main[3] = zero;
#pragma unroll
        for (int i = 0; i < tail_addrs(V); ++i) ad.tail[i] = (uint32_t)tail0[i] + start + tail_plane;
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(ad.main[i]));
#pragma unroll
        for (int i = 0; i < tail_addrs(V); ++i) asm volatile("" : "+v"(ad.tail[i]));
        auto none = [](int) { return 0u; };
        const int n_clean = it.series_hi - it.series_lo;
        for (int b = 0; b + kUnroll <= n_clean; b += kUnroll) {
            block<V, 2, MPV, false, 0, kPosBytes>(ad, plane, fa, cinit, none, h, ac, cb);
            if constexpr (kUnroll == 2) block<V, 2, MPV, false, 1, kPosBytes>(ad, plane, fa, cinit, none, h, ac, cb);
#pragma unroll
            for (int i = 0; i < 4; ++i) ad.main[i] += i == 3 ? step3 : step;
#pragma unroll
            for (int i = 0; i < tail_addrs(V); ++i) ad.tail[i] += step;
        }
        if (n_clean % kUnroll) block<V, 2, MPV, false, 0, kPosBytes>(ad, plane, fa, cinit, none, h, ac, cb);
        for (int b = it.series_hi; b < n_blocks; ++b) edge(b);

        // the features of the lane's series, rows 2 i + h
        const float2 *div = reinterpret_cast<const float2 *>(a.div_O) + it.r_off + h * kRegs;
        const bool mine = s0 + n < n_series;
        float *out = a.S + ((int64_t)(it.r_off + h) * a.s_rows + series0 + s0 + n) * (MPV ? 3 : 2);
#pragma unroll
        for (int i = 0; i < kRegs; ++i) {
            const uint32_t packed = ac.cnt[i / 2];  // see run_split_item
            const uint32_t lo16 = (0u - packed) & 0xffffu;
            const uint32_t c = (i & 1) ? (lo16 - ((packed + lo16) >> 16)) & 0xffffu : lo16;
            // (float)c / (float)O correctly rounded: a quotient estimate from
            // the rounded reciprocal, corrected once by the exact remainder
            // (Markstein 1990)
            const float2 d = div[i];
            const float fc = (float)c, q = fc * d.y;
            const float ppv = fmaf(fmaf(-q, d.x, fc), d.y, q);
            const float m = 0.0f - ac.mn[i];
            float *f = out + (int64_t)(2 * i) * a.s_rows * (MPV ? 3 : 2);
            if (mine && 2 * i + h < it.n_rows) {
#if ROCKET_CHECKED
                if (f < a.S || f + (MPV ? 3 : 2) > a.S + a.s_floats) {
                    atomicOr(&g_rocket_checks, kCheckStore);
                    continue;
                }
#endif
                if (MPV) {
                    f[0] = ppv;
                    f[1] = m;
                    f[2] = c > 0 ? ac.sum(i) / fc : 0.0f;
                } else {
                    *reinterpret_cast<float2 *>(f) = make_float2(ppv, m);
                }
            }
        }
    }
}

// The tasks of one variant, as run_split_items: items, or where those are few
// (sh = 1) items x the workgroup's two tiles of 32 series.
template <int V, int MPV>
__device__ __forceinline__ void run_series_items(int *next_item, int idx, SplitItem it, int beg, int n_items, int sh,
                                                 const SplitArgs &a, uint32_t lds0, uint32_t plane, int64_t series0,
                                                 int n_series, int lane, const CheckBounds &cb) {
    const int n_tasks = n_items << sh;
    while (idx < n_tasks) {
        const int first = sh ? (idx & 1) * rocket::kSplitTile : 0;
        run_series_item<V, MPV>(it, a, lds0, plane, series0, first,
                                sh ? min(n_series, first + rocket::kSplitTile) : n_series, lane, cb);
        int nx = 0;
        if (lane == 0) nx = atomicAdd(next_item, 1);
        idx = __builtin_amdgcn_readfirstlane(__shfl(nx, 0, 64));
        if (idx < n_tasks) it = load_split_item(as_const(a.items) + as_const(a.order)[beg + (idx >> sh)]);
    }
}

constexpr int kSeriesBlock = 256;
constexpr int kSeriesRounds = 4;  // workgroups per CU that a launch splits its items into

template <int MPV>
__global__ __launch_bounds__(kSeriesBlock, MPV ? 2 : 3) void rocket_split_series_kernel(SplitArgs a) {
    extern __shared__ __align__(16) uint32_t smem[];
    __shared__ int next_item;
    const int lane = threadIdx.x & (rocket::kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / rocket::kWave);
    const int64_t b = blockIdx.x;
    const int xcd = (int)(b % kXcds);
    const int64_t local = b / kXcds;
    const int64_t per_variant = a.groups_per_xcd * a.nsplit;
    const int variant = a.variants[(int)(local / per_variant)];
    const int64_t rest = local % per_variant;
    const int64_t group = xcd * a.groups_per_xcd + rest / a.nsplit;
    const int split = (int)(rest % a.nsplit);
    const int beg = as_const(a.split_begin)[variant * a.nsplit + split];
    const int n_items = as_const(a.split_begin)[variant * a.nsplit + split + 1] - beg;
    const int64_t first = group * rocket::kWave;
    if (n_items == 0 || first >= a.n_rows) return;
    const int n_series = (int)min((int64_t)rocket::kWave, a.n_rows - first);
    constexpr int kWaves = kSeriesBlock / rocket::kWave;
    const int sh = n_items < kWaves || (n_items < 2 * kWaves && a.L * rocket::kSplitTile >= kPartWork) ? 1 : 0;
    const SplitItem it0 =
        load_split_item(as_const(a.items) + as_const(a.order)[beg + min(wave >> sh, n_items - 1)]);
    // stage: lane = series, so that a position's 64 words are written at once
    const uint32_t plane = 4u * (uint32_t)a.plane_words;
    uint32_t *w0 = smem + kSM * rocket::kWave + lane, *w1 = w0 + plane / 4;
    for (int m = wave; m < 2 * kSM; m += kSeriesBlock / rocket::kWave) {
        const int pos = m < kSM ? m - kSM : a.L + m - kSM;
        w0[pos * rocket::kWave] = w1[pos * rocket::kWave] = 0u;
    }
    const float *x = a.X + (a.row0 + first + min(lane, n_series - 1)) * (int64_t)a.L;
    if (a.vec4) {
        for (int e = wave; e < a.L / 4; e += kSeriesBlock / rocket::kWave) {
            const float4 v = reinterpret_cast<const float4 *>(x)[e];
            split_words(v.x, w0[4 * e * rocket::kWave], w1[4 * e * rocket::kWave]);
            split_words(v.y, w0[(4 * e + 1) * rocket::kWave], w1[(4 * e + 1) * rocket::kWave]);
            split_words(v.z, w0[(4 * e + 2) * rocket::kWave], w1[(4 * e + 2) * rocket::kWave]);
            split_words(v.w, w0[(4 * e + 3) * rocket::kWave], w1[(4 * e + 3) * rocket::kWave]);
        }
    } else {
        for (int e = wave; e < a.L; e += kSeriesBlock / rocket::kWave)
            split_words(x[e], w0[e * rocket::kWave], w1[e * rocket::kWave]);
    }
    if (threadIdx.x == 0) next_item = kSeriesBlock / rocket::kWave;
    __syncthreads();
    const uint32_t lds0 = (uint32_t)(__UINTPTR_TYPE__)(lds_out *)smem;
    const CheckBounds cb{lds0 + 2 * plane, nullptr, nullptr};
    switch (variant) {
        case 0: run_series_items<0, MPV>(&next_item, wave, it0, beg, n_items, sh, a, lds0, plane, first, n_series, lane, cb); break;
        case 1: run_series_items<1, MPV>(&next_item, wave, it0, beg, n_items, sh, a, lds0, plane, first, n_series, lane, cb); break;
        default: run_series_items<2, MPV>(&next_item, wave, it0, beg, n_items, sh, a, lds0, plane, first, n_series, lane, cb); break;
    }
}

// Workgroup shapes.  The kernel's registers (168, with MPV 205 to 209) allow
// three wavefronts per SIMD (with MPV two), so a CU holds 12 (8): three
// workgroups of 256 threads with a third of the 160 KB of LDS each, two of 384,
// or one of 768 for rows that take more than half (with MPV two of 256, one of
// 512).
struct Shape {
    int block;
    int plane;  // bytes of a plane; 0: given at run time
};
constexpr Shape kShapes[2][3] = {{{256, 26624}, {384, 40704}, {768, 0}}, {{256, 40704}, {256, 40704}, {512, 0}}};

// chains: see Acc (1 up to 128 samples, whose rows never take shape 2).
const void *kernel_fn(int shape, int chains) {
    if (chains > 0 && shape == 2) return (const void *)rocket_split_kernel<512, 0, 2>;
    if (chains > 0)
        return chains == 1 ? (const void *)rocket_split_kernel<256, 40704, 1>
                           : (const void *)rocket_split_kernel<256, 40704, 2>;
    switch (shape) {
        case 0: return (const void *)rocket_split_kernel<256, 26624, 0>;
        case 1: return (const void *)rocket_split_kernel<384, 40704, 0>;
        default: return (const void *)rocket_split_kernel<768, 0, 0>;
    }
}

// Copies of host tables in one device allocation (a plan is made of many small
// ones, and an allocation costs as much as their planning): sized by the first
// walk over the tables, filled by the second.
struct TablePool {
    char *base = nullptr;
    size_t used = 0;
    template <typename T>
    hipError_t add(const std::vector<T> &h, T **d) {
        const size_t at = used;
        used += (h.size() * sizeof(T) + 255) / 256 * 256;
        if (!base || h.empty()) return hipSuccess;
        *d = reinterpret_cast<T *>(base + at);
        return hipMemcpy(*d, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice);
    }
};

constexpr int kMaxDevices = 64;
std::mutex g_lds_mu;
bool g_lds_allowed[kMaxDevices];

// The kernels' dynamic LDS limit, raised once per device.
hipError_t allow_lds(int device, int64_t limit) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_lds_mu);
    if (g_lds_allowed[device]) return hipSuccess;
    for (int sel = 0; sel < 9; ++sel) {
        const hipError_t e = hipFuncSetAttribute(kernel_fn(sel / 3, sel % 3),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)limit);
        if (e != hipSuccess) return e;
    }
    for (const void *fn : {(const void *)rocket_split_series_kernel<0>, (const void *)rocket_split_series_kernel<1>}) {
        const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)limit);
        if (e != hipSuccess) return e;
    }
    g_lds_allowed[device] = true;
    return hipSuccess;
}

}  // namespace

namespace rocket {

struct SplitDevice {
    SplitPlan host;
    int shape = 0, rows = 1, n_cu = 0;
    int64_t lds = 0, lds_room = 0;
    int32_t plane_words = 0;
    bool mpv = false;
    void *tables = nullptr;  // the allocation that the following point into
    SplitItem *items = nullptr;
    uint32_t *a = nullptr;
    float *cinit = nullptr;
    int32_t *kid = nullptr, *order = nullptr, *split_begin = nullptr;
    double *inv_O = nullptr;
    float *div_O = nullptr;
};

void split_destroy(SplitDevice *d) {
    if (!d) return;
    if (d->tables) (void)hipFree(d->tables);
    delete d;
}

bool split_fits(int32_t L, int64_t lds_limit) {
    return 2 * 4 * ((int64_t)L + kMargin + kEndZeros) + 256 <= lds_limit;
}

int64_t split_series_lds(int32_t L) { return 2 * (int64_t)kPosBytes * (L + 2 * kSM); }
const std::vector<int32_t> &split_slot_kernels(const SplitDevice *d) { return d->host.kid; }

rocket_status split_launch_series(const SplitDevice *d, const float *X, int64_t n, int32_t K, float *S, int64_t s_rows,
                                  hipStream_t s) {
    const SplitPlan &P = d->host;
    const int64_t groups = (n + kWave - 1) / kWave;
    int64_t present = 0;
    for (int v = 0; v < kSplitVariants; ++v) present += P.split_begin[v + 1] > P.split_begin[v];
    // at most kSeriesRounds workgroups per CU (LDS and registers let two to
    // three run at once), with at least two items per wavefront once every CU
    // has a workgroup (5,000 series of 128 samples, 1,000 kernels: 322 us with
    // that bound at any size, 200 now)
    const int64_t n_cu = std::max(d->n_cu, 1);
    int li = 0;
    while (li + 1 < kNumSplitLayouts && groups * kSplitCounts[li + 1] * present <= kSeriesRounds * n_cu &&
           ((int64_t)P.items.size() / present / kSplitCounts[li + 1] >= 2 * (kSeriesBlock / kWave) ||
            groups * present * kSplitCounts[li] < n_cu))
        ++li;
    SplitArgs a{};
    a.X = X;
    a.L = P.L;
    a.K = K;
    a.items = d->items;
    a.a = d->a;
    a.cinit = d->cinit;
    a.kid = d->kid;
    a.inv_O = d->inv_O;
    a.div_O = d->div_O;
    a.order = d->order;
    a.split_begin = d->split_begin + P.layout_off[li];
    a.nsplit = kSplitCounts[li];
    const int32_t *sb = P.split_begin.data() + P.layout_off[li];
    for (int v = kSplitVariants - 1; v >= 0; --v)
        if (sb[(v + 1) * a.nsplit] > sb[v * a.nsplit]) a.variants[a.n_variants++] = v;
    a.n_rows = n;
    a.groups_per_xcd = (groups + kXcds - 1) / kXcds;
    a.plane_words = (int32_t)(split_series_lds(P.L) / 8);
    a.vec4 = (P.L % 4 == 0 && ((uintptr_t)X % 16) == 0) ? 1 : 0;
    a.S = S;
    a.s_rows = s_rows;
    a.s_floats = (int64_t)P.kid.size() * s_rows * (d->mpv ? 3 : 2);
    const unsigned nb = (unsigned)(kXcds * a.groups_per_xcd * a.nsplit * a.n_variants);
    void *args[] = {&a};
    const void *fn = d->mpv ? (const void *)rocket_split_series_kernel<1> : (const void *)rocket_split_series_kernel<0>;
    if (hipLaunchKernel(fn, dim3(nb), dim3(kSeriesBlock), args, (size_t)split_series_lds(P.L), s) != hipSuccess ||
        hipGetLastError() != hipSuccess)
        return ROCKET_ERR_HIP;
    return ROCKET_OK;
}
int64_t split_lds_bytes(const SplitDevice *d) { return d->lds; }
double split_rest_cost(const SplitDevice *d) { return d->host.rest_cost; }
int split_rows_per_block(const SplitDevice *d) { return d->rows; }
int64_t split_n_items(const SplitDevice *d) { return (int64_t)d->host.items.size(); }
int64_t split_n_rest(const SplitDevice *d) { return (int64_t)d->host.rest.size(); }
int64_t split_n_buckets(const SplitDevice *d) { return d->host.n_buckets; }
int64_t split_lds_room(const SplitDevice *d) { return d->lds_room; }
bool split_one_per_cu(const SplitDevice *d) { return d->shape == 2; }

hipError_t split_create(SplitPlan &&plan, int device, int n_cu, int64_t lds_limit, bool mpv, SplitDevice **out) {
    *out = nullptr;
    SplitDevice *d = new (std::nothrow) SplitDevice();
    if (!d) return hipErrorOutOfMemory;
    d->host = std::move(plan);
    d->n_cu = n_cu;
    d->mpv = mpv;
    const int64_t L = d->host.L, pitch = L + kMargin;
    const int64_t row_plane = 4 * (pitch + kEndZeros);  // one row
    const Shape *shapes = kShapes[mpv ? 1 : 0];
    d->shape = row_plane <= shapes[0].plane ? 0 : (row_plane <= shapes[1].plane ? 1 : 2);
    const int64_t plane = d->shape == 2 ? (row_plane + 15) / 16 * 16 : shapes[d->shape].plane;
    d->rows = d->shape == 2 ? 1 : (int)((plane / 4 - kEndZeros) / pitch);
    d->plane_words = (int32_t)(plane / 4);
    d->lds = 2 * plane;
    TablePool pool;
    auto walk = [&]() {
        hipError_t e = pool.add(d->host.items, &d->items);
        if (e == hipSuccess) e = pool.add(d->host.a, &d->a);
        if (e == hipSuccess) e = pool.add(d->host.cinit, &d->cinit);
        if (e == hipSuccess) e = pool.add(d->host.kid, &d->kid);
        if (e == hipSuccess) e = pool.add(d->host.inv_O, &d->inv_O);
        if (e == hipSuccess && d->host.L <= kSeriesMaxL) e = pool.add(d->host.div_O, &d->div_O);
        if (e == hipSuccess) e = pool.add(d->host.order, &d->order);
        if (e == hipSuccess) e = pool.add(d->host.split_begin, &d->split_begin);
        return e;
    };
    hipError_t e = walk();
    if (e == hipSuccess) e = hipMalloc(&d->tables, std::max<size_t>(pool.used, 256));
    pool = TablePool{static_cast<char *>(d->tables)};
    if (e == hipSuccess) e = walk();
    d->lds_room = lds_limit - 256;  // the rest for the workgroup's own variables
    if (e == hipSuccess) e = allow_lds(device, d->lds_room);
    if (e != hipSuccess) {
        split_destroy(d);
        return e;
    }
    *out = d;
    return hipSuccess;
}

rocket_status split_launch(const SplitDevice *d, const float *X, int64_t n, int32_t K, float *F, const FusedArgs *fp32,
                           int64_t fp32_lds, hipStream_t s) {
    const int block = kShapes[d->mpv ? 1 : 0][d->shape].block;
    const SplitPlan &P = d->host;
    int64_t present = 0;
    for (int v = 0; v < kSplitVariants; ++v) present += P.split_begin[v + 1] > P.split_begin[v];
    if (present == 0) return ROCKET_OK;
    // as the fp32 launch: enough workgroups to fill the chip several times
    // over, but a few items per wavefront once it is full twice
    const int64_t per_variant = (int64_t)P.items.size() / present;
    const int64_t resident = (int64_t)std::max(d->n_cu, 1) * ((d->mpv ? 512 : 768) / block);
    // few series: fewer of them per workgroup, down to one, before their items
    // are split over more workgroups than wavefronts have items for
    const int64_t spread = std::max<int64_t>(1, n * present / resident);
    const int R = (int)std::min<int64_t>(d->rows, spread);
    const int64_t groups = (n + R - 1) / R;
    int li = 0;
    while (li + 1 < kNumSplitLayouts && groups * present * kSplitCounts[li] < 4 * resident &&
           (per_variant / kSplitCounts[li + 1] >= 2 * (block / kWave) ||
            groups * present * kSplitCounts[li] < resident / 2))
        ++li;
    SplitArgs a;
    a.X = X;
    a.F = F;
    a.L = P.L;
    a.K = K;
    a.items = d->items;
    a.a = d->a;
    a.cinit = d->cinit;
    a.kid = d->kid;
    a.inv_O = d->inv_O;
    a.order = d->order;
    a.split_begin = d->split_begin + P.layout_off[li];
    a.nsplit = kSplitCounts[li];
    a.n_variants = 0;
    const int32_t *sb = P.split_begin.data() + P.layout_off[li];
    for (int v = kSplitVariants - 1; v >= 0; --v)
        if (sb[(v + 1) * a.nsplit] > sb[v * a.nsplit]) a.variants[a.n_variants++] = v;
    a.rows_per_block = R;
    a.part_cap = R >= 4 ? 2 : (R >= 2 ? 1 : 0);
    a.part_even = ((int64_t)R * P.L >> a.part_cap) >= kPartWork ? 1 : 0;
    a.pitch = P.L + kMargin;
    a.plane_words = d->plane_words;
    a.vec4 = (P.L % 4 == 0 && ((uintptr_t)X % 16) == 0) ? 1 : 0;
    FusedArgs q{};
    if (fp32) q = *fp32;
    const size_t lds = (size_t)std::max(d->lds, fp32 ? fp32_lds : 0);
    // rows of one launch: each part at most 2^30 workgroups
    const int64_t most = (int64_t)1 << 30;
    int64_t max_rows = (most / (a.nsplit * a.n_variants) / kXcds - 1) * kXcds * R;
    if (fp32)
        max_rows = std::min(max_rows, (most / (q.nsplit * q.n_variants) / kXcds - 1) * kXcds * q.rows_per_block);
    for (int64_t r0 = 0; r0 < n; r0 += max_rows) {
        a.row0 = r0;
        a.n_rows = std::min<int64_t>(max_rows, n - r0);
        auto share = [&](int64_t rows, int32_t *shift, int64_t *groups_per) {
            const int64_t groups = (a.n_rows + rows - 1) / rows;
            *shift = xcd_shift(groups);
            *groups_per = (groups + (1 << *shift) - 1) >> *shift;
            return *groups_per << *shift;
        };
        a.blocks = (uint32_t)(share(R, &a.xcd_shift, &a.groups_per_xcd) * a.nsplit * a.n_variants);
        uint32_t blocks = a.blocks;
        if (fp32) {
            q.row0 = r0;
            q.n_rows = a.n_rows;
            blocks += (uint32_t)(share(q.rows_per_block, &q.xcd_shift, &q.groups_per_xcd) * q.nsplit * q.n_variants);
        }
        void *args[] = {&a, &q};
        if (hipLaunchKernel(kernel_fn(d->shape, !d->mpv ? 0 : (P.L <= kSeriesMaxL ? 1 : 2)), dim3(blocks), dim3(block), args, lds, s) != hipSuccess ||
            hipGetLastError() != hipSuccess)
            return ROCKET_ERR_HIP;
    }
    return ROCKET_OK;
}

rocket_status split_check_flags(uint32_t *flags) {
#if ROCKET_CHECKED
    uint32_t v = 0, zero = 0;
    if (hipMemcpyFromSymbol(&v, HIP_SYMBOL(g_rocket_checks), sizeof(v)) != hipSuccess ||
        hipMemcpyToSymbol(HIP_SYMBOL(g_rocket_checks), &zero, sizeof(zero)) != hipSuccess)
        return ROCKET_ERR_HIP;
    *flags |= v;
#endif
    (void)flags;
    return ROCKET_OK;
}

}  // namespace rocket
