// fp32 work items of the ROCKET transform: tile reads, the MFMA, VALU and
// Toeplitz items, the wavefront reductions and the staging of series.  Used
// by the fused kernels (transform.hip) and by the split kernel, which runs
// the kernels its own items leave over beside them (split.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "rocket_internal.h"

namespace rocket {

// Arguments of the kernels that run fp32 items.
struct FusedArgs {
    const float *X;
    float *F;
    int64_t row0;      // first row of this launch (rows are independent)
    int64_t n_rows;    // rows in this launch
    int32_t L;
    int32_t K;
    int32_t nf;        // features per kernel in F: 2 (PPV, MAX) or 3 (+ MPV); 1 for
                       // MINIROCKET, whose K is then its feature count
    int32_t C;         // channels per series
    const float *thr;     // MINIROCKET items: per item [nq][4] thresholds
    const ItemDesc *items;
    const float *wpk;
    const float *bias;
    const int32_t *kid;
    const int32_t *order;
    const int32_t *split_begin;  // n_variants * nsplit + 1 offsets into order
    int32_t nsplit;
    int32_t n_variants;          // variants that have items, launched variant-major
    int32_t variants[kNumVariants];
    int32_t xcd_shift;           // workgroup b belongs to XCD share b mod 2^xcd_shift (3: its XCD; 0: one share)
    int64_t groups_per_xcd;      // row groups (of rows_per_block series) per share
    int32_t halo_lo;
    int32_t row_stride;
    int32_t tail_pad;        // zero floats staged after the last row
    int32_t rows_per_block;  // series staged together in one workgroup's LDS
    int32_t vec4;            // 1: rows are staged with 16-byte loads and LDS writes (L, halo_lo and
                             // row_stride multiples of 4 floats, X 16-byte aligned)
    float *S;                // series-lane layout: features in slot order (see below)
    int64_t s_rows;          // rows one slot column of S holds
    int64_t s_floats;        // floats of S this launch may write (bounds of checked builds)
};

}  // namespace rocket

using rocket::FusedArgs;
using rocket::ItemDesc;

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
constexpr uint64_t kNegInfPair = 0xff800000ff800000ull;  // two fp32 -inf

// ---------------------------------------------------------------------------
// Checked build (compiled with ROCKET_CHECKED=1 into librocket_checked.so):
// every LDS tile read is checked against the bytes its workgroup staged,
// every feature store of the workgroup kernels against the rows and columns
// of its launch, and every slot column the series-lane permutation reads
// against the plan's slots.  A failed check sets a bit of g_rocket_checks
// (read and cleared by rocket_check_flags) and the access is redirected
// inside the buffer or skipped, so a wrong index never reads or writes
// outside it.  The product build compiles none of this.
// ---------------------------------------------------------------------------
#ifndef ROCKET_CHECKED
#define ROCKET_CHECKED 0
#endif
[[maybe_unused]] constexpr uint32_t kCheckLdsRead = 1u;  // an LDS tile read outside the staged bytes
[[maybe_unused]] constexpr uint32_t kCheckStore = 2u;    // a feature store outside its rows / columns
[[maybe_unused]] constexpr uint32_t kCheckSlotRead = 4u; // a read of the slot-ordered buffer outside its columns
#if ROCKET_CHECKED
static __device__ unsigned int g_rocket_checks;
static __shared__ uint32_t g_check_lds_lo, g_check_lds_hi;  // staged LDS bytes [lo, hi) of the workgroup
static __shared__ float *g_check_out_lo;              // the launch's output floats [lo, hi)
static __shared__ float *g_check_out_hi;
__device__ __forceinline__ void check_failed(uint32_t bit) {
    if ((threadIdx.x & 63) == 0) atomicOr(&g_rocket_checks, bit);
}
#endif

// The LDS byte address m of a read of `bytes` bytes (wave-uniform), checked
// in checked builds; a read outside the staged bytes goes to their start.
__device__ __forceinline__ uint32_t lds_checked(uint32_t m, uint32_t bytes) {
#if ROCKET_CHECKED
    // the bounds come from LDS into vector registers; the result goes to a
    // scalar operand (M0), so it is made wave-uniform explicitly (it is
    // uniform: m and the bounds are)
    const uint32_t lo = __builtin_amdgcn_readfirstlane(g_check_lds_lo);
    const uint32_t hi = __builtin_amdgcn_readfirstlane(g_check_lds_hi);
    uint32_t r = m;
    if (m < lo || m + bytes > hi) {
        check_failed(kCheckLdsRead);
        r = lo;
    }
    return __builtin_amdgcn_readfirstlane(r);
#endif
    (void)bytes;
    return m;
}

// Whether the n floats at f lie in the launch's output (always true in the
// product build).
__device__ __forceinline__ bool store_checked(const float *f, int n) {
#if ROCKET_CHECKED
    if (f < g_check_out_lo || f + n > g_check_out_hi) {
        check_failed(kCheckStore);
        return false;
    }
#endif
    (void)f;
    (void)n;
    return true;
}

// Record a workgroup's staged LDS bytes and its launch's output range
// (checked builds; thread 0, before the workgroup's barrier).
__device__ __forceinline__ void set_check_bounds(const float *smem, int64_t staged_floats, float *out_lo,
                                                 float *out_hi) {
#if ROCKET_CHECKED
    if (threadIdx.x == 0) {
        g_check_lds_lo = (uint32_t)(__UINTPTR_TYPE__)(__attribute__((address_space(3))) const float *)smem;
        g_check_lds_hi = g_check_lds_lo + 4u * (uint32_t)staged_floats;
        g_check_out_lo = out_lo;
        g_check_out_hi = out_hi;
    }
#endif
    (void)smem;
    (void)staged_floats;
    (void)out_lo;
    (void)out_hi;
}

// Read-only tables indexed by wavefront-uniform values are read through the
// constant address space, which lets the compiler use scalar loads.
template <typename T>
using ConstPtr = const __attribute__((address_space(4))) T *;
template <typename T>
__device__ __forceinline__ ConstPtr<T> as_const(const T *p) {
    return (ConstPtr<T>)(p);
}

// LDS byte address of a pointer into the kernel's shared memory.
typedef __attribute__((address_space(3))) const float lds_cfloat;
__device__ __forceinline__ uint32_t lds_addr(const float *p) {
    return (uint32_t)(__UINTPTR_TYPE__)(lds_cfloat *)p;
}

// The series values of up to 4 tiles under one tap: NT reads of 64
// consecutive floats, 256 bytes apart, the first at LDS byte address m
// (wavefront-uniform).  ds_read_addtid_b32 reads the dword at
// M0 + offset + 4 * lane, so the address comes from a scalar register and no
// vector instruction computes it.  M0 is written right before the reads
// (one wait state between the write and its first use) and is not used by
// compiled code in these kernels.  The reads complete before the asm block
// ends (lgkmcnt(0)), so the outputs are ready when the compiler sees them.
template <int NT>
__device__ __forceinline__ void lds_tiles_raw(uint32_t m, float (&xv)[NT]);
template <>
__device__ __forceinline__ void lds_tiles_raw<1>(uint32_t m, float (&xv)[1]) {
    asm volatile(
        "s_mov_b32 m0, %1\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %0\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=v"(xv[0])
        : "s"(m)
        : "memory");
}
template <>
__device__ __forceinline__ void lds_tiles_raw<2>(uint32_t m, float (&xv)[2]) {
    asm volatile(
        "s_mov_b32 m0, %2\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %0\n\tds_read_addtid_b32 %1 offset:256\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(xv[0]), "=&v"(xv[1])
        : "s"(m)
        : "memory");
}
template <>
__device__ __forceinline__ void lds_tiles_raw<3>(uint32_t m, float (&xv)[3]) {
    asm volatile(
        "s_mov_b32 m0, %3\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %0\n\tds_read_addtid_b32 %1 offset:256\n\t"
        "ds_read_addtid_b32 %2 offset:512\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(xv[0]), "=&v"(xv[1]), "=&v"(xv[2])
        : "s"(m)
        : "memory");
}
template <>
__device__ __forceinline__ void lds_tiles_raw<4>(uint32_t m, float (&xv)[4]) {
    asm volatile(
        "s_mov_b32 m0, %4\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %0\n\tds_read_addtid_b32 %1 offset:256\n\t"
        "ds_read_addtid_b32 %2 offset:512\n\tds_read_addtid_b32 %3 offset:768\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(xv[0]), "=&v"(xv[1]), "=&v"(xv[2]), "=&v"(xv[3])
        : "s"(m)
        : "memory");
}
// 5..8 tiles: all reads from one M0, then two waits.  lds_tiles waits until
// at most NT-4 reads are in flight (lgkmcnt(NT-4)); LDS reads complete in
// order, so tiles 0-3 are ready and their MFMAs can issue while the rest
// arrive.  lds_tiles_rest then waits for the rest: it takes tiles 4.. as
// operands and returns them, so no use of them precedes it.
template <int NT>
__device__ __forceinline__ void lds_tiles_rest(float (&xv)[NT]);

template <>
__device__ __forceinline__ void lds_tiles_raw<5>(uint32_t m, float (&xv)[5]) {
    asm volatile(
        "s_mov_b32 m0, %5\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %0\n\t"
        "ds_read_addtid_b32 %1 offset:256\n\t"
        "ds_read_addtid_b32 %2 offset:512\n\t"
        "ds_read_addtid_b32 %3 offset:768\n\t"
        "ds_read_addtid_b32 %4 offset:1024\n\t"
        "s_waitcnt lgkmcnt(1)"
        : "=&v"(xv[0]), "=&v"(xv[1]), "=&v"(xv[2]), "=&v"(xv[3]), "=&v"(xv[4])
        : "s"(m)
        : "memory");
}
template <>
__device__ __forceinline__ void lds_tiles_rest<5>(float (&xv)[5]) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(xv[4]) : : "memory");
}

template <>
__device__ __forceinline__ void lds_tiles_raw<6>(uint32_t m, float (&xv)[6]) {
    asm volatile(
        "s_mov_b32 m0, %6\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %0\n\t"
        "ds_read_addtid_b32 %1 offset:256\n\t"
        "ds_read_addtid_b32 %2 offset:512\n\t"
        "ds_read_addtid_b32 %3 offset:768\n\t"
        "ds_read_addtid_b32 %4 offset:1024\n\t"
        "ds_read_addtid_b32 %5 offset:1280\n\t"
        "s_waitcnt lgkmcnt(2)"
        : "=&v"(xv[0]), "=&v"(xv[1]), "=&v"(xv[2]), "=&v"(xv[3]), "=&v"(xv[4]), "=&v"(xv[5])
        : "s"(m)
        : "memory");
}
template <>
__device__ __forceinline__ void lds_tiles_rest<6>(float (&xv)[6]) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(xv[4]), "+v"(xv[5]) : : "memory");
}

template <>
__device__ __forceinline__ void lds_tiles_raw<7>(uint32_t m, float (&xv)[7]) {
    asm volatile(
        "s_mov_b32 m0, %7\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %0\n\t"
        "ds_read_addtid_b32 %1 offset:256\n\t"
        "ds_read_addtid_b32 %2 offset:512\n\t"
        "ds_read_addtid_b32 %3 offset:768\n\t"
        "ds_read_addtid_b32 %4 offset:1024\n\t"
        "ds_read_addtid_b32 %5 offset:1280\n\t"
        "ds_read_addtid_b32 %6 offset:1536\n\t"
        "s_waitcnt lgkmcnt(3)"
        : "=&v"(xv[0]), "=&v"(xv[1]), "=&v"(xv[2]), "=&v"(xv[3]), "=&v"(xv[4]), "=&v"(xv[5]), "=&v"(xv[6])
        : "s"(m)
        : "memory");
}
template <>
__device__ __forceinline__ void lds_tiles_rest<7>(float (&xv)[7]) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(xv[4]), "+v"(xv[5]), "+v"(xv[6]) : : "memory");
}

template <>
__device__ __forceinline__ void lds_tiles_raw<8>(uint32_t m, float (&xv)[8]) {
    asm volatile(
        "s_mov_b32 m0, %8\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %0\n\t"
        "ds_read_addtid_b32 %1 offset:256\n\t"
        "ds_read_addtid_b32 %2 offset:512\n\t"
        "ds_read_addtid_b32 %3 offset:768\n\t"
        "ds_read_addtid_b32 %4 offset:1024\n\t"
        "ds_read_addtid_b32 %5 offset:1280\n\t"
        "ds_read_addtid_b32 %6 offset:1536\n\t"
        "ds_read_addtid_b32 %7 offset:1792\n\t"
        "s_waitcnt lgkmcnt(4)"
        : "=&v"(xv[0]), "=&v"(xv[1]), "=&v"(xv[2]), "=&v"(xv[3]), "=&v"(xv[4]), "=&v"(xv[5]), "=&v"(xv[6]), "=&v"(xv[7])
        : "s"(m)
        : "memory");
}
template <>
__device__ __forceinline__ void lds_tiles_rest<8>(float (&xv)[8]) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(xv[4]), "+v"(xv[5]), "+v"(xv[6]), "+v"(xv[7]) : : "memory");
}

// The reads of lds_tiles_raw, with the address checked in checked builds.
template <int NT>
__device__ __forceinline__ void lds_tiles(uint32_t m, float (&xv)[NT]) {
    lds_tiles_raw<NT>(lds_checked(m, 256u * NT), xv);
}

// The reads of lds_tiles_raw<NT> (NT <= 4) without the wait: the values
// arrive in xv once lds_wait<NT, KEEP> has run after them.
template <int NT>
__device__ __forceinline__ void lds_issue_raw(uint32_t m, float (&xv)[NT]);
template <>
__device__ __forceinline__ void lds_issue_raw<1>(uint32_t m, float (&xv)[1]) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tds_read_addtid_b32 %0" : "=v"(xv[0]) : "s"(m) : "memory");
}
template <>
__device__ __forceinline__ void lds_issue_raw<2>(uint32_t m, float (&xv)[2]) {
    asm volatile(
        "s_mov_b32 m0, %2\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %0\n\tds_read_addtid_b32 %1 offset:256"
        : "=&v"(xv[0]), "=&v"(xv[1])
        : "s"(m)
        : "memory");
}
template <>
__device__ __forceinline__ void lds_issue_raw<3>(uint32_t m, float (&xv)[3]) {
    asm volatile(
        "s_mov_b32 m0, %3\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %0\n\tds_read_addtid_b32 %1 offset:256\n\t"
        "ds_read_addtid_b32 %2 offset:512"
        : "=&v"(xv[0]), "=&v"(xv[1]), "=&v"(xv[2])
        : "s"(m)
        : "memory");
}
template <>
__device__ __forceinline__ void lds_issue_raw<4>(uint32_t m, float (&xv)[4]) {
    asm volatile(
        "s_mov_b32 m0, %4\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %0\n\tds_read_addtid_b32 %1 offset:256\n\t"
        "ds_read_addtid_b32 %2 offset:512\n\tds_read_addtid_b32 %3 offset:768"
        : "=&v"(xv[0]), "=&v"(xv[1]), "=&v"(xv[2]), "=&v"(xv[3])
        : "s"(m)
        : "memory");
}
template <int NT>
__device__ __forceinline__ void lds_issue(uint32_t m, float (&xv)[NT]) {
    lds_issue_raw<NT>(lds_checked(m, 256u * NT), xv);
}

// Waits until at most KEEP LDS reads are in flight.  LDS reads complete in
// order, so the reads issued before the last KEEP (xv among them) have
// arrived; xv passes through the statement, so nothing reads it earlier.
template <int KEEP, int NT>
struct LdsWait;
template <int KEEP>
struct LdsWait<KEEP, 1> {
    __device__ __forceinline__ static void run(float (&xv)[1]) {
        asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(xv[0]) : "n"(KEEP) : "memory");
    }
};
template <int KEEP>
struct LdsWait<KEEP, 2> {
    __device__ __forceinline__ static void run(float (&xv)[2]) {
        asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(xv[0]), "+v"(xv[1]) : "n"(KEEP) : "memory");
    }
};
template <int KEEP>
struct LdsWait<KEEP, 3> {
    __device__ __forceinline__ static void run(float (&xv)[3]) {
        asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(xv[0]), "+v"(xv[1]), "+v"(xv[2]) : "n"(KEEP) : "memory");
    }
};
template <int KEEP>
struct LdsWait<KEEP, 4> {
    __device__ __forceinline__ static void run(float (&xv)[4]) {
        asm volatile("s_waitcnt lgkmcnt(%4)"
                     : "+v"(xv[0]), "+v"(xv[1]), "+v"(xv[2]), "+v"(xv[3])
                     : "n"(KEEP)
                     : "memory");
    }
};
template <int NT, int KEEP>
__device__ __forceinline__ void lds_wait(float (&xv)[NT]) {
    LdsWait<KEEP, NT>::run(xv);
}

// NC tiles (256 bytes apart) at each of P bases sb bytes apart, the first at
// m: P runs of reads under one M0 each, M0 advanced by sb between runs (one
// wait state after every M0 write).  Tiles are numbered base-major.  As for
// lds_tiles, at most NC * P - 4 reads are left in flight on return when
// NC * P > 4 (lds_tiles_rest then waits for the rest).
template <int NC, int P>
__device__ __forceinline__ void lds_multi_raw(uint32_t m, uint32_t sb, float (&xv)[NC * P]);
template <>
__device__ __forceinline__ void lds_multi_raw<1, 4>(uint32_t m, uint32_t sb, float (&xv)[4]) {
    asm volatile(
        "s_mov_b32 m0, %4\n\ts_nop 0\n\tds_read_addtid_b32 %0\n\t"
        "s_add_u32 m0, m0, %5\n\ts_nop 0\n\tds_read_addtid_b32 %1\n\t"
        "s_add_u32 m0, m0, %5\n\ts_nop 0\n\tds_read_addtid_b32 %2\n\t"
        "s_add_u32 m0, m0, %5\n\ts_nop 0\n\tds_read_addtid_b32 %3\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(xv[0]), "=&v"(xv[1]), "=&v"(xv[2]), "=&v"(xv[3])
        : "s"(m), "s"(sb)
        : "memory", "scc");
}
template <>
__device__ __forceinline__ void lds_multi_raw<2, 4>(uint32_t m, uint32_t sb, float (&xv)[8]) {
    asm volatile(
        "s_mov_b32 m0, %8\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %0\n\tds_read_addtid_b32 %1 offset:256\n\t"
        "s_add_u32 m0, m0, %9\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %2\n\tds_read_addtid_b32 %3 offset:256\n\t"
        "s_add_u32 m0, m0, %9\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %4\n\tds_read_addtid_b32 %5 offset:256\n\t"
        "s_add_u32 m0, m0, %9\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %6\n\tds_read_addtid_b32 %7 offset:256\n\t"
        "s_waitcnt lgkmcnt(4)"
        : "=&v"(xv[0]), "=&v"(xv[1]), "=&v"(xv[2]), "=&v"(xv[3]), "=&v"(xv[4]), "=&v"(xv[5]), "=&v"(xv[6]), "=&v"(xv[7])
        : "s"(m), "s"(sb)
        : "memory", "scc");
}
template <>
__device__ __forceinline__ void lds_multi_raw<3, 2>(uint32_t m, uint32_t sb, float (&xv)[6]) {
    asm volatile(
        "s_mov_b32 m0, %6\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %0\n\tds_read_addtid_b32 %1 offset:256\n\tds_read_addtid_b32 %2 offset:512\n\t"
        "s_add_u32 m0, m0, %7\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %3\n\tds_read_addtid_b32 %4 offset:256\n\tds_read_addtid_b32 %5 offset:512\n\t"
        "s_waitcnt lgkmcnt(2)"
        : "=&v"(xv[0]), "=&v"(xv[1]), "=&v"(xv[2]), "=&v"(xv[3]), "=&v"(xv[4]), "=&v"(xv[5])
        : "s"(m), "s"(sb)
        : "memory", "scc");
}
template <>
__device__ __forceinline__ void lds_multi_raw<4, 2>(uint32_t m, uint32_t sb, float (&xv)[8]) {
    asm volatile(
        "s_mov_b32 m0, %8\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %0\n\tds_read_addtid_b32 %1 offset:256\n\t"
        "ds_read_addtid_b32 %2 offset:512\n\tds_read_addtid_b32 %3 offset:768\n\t"
        "s_add_u32 m0, m0, %9\n\ts_nop 0\n\t"
        "ds_read_addtid_b32 %4\n\tds_read_addtid_b32 %5 offset:256\n\t"
        "ds_read_addtid_b32 %6 offset:512\n\tds_read_addtid_b32 %7 offset:768\n\t"
        "s_waitcnt lgkmcnt(4)"
        : "=&v"(xv[0]), "=&v"(xv[1]), "=&v"(xv[2]), "=&v"(xv[3]), "=&v"(xv[4]), "=&v"(xv[5]), "=&v"(xv[6]), "=&v"(xv[7])
        : "s"(m), "s"(sb)
        : "memory", "scc");
}

namespace {

constexpr int kMaxRowsPerBlock = 7;
constexpr int kXcds = 8;          // MI355X: 8 XCDs, workgroups dealt round-robin
constexpr int kXcdShift = 3;
constexpr int kTile = rocket::kTile;

// DPP controls (GFX9 encoding)
constexpr int kDppQuadSwap1 = 0xB1;   // quad_perm(1,0,3,2)
constexpr int kDppQuadSwap2 = 0x4E;   // quad_perm(2,3,0,1)
constexpr int kDppRowHalfMirror = 0x141;
constexpr int kDppRowMirror = 0x140;
constexpr int kDppRowRor8 = 0x128;     // row_ror:8 (lane i of a row reads lane i^8)

// Where a block's series values come from.  m0(j) is the LDS byte address
// of lane 0's value under tap j in the block's first tile; lane l reads 4*l
// bytes further and tile u of the block 256*u bytes further.  channel(off)
// moves to another channel's row (off floats further).
//   PaddedTiles:  the row sits in LDS with zero margins wide enough for
//                 every tap of every real output (and the tail pad after
//                 the last row for the lanes past O), so tap j is d floats
//                 after tap j-1.
//   ClampedTiles: the row sits in LDS with kClampMargin zeros on each side
//                 (long series, whose full margins would not fit).  The
//                 series index of lane 0 under tap j is clamped into
//                 [-kClampMargin, L] on the scalar unit: a block whose
//                 positions all lie left (right) of the series then reads
//                 zeros from the left (right) margin, and a block that
//                 overlaps the series is not moved, so every read stays in
//                 the margins and yields the zero-padded value.
struct PaddedTiles {
    uint32_t base;  // LDS byte address of lane 0's value under tap 0
    int d;
    __device__ __forceinline__ uint32_t m0(int j) const { return base + 4u * (uint32_t)(j * d); }
    __device__ __forceinline__ PaddedTiles channel(int off) const {
        return PaddedTiles{base + 4u * (uint32_t)off, d};
    }
};

struct ClampedTiles {
    uint32_t row;  // LDS byte address of series index 0
    int b0;        // series index under tap 0 of lane 0
    int d;
    int L;
    __device__ __forceinline__ uint32_t m0(int j) const {
        const int b = min(max(b0 + j * d, -rocket::kClampMargin), L);
        return row + 4u * (uint32_t)b;
    }
    __device__ __forceinline__ ClampedTiles channel(int off) const {
        return ClampedTiles{row + 4u * (uint32_t)off, b0, d, L};
    }
};

// The padded layout with each block's series offset clamped to at most L
// (Toeplitz items' last super-tile, whose taps reach up to (sigma - 1) d past
// the other blocks): a block that starts at or past L holds no real output
// that reads a series value, only zero padding, so it reads the zeros at L
// instead and every read stays inside the row's margins and the tail pad.
struct RightClampedTiles {
    uint32_t row;  // LDS byte address of series index 0
    int b0;        // series index under tap 0 of lane 0
    int d;
    int L;
    __device__ __forceinline__ uint32_t m0(int j) const { return row + 4u * (uint32_t)min(b0 + j * d, L); }
};

// The reads of lds_multi_raw, every run's address checked in checked
// builds (a failed run sends every run to the start of the staged bytes).
template <int NC, int P>
__device__ __forceinline__ void lds_multi(uint32_t m, uint32_t sb, float (&xv)[NC * P]) {
#if ROCKET_CHECKED
    bool ok = true;
#pragma unroll
    for (int k = 0; k < P; ++k) ok = ok && lds_checked(m + (uint32_t)k * sb, 256u * NC) == m + (uint32_t)k * sb;
    if (!ok) {
        m = g_check_lds_lo;
        sb = 0;
    }
    m = __builtin_amdgcn_readfirstlane(m);
    sb = __builtin_amdgcn_readfirstlane(sb);
#endif
    lds_multi_raw<NC, P>(m, sb, xv);
}

// The padded layout for P runs of NC tiles each, run k sb bytes after run 0
// (P super-tiles of a Toeplitz item whose super-tiles hold NC chunks): tile
// u is chunk u % NC of run u / NC.
template <int NC, int P>
struct MultiTiles {
    uint32_t base;  // LDS byte address of lane 0's value under tap 0, run 0
    int d;
    uint32_t sb;    // bytes from one run to the next
    __device__ __forceinline__ uint32_t m0(int j) const { return base + 4u * (uint32_t)(j * d); }
};

// How the tiles of one block group: 0 for one run (the block's last tile is
// the row's or super-tile's last), NC for MultiTiles (every run's last
// tile is its super-tile's last chunk).
template <typename Src>
struct TileRuns {
    static constexpr int nc = 0;
};
template <int NC, int P>
struct TileRuns<MultiTiles<NC, P>> {
    static constexpr int nc = NC;
};
__device__ constexpr bool run_last(int u, int nt, int nc) { return nc ? (u % nc == nc - 1) : (u == nt - 1); }

// The series values of a block's tiles under tap j.
template <int NT, typename Src>
__device__ __forceinline__ void read_tiles(const Src &src, int j, float (&xv)[NT]) {
    lds_tiles<NT>(src.m0(j), xv);
}

// Sources whose next tap's reads tile_mfma issues before the current tap's
// MFMAs (blocks of up to 4 tiles).  Only the series-lane reads: in the
// fused kernel the second set of tile registers lowers the occupancy from 5
// to 4 wavefronts per SIMD (100-thousand-series calls 2.2 % slower), while
// the series-lane kernel keeps its register count (a million 64-sample
// series: 0.4 % faster).
template <typename Src>
struct PipelinedReads {
    static constexpr bool value = false;
};
template <int NT, int NC, int P>
__device__ __forceinline__ void read_tiles(const MultiTiles<NC, P> &src, int j, float (&xv)[NT]) {
    static_assert(NT == NC * P, "one block reads all of its runs");
    lds_multi<NC, P>(src.m0(j), src.sb, xv);
}

// Per-series accumulators of one work item, per lane and kernel slot: the
// running max, the positive count (wavefront-uniform, scalar registers) and,
// when MPV is computed, the sum of the positive values.
template <int G>
struct RowAcc {
    v4f mx[G];
    uint32_t cnt[G][4];
    v4f ps[G];
};

// Multichannel items (Sec. 3.3): where the item's weights and channel rows
// are.  w is the lane's first packed weight (slot lane & 3); the weights of
// the item's ci-th channel, group g, tap j are at w[((ci*G + g)*ELL + j)*4].
// The channels are the set bits of mask, in ascending order; the row of
// channel c sits c*cstride floats after the series' first row.
struct McCtx {
    const float *w;
    uint64_t mask;
    int n_ch;
    int cstride;
};

// One channel's A-operand weights of a multichannel item (wp: its first).
template <int ELL, int G>
__device__ __forceinline__ void load_channel_weights(const float *wp, float (&wc)[G][ELL]) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int j = 0; j < ELL; ++j) wc[g][j] = wp[(g * ELL + j) * 4];
}

// The contraction of one block of NT tiles over the taps of one channel:
// tap j of every tile and kernel group is issued before tap j+1, so the
// wavefront keeps NT*G independent MFMA accumulation chains in flight.  With
// FIRST set each chain starts from its start value (the slots' biases, or,
// in the last tile of a row, -inf on lanes past the last output); without
// it the chains continue from acc (the next channel of a multichannel item).
template <int ELL, int G, int NT, bool LAST, bool FIRST, typename Src>
__device__ __forceinline__ void tile_mfma(const Src &src, const float (&wa)[G][ELL],
                                          const v4f (&binit)[G], const v4f (&blast)[G],
                                          v4f (&acc)[NT][G]) {
    if constexpr (NT <= 4 && PipelinedReads<Src>::value) {
        // tap j + 1's reads are in flight while tap j's MFMAs issue
        float xv[2][NT];
        lds_issue<NT>(src.m0(0), xv[0]);
#pragma unroll
        for (int j = 0; j < ELL; ++j) {
            if (j + 1 < ELL) {
                lds_issue<NT>(src.m0(j + 1), xv[(j + 1) & 1]);
                lds_wait<NT, NT>(xv[j & 1]);
            } else {
                lds_wait<NT, 0>(xv[j & 1]);
            }
#pragma unroll
            for (int u = 0; u < NT; ++u)
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const v4f c = (FIRST && j == 0)
                                      ? ((LAST && run_last(u, NT, TileRuns<Src>::nc)) ? blast[g] : binit[g])
                                      : acc[u][g];
                    acc[u][g] = __builtin_amdgcn_mfma_f32_4x4x1f32(wa[g][j], xv[j & 1][u], c, 0, 0, 0);
                }
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < ELL; ++j) {
        float xv[NT];
        read_tiles<NT>(src, j, xv);
        constexpr int NA = NT > 4 ? 4 : NT;  // tiles ready after lds_tiles
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            if (NT > 4 && u == NA) {
                // tiles 4..: wait for the rest of the reads only now, after
                // the MFMAs of tiles 0-3 (the barriers keep this order)
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (NT > 4) lds_tiles_rest<NT>(xv);
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const v4f c = (FIRST && j == 0)
                                  ? ((LAST && run_last(u, NT, TileRuns<Src>::nc)) ? blast[g] : binit[g])
                                  : acc[u][g];
                acc[u][g] = __builtin_amdgcn_mfma_f32_4x4x1f32(wa[g][j], xv[u], c, 0, 0, 0);
            }
        }
        if (NT > 4) __builtin_amdgcn_sched_barrier(0);
    }
}

// Fold NT tiles of finished dot products into the row accumulators.  A chain
// started at -inf stays -inf, so MAX folds every result (v_max3 over pairs of
// tiles), the positive count is a ballot of y > 0 popcounted on the scalar
// unit, and the MPV numerator adds max(y, 0).
template <int G, int NT, bool MPV>
__device__ __forceinline__ void block_reduce(const v4f (&acc)[NT][G], RowAcc<G> &ra) {
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                ra.cnt[g][v] += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(acc[u][g][v] > 0.0f));
    if (MPV) {
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int v = 0; v < 4; ++v) ra.ps[g][v] += fmaxf(acc[u][g][v], 0.0f);
    }
#pragma unroll
    for (int u = 0; u + 1 < NT; u += 2)
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                ra.mx[g][v] = fmaxf(fmaxf(ra.mx[g][v], acc[u][g][v]), acc[u + 1][g][v]);
    if (NT % 2 == 1) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int v = 0; v < 4; ++v) ra.mx[g][v] = fmaxf(ra.mx[g][v], acc[NT - 1][g][v]);
    }
}

// One block of NT tiles.  Univariate items keep their weights in registers
// (wa); multichannel items (MC) run the MFMA chains over every channel of
// their mask, reading each channel's weights in turn: the next channel's
// weights are loaded while the current channel's MFMAs run, and the channel
// numbers come from the mask (s_ff1) without a memory access.  The scheduling
// barriers keep the block's MFMAs in one run and its reduction in another:
// on gfx950 fp32 MFMA and VALU instructions of a SIMD do not execute at the
// same time, and a VALU instruction placed between two MFMAs of a wavefront
// costs more than the same instruction in a run of VALU work.
template <int ELL, int G, int NT, bool LAST, bool MPV, bool MC, typename Src>
__device__ __forceinline__ void tile_block(const Src &src, const float (&wa)[G][ELL],
                                           const McCtx &mc, const v4f (&binit)[G],
                                           const v4f (&blast)[G], RowAcc<G> &ra) {
    v4f acc[NT][G];
    if constexpr (!MC) {
        tile_mfma<ELL, G, NT, LAST, true>(src, wa, binit, blast, acc);
    } else {
        float wc[G][ELL], wn[G][ELL];
        uint64_t m = mc.mask;
        int c = (int)__builtin_ctzll(m);
        m &= m - 1;
        load_channel_weights<ELL, G>(mc.w, wc);
        for (int ci = 0; ci < mc.n_ch; ++ci) {
            int cn = 0;
            if (ci + 1 < mc.n_ch) {
                load_channel_weights<ELL, G>(mc.w + (ci + 1) * (G * ELL * 4), wn);
                cn = (int)__builtin_ctzll(m);
                m &= m - 1;
            }
            const Src s = src.channel(c * mc.cstride);
            if (ci == 0)
                tile_mfma<ELL, G, NT, LAST, true>(s, wc, binit, blast, acc);
            else
                tile_mfma<ELL, G, NT, LAST, false>(s, wc, binit, blast, acc);
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int j = 0; j < ELL; ++j) wc[g][j] = wn[g][j];
            c = cn;
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // raised wave priority while the reduction runs: a wavefront that has
    // finished its MFMAs gets its vector work issued first (measured: 0.4 %
    // faster passes over 100,000 series of 1,000 samples, 0.7 % faster long
    // series; same results)
    __builtin_amdgcn_s_setprio(1);
    block_reduce<G, NT, MPV>(acc, ra);
    __builtin_amdgcn_s_setprio(0);
}

// The last block of a row: its tile count nv (1..N) selects a code copy.
// (LASTB false: a block of nv tiles whose last tile is not the row's last.)
template <int ELL, int G, int N, bool MPV, bool MC, typename Src, bool LASTB = true>
struct TailTiles {
    __device__ __forceinline__ static void run(int nv, const Src &src, const float (&wa)[G][ELL],
                                               const McCtx &mc, const v4f (&binit)[G],
                                               const v4f (&blast)[G], RowAcc<G> &ra) {
        if (nv == N)
            tile_block<ELL, G, N, LASTB, MPV, MC>(src, wa, mc, binit, blast, ra);
        else
            TailTiles<ELL, G, N - 1, MPV, MC, Src, LASTB>::run(nv, src, wa, mc, binit, blast, ra);
    }
};

template <int ELL, int G, bool MPV, bool MC, typename Src, bool LASTB>
struct TailTiles<ELL, G, 0, MPV, MC, Src, LASTB> {
    __device__ __forceinline__ static void run(int, const Src &, const float (&)[G][ELL],
                                               const McCtx &, const v4f (&)[G], const v4f (&)[G],
                                               RowAcc<G> &) {}
};

// The last block of a row and then the row's epilogue, a code copy per
// tile count nv (1..N): each copy reduces and writes the features from the
// registers its own block left the accumulators in (one epilogue after the
// copies would first have to move them into common registers).
template <int ELL, int G, int N, bool MPV, bool MC, typename Src>
struct TailTilesThen {
    template <typename Epi>
    __device__ __forceinline__ static void run(int nv, const Src &src, const float (&wa)[G][ELL],
                                               const McCtx &mc, const v4f (&binit)[G],
                                               const v4f (&blast)[G], RowAcc<G> &ra, const Epi &epi) {
        if (nv == N) {
            tile_block<ELL, G, N, true, MPV, MC>(src, wa, mc, binit, blast, ra);
            epi(ra);
        } else {
            TailTilesThen<ELL, G, N - 1, MPV, MC, Src>::run(nv, src, wa, mc, binit, blast, ra, epi);
        }
    }
};
template <int ELL, int G, bool MPV, bool MC, typename Src>
struct TailTilesThen<ELL, G, 0, MPV, MC, Src> {
    template <typename Epi>
    __device__ __forceinline__ static void run(int, const Src &, const float (&)[G][ELL], const McCtx &,
                                               const v4f (&)[G], const v4f (&)[G], RowAcc<G> &, const Epi &) {}
};

// Combining operations of the wavefront reductions: max for MAX, sum for
// the MPV numerator.
struct OpMax {
    __device__ __forceinline__ static float f(float a, float b) { return fmaxf(a, b); }
};
struct OpSum {
    __device__ __forceinline__ static float f(float a, float b) { return a + b; }
};

template <typename Op, int CTRL>
__device__ __forceinline__ float dpp_row_step(float v) {
    // every lane of a full row reads a valid lane for these controls, so the
    // move can fold into the combining instruction's DPP source
    const int moved = __builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true);
    return Op::f(v, __int_as_float(moved));
}

// Lane-wise combination of two registers after swapping the upper 32 lanes
// of a with the lower 32 lanes of b: lanes 0-31 then reduce a over lane pairs
// (i, i+32), lanes 32-63 reduce b.
template <typename Op>
__device__ __forceinline__ float fold32(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return Op::f(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// The same with 16-lane rows: odd rows of a swap with even rows of b, so
// rows 0 and 2 of the result reduce a over row pairs, rows 1 and 3 reduce b.
template <typename Op>
__device__ __forceinline__ float fold16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return Op::f(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Reduction within each 16-lane row, broadcast to the row.
template <typename Op>
__device__ __forceinline__ float row_reduce(float v) {
    v = dpp_row_step<Op, kDppQuadSwap1>(v);
    v = dpp_row_step<Op, kDppQuadSwap2>(v);
    v = dpp_row_step<Op, kDppRowHalfMirror>(v);
    v = dpp_row_step<Op, kDppRowMirror>(v);
    return v;
}

// Reduce the 4 slot values of one group over the wavefront: on return, the
// lanes of 16-lane row q hold the result of slot slot_of_row(q).
template <typename Op>
__device__ __forceinline__ float reduce4(const v4f &m) {
    return row_reduce<Op>(fold16<Op>(fold32<Op>(m[0], m[1]), fold32<Op>(m[2], m[3])));
}
// fold32(m0, m1): lanes 0-31 slot 0, lanes 32-63 slot 1; fold16 of
// (slot0|slot1) and (slot2|slot3): row 0 slot 0, row 1 slot 2, row 2 slot 1,
// row 3 slot 3.
__device__ constexpr int slot_of_row(int q) { return ((q & 1) << 1) | (q >> 1); }

// The same for the 8 slots of two groups at once: after the 32- and 16-lane
// folds of each group, the two 16-lane rows q of the groups fold over lane
// pairs (i, i+8) into one register (lanes 0-7 of the row keep group 0,
// lanes 8-15 group 1), and three DPP steps finish each 8-lane half-row.  On
// return the lanes 16q + 8h .. 16q + 8h + 7 hold slot slot_of_row(q) of
// group h.  18 vector instructions for 8 slots, against 20 for two reduce4.
template <typename Op>
__device__ __forceinline__ float reduce8(const v4f &m0, const v4f &m1, bool hi8) {
    const float e = fold16<Op>(fold32<Op>(m0[0], m0[1]), fold32<Op>(m0[2], m0[3]));
    const float h = fold16<Op>(fold32<Op>(m1[0], m1[1]), fold32<Op>(m1[2], m1[3]));
    const float re = dpp_row_step<Op, kDppRowRor8>(e);
    const float rh = dpp_row_step<Op, kDppRowRor8>(h);
    float v = hi8 ? rh : re;
    v = dpp_row_step<Op, kDppQuadSwap1>(v);
    v = dpp_row_step<Op, kDppQuadSwap2>(v);
    return dpp_row_step<Op, kDppRowHalfMirror>(v);
}

// The writer lane of a kernel slot after the wavefront reduction (-1: the
// lane writes nothing): lane 16q writes slot slot_of_row(q) of a 4-kernel
// item; lane 16q + 8h writes slot slot_of_row(q) of group h of an 8-kernel
// item.  Returns the slot index 4h + v, or -1.
template <int G>
__device__ __forceinline__ int writer_slot(int lane) {
    if (G == 1) return (lane & 15) == 0 ? slot_of_row(lane >> 4) : -1;
    return (lane & 7) == 0 ? 4 * ((lane >> 3) & 1) + slot_of_row(lane >> 4) : -1;
}

template <int G, bool MPV>
__device__ __forceinline__ void init_row(RowAcc<G> &ra) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
        // -inf into the four running maxima with two 64-bit moves
        v2f lo, hi;
        asm volatile("v_mov_b64 %0, %2\n\tv_mov_b64 %1, %2" : "=v"(lo), "=v"(hi) : "s"(kNegInfPair));
        ra.mx[g] = v4f{lo[0], lo[1], hi[0], hi[1]};
        if (MPV) ra.ps[g] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int v = 0; v < 4; ++v) ra.cnt[g][v] = 0;
    }
}

// One kernel's features from its writer lane: PPV = c / O, MAX, and MPV.
template <bool MPV>
__device__ __forceinline__ void write_features(uint32_t c, float m, float psum, int ok, double inv_O,
                                               float *Frow) {
    // (float)c / (float)O, correctly rounded: for c <= O < 2^24 the quotient
    // is never a float midpoint and lies at least 2^-49 (relative) from one,
    // while c * fl64(1/O) is within 2^-52 of it, so rounding the double
    // product to float gives the same float as the fp32 division
    const float ppv = (float)((double)c * inv_O);
    if (!store_checked(Frow + (MPV ? 3 : 2) * (int64_t)ok, MPV ? 3 : 2)) return;
    if (MPV) {
        // rows of 3 floats: 4-byte aligned only
        float *f = Frow + 3 * (int64_t)ok;
        f[0] = ppv;
        f[1] = m;
        f[2] = c > 0 ? psum / (float)c : 0.0f;
    } else {
        float2 res;
        res.x = ppv;
        res.y = m;
        *reinterpret_cast<float2 *>(Frow + 2 * (int64_t)ok) = res;
    }
}

// MAX (and the MPV numerator) over the wavefront (counts are already
// scalar), then per kernel {PPV, MAX} (or {PPV, MAX, MPV}), written by the
// writer lanes (writer_slot); okid is the kernel id the lane writes, or -1.
template <int G, bool MPV>
__device__ __forceinline__ void write_row(const RowAcc<G> &ra, int okid, double inv_O, float *Frow,
                                          bool hi8) {
    if constexpr (G == 1) {
        const float m = reduce4<OpMax>(ra.mx[0]);
        const float psum = MPV ? reduce4<OpSum>(ra.ps[0]) : 0.0f;
        // the count of slot slot_of_row(q) into writer lane 16q (scalar to
        // lane moves: one instruction each, no lane masks)
        uint32_t c;
        asm volatile(
            "v_writelane_b32 %0, %1, 0\n\t"
            "v_writelane_b32 %0, %2, 16\n\t"
            "v_writelane_b32 %0, %3, 32\n\t"
            "v_writelane_b32 %0, %4, 48"
            : "=&v"(c)
            : "s"(ra.cnt[0][slot_of_row(0)]), "s"(ra.cnt[0][slot_of_row(1)]), "s"(ra.cnt[0][slot_of_row(2)]),
              "s"(ra.cnt[0][slot_of_row(3)]));
        if (okid >= 0) write_features<MPV>(c, m, psum, okid, inv_O, Frow);
    } else {
        const float m = reduce8<OpMax>(ra.mx[0], ra.mx[1], hi8);
        const float psum = MPV ? reduce8<OpSum>(ra.ps[0], ra.ps[1], hi8) : 0.0f;
        // the count of slot slot_of_row(q) of group h into lane 16q + 8h
        uint32_t c;
        asm volatile(
            "v_writelane_b32 %0, %1, 0\n\t"
            "v_writelane_b32 %0, %2, 8\n\t"
            "v_writelane_b32 %0, %3, 16\n\t"
            "v_writelane_b32 %0, %4, 24\n\t"
            "v_writelane_b32 %0, %5, 32\n\t"
            "v_writelane_b32 %0, %6, 40\n\t"
            "v_writelane_b32 %0, %7, 48\n\t"
            "v_writelane_b32 %0, %8, 56"
            : "=&v"(c)
            : "s"(ra.cnt[0][slot_of_row(0)]), "s"(ra.cnt[1][slot_of_row(0)]), "s"(ra.cnt[0][slot_of_row(1)]),
              "s"(ra.cnt[1][slot_of_row(1)]), "s"(ra.cnt[0][slot_of_row(2)]), "s"(ra.cnt[1][slot_of_row(2)]),
              "s"(ra.cnt[0][slot_of_row(3)]), "s"(ra.cnt[1][slot_of_row(3)]));
        if (okid >= 0) write_features<MPV>(c, m, psum, okid, inv_O, Frow);
    }
}

// The row epilogue of run_item as a function object (write_row with the
// item's writer lane, 1/O and the row's F pointer).
template <int G, bool MPV>
struct RowWriter {
    int okid;
    double inv_O;
    float *Frow;
    bool hi8;
    __device__ __forceinline__ void operator()(const RowAcc<G> &ra) const {
        write_row<G, MPV>(ra, okid, inv_O, Frow, hi8);
    }
};

// One work item over the `nrows` series staged in LDS: the item's weights
// are loaded once and reused for every series.  Each series runs the item's
// tiles in blocks of NT (the last block holds the remaining 1..NT tiles).
template <int ELL, int G, bool CLAMP, bool MPV, bool MC>
__device__ __forceinline__ void run_item(const ItemDesc &it, const float *rows0, int nrows,
                                         const FusedArgs &a, float *F0, int lane) {
    constexpr int NT = rocket::kTilesPerBlock[G - 1];
    // A operand: lane holds the weight of kernel slot (lane & 3) for every
    // tap; univariate items keep them in registers for the whole item,
    // multichannel ones read each channel's weights per block (McCtx)
    float wa[G][ELL];
    if constexpr (!MC) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int j = 0; j < ELL; ++j) wa[g][j] = a.wpk[it.w_off + (g * ELL + j) * 4 + (lane & 3)];
    }
    McCtx mc{};
    if constexpr (MC)
        mc = McCtx{a.wpk + it.w_off + (lane & 3), ((uint64_t)it.ch_mask[1] << 32) | it.ch_mask[0], it.n_ch,
                   a.row_stride};
    const int row_pitch = a.C * a.row_stride;  // floats per staged series (LDS offsets fit 32 bits)
    // C operand of the first tap: the bias of block row v (kernel slot v),
    // and in the last tile of a series -inf on the lanes past the last
    // output, so that they change no feature
    const int rem = it.O - (it.n_tiles - 1) * kTile;  // real outputs in the last tile, 1..64
    v4f binit[G], blast[G];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float b = as_const(a.bias)[it.k_off + 4 * g + v];
            // copied into a vector register once per item (an opaque copy,
            // so the compiler keeps it there instead of copying the scalar
            // bias again before every block)
            float bv;
            asm volatile("v_mov_b32 %0, %1" : "=v"(bv) : "s"(b));
            binit[g][v] = bv;
            blast[g][v] = lane < rem ? bv : -INFINITY;
        }
    const int nfull = (it.n_tiles - 1) / NT;  // full blocks before the last block
    const int nv = it.n_tiles - nfull * NT;   // tiles in the last block, 1..NT
    // the kernel id this lane writes after the reduction (-1: not a writer,
    // or an empty slot)
    const int wslot = writer_slot<G>(lane);
    const int okid = wslot >= 0 ? a.kid[it.k_off + wslot] : -1;
    const bool hi8 = (lane & 8) != 0;
    const int64_t f_stride = (int64_t)a.nf * a.K;
    for (int r = 0; r < nrows; ++r) {
        RowAcc<G> ra;
        init_row<G, MPV>(ra);
        const uint32_t row = lds_addr(rows0 + r * row_pitch);  // series index 0
        // block b starts at output b*NT*64; its lane 0 reads series index
        // b*NT*64 - p under tap 0 (a wavefront-uniform offset)
        for (int blk = 0; blk < nfull; ++blk) {
            const int b0 = blk * (NT * kTile) - it.p;
            if constexpr (CLAMP)
                tile_block<ELL, G, NT, false, MPV, MC>(ClampedTiles{row, b0, it.d, a.L}, wa, mc, binit,
                                                       blast, ra);
            else
                tile_block<ELL, G, NT, false, MPV, MC>(PaddedTiles{row + 4u * (uint32_t)b0, it.d}, wa,
                                                       mc, binit, blast, ra);
        }
        const int b0 = nfull * (NT * kTile) - it.p;
        const RowWriter<G, MPV> epi{okid, it.inv_O, F0 + r * f_stride, hi8};
        if constexpr (CLAMP)
            TailTilesThen<ELL, G, NT, MPV, MC, ClampedTiles>::run(nv, ClampedTiles{row, b0, it.d, a.L}, wa, mc,
                                                                  binit, blast, ra, epi);
        else
            TailTilesThen<ELL, G, NT, MPV, MC, PaddedTiles>::run(
                nv, PaddedTiles{row + 4u * (uint32_t)b0, it.d}, wa, mc, binit, blast, ra, epi);
    }
}

__device__ __forceinline__ ItemDesc load_item(ConstPtr<ItemDesc> p) {
    ItemDesc it;
    it.variant = p->variant;
    it.d = p->d;
    it.p = p->p;
    it.O = p->O;
    it.n_tiles = p->n_tiles;
    it.w_off = p->w_off;
    it.k_off = p->k_off;
    it.cost = p->cost;
    it.n_ch = p->n_ch;
    it.ch_off = p->ch_off;
    it.t_off = p->t_off;
    it.nq = p->nq;
    it.ch_mask[0] = p->ch_mask[0];
    it.ch_mask[1] = p->ch_mask[1];
    it.inv_O = p->inv_O;
    return it;
}

// Items of one variant, taken one at a time from the workgroup's counter.
template <int ELL, int G, bool CLAMP, bool MPV, bool MC>
__device__ __forceinline__ void run_items(int *next_item, int beg, int cnt_items,
                                          const float *rows0, int nrows, const FusedArgs &a,
                                          float *F0, int lane) {
    while (true) {
        int idx = 0;
        if (lane == 0) idx = atomicAdd(next_item, 1);
        idx = __builtin_amdgcn_readfirstlane(__shfl(idx, 0, 64));
        if (idx >= cnt_items) break;
        const ItemDesc it = load_item(as_const(a.items) + as_const(a.order)[beg + idx]);
        run_item<ELL, G, CLAMP, MPV, MC>(it, rows0, nrows, a, F0, lane);
    }
}

// What one workgroup does: a row group, one variant, one split of its items.
// ---------------------------------------------------------------------------
// VALU items: the one or two kernels left over in a bucket of a long-series
// plan.  A 4-slot MFMA group would run them with 3 or 2 empty slots, and
// each empty slot still costs its share of the MFMA and of the reduction; on
// the VALU each kernel costs one fp32 FMA per tap and tile (4.5 cycles
// against 8.7 for the 4-slot MFMA) and one result register to reduce.  The
// tiles, blocks (8 tiles), series reads and the -inf start of lanes past O
// are those of a one-group MFMA item; the weights and biases are scalars.
// ---------------------------------------------------------------------------

template <int NK>
struct ValuAcc {
    float mx[NK];
    uint32_t cnt[NK];
    float ps[NK];
};

template <int ELL, int NK, int NT, bool LAST, bool MPV, typename Src>
__device__ __forceinline__ void valu_block(const Src &src, const float (&w)[NK][ELL], const float (&binit)[NK],
                                           const float (&blast)[NK], ValuAcc<NK> &va) {
    float acc[NT][NK];
#pragma unroll
    for (int j = 0; j < ELL; ++j) {
        float xv[NT];
        lds_tiles<NT>(src.m0(j), xv);
        if constexpr (NT > 4) lds_tiles_rest<NT>(xv);
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int c = 0; c < NK; ++c) {
                const float a0 = (j == 0) ? ((LAST && u == NT - 1) ? blast[c] : binit[c]) : acc[u][c];
                acc[u][c] = fmaf(w[c][j], xv[u], a0);
            }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int c = 0; c < NK; ++c) va.cnt[c] += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(acc[u][c] > 0.0f));
    if (MPV) {
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int c = 0; c < NK; ++c) va.ps[c] += fmaxf(acc[u][c], 0.0f);
    }
#pragma unroll
    for (int u = 0; u + 1 < NT; u += 2)
#pragma unroll
        for (int c = 0; c < NK; ++c) va.mx[c] = fmaxf(fmaxf(va.mx[c], acc[u][c]), acc[u + 1][c]);
    if (NT % 2 == 1) {
#pragma unroll
        for (int c = 0; c < NK; ++c) va.mx[c] = fmaxf(va.mx[c], acc[NT - 1][c]);
    }
}

template <int ELL, int NK, int N, bool MPV, typename Src>
struct ValuTail {
    __device__ __forceinline__ static void run(int nv, const Src &src, const float (&w)[NK][ELL],
                                               const float (&binit)[NK], const float (&blast)[NK],
                                               ValuAcc<NK> &va) {
        if (nv == N)
            valu_block<ELL, NK, N, true, MPV>(src, w, binit, blast, va);
        else
            ValuTail<ELL, NK, N - 1, MPV, Src>::run(nv, src, w, binit, blast, va);
    }
};
template <int ELL, int NK, bool MPV, typename Src>
struct ValuTail<ELL, NK, 0, MPV, Src> {
    __device__ __forceinline__ static void run(int, const Src &, const float (&)[NK][ELL], const float (&)[NK],
                                               const float (&)[NK], ValuAcc<NK> &) {}
};

// Combine over the whole wavefront (every lane gets the result).
template <typename Op>
__device__ __forceinline__ float wave_all(float v) {
    return row_reduce<Op>(fold16<Op>(fold32<Op>(v, v), fold32<Op>(v, v)));
}

template <int ELL, int NK, bool CLAMP, bool MPV>
__device__ __forceinline__ void run_valu_item(const ItemDesc &it, const float *rows0, int nrows, const FusedArgs &a,
                                              float *F0, int lane) {
    constexpr int NT = rocket::kTilesPerBlock[0];
    // weights and biases are the same on every lane: scalar registers
    float w[NK][ELL], binit[NK], blast[NK];
    const int rem = it.O - (it.n_tiles - 1) * kTile;
#pragma unroll
    for (int c = 0; c < NK; ++c) {
#pragma unroll
        for (int j = 0; j < ELL; ++j) w[c][j] = as_const(a.wpk)[it.w_off + j * 4 + c];
        const float b = as_const(a.bias)[it.k_off + c];
        float bv;
        asm volatile("v_mov_b32 %0, %1" : "=v"(bv) : "s"(b));
        binit[c] = bv;
        blast[c] = lane < rem ? bv : -INFINITY;
    }
    int kid[NK];
#pragma unroll
    for (int c = 0; c < NK; ++c) kid[c] = as_const(a.kid)[it.k_off + c];
    const int row_pitch = a.C * a.row_stride;
    const int nfull = (it.n_tiles - 1) / NT;
    const int nv = it.n_tiles - nfull * NT;
    const int64_t f_stride = (int64_t)a.nf * a.K;
    for (int r = 0; r < nrows; ++r) {
        ValuAcc<NK> va;
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            va.mx[c] = -INFINITY;
            va.cnt[c] = 0;
            va.ps[c] = 0.0f;
        }
        const uint32_t row = lds_addr(rows0 + r * row_pitch);
        for (int blk = 0; blk < nfull; ++blk) {
            const int b0 = blk * (NT * kTile) - it.p;
            if constexpr (CLAMP)
                valu_block<ELL, NK, NT, false, MPV>(ClampedTiles{row, b0, it.d, a.L}, w, binit, blast, va);
            else
                valu_block<ELL, NK, NT, false, MPV>(PaddedTiles{row + 4u * (uint32_t)b0, it.d}, w, binit, blast, va);
        }
        const int b0 = nfull * (NT * kTile) - it.p;
        if constexpr (CLAMP)
            ValuTail<ELL, NK, NT, MPV, ClampedTiles>::run(nv, ClampedTiles{row, b0, it.d, a.L}, w, binit, blast, va);
        else
            ValuTail<ELL, NK, NT, MPV, PaddedTiles>::run(nv, PaddedTiles{row + 4u * (uint32_t)b0, it.d}, w, binit,
                                                         blast, va);
        float m[NK], psum[NK];
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            m[c] = wave_all<OpMax>(va.mx[c]);
            psum[c] = MPV ? wave_all<OpSum>(va.ps[c]) : 0.0f;
        }
        if (lane == 0) {
#pragma unroll
            for (int c = 0; c < NK; ++c)
                write_features<MPV>(va.cnt[c], m[c], psum[c], kid[c], it.inv_O, F0 + r * f_stride);
        }
    }
}

template <int ELL, int NK, bool CLAMP, bool MPV>
__device__ __forceinline__ void run_valu_items(int *next_item, int beg, int cnt_items, const float *rows0, int nrows,
                                               const FusedArgs &a, float *F0, int lane) {
    while (true) {
        int idx = 0;
        if (lane == 0) idx = atomicAdd(next_item, 1);
        idx = __builtin_amdgcn_readfirstlane(__shfl(idx, 0, 64));
        if (idx >= cnt_items) break;
        const ItemDesc it = load_item(as_const(a.items) + as_const(a.order)[beg + idx]);
        run_valu_item<ELL, NK, CLAMP, MPV>(it, rows0, nrows, a, F0, lane);
    }
}

// ---------------------------------------------------------------------------
// Toeplitz items: the one (NK = 1) or two (NK = 2) kernels left over in a
// bucket at a large dilation d.  The 4 slots of one MFMA group hold the same
// kernel at SIGMA = 4 / NK shifts: slot s is kernel s / SIGMA shifted by
// h = s % SIGMA taps (weight w[m - h] at tap m, ELL + SIGMA - 1 taps), so the
// MFMA chain of lane l reading series index t0 - p + m d + l at tap m
// computes, in slot s, the output at position t0 + l + h d.  Outputs come in
// super-tiles of SIGMA d consecutive positions per kernel: ceil(d / 64)
// chunks at t0 = T + 64 c cover positions T .. T + d - 1 for shift 0 and the
// same plus h d for shift h; lanes with 64 c + l >= d (the last chunk) start
// from -inf, as lanes past O do in an MFMA item's last tile.  The last,
// partial super-tile masks each slot on its own (positions below O) and, in
// the padded layout, clamps its block offsets to at most L (its taps reach
// past the row's margin; see RightClampedTiles).  One
// MFMA chain of ELL + SIGMA - 1 taps thus yields 4 x 64 outputs, where a
// VALU item spends ELL fp32 FMAs per 64 outputs and kernel.
// ---------------------------------------------------------------------------
// Whole super-tiles of NC chunks, P per block (padded rows): the block's
// tiles are the NC chunks of each of P consecutive super-tiles, each
// super-tile's last chunk starting from blast.  Returns the super-tiles
// done, a multiple of P; the caller runs the rest one per block.
template <int TAPS, int NC, int P, bool MPV>
__device__ __forceinline__ int toep_runs(uint32_t row, int p, int d, int span, int s_full,
                                         const float (&wa)[1][TAPS], const v4f (&binit)[1],
                                         const v4f (&blast)[1], RowAcc<1> &ra) {
    const McCtx mc{};
    const int groups = s_full / P;
    const uint32_t sb = 4u * (uint32_t)span;
    for (int gi = 0; gi < groups; ++gi) {
        const int b0 = gi * P * span - p;
        tile_block<TAPS, 1, NC * P, true, MPV, false>(MultiTiles<NC, P>{row + 4u * (uint32_t)b0, d, sb}, wa, mc,
                                                       binit, blast, ra);
    }
    return groups * P;
}

template <int ELL, int NK, bool CLAMP, bool MPV>
__device__ __forceinline__ void run_toep_item(const ItemDesc &it, const float *rows0, int nrows,
                                              const FusedArgs &a, float *F0, int lane) {
    constexpr int SIGMA = 4 / NK;
    constexpr int TAPS = ELL + SIGMA - 1;
    constexpr int NT = rocket::kTilesPerBlock[0];
    float wa[1][TAPS];
#pragma unroll
    for (int j = 0; j < TAPS; ++j) wa[0][j] = a.wpk[it.w_off + j * 4 + (lane & 3)];
    const int d = it.d;
    const int nc = it.n_tiles;                // chunks per super-tile
    const int remc = d - (nc - 1) * kTile;    // positions of a super-tile's last chunk, 1..64
    v4f binit[1], blast[1];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const float b = as_const(a.bias)[it.k_off + v];
        float bv;
        asm volatile("v_mov_b32 %0, %1" : "=v"(bv) : "s"(b));
        binit[0][v] = bv;
        blast[0][v] = lane < remc ? bv : -INFINITY;
    }
    int kid[NK];
#pragma unroll
    for (int q = 0; q < NK; ++q) kid[q] = as_const(a.kid)[it.k_off + q * SIGMA];
    const int span = SIGMA * d;
    const int s_full = it.O / span;
    const int rest = it.O - s_full * span;
    const int nlast = rest > 0 ? (min(rest, d) + kTile - 1) / kTile : 0;
    const int nblk = (nc + NT - 1) / NT;  // blocks per super-tile
    const int bsz = nc / nblk, bextra = nc % nblk;
    const McCtx mc{};
    const int row_pitch = a.row_stride;
    const int64_t f_stride = (int64_t)a.nf * a.K;
    for (int r = 0; r < nrows; ++r) {
        RowAcc<1> ra;
        init_row<1, MPV>(ra);
        const uint32_t row = lds_addr(rows0 + r * row_pitch);
        // super-tiles of at most 4 chunks: several per block (padded rows)
        int st0 = 0;
        if constexpr (!CLAMP) {
            switch (nc) {
                case 1: st0 = toep_runs<TAPS, 1, 4, MPV>(row, it.p, d, span, s_full, wa, binit, blast, ra); break;
                case 2: st0 = toep_runs<TAPS, 2, 4, MPV>(row, it.p, d, span, s_full, wa, binit, blast, ra); break;
                case 3: st0 = toep_runs<TAPS, 3, 2, MPV>(row, it.p, d, span, s_full, wa, binit, blast, ra); break;
                case 4: st0 = toep_runs<TAPS, 4, 2, MPV>(row, it.p, d, span, s_full, wa, binit, blast, ra); break;
                default: break;
            }
        }
        for (int st = st0; st < s_full; ++st) {
            const int T = st * span;
            // nblk blocks of nearly equal size (the first nc % nblk one tile
            // larger), so that no block is left with one or two tiles
            int c0 = 0;
            for (int blk = 0; blk + 1 < nblk; ++blk) {
                const int sz = bsz + (blk < bextra ? 1 : 0);
                const int b0 = T + c0 * kTile - it.p;
                if constexpr (CLAMP)
                    TailTiles<TAPS, 1, NT, MPV, false, ClampedTiles, false>::run(sz, ClampedTiles{row, b0, d, a.L}, wa,
                                                                                 mc, binit, blast, ra);
                else
                    TailTiles<TAPS, 1, NT, MPV, false, PaddedTiles, false>::run(
                        sz, PaddedTiles{row + 4u * (uint32_t)b0, d}, wa, mc, binit, blast, ra);
                c0 += sz;
            }
            const int b0 = T + c0 * kTile - it.p;
            if constexpr (CLAMP)
                TailTiles<TAPS, 1, NT, MPV, false, ClampedTiles>::run(nc - c0, ClampedTiles{row, b0, d, a.L}, wa, mc,
                                                                      binit, blast, ra);
            else
                TailTiles<TAPS, 1, NT, MPV, false, PaddedTiles>::run(nc - c0, PaddedTiles{row + 4u * (uint32_t)b0, d},
                                                                     wa, mc, binit, blast, ra);
        }
        // the last, partial super-tile: chunk by chunk, each slot valid on
        // the lanes whose position is in its chunk's d and below O
        const int T = s_full * span;
        for (int c = 0; c < nlast; ++c) {
            v4f bm[1];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int lim = min(d - c * kTile, it.O - T - c * kTile - (v % SIGMA) * d);
                bm[0][v] = lane < lim ? binit[0][v] : -INFINITY;
            }
            const int b0 = T + c * kTile - it.p;
            if constexpr (CLAMP)
                tile_block<TAPS, 1, 1, true, MPV, false>(ClampedTiles{row, b0, d, a.L}, wa, mc, binit, bm, ra);
            else
                tile_block<TAPS, 1, 1, true, MPV, false>(RightClampedTiles{row, b0, d, a.L}, wa, mc, binit, bm, ra);
        }
        // each kernel's features from its SIGMA slots
#pragma unroll
        for (int q = 0; q < NK; ++q) {
            uint32_t cnt = 0;
            float m = ra.mx[0][q * SIGMA], ps = MPV ? ra.ps[0][q * SIGMA] : 0.0f;
#pragma unroll
            for (int h = 0; h < SIGMA; ++h) cnt += ra.cnt[0][q * SIGMA + h];
#pragma unroll
            for (int h = 1; h < SIGMA; ++h) {
                m = fmaxf(m, ra.mx[0][q * SIGMA + h]);
                if (MPV) ps += ra.ps[0][q * SIGMA + h];
            }
            m = wave_all<OpMax>(m);
            if (MPV) ps = wave_all<OpSum>(ps);
            if (lane == 0 && kid[q] >= 0) write_features<MPV>(cnt, m, ps, kid[q], it.inv_O, F0 + r * f_stride);
        }
    }
}

template <int ELL, int NK, bool CLAMP, bool MPV>
__device__ __forceinline__ void run_toep_items(int *next_item, int beg, int cnt_items, const float *rows0, int nrows,
                                               const FusedArgs &a, float *F0, int lane) {
    while (true) {
        int idx = 0;
        if (lane == 0) idx = atomicAdd(next_item, 1);
        idx = __builtin_amdgcn_readfirstlane(__shfl(idx, 0, 64));
        if (idx >= cnt_items) break;
        const ItemDesc it = load_item(as_const(a.items) + as_const(a.order)[beg + idx]);
        run_toep_item<ELL, NK, CLAMP, MPV>(it, rows0, nrows, a, F0, lane);
    }
}

struct GroupWork {
    int variant;
    int beg;        // first entry of the items' order
    int cnt_items;
    int nrows;      // series staged
    int64_t grow;   // first series (global row)
};

// Row groups go to the XCDs in equal shares, unless that would leave a fifth of
// the chip without work (one series would run on one XCD alone): then the
// workgroups are dealt to the XCDs one by one.  One series, us: 500 samples,
// 10,000 kernels 15.3 -> 9.0, 16,000 samples 513 -> 180; with balanced shares
// (16 and 50 series of 64 to 200 samples) the shares measured 5 % faster.
inline int32_t xcd_shift(int64_t groups) {
    const int64_t slots = (groups + kXcds - 1) / kXcds * kXcds;
    return 5 * groups < 4 * slots ? 0 : kXcdShift;
}

// The row group and the split of workgroup `rest` of a variant (the vi-th of
// the launch) in an XCD's share.  In one share of all XCDs (xcd_shift 0) the
// groups go fastest and each variant starts at another split: the splits that
// have items are the first ones, and with a power of two of splits going
// fastest they would meet on the same few XCDs (6 series of 12,428 samples, 241
// kernels: 103 us).
__device__ __forceinline__ int group_split(int xcd, int xcd_shift, int64_t groups, int nsplit, int vi, int64_t rest,
                                           int64_t &group) {
    if (xcd_shift == 0) {
        group = rest % groups;
        return ((int)(rest / groups) + 5 * vi) & (nsplit - 1);  // nsplit is a power of two
    }
    group = xcd * groups + (rest >> __builtin_ctz(nsplit));
    return (int)rest & (nsplit - 1);
}

// Workgroup = (variant, row group, split).  Workgroup b of the launch's fp32
// part runs on XCD b % 8.
// Every XCD takes its own share of the row groups and walks them variant by
// variant, so all XCDs get the same mix of work while the CUs of an XCD run
// one code variant at a time.  Returns false when the workgroup has nothing
// to do (uniformly for the whole workgroup).
__device__ __forceinline__ bool group_work(const FusedArgs &a, int64_t b, GroupWork &w) {
    const int xcd = (int)b & ((1 << a.xcd_shift) - 1);
    const int64_t local = b >> a.xcd_shift;
    const int64_t per_variant = a.groups_per_xcd * a.nsplit;
    const int vi = (int)(local / per_variant);
    const int64_t rest = local % per_variant;
    int64_t group;
    const int split = group_split(xcd, a.xcd_shift, a.groups_per_xcd, a.nsplit, vi, rest, group);
    w.variant = a.variants[vi];
    w.beg = as_const(a.split_begin)[w.variant * a.nsplit + split];
    w.cnt_items = as_const(a.split_begin)[w.variant * a.nsplit + split + 1] - w.beg;
    const int64_t first = group * a.rows_per_block;
    if (w.cnt_items == 0 || first >= a.n_rows) return false;
    w.nrows = (int)min((int64_t)a.rows_per_block, a.n_rows - first);
    w.grow = a.row0 + first;
    return true;
}

// Stages the group's series (every channel) with their zero margins into
// smem, coalesced (channel c of row r at (r*C + c)*row_stride), and the tail
// pad after them.
template <int BLOCK>
__device__ __forceinline__ bool stage_group(const FusedArgs &a, int64_t b, float *smem, int *next_item,
                                            GroupWork &w) {
    if (!group_work(a, b, w)) return false;
    if (a.vec4) {
        // 4 floats per lane: the series and both margins are whole 16-byte
        // words, so no word straddles a margin
        const int stride4 = a.row_stride >> 2, lo4 = a.halo_lo >> 2, L4 = a.L >> 2;
        for (int rc = 0; rc < w.nrows * a.C; ++rc) {
            const float4 *x = reinterpret_cast<const float4 *>(a.X + ((w.grow * a.C) + rc) * (int64_t)a.L);
            float4 *dst = reinterpret_cast<float4 *>(smem + rc * a.row_stride);
            for (int e = threadIdx.x; e < stride4; e += BLOCK) {
                const int m = e - lo4;
                dst[e] = (m >= 0 && m < L4) ? x[m] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
        }
    } else {
        for (int rc = 0; rc < w.nrows * a.C; ++rc) {
            const float *x = a.X + ((w.grow * a.C) + rc) * (int64_t)a.L;
            float *dst = smem + rc * a.row_stride;
            for (int e = threadIdx.x; e < a.row_stride; e += BLOCK) {
                const int m = e - a.halo_lo;
                dst[e] = (m >= 0 && m < a.L) ? x[m] : 0.0f;
            }
        }
    }
    // zeros after the last row: lanes past the last output of an item read
    // up to tail_pad floats past it
    for (int e = threadIdx.x; e < a.tail_pad; e += BLOCK) smem[w.nrows * a.C * a.row_stride + e] = 0.0f;
    set_check_bounds(smem, (int64_t)w.nrows * a.C * a.row_stride + a.tail_pad,
                     a.F + a.row0 * (int64_t)a.nf * a.K, a.F + (a.row0 + a.n_rows) * (int64_t)a.nf * a.K);
    if (threadIdx.x == 0) *next_item = 0;
    __syncthreads();
    return true;
}

// The univariate MFMA and VALU items of one variant over the staged series.
template <bool CLAMP, bool MPV>
__device__ __forceinline__ void run_variant(int *next_item, const GroupWork &w, const FusedArgs &a, const float *rows0,
                                            float *F0, int lane) {
    const int beg = w.beg, cnt = w.cnt_items, nr = w.nrows;
    switch (w.variant) {
        case 0: run_items<7, 1, CLAMP, MPV, false>(next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 1: run_items<7, 2, CLAMP, MPV, false>(next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 2: run_items<9, 1, CLAMP, MPV, false>(next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 3: run_items<9, 2, CLAMP, MPV, false>(next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 4: run_items<11, 1, CLAMP, MPV, false>(next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 5: run_items<11, 2, CLAMP, MPV, false>(next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        // VALU items (univariate long-series plans)
        case 6: run_valu_items<7, 1, CLAMP, MPV>(next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 7: run_valu_items<7, 2, CLAMP, MPV>(next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 8: run_valu_items<9, 1, CLAMP, MPV>(next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 9: run_valu_items<9, 2, CLAMP, MPV>(next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        case 10: run_valu_items<11, 1, CLAMP, MPV>(next_item, beg, cnt, rows0, nr, a, F0, lane); break;
        default: run_valu_items<11, 2, CLAMP, MPV>(next_item, beg, cnt, rows0, nr, a, F0, lane); break;
    }
}

}  // namespace
