// Device helpers shared by the two- and three-dimensional steps: wrapped row indices, accesses
// at a uniform base plus a lane's byte offset, reciprocals.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tcg {
namespace {

__device__ __forceinline__ int wrapi(int a, int n)
{
    int r = a % n;
    return r < 0 ? r + n : r;
}

// Successive row indices modulo n, the same in every lane: wrapped once at the start, then
// advanced by one per row on the scalar unit.  (Integer division has no scalar instruction:
// a % n per row would move every row address of the march into vector registers.)
struct RowCursor {
    int r, n;
    __device__ RowCursor(int a, int n_) : r(__builtin_amdgcn_readfirstlane(wrapi(a, n_))), n(n_) {}
    // the current row, then advance
    __device__ int next()
    {
        const int c = r;
        r = r + 1 == n ? 0 : r + 1;
        return c;
    }
};

// Row pointers that are the same in every lane are rebuilt from scalar registers in the
// global address space, opaque to the optimiser, so that they are not re-associated with
// the per-lane column offset (which would turn every access into a hoisted 64-bit
// per-lane address) and every access compiles to the scalar-base + 32-bit vector-offset
// form of the global load/store.
__device__ __forceinline__ uint64_t uniform_u64(uint64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

template <typename T>
__device__ __forceinline__ T ld_at(const T* base, unsigned byte_off)
{
    typedef const __attribute__((address_space(1))) char gchar;
    typedef const __attribute__((address_space(1))) T gT;
    gchar* b = (gchar*)uniform_u64(reinterpret_cast<uint64_t>(base));
    return *(gT*)(b + byte_off);
}
// Stores of the new state are non-temporal: nothing reads them again within the step, and
// keeping them out of the caches leaves the caches to the halo rows and columns that
// neighbouring workgroups re-read (measured: +1% at 512 threads, +19% at 256, FP64).
template <typename T>
__device__ __forceinline__ void st_at(T* base, unsigned byte_off, T v)
{
    typedef __attribute__((address_space(1))) char gchar;
    typedef __attribute__((address_space(1))) T gT;
    gchar* b = (gchar*)uniform_u64(reinterpret_cast<uint64_t>(base));
    __builtin_nontemporal_store(v, (gT*)(b + byte_off));
}

template <typename T>
__device__ __forceinline__ void st_plain(T* base, unsigned byte_off, T v)
{
    typedef __attribute__((address_space(1))) char gchar;
    typedef __attribute__((address_space(1))) T gT;
    gchar* b = (gchar*)uniform_u64(reinterpret_cast<uint64_t>(base));
    *(gT*)(b + byte_off) = v;
}

// A per-lane byte offset the optimiser must take as new: left alone, it widens the offset to 64
// bits outside the loop and every access takes a 64-bit vector addition.
__device__ __forceinline__ void refresh(uint32_t& o) { asm volatile("" : "+v"(o)); }

// Access at a scalar base address (pinned there: plane offsets hoisted out of a loop end up in
// vector registers, at four instructions per access) plus a 32-bit lane offset.  Stores are
// non-temporal, as st_at's.
template <typename T>
__device__ __forceinline__ T ld_sbase(uint64_t& base, uint32_t byte_off)
{
    typedef const __attribute__((address_space(1))) char gchar;
    typedef const __attribute__((address_space(1))) T gT;
    asm volatile("" : "+s"(base));
    return *(gT*)((gchar*)base + byte_off);
}
template <typename T>
__device__ __forceinline__ void st_sbase(uint64_t& base, uint32_t byte_off, T v)
{
    typedef __attribute__((address_space(1))) char gchar;
    typedef __attribute__((address_space(1))) T gT;
    asm volatile("" : "+s"(base));
    __builtin_nontemporal_store(v, (gT*)((gchar*)base + byte_off));
}

// The plane stride as a value the optimiser must take afresh at each row: left alone, it
// hoists the 18 or 27 plane offsets of a row out of the march loop and keeps them all live
// in scalar registers, which then spill to vector lanes (FP32 storage: 91 spilled scalars,
// about 190 lane moves per row).  Recomputed per row they cost a few scalar multiplies.
__device__ __forceinline__ int64_t fresh_stride(int64_t s)
{
    asm volatile("" : "+s"(s));
    return s;
}

// 1/x for a positive normal x (densities, relaxation-time denominators): the hardware
// reciprocal estimate y refined to within about an ulp, in place of the IEEE division
// sequence: with e = 1 - x y (the estimate's relative error, below 2^-23 in FP64), by
// y (1 + e + e^2) in FP64, whose error is e^3, and by a Newton step y (1 + e) in FP32.
template <typename C>
__device__ __forceinline__ C recip(C x)
{
    if constexpr (sizeof(C) == 8) {
        const double y = __builtin_amdgcn_rcp(x);
        const double e = fma(-x, y, 1.0);
        return fma(y, fma(e, e, e), y);
    } else {
        const float y = __builtin_amdgcn_rcpf(x);
        return fmaf(y, fmaf(-x, y, 1.0f), y);
    }
}

// 1/sqrt(s) for a positive normal s, the same way: with e = 1 - s y^2, y (1 + e/2 + 3 e^2/8) in
// FP64 and a Newton step in FP32.
template <typename C>
__device__ __forceinline__ C rsqrt_nr(C s)
{
    if constexpr (sizeof(C) == 8) {
        const double y = __builtin_amdgcn_rsq(s);
        const double e = fma(-s * y, y, 1.0);
        return fma(y * e, fma(0.375, e, 0.5), y);
    } else {
        const float y = __builtin_amdgcn_rsqf(s);
        const float h = 0.5f * y;
        return fmaf(y, fmaf(-s * y, h, 0.5f), y);
    }
}

}  // namespace
}  // namespace tcg
