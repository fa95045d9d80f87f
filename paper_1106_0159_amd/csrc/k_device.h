// Device helpers shared by the Legendre kernels (FP64 and mixed precision).
#pragma once

#include "sht_internal.h"

namespace sht {

// Workgroups are dispatched to the XCDs in turn (workgroup b runs on XCD
// b mod kXcds).  The launchers round the number of m values up to a multiple
// of kMBlock * kXcds, and the k-th workgroup of XCD x takes part k % parts of
// the m value 64 j + 8 x' + r, with (j, r, part) counted out of k (r fastest
// after the part) and x' = x on even j, 7 - x on odd j.  So the parts (slot
// tiles or groups) of one m share one XCD's L2 for its coefficient column,
// the 8 consecutive m whose entries fill one 128-byte line of a Delta row are
// written (read) through the same L2, m still ascends in launch order, and
// the snake order keeps the XCDs' shares of the work equal.  Within an XCD the
// dispatcher deals workgroups to its 4 shader engines in turn and waits for the
// one whose turn it is: with an even number of parts each engine would get the
// same parts of every m, the short polar tiles or the long equatorial ones, and
// the first would idle (a fifth of the CU time at 4 tiles), so the parts of
// successive m start one further on.  Synthesis at HEALPix 2048 / lmax 4096 (4
// tiles) 3.05 -> 2.60 ms, 1024 / 2048 (2 tiles) 424 -> 408 us; analysis at 2048
// / 4096 (2 groups) 4.97 -> 4.21 ms with the ring stage (all with a recurrence of 6
// operations for two degrees instead of 7).  A grid that is all resident at
// once waits for nothing and keeps the plain order (HEALPix 347: 85 us, turned 88).
constexpr int kXcds = 8;
constexpr int kMBlock = 8;  // m values per 128-byte line of a Delta row
constexpr unsigned kTurnMin = 2048;  // workgroups, 8 per CU
struct MPart {
    int m, part;
};
__device__ __forceinline__ MPart xcd_m_part(int parts) {
    const int x = blockIdx.x % kXcds, k = blockIdx.x / kXcds;
    const int per = kMBlock * parts;
    const int j = k / per, rem = k - j * per;
    const int xs = (j & 1) ? kXcds - 1 - x : x;
    const int r = rem / parts;
    const int turn = parts % 2 || gridDim.x < kTurnMin ? 0 : parts == 2 ? r / 2 : r;
    return {(j * kXcds + xs) * kMBlock + r, (rem + turn) % parts};
}

// number of m values launched: mmax + 1 rounded up to a multiple of kMBlock * kXcds
inline int64_t padded_m(int mmax) {
    constexpr int64_t q = (int64_t)kMBlock * kXcds;
    return ((int64_t)mmax + q) / q * q;
}
inline bool grid_ok(int64_t n) { return n > 0 && n < (int64_t)INT32_MAX; }

// One load from each of the first 128-byte lines, one per thread, of p[stride * i],
// i0 <= i <= i1 (addresses clamped to i1, so every load is in bounds).  The
// workgroup's pass over a coefficient column brings it into this XCD's L2
// ahead of the wave-uniform loads that use it; the value is only handed to an
// empty asm at the end of the kernel, so nothing waits for it before then.
__device__ __forceinline__ double warm_l2(const double *p, int stride, int i0, int i1) {
    const int per_line = 16 / stride;  // entries per 128 bytes
    const int i = min(i0 + per_line * (int)threadIdx.x, i1);
    return p[(int64_t)stride * i];
}

// Wave-wide min / max, returned as a wave-uniform (scalar) value so that
// loops bounded by it stay uniform and their coefficient loads scalar.  Lane
// exchanges in registers (DPP within a row of 16, then the permlane swaps):
// six dependent LDS permutes instead would add about 0.2 us to every kernel's start.
template <class Op>
__device__ __forceinline__ int wave_reduce(int v, Op op) {
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, false));   // quad_perm [1,0,3,2]
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, false));   // quad_perm [2,3,0,1]
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, false));  // row_half_mirror
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, false));  // row_mirror
    const auto r16 = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
    v = op((int)r16[0], (int)r16[1]);
    const auto r32 = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
    return __builtin_amdgcn_readfirstlane(op((int)r32[0], (int)r32[1]));
}
__device__ __forceinline__ int wave_min(int v) {
    return wave_reduce(v, [](int a, int b) { return min(a, b); });
}
__device__ __forceinline__ int wave_max(int v) {
    return wave_reduce(v, [](int a, int b) { return max(a, b); });
}

// Read-only coefficient data (recurrence coefficients, scaled a_lm) seen
// through the constant address space: nothing a kernel stores may alias it,
// so loads at wave-uniform addresses become scalar (SGPR) loads.  (Pointers
// taken from a struct lose the __restrict__ that tells the compiler so.)
template <class T>
using const_ptr = const __attribute__((address_space(4))) T *;
template <class T>
__device__ __forceinline__ const_ptr<T> ro(const T *p) {
    return (const_ptr<T>)p;
}
// complex entries of such an array (re, im interleaved), loaded 16 bytes at a time
typedef double dvec2 __attribute__((ext_vector_type(2)));
struct ConstC {
    const_ptr<dvec2> p;
    __device__ __forceinline__ double2 operator[](int64_t i) const {
        const dvec2 v = p[i];
        return make_double2(v.x, v.y);
    }
};
__device__ __forceinline__ ConstC ro(const double2 *p) { return ConstC{ro(reinterpret_cast<const dvec2 *>(p))}; }

// A wave-uniform 64-bit value restated as such (for addresses that must stay
// on scalar registers).
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

}  // namespace sht
