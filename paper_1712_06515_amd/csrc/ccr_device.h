// Device helpers shared by the kernel sources: complex arithmetic, small DFTs, uniform loads and
// the device views of the band and work-item tables.
#pragma once

#include <hip/hip_runtime.h>

#include "ccr_internal.h"

namespace ccr {
namespace {

// Two 32-bit lanes: the data operand of the 64-bit buffer store builtin.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// ------------------------------------------------------------------ complex helpers
template <typename T> struct C2;
template <> struct C2<float> { using type = float2; };
template <> struct C2<double> { using type = double2; };
template <typename T> using c2 = typename C2<T>::type;

template <typename T> __device__ __forceinline__ c2<T> mk(T re, T im) { c2<T> v; v.x = re; v.y = im; return v; }
template <typename T> __device__ __forceinline__ c2<T> cadd(c2<T> a, c2<T> b) { return mk<T>(a.x + b.x, a.y + b.y); }
template <typename T> __device__ __forceinline__ c2<T> csub(c2<T> a, c2<T> b) { return mk<T>(a.x - b.x, a.y - b.y); }
template <typename T> __device__ __forceinline__ c2<T> cmul(c2<T> a, c2<T> b) {
    return mk<T>(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
template <typename T> __device__ __forceinline__ c2<T> cscale(c2<T> a, T s) { return mk<T>(a.x * s, a.y * s); }
// multiply by -i
template <typename T> __device__ __forceinline__ c2<T> cmul_mi(c2<T> a) { return mk<T>(a.y, -a.x); }

template <typename T> __device__ __forceinline__ const c2<T> *twiddles(const BandDev &B);
template <> __device__ __forceinline__ const float2 *twiddles<float>(const BandDev &B) { return B.tw32; }
template <> __device__ __forceinline__ const double2 *twiddles<double>(const BandDev &B) { return B.tw64; }

// Orders the LDS accesses of one wavefront around this point (compiler ordering only: the
// hardware executes a wavefront's LDS operations in issue order).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 4-point forward DFT in place: (a0, a1, a2, a3) -> sum_n a_n exp(-2 pi i n k / 4).
template <typename T>
__device__ __forceinline__ void dft4(c2<T> &a0, c2<T> &a1, c2<T> &a2, c2<T> &a3) {
    const c2<T> t0 = cadd<T>(a0, a2), t1 = csub<T>(a0, a2);
    const c2<T> t2 = cadd<T>(a1, a3), t3 = cmul_mi<T>(csub<T>(a1, a3));
    a0 = cadd<T>(t0, t2);
    a2 = csub<T>(t0, t2);
    a1 = cadd<T>(t1, t3);
    a3 = csub<T>(t1, t3);
}

// 4-point DFT whose last input is zero.
template <typename T>
__device__ __forceinline__ void dft4_z(c2<T> &a0, c2<T> &a1, c2<T> &a2, c2<T> &a3) {
    const c2<T> t0 = cadd<T>(a0, a2), t1 = csub<T>(a0, a2);
    const c2<T> t3 = cmul_mi<T>(a1);
    a0 = cadd<T>(t0, a1);
    a2 = csub<T>(t0, a1);
    a3 = csub<T>(t1, t3);
    a1 = cadd<T>(t1, t3);
}

// 16-point forward DFT in registers, n = 4a + b, k = c + 4d: 4-point DFTs over a, twiddles
// W16^(b c), 4-point DFTs over b.  On return A[k] is held in v[4 (k % 4) + k / 4].  Z4: the
// inputs v[12..15] are zero (their values are not read).
template <typename T, bool Z4 = false>
__device__ __forceinline__ void dft16(c2<T> *v) {
    const T c1 = (T)0.92387953251128675613, s1 = (T)0.38268343236508977173, h = (T)0.70710678118654752440;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if constexpr (Z4) dft4_z<T>(v[b], v[4 + b], v[8 + b], v[12 + b]);
        else dft4<T>(v[b], v[4 + b], v[8 + b], v[12 + b]);
    }
    // v[4c + b] *= W16^(b c)
    v[5] = cmul<T>(v[5], mk<T>(c1, -s1));    // b1 c1: W^1
    v[6] = cmul<T>(v[6], mk<T>(h, -h));      // b2 c1: W^2
    v[7] = cmul<T>(v[7], mk<T>(s1, -c1));    // b3 c1: W^3
    v[9] = cmul<T>(v[9], mk<T>(h, -h));      // b1 c2: W^2
    v[10] = cmul_mi<T>(v[10]);               // b2 c2: W^4 = -i
    v[11] = cmul<T>(v[11], mk<T>(-h, -h));   // b3 c2: W^6
    v[13] = cmul<T>(v[13], mk<T>(s1, -c1));  // b1 c3: W^3
    v[14] = cmul<T>(v[14], mk<T>(-h, -h));   // b2 c3: W^6
    v[15] = cmul<T>(v[15], mk<T>(-c1, s1));  // b3 c3: W^9
#pragma unroll
    for (int c = 0; c < 4; ++c) dft4<T>(v[4 * c], v[4 * c + 1], v[4 * c + 2], v[4 * c + 3]);
}

// 8-point forward DFT in place, natural order: 4-point DFTs of the even and odd inputs, then
// X[k] = E[k] + W8^k O[k], X[k + 4] = E[k] - W8^k O[k].
template <typename T>
__device__ __forceinline__ void dft8(c2<T> *v) {
    const T h = (T)0.70710678118654752440;
    c2<T> e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6], o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
    dft4<T>(e0, e1, e2, e3);
    dft4<T>(o0, o1, o2, o3);
    o1 = cmul<T>(o1, mk<T>(h, -h));
    o2 = cmul_mi<T>(o2);
    o3 = cmul<T>(o3, mk<T>(-h, -h));
    v[0] = cadd<T>(e0, o0);
    v[4] = csub<T>(e0, o0);
    v[1] = cadd<T>(e1, o1);
    v[5] = csub<T>(e1, o1);
    v[2] = cadd<T>(e2, o2);
    v[6] = csub<T>(e2, o2);
    v[3] = cadd<T>(e3, o3);
    v[7] = csub<T>(e3, o3);
}

// Load of a table entry that is the same for every lane (uniform index into memory the kernel
// does not write), through the constant address space: a scalar load, whose wait does not wait
// for the wavefront's outstanding vector loads.
template <typename T> __device__ __forceinline__ T ld_uniform(const T *p, int i) {
    i = __builtin_amdgcn_readfirstlane(i);
    return ((const __attribute__((address_space(4))) T *)p)[i];
}
__device__ __forceinline__ float2 ld_uniform_f2(const float2 *p, int i) {
    const unsigned long long v = ld_uniform(reinterpret_cast<const unsigned long long *>(p), i);
    return make_float2(__uint_as_float((unsigned)v), __uint_as_float((unsigned)(v >> 32)));
}

// Pointers loaded from a device table are generic, and loads through generic pointers are
// slower than global loads (and hold more registers).  as_global() re-derives such a pointer
// from `base`, a kernel argument in global memory, as base + (p - base): the same 64-bit
// address, now known to the compiler to be global memory.
typedef __attribute__((address_space(1))) char gchar;
template <typename T> __device__ __forceinline__ T *as_global(T *p, const gchar *base) {
    const gchar *q = base + ((const char *)p - (const char *)base);
    return (T *)q;
}

// A copy of a band descriptor from the device band table with every pointer re-derived as a
// global-memory pointer.
__device__ __forceinline__ BandDev global_view(const BandDev &b, const void *base_) {
    const gchar *base = (const gchar *)base_;
    BandDev g = b;
    g.x = as_global(b.x, base);
    g.mask = as_global(b.mask, base);
    g.anchors = as_global(b.anchors, base);
    g.earth = as_global(b.earth, base);
    g.win64 = as_global(b.win64, base);
    g.win32 = as_global(b.win32, base);
    g.cheb_x = as_global(b.cheb_x, base);
    g.mono = as_global(b.mono, base);
    g.tw64 = as_global(b.tw64, base);
    g.tw32 = as_global(b.tw32, base);
    g.bin_m = as_global(b.bin_m, base);
    g.bin_p = as_global(b.bin_p, base);
    g.bin_kb = as_global(b.bin_kb, base);
    g.bin_pos = as_global(b.bin_pos, base);
    g.segw = as_global(b.segw, base);
    g.active = as_global(b.active, base);
    g.work = as_global(b.work, base);
    g.seg_work = as_global(b.seg_work, base);
    g.tmpl = as_global(b.tmpl, base);
    g.lagph = as_global(b.lagph, base);
    g.seg_any = as_global(b.seg_any, base);
    g.col_bin = as_global(b.col_bin, base);
    g.class_start = as_global(b.class_start, base);
    g.zero256 = as_global(b.zero256, base);
    g.bin_col = as_global(b.bin_col, base);
    g.farrow = as_global(b.farrow, base);
    g.cls_m0 = as_global(b.cls_m0, base);
    if (b.pw) g.pw = as_global(b.pw, base);
    if (b.pwf) g.pwf = as_global(b.pwf, base);
    g.segwd = as_global(b.segwd, base);
    g.seg_bits = as_global(b.seg_bits, base);
    if (b.lag.on) {
        g.lag.tw32 = as_global(b.lag.tw32, base);
        g.lag.tw64 = as_global(b.lag.tw64, base);
        g.lag.g0 = as_global(b.lag.g0, base);
        g.lag.frac = as_global(b.lag.frac, base);
        g.lag.wt = as_global(b.lag.wt, base);
        if (b.lag.pairw) g.lag.pairw = as_global(b.lag.pairw, base);
    }
    return g;
}

// The item owning block b of a stage: the last item whose first block is <= b.
__device__ __forceinline__ int find_item(const WorkItem *__restrict__ items, int n_items, int stage, int b) {
    int lo = 0, hi = n_items - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (items[mid].first[stage] <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

}  // namespace
}  // namespace ccr
