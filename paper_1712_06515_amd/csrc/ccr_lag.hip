// Spectra and pair sums on a lag-resolved frequency grid.
//
// With every segment's transform referenced to the segment's own first sample, the pair term
// at segment lag d = K - L is
//   S_d(f) = sum_K conj(F_K(f)) F_{K-d}(f),   rho(f) = sum_d Re[e^{2 pi i f d N_K} S_d(f)]
// (f in cycles per sample; weights left out).  S_d is the Fourier transform of the segments'
// sample correlation, whose sample lags lie within +-(N_K - 1), whatever d and however many
// segments are summed.  A frequency grid of N_G >= 2 N_K - 1 points therefore determines every
// S_d, and its values at the output bins (N_FFT points, 4.6 (2R + 1) N_K and up) follow by
// band-limited interpolation once per template, after the sum over segments, instead of a
// transform at every output bin in every segment: 2 transforms of 1024 points a segment in
// place of 32 for the 240-day, lag-4 band, and no per-segment phase rotation.
//
//   k_lag         transforms and pair sums: S_d on the grid's bins inside the band plus the
//                 interpolation margin, per (template, chunk of segments, residue class)
//   k_lag_reduce  chunk sums
//   k_lag_finish  interpolation to the output bins, lag phases, sqrt(2) / N
//
// Accuracy.  Errors of S_d at one grid point reach the bins within half the taps of it, so they are
// relative to the largest S_d there, where a transform at the bin itself rounds relative to the bin's own
// value.  Against the FP64 path on noise and signals up to rho ~ 1e3 the error is smaller than that of the
// kernels before the grid at every lag (rms 2.1 - 2.8e-7 in place of 2.5 - 7.8e-7).  Beside a signal of
// rho = 1e4, 1e6 and 1e7 and up the worst bin at lags above 0 is off by 3e-5, 1 to 3e-4 and 1e-3 of max(|rho|, 1)
// (before: 3e-6, 2e-5, 6e-5), from the FP32 rounding of the products at the peak (6e-8 of it, over the
// root of the segments) and the taps' stop band (3e-10 of it); at lag 0 less than before at any strength.
// FP64: the same as before below 1e6, up to 3.4 times at 2e7 (1.2e-10 -> 4.2e-10).
#include <type_traits>

#include "ccr_device.h"
#include "ccr_internal.h"

namespace ccr {
namespace {

// ------------------------------------------------------------------ one-wavefront FFT

// Exchange of a lane's V complex values through a T array: the real parts, then the imaginary
// parts (half the LDS of a complex exchange; every lane has stored its real parts before any
// register is overwritten, and a wavefront's LDS operations execute in issue order).
// wr(k) is the value index and LDS index of store k, rd(r) the LDS index of load r.
template <typename T, int V, typename WI, typename WP, typename RD>
__device__ __forceinline__ void exchange(c2<T> *v, T *ex, WI wi, WP wp, RD rd) {
#pragma unroll
    for (int k = 0; k < V; ++k) ex[wp(k)] = v[wi(k)].x;
    wave_sync();
#pragma unroll
    for (int r = 0; r < V; ++r) v[r].x = ex[rd(r)];
    wave_sync();
#pragma unroll
    for (int k = 0; k < V; ++k) ex[wp(k)] = v[wi(k)].y;
    wave_sync();
#pragma unroll
    for (int r = 0; r < V; ++r) v[r].y = ex[rd(r)];
    wave_sync();
}

// Pass twiddles of this lane for the NS-point FFT of residue class p (q = p + P m0, W = W_{N_G},
// N_G = P NS; `tw` holds its N_G powers).  The class's input twiddle W^(q s), s = lane + 64 r,
// splits into the uniform W^(64 q r), applied to the input, and W^(q lane), which commutes
// through the first pass (a DFT over r for one lane) and is folded into the second pass's
// twiddles: its butterfly l reads first-pass outputs of butterfly (l + 64 r) / V.
// Index of this lane's factor in `tw`: a(r), r < V, of the second pass; b(r), r >= 1, of the third
// (1024 points: b(4 j + r) of its butterfly j); c(r), r >= 1, of the fourth (256 points).
template <int NS> struct LagIdx;
template <> struct LagIdx<1024> {
    static constexpr int NA = 16, NB = 16, NC [[maybe_unused]] = 0;
    static __device__ __forceinline__ unsigned a(int r, int P, int q, int lane) {
        return ((unsigned)(r * (lane & 15) * 4 * P) + (unsigned)q * (unsigned)((lane >> 4) + 4 * r)) % (unsigned)(P * 1024);
    }
    static __device__ __forceinline__ unsigned b(int r, int P, int lane) {
        return (unsigned)((r & 3) * (lane + 64 * (r >> 2)) * P) % (unsigned)(P * 1024);
    }
    static __device__ __forceinline__ unsigned c(int, int, int) { return 0; }
};
template <> struct LagIdx<512> {
    static constexpr int NA = 8, NB = 8, NC = 0;
    static __device__ __forceinline__ unsigned a(int r, int P, int q, int lane) {
        return ((unsigned)(r * (lane & 7) * 8 * P) + (unsigned)q * (unsigned)((lane >> 3) + 8 * r)) % (unsigned)(P * 512);
    }
    static __device__ __forceinline__ unsigned b(int r, int P, int lane) {
        return (unsigned)(r * lane * P) % (unsigned)(P * 512);
    }
    static __device__ __forceinline__ unsigned c(int, int, int) { return 0; }
};
template <> struct LagIdx<256> {
    static constexpr int NA = 4, NB = 4, NC = 4;
    static __device__ __forceinline__ unsigned a(int r, int P, int q, int lane) {
        return ((unsigned)(r * (lane & 3) * 16 * P) + (unsigned)q * (unsigned)((lane >> 2) + 16 * r)) % (unsigned)(P * 256);
    }
    static __device__ __forceinline__ unsigned b(int r, int P, int lane) {
        return (unsigned)(r * (lane & 15) * 4 * P) % (unsigned)(P * 256);
    }
    static __device__ __forceinline__ unsigned c(int r, int P, int lane) {
        return (unsigned)(r * lane * P) % (unsigned)(P * 256);
    }
};

// The factors in registers, or (1024 points) in LDS, one copy a workgroup: 56 registers a lane
// less, which is what lets four wavefronts share a SIMD.
template <typename T, int NS, bool LDS> struct LagTw;
template <typename T, int NS> struct LagTw<T, NS, false> {
    using I = LagIdx<NS>;
    c2<T> va[I::NA], vb[I::NB], vc[I::NC > 0 ? I::NC : 1];
    __device__ __forceinline__ void load(const c2<T> *tw, c2<T> *, int P, int q, int lane) {
#pragma unroll
        for (int r = 0; r < I::NA; ++r) va[r] = tw[I::a(r, P, q, lane)];
#pragma unroll
        for (int r = 1; r < I::NB; ++r) vb[r] = tw[I::b(r, P, lane)];
#pragma unroll
        for (int r = 1; r < I::NC; ++r) vc[r] = tw[I::c(r, P, lane)];
    }
    __device__ __forceinline__ c2<T> a(int r) const { return va[r]; }
    __device__ __forceinline__ c2<T> b(int r) const { return vb[r]; }
    __device__ __forceinline__ c2<T> c(int r) const { return vc[r]; }
};
template <typename T, int NS> struct LagTw<T, NS, true> {
    using I = LagIdx<NS>;
    const c2<T> *l;
    __device__ __forceinline__ void load(const c2<T> *tw, c2<T> *lds, int P, int q, int lane) {
        for (int e = threadIdx.x; e < 64 * (I::NA + I::NB); e += blockDim.x) {
            const int r = e >> 6, ln = e & 63;
            lds[e] = tw[r < I::NA ? I::a(r, P, q, ln) : I::b(r - I::NA, P, ln)];
        }
        l = lds + lane;
        __syncthreads();
    }
    __device__ __forceinline__ c2<T> a(int r) const { return l[64 * r]; }
    __device__ __forceinline__ c2<T> b(int r) const { return l[64 * (I::NA + r)]; }
    __device__ __forceinline__ c2<T> c(int) const { return l[0]; }
};

// 256 points, FP32: four transforms a wavefront, 16 lanes each (lane t of a group holds x[t + 16 r]
// in v[r]): passes of radix 16 and 16 with one exchange where the 64-lane form takes three, at the
// same arithmetic a transform and a quarter of the per-unit overhead (six bands of 3 detectors with
// lag 1, whole call: 8.5 -> 8.3 ms; same-time pairs: see k_lag_same).  l: the factors
// W256^(k t) W^(q t) of the first pass's output k, q as above (16 x 16, LDS, one copy a workgroup;
// the groups' reads coincide), times `scale`, which multiplies the spectra.
struct LagTwQuad {
    const float2 *l;
    __device__ __forceinline__ void load(const float2 *tw, float2 *lds, int P, int q, int lane, float scale = 1.0f) {
        for (int e = threadIdx.x; e < 256; e += blockDim.x)
            lds[e] = cscale<float>(tw[((unsigned)(P * (e >> 4) + q) * (unsigned)(e & 15)) % (unsigned)(P * 256)], scale);
        l = lds + (lane & 15);
        __syncthreads();
    }
    __device__ __forceinline__ float2 a(int k) const { return l[16 * k]; }
};

// One group's transform through `ex` (16 rows of 17); on return X[t + 16 k] is in v[4 (k % 4) + k / 4].
// Groups without a unit (on = false) leave LDS alone.  Z4: the inputs v[12..15] are zero (not read).
template <bool Z4 = false>
__device__ __forceinline__ void lag_fft_quad(float2 *v, float *ex, const LagTwQuad &tw, int t, bool on) {
    dft16<float, Z4>(v);
#pragma unroll
    for (int k = 0; k < 16; ++k) v[4 * (k & 3) + (k >> 2)] = cmul<float>(v[4 * (k & 3) + (k >> 2)], tw.a(k));
    if (on) {
#pragma unroll
        for (int k = 0; k < 16; ++k) ex[17 * k + t] = v[4 * (k & 3) + (k >> 2)].x;
        wave_sync();
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r].x = ex[17 * t + r];
        wave_sync();
#pragma unroll
        for (int k = 0; k < 16; ++k) ex[17 * k + t] = v[4 * (k & 3) + (k >> 2)].y;
        wave_sync();
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r].y = ex[17 * t + r];
    }
    dft16<float>(v);
}

// NS-point forward FFT of one wavefront (V = NS / 64 values a lane, x[l + 64 r] in v[r] on
// entry, X[l + 64 J] in v[J] on return), self-sorting passes of radix 16, 16, 4 (1024, FP32), 8, 8, 8
// (512) or 4, 4, 4, 4 (256, FP64): a pass of radix V with stride Ns has butterfly l read a[l + 64 r],
// twiddle input r and write output r to (l / Ns) V Ns + l % Ns + r Ns.  Between passes the values
// go through `ex` (at most NS + 64 entries), padded so that the lanes served together -- 32 for
// 4-byte values, 16 for 8-byte ones -- fall on distinct banks on both sides: 4-byte values at
// i + i / 32 in the first exchange and with 16 (8) entries after each 256 (64) in the second,
// 8-byte values at i + i / V.  By the counters that holds for 4-byte values (no conflict cycles); in
// FP64 0.30 (512 points) to 0.37 (256) of the LDS cycles are still conflicts.
template <typename T, bool L>
__device__ __forceinline__ void lag_fft(c2<T> *v, T *ex, const LagTw<T, 1024, L> &t, int lane) {
    const int g = lane >> 4, k = lane & 15;
    auto perm = [](int i) { return 4 * (i & 3) + (i >> 2); };
    dft16<T>(v);
    static_assert(sizeof(T) == 4, "1024 points: FP32 only");
    exchange<T, 16>(v, ex, perm, [&](int i) { return 16 * lane + (lane >> 1) + i; },
                    [&](int r) { return lane + (lane >> 5) + 66 * r; });
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = cmul<T>(v[r], t.a(r));
    dft16<T>(v);
    exchange<T, 16>(v, ex, perm, [&](int i) { return 272 * g + k + 16 * i; },
                    [&](int r) { return lane + 64 * (r & 3) + 272 * (r >> 2); });
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // v[j + 4 r] = a[l + 64 j + 256 r]
#pragma unroll
        for (int r = 1; r < 4; ++r) v[j + 4 * r] = cmul<T>(v[j + 4 * r], t.b(4 * j + r));
        dft4<T>(v[j], v[j + 4], v[j + 8], v[j + 12]);
    }
}

template <typename T, bool L>
__device__ __forceinline__ void lag_fft(c2<T> *v, T *ex, const LagTw<T, 512, L> &t, int lane) {
    const int g = lane >> 3, k = lane & 7;
    auto id = [](int i) { return i; };
    dft8<T>(v);
    if constexpr (sizeof(T) == 4)
        exchange<T, 8>(v, ex, id, [&](int i) { return 8 * lane + (lane >> 2) + i; },
                       [&](int r) { return lane + (lane >> 5) + 66 * r; });
    else
        exchange<T, 8>(v, ex, id, [&](int i) { return 9 * lane + i; }, [&](int r) { return lane + g + 72 * r; });
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = cmul<T>(v[r], t.a(r));
    dft8<T>(v);
    if constexpr (sizeof(T) == 4)
        exchange<T, 8>(v, ex, id, [&](int i) { return 72 * g + k + 8 * i; }, [&](int r) { return lane + 72 * r; });
    else
        exchange<T, 8>(v, ex, id, [&](int i) { return 72 * g + k + 9 * i; }, [&](int r) { return lane + g + 72 * r; });
#pragma unroll
    for (int r = 1; r < 8; ++r) v[r] = cmul<T>(v[r], t.b(r));
    dft8<T>(v);
}

template <typename T, bool L>
__device__ __forceinline__ void lag_fft(c2<T> *v, T *ex, const LagTw<T, 256, L> &t, int lane) {
    const int g4 = lane >> 2, k4 = lane & 3, g16 = lane >> 4, k16 = lane & 15;
    auto id = [](int i) { return i; };
    auto rd = [&](int r) { return lane + g4 + 80 * r; };
    static_assert(sizeof(T) == 8, "256 points in FP32 run four to a wavefront");
    dft4<T>(v[0], v[1], v[2], v[3]);
    exchange<T, 4>(v, ex, id, [&](int i) { return 5 * lane + i; }, rd);
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = cmul<T>(v[r], t.a(r));
    dft4<T>(v[0], v[1], v[2], v[3]);
    exchange<T, 4>(v, ex, id, [&](int i) { return 20 * g4 + k4 + 5 * i; }, rd);
#pragma unroll
    for (int r = 1; r < 4; ++r) v[r] = cmul<T>(v[r], t.b(r));
    dft4<T>(v[0], v[1], v[2], v[3]);
    exchange<T, 4>(v, ex, id, [&](int i) { return 80 * g16 + k16 + (k16 >> 2) + 20 * i; }, rd);
#pragma unroll
    for (int r = 1; r < 4; ++r) v[r] = cmul<T>(v[r], t.c(r));
    dft4<T>(v[0], v[1], v[2], v[3]);
}

// ------------------------------------------------------------------ uniform reads and buffer loads

template <typename T> __device__ __forceinline__ c2<T> ld_uniform_c2(const c2<T> *p, int i);
template <> __device__ __forceinline__ float2 ld_uniform_c2<float>(const float2 *p, int i) { return ld_uniform_f2(p, i); }
template <> __device__ __forceinline__ double2 ld_uniform_c2<double>(const double2 *p, int i) {
    const double *d = reinterpret_cast<const double *>(p);
    return make_double2(ld_uniform(d, 2 * i), ld_uniform(d, 2 * i + 1));
}

// Byte offset past any series (with room for a row's offset): reads there give zero.
constexpr unsigned kLagNone = 0xffff0000u;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// Value at byte offset `lane` + 64 r values (`lane`: the lane's own byte offset, opaque to the
// compiler so that the rows' offsets stay additions, which the load's immediate field holds).
template <typename T> __device__ __forceinline__ c2<T> ld_buf(__amdgpu_buffer_rsrc_t rs, int lane, int r);
template <> __device__ __forceinline__ float2 ld_buf<float>(__amdgpu_buffer_rsrc_t rs, int lane, int r) {
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, lane + 512 * r, 0, 0));
}
template <> __device__ __forceinline__ double2 ld_buf<double>(__amdgpu_buffer_rsrc_t rs, int lane, int r) {
    return __builtin_bit_cast(double2, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(rs, lane + 1024 * r, 0, 0));
}

template <typename T> struct LagTab;
template <> struct LagTab<float> {
    static __device__ __forceinline__ const float2 *tw(const LagDev &G) { return G.tw32; }
    static __device__ __forceinline__ const float2 *step(const LagDev &G) { return G.step32; }
    static __device__ __forceinline__ const float2 *segw(const LagDev &G) { return G.segwf; }
    static __device__ __forceinline__ const float2 *pw(const BandDev &B) { return B.pwf; }
};
template <> struct LagTab<double> {
    static __device__ __forceinline__ const double2 *tw(const LagDev &G) { return G.tw64; }
    static __device__ __forceinline__ const double2 *step(const LagDev &G) { return G.step64; }
    static __device__ __forceinline__ const double2 *segw(const LagDev &G) { return G.segwd; }
    static __device__ __forceinline__ const double2 *pw(const BandDev &B) { return B.pw; }
};

// ------------------------------------------------------------------ spectra and pair sums

// The detectors a workgroup sums over: all of them (both pair kinds, or lag 0), one (pairs
// within a detector: one problem a detector) or two (pairs across detectors with lags: one
// problem a pair of detectors).
struct LagDets {
    int n, d0, d1;
    __device__ __forceinline__ int at(int i) const { return i == 0 ? d0 : (i == 1 ? d1 : i); }
};

// Streams of one grid column at the step's kLagSegs segments from the spectra in LDS: NST = 2:
// the sums over the detectors of hat a_X F_X and hat b_X F_X (n[t] = {A, B}); NST = 4 (two
// detectors, pairs across them only): {a_0, a_1, b_0, b_1}.  s0[t]: the same-time products of the
// pairs X < Y, Re[conj(a_X) a_Y + conj(b_X) b_Y], or for Gamma^circ Im[conj(b_X) a_Y - conj(a_X) b_Y]
// (a workgroup with more than one detector always sums pairs across them; in FP64 s0[t] adds up
// over the step).  PS (per-sample antenna functions): the two streams are transforms of their own.
// DET64 (lag 0 in FP32, no halo): each detector's product goes to acc0 in FP64 by itself, as in the
// path these bands had before the grid.  WR: the weights with the part that rounding them to FP32
// leaves, for the bands whose pair weights were formed in FP64 before the grid (four more
// instructions a spectrum: six bands of 3 detectors, three of them such, 8.00 -> 8.13 ms).
template <typename T, int ND, int NST, bool PS, bool WR, bool DET64>
__device__ __forceinline__ void lag_gather(const BandDev &B, const LagDets &D, const char *slots, int slot_bytes,
                                           int col, int Kb, int nd, bool circ, T (&s0)[kLagSegs], c2<T> (&n)[kLagSegs][NST],
                                           double &acc0) {
    const int NDr = ND > 0 ? ND : nd;
    constexpr int NM = ND > 0 ? ND : CCR_MAX_DET_K;
#pragma unroll
    for (int t = 0; t < kLagSegs; ++t) {
        c2<T> A = mk<T>((T)0, (T)0), Bs = A;
        T z = sizeof(T) == 8 && t > 0 ? s0[t > 0 ? t - 1 : 0] : (T)0;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            if (ND == 0 && i >= nd) continue;  // uniform
            const int u = (t * NDr + i) * (PS ? 2 : 1);
            const c2<T> f = reinterpret_cast<const c2<T> *>(slots + (size_t)u * slot_bytes)[col];
            c2<T> a, b;
            if constexpr (PS) {
                a = f;
                b = reinterpret_cast<const c2<T> *>(slots + (size_t)(u + 1) * slot_bytes)[col];
            } else {
                const int e = D.at(i) * (B.n_seg + 2 * kLagSegs) + kLagSegs + Kb + t;
                const c2<T> w = ld_uniform_c2<T>(LagTab<T>::segw(B.lag), e);
                if constexpr (WR) {  // and what is left of the FP64 weights: one rounding, of the product
                    const float2 r = ld_uniform_f2(B.lag.segwl, e);
                    a = mk<T>(fma(f.x, w.x, f.x * r.x), fma(f.y, w.x, f.y * r.x));
                    b = mk<T>(fma(f.x, w.y, f.x * r.y), fma(f.y, w.y, f.y * r.y));
                } else {
                    a = cscale<T>(f, w.x);
                    b = cscale<T>(f, w.y);
                }
            }
            if (i > 0) {
                if constexpr (DET64) z = (T)0;
                if (circ) {
                    z = fma(Bs.x, a.y, fma(-Bs.y, a.x, z));
                    z = fma(-A.x, b.y, fma(A.y, b.x, z));
                } else {
                    z = fma(A.x, a.x, fma(A.y, a.y, z));
                    z = fma(Bs.x, b.x, fma(Bs.y, b.y, z));
                }
                if constexpr (DET64) acc0 += (double)z;
            }
            if constexpr (NST == 4) {
                n[t][i & 1] = a;
                n[t][2 + (i & 1)] = b;
            }
            A = i == 0 ? a : cadd<T>(A, a);
            Bs = i == 0 ? b : cadd<T>(Bs, b);
        }
        if constexpr (NST == 2) {
            n[t][0] = A;
            n[t][1] = Bs;
        }
        s0[t] = z;
    }
}

// One workgroup of W wavefronts: residue class p of the grid (grid index p + P (m0 + i), i <
// span), chunk c of segments [K0, K1) with the RM >= R segments before it as halo, one
// template.  Steps of kLagSegs segments:
//   Transforms.  Unit (segment, detector[, stream]): one wavefront reads the segment's N_K
//   samples (rows past N_S fold onto the first N_S: the grid's classes need sums over residues
//   mod N_S only), applies the class's input twiddle, transforms them and writes the class's
//   bins inside the band to the unit's LDS slot, which also serves as the transform's exchange
//   buffer.  Units of absent segments write zeros.  The next unit's input is loaded meanwhile.
//   Pair sums.  Lane j of the workgroup owns column j: it forms the step's streams, multiplies each
//   segment's with those of the RM segments before it -- the step's own or the last step's, kept in
//   registers -- and adds them to S_1 .. S_RM (lags above R are computed and dropped).  FP32 products
//   of a segment and lag are summed in FP32 (at lag 0 alone: of a segment and detector), the sums in
//   FP64.
// Two barriers a step.  Partials: [comp][P][span], comp 0: S_0 (same-time pairs across
// detectors), 2 d - 1 and 2 d: Re and Im of S_d.
//
// Bound at 1024 points, lag 4: VALU issue (83 % busy; transforms ~70 % of the instructions).  FP64: not
// the arithmetic (22 % busy) but latency at two wavefronts a SIMD (6.6 - 7 a CU): 226 registers, of
// which the twiddles take 64, ~75 spilled scalars, and the exchanges' bank conflicts.
// Registers: the 1024-point lag-4 form holds its 128 with 20 vector and 73 scalar registers spilled (40
// bytes a lane), the 512-point FP64 forms for pairs across detectors only spill 82 and 91 vector
// registers (about 300 bytes a lane: streams of both detectors are kept; 256 points would hold them, which
// the planner's instruction counts do not see), the quad forms ~94 scalars.
// 60 templates of the 240-day, lag-4 band: transforms at every output bin with window sums over
// an LDS ring of spectra 80.4 ms; this kernel with two columns a lane, twiddles in registers (256,
// two wavefronts a SIMD), per-unit scalar searches and one bank conflict a read 10.9 ms; one
// column a lane and twiddles in LDS (four wavefronts a SIMD), halo as whole steps, fused
// multiply-adds in the products 8.4 ms; conflict-free padding and table lookups for the activity
// masks and weights 7.25 ms; segments added in FP64 one by one (fewer sums held) 6.87 ms.  FP64, 5
// templates of 120 days: 23.4 ms (spectra through memory) -> 0.95 ms.
template <typename T, int NS, int RM, bool CR, bool PS, int CM>
__device__ __forceinline__ void lag_body(const BandDev &B, const c2<T> *__restrict__ y, double *__restrict__ part,
                                         int k_chunk, int n_chunks, int c, int sub, int p, int tb) {
    extern __shared__ __align__(16) char smem[];
    constexpr bool QUAD = lag_quad(NS, sizeof(T) == 8);
    constexpr int V = lag_values(NS, sizeof(T) == 8);  // values a lane
    constexpr int RL = NS / V;                          // input row: lanes of one transform
    constexpr int GR = 64 / RL;                         // transforms a wavefront takes at once
    constexpr int S = PS ? 2 : 1;
    constexpr int NST = CR ? 4 : 2;
    constexpr bool LTW = lag_tw_lds(NS, sizeof(T) == 8) > 0;
    constexpr bool ALL64 = sizeof(T) == 8;  // a step's products have one sum
    constexpr bool DET64 = RM == 0 && !ALL64;
    const LagDev &G = B.lag;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int W = blockDim.x >> 6;
    const int n_k = B.n_k, R = B.R, P = G.P, span = G.span, nf = G.nfold;
    constexpr bool WR = (CM & 4) != 0;
    const bool circ = (CM & 3) == 2 ? B.weight != 0 : (CM & 3) == 1;
    // the workgroup's detectors
    LagDets D{B.Q, 0, 1};
    if (G.n_sub > 1 || CR) {
        if (!(B.pairs & 1)) {
            D = LagDets{1, sub, sub};
        } else {
            int X = 0, r = sub;
            while (r >= B.Q - 1 - X) {
                r -= B.Q - 1 - X;
                ++X;
            }
            D = LagDets{2, X, X + 1 + r};
        }
    }
    const int nd = D.n;
    const int slot_bytes = G.slot_bytes;
    const int nunit = kLagSegs * nd;  // units of a step (times the streams)

    std::conditional_t<QUAD, LagTwQuad, LagTw<T, NS, LTW>> tw;
    tw.load(LagTab<T>::tw(G), reinterpret_cast<c2<T> *>(smem), P, (p + P * G.m0) % G.ng, lane);
    char *slots = smem + lag_tw_lds(NS, sizeof(T) == 8);
    const c2<T> *step = LagTab<T>::step(G) + (size_t)p * V * nf;

    // steps of kLagSegs segments from K0 on, after one of halo segments (of which the R before K0 count)
    const int K0 = c * k_chunk, K1 = min(B.n_seg, K0 + k_chunk), Kh = max(0, K0 - R);
    const int Ks = RM > 0 && K0 > 0 ? K0 - kLagSegs : K0;
    const int64_t nr = (int64_t)B.n_seg * n_k;
    const c2<T> *yb = y + (size_t)tb * B.Q * nr;

    // active units of the step at Kb: bit t nd + i.  The table holds them per first segment (with a
    // step of zeros at either end); the chunk's ends cut the first and the last step.
    const uint32_t *tab = G.step_bits + (size_t)sub * (B.n_seg + 2 * kLagSegs) + kLagSegs;
    auto step_mask = [&](int Kb) -> unsigned {
        unsigned m = ld_uniform(tab, Kb);
        if (Kb < Kh) m &= ~0u << ((Kh - Kb) * nd);
        if (Kb + kLagSegs > K1) m &= (1u << ((K1 - Kb) * nd)) - 1u;
        return m;
    };
    const unsigned all = nunit >= 32 ? ~0u : (1u << nunit) - 1u;
    // n-th set bit of m (from 0), n < popcount(m)
    auto nth = [&](unsigned m, int n) -> int {
        if (m == all) return n;
        if constexpr (GR == 1) {  // uniform
            for (int k = 0; k < n; ++k) m &= m - 1;
            return __builtin_ctz(m);
        } else {  // a lane each: by halves
            int pos = 0;
#pragma unroll
            for (int w = 16; w > 0; w >>= 1) {
                const int low = __builtin_popcount((m >> pos) & ((1u << w) - 1u));
                if (n >= low) {
                    n -= low;
                    pos += w;
                }
            }
            return pos;
        }
    };
    const unsigned rnd = (65536u + nd - 1) / nd;  // u / nd = u rnd >> 16 for u < 32, nd <= 8
    const int tl = lane & (RL - 1);               // lane within the transform's row
    int lo = tl * (int)sizeof(c2<T>);
    asm("" : "+v"(lo));
    // input of segment K of detector det; reads past its N_K samples give zero (on = false: all)
    auto src = [&](const c2<T> *base, int det, int K, bool on) {
        return __builtin_amdgcn_make_buffer_rsrc((void *)(base + (size_t)det * nr + (size_t)K * n_k), (short)0,
                                                 on ? n_k * (int)sizeof(c2<T>) : 0, 0x00020000);
    };
    // four transforms a wavefront: every lane reads at its own group's byte offset `at` into the
    // template's series (or its weights, laid out alike); rows past N_K and groups without a unit
    // read past the range, which gives zero
    auto ld_quad = [&](__amdgpu_buffer_rsrc_t rs, unsigned at, unsigned at_last, int n, int r) -> float2 {
        const int s0 = RL * r;
        const unsigned o = s0 + RL <= n ? at : (s0 < n ? at_last : kLagNone);
        return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(o + (unsigned)(s0 * 8)), 0, 0));
    };
    // n_k, opaque: a row's comparison with it is redone (two scalar instructions) instead of held
    auto fresh = [](int n) {
        asm volatile("" : "+s"(n));
        return n;
    };
    auto last_of = [&](unsigned at) { return tl < n_k % RL ? at : kLagNone; };
    auto whole = [&](const c2<T> *base) {
        return __builtin_amdgcn_make_buffer_rsrc((void *)base, (short)0, (int)(unsigned)(B.Q * nr * 8), 0x00020000);
    };
    // this wavefront's (unit, stream) pairs in order: number GR in + group of the step at iK; nxt holds
    // their input, ip their place (unit S + stream, -1: none; of this lane's group), iat its offset
    c2<T> nxt[V];
    int iK = Ks, in = wv, ip = -1;
    unsigned iat = kLagNone;
    bool have = false;
    unsigned im = step_mask(Ks);
    auto seek = [&]() {  // to the first pairs at or after the iterator's place
        int cnt = __builtin_popcount(im) * S;
        while (GR * in >= cnt && iK + kLagSegs < K1) {
            iK += kLagSegs;
            im = step_mask(iK);
            in = wv;
            cnt = __builtin_popcount(im) * S;
        }
        have = GR * in < cnt;
        if constexpr (QUAD) {
            const int n = GR * in + (lane >> 4);
            ip = n < cnt ? nth(im, n / S) * S + n % S : -1;
            const int u = max(ip, 0) / S, t = (int)((unsigned)u * rnd >> 16), i = u - t * nd;
            iat = ip < 0 ? kLagNone : (unsigned)(D.at(i) * nr + (int64_t)(iK + t) * n_k) * 8u + (unsigned)lo;
            const __amdgpu_buffer_rsrc_t rs = whole(yb);
            const unsigned last = last_of(iat);
            const int nk = fresh(n_k);
#pragma unroll
            for (int r = 0; r < V; ++r) nxt[r] = ld_quad(rs, iat, last, nk, r);
        } else {
            ip = have ? nth(im, in / S) * S + in % S : -1;
            const int u = max(ip, 0) / S, t = (int)((unsigned)u * rnd >> 16), i = u - t * nd;
            const __amdgpu_buffer_rsrc_t rs = src(yb, D.at(i), have ? iK + t : 0, have);
#pragma unroll
            for (int r = 0; r < V; ++r) nxt[r] = ld_buf<T>(rs, lo, r);
        }
    };
    seek();

    c2<T> hist[RM > 0 ? RM : 1][NST];
    double acc0 = 0.0, acc[RM > 0 ? 2 * RM : 1];
#pragma unroll
    for (int k = 0; k < (RM > 0 ? 2 * RM : 1); ++k) acc[k] = 0.0;
#pragma unroll
    for (int d = 0; d < (RM > 0 ? RM : 1); ++d)
#pragma unroll
        for (int j = 0; j < NST; ++j) hist[d][j] = mk<T>((T)0, (T)0);
    const int col = min((int)threadIdx.x, span - 1);

#pragma unroll 1
    for (int Kb = Ks; Kb < K1; Kb += kLagSegs) {
        const unsigned mask = step_mask(Kb);
        if (mask == 0) {  // no spectra in the step (uniform over the workgroup)
#pragma unroll
            for (int d = 0; d < (RM > 0 ? RM : 1); ++d)
#pragma unroll
                for (int j = 0; j < NST; ++j) hist[d][j] = mk<T>((T)0, (T)0);
            continue;
        }
        // transforms of this wavefront's pairs
#pragma unroll 1
        while (have && iK == Kb) {
            const int pl = ip, s = PS ? max(pl, 0) % S : 0;
            const unsigned at = iat;
            const int u = max(pl, 0) / S, t = (int)((unsigned)u * rnd >> 16), i = u - t * nd;
            char *slot = slots + (size_t)max(pl, 0) * slot_bytes;
            // input row r + V j (j > 0: rows past N_S) and its weight
            auto from = [&](const c2<T> *base) {
                if constexpr (QUAD) return whole(base);
                else return src(base, D.at(i), Kb + t, true);
            };
            auto row = [&](__amdgpu_buffer_rsrc_t rs, int r) -> c2<T> {
                if constexpr (QUAD) return ld_quad(rs, at, last_of(at), n_k, r);
                else return ld_buf<T>(rs, lo, r);
            };
            c2<T> v[V];
            if constexpr (PS) {
                const __amdgpu_buffer_rsrc_t rw = from(LagTab<T>::pw(B));
#pragma unroll
                for (int r = 0; r < V; ++r) {
                    const c2<T> w = row(rw, r);
                    v[r] = cscale<T>(nxt[r], s ? w.y : w.x);
                }
                if (p > 0) {
#pragma unroll
                    for (int r = 0; r < V; ++r) v[r] = cmul<T>(v[r], ld_uniform_c2<T>(step, r));
                }
            } else if (p > 0) {
#pragma unroll
                for (int r = 0; r < V; ++r) v[r] = cmul<T>(nxt[r], ld_uniform_c2<T>(step, r));
            } else {
#pragma unroll
                for (int r = 0; r < V; ++r) v[r] = nxt[r];
            }
            // the next input is loaded while this one is transformed
            in += W;
            seek();
            for (int j = 1; j < nf; ++j) {
                const __amdgpu_buffer_rsrc_t rs = from(yb), rw = from(PS ? LagTab<T>::pw(B) : yb);
#pragma unroll
                for (int r = 0; r < V; ++r) {
                    if (RL * r + NS * j >= n_k) continue;  // uniform
                    c2<T> z = row(rs, r + V * j);
                    if constexpr (PS) {
                        const c2<T> w = row(rw, r + V * j);
                        z = cscale<T>(z, s ? w.y : w.x);
                    }
                    v[r] = cadd<T>(v[r], cmul<T>(z, ld_uniform_c2<T>(step, r + V * j)));
                }
            }
            if constexpr (QUAD) {
                lag_fft_quad(v, reinterpret_cast<float *>(slot), tw, tl, pl >= 0);
                if (pl >= 0) {
                    wave_sync();
#pragma unroll
                    for (int k = 0; k < 16; ++k)
                        if (16 * k < span) reinterpret_cast<c2<T> *>(slot)[tl + 16 * k] = v[4 * (k & 3) + (k >> 2)];
                }
            } else {
                lag_fft<T>(v, reinterpret_cast<T *>(slot), tw, lane);
                wave_sync();
#pragma unroll
                for (int J = 0; J < V; ++J)
                    if (64 * J < span) reinterpret_cast<c2<T> *>(slot)[lane + 64 * J] = v[J];
            }
        }
        // zeros for the units without a spectrum
        {
            unsigned off = ~mask & all;
            for (int k = 0; off; off &= off - 1, ++k) {
                if (k % W != wv) continue;
                c2<T> *slot = reinterpret_cast<c2<T> *>(slots + (size_t)(__builtin_ctz(off) * S) * slot_bytes);
                for (int e = lane; e < S * slot_bytes / (int)sizeof(c2<T>); e += 64) slot[e] = mk<T>((T)0, (T)0);
            }
        }
        __syncthreads();
        if (wv * 64 < span) {  // uniform: some lane of this wavefront has a column
            c2<T> n[kLagSegs][NST];
            T s0[kLagSegs];
            if constexpr (CR) {
                lag_gather<T, 2, NST, PS, WR, DET64>(B, D, slots, slot_bytes, col, Kb, nd, circ, s0, n, acc0);
            } else {
                switch (nd) {
                    case 1: lag_gather<T, 1, NST, PS, WR, DET64>(B, D, slots, slot_bytes, col, Kb, nd, circ, s0, n, acc0); break;
                    case 2: lag_gather<T, 2, NST, PS, WR, DET64>(B, D, slots, slot_bytes, col, Kb, nd, circ, s0, n, acc0); break;
                    case 3: lag_gather<T, 3, NST, PS, WR, DET64>(B, D, slots, slot_bytes, col, Kb, nd, circ, s0, n, acc0); break;
                    default: lag_gather<T, 0, NST, PS, WR, DET64>(B, D, slots, slot_bytes, col, Kb, nd, circ, s0, n, acc0); break;
                }
            }
            if (Kb >= K0) {  // uniform; halo segments only enter the history
#pragma unroll
                for (int t = ALL64 ? kLagSegs - 1 : 0; t < kLagSegs && !DET64; ++t) acc0 += (double)s0[t];
                if constexpr (RM > 0) {
                    T st[2 * RM];
#pragma unroll
                    for (int k = 0; k < 2 * RM; ++k) st[k] = (T)0;
#pragma unroll
                    for (int t = 0; t < kLagSegs; ++t) {
                        // x[j]: the stream multiplied with the earlier segment's stream h[j]
                        c2<T> x[NST];
                        if constexpr (NST == 2) {
                            x[0] = circ ? n[t][1] : n[t][0];
                            x[1] = circ ? mk<T>(-n[t][0].x, -n[t][0].y) : n[t][1];
                        } else {
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                x[j] = circ ? n[t][3 - j] : n[t][1 - j];
                                x[2 + j] = circ ? mk<T>(-n[t][1 - j].x, -n[t][1 - j].y) : n[t][3 - j];
                            }
                        }
#pragma unroll
                        for (int d = 1; d <= RM; ++d) {
                            T re = ALL64 ? st[2 * d - 2] : (T)0, im = ALL64 ? st[2 * d - 1] : (T)0;
#pragma unroll
                            for (int j = 0; j < NST; ++j) {
                                const c2<T> h = t >= d ? n[t >= d ? t - d : 0][j] : hist[d > t ? d - t - 1 : 0][j];
                                re = fma(x[j].x, h.x, fma(x[j].y, h.y, re));
                                im = fma(x[j].x, h.y, fma(-x[j].y, h.x, im));
                            }
                            if constexpr (ALL64) {
                                st[2 * d - 2] = re;
                                st[2 * d - 1] = im;
                            } else {
                                acc[2 * d - 2] += (double)re;
                                acc[2 * d - 1] += (double)im;
                            }
                        }
                    }
                    if constexpr (ALL64) {
#pragma unroll
                        for (int k = 0; k < 2 * RM; ++k) acc[k] += (double)st[k];
                    }
                }
            }
            // the step's last RM segments become the history (kLagSegs >= RM)
            if constexpr (RM > 0) {
#pragma unroll
                for (int d = 0; d < RM; ++d)
#pragma unroll
                    for (int j = 0; j < NST; ++j) hist[d][j] = n[kLagSegs - 1 - d][j];
            }
        }
        __syncthreads();
    }
    if ((int)threadIdx.x >= span) return;
    const int nc = 2 * R + 1;
    double *o = part + (((size_t)tb * n_chunks + c) * G.n_sub + sub) * nc * P * span + (size_t)p * span + threadIdx.x;
    o[0] = acc0;
    if constexpr (RM > 0) {
#pragma unroll
        for (int k = 0; k < 2 * RM; ++k)
            if (k + 1 < nc) o[(size_t)(k + 1) * P * span] = acc[k];
    }
}

// ------------------------------------------------------------------ same-time pairs, 256 points

// First index of the ascending list x[0 .. n) with x >= key, by the whole wavefront (64 probes a round).
__device__ __forceinline__ int lower_wave(const int *x, int n, int key, int lane) {
    int a = 0;
    while (n > 0) {
        const int step = (n + 63) >> 6, i = lane * step;
        const int below = __builtin_popcountll(__ballot(i < n && x[i] < key));
        if (below == 0) return a;
        // x[a + (below - 1) step] < key <= x[a + below step], where that exists
        const int lo = (below - 1) * step + 1, hi = min(n, below * step);
        a += lo;
        x += lo;
        n = hi - lo;
    }
    return a;
}

// Same-time pair sums (R = 0) of a 256-point grid without LDS slots or barriers: a wavefront takes
// four segments at once, a 16-lane group each, and transforms one detector after the other, so that
// every detector's spectrum of a segment lies in the same registers of the same lanes and the
// products are formed there.  The groups take consecutive entries of seg_any, the segments with a
// pair (gaps cost nothing); the workgroup's four wavefronts take the chunk's quadruples in turn and
// add up at the end.  A lane keeps outputs t + 16 k, k < NO (16 NO >= span; the second pass is
// pruned to them at compile time).  NR: input rows of 16 that hold samples, 8, 12 or 16 for N_K up to
// 128, 192 or 256; of 12 and 16 all but the last four are full, and only these need their ends looked at.
// The pairs of detector Y with those before it add F_Y . sum_X (wa_Y u_X + wb_Y v_X) G_X (a product
// of 2-vectors) with weights wa, wb = hat a, hat b times the scale, u = wa, v = wb and G = F; for
// Gamma^circ u = wb, v = -wa and G = i F.  QK = 2 to 4 detectors: the G_X are kept as they are and the
// pair weights wa_Y u_X + wb_Y v_X come from the band's table (formed in FP64, rounded once: as
// products of FP32 factors they were off by up to three roundings); any other number (QK = 0): as the
// sums of u_X G_X and of v_X G_X.  The twiddles carry a power of two (G.scale) that keeps unweighted
// products of spectra as far from FP32's ends as weighted ones, whatever the data's unit.
//
// (One workgroup for both classes, in step so that they read the segments together: 4.33 ms instead
// of 4.06, though the two read the series 1.9 times over: that traffic does not set the time.)
// Bound: VALU issue, one instruction in 3.6 cycles of a SIMD (the derived share of profiles, which takes
// every instruction for four cycles, reads 1.1), ~112 instructions a transform of which ~95 are its
// passes and twiddles; four wavefronts a SIMD.  512 templates of the 120-day band (2 detectors, 30 % gaps,
// two classes of 179-sample segments, 137 bins): the 256-point spectra + pairs kernel, which runs
// every step through an LDS ring, 7.2 ms; k_lag with four transforms a wavefront 6.5 ms; this kernel
// 4.8 ms, with chunks of up to 1024 segments (a wavefront gets ~35 steps, not 9) 4.25 ms, with one
// weight a pair in place of the two sums for 2 and 3 detectors 4.06 ms; 4.1 with the weights from the table.
template <int NO, int NR, int QK>
__device__ __forceinline__ void lag_same_body(const BandDev &B, const float2 *__restrict__ y, double *__restrict__ part,
                                              int k_chunk, int n_chunks, int c, int sub, int p, int tb) {
    extern __shared__ __align__(16) char smem[];
    constexpr int NF = NR == 8 ? 0 : NR - 4;  // full rows
    const LagDev &G = B.lag;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int g = lane >> 4, t = lane & 15;
    const int n_k = B.n_k, Q = QK > 0 ? QK : B.Q, P = G.P, span = G.span;
    const bool circ = B.weight != 0;
    LagTwQuad tw;
    tw.load(G.tw32, reinterpret_cast<float2 *>(smem), P, (p + P * G.m0) % G.ng, lane, G.scale);
    char *ex = smem + lag_tw_lds(256, false) + wv * 4 * kLagQuadSlot;
    const float2 *step = G.step32 + (size_t)p * 16;

    // entries [lo, hi) of seg_any; pairs within a detector only: none
    const int K0 = c * k_chunk, K1 = min(B.n_seg, K0 + k_chunk);
    const int lo = lower_wave(B.seg_any, B.n_seg_any, K0, lane);
    const int hi = (B.pairs & 1) ? lower_wave(B.seg_any, B.n_seg_any, K1, lane) : lo;
    const unsigned nr = (unsigned)(B.n_seg * n_k);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(y + (size_t)tb * Q * nr), (short)0, (int)((unsigned)Q * nr * 8u), 0x00020000);
    const int nlast = n_k & 15;

    auto seg = [&](int e) { return e < hi ? B.seg_any[e] : -1; };
    auto det_bits = [&](int K) { return K >= 0 ? B.seg_bits[K] : 0u; };
    constexpr int NPW = QK > 0 ? QK * (QK - 1) / 2 : 1;
    float2 nxt[NR], wn = make_float2(0.0f, 0.0f);
    float pwn[QK > 1 ? QK - 1 : 1];
    // input of detector i of this group's segment K and its weights, or those of its pairs with the
    // detectors before it; on: it has a spectrum.  Rows past N_K and segments without one read past the
    // buffer's range, which gives zero.
    auto load = [&](int K, bool on, int i) {
        const unsigned at = on ? ((unsigned)i * nr + (unsigned)(K * n_k + t)) * 8u : kLagNone;
        const unsigned last = t < nlast ? at : kLagNone;
        int n = n_k;
        asm volatile("" : "+s"(n));  // the rows' comparisons are redone (two scalar instructions each), not held
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const unsigned o = r < NF || 16 * r + 16 <= n ? at : (16 * r < n ? last : kLagNone);
            nxt[r] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(o + 128u * r), 0, 0));
        }
        if constexpr (QK > 0) {
#pragma unroll
            for (int X = 0; X < QK - 1; ++X)
                if (X < i) pwn[X] = on ? G.pairw[K * NPW + i * (i - 1) / 2 + X] : 0.0f;
        } else {
            wn = make_float2(0.0f, 0.0f);
            if (on) wn = G.segwf[i * (B.n_seg + 2 * kLagSegs) + kLagSegs + K];
        }
    };

    double acc[NO];
#pragma unroll
    for (int k = 0; k < NO; ++k) acc[k] = 0.0;
    // the input is loaded one transform ahead, a step's activity bits one step and its segment two
    int eb = lo + 4 * wv;
    int Ka = seg(eb + g), Kb = seg(eb + 16 + g);
    unsigned ba = det_bits(Ka);
    load(Ka, ba & 1u, 0);
#pragma unroll 1
    for (; eb < hi; eb += 16) {
        const unsigned bb = det_bits(Kb);
        const int Kc = seg(eb + 32 + g);
        // spectra of detector i, while the next input is loaded (a step without the detector costs
        // its transform all the same: a branch round it took a quarter of the registers)
        auto spectra = [&](float2 *v, int i) {
            if (p > 0) {
#pragma unroll
                for (int r = 0; r < NR; ++r) v[r] = cmul<float>(nxt[r], ld_uniform_c2<float>(step, r));
            } else {
#pragma unroll
                for (int r = 0; r < NR; ++r) v[r] = nxt[r];
            }
            if (i + 1 < Q) load(Ka, (ba >> (i + 1)) & 1u, i + 1);
            else load(Kb, bb & 1u, 0);
            if constexpr (NR == 8) {
#pragma unroll
                for (int r = 8; r < 12; ++r) v[r] = make_float2(0.0f, 0.0f);
            }
            lag_fft_quad<(NR <= 12)>(v, reinterpret_cast<float *>(ex + g * kLagQuadSlot), tw, t, true);
            wave_sync();
        };
        auto turned = [&](float2 f) { return circ ? make_float2(-f.y, f.x) : f; };
        if constexpr (QK > 0) {
            float2 G_[QK - 1][NO];
#pragma unroll
            for (int i = 0; i < QK; ++i) {
                float pw[QK - 1];
#pragma unroll
                for (int X = 0; X < QK - 1; ++X) pw[X] = pwn[X];
                float2 v[16];
                spectra(v, i);
#pragma unroll
                for (int k = 0; k < NO; ++k) {
                    const float2 f = v[4 * (k & 3) + (k >> 2)];
                    if (i == 1) {
                        acc[k] += (double)(pw[0] * fma(f.x, G_[0][k].x, f.y * G_[0][k].y));
                    } else if (i > 1) {
                        float cx = pw[i - 1] * G_[i - 1][k].x, cy = pw[i - 1] * G_[i - 1][k].y;
#pragma unroll
                        for (int X = i - 2; X >= 0; --X) {
                            cx = fma(pw[X], G_[X][k].x, cx);
                            cy = fma(pw[X], G_[X][k].y, cy);
                        }
                        acc[k] += (double)fma(f.x, cx, f.y * cy);
                    }
                    if (i + 1 < QK) G_[i][k] = turned(f);
                }
            }
        } else {
            float2 A[NO], Bs[NO];
#pragma unroll 1
            for (int i = 0; i < Q; ++i) {
                const float2 w = wn, uv = circ ? make_float2(w.y, -w.x) : w;
                float2 v[16];
                spectra(v, i);
                if (i == 0) {
#pragma unroll
                    for (int k = 0; k < NO; ++k) {
                        const float2 f = turned(v[4 * (k & 3) + (k >> 2)]);
                        A[k] = cscale<float>(f, uv.x);
                        Bs[k] = cscale<float>(f, uv.y);
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < NO; ++k) {
                        const float2 f = v[4 * (k & 3) + (k >> 2)], h = turned(f);
                        const float cx = fma(w.x, A[k].x, w.y * Bs[k].x), cy = fma(w.x, A[k].y, w.y * Bs[k].y);
                        acc[k] += (double)fma(f.x, cx, f.y * cy);
                        A[k] = make_float2(fma(uv.x, h.x, A[k].x), fma(uv.x, h.y, A[k].y));
                        Bs[k] = make_float2(fma(uv.y, h.x, Bs[k].x), fma(uv.y, h.y, Bs[k].y));
                    }
                }
            }
        }
        Ka = Kb;
        ba = bb;
        Kb = Kc;
    }
    // the groups, then the wavefronts (each through its own exchange area)
    double *red = reinterpret_cast<double *>(ex);
#pragma unroll
    for (int k = 0; k < NO; ++k) {
        double v = acc[k];
        v += __shfl_xor(v, 16);
        v += __shfl_xor(v, 32);
        if (g == 0) red[16 * k + t] = v;
    }
    __syncthreads();
    const int x = threadIdx.x;
    if (x >= span) return;
    const char *r0 = smem + lag_tw_lds(256, false) + 8 * x;
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w) v += *reinterpret_cast<const double *>(r0 + w * 4 * kLagQuadSlot);
    part[(((size_t)tb * n_chunks + c) * G.n_sub + sub) * P * span + (size_t)p * span + x] = v;
}

// Blocks of an item: G = n_tmpl n_chunks n_sub groups of P class workgroups; the dispatcher
// hands workgroups to the 8 XCDs in turn, so a group's classes get indices with equal value mod
// 8 and read the group's resampled series through one XCD's L2.
struct LagPlace {
    int c, sub, p, t;  // chunk, problem, class, template
};
__device__ __forceinline__ LagPlace lag_place(const WorkItem &it, const LagDev &L) {
    const int l = blockIdx.x - it.first[kStSpectra];
    const int P = L.P, G = it.n_tmpl * it.n_chunks * L.n_sub;
    const int full = (G >> 3) * 8 * P;
    int g, p;
    if (l < full) {
        const int r = l >> 3;
        p = r % P;
        g = (r / P) * 8 + (l & 7);
    } else {
        g = (G >> 3) * 8 + (l - full) / P;
        p = (l - full) % P;
    }
    const int per = it.n_chunks * L.n_sub;
    return {(g % per) / L.n_sub, g % L.n_sub, p, g / per};
}

template <typename T, int NS, int RM, bool CR, bool PS, int CM>
__global__ void __launch_bounds__(lag_max_threads(NS, sizeof(T) == 8))
k_lag(const BandDev *__restrict__ bands, const WorkItem *__restrict__ items, int n_items,
      const c2<T> *__restrict__ y, double *__restrict__ part) {
    const WorkItem &it = items[find_item(items, n_items, kStSpectra, blockIdx.x)];
    const BandDev B = global_view(bands[it.band], bands);
    const LagPlace w = lag_place(it, B.lag);
    lag_body<T, NS, RM, CR, PS, CM>(B, y + it.y_off, part + it.part_off, it.k_chunk, it.n_chunks, w.c, w.sub, w.p, w.t);
}

template <int NO, int NR, int QK>
__global__ void __launch_bounds__(256, NO > 6 ? 2 : (QK == 2 && NR <= 12 ? 4 : 3))
k_lag_same(const BandDev *__restrict__ bands, const WorkItem *__restrict__ items, int n_items,
           const float2 *__restrict__ y, double *__restrict__ part) {
    const WorkItem &it = items[find_item(items, n_items, kStSpectra, blockIdx.x)];
    const BandDev B = global_view(bands[it.band], bands);
    const LagPlace w = lag_place(it, B.lag);
    lag_same_body<NO, NR, QK>(B, y + it.y_off, part + it.part_off, it.k_chunk, it.n_chunks, w.c, w.sub, w.p, w.t);
}

// ------------------------------------------------------------------ interpolation to the output bins

// Sum of a template's chunk (and detector) partials into the first one, one thread per component
// and column, in chunk order.  A kernel of its own: a bin's interpolation reaches ~100 columns, so
// summing them where they are used read every partial 4 times over and left calls of few templates
// on a few workgroups.
__global__ void __launch_bounds__(kLagFinThreads)
k_lag_reduce(const BandDev *__restrict__ bands, const WorkItem *__restrict__ items, int n_items,
             double *__restrict__ part_) {
    const WorkItem &it = items[find_item(items, n_items, kStPairs, blockIdx.x)];
    const LagDev &G = bands[it.band].lag;
    const int l = blockIdx.x - it.first[kStPairs], gx = it.gx[kStPairs];
    const int n = (2 * bands[it.band].R + 1) * G.P * G.span, np = it.n_chunks * G.n_sub;
    const int x = (l % gx) * kLagFinThreads + threadIdx.x;
    if (x >= n) return;
    double *o = part_ + it.part_off + (size_t)(l / gx) * np * n + x;
    double v = 0.0;
#pragma unroll 8
    for (int k = 0; k < np; ++k) v += o[(size_t)k * n];
    o[0] = v;
}

// rho of kLagFinThreads consecutive bins of one template: per lag, the grid columns the block's
// bins reach go to LDS, then each bin takes its `taps`-point interpolation (weights by the bin's
// fraction of a grid step) and adds Re (Gamma^circ: Im) of e^{2 pi i kbar d N_K / N_FFT} S_d.
__global__ void __launch_bounds__(kLagFinThreads)
k_lag_finish(const BandDev *__restrict__ bands, const WorkItem *__restrict__ items, int n_items,
             const double *__restrict__ part_) {
    extern __shared__ __align__(16) char smem[];
    const WorkItem &it = items[find_item(items, n_items, kStFinish, blockIdx.x)];
    const BandDev B = global_view(bands[it.band], bands);
    const LagDev &G = B.lag;
    const int l = blockIdx.x - it.first[kStFinish], gx = it.gx[kStFinish];
    const int t = l / gx, b0 = (l % gx) * kLagFinThreads, b1 = min(B.n_f, b0 + kLagFinThreads);
    const int r0 = G.g0[b0], ncol = G.g0[b1 - 1] + G.taps - r0;
    const int R = B.R, P = G.P, span = G.span;
    const size_t plane = (size_t)P * span;
    const double *part = part_ + it.part_off + (size_t)t * it.n_chunks * G.n_sub * (2 * R + 1) * plane;
    double2 *S = reinterpret_cast<double2 *>(smem);
    const int i = min(b0 + (int)threadIdx.x, b1 - 1);
    const double *w = G.wt + (size_t)G.frac[i] * G.taps;
    const double2 *s = S + (G.g0[i] - r0);
    double rho = 0.0;
    for (int d = 0; d <= R; ++d) {
        for (int x = threadIdx.x; x < ncol; x += kLagFinThreads) {
            int rel = r0 + x;
            if (G.wrap) rel %= G.ng;
            const double *src = part + (size_t)(d == 0 ? 0 : 2 * d - 1) * plane + (size_t)(rel % P) * span + rel / P;
            S[x] = make_double2(src[0], d > 0 ? src[plane] : 0.0);
        }
        __syncthreads();
        double re = 0.0, im = 0.0;
#pragma unroll 4
        for (int j = 0; j < G.taps; ++j) {
            re = fma(w[j], s[j].x, re);
            im = fma(w[j], s[j].y, im);
        }
        if (d == 0) {
            rho = re;
        } else {
            const int e = (int)(((int64_t)B.bin_kb[i] * (((int64_t)d * B.n_k) % B.n_fft)) % B.n_fft);
            const double2 ph = B.tw64[e];  // exp(-2 pi i e / N_FFT)
            rho += B.weight != 0 ? im * ph.x - re * ph.y : re * ph.x + im * ph.y;
        }
        __syncthreads();
    }
    if (b0 + (int)threadIdx.x >= b1) return;
    void *out = as_global(it.out, (const gchar *)part_);
    const double v = rho * it.factor;
    if (it.out_fp64) static_cast<double *>(out)[(size_t)t * B.n_f + i] = v;
    else static_cast<float *>(out)[(size_t)t * B.n_f + i] = (float)v;
}

}  // namespace

// ------------------------------------------------------------------ launchers

template <typename T, int NS>
static void launch_lag_t(const LagKey &k, const BandDev *bands, const WorkItem *items, int n_items, int blocks,
                         size_t lds, const void *y, double *part, hipStream_t stream) {
#define CCR_LAG(RM_, CR_, PS_, CM_)                                                                              \
    hipLaunchKernelGGL((k_lag<T, NS, RM_, CR_, PS_, CM_>), dim3(blocks), dim3(64 * k.waves), lds, stream, bands, \
                       items, n_items, (const c2<T> *)y, part)
    // CM: weight Gamma^ave (0) or Gamma^circ (1), or read at run time (2); 4: Gamma^ave with the weights'
    // FP32 rests.  The weight is compiled in for pairs of both kinds with per-segment weights; the other forms
    // run transforms of up to 512 points (the planner's choice)
    if (k.cross || k.ps) {
        if constexpr (NS <= 512) {
            if (k.cross && k.ps) CCR_LAG(4, true, true, 2);
            else if (k.cross && k.rest) {
                if constexpr (sizeof(T) == 4) CCR_LAG(4, true, false, 4);
            } else if (k.cross) CCR_LAG(4, true, false, 2);
            else if (k.rm == 0) CCR_LAG(0, false, true, 2);
            else CCR_LAG(4, false, true, 2);
        }
    } else if (k.circ) {
        if (k.rm == 0) CCR_LAG(0, false, false, 1);
        else if (k.rm == 1) CCR_LAG(1, false, false, 1);
        else CCR_LAG(4, false, false, 1);
    } else if (NS <= 512 && sizeof(T) == 4 && k.rest) {
        if constexpr (NS <= 512 && sizeof(T) == 4) {
            if (k.rm == 1) CCR_LAG(1, false, false, 4);
            else if (k.rm == 2) CCR_LAG(2, false, false, 4);
            else CCR_LAG(4, false, false, 4);
        }
    } else {
        if (k.rm == 0) CCR_LAG(0, false, false, 0);
        else if (k.rm == 1) CCR_LAG(1, false, false, 0);
        else if (k.rm == 2) CCR_LAG(2, false, false, 0);
        else CCR_LAG(4, false, false, 0);
    }
#undef CCR_LAG
}

hipError_t launch_lag_m(const LagKey &k, const BandDev *bands, const WorkItem *items, int n_items, int blocks,
                        bool fp64, size_t lds, const void *y, double *part, hipStream_t stream) {
    if (blocks == 0) return hipSuccess;
    if (k.same > 0) {
#define CCR_SAME(NO_, NR_, QK_)                                                                            \
    hipLaunchKernelGGL((k_lag_same<NO_, NR_, QK_>), dim3(blocks), dim3(256), lds, stream, bands, items, n_items, \
                       (const float2 *)y, part)
#define CCR_SAME_Q(NO_, NR_)                   \
    if (k.dets == 2) CCR_SAME(NO_, NR_, 2);    \
    else if (k.dets == 3) CCR_SAME(NO_, NR_, 3); \
    else if (k.dets == 4) CCR_SAME(NO_, NR_, 4); \
    else CCR_SAME(NO_, NR_, 0)
        switch (k.same + k.rows) {
            case 6 + 8: CCR_SAME_Q(6, 8); break;
            case 6 + 12: CCR_SAME_Q(6, 12); break;
            case 6 + 16: CCR_SAME_Q(6, 16); break;
            case 16 + 8: CCR_SAME_Q(16, 8); break;
            case 16 + 12: CCR_SAME_Q(16, 12); break;
            case 16 + 16: CCR_SAME_Q(16, 16); break;
            default: return hipErrorInvalidValue;
        }
#undef CCR_SAME_Q
#undef CCR_SAME
        return hipGetLastError();
    }
    if (fp64) {
        if (k.ns == 512) launch_lag_t<double, 512>(k, bands, items, n_items, blocks, lds, y, part, stream);
        else if (k.ns == 256) launch_lag_t<double, 256>(k, bands, items, n_items, blocks, lds, y, part, stream);
        else return hipErrorInvalidValue;
    } else {
        if (k.ns == 1024) launch_lag_t<float, 1024>(k, bands, items, n_items, blocks, lds, y, part, stream);
        else if (k.ns == 512) launch_lag_t<float, 512>(k, bands, items, n_items, blocks, lds, y, part, stream);
        else if (k.ns == 256) launch_lag_t<float, 256>(k, bands, items, n_items, blocks, lds, y, part, stream);
        else return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_lag_finish_m(const BandDev *bands, const WorkItem *items, int n_items, int reduce_blocks,
                               int blocks, size_t lds, double *part, hipStream_t stream) {
    if (blocks == 0) return hipSuccess;
    if (reduce_blocks > 0)
        hipLaunchKernelGGL(k_lag_reduce, dim3(reduce_blocks), dim3(kLagFinThreads), 0, stream, bands, items, n_items, part);
    hipLaunchKernelGGL(k_lag_finish, dim3(blocks), dim3(kLagFinThreads), lds, stream, bands, items, n_items, part);
    return hipGetLastError();
}

}  // namespace ccr
