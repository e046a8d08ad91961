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
//   k_lag_finish  chunk sums, interpolation to the output bins, lag phases, sqrt(2) / N
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
template <typename T, int NS> struct LagTw;
template <typename T> struct LagTw<T, 1024> {
    c2<T> a[16], b[4][3];
    __device__ __forceinline__ void load(const c2<T> *tw, int P, int q, int lane) {
        const unsigned N = (unsigned)P * 1024;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            a[r] = tw[((unsigned)(r * (lane & 15) * 4 * P) + (unsigned)q * (unsigned)((lane >> 4) + 4 * r)) % N];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 1; r < 4; ++r) b[j][r - 1] = tw[(unsigned)(r * (lane + 64 * j) * P) % N];
    }
};
template <typename T> struct LagTw<T, 512> {
    c2<T> a[8], b[7];
    __device__ __forceinline__ void load(const c2<T> *tw, int P, int q, int lane) {
        const unsigned N = (unsigned)P * 512;
#pragma unroll
        for (int r = 0; r < 8; ++r)
            a[r] = tw[((unsigned)(r * (lane & 7) * 8 * P) + (unsigned)q * (unsigned)((lane >> 3) + 8 * r)) % N];
#pragma unroll
        for (int r = 1; r < 8; ++r) b[r - 1] = tw[(unsigned)(r * lane * P) % N];
    }
};
template <typename T> struct LagTw<T, 256> {
    c2<T> a[4], b[3], c[3];
    __device__ __forceinline__ void load(const c2<T> *tw, int P, int q, int lane) {
        const unsigned N = (unsigned)P * 256;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            a[r] = tw[((unsigned)(r * (lane & 3) * 16 * P) + (unsigned)q * (unsigned)((lane >> 2) + 16 * r)) % N];
#pragma unroll
        for (int r = 1; r < 4; ++r) {
            b[r - 1] = tw[(unsigned)(r * (lane & 15) * 4 * P) % N];
            c[r - 1] = tw[(unsigned)(r * lane * P) % N];
        }
    }
};

// NS-point forward FFT of one wavefront (V = NS / 64 values a lane, x[l + 64 r] in v[r] on
// entry, X[l + 64 J] in v[J] on return), self-sorting passes of radix 16, 16, 4 (1024), 8, 8, 8
// (512) or 4, 4, 4, 4 (256): a pass of radix V with stride Ns has butterfly l read a[l + 64 r],
// twiddle input r and write output r to (l / Ns) V Ns + l % Ns + r Ns.  Between passes the values
// go through `ex` (NS + NS / V entries), index i at i + i / V.
template <typename T>
__device__ __forceinline__ void lag_fft(c2<T> *v, T *ex, const LagTw<T, 1024> &t, int lane) {
    const int g = lane >> 4, k = lane & 15;
    auto perm = [](int i) { return 4 * (i & 3) + (i >> 2); };
    dft16<T>(v);
    exchange<T, 16>(v, ex, perm, [&](int i) { return 17 * lane + i; }, [&](int r) { return lane + g + 68 * r; });
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = cmul<T>(v[r], t.a[r]);
    dft16<T>(v);
    exchange<T, 16>(v, ex, perm, [&](int i) { return 272 * g + k + 17 * i; },
                    [&](int r) { return lane + g + 68 * (r & 3) + 272 * (r >> 2); });
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // v[j + 4 r] = a[l + 64 j + 256 r]
#pragma unroll
        for (int r = 1; r < 4; ++r) v[j + 4 * r] = cmul<T>(v[j + 4 * r], t.b[j][r - 1]);
        dft4<T>(v[j], v[j + 4], v[j + 8], v[j + 12]);
    }
}

template <typename T>
__device__ __forceinline__ void lag_fft(c2<T> *v, T *ex, const LagTw<T, 512> &t, int lane) {
    const int g = lane >> 3, k = lane & 7;
    auto id = [](int i) { return i; };
    auto rd = [&](int r) { return lane + g + 72 * r; };
    dft8<T>(v);
    exchange<T, 8>(v, ex, id, [&](int i) { return 9 * lane + i; }, rd);
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = cmul<T>(v[r], t.a[r]);
    dft8<T>(v);
    exchange<T, 8>(v, ex, id, [&](int i) { return 72 * g + k + 9 * i; }, rd);
#pragma unroll
    for (int r = 1; r < 8; ++r) v[r] = cmul<T>(v[r], t.b[r - 1]);
    dft8<T>(v);
}

template <typename T>
__device__ __forceinline__ void lag_fft(c2<T> *v, T *ex, const LagTw<T, 256> &t, int lane) {
    const int g4 = lane >> 2, k4 = lane & 3, g16 = lane >> 4, k16 = lane & 15;
    auto id = [](int i) { return i; };
    auto rd = [&](int r) { return lane + g4 + 80 * r; };
    dft4<T>(v[0], v[1], v[2], v[3]);
    exchange<T, 4>(v, ex, id, [&](int i) { return 5 * lane + i; }, rd);
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = cmul<T>(v[r], t.a[r]);
    dft4<T>(v[0], v[1], v[2], v[3]);
    exchange<T, 4>(v, ex, id, [&](int i) { return 20 * g4 + k4 + 5 * i; }, rd);
#pragma unroll
    for (int r = 1; r < 4; ++r) v[r] = cmul<T>(v[r], t.b[r - 1]);
    dft4<T>(v[0], v[1], v[2], v[3]);
    exchange<T, 4>(v, ex, id, [&](int i) { return 80 * g16 + k16 + (k16 >> 2) + 20 * i; }, rd);
#pragma unroll
    for (int r = 1; r < 4; ++r) v[r] = cmul<T>(v[r], t.c[r - 1]);
    dft4<T>(v[0], v[1], v[2], v[3]);
}

// ------------------------------------------------------------------ uniform reads and buffer loads

template <typename T> __device__ __forceinline__ c2<T> ld_uniform_c2(const c2<T> *p, int i);
template <> __device__ __forceinline__ float2 ld_uniform_c2<float>(const float2 *p, int i) { return ld_uniform_f2(p, i); }
template <> __device__ __forceinline__ double2 ld_uniform_c2<double>(const double2 *p, int i) {
    const double *d = reinterpret_cast<const double *>(p);
    return make_double2(ld_uniform(d, 2 * i), ld_uniform(d, 2 * i + 1));
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <typename T> __device__ __forceinline__ c2<T> ld_buf(__amdgpu_buffer_rsrc_t rs, int i);
template <> __device__ __forceinline__ float2 ld_buf<float>(__amdgpu_buffer_rsrc_t rs, int i) {
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, i * 8, 0, 0));
}
template <> __device__ __forceinline__ double2 ld_buf<double>(__amdgpu_buffer_rsrc_t rs, int i) {
    return __builtin_bit_cast(double2, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(rs, i * 16, 0, 0));
}

template <typename T> struct LagTab;
template <> struct LagTab<float> {
    static __device__ __forceinline__ const float2 *tw(const LagDev &G) { return G.tw32; }
    static __device__ __forceinline__ const float2 *step(const LagDev &G) { return G.step32; }
    static __device__ __forceinline__ const float2 *segw(const BandDev &B) { return B.segwf; }
    static __device__ __forceinline__ const float2 *pw(const BandDev &B) { return B.pwf; }
};
template <> struct LagTab<double> {
    static __device__ __forceinline__ const double2 *tw(const LagDev &G) { return G.tw64; }
    static __device__ __forceinline__ const double2 *step(const LagDev &G) { return G.step64; }
    static __device__ __forceinline__ const double2 *segw(const BandDev &B) { return B.segwd; }
    static __device__ __forceinline__ const double2 *pw(const BandDev &B) { return B.pw; }
};

// ------------------------------------------------------------------ spectra and pair sums

// The detectors a workgroup sums over: all of them (both pair kinds, or lag 0), one (pairs
// within a detector: one problem a detector) or two (pairs across detectors with lags: one
// problem a pair of detectors).
struct LagDets {
    int n, d0, d1;
    __device__ __forceinline__ int at(int i) const { return i == 0 ? d0 : (i == 1 ? d1 : i); }
    // activity of segment K's spectra, bit i for detector at(i)
    __device__ __forceinline__ unsigned bits(unsigned b) const {
        if (n == 1) return (b >> d0) & 1u;
        if (n == 2) return ((b >> d0) & 1u) | (((b >> d1) & 1u) << 1);
        return b;
    }
};

// Streams of one grid column at the step's kLagSegs segments from the spectra in LDS: NST = 2:
// the sums over the detectors of hat a_X F_X and hat b_X F_X (n[t] = {A, B}); NST = 4 (two
// detectors, pairs across them only): {a_0, a_1, b_0, b_1}.  s0: the same-time products of the
// pairs X < Y, Re[conj(a_X) a_Y + conj(b_X) b_Y], or for Gamma^circ Im[conj(b_X) a_Y - conj(a_X) b_Y],
// of the segments from t0 on (the ones before them are halo); null with no pairs across detectors.
// PS (per-sample antenna functions): the two streams are transforms of their own.
template <typename T, int ND, int NST, bool PS>
__device__ __forceinline__ void lag_gather(const BandDev &B, const LagDets &D, const char *slots, int slot_bytes,
                                           int col, int Kb, int nd, bool circ, bool cross, int t0, T &s0,
                                           c2<T> (&n)[kLagSegs][NST]) {
    const int NDr = ND > 0 ? ND : nd;
    constexpr int NM = ND > 0 ? ND : CCR_MAX_DET_K;
#pragma unroll
    for (int t = 0; t < kLagSegs; ++t) {
        c2<T> A = mk<T>((T)0, (T)0), Bs = A;
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
                const c2<T> w = ld_uniform_c2<T>(LagTab<T>::segw(B), D.at(i) * B.n_seg + min(Kb + t, B.n_seg - 1));
                a = cscale<T>(f, w.x);
                b = cscale<T>(f, w.y);
            }
            if (i > 0 && cross && t >= t0) {
                if (circ) s0 += (Bs.x * a.y - Bs.y * a.x) - (A.x * b.y - A.y * b.x);
                else s0 += (A.x * a.x + A.y * a.y) + (Bs.x * b.x + Bs.y * b.y);
            }
            if constexpr (NST == 4) {
                n[t][i & 1] = a;
                n[t][2 + (i & 1)] = b;
            }
            A = cadd<T>(A, a);
            Bs = cadd<T>(Bs, b);
        }
        if constexpr (NST == 2) {
            n[t][0] = A;
            n[t][1] = Bs;
        }
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
//   Pair sums.  Lane j of the workgroup owns columns j + 64 W u (u < U): it forms the step's
//   streams, multiplies each segment's with those of the RM segments before it -- the step's own
//   or the last step's, kept in registers -- and adds them to S_1 .. S_RM (lags above R are
//   computed and dropped).  FP32 products of a step are summed in FP32, steps in FP64.
// Two barriers a step.  Partials: [comp][P][span], comp 0: S_0 (same-time pairs across
// detectors), 2 d - 1 and 2 d: Re and Im of S_d.
//
// Bound: VALU issue (transforms ~3/4 of the instructions, pair sums ~1/4 at lag 4).  Against the
// transform at every output bin with window sums over an LDS ring of spectra: 1300 -> 175 ms for
// 1002 templates of the 240-day, lag-4 band; in FP64 (spectra through memory, then pair sums)
// 23.4 -> 1.7 ms for 5 templates of 120 days of it.
template <typename T, int NS, int U, int RM, bool CR, bool PS>
__device__ __forceinline__ void lag_body(const BandDev &B, const c2<T> *__restrict__ y, double *__restrict__ part,
                                         int k_chunk, int n_chunks, int c, int sub, int p, int tb) {
    extern __shared__ __align__(16) char smem[];
    constexpr int V = NS / 64;
    constexpr int S = PS ? 2 : 1;
    constexpr int NST = CR ? 4 : 2;
    const LagDev &G = B.lag;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int W = blockDim.x >> 6;
    const int n_k = B.n_k, R = B.R, P = G.P, span = G.span, nf = G.nfold;
    const bool circ = B.weight != 0, cross = (B.pairs & 1) != 0;
    // the workgroup's detectors
    LagDets D{B.Q, 0, 1};
    if (G.n_sub > 1 || CR) {
        if (!cross) {
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

    const int q = (p + P * G.m0) % G.ng;
    LagTw<T, NS> tw;
    tw.load(LagTab<T>::tw(G), P, q, lane);
    const c2<T> *step = LagTab<T>::step(G) + (size_t)p * V * nf;

    const int K0 = c * k_chunk, K1 = min(B.n_seg, K0 + k_chunk);
    const int Kh = max(0, K0 - R);
    const int64_t nr = (int64_t)B.n_seg * n_k;
    const c2<T> *yb = y + (size_t)tb * B.Q * nr;

    // active units of the step at Kb: bit t nd + i
    auto step_mask = [&](int Kb) -> unsigned {
        unsigned m = 0;
#pragma unroll
        for (int t = 0; t < kLagSegs; ++t)
            if (Kb + t < K1) m |= D.bits(ld_uniform(B.seg_bits, Kb + t)) << (t * nd);
        return m;
    };
    // n-th set bit of m (from 0), -1 if there is none
    auto nth = [](unsigned m, int n) -> int {
        for (int k = 0; k < n && m; ++k) m &= m - 1;
        return m ? __builtin_ctz(m) : -1;
    };
    auto src = [&](const c2<T> *base, int det, int K) {
        return __builtin_amdgcn_make_buffer_rsrc((void *)(base + (size_t)det * nr + (size_t)K * n_k), (short)0,
                                                 n_k * (int)sizeof(c2<T>), 0x00020000);
    };
    c2<T> nxt[V];
    auto load = [&](int Kb, int unit) {
        const int t = unit / nd, i = unit - t * nd;
        const __amdgpu_buffer_rsrc_t rs = src(yb, D.at(i), Kb + t);
#pragma unroll
        for (int r = 0; r < V; ++r) nxt[r] = ld_buf<T>(rs, lane + 64 * r);
    };

    c2<T> hist[U][RM > 0 ? RM : 1][NST];
    double acc0[U], acc[U][RM > 0 ? 2 * RM : 1];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        acc0[u] = 0.0;
#pragma unroll
        for (int k = 0; k < (RM > 0 ? 2 * RM : 1); ++k) acc[u][k] = 0.0;
#pragma unroll
        for (int d = 0; d < (RM > 0 ? RM : 1); ++d)
#pragma unroll
            for (int j = 0; j < NST; ++j) hist[u][d][j] = mk<T>((T)0, (T)0);
    }

    unsigned mask = step_mask(Kh);
    {
        const int u0 = nth(mask, wv / S);
        if (u0 >= 0) load(Kh, u0);
    }
    for (int Kb = Kh; Kb < K1; Kb += kLagSegs) {
        const unsigned nmask = Kb + kLagSegs < K1 ? step_mask(Kb + kLagSegs) : 0u;
        const int nu0 = nth(nmask, wv / S);
        if (mask == 0) {  // no spectra in the step (uniform over the workgroup)
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int d = 0; d < (RM > 0 ? RM : 1); ++d)
#pragma unroll
                    for (int j = 0; j < NST; ++j) hist[u][d][j] = mk<T>((T)0, (T)0);
            if (nu0 >= 0) load(Kb + kLagSegs, nu0);
            mask = nmask;
            continue;
        }
        // transforms: this wavefront takes active (unit, stream) numbers wv, wv + W, ...
        int nn = wv;
        int unit = nth(mask, nn / S);
        if (unit < 0 && nu0 >= 0) load(Kb + kLagSegs, nu0);
#pragma unroll 1
        while (unit >= 0) {
            const int s = PS ? nn % S : 0;
            const int t = unit / nd, i = unit - t * nd;
            char *slot = smem + (size_t)(unit * S + s) * slot_bytes;
            c2<T> v[V];
#pragma unroll
            for (int r = 0; r < V; ++r) v[r] = nxt[r];
            // the next input: this wavefront's next unit of the step, or its first of the next step
            nn += W;
            const int un = nth(mask, nn / S);
            if (un >= 0) load(Kb, un);
            else if (nu0 >= 0) load(Kb + kLagSegs, nu0);
            if constexpr (PS) {
                const __amdgpu_buffer_rsrc_t rw = src(LagTab<T>::pw(B), D.at(i), Kb + t);
#pragma unroll
                for (int r = 0; r < V; ++r) {
                    const c2<T> w = ld_buf<T>(rw, lane + 64 * r);
                    v[r] = cscale<T>(v[r], s ? w.y : w.x);
                }
            }
            if (p > 0) {
#pragma unroll
                for (int r = 0; r < V; ++r) v[r] = cmul<T>(v[r], ld_uniform_c2<T>(step, r));
            }
            for (int j = 1; j < nf; ++j) {
                const __amdgpu_buffer_rsrc_t rs = src(yb, D.at(i), Kb + t);
                const __amdgpu_buffer_rsrc_t rw = src(PS ? LagTab<T>::pw(B) : yb, D.at(i), Kb + t);
#pragma unroll
                for (int r = 0; r < V; ++r) {
                    if (64 * r + NS * j >= n_k) continue;  // uniform
                    c2<T> z = ld_buf<T>(rs, lane + 64 * r + NS * j);
                    if constexpr (PS) {
                        const c2<T> w = ld_buf<T>(rw, lane + 64 * r + NS * j);
                        z = cscale<T>(z, s ? w.y : w.x);
                    }
                    v[r] = cadd<T>(v[r], cmul<T>(z, ld_uniform_c2<T>(step, r + V * j)));
                }
            }
            lag_fft<T>(v, reinterpret_cast<T *>(slot), tw, lane);
            wave_sync();
#pragma unroll
            for (int J = 0; J < V; ++J)
                if (64 * J < span) reinterpret_cast<c2<T> *>(slot)[lane + 64 * J] = v[J];
            unit = un;
        }
        // zeros for the units without a spectrum
        {
            unsigned off = ~mask & (nunit >= 32 ? ~0u : (1u << nunit) - 1u);
            for (int k = 0; off; off &= off - 1, ++k) {
                if (k % W != wv) continue;
                c2<T> *slot = reinterpret_cast<c2<T> *>(smem + (size_t)(__builtin_ctz(off) * S) * slot_bytes);
                for (int e = lane; e < S * slot_bytes / (int)sizeof(c2<T>); e += 64) slot[e] = mk<T>((T)0, (T)0);
            }
        }
        __syncthreads();
        const int t0 = max(0, K0 - Kb);  // halo segments before t0 only enter the history
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (wv * 64 + 64 * W * u >= span) continue;  // uniform: no lane of this wavefront has a column
            const int col = min((int)threadIdx.x + 64 * W * u, span - 1);
            c2<T> n[kLagSegs][NST];
            T s0 = (T)0;
            if constexpr (CR) {
                lag_gather<T, 2, NST, PS>(B, D, smem, slot_bytes, col, Kb, nd, circ, cross, t0, s0, n);
            } else {
                switch (nd) {
                    case 1: lag_gather<T, 1, NST, PS>(B, D, smem, slot_bytes, col, Kb, nd, circ, cross, t0, s0, n); break;
                    case 2: lag_gather<T, 2, NST, PS>(B, D, smem, slot_bytes, col, Kb, nd, circ, cross, t0, s0, n); break;
                    case 3: lag_gather<T, 3, NST, PS>(B, D, smem, slot_bytes, col, Kb, nd, circ, cross, t0, s0, n); break;
                    default: lag_gather<T, 0, NST, PS>(B, D, smem, slot_bytes, col, Kb, nd, circ, cross, t0, s0, n); break;
                }
            }
            acc0[u] += (double)s0;
            if constexpr (RM > 0) {
                T st[2 * RM];
#pragma unroll
                for (int k = 0; k < 2 * RM; ++k) st[k] = (T)0;
#pragma unroll
                for (int t = 0; t < kLagSegs; ++t) {
                    if (t < t0) continue;  // uniform
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
#pragma unroll
                        for (int j = 0; j < NST; ++j) {
                            const c2<T> h = t - d >= 0 ? n[t - d >= 0 ? t - d : 0][j] : hist[u][d - t - 1 >= 0 ? d - t - 1 : 0][j];
                            st[2 * d - 2] += x[j].x * h.x + x[j].y * h.y;
                            st[2 * d - 1] += x[j].x * h.y - x[j].y * h.x;
                        }
                    }
                }
#pragma unroll
                for (int k = 0; k < 2 * RM; ++k) acc[u][k] += (double)st[k];
                // the step's last RM segments become the history (kLagSegs >= RM)
#pragma unroll
                for (int d = 0; d < RM; ++d)
#pragma unroll
                    for (int j = 0; j < NST; ++j) hist[u][d][j] = n[kLagSegs - 1 - d][j];
            }
        }
        __syncthreads();
        mask = nmask;
    }
    const int nc = 2 * R + 1;
    double *o = part + (((size_t)tb * n_chunks + c) * G.n_sub + sub) * nc * P * span + (size_t)p * span;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int col = threadIdx.x + 64 * W * u;
        if (col >= span) continue;
        o[col] = acc0[u];
        if constexpr (RM > 0) {
#pragma unroll
            for (int k = 0; k < 2 * RM; ++k)
                if (k + 1 < nc) o[(size_t)(k + 1) * P * span + col] = acc[u][k];
        }
    }
}

// Blocks of an item: G = n_tmpl n_chunks n_sub groups of P class workgroups; the dispatcher
// hands workgroups to the 8 XCDs in turn, so a group's classes get indices with equal value mod
// 8 and read the group's resampled series through one XCD's L2.
template <typename T, int NS, int U, int RM, bool CR, bool PS>
__global__ void __launch_bounds__(512)
k_lag(const BandDev *__restrict__ bands, const WorkItem *__restrict__ items, int n_items,
      const c2<T> *__restrict__ y, double *__restrict__ part) {
    const WorkItem &it = items[find_item(items, n_items, kStSpectra, blockIdx.x)];
    const BandDev B = global_view(bands[it.band], bands);
    const int l = blockIdx.x - it.first[kStSpectra];
    const int P = B.lag.P, G = it.n_tmpl * it.n_chunks * B.lag.n_sub;
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
    const int per = it.n_chunks * B.lag.n_sub;
    lag_body<T, NS, U, RM, CR, PS>(B, y + it.y_off, part + it.part_off, it.k_chunk, it.n_chunks,
                                   (g % per) / B.lag.n_sub, g % B.lag.n_sub, p, g / per);
}

// ------------------------------------------------------------------ interpolation to the output bins

// rho of kLagFinThreads * bpt consecutive bins of one template: per lag, the chunk (and
// detector) partials of the grid columns the block's bins reach are summed into LDS, then each
// bin takes its `taps`-point interpolation (weights by the bin's fraction of a grid step, exact
// to LagDev's design error) and adds Re (Gamma^circ: Im) of e^{2 pi i kbar d N_K / N_FFT} S_d.
// Sums in FP64, in chunk order.
__global__ void __launch_bounds__(kLagFinThreads)
k_lag_finish(const BandDev *__restrict__ bands, const WorkItem *__restrict__ items, int n_items,
             const double *__restrict__ part_) {
    extern __shared__ __align__(16) char smem[];
    const WorkItem &it = items[find_item(items, n_items, kStFinish, blockIdx.x)];
    const BandDev B = global_view(bands[it.band], bands);
    const LagDev &G = B.lag;
    const int l = blockIdx.x - it.first[kStFinish], gx = it.gx[kStFinish];
    const int t = l / gx, bpt = G.fin_bpt;
    const int b0 = (l % gx) * kLagFinThreads * bpt, b1 = min(B.n_f, b0 + kLagFinThreads * bpt);
    const int r0 = G.g0[b0], ncol = G.g0[b1 - 1] + G.taps - r0;
    const int R = B.R, P = G.P, span = G.span, nc = 2 * R + 1, np = it.n_chunks * G.n_sub;
    const size_t plane = (size_t)P * span;
    const double *part = part_ + it.part_off + (size_t)t * np * nc * plane;
    double2 *S = reinterpret_cast<double2 *>(smem);
    double rho[kLagFinBins];
#pragma unroll
    for (int k = 0; k < kLagFinBins; ++k) rho[k] = 0.0;
    for (int d = 0; d <= R; ++d) {
        for (int x = threadIdx.x; x < ncol; x += kLagFinThreads) {
            int rel = r0 + x;
            if (G.wrap) rel %= G.ng;
            const double *src = part + (size_t)(d == 0 ? 0 : 2 * d - 1) * plane + (size_t)(rel % P) * span + rel / P;
            double re = 0.0, im = 0.0;
            for (int k = 0; k < np; ++k) {
                re += src[(size_t)k * nc * plane];
                if (d > 0) im += src[(size_t)k * nc * plane + plane];
            }
            S[x] = make_double2(re, im);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kLagFinBins; ++k) {
            const int i = b0 + threadIdx.x + kLagFinThreads * k;
            if (k >= bpt || i >= b1) continue;
            const double *w = G.wt + (size_t)G.frac[i] * G.taps;
            const double2 *s = S + (G.g0[i] - r0);
            double re = 0.0, im = 0.0;
            for (int j = 0; j < G.taps; ++j) {
                re = fma(w[j], s[j].x, re);
                im = fma(w[j], s[j].y, im);
            }
            if (d == 0) {
                rho[k] = re;
            } else {
                const int e = (int)(((int64_t)B.bin_kb[i] * (((int64_t)d * B.n_k) % B.n_fft)) % B.n_fft);
                const double2 ph = B.tw64[e];  // exp(-2 pi i e / N_FFT)
                rho[k] += B.weight != 0 ? im * ph.x - re * ph.y : re * ph.x + im * ph.y;
            }
        }
        __syncthreads();
    }
    void *out = as_global(it.out, (const gchar *)part_);
#pragma unroll
    for (int k = 0; k < kLagFinBins; ++k) {
        const int i = b0 + threadIdx.x + kLagFinThreads * k;
        if (k >= bpt || i >= b1) continue;
        const double v = rho[k] * it.factor;
        if (it.out_fp64) static_cast<double *>(out)[(size_t)t * B.n_f + i] = v;
        else static_cast<float *>(out)[(size_t)t * B.n_f + i] = (float)v;
    }
}

}  // namespace

// ------------------------------------------------------------------ launchers

template <typename T, int NS, int U>
static void launch_lag_t(const LagKey &k, const BandDev *bands, const WorkItem *items, int n_items, int blocks,
                         size_t lds, const void *y, double *part, hipStream_t stream) {
#define CCR_LAG(RM_, CR_, PS_)                                                                                        \
    hipLaunchKernelGGL((k_lag<T, NS, U, RM_, CR_, PS_>), dim3(blocks), dim3(64 * k.waves), lds, stream, bands, items, \
                       n_items, (const c2<T> *)y, part)
    if (k.cross) {
        if (k.ps) CCR_LAG(4, true, true);
        else CCR_LAG(4, true, false);
    } else if (k.ps) {
        if (k.rm == 0) CCR_LAG(0, false, true);
        else CCR_LAG(4, false, true);
    } else {
        if (k.rm == 0) CCR_LAG(0, false, false);
        else if (k.rm == 1) CCR_LAG(1, false, false);
        else if (k.rm == 2) CCR_LAG(2, false, false);
        else CCR_LAG(4, false, false);
    }
#undef CCR_LAG
}

hipError_t launch_lag_m(const LagKey &k, const BandDev *bands, const WorkItem *items, int n_items, int blocks,
                        bool fp64, size_t lds, const void *y, double *part, hipStream_t stream) {
    if (blocks == 0) return hipSuccess;
    if (fp64) {
        if (k.ns == 512) launch_lag_t<double, 512, 1>(k, bands, items, n_items, blocks, lds, y, part, stream);
        else if (k.ns == 256) launch_lag_t<double, 256, 1>(k, bands, items, n_items, blocks, lds, y, part, stream);
        else return hipErrorInvalidValue;
    } else {
        if (k.ns == 1024) launch_lag_t<float, 1024, 2>(k, bands, items, n_items, blocks, lds, y, part, stream);
        else if (k.ns == 512) launch_lag_t<float, 512, 1>(k, bands, items, n_items, blocks, lds, y, part, stream);
        else if (k.ns == 256) launch_lag_t<float, 256, 1>(k, bands, items, n_items, blocks, lds, y, part, stream);
        else return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_lag_finish_m(const BandDev *bands, const WorkItem *items, int n_items, int blocks, size_t lds,
                               const double *part, hipStream_t stream) {
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_lag_finish, dim3(blocks), dim3(kLagFinThreads), lds, stream, bands, items, n_items, part);
    return hipGetLastError();
}

}  // namespace ccr
