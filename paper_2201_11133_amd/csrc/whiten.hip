// Whitening front end ("Data preparation"): the Welch PSD of each channel of a two-detector
// stream, whitening of the stream by that PSD as one transform over the whole stream, and scaling
// of each channel to unit standard deviation.
//
// Both channels travel in one complex sequence z[t] = x0[t] + i x1[t]; the spectra of the two real
// channels separate as X0[k] = (Z[k] + conj Z[N-k]) / 2 and X1[k] = (Z[k] - conj Z[N-k]) / 2i.
// Transforms are decimation-in-time (radix-2 stages taken three at a time), in registers with exchanges
// through LDS from 256 points on, in LDS below, up to 16384 points. A stream of L = N1 N2 samples takes the four-step route: N2 transforms of length N1 down
// the columns t = n1 N2 + n2, a twiddle e^(-2 pi i n2 k1 / L), N1 transforms of length N2 along
// the rows; the spectrum is kept transposed (bin k1 + N1 k2 at k1 N2 + k2), which is the order
// the inverse reads back.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "gwd_internal.h"

namespace gwd {

constexpr int WH_SMALL = 64;                  // threads of the transforms of up to 128 points
constexpr int WH_SMALLN = 128;
constexpr int WH_MAXLOG = 14;                 // largest transform in one workgroup: 16384 points
constexpr int WH_TW = 1 << (WH_MAXLOG - 1);   // twiddle table tw[t] = e^(-2 pi i t / 16384), t < 8192

// a b, the imaginary part with a.y b.x fused (ALT: with a.x b.y): the fused product is written out, so that
// every form of a transform rounds alike.
template <bool ALT = false>
__device__ inline float2 cmul(float2 a, float2 b) {
    return make_float2(fmaf(a.x, b.x, -(a.y * b.y)), ALT ? fmaf(a.x, b.y, a.y * b.x) : fmaf(a.y, b.x, a.x * b.y));
}

__device__ inline int bitrev(int j, int logn) { return (int)(__brev((unsigned)j) >> (32 - logn)); }

// Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous range of transforms so
// that the neighbouring columns that share cache lines in the strided passes meet in one L2.
__device__ inline int64_t xcd_block(int64_t nblk) {
    const int64_t b = blockIdx.x;
    return (nblk & 7) ? b : (b & 7) * (nblk >> 3) + (b >> 3);
}

// e^(sign 2 pi i e / L) for an exact integer e < L (L a power of two), in float64
__device__ inline double2 twiddle_l(int64_t e, int logl, bool inverse) {
    double s, c;
    sincospi((inverse ? 2.0 : -2.0) * ldexp((double)e, -logl), &s, &c);
    return make_double2(c, s);
}

// The twiddles e^(sign 2 pi i a k / L) of one row or column, k = k0 + stride i for i = 0, 1, ..:
// a float64 sincospi for the first and for the step, then float64 complex products, each rounded to
// float32 when used. After 31 products the float64 value is within about 1e-14, far below the rounding.
// (Forward column and inverse row passes over 2^24 samples, then with their transforms in LDS: 138 and 111 us
// with it, 150 and 118 us with a sincospi per element.)
struct TwiddleRun {
    double2 w, step;
    __device__ TwiddleRun(int64_t a, int k0, int stride, int logl, bool inverse) {
        const int64_t mask = (1ll << logl) - 1;
        w = twiddle_l((a * k0) & mask, logl, inverse);
        step = twiddle_l((a * stride) & mask, logl, inverse);
    }
    __device__ float2 next() {
        const float2 r = make_float2((float)w.x, (float)w.y);
        w = make_double2(w.x * step.x - w.y * step.y, w.x * step.y + w.y * step.x);
        return r;
    }
};

__global__ void wh_twiddle_kernel(float2* tw) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < WH_TW) {
        double s, c;
        sincospi(-2.0 * ldexp((double)t, -WH_MAXLOG), &s, &c);
        tw[t] = make_float2((float)c, (float)s);
    }
}

// In-place radix-2 DIT transform of s[0, 2^logn) (input already in bit-reversed order, output in
// natural order); the inverse uses the conjugate twiddles and does not scale. Stages go in threes
// (radix 2^3): a thread takes eight points base + j + m half (m = 0..7) through the three stages in
// registers, so LDS is read and written once per three stages; the last one or two run as a pair or
// alone.
__device__ inline float2 tw_at(const float2* __restrict__ tw, int i, bool inverse) {
    float2 w = tw[i];
    if (inverse) w.y = -w.y;
    return w;
}

template <bool ALT = false>
__device__ inline void bfly(float2& a, float2& b, float2 w) {
#pragma clang fp contract(off)   // (a windowed sample keeps its rounding)
    const float2 c = cmul<ALT>(b, w);
    b = make_float2(a.x - c.x, a.y - c.y);
    a = make_float2(a.x + c.x, a.y + c.y);
}

__device__ void lds_fft(float2* s, int logn, const float2* __restrict__ tw, bool inverse) {
    const int n = 1 << logn;
    int lh = 0;
    for (; lh + 2 < logn; lh += 3) {   // three stages per pass: eight points base + j + m half per thread
        const int half = 1 << lh;
        __syncthreads();
        for (int b = threadIdx.x; b < (n >> 3); b += blockDim.x) {
            const int j = b & (half - 1);
            const int base = ((b - j) << 3) + j;
            float2 a[8];
#pragma unroll
            for (int m = 0; m < 8; ++m) a[m] = s[base + m * half];
            const float2 w1 = tw_at(tw, j << (WH_MAXLOG - 1 - lh), inverse);           // W_(2 half)^j
#pragma unroll
            for (int m = 0; m < 8; m += 2) bfly(a[m], a[m + 1], w1);
            const float2 w2 = tw_at(tw, j << (WH_MAXLOG - 2 - lh), inverse);           // W_(4 half)^j
            const float2 w3 = tw_at(tw, (j + half) << (WH_MAXLOG - 2 - lh), inverse);  // W_(4 half)^(j + half)
#pragma unroll
            for (int g = 0; g < 8; g += 4) {
                bfly<true>(a[g], a[g + 2], w2);
                bfly(a[g + 1], a[g + 3], w3);
            }
            bfly<true>(a[0], a[4], tw_at(tw, j << (WH_MAXLOG - 3 - lh), inverse));       // W_(8 half)^(j + m half)
#pragma unroll
            for (int m = 1; m < 4; ++m) bfly(a[m], a[m + 4], tw_at(tw, (j + m * half) << (WH_MAXLOG - 3 - lh), inverse));
#pragma unroll
            for (int m = 0; m < 8; ++m) s[base + m * half] = a[m];
        }
    }
    if (lh + 1 < logn) {   // two stages left
        const int half = 1 << lh;
        __syncthreads();
        for (int b = threadIdx.x; b < (n >> 2); b += blockDim.x) {
            const int j = b & (half - 1);
            const int base = ((b - j) << 2) + j;
            float2 a0 = s[base], a1 = s[base + half], a2 = s[base + 2 * half], a3 = s[base + 3 * half];
            const float2 w1 = tw_at(tw, j << (WH_MAXLOG - 1 - lh), inverse);
            bfly(a0, a1, w1);
            bfly(a2, a3, w1);
            bfly<true>(a0, a2, tw_at(tw, j << (WH_MAXLOG - 2 - lh), inverse));
            bfly(a1, a3, tw_at(tw, (j + half) << (WH_MAXLOG - 2 - lh), inverse));
            s[base] = a0;
            s[base + half] = a1;
            s[base + 2 * half] = a2;
            s[base + 3 * half] = a3;
        }
    } else if (lh < logn) {   // one stage left
        const int half = 1 << lh;
        __syncthreads();
        for (int b = threadIdx.x; b < (n >> 1); b += blockDim.x) {
            const int j = b & (half - 1);
            const int i0 = ((b - j) << 1) + j;
            float2 a0 = s[i0], a1 = s[i0 + half];
            bfly(a0, a1, tw_at(tw, j << (WH_MAXLOG - 1 - lh), inverse));
            s[i0] = a0;
            s[i0 + half] = a1;
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------- transforms of 256 points and more
// The same radix-2 stages, three at a time, with the points in registers: a transform of N points runs on
// TC threads, thread t holds the points t + TC i. The first pass reads its points where the caller loaded
// them from memory and the last leaves them in natural order, so only the exchanges between passes go
// through LDS, in one padded buffer (8 points, then one unused: the writes of the first passes are strided
// by 8 points). Each pass merges sub-transforms l, l + N/8, .. of Ns points (in the stages' own order, the
// bits of the merge index reversed) and writes them in natural order, so nothing is ever bit-reversed in
// LDS: bit-reversed stores met in one bank, and they and the strided first pass bounded these kernels.
// The operations and their order are those of lds_fft. 2^24 samples, 4096-point columns and rows: forward
// columns 150 -> 124 us, forward rows 146 -> 102, spectrum division and inverse rows 194 -> 102, inverse
// columns 138 -> 91; Welch of 2,047 segments of 16384: 374 -> 188 us. Each pass moves 268 MB, 54 us at the
// rate of a large copy; the strided gathers of 16 bytes per row bound the column passes.
template <int LOGN, int MAXT>
struct RegFft {
    static constexpr int N = 1 << LOGN;
    static constexpr int TC = N / 8 < MAXT ? N / 8 : MAXT;   // threads per transform
    static constexpr int P = N / TC;                          // points per thread
    static constexpr int LDS = N + N / 8;                     // float2 per transform in flight
    static __device__ int pad(int a) { return a + (a >> 3); }

    // three stages (or R = 4, 2: the last two or one) at half = Ns on v[m], m in stage order
    template <int R>
    static __device__ void stages(float2 (&a)[R], int lh, int k, const float2* __restrict__ tw, bool inverse) {
        const int half = 1 << lh;
        const float2 w1 = tw_at(tw, k << (WH_MAXLOG - 1 - lh), inverse);
#pragma unroll
        for (int m = 0; m < R; m += 2) bfly(a[m], a[m + 1], w1);
        if constexpr (R >= 4) {
            const float2 w2 = tw_at(tw, k << (WH_MAXLOG - 2 - lh), inverse);
            const float2 w3 = tw_at(tw, (k + half) << (WH_MAXLOG - 2 - lh), inverse);
#pragma unroll
            for (int g = 0; g < R; g += 4) {
                bfly<true>(a[g], a[g + 2], w2);
                bfly(a[g + 1], a[g + 3], w3);
            }
        }
        if constexpr (R >= 8) {
            bfly<true>(a[0], a[4], tw_at(tw, k << (WH_MAXLOG - 3 - lh), inverse));
#pragma unroll
            for (int m = 1; m < 4; ++m) bfly(a[m], a[m + 4], tw_at(tw, (k + m * half) << (WH_MAXLOG - 3 - lh), inverse));
        }
    }
    static constexpr int rev(int m, int R) {
        return R == 8 ? ((m & 1) << 2) | (m & 2) | (m >> 2) : R == 4 ? ((m & 1) << 1) | (m >> 1) : m;
    }
    // one pass of radix R over the points of C transforms
    template <int R, int C>
    static __device__ void pass(float2 (&v)[C][P], int lh, int t, const float2* __restrict__ tw, bool inverse) {
#pragma unroll
        for (int b = 0; b < P / R; ++b) {
            const int k = (t + TC * b) & ((1 << lh) - 1);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                float2 a[R];
#pragma unroll
                for (int m = 0; m < R; ++m) a[m] = v[c][b + rev(m, R) * (P / R)];
                stages<R>(a, lh, k, tw, inverse);
#pragma unroll
                for (int m = 0; m < R; ++m) v[c][b + m * (P / R)] = a[m];
            }
            if (P > 8) __builtin_amdgcn_sched_barrier(0);   // (one butterfly's twiddles at a time: registers)
        }
    }
    // v[c][i] = point t + TC i of transform c, before and after; s: C LDS floats2 buffers of LDS each
    template <int C>
    static __device__ void run(float2 (&v)[C][P], float2* s, int t, const float2* __restrict__ tw, bool inverse) {
        constexpr int R8 = (LOGN % 3 == 0) ? LOGN / 3 - 1 : LOGN / 3;   // radix-8 passes before the last pass
#pragma unroll
        for (int p = 0; p < R8; ++p) {
            const int lh = 3 * p;
            pass<8, C>(v, lh, t, tw, inverse);
            if (p > 0) __syncthreads();   // the previous exchange is read
#pragma unroll
            for (int b = 0; b < P / 8; ++b) {
                const int j = t + TC * b, at = ((j >> lh) << (lh + 3)) + (j & ((1 << lh) - 1));
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int m = 0; m < 8; ++m) s[c * LDS + pad(at + (m << lh))] = v[c][b + m * (P / 8)];
            }
            __syncthreads();
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int i = 0; i < P; ++i) v[c][i] = s[c * LDS + pad(t + TC * i)];
        }
        pass<(LOGN % 3 == 0) ? 8 : (LOGN % 3 == 1) ? 2 : 4, C>(v, 3 * R8, t, tw, inverse);
    }
};

// Strided passes: workgroups of G transforms groups of C adjacent columns each.
template <int LOGN>
struct ColFft : RegFft<LOGN, 512> {
    using F = RegFft<LOGN, 512>;
    static constexpr int BT = F::TC < 64 ? 64 : F::TC;   // threads per workgroup
    static constexpr int G = BT / F::TC;
    static constexpr int C = F::P <= 16 ? 2 : 1;
    static constexpr int COLS = G * C;
};

// The four passes over a stream on register transforms (the small forms below say what each computes). vec:
// the channels are interleaved (x1 = x0 + 1, element stride 2) and 16-byte aligned, so a row's two
// columns are one 16-byte load.
template <int LOGN>
__global__ __launch_bounds__(ColFft<LOGN>::BT) void wh_cols_fwd_reg(const float* x0, const float* x1, int64_t es, int vec,
                                                                    int logn2, const float2* tw, float2* A) {
    using K = ColFft<LOGN>;
    __shared__ float2 s[K::G * K::C * K::LDS];
    const int t = threadIdx.x % K::TC, g = threadIdx.x / K::TC;
    const int64_t n2 = xcd_block((1ll << logn2) / K::COLS) * K::COLS + g * K::C;
    float2 v[K::C][K::P];
#pragma unroll
    for (int i = 0; i < K::P; ++i) {
        const int64_t at = ((int64_t)(t + K::TC * i) << logn2) + n2;
        if (K::C == 2 && vec) {
            const float4 q = *reinterpret_cast<const float4*>(x0 + 2 * at);
            v[0][i] = make_float2(q.x, q.y);
            v[K::C - 1][i] = make_float2(q.z, q.w);
        } else {
#pragma unroll
            for (int c = 0; c < K::C; ++c) v[c][i] = make_float2(x0[(at + c) * es], x1[(at + c) * es]);
        }
    }
    K::template run<K::C>(v, s + g * K::C * K::LDS, t, tw, false);
#pragma unroll
    for (int c = 0; c < K::C; ++c) {
        float2* out = A + ((n2 + c) << LOGN);
        TwiddleRun tr(n2 + c, t, K::TC, LOGN + logn2, false);
#pragma unroll
        for (int i = 0; i < K::P; ++i) out[t + K::TC * i] = cmul(v[c][i], tr.next());
    }
}

template <int LOGN>
__global__ __launch_bounds__(ColFft<LOGN>::BT) void wh_rows_fwd_reg(const float2* A, int logn1, const float2* tw, float2* T) {
    using K = ColFft<LOGN>;
    __shared__ float2 s[K::G * K::C * K::LDS];
    const int t = threadIdx.x % K::TC, g = threadIdx.x / K::TC;
    const int64_t k1 = xcd_block((1ll << logn1) / K::COLS) * K::COLS + g * K::C;
    float2 v[K::C][K::P];
#pragma unroll
    for (int i = 0; i < K::P; ++i) {
        const float2* src = A + ((int64_t)(t + K::TC * i) << logn1) + k1;
        if (K::C == 2) {
            const float4 q = *reinterpret_cast<const float4*>(src);
            v[0][i] = make_float2(q.x, q.y);
            v[K::C - 1][i] = make_float2(q.z, q.w);
        } else {
            v[0][i] = src[0];
        }
    }
    K::template run<K::C>(v, s + g * K::C * K::LDS, t, tw, false);
#pragma unroll
    for (int c = 0; c < K::C; ++c)
#pragma unroll
        for (int i = 0; i < K::P; ++i) T[((k1 + c) << LOGN) + t + K::TC * i] = v[c][i];
}

template <int LOGN>
__global__ __launch_bounds__(ColFft<LOGN>::BT) void wh_rows_inv_reg(const float2* T, int logn1, const float2* tw, float2* C) {
    using K = ColFft<LOGN>;
    __shared__ float2 s[K::G * K::LDS];
    const int t = threadIdx.x % K::TC, g = threadIdx.x / K::TC;
    const int64_t k1 = (int64_t)blockIdx.x * K::G + g;
    float2 v[1][K::P];
#pragma unroll
    for (int i = 0; i < K::P; ++i) v[0][i] = T[(k1 << LOGN) + t + K::TC * i];
    K::template run<1>(v, s + g * K::LDS, t, tw, true);
    TwiddleRun tr(k1, t, K::TC, logn1 + LOGN, true);
#pragma unroll
    for (int i = 0; i < K::P; ++i) C[(k1 << LOGN) + t + K::TC * i] = cmul(v[0][i], tr.next());
}

// 1 / (L sqrt(P_c(f_k) fs / 2)): the PSD linearly interpolated at bin k of L (grid position
// k n / L), with the inverse transform's 1/L folded in.
__device__ inline float wh_coef(const double* psd, int h, int c, int64_t k, int sh, int logl, double fs) {
    const int64_t j = k >> sh;
    const double fr = ldexp((double)(k & ((1ll << sh) - 1)), -sh);
    const double* p = psd + (int64_t)c * h;
    const double pk = fr == 0.0 ? p[j] : p[j] * (1.0 - fr) + p[j + 1] * fr;
    // 1 / sqrt by the hardware estimate and two Newton steps (to a few float64 ulp; a square root and a
    // division in float64 were most of the spectrum pass); 0 and infinity keep their estimates
    const double q = pk * fs * 0.5;
    double r = __builtin_amdgcn_rsq(q);
    if (r > 0.0 && r < INFINITY) {
        r = r * fma(-0.5 * q * r, r, 1.5);
        r = r * fma(-0.5 * q * r, r, 1.5);
    }
    return (float)ldexp(r, -logl);
}

// The spectrum division of the bin pair z (bin k <= L - k) and zp (bin L - k): separate the channels, scale
// each by its coefficient, recombine.
__device__ inline void wh_divide(float2& z, float2& zp, const double* psd, int h, int64_t k, int sh, int logl, double fs) {
    const float2 X0 = make_float2(0.5f * (z.x + zp.x), 0.5f * (z.y - zp.y));
    const float2 X1 = make_float2(0.5f * (z.y + zp.y), -0.5f * (z.x - zp.x));
    const float a0 = wh_coef(psd, h, 0, k, sh, logl, fs);
    const float a1 = wh_coef(psd, h, 1, k, sh, logl, fs);
    z = make_float2(a0 * X0.x - a1 * X1.y, a0 * X0.y + a1 * X1.x);
    zp = make_float2(a0 * X0.x + a1 * X1.y, a1 * X1.x - a0 * X0.y);
}

// The spectrum division and the inverse row pass in one: workgroup group q takes rows q and N1 - q, which
// hold each other's bin pairs (element k2 of row q meets N2 - 1 - k2 of row N1 - q; rows 0 and N1 / 2 meet
// themselves), so the divided spectrum never goes through memory (2^24 samples: 75 + 118 us for the two
// passes before).
template <int LOGN>
__global__ __launch_bounds__(ColFft<LOGN>::BT) void wh_divide_rows_inv_reg(const float2* T, int logn1, const double* psd,
                                                                           int logn, double fs, const float2* tw, float2* C) {
    using K = ColFft<LOGN>;
    static_assert(K::C == 2, "two rows in registers");
    __shared__ float2 lds[K::G * 2 * K::LDS];
    const int t = threadIdx.x % K::TC, g = threadIdx.x / K::TC;
    const int64_t n1c = 1ll << logn1, q = (int64_t)blockIdx.x * K::G + g, ka = min(q, n1c / 2), kb = (n1c - ka) & (n1c - 1);
    const int logl = logn1 + LOGN, h = (1 << logn) / 2 + 1, sh = logl - logn;
    float2* s = lds + g * 2 * K::LDS;
    float2 v[2][K::P];
#pragma unroll
    for (int i = 0; i < K::P; ++i) {
        v[0][i] = T[(ka << LOGN) + t + K::TC * i];
        v[1][i] = T[(kb << LOGN) + t + K::TC * i];
        s[K::pad(t + K::TC * i)] = v[1][i];
    }
    __syncthreads();
    const bool own = ka == kb;   // the row meets itself
#pragma unroll
    for (int i = 0; i < K::P; ++i) {
        const int k2 = t + K::TC * i, p2 = (ka == 0 ? K::N - k2 : K::N - 1 - k2) & (K::N - 1);
        const int64_t k = ka + ((int64_t)k2 << logn1), kp = kb + ((int64_t)p2 << logn1);
        float2 zp = s[K::pad(p2)];
        if (k <= kp) wh_divide(v[0][i], zp, psd, h, k, sh, logl, fs);
        else wh_divide(zp, v[0][i], psd, h, kp, sh, logl, fs);
        if (!own) s[K::pad(p2)] = zp;   // (each element of row N1 - q is read and written by one thread)
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < K::P; ++i) v[1][i] = s[K::pad(t + K::TC * i)];
    __syncthreads();
    K::template run<2>(v, s, t, tw, true);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int64_t k1 = c ? kb : ka;
        TwiddleRun tr(k1, t, K::TC, logl, true);
        if (q > n1c / 2 || (c == 1 && own)) continue;
#pragma unroll
        for (int i = 0; i < K::P; ++i) C[(k1 << LOGN) + t + K::TC * i] = cmul(v[c][i], tr.next());
    }
}

template <int LOGN>
__global__ __launch_bounds__(ColFft<LOGN>::BT) void wh_cols_inv_reg(const float2* C, int logn2, const float2* tw, float2* yt,
                                                                    double* part) {
    using K = ColFft<LOGN>;
    __shared__ float2 s[K::G * K::C * K::LDS];
    const int t = threadIdx.x % K::TC, g = threadIdx.x / K::TC;
    const int64_t blk = xcd_block((1ll << logn2) / K::COLS), n2 = blk * K::COLS + g * K::C;
    float2 v[K::C][K::P];
#pragma unroll
    for (int i = 0; i < K::P; ++i) {
        const float2* src = C + ((int64_t)(t + K::TC * i) << logn2) + n2;
        if (K::C == 2) {
            const float4 q = *reinterpret_cast<const float4*>(src);
            v[0][i] = make_float2(q.x, q.y);
            v[K::C - 1][i] = make_float2(q.z, q.w);
        } else {
            v[0][i] = src[0];
        }
    }
    K::template run<K::C>(v, s + g * K::C * K::LDS, t, tw, true);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < K::C; ++c)
#pragma unroll
        for (int i = 0; i < K::P; ++i) {
            const float2 y = v[c][i];
            yt[((n2 + c) << LOGN) + t + K::TC * i] = y;
            acc[0] += y.x;
            acc[1] += (double)y.x * y.x;
            acc[2] += y.y;
            acc[3] += (double)y.y * y.y;
        }
    // the workgroup's sums: within each wave, then the waves in order
    __syncthreads();
    double* red = (double*)s;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        for (int o = 32; o > 0; o >>= 1) acc[q] += __shfl_xor(acc[q], o);
        if ((threadIdx.x & 63) == 0) red[(threadIdx.x >> 6) * 4 + q] = acc[q];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        double sum = 0.0;
        for (int w = 0; w < K::BT / 64; ++w) sum += red[w * 4 + threadIdx.x];
        part[blk * 4 + threadIdx.x] = sum;
    }
}

// The Welch kernel below on register transforms (one per workgroup; 2^14 points on 1024 threads, whose
// points, window and sums fit 128 registers).
template <int LOGN>
using WelchFft = RegFft<LOGN, LOGN == 14 ? 1024 : 512>;
template <int LOGN>
__global__ __launch_bounds__((WelchFft<LOGN>::TC)) void wh_welch_reg(const float* x0, const float* x1, int64_t es,
                                                                         int64_t nseg, const float2* tw, double* part) {
    using F = WelchFft<LOGN>;
    constexpr int N = F::N, H = N / 2 + 1, NB = F::P / 2;   // bins t + TC i, i < NB, and bin N/2 in thread 0
    __shared__ float2 s[F::LDS];
    const int t = threadIdx.x;
    const int64_t g = blockIdx.x, G = gridDim.x;
    const int64_t s0 = nseg * g / G, s1 = nseg * (g + 1) / G;
    double acc0[NB + 1], acc1[NB + 1];
    float win[F::P];
#pragma unroll
    for (int i = 0; i <= NB; ++i) acc0[i] = acc1[i] = 0.0;
#pragma unroll
    for (int i = 0; i < F::P; ++i) win[i] = (float)(0.5 - 0.5 * cospi(ldexp((double)(t + F::TC * i), 1 - LOGN)));
    for (int64_t seg = s0; seg < s1; ++seg) {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));   // (twiddles and LDS addresses are formed per segment, not kept in registers)
        const int64_t t0 = seg * (N / 2) + t;
        float2 v[1][F::P];
#pragma unroll
        for (int i = 0; i < F::P; ++i) {
            const int64_t at = (t0 + F::TC * i) * es;
            v[0][i] = make_float2(win[i] * x0[at], win[i] * x1[at]);
        }
        __syncthreads();   // the previous segment's spectrum has been read
        F::template run<1>(v, s, t, tw, false);
        __syncthreads();   // the last exchange is read
#pragma unroll
        for (int i = 0; i < F::P; ++i) s[F::pad(t + F::TC * i)] = v[0][i];
        __syncthreads();
        auto add = [&](int i, float2 z, float2 zp) {
            const double a0 = 0.5 * ((double)z.x + zp.x), b0 = 0.5 * ((double)z.y - zp.y);
            const double a1 = 0.5 * ((double)z.y + zp.y), b1 = -0.5 * ((double)z.x - zp.x);
            acc0[i] += a0 * a0 + b0 * b0;
            acc1[i] += a1 * a1 + b1 * b1;
        };
#pragma unroll
        for (int i = 0; i < NB; ++i) add(i, v[0][i], s[F::pad((N - (t + F::TC * i)) & (N - 1))]);
        if (t == 0) add(NB, v[0][NB], v[0][NB]);
    }
    double* out = part + g * 2 * H;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        out[t + F::TC * i] = acc0[i];
        out[H + t + F::TC * i] = acc1[i];
    }
    if (t == 0) {
        out[N / 2] = acc0[NB];
        out[H + N / 2] = acc1[NB];
    }
}

// Welch: workgroup g takes the contiguous run of segments [nseg g / G, nseg (g + 1) / G) in order.
// Each segment: both channels windowed into one complex sequence, transformed, separated; every
// thread keeps |X_c[k]|^2 summed in float64 registers for its bins k = tid + 64 i, and the run's sums
// go to part[(g * 2 + c) * h + k], h = n/2 + 1.
__global__ __launch_bounds__(WH_SMALL) void wh_welch_kernel(const float* x0, const float* x1, int64_t es,
                                                             int logn, int64_t nseg, const float2* tw,
                                                             double* part) {
    __shared__ float2 s[WH_SMALLN];
    constexpr int NB = (WH_SMALLN / 2 + WH_SMALL) / WH_SMALL;   // bins per thread
    constexpr int NW = WH_SMALLN / WH_SMALL;                               // samples per thread
    const int n = 1 << logn;
    const int h = n / 2 + 1;
    const int64_t g = blockIdx.x, G = gridDim.x;
    const int64_t s0 = nseg * g / G, s1 = nseg * (g + 1) / G;
    double acc0[NB], acc1[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) acc0[i] = acc1[i] = 0.0;
    // the window of this thread's samples, once for all segments
    float win[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i)
        win[i] = (float)(0.5 - 0.5 * cospi(ldexp((double)(threadIdx.x + WH_SMALL * i), 1 - logn)));
    for (int64_t seg = s0; seg < s1; ++seg) {
        const int64_t t0 = seg * (n / 2);
        __syncthreads();   // the previous segment's spectrum has been read
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const int j = threadIdx.x + WH_SMALL * i;
            if (j < n) {
                const int64_t t = (t0 + j) * es;
                s[bitrev(j, logn)] = make_float2(win[i] * x0[t], win[i] * x1[t]);
            }
        }
        lds_fft(s, logn, tw, false);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int k = threadIdx.x + WH_SMALL * i;
            if (k < h) {
                const float2 z = s[k], zp = s[(n - k) & (n - 1)];
                const double a0 = 0.5 * ((double)z.x + zp.x), b0 = 0.5 * ((double)z.y - zp.y);
                const double a1 = 0.5 * ((double)z.y + zp.y), b1 = -0.5 * ((double)z.x - zp.x);
                acc0[i] += a0 * a0 + b0 * b0;
                acc1[i] += a1 * a1 + b1 * b1;
            }
        }
    }
    double* out = part + g * 2 * h;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int k = threadIdx.x + WH_SMALL * i;
        if (k < h) {
            out[k] = acc0[i];
            out[h + k] = acc1[i];
        }
    }
}

// The workgroups' sums added in workgroup order, in two fixed levels: WH_RG contiguous runs of
// workgroups, then the runs; scaled to the one-sided density.
constexpr int WH_RG = 16;

__global__ void wh_welch_runs_kernel(const double* part, int64_t groups, int h, double* runs) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 2 * h) return;
    const int64_t y = blockIdx.y;
    const int64_t g0 = groups * y / WH_RG, g1 = groups * (y + 1) / WH_RG;
    double acc = 0.0;
    for (int64_t g = g0; g < g1; ++g) acc += part[g * 2 * h + i];
    runs[y * 2 * h + i] = acc;
}

__global__ void wh_welch_reduce_kernel(const double* runs, int h, double scale, double* psd) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 2 * h) return;
    const int k = i % h;
    double acc = 0.0;
    for (int y = 0; y < WH_RG; ++y) acc += runs[(int64_t)y * 2 * h + i];
    psd[i] = acc * scale * ((k == 0 || k == h - 1) ? 1.0 : 2.0);
}

// Forward column pass: workgroup n2 transforms z[n1 N2 + n2] over n1 and writes
// A[n2 N1 + k1] = Z_n2[k1] e^(-2 pi i n2 k1 / L).
__global__ __launch_bounds__(WH_SMALL) void wh_cols_fwd_kernel(const float* x0, const float* x1, int64_t es, int logn1,
                                                              int logn2, const float2* tw, float2* A) {
    __shared__ float2 s[WH_SMALLN];
    const int n1c = 1 << logn1;
    const int64_t n2 = blockIdx.x;
    for (int j = threadIdx.x; j < n1c; j += blockDim.x) {
        const int64_t t = ((int64_t)j << logn2) + n2;
        s[bitrev(j, logn1)] = make_float2(x0[t * es], x1[t * es]);
    }
    lds_fft(s, logn1, tw, false);
    float2* out = A + (n2 << logn1);
    TwiddleRun tr(n2, threadIdx.x, WH_SMALL, logn1 + logn2, false);
    for (int k1 = threadIdx.x; k1 < n1c; k1 += blockDim.x) out[k1] = cmul(s[k1], tr.next());
}

// Forward row pass: workgroup k1 transforms A[n2 N1 + k1] over n2 and writes T[k1 N2 + k2].
__global__ __launch_bounds__(WH_SMALL) void wh_rows_fwd_kernel(const float2* A, int logn1, int logn2, const float2* tw,
                                                              float2* T) {
    __shared__ float2 s[WH_SMALLN];
    const int n2c = 1 << logn2;
    const int64_t k1 = blockIdx.x;
    for (int j = threadIdx.x; j < n2c; j += blockDim.x) s[bitrev(j, logn2)] = A[((int64_t)j << logn1) + k1];
    lds_fft(s, logn2, tw, false);
    for (int k2 = threadIdx.x; k2 < n2c; k2 += blockDim.x) T[(k1 << logn2) + k2] = s[k2];
}

// Spectrum division on the transposed spectrum, in place. The thread of bin k <= L - k handles the
// pair (k, L - k): separate the channels, scale each by its coefficient, recombine.
__global__ void wh_spectrum_kernel(float2* T, int logn1, int logn2, const double* psd, int logn, double fs) {
    const int logl = logn1 + logn2;
    const int64_t L = 1ll << logl;
    const int h = (1 << logn) / 2 + 1;
    const int sh = logl - logn;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < L; p += step) {
        const int64_t k = (p >> logn2) + ((p & ((1ll << logn2) - 1)) << logn1);
        const int64_t kp = (L - k) & (L - 1);
        if (k > kp) continue;
        const int64_t pp = ((kp & ((1ll << logn1) - 1)) << logn2) + (kp >> logn1);
        float2 z = T[p], zp = T[pp];
        wh_divide(z, zp, psd, h, k, sh, logl, fs);
        T[p] = z;
        if (pp != p) T[pp] = zp;
    }
}

// Inverse row pass: workgroup k1 inverse-transforms T[k1 N2 + k2] over k2 and writes
// C[k1 N2 + n2] = c_k1[n2] e^(+2 pi i n2 k1 / L).
__global__ __launch_bounds__(WH_SMALL) void wh_rows_inv_kernel(const float2* T, int logn1, int logn2, const float2* tw,
                                                              float2* C) {
    __shared__ float2 s[WH_SMALLN];
    const int n2c = 1 << logn2;
    const int64_t k1 = blockIdx.x;
    for (int j = threadIdx.x; j < n2c; j += blockDim.x) s[bitrev(j, logn2)] = T[(k1 << logn2) + j];
    lds_fft(s, logn2, tw, true);
    TwiddleRun tr(k1, threadIdx.x, WH_SMALL, logn1 + logn2, true);
    for (int n2 = threadIdx.x; n2 < n2c; n2 += blockDim.x) C[(k1 << logn2) + n2] = cmul(s[n2], tr.next());
}

// Inverse column pass: workgroup n2 inverse-transforms C[k1 N2 + n2] over k1 into column n2 of y (channel 0
// real part, channel 1 imaginary part), stored contiguously as yt[n2 N1 + n1] (the interleaved output is
// written by the transpose below), and leaves its float64 sums of y and y^2 per channel in
// part[n2 * 4 + {0..3}].
__global__ __launch_bounds__(WH_SMALL) void wh_cols_inv_kernel(const float2* C, int logn1, int logn2, const float2* tw,
                                                              float2* yt, double* part) {
    __shared__ float2 s[WH_SMALLN];
    const int n1c = 1 << logn1;
    const int64_t n2 = blockIdx.x;
    for (int j = threadIdx.x; j < n1c; j += blockDim.x) s[bitrev(j, logn1)] = C[((int64_t)j << logn2) + n2];
    lds_fft(s, logn1, tw, true);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int j = threadIdx.x; j < n1c; j += blockDim.x) {
        const float2 y = s[j];
        yt[(n2 << logn1) + j] = y;
        acc[0] += y.x;
        acc[1] += (double)y.x * y.x;
        acc[2] += y.y;
        acc[3] += (double)y.y * y.y;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        for (int o = 32; o > 0; o >>= 1) acc[q] += __shfl_xor(acc[q], o);
        if (threadIdx.x == 0) part[n2 * 4 + q] = acc[q];
    }
}

// 1 / sigma per channel from the per-workgroup sums (fixed summation order).
__global__ void wh_sigma_kernel(const double* part, int64_t nblk, int logl, float* inv_sigma) {
    __shared__ double red[4][256];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t b = threadIdx.x; b < nblk; b += blockDim.x)
        for (int q = 0; q < 4; ++q) acc[q] += part[b * 4 + q];
    for (int q = 0; q < 4; ++q) red[q][threadIdx.x] = acc[q];
    for (int w = 128; w > 0; w >>= 1) {
        __syncthreads();
        if ((int)threadIdx.x < w)
            for (int q = 0; q < 4; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + w];
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const double inv_l = ldexp(1.0, -logl);
        const double mean = red[2 * threadIdx.x][0] * inv_l;
        const double var = red[2 * threadIdx.x + 1][0] * inv_l - mean * mean;
        inv_sigma[threadIdx.x] = (float)(1.0 / sqrt(var));
    }
}

// out[n1 N2 + n2] = yt[n2 N1 + n1] * (1 / sigma per channel, or 1 without normalisation), through a
// 32 x 32 LDS tile so that both the reads (along n1) and the writes (along n2) are contiguous.
constexpr int WH_TT = 32;

__global__ __launch_bounds__(256) void wh_transpose_kernel(const float2* yt, int logn1, int logn2,
                                                         const float* inv_sigma, float2* out) {
    __shared__ float2 tile[WH_TT][WH_TT + 1];
    const int n1c = 1 << logn1, n2c = 1 << logn2;
    const int b1 = blockIdx.x * WH_TT, b2 = blockIdx.y * WH_TT;
    const float s0 = inv_sigma ? inv_sigma[0] : 1.0f, s1 = inv_sigma ? inv_sigma[1] : 1.0f;
    const int tx = threadIdx.x & (WH_TT - 1), ty = threadIdx.x / WH_TT;   // 32 x 8 threads
    for (int r = ty; r < WH_TT; r += 256 / WH_TT) {
        const int n2 = b2 + r, n1 = b1 + tx;
        if (n2 < n2c && n1 < n1c) tile[r][tx] = yt[((int64_t)n2 << logn1) + n1];
    }
    __syncthreads();
    for (int r = ty; r < WH_TT; r += 256 / WH_TT) {
        const int n1 = b1 + r, n2 = b2 + tx;
        if (n1 < n1c && n2 < n2c) {
            const float2 y = tile[tx][r];
            out[((int64_t)n1 << logn2) + n2] = make_float2(y.x * s0, y.y * s1);
        }
    }
}

// grow-only device workspace (twiddle table first), shared by the calls of the process
struct WhitenWs {
    std::mutex mu;
    void* buf = nullptr;
    int64_t bytes = 0;
    int device = -1;
};
static WhitenWs g_wh;

constexpr int64_t WH_TW_BYTES = (int64_t)WH_TW * 8;

static gwd_status wh_workspace(int64_t need, hipStream_t st, char** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    need += WH_TW_BYTES;
    if (g_wh.bytes < need || g_wh.device != dev) {
        if (g_wh.buf) {
            (void)hipDeviceSynchronize();
            (void)hipFree(g_wh.buf);
            g_wh.buf = nullptr;
            g_wh.bytes = 0;
        }
        e = hipMalloc(&g_wh.buf, need);
        if (e != hipSuccess) return hip_fail(e, "hipMalloc(whitening workspace)");
        g_wh.bytes = need;
        g_wh.device = dev;
        hipLaunchKernelGGL(wh_twiddle_kernel, dim3(WH_TW / 256), dim3(256), 0, st, (float2*)g_wh.buf);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(st);   // the table serves calls on any stream
        if (e != hipSuccess) return hip_fail(e, "twiddle table");
    }
    *out = (char*)g_wh.buf;
    return GWD_OK;
}

// f(constant logn) for the sizes the register transforms are built for (smaller ones are latency-bound
// either way and stay on lds_fft, which takes any size); false for others.
template <class F>
static bool reg_fft_size(int logn, F f) {
    switch (logn) {
        case 8: f(std::integral_constant<int, 8>{}); return true;
        case 9: f(std::integral_constant<int, 9>{}); return true;
        case 10: f(std::integral_constant<int, 10>{}); return true;
        case 11: f(std::integral_constant<int, 11>{}); return true;
        case 12: f(std::integral_constant<int, 12>{}); return true;
        case 13: f(std::integral_constant<int, 13>{}); return true;
        case 14: f(std::integral_constant<int, 14>{}); return true;
        default: return false;
    }
}

static int log2_exact(int64_t v) {
    if (v <= 0 || (v & (v - 1))) return -1;
    int l = 0;
    while ((1ll << l) < v) ++l;
    return l;
}

static gwd_status check_stream(const gwd_stream* src, const char* who) {
    if (!src || !src->ch[0] || !src->ch[1]) { set_error("%s: NULL stream or channel pointer", who); return GWD_ERR_ARG; }
    if (src->elem_stride < 1 || src->length < 0) { set_error("%s: elem_stride < 1 or negative length", who); return GWD_ERR_ARG; }
    if (((uintptr_t)src->ch[0] & 3) || ((uintptr_t)src->ch[1] & 3)) { set_error("%s: misaligned channel pointer", who); return GWD_ERR_ARG; }
    return GWD_OK;
}

static gwd_status check_fs_n(int32_t nperseg, double fs, const char* who, int* logn) {
    *logn = log2_exact(nperseg);
    if (*logn < 4 || *logn > WH_MAXLOG) { set_error("%s: nperseg must be a power of two in [16, 16384]", who); return GWD_ERR_ARG; }
    if (!(fs > 0.0) || !std::isfinite(fs)) { set_error("%s: fs must be positive and finite", who); return GWD_ERR_ARG; }
    return GWD_OK;
}

}  // namespace gwd

using namespace gwd;

gwd_status gwd_welch_psd(const gwd_stream* src, int32_t nperseg, double fs, double* psd, void* hip_stream) {
    gwd_status r = check_stream(src, "gwd_welch_psd");
    if (r != GWD_OK) return r;
    int logn = 0;
    r = check_fs_n(nperseg, fs, "gwd_welch_psd", &logn);
    if (r != GWD_OK) return r;
    if (!psd || ((uintptr_t)psd & 7)) { set_error("gwd_welch_psd: NULL or misaligned psd"); return GWD_ERR_ARG; }
    if (src->length < nperseg) { set_error("gwd_welch_psd: stream shorter than one segment"); return GWD_ERR_SHAPE; }
    const int64_t nseg = (src->length - nperseg) / (nperseg / 2) + 1;
    if (nseg > 0x7fffffff) { set_error("gwd_welch_psd: too many segments"); return GWD_ERR_SHAPE; }
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) { set_error("gwd_welch_psd: no HIP device"); return GWD_ERR_NO_DEVICE; }
    hipStream_t st = (hipStream_t)hip_stream;
    const int h = nperseg / 2 + 1;
    // one workgroup per CU for the 128 KB transforms, four for the 32 KB ones, none without a segment
    const int64_t groups = std::min<int64_t>(nseg, logn > 12 ? 256 : 1024);
    std::lock_guard<std::mutex> lock(g_wh.mu);
    char* ws = nullptr;
    r = wh_workspace((groups + WH_RG) * 2 * h * 8, st, &ws);
    if (r != GWD_OK) return r;
    const float2* tw = (const float2*)ws;
    double* part = (double*)(ws + WH_TW_BYTES);
    double* runs = part + groups * 2 * h;
    if (!reg_fft_size(logn, [&](auto n) {
            constexpr int LOGN = decltype(n)::value;
            hipLaunchKernelGGL(wh_welch_reg<LOGN>, dim3((unsigned)groups), dim3(WelchFft<LOGN>::TC), 0, st, src->ch[0],
                               src->ch[1], src->elem_stride, nseg, tw, part);
        }))
        hipLaunchKernelGGL(wh_welch_kernel, dim3((unsigned)groups), dim3(WH_SMALL), 0, st, src->ch[0], src->ch[1],
                           src->elem_stride, logn, nseg, tw, part);
    // sum of the squared periodic Hann window: 3n/8
    const double scale = 1.0 / ((double)nseg * fs * (3.0 * nperseg / 8.0));
    hipLaunchKernelGGL(wh_welch_runs_kernel, dim3((2 * h + 255) / 256, WH_RG), dim3(256), 0, st, (const double*)part, groups,
                       h, runs);
    hipLaunchKernelGGL(wh_welch_reduce_kernel, dim3((2 * h + 255) / 256), dim3(256), 0, st, (const double*)runs, h, scale,
                       psd);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? GWD_OK : hip_fail(e, "Welch kernel launch");
}

gwd_status gwd_whiten(const gwd_stream* src, const double* psd, int32_t nperseg, double fs, int32_t normalize,
                      float* dst, void* hip_stream) {
    gwd_status r = check_stream(src, "gwd_whiten");
    if (r != GWD_OK) return r;
    int logn = 0;
    r = check_fs_n(nperseg, fs, "gwd_whiten", &logn);
    if (r != GWD_OK) return r;
    if (!psd || ((uintptr_t)psd & 7)) { set_error("gwd_whiten: NULL or misaligned psd"); return GWD_ERR_ARG; }
    if (!dst || ((uintptr_t)dst & 7)) { set_error("gwd_whiten: NULL or misaligned output"); return GWD_ERR_ARG; }
    if (normalize != 0 && normalize != 1) { set_error("gwd_whiten: normalize must be 0 or 1"); return GWD_ERR_ARG; }
    const int logl = log2_exact(src->length);
    if (logl < 4 || logl > 2 * WH_MAXLOG) { set_error("gwd_whiten: length must be a power of two in [16, 2^28]"); return GWD_ERR_SHAPE; }
    if (logn > logl) { set_error("gwd_whiten: nperseg longer than the stream"); return GWD_ERR_SHAPE; }
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) { set_error("gwd_whiten: no HIP device"); return GWD_ERR_NO_DEVICE; }
    hipStream_t st = (hipStream_t)hip_stream;
    const int logn1 = (logl + 1) / 2, logn2 = logl / 2;
    const int64_t L = 1ll << logl, n1c = 1ll << logn1, n2c = 1ll << logn2;
    std::lock_guard<std::mutex> lock(g_wh.mu);
    char* ws = nullptr;
    r = wh_workspace(2 * L * 8 + n2c * 32 + 16, st, &ws);
    if (r != GWD_OK) return r;
    const float2* tw = (const float2*)ws;
    float2* A = (float2*)(ws + WH_TW_BYTES);
    float2* T = A + L;
    double* part = (double*)(T + L);
    float* inv_sigma = (float*)(part + 4 * n2c);
    const int vec_in = src->elem_stride == 2 && src->ch[1] == src->ch[0] + 1 && ((uintptr_t)src->ch[0] & 15) == 0;
    int64_t nblk_c = n2c;   // workgroups of the column passes
    if (!reg_fft_size(logn1, [&](auto n) {
            using K = ColFft<decltype(n)::value>;
            nblk_c = n2c / K::COLS;
            hipLaunchKernelGGL(wh_cols_fwd_reg<decltype(n)::value>, dim3((unsigned)nblk_c), dim3(K::BT), 0, st, src->ch[0],
                               src->ch[1], src->elem_stride, vec_in, logn2, tw, A);
        }))
        hipLaunchKernelGGL(wh_cols_fwd_kernel, dim3((unsigned)n2c), dim3(WH_SMALL), 0, st, src->ch[0], src->ch[1],
                           src->elem_stride, logn1, logn2, tw, A);
    if (!reg_fft_size(logn2, [&](auto n) {
            using K = ColFft<decltype(n)::value>;
            hipLaunchKernelGGL(wh_rows_fwd_reg<decltype(n)::value>, dim3((unsigned)(n1c / K::COLS)), dim3(K::BT), 0, st,
                               (const float2*)A, logn1, tw, T);
        }))
        hipLaunchKernelGGL(wh_rows_fwd_kernel, dim3((unsigned)n1c), dim3(WH_SMALL), 0, st, (const float2*)A, logn1, logn2,
                           tw, T);
    const unsigned sblocks = (unsigned)std::min<int64_t>((L + 255) / 256, 16384);
    if (logn2 <= 13 && reg_fft_size(logn2, [&](auto n) {   // (rows of 2^14 points do not fit in pairs)
            constexpr int LOGN = decltype(n)::value < 14 ? decltype(n)::value : 13;
            using K = ColFft<LOGN>;
            hipLaunchKernelGGL(wh_divide_rows_inv_reg<LOGN>, dim3((unsigned)((n1c / 2 + K::G) / K::G)), dim3(K::BT), 0, st,
                               (const float2*)T, logn1, psd, logn, fs, tw, A);
        })) {
    } else {
        hipLaunchKernelGGL(wh_spectrum_kernel, dim3(sblocks), dim3(256), 0, st, T, logn1, logn2, psd, logn, fs);
        if (logn2 == 14)
            hipLaunchKernelGGL(wh_rows_inv_reg<14>, dim3((unsigned)n1c), dim3(ColFft<14>::BT), 0, st, (const float2*)T, logn1,
                               tw, A);
        else
            hipLaunchKernelGGL(wh_rows_inv_kernel, dim3((unsigned)n1c), dim3(WH_SMALL), 0, st, (const float2*)T, logn1,
                               logn2, tw, A);
    }
    // the columns of y go to T (free again), then one transpose writes the interleaved output
    if (!reg_fft_size(logn1, [&](auto n) {
            using K = ColFft<decltype(n)::value>;
            hipLaunchKernelGGL(wh_cols_inv_reg<decltype(n)::value>, dim3((unsigned)nblk_c), dim3(K::BT), 0, st,
                               (const float2*)A, logn2, tw, T, part);
        }))
        hipLaunchKernelGGL(wh_cols_inv_kernel, dim3((unsigned)n2c), dim3(WH_SMALL), 0, st, (const float2*)A, logn1, logn2, tw,
                           T, part);
    if (normalize)
        hipLaunchKernelGGL(wh_sigma_kernel, dim3(1), dim3(256), 0, st, (const double*)part, nblk_c, logl, inv_sigma);
    const dim3 tgrid((unsigned)((n1c + WH_TT - 1) / WH_TT), (unsigned)((n2c + WH_TT - 1) / WH_TT));
    hipLaunchKernelGGL(wh_transpose_kernel, tgrid, dim3(256), 0, st, (const float2*)T, logn1, logn2,
                       normalize ? (const float*)inv_sigma : (const float*)nullptr, (float2*)dst);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? GWD_OK : hip_fail(e, "whitening kernel launch");
}
