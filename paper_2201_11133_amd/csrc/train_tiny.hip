// Training of the small plain member (four causal convolutions, 16 channels, ReLU, 1x1 to a logit)
// in float or double; double is used for the finite-difference gradient check on the device.
//
// The member is 3,232 flop per time step, so a step is bound by launches and latency, not by
// arithmetic (64 windows: 2.5 GFLOP with the backward, 16 us at the fp32 matrix rate). Both passes
// keep one time step per thread and carry it through all four layers in one kernel: a row's 16
// channels stay in registers, LDS holds only what neighbouring rows read (the dilation taps), and the
// weights, the same for every lane, are scalar operands. A tile recomputes the few rows its
// neighbours own (14 in the forward, 16 in the backward of 256), which costs less than a launch. The
// weight gradients are sums over all rows in a fixed order, taken by a second kernel.
#include "train_internal.h"

namespace gwd {

constexpr int TC = 16;
constexpr int TN = 256;                   // threads (time steps) per tile
constexpr int TF_HALO = 14;               // forward: rows left of the tile (dilations 2 + 4 + 8)
constexpr int TF_ROWS = TN - TF_HALO;
constexpr int TB_HALO = 16;               // backward: rows right of the tile (8 + 4 + 2 + 1, rounded)
constexpr int TB_ROWS = TN - TB_HALO;
constexpr int T_PARAMS = 80 + 3 * 528 + 17;
constexpr int T_RES = 256;                // weight gradients: partial sums by row index mod 256

// blob offsets: conv0 (W [16][2][2], b [16]) = 80 values, conv1..3 (W [16][16][2], b) = 528 each, out W [16], b [1]
__host__ __device__ constexpr int tiny_off(int layer) { return layer == 0 ? 0 : 80 + 528 * (layer - 1); }
__host__ __device__ constexpr int tiny_cin(int layer) { return layer == 0 ? 2 : TC; }

// LDS rows of 16 channels, padded so that 16-byte accesses of consecutive rows spread over the banks.
template <class T>
constexpr int tiny_ld() { return TC + 16 / (int)sizeof(T); }

// The 16 channels of one row, as 16-byte accesses (LDS rows, and rows of ys: 4-byte aligned is enough
// for global memory).
template <class T>
__device__ inline void load_row(const T* p, T (&v)[TC]) {
    typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
    constexpr int E = 16 / sizeof(T);
#pragma unroll
    for (int i = 0; i < TC / E; ++i) {
        const vec x = *(const vec*)(p + E * i);
#pragma unroll
        for (int j = 0; j < E; ++j) v[E * i + j] = x[j];
    }
}
template <class T>
__device__ inline void store_row(T* p, const T (&v)[TC]) {
    typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
    constexpr int E = 16 / sizeof(T);
#pragma unroll
    for (int i = 0; i < TC / E; ++i) {
        vec x;
#pragma unroll
        for (int j = 0; j < E; ++j) x[j] = v[E * i + j];
        *(vec*)(p + E * i) = x;
    }
}

// acc[o] = b[o] + sum_c (W[o][c][0] xo[c] + W[o][c][1] xc[c]), channel by channel, the tap at t - d
// only where it lies inside the window (`tap`). An output's weights are consecutive: wide scalar loads.
template <class T, int CIN>
__device__ inline void tiny_conv(const T* __restrict__ W, const T (&xo)[CIN], const T (&xc)[CIN], bool tap, T (&acc)[TC]) {
    const T* b = W + TC * CIN * 2;
#pragma unroll
    for (int o = 0; o < TC; ++o) {
        T s = b[o];
#pragma unroll
        for (int c = 0; c < CIN; ++c) {
            const T far = s + W[(o * CIN + c) * 2 + 0] * xo[c];
            s = tap ? far : s;
            s += W[(o * CIN + c) * 2 + 1] * xc[c];
        }
        acc[o] = s;
    }
}

// Layer outputs ys [4][M][16] and logits z [M] of windows u [M][2]. Block: one tile of TF_ROWS rows of
// one window, thread tid the row t0 - TF_HALO + tid. 64 windows of 4096: 744 us (one launch per layer,
// one output per thread, every weight a vector load) -> 46 us.
template <class T>
__global__ __launch_bounds__(TN) void tiny_fwd_kernel(const T* __restrict__ blob, const float* __restrict__ u,
                                                      int64_t M, int Tw, int tiles, T* __restrict__ ys, T* __restrict__ z) {
    constexpr int LD = tiny_ld<T>();
    __shared__ __attribute__((aligned(16))) T y[2][TN][LD];
    const int tid = threadIdx.x;
    const int64_t b = blockIdx.x / tiles;
    const int t = (int)(blockIdx.x - b * tiles) * TF_ROWS - TF_HALO + tid;
    const bool in = t >= 0 && t < Tw, own = in && tid >= TF_HALO;
    const int64_t row = b * Tw + t;
    T acc[TC];
    {
        T xc[2] = {}, xo[2] = {};
        if (in) {
            xc[0] = (T)u[2 * row];
            xc[1] = (T)u[2 * row + 1];
            if (t >= 1) {
                xo[0] = (T)u[2 * row - 2];
                xo[1] = (T)u[2 * row - 1];
            }
        }
        tiny_conv<T, 2>(blob, xo, xc, t >= 1, acc);
    }
#pragma unroll
    for (int layer = 0; layer < 4; ++layer) {
#pragma unroll
        for (int o = 0; o < TC; ++o) acc[o] = acc[o] > (T)0 ? acc[o] : (T)0;
        if (own) store_row(ys + ((int64_t)layer * M + row) * TC, acc);
        if (layer == 3) break;
        store_row(y[layer & 1][tid], acc);
        __syncthreads();
        const int d = 2 << layer;
        T xo[TC], xc[TC];
        load_row(y[layer & 1][tid >= d ? tid - d : 0], xo);   // (rows left of the halo feed halo rows only)
#pragma unroll
        for (int o = 0; o < TC; ++o) xc[o] = acc[o];
        tiny_conv<T, TC>(blob + tiny_off(layer + 1), xo, xc, t >= d, acc);
    }
    if (own) {
        const T* w = blob + tiny_off(4);
        T s = w[TC];
#pragma unroll
        for (int c = 0; c < TC; ++c) s += w[c] * acc[c];
        z[row] = s;
    }
}

// dL/dwindows of one row, from dL/dpre of conv 0 at the row (dp) and at the next one (only where `tap`).
template <class T>
__device__ inline void tiny_du_row(const T* __restrict__ blob, const T (&dp)[TC], const T* next, bool tap, T* du) {
    T s0 = 0, s1 = 0;
#pragma unroll
    for (int o = 0; o < TC; ++o) {
        s0 += dp[o] * blob[4 * o + 1];
        s1 += dp[o] * blob[4 * o + 3];
        if (tap) {
            s0 += next[o] * blob[4 * o + 0];
            s1 += next[o] * blob[4 * o + 2];
        }
    }
    du[0] = s0;
    du[1] = s1;
}

// dL/dpre of every layer dp [4][M][16] and, if du, dL/dwindows. Block: one tile of TB_ROWS rows of one
// window, thread tid the row t0 + tid, the layers in reverse with dL/dpre of its row in registers and, for
// the taps of the rows to the left, in LDS. ym: rows from one layer of ys to the next (M is that of dp).
// 64 windows of 4096: 295 us (three launches per layer) -> 37 us.
template <class T>
__global__ __launch_bounds__(TN) void tiny_bwd_kernel(const T* __restrict__ blob, const T* __restrict__ ys,
                                                      const T* __restrict__ dz, int64_t M, int64_t ym, int Tw, int tiles,
                                                      T* __restrict__ du, T* __restrict__ dpre) {
    constexpr int LD = tiny_ld<T>();
    __shared__ __attribute__((aligned(16))) T D[2][TN][LD];
    const int tid = threadIdx.x;
    const int64_t b = blockIdx.x / tiles;
    const int t = (int)(blockIdx.x - b * tiles) * TB_ROWS + tid;
    const bool in = t < Tw, own = in && tid < TB_ROWS;
    const int64_t row = b * Tw + t;
    // rows past the window: their loads read the window's last row, their dL/dpre is zero
    const int64_t lrow = in ? row : b * Tw + Tw - 1;
    T y[TC], dp[TC];
    {
        const T g = dz[lrow];
        load_row(ys + ((int64_t)3 * ym + lrow) * TC, y);
        const T* wo = blob + tiny_off(4);
#pragma unroll
        for (int c = 0; c < TC; ++c) {
            const T v = g * wo[c];
            dp[c] = in && y[c] > (T)0 ? v : (T)0;
        }
    }
#pragma unroll
    for (int layer = 3; layer >= 1; --layer) {
        const int d = 1 << layer;
        store_row(D[layer & 1][tid], dp);
        if (own) store_row(dpre + ((int64_t)layer * M + row) * TC, dp);
        load_row(ys + ((int64_t)(layer - 1) * ym + lrow) * TC, y);
        __syncthreads();
        // dL/dy of the layer below, then through its ReLU
        const T* W = blob + tiny_off(layer);
        const bool tap = t + d < Tw;
        T dn[TC];
        load_row(D[layer & 1][tid + d < TN ? tid + d : TN - 1], dn);   // (past the halo: rows nobody uses)
        T s[TC] = {}, w[2 * TC], wn[2 * TC];   // an output's weights are consecutive: wide scalar loads
#pragma unroll
        for (int i = 0; i < 2 * TC; ++i) wn[i] = W[i];
#pragma unroll
        for (int o = 0; o < TC; ++o) {
#pragma unroll
            for (int i = 0; i < 2 * TC; ++i) w[i] = wn[i];
            if (o + 1 < TC) {
#pragma unroll
                for (int i = 0; i < 2 * TC; ++i) wn[i] = W[(o + 1) * 2 * TC + i];
            }
            __builtin_amdgcn_sched_barrier(0);   // one output's weights in flight during the one before
#pragma unroll
            for (int c = 0; c < TC; ++c) {
                s[c] += dp[o] * w[2 * c + 1];
                const T both = s[c] + dn[o] * w[2 * c];
                s[c] = tap ? both : s[c];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int c = 0; c < TC; ++c) dp[c] = in && y[c] > (T)0 ? s[c] : (T)0;
    }
    if (own) store_row(dpre + row * TC, dp);
    if (!du) return;
    store_row(D[0][tid], dp);
    __syncthreads();
    if (own) tiny_du_row(blob, dp, D[0][tid + 1], t + 1 < Tw, du + 2 * row);
}

// dL/dwindows alone, from dL/dpre of conv 0, for a du that shares memory with what the kernels above and below
// read (an in-place gradient): it runs after them.
template <class T>
__global__ __launch_bounds__(TN) void tiny_du_kernel(const T* __restrict__ blob, const T* __restrict__ dpre, int64_t M,
                                                     int Tw, T* __restrict__ du) {
    const int64_t row = (int64_t)blockIdx.x * TN + threadIdx.x;
    if (row >= M) return;
    T dp[TC];
    load_row(dpre + row * TC, dp);
    tiny_du_row(blob, dp, dpre + (row + 1) * TC, row % Tw + 1 < Tw, du + 2 * row);
}

// Weight gradients, first level: part[j][p] = sum over the rows r = j (mod T_RES), in ascending order, of
// parameter p's term: a serial chain over M / 256 rows for each of 256 x 1,681 sums. Block (group, four
// consecutive residues j, one per wave): groups 0-2 the conv layers 1-3, lane (o pair, c pair) of both taps,
// group 3 conv 0 and the output layer. T_STEP steps (64 rows) of each operand go through LDS as one 16-byte
// load per thread, T_DEEP stages ahead: with every lane loading its own operands the vector-memory
// instructions bounded it. more: the rows go on from those of the call before (whole windows, a multiple of
// T_RES rows so far), whose sums are in part. 64 windows of 4096: 2,660 us (one block per parameter walking every row),
// 337 us with a block per residue reading its operands directly, 105 us now; the 200 MB it reads
// take 40 us at the rate of a large copy.
constexpr int T_STEP = 16, T_DEEP = 3;

// Stage `st` of one operand with 16 channels (rows r - back): registers, then LDS [64 rows][16].
template <class T>
struct TinyStage {
    typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
    static constexpr int NV = sizeof(T) / 4;
    vec v[NV];
    __device__ void load(const T* __restrict__ src, int st, int j0, int back, int64_t M, int tid) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int e = (tid + 256 * k) * (16 / (int)sizeof(T)), q = e / TC;
            const int64_t r = (int64_t)T_RES * (st * T_STEP + (q >> 2)) + j0 + (q & 3) - back;
            v[k] = *(const vec*)(src + min(max(r, (int64_t)0), M - 1) * TC + e % TC);   // (rows outside are not added)
        }
    }
    __device__ void store(T* lds, int tid) const {
#pragma unroll
        for (int k = 0; k < NV; ++k) *(vec*)(lds + (tid + 256 * k) * (16 / (int)sizeof(T))) = v[k];
    }
};

template <class T>
__global__ __launch_bounds__(256) void tiny_wgrad_kernel(const float* __restrict__ u, const T* __restrict__ ys,
                                                         const T* __restrict__ dpre, const T* __restrict__ dz, int64_t M,
                                                         int64_t ym, int Tw, int more, T* __restrict__ part) {
    constexpr int SZ = T_STEP * 4 * TC;
    __shared__ __attribute__((aligned(16))) T sd[2][SZ], sx[2][SZ], so[2][SZ];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int group = blockIdx.x & 3, j0 = 4 * (blockIdx.x >> 2), j = j0 + wave;
    T* out = part + (int64_t)j * T_PARAMS;
    const int64_t n = M > j ? (M - j + T_RES - 1) / T_RES : 0;                       // rows of this wave's residue
    const int nst = (int)((M > j0 ? (M - j0 + T_RES - 1) / T_RES : 0) + T_STEP - 1) / T_STEP;   // stages (uniform)
    int t = j % Tw;                                // time step of the row being added
    const int step = T_RES % Tw;
    if (group < 3) {
        const int layer = group + 1, d = 1 << layer, o = 2 * (lane >> 3), c = 2 * (lane & 7);
        const T* D = dpre + (int64_t)layer * M * TC;
        const T* X = ys + (int64_t)(layer - 1) * ym * TC;
        TinyStage<T> pd[T_DEEP], px[T_DEEP], po[T_DEEP];
        auto load = [&](int k, int st) __attribute__((always_inline)) {
            pd[k].load(D, st, j0, 0, M, tid);
            px[k].load(X, st, j0, 0, M, tid);
            po[k].load(X, st, j0, d, M, tid);
        };
        T a[2][2][2] = {}, ab[2] = {};             // [o][c][tap], biases
        T* w = out + tiny_off(layer);
        if (more)
#pragma unroll
            for (int oi = 0; oi < 2; ++oi) {
#pragma unroll
                for (int ci = 0; ci < 2; ++ci)
#pragma unroll
                    for (int tap = 0; tap < 2; ++tap) a[oi][ci][tap] = w[((o + oi) * TC + c + ci) * 2 + tap];
                ab[oi] = w[TC * TC * 2 + o + oi];
            }
#pragma unroll
        for (int k = 0; k < T_DEEP; ++k) load(k, k);
        for (int st0 = 0; st0 < nst; st0 += T_DEEP)
#pragma unroll
            for (int k = 0; k < T_DEEP; ++k) {
                const int st = st0 + k, bf = st & 1;
                if (st >= nst) break;              // uniform over the block
                pd[k].store(sd[bf], tid);
                px[k].store(sx[bf], tid);
                po[k].store(so[bf], tid);
                __syncthreads();                   // (the other buffer is read before its next store's barrier)
                load(k, st + T_DEEP);
                const int rows = (int)min((int64_t)T_STEP, n - (int64_t)st * T_STEP);
                auto add = [&](int i) __attribute__((always_inline)) {
                    const int q = (4 * i + wave) * TC;
                    const T d0 = sd[bf][q + o], d1 = sd[bf][q + o + 1];
                    const T x0 = sx[bf][q + c], x1 = sx[bf][q + c + 1];
                    const T y0 = so[bf][q + c], y1 = so[bf][q + c + 1];
                    const bool tap = t >= d;       // uniform over the wave
                    const T s00 = a[0][0][0] + d0 * y0, s01 = a[0][1][0] + d0 * y1;
                    const T s10 = a[1][0][0] + d1 * y0, s11 = a[1][1][0] + d1 * y1;
                    a[0][0][0] = tap ? s00 : a[0][0][0];
                    a[0][1][0] = tap ? s01 : a[0][1][0];
                    a[1][0][0] = tap ? s10 : a[1][0][0];
                    a[1][1][0] = tap ? s11 : a[1][1][0];
                    a[0][0][1] += d0 * x0;
                    a[0][1][1] += d0 * x1;
                    a[1][0][1] += d1 * x0;
                    a[1][1][1] += d1 * x1;
                    ab[0] += d0;
                    ab[1] += d1;
                    t += step;
                    t -= t >= Tw ? Tw : 0;
                };
                if (rows == T_STEP) {              // whole stages unrolled: later rows' LDS reads overlap the sums
#pragma unroll
                    for (int i = 0; i < T_STEP; ++i) add(i);
                } else {
                    for (int i = 0; i < rows; ++i) add(i);
                }
            }
#pragma unroll
        for (int oi = 0; oi < 2; ++oi) {
#pragma unroll
            for (int ci = 0; ci < 2; ++ci)
#pragma unroll
                for (int tap = 0; tap < 2; ++tap) w[((o + oi) * TC + c + ci) * 2 + tap] = a[oi][ci][tap];
            if (c == 0) w[TC * TC * 2 + o + oi] = ab[oi];
        }
        return;
    }
    // conv 0: lane (o, c, tap) a weight; the output layer and the biases: lanes 0-15 conv 0's biases,
    // 16-31 the output weights, 32 their bias. so: [64 rows] dz, u(t) and u(t - 1).
    TinyStage<T> pd[T_DEEP], py[T_DEEP];
    T pz[T_DEEP][5];
    auto load = [&](int k, int st) __attribute__((always_inline)) {
        pd[k].load(dpre, st, j0, 0, M, tid);
        py[k].load(ys + 3 * ym * TC, st, j0, 0, M, tid);
        const int64_t r = min((int64_t)T_RES * (st * T_STEP + (lane >> 2)) + j0 + (lane & 3), M - 1);
        const int64_t rp = max(r - 1, (int64_t)0);
        pz[k][0] = dz[r];
        pz[k][1] = (T)u[2 * r];
        pz[k][2] = (T)u[2 * r + 1];
        pz[k][3] = (T)u[2 * rp];
        pz[k][4] = (T)u[2 * rp + 1];
    };
    const int o = lane >> 2, c = (lane >> 1) & 1, tap = lane & 1;
    T a0 = 0, a1 = 0;
    T* w1 = lane < 16 ? out + 64 + lane : out + tiny_off(4) + min(lane, 32) - 16;
    if (more) {
        a0 = out[lane];
        a1 = *w1;
    }
#pragma unroll
    for (int k = 0; k < T_DEEP; ++k) load(k, k);
    for (int st0 = 0; st0 < nst; st0 += T_DEEP)
#pragma unroll
        for (int k = 0; k < T_DEEP; ++k) {
            const int st = st0 + k, bf = st & 1;
            if (st >= nst) break;
            pd[k].store(sd[bf], tid);
            py[k].store(sx[bf], tid);
            if (tid < 64)
#pragma unroll
                for (int e = 0; e < 5; ++e) so[bf][8 * tid + e] = pz[k][e];
            __syncthreads();
            load(k, st + T_DEEP);
            const int rows = (int)min((int64_t)T_STEP, n - (int64_t)st * T_STEP);
            auto add = [&](int i) __attribute__((always_inline)) {
                const int q = 4 * i + wave;
                const T z = so[bf][8 * q];
                const T dv = sd[bf][q * TC + o], xv = so[bf][8 * q + (tap ? 1 : 3) + c];
                const T s0 = a0 + dv * xv;
                a0 = tap || t >= 1 ? s0 : a0;
                // one multiply-add for all three sums (a product with 1 is exact)
                const T p0 = lane < 16 ? sd[bf][q * TC + (lane & 15)] : z;
                const T p1 = lane >= 16 && lane < 32 ? sx[bf][q * TC + (lane & 15)] : (T)1;
                a1 += p0 * p1;
                t += step;
                t -= t >= Tw ? Tw : 0;
            };
            if (rows == T_STEP) {
#pragma unroll
                for (int i = 0; i < T_STEP; ++i) add(i);
            } else {
                for (int i = 0; i < rows; ++i) add(i);
            }
        }
    out[lane] = a0;
    if (lane < 33) *w1 = a1;
}

// grad[p] = the residues' sums added pairwise (j + 128, + 64, .. + 1).
template <class T>
__global__ __launch_bounds__(256) void tiny_reduce_kernel(const T* __restrict__ part, T* __restrict__ grad) {
    __shared__ T red[16][16];
    const int p = threadIdx.x & 15, run = threadIdx.x >> 4, i = blockIdx.x * 16 + p;
    T v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = i < T_PARAMS ? part[(int64_t)(run + 16 * k) * T_PARAMS + i] : (T)0;
#pragma unroll
    for (int w = 8; w > 0; w >>= 1)
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (k < w) v[k] += v[k + w];
    red[run][p] = v[0];
    for (int w = 8; w > 0; w >>= 1) {
        __syncthreads();
        if (run < w) red[run][p] += red[run + w][p];
    }
    if (run == 0 && i < T_PARAMS) grad[i] = red[0][p];
}

// dL/dpre of `windows` windows at a time, then the partial sums.
int64_t tiny_train_backward_scratch(int windows, int Tw) { return 4 * (int64_t)windows * Tw * TC + T_RES * T_PARAMS; }

// Windows at a time where device memory does not hold the scratch of all B: about a quarter, and a multiple of
// T_RES rows, so that the sums keep their order (B: no such number).
int tiny_train_windows(int B, int Tw) {
    int unit = T_RES;   // windows of a multiple of T_RES rows
    while (unit > 1 && (int64_t)(unit / 2) * Tw % T_RES == 0) unit /= 2;
    const int w = (B / 4 + unit - 1) / unit * unit;
    return w < 1 || w > B ? B : w;
}

template <class T>
hipError_t tiny_train_forward(const T* blob, const float* u, int B, int Tw, T* ys, T* logits, hipStream_t st) {
    const int tiles = (Tw + TF_ROWS - 1) / TF_ROWS;
    hipLaunchKernelGGL(tiny_fwd_kernel<T>, dim3((unsigned)((int64_t)B * tiles)), dim3(TN), 0, st, blob, u,
                       (int64_t)B * Tw, Tw, tiles, ys, logits);
    return hipGetLastError();
}

template <class T>
hipError_t tiny_train_backward(const T* blob, const float* u, int B, int windows, int Tw, const T* ys, const T* dz, T* grad,
                               T* scratch, T* du, hipStream_t st) {
    const int64_t M = (int64_t)B * Tw;
    const int tiles = (Tw + TB_ROWS - 1) / TB_ROWS;
    T* part = scratch + 4 * (int64_t)windows * Tw * TC;
    const auto meets = [&](const void* p, int64_t bytes) {
        const uintptr_t a = (uintptr_t)du, b = (uintptr_t)p;
        return du && a < b + (uint64_t)bytes && b < a + (uint64_t)(2 * M * (int64_t)sizeof(T));
    };
    const bool last = meets(u, 2 * M * 4) || meets(dz, M * (int64_t)sizeof(T)) || meets(ys, 4 * M * TC * (int64_t)sizeof(T));
    if (last && windows < B) return hipErrorOutOfMemory;   // (it needs every window's dL/dpre at the end)
    for (int b0 = 0; b0 < B; b0 += windows) {
        const int nb = B - b0 < windows ? B - b0 : windows;
        const int64_t r0 = (int64_t)b0 * Tw, m = (int64_t)nb * Tw;
        hipLaunchKernelGGL(tiny_bwd_kernel<T>, dim3((unsigned)((int64_t)nb * tiles)), dim3(TN), 0, st, blob, ys + r0 * TC,
                           dz + r0, m, M, Tw, tiles, last || !du ? nullptr : du + 2 * r0, scratch);
        hipLaunchKernelGGL(tiny_wgrad_kernel<T>, dim3(T_RES), dim3(256), 0, st, u + 2 * r0, ys + r0 * TC, (const T*)scratch,
                           dz + r0, m, M, Tw, b0 > 0 ? 1 : 0, part);
    }
    hipLaunchKernelGGL(tiny_reduce_kernel<T>, dim3((T_PARAMS + 15) / 16), dim3(256), 0, st, (const T*)part, grad);
    if (last)
        hipLaunchKernelGGL(tiny_du_kernel<T>, dim3((unsigned)((M + TN - 1) / TN)), dim3(TN), 0, st, blob, (const T*)scratch,
                           M, Tw, du);
    return hipGetLastError();
}

template hipError_t tiny_train_forward<float>(const float*, const float*, int, int, float*, float*, hipStream_t);
template hipError_t tiny_train_forward<double>(const double*, const float*, int, int, double*, double*, hipStream_t);
template hipError_t tiny_train_backward<float>(const float*, const float*, int, int, int, const float*, const float*,
                                               float*, float*, float*, hipStream_t);
template hipError_t tiny_train_backward<double>(const double*, const float*, int, int, int, const double*, const double*,
                                                double*, double*, double*, hipStream_t);

}  // namespace gwd
