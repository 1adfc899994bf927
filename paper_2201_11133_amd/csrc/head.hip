// Head, stitching and ensemble minimum; and the complete forward pass of the small plain member.
//
// Head of the gated member: logit = w_h2 . act(W_h1 ReLU(skip) + b_h1) + b_h2 per time step
// ("AI architecture": the network ends in convolutional layers that give one classification
// output per time step). Only the rows a window owns are computed in the stitched output modes.
// The ensemble score is the running minimum over members (Results, "Event Detection": a sample
// counts only if every member flags it).
#include "gwd_internal.h"
#include "head_common.h"
#include "layer_common.h"

namespace gwd {

__global__ __launch_bounds__(256) void head_kernel(HeadArgs p) {
    __shared__ __attribute__((aligned(16))) float sk[kBM * kHS];
    __shared__ float part[4][kBM];
    const int b = blockIdx.x / p.tiles;
    const int t0 = (p.tile_first + blockIdx.x - b * p.tiles) * kBM;
    const int64_t gw = p.wins ? p.wins[b] : p.win_base + b;
    const StreamDesc sd = p.streams[find_stream(p.streams, p.n_streams, gw)];
    const int64_t k = gw - sd.win_begin;
    int lo, hi;
    owner_rows(p.o, k, sd.length, lo, hi);
    if (t0 + kBM <= lo || t0 >= hi) return;  // uniform over the block
    // the launch's members in order: the thread that writes a sample's score takes the running minimum
    for (int mem = 0; mem < p.n_mem; ++mem) {
        if (mem > 0) __syncthreads();   // the LDS of the member before is read
        head_tile(p, sd, gw, k, t0, lo, hi, p.skip + mem * p.act_stride + (gw - p.win_base) * p.o.T * kC, sk, part, mem);
    }
}

hipError_t wavenet_layers_f32(gwd_model* m, const FwdBatch& fb, float* x_a, float* x_b, float* skip,
                              hipStream_t st);
hipError_t wavenet_layers_bf16(gwd_model* m, const FwdBatch& fb, float* x_a, float* x_b, float* skip,
                               hipStream_t st);
hipError_t wavenet_layers_fp8(gwd_model* m, const FwdBatch& fb, float* x_a, float* x_b, float* skip,
                              hipStream_t st);

static OutDesc out_desc(const FwdBatch& fb) {
    OutDesc o;
    o.out_mode = fb.out_mode;
    o.member = fb.member;
    o.T = fb.T;
    o.S = fb.S;
    o.out = fb.out;
    o.sum_L = fb.sum_L;
    o.total_win = fb.total_win;
    return o;
}

hipError_t launch_wavenet_forward(gwd_model* m, const FwdBatch& fb, float* x_a, float* x_b, float* skip,
                                  hipStream_t st) {
    hipError_t e;
    switch (m->prec) {
        case GWD_FP32: e = wavenet_layers_f32(m, fb, x_a, x_b, skip, st); break;
        case GWD_BF16: e = wavenet_layers_bf16(m, fb, x_a, x_b, skip, st); break;
        default: e = wavenet_layers_fp8(m, fb, x_a, x_b, skip, st); break;
    }
    if (e != hipSuccess) return e;
    const MemberWeights& mw = m->members[fb.member];
    const float* base = (const float*)mw.base;
    HeadArgs h{};
    h.skip = skip;
    h.n_mem = fb.n_group;
    h.act_stride = fb.act_stride;
    for (int i = 0; i < fb.n_group; ++i) h.mem_off[i] = (const char*)m->members[fb.member + i].base - (const char*)mw.base;
    h.h1w = base + mw.h1w;
    h.h1b = base + mw.h1b;
    h.h2w = base + mw.h2w;
    h.h2b = base + mw.h2b;
    h.mid_relu = m->arch.head_mid_relu;
    h.streams = fb.streams;
    h.n_streams = fb.n_streams;
    h.win_base = fb.win_base;
    h.o = out_desc(fb);
    h.wins = nullptr;
    const int tpw = fb.T / kBM;
    if (fb.out_mode == 2) {  // every row of every window
        h.tile_first = 0;
        h.tiles = tpw;
        hipLaunchKernelGGL(head_kernel, dim3(fb.nb * tpw), dim3(256), 0, st, h);
        return hipGetLastError();
    }
    // the tail rows [T - S, T) of every window, then the head rows of the windows that start a stream
    h.tile_first = (fb.T - fb.S) / kBM;
    h.tiles = tpw - h.tile_first;
    hipLaunchKernelGGL(head_kernel, dim3(fb.nb * h.tiles), dim3(256), 0, st, h);
    if (fb.n_first > 0 && h.tile_first > 0) {
        h.wins = fb.firsts + fb.first_idx;
        h.tiles = h.tile_first;
        h.tile_first = 0;
        hipLaunchKernelGGL(head_kernel, dim3(fb.n_first * h.tiles), dim3(256), 0, st, h);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- small plain member (kind 0)
// Four causal convolutions 2 -> 16 -> 16 -> 16 -> 16 (kernel 2, dilations 1, 2, 4, 8, ReLU), then a
// 1x1 to one logit, all in one kernel: one time step per thread, its 16 channels in registers through
// all layers. LDS holds the rows only for the taps at t - d, and the weights, the same for every lane,
// are scalar operands (read from LDS by each lane for each output, they bounded the kernel). A tile is
// TINY_ROWS output rows of one window and the TINY_HALO rows left of them that the later layers need.
// 64 windows of 4096 in FP32: 123 us (16 outputs of a row on 16 threads) -> 26 us.
constexpr int TINY_N = 256;
constexpr int TINY_HALO = 14;
constexpr int TINY_ROWS = TINY_N - TINY_HALO;
constexpr int TINY_C = 16;
constexpr int TINY_LD = TINY_C + 4;   // padded LDS row: 16-byte accesses of consecutive rows spread over the banks

struct TinyArgs {
    const StreamDesc* streams;
    int n_streams;
    int64_t win_base;
    int tiles_per_window;
    OutDesc o;
};

// Operand rounding of the reduced-precision forms: P = 0 fp32 (none), 1 bf16 (nearest even),
// 2 E4M3 (nearest even, saturated at +/-448; NaN stays NaN).
template <int P>
__device__ inline float tiny_round(float v) {
    if constexpr (P == 1) return (float)(__bf16)v;
    if constexpr (P == 2) {
        v = fabsf(v) > 448.f ? copysignf(448.f, v) : v;
        return __builtin_amdgcn_cvt_f32_fp8((int)__builtin_amdgcn_cvt_pk_fp8_f32(v, v, 0, false), 0);
    }
    return v;
}

// One convolution of one row: acc[o] from xc (row t) and xo (row t - d, zero before the window), channel
// by channel, then ReLU and the operand rounding; zero for rows before the window.
template <int P, int CIN>
__device__ inline void tiny_conv(const float* __restrict__ W, const float* __restrict__ sc, const float (&xo)[CIN],
                                 const float (&xc)[CIN], bool in, float (&acc)[TINY_C]) {
    const float* B = W + TINY_C * CIN * 2;
#pragma unroll
    for (int o = 0; o < TINY_C; ++o) {   // (an output's weights are consecutive: wide scalar loads)
        float s = P == 2 ? 0.f : B[o];
#pragma unroll
        for (int c = 0; c < CIN; ++c) {
            s = fmaf(W[(o * CIN + c) * 2 + 0], xo[c], s);
            s = fmaf(W[(o * CIN + c) * 2 + 1], xc[c], s);
        }
        if (P == 2) s = fmaf(s, sc[o], B[o]);
        acc[o] = in ? tiny_round<P>(fmaxf(s, 0.f)) : 0.f;
    }
}

// P as above. BF16: operands rounded to bf16, products exact in fp32 and accumulated in fp32 from
// the bias (the arithmetic of the bf16 matrix instruction). FP8: E4M3 operands (weights as codes,
// activations with unit scale), fp32 accumulation, then the channel scale and the bias. Each layer's
// output is stored in the operand format; the logit stays fp32.
// W: the packed blob (1,681 floats, operand values), then kTinyScales channel scales.
template <int P>
__global__ __launch_bounds__(TINY_N) void tiny_forward_kernel(TinyArgs p, const float* __restrict__ W) {
    __shared__ __attribute__((aligned(16))) float y[2][TINY_N][TINY_LD];
    const int tid = threadIdx.x;
    const int b = blockIdx.x / p.tiles_per_window;
    const int64_t gw = p.win_base + b;
    const StreamDesc sd = p.streams[find_stream(p.streams, p.n_streams, gw)];
    const int64_t k = gw - sd.win_begin;
    int lo, hi;
    owner_rows(p.o, k, sd.length, lo, hi);
    const int t0 = lo + (blockIdx.x - b * p.tiles_per_window) * TINY_ROWS;   // the tile's first output row
    if (t0 >= hi) return;  // uniform over the block
    const float* sc = W + 1681;
    const int t = t0 - TINY_HALO + tid;
    const bool in = t >= 0;
    const int64_t smp = k * (int64_t)p.o.S + t;   // sample of row t
    float acc[TINY_C];
    {
        float xc[2] = {0.f, 0.f}, xo[2] = {0.f, 0.f};
        if (in && smp < sd.length) {
            xc[0] = tiny_round<P>(sd.ch0[smp * sd.stride]);
            xc[1] = tiny_round<P>(sd.ch1[smp * sd.stride]);
        }
        if (t >= 1 && smp - 1 < sd.length) {
            xo[0] = tiny_round<P>(sd.ch0[(smp - 1) * sd.stride]);
            xo[1] = tiny_round<P>(sd.ch1[(smp - 1) * sd.stride]);
        }
        tiny_conv<P, 2>(W, sc, xo, xc, in, acc);
    }
    // blob offsets: conv0 W[16][2][2] b[16] (80), conv1..3 W[16][16][2] b[16] (528 each), out W[16] b[1]
#pragma unroll
    for (int layer = 1; layer < 4; ++layer) {
        const int d = 1 << layer;
        float(*yb)[TINY_LD] = y[layer & 1];
#pragma unroll
        for (int o = 0; o < TINY_C; o += 4) *(float4*)&yb[tid][o] = make_float4(acc[o], acc[o + 1], acc[o + 2], acc[o + 3]);
        __syncthreads();
        float xo[TINY_C], xc[TINY_C];
#pragma unroll
        for (int o = 0; o < TINY_C; ++o) {
            xc[o] = acc[o];
            xo[o] = yb[tid >= d ? tid - d : 0][o];   // rows left of the halo feed halo rows only; rows before the window are zero
        }
        int zl = 0;
        asm volatile("" : "+s"(zl));   // (keeps the layer's scalar weight loads behind the layers before it)
        tiny_conv<P, TINY_C>(W + zl + 80 + 528 * (layer - 1), sc + zl + 16 * layer, xo, xc, in, acc);
    }
    if (tid < TINY_HALO || t >= hi) return;
    const float* Wo = W + 80 + 3 * 528;
    float z = 0.f;
#pragma unroll
    for (int c = 0; c < TINY_C; ++c) z = fmaf(Wo[c], acc[c], z);
    z = P == 2 ? fmaf(z, sc[tiny_scale_index(4, 0)], Wo[TINY_C]) : z + Wo[TINY_C];
    emit_logit(p.o, sd, gw, k, t, z);
}

hipError_t launch_tiny_forward(const gwd_model* m, const FwdBatch& fb, hipStream_t st) {
    TinyArgs a;
    const float* blob = (const float*)m->members[fb.member].base + m->members[fb.member].blob;
    a.streams = fb.streams;
    a.n_streams = fb.n_streams;
    a.win_base = fb.win_base;
    // the rows a window owns: all of its stream's first window (and every window in mode 2)
    a.tiles_per_window = (fb.T + TINY_ROWS - 1) / TINY_ROWS;
    a.o = out_desc(fb);
    const dim3 grid(fb.nb * a.tiles_per_window);
    if (m->prec == GWD_BF16) hipLaunchKernelGGL(tiny_forward_kernel<1>, grid, dim3(TINY_N), 0, st, a, blob);
    else if (m->prec == GWD_FP8_E4M3) hipLaunchKernelGGL(tiny_forward_kernel<2>, grid, dim3(TINY_N), 0, st, a, blob);
    else hipLaunchKernelGGL(tiny_forward_kernel<0>, grid, dim3(TINY_N), 0, st, a, blob);
    return hipGetLastError();
}

}  // namespace gwd

namespace gwd {
hipError_t layer_debug_f32(gwd_model* m, int member, int l, const float* x_in, int nb, int T, float* pre_out,
                           float* x_out, float* skip, hipStream_t st);
hipError_t layer_debug_bf16(gwd_model* m, int member, int l, const float* x_in, int nb, int T, float* pre_out,
                            float* x_out, float* skip, hipStream_t st);
hipError_t layer_debug_fp8(gwd_model* m, int member, int l, const float* x_in, int nb, int T, float* pre_out,
                           float* x_out, float* skip, hipStream_t st);

// Device completion stamp: the 64-bit wall clock (constant rate) when the stream reaches this point.
__global__ void stamp_kernel(unsigned long long* slot) {
    if (threadIdx.x == 0) *slot = wall_clock64();
}
hipError_t launch_stamp(unsigned long long* slot, hipStream_t st) {
    hipLaunchKernelGGL(stamp_kernel, dim3(1), dim3(64), 0, st, slot);
    return hipGetLastError();
}

hipError_t layer_production_f32(gwd_model*, int, void*, void*, float*, const FwdBatch&, hipStream_t);
hipError_t layer_production_bf16(gwd_model*, int, void*, void*, float*, const FwdBatch&, hipStream_t);
hipError_t layer_production_fp8(gwd_model*, int, void*, void*, float*, const FwdBatch&, hipStream_t);

hipError_t launch_layer_production(gwd_model* m, int layer, void* x_in, void* x_out, float* skip, const FwdBatch& fb,
                                   hipStream_t st) {
    switch (m->prec) {
        case GWD_FP32: return layer_production_f32(m, layer, x_in, x_out, skip, fb, st);
        case GWD_BF16: return layer_production_bf16(m, layer, x_in, x_out, skip, fb, st);
        default: return layer_production_fp8(m, layer, x_in, x_out, skip, fb, st);
    }
}

int layers_per_launch_lp(const gwd_model* m, int l);
int layers_per_launch(const gwd_model* m, int l) {
    return (m->prec == GWD_BF16 || m->prec == GWD_FP8_E4M3) ? layers_per_launch_lp(m, l) : 1;
}

hipError_t launch_layer_debug(gwd_model* m, int member, int layer, const float* x_in, int nb, int T, float* pre_out,
                              float* x_out, float* skip, hipStream_t st) {
    switch (m->prec) {
        case GWD_FP32: return layer_debug_f32(m, member, layer, x_in, nb, T, pre_out, x_out, skip, st);
        case GWD_BF16: return layer_debug_bf16(m, member, layer, x_in, nb, T, pre_out, x_out, skip, st);
        default: return layer_debug_fp8(m, member, layer, x_in, nb, T, pre_out, x_out, skip, st);
    }
}
}  // namespace gwd
