// Training kernels: generic FP32 MFMA GEMMs with row-shifted operands, reductions, elementwise
// backward steps, Adam. ("AI ensemble construction": each member is trained as a per-timestep
// classifier from random initialisation.)
//
// Row index `row` = b * T + t addresses time step t of window b; an operand part with shift s reads
// row b * T + (t + s) and is zero when t + s falls outside [0, T) (each window has zero context, so
// a dilation tap never crosses windows).
#include <algorithm>

#include "gwd_internal.h"
#include "train_internal.h"

namespace gwd {

typedef float floatx16 __attribute__((ext_vector_type(16)));
#define MFMA32(a, b, c) __builtin_amdgcn_mfma_f32_32x32x2f32((a), (b), (c), 0, 0, 0)

// ---- row GEMM: C[M, N] = beta * C + sum_p A_p[M, K_p] B_p[K_p, N] (optionally masked: C *= (mask > 0)), in
// two forms. With bf16 operands (fp32 accumulation), for BF16/FP8 models: B is packed
// once per call into bt in MFMA fragment order (parts stacked along k), so a wave's B fragment is one
// 1 KB load from L2; A rows are read from HBM once per 128 x 128 output tile and rounded to bf16 as
// they are staged.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx8 __attribute__((ext_vector_type(8)));
constexpr int BN = 128;       // columns per block
constexpr int BK = 64;        // k per staged chunk
constexpr int AROW = BK + 8;  // bf16 per LDS row (144 B: conflict-free 16-byte fragment reads)

// Gate backward of one (row, channel c): from the pre-activations (filter pf, gate pg) and dg, the
// gate output g = tanh(pf) sigma(pg) and dpre for both halves, in bf16 (the dg GEMM's epilogue).
__device__ inline void gate_bwd_one(float pf, float pg, float d, uint16_t& g, uint16_t& df, uint16_t& dgt) {
    const float th = tanhf(pf), sg = 1.f / (1.f + expf(-pg));
    g = __builtin_bit_cast(uint16_t, (__bf16)(th * sg));
    df = __builtin_bit_cast(uint16_t, (__bf16)(d * sg * (1.f - th * th)));
    dgt = __builtin_bit_cast(uint16_t, (__bf16)(d * th * sg * (1.f - sg)));
}

// The same in fp32.
__device__ inline void gate_bwd_f32(float pf, float pg, float d, float& g, float& df, float& dgt) {
    const float th = tanhf(pf), sg = 1.f / (1.f + expf(-pg));
    g = th * sg;
    df = d * sg * (1.f - th * th);
    dgt = d * th * sg * (1.f - sg);
}

// bt in MFMA fragment order: the 16-byte fragment of lane (h, r) for column tile nt (32 columns) and
// k step ks (16 k) sits at fragment index (nt Ktot / 16 + ks) 64 + 32 h + r and holds B(k, 32 nt + r)
// for k = 16 ks + 8 h .. + 8, so a wave's fragment load is 1 KB of consecutive bytes.
__global__ __launch_bounds__(256) void pack_bt_kernel(GemmRowsArgs a, int Ktot) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;  // i = n Ktot + k
    if (i >= (int64_t)a.N * Ktot) return;
    const int n = (int)(i / Ktot);
    const int kk = (int)(i - (int64_t)n * Ktot);
    int k = kk, p = 0;
    while (p + 1 < a.nparts && k >= a.A[p].K) {
        k -= a.A[p].K;
        ++p;
    }
    const BPart& bp = a.B[p];
    const int64_t f = ((int64_t)(n >> 5) * (Ktot >> 4) + (kk >> 4)) * 64 + ((kk >> 3) & 1) * 32 + (n & 31);
    a.bt[f * 8 + (kk & 7)] = __builtin_bit_cast(uint16_t, (__bf16)bp.ptr[(int64_t)k * bp.ld + (int64_t)n * bp.es]);
}

__device__ inline uint4 bf16_pack8(float4 lo, float4 hi) {
    const floatx8 f = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    return __builtin_bit_cast(uint4, __builtin_convertvector(f, bf16x8));
}
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// four fp32 (as raw bits) -> four bf16, rounded to nearest even
__device__ inline u32x2 bf16_pack4(u32x4 v) {
    return __builtin_bit_cast(u32x2, __builtin_convertvector(__builtin_bit_cast(floatx4, v), bf16x4));
}

constexpr int EP = BN + 4;     // floats per row of the epilogue's LDS stage

// The row GEMMs' epilogue: the block's 64 RB x 128 tile (wave (wr, wc): rows 32 RB wr .. + 32 RB, columns
// 64 wc .. + 64) staged through LDS 64 rows at a time; each thread then takes 4 consecutive columns (cq) of 8 rows, all
// its loads (C for beta, the mask, or the gate's pre-activations) issued before the first store.
template <int RB>
__device__ __forceinline__ void rows_epilogue(const GemmRowsArgs& a, const floatx16 (&acc)[RB][2], float* Ep, int64_t row0,
                                              int col0) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = wave & 1, wc = wave >> 1, r = lane & 31, h = lane >> 5;
    const int cq = 4 * (tid & 31);
    const int n4 = col0 + cq;
    for (int pass = 0; pass < RB; ++pass) {
        __syncthreads();  // the products' (or the previous pass's) LDS reads are done
        if (RB == 1 || wr == pass) {
#pragma unroll
            for (int i = 0; i < RB; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        Ep[(32 * (RB == 1 ? wr : i) + 8 * (e >> 2) + 4 * h + (e & 3)) * EP + 64 * wc + 32 * c + r] = acc[i][c][e];
        }
        __syncthreads();
        const int64_t rbase = row0 + 64 * pass + (tid >> 5);   // + 8 it
        if (a.gpre) {
            // gate backward (N = 128, one column block): g, dpre from the bf16 pre-activations and dg
            u32x2 pf[8], pg[8];
#pragma unroll
            for (int it = 0; it < 8; ++it) {
                const int64_t row = rbase + 8 * it;
                pf[it] = *(const u32x2*)(a.gpre + row * 2 * kC + cq);
                pg[it] = *(const u32x2*)(a.gpre + row * 2 * kC + kC + cq);
            }
#pragma unroll
            for (int it = 0; it < 8; ++it) {
                const int64_t row = rbase + 8 * it;
                const float4 d = *(const float4*)&Ep[(8 * it + (tid >> 5)) * EP + cq];
                const float fv[4] = {__uint_as_float(pf[it][0] << 16), __uint_as_float(pf[it][0] & 0xffff0000u),
                                     __uint_as_float(pf[it][1] << 16), __uint_as_float(pf[it][1] & 0xffff0000u)};
                const float gv[4] = {__uint_as_float(pg[it][0] << 16), __uint_as_float(pg[it][0] & 0xffff0000u),
                                     __uint_as_float(pg[it][1] << 16), __uint_as_float(pg[it][1] & 0xffff0000u)};
                const float dv[4] = {d.x, d.y, d.z, d.w};
                uint16_t go[4], fo[4], so[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) gate_bwd_one(fv[j], gv[j], dv[j], go[j], fo[j], so[j]);
                *(uint2*)(a.g16 + row * kC + cq) = make_uint2(go[0] | ((uint32_t)go[1] << 16), go[2] | ((uint32_t)go[3] << 16));
                *(uint2*)(a.dpre16 + row * 2 * kC + cq) =
                    make_uint2(fo[0] | ((uint32_t)fo[1] << 16), fo[2] | ((uint32_t)fo[3] << 16));
                *(uint2*)(a.dpre16 + row * 2 * kC + kC + cq) =
                    make_uint2(so[0] | ((uint32_t)so[1] << 16), so[2] | ((uint32_t)so[3] << 16));
                if (a.C) *(float4*)(a.C + row * a.ldc + cq) = d;
            }
            continue;
        }
        if (a.gpre32) {
            // the same in fp32
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float4 pf[4], pg[4];
#pragma unroll
                for (int it = 0; it < 4; ++it) {
                    const int64_t row = rbase + 8 * (4 * q + it);
                    pf[it] = *(const float4*)(a.gpre32 + row * 2 * kC + cq);
                    pg[it] = *(const float4*)(a.gpre32 + row * 2 * kC + kC + cq);
                }
#pragma unroll
                for (int it = 0; it < 4; ++it) {
                    const int64_t row = rbase + 8 * (4 * q + it);
                    const float4 d = *(const float4*)&Ep[(8 * (4 * q + it) + (tid >> 5)) * EP + cq];
                    const float fv[4] = {pf[it].x, pf[it].y, pf[it].z, pf[it].w}, gv[4] = {pg[it].x, pg[it].y, pg[it].z, pg[it].w};
                    const float dv[4] = {d.x, d.y, d.z, d.w};
                    float go[4], fo[4], so[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) gate_bwd_f32(fv[j], gv[j], dv[j], go[j], fo[j], so[j]);
                    *(float4*)(a.g32 + row * kC + cq) = make_float4(go[0], go[1], go[2], go[3]);
                    *(float4*)(a.dpre32 + row * 2 * kC + cq) = make_float4(fo[0], fo[1], fo[2], fo[3]);
                    *(float4*)(a.dpre32 + row * 2 * kC + kC + cq) = make_float4(so[0], so[1], so[2], so[3]);
                    if (a.C) *(float4*)(a.C + row * a.ldc + cq) = d;
                }
            }
            continue;
        }
        float4 cv[8], mv[8];
        if (a.beta != 0.f) {
#pragma unroll
            for (int it = 0; it < 8; ++it) cv[it] = *(const float4*)(a.C + (rbase + 8 * it) * a.ldc + n4);
        }
        if (a.mask) {
#pragma unroll
            for (int it = 0; it < 8; ++it) mv[it] = *(const float4*)(a.mask + (rbase + 8 * it) * a.ldm + n4);
        }
        const float4 bv = a.bias ? *(const float4*)(a.bias + n4) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            const float4 d = *(const float4*)&Ep[(8 * it + (tid >> 5)) * EP + cq];
            float v[4] = {d.x, d.y, d.z, d.w};
            const float b4[4] = {bv.x, bv.y, bv.z, bv.w};
            const float c4[4] = {cv[it].x, cv[it].y, cv[it].z, cv[it].w};
            const float m4[4] = {mv[it].x, mv[it].y, mv[it].z, mv[it].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (a.bias) v[j] += b4[j];
                if (a.beta != 0.f) v[j] += a.beta * c4[j];
                if (a.mask) v[j] = (m4[j] > 0.f) ? v[j] : 0.f;
            }
            *(float4*)(a.C + (rbase + 8 * it) * a.ldc + n4) = make_float4(v[0], v[1], v[2], v[3]);
            if (a.c16)
                *(u32x2*)(a.c16 + (rbase + 8 * it) * a.ldc + n4) =
                    bf16_pack4(u32x4{__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])});
        }
    }
}

// One block: 128 rows x 128 columns; wave (wr, wc) owns rows 64 wr .. + 64 (two row blocks) and columns
// 64 wc .. + 64 (two column tiles), so each B fragment feeds two products and each A fragment two.
// The next chunk's A rows are requested before the current chunk's products, and the chunk's B
// fragments before its staging barrier. Products per output in k order (part by part, chunk by
// chunk, 16-k steps ascending).
constexpr int BR2 = 128;      // rows per block

__device__ inline void rows_chunk(const GemmRowsArgs& a, int ci, int& p, int& k0) {
    const int n0 = a.A[0].K / BK;
    p = ci < n0 ? 0 : 1;
    k0 = BK * (ci < n0 ? ci : ci - n0);
}

constexpr int ROWS_LDS = (64 * EP * 4 > BR2 * AROW * 2) ? 64 * EP * 4 : BR2 * AROW * 2;

__global__ __launch_bounds__(256) void gemm_rows_bf16_kernel(GemmRowsArgs a, int Ktot) {
    __shared__ __attribute__((aligned(16))) uint8_t smem[ROWS_LDS];
    uint16_t* As = (uint16_t*)smem;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = wave & 1, wc = wave >> 1;
    const int r = lane & 31, h = lane >> 5;
    const int ntn = a.N / BN;
    const int64_t row0 = (int64_t)(blockIdx.x / ntn) * BR2;
    const int col0 = (blockIdx.x % ntn) * BN;
    // staging of one chunk (64 k) of the block's 128 rows: thread tid stages block rows tid / 8 + 32 i
    // (i < 4), 16 bytes at column group tid % 8 of every 128 bytes of the row, so each load instruction
    // covers whole 128-byte lines (bf16 parts one load per row, fp32 parts two). tw[i]: the row's time
    // step in its window, for the shifted parts' zero rows.
    const int64_t b0 = row0 / a.T;
    const int t0 = (int)(row0 - b0 * a.T);
    const int sr = tid >> 3, sc = tid & 7;
    int tw[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int t = t0 + sr + 32 * i;
        while (t >= a.T) t -= a.T;
        tw[i] = t;
    }
    const int nch = Ktot / BK;
    // rows whose shifted source leaves the window read the (valid) unshifted row and are set to zero
    // as they are staged (masking at the load would let the compiler turn it into a conditional load)
    auto row_ok = [&](int sh, int i) { return (unsigned)(tw[i] + sh) < (unsigned)a.T; };
    auto load_raw = [&](int ci, u32x4 (&raw)[8]) __attribute__((always_inline)) {
        int p, k0;
        rows_chunk(a, ci, p, k0);
        const APart& ap = a.A[p];
        const int sh = ap.shift;
        if (ap.p16) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t row = row0 + sr + 32 * i + (row_ok(sh, i) ? sh : 0);
                raw[2 * i] = *(const u32x4*)(ap.p16 + row * ap.ld + k0 + 8 * sc);
                raw[2 * i + 1] = u32x4{0, 0, 0, 0};  // (both paths write raw[0..7] in one order)
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t row = row0 + sr + 32 * i + (row_ok(sh, i) ? sh : 0);
#pragma unroll
                for (int j = 0; j < 2; ++j) raw[2 * i + j] = *(const u32x4*)(ap.ptr + row * ap.ld + k0 + 4 * sc + 32 * j);
            }
        }
    };
    // this wave's B fragments: column tile (col0 + 64 wc) / 32 + c, k step ks at + ks 64 fragments
    const uint16_t* bfr = a.bt + ((int64_t)((col0 + 64 * wc) >> 5) * (Ktot >> 4) * 64 + lane) * 8;
    const int64_t ctile = (int64_t)(Ktot >> 4) * 64 * 8;   // elements per column tile
    floatx16 acc[2][2] = {};
    u32x4 raw[8];
    load_raw(0, raw);
    for (int ci = 0; ci < nch; ++ci) {
        int p, k0;
        rows_chunk(a, ci, p, k0);
        const bool is16 = a.A[p].p16 != nullptr;
        bf16x8 bf[4][2];
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4)
#pragma unroll
            for (int c = 0; c < 2; ++c) bf[s4][c] = *(const bf16x8*)(bfr + c * ctile + (int64_t)(4 * ci + s4) * 64 * 8);
        __syncthreads();  // the previous chunk's fragments are read
        const int sh = a.A[p].shift;
        if (is16) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *(u32x4*)&As[(sr + 32 * i) * AROW + 8 * sc] = row_ok(sh, i) ? raw[2 * i] : u32x4{0, 0, 0, 0};
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    *(u32x2*)&As[(sr + 32 * i) * AROW + 4 * sc + 32 * j] =
                        row_ok(sh, i) ? bf16_pack4(raw[2 * i + j]) : u32x2{0, 0};
        }
        __syncthreads();
        if (ci + 1 < nch) load_raw(ci + 1, raw);   // in flight during this chunk's products
#pragma unroll
        for (int s4 = 0; s4 < BK / 16; ++s4) {
            bf16x8 av[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) av[i] = *(const bf16x8*)&As[(64 * wr + 32 * i + r) * AROW + 16 * s4 + 8 * h];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    acc[i][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i], bf[s4][c], acc[i][c], 0, 0, 0);
        }
    }
    rows_epilogue<2>(a, acc, (float*)smem, row0, col0);
}

// The row GEMM in fp32 (v_mfma_f32_32x32x2f32), for FP32 models and the training forward's head: the same
// tile, waves and epilogue, chunks of 32 k. B is packed once per call so that a lane's operands of four
// steps are one 16-byte load; A rows go through LDS at a stride of 33 floats (conflict-free operand reads).
// Products per output in k order. The matrix cores bound it: 32,768 rows x 512 x 128 take 28 us at 154
// TFLOP/s and 45 us here; the 63 products of a backward over them 2.4 ms with the gate's backward in the
// epilogue (64 x 64 tiles, B read from the canonical weights by every block: 3.6 ms and 0.6 ms for the gate).
// RB = 1, 64 rows per block, while 128 would leave a block or less per CU (32,768 rows: 42 | 39 us on average).
constexpr int FK = 32, FLD = FK + 1;
__global__ __launch_bounds__(256) void pack_btf_kernel(GemmRowsArgs a, int Ktot) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;  // i = n Ktot + k
    if (i >= (int64_t)a.N * Ktot) return;
    const int n = (int)(i / Ktot);
    const int kk = (int)(i - (int64_t)n * Ktot);
    int k = kk, p = 0;
    while (p + 1 < a.nparts && k >= a.A[p].K) {
        k -= a.A[p].K;
        ++p;
    }
    const BPart& bp = a.B[p];
    // column tile, group of 8 k, lane (h = k & 1, column), step of the group
    const int64_t f = (((int64_t)(n >> 5) * (Ktot >> 3) + (kk >> 3)) * 64 + (kk & 1) * 32 + (n & 31)) * 4 + ((kk & 7) >> 1);
    a.btf[f] = bp.ptr[(int64_t)k * bp.ld + (int64_t)n * bp.es];
}

template <int RB, bool RELU>
__global__ __launch_bounds__(256) void gemm_rows_f32_kernel(GemmRowsArgs a, int Ktot) {
    __shared__ __attribute__((aligned(16))) float smem[64 * EP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = wave & 1, wc = wave >> 1, r = lane & 31, h = lane >> 5;
    const int ntn = a.N / BN;
    const int64_t row0 = (int64_t)(blockIdx.x / ntn) * 64 * RB;
    const int col0 = (blockIdx.x % ntn) * BN;
    const int t0 = (int)(row0 % a.T);
    const int sr = tid >> 3, sc = tid & 7;   // staging: rows sr + 32 i, k 4 sc .. + 4
    int tw[2 * RB];
#pragma unroll
    for (int i = 0; i < 2 * RB; ++i) {
        int t = t0 + sr + 32 * i;
        while (t >= a.T) t -= a.T;
        tw[i] = t;
    }
    auto row_ok = [&](int sh, int i) { return (unsigned)(tw[i] + sh) < (unsigned)a.T; };
    const int nch = Ktot / FK, n0 = a.A[0].K / FK;
    auto load = [&](int ci, float4 (&raw)[2 * RB]) __attribute__((always_inline)) {
        const APart& ap = a.A[ci < n0 ? 0 : 1];
        const int k0 = FK * (ci < n0 ? ci : ci - n0);
#pragma unroll
        for (int i = 0; i < 2 * RB; ++i)   // (rows whose source leaves the window read the unshifted row and are zeroed below)
            raw[i] = *(const float4*)(ap.ptr + (row0 + sr + 32 * i + (row_ok(ap.shift, i) ? ap.shift : 0)) * ap.ld + k0 + 4 * sc);
    };
    const float* bfr = a.btf + ((int64_t)((col0 + 64 * wc) >> 5) * (Ktot >> 3) * 64 + lane) * 4;
    const int64_t ctile = (int64_t)(Ktot >> 3) * 64 * 4;
    floatx16 acc[RB][2] = {};
    float4 raw[2 * RB];
    load(0, raw);
    for (int ci = 0; ci < nch; ++ci) {
        float4 bf[4][2];
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int c = 0; c < 2; ++c) bf[g][c] = *(const float4*)(bfr + c * ctile + (int64_t)(4 * ci + g) * 64 * 4);
        __syncthreads();  // the previous chunk's operands are read
        const int sh = a.A[ci < n0 ? 0 : 1].shift;
        if (RELU)   // (a.relu_a; tested in the loop it cost an FP32 pass 0.3 %)
#pragma unroll
            for (int i = 0; i < 2 * RB; ++i)
                raw[i] = make_float4(fmaxf(raw[i].x, 0.f), fmaxf(raw[i].y, 0.f), fmaxf(raw[i].z, 0.f), fmaxf(raw[i].w, 0.f));
#pragma unroll
        for (int i = 0; i < 2 * RB; ++i) {
            const bool ok = row_ok(sh, i);
            float* dst = &smem[(sr + 32 * i) * FLD + 4 * sc];
            dst[0] = ok ? raw[i].x : 0.f;
            dst[1] = ok ? raw[i].y : 0.f;
            dst[2] = ok ? raw[i].z : 0.f;
            dst[3] = ok ? raw[i].w : 0.f;
        }
        __syncthreads();
        if (ci + 1 < nch) load(ci + 1, raw);   // in flight during this chunk's products
#pragma unroll
        for (int s = 0; s < FK / 2; ++s) {
            float av[RB];
#pragma unroll
            for (int i = 0; i < RB; ++i) av[i] = smem[(32 * RB * wr + 32 * i + r) * FLD + 2 * s + h];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float4& b4 = bf[s >> 2][c];
                const float bv = (s & 3) == 0 ? b4.x : (s & 3) == 1 ? b4.y : (s & 3) == 2 ? b4.z : b4.w;
#pragma unroll
                for (int i = 0; i < RB; ++i) acc[i][c] = MFMA32(av[i], bv, acc[i][c]);
            }
        }
    }
    rows_epilogue<RB>(a, acc, smem, row0, col0);
}

// Block -> (output tile, row chunk) of the weight-gradient GEMMs. Blocks are dispatched round-robin
// over the 8 XCDs, each with its own L2; the tiles of one chunk read the same rows, so they are put
// on one XCD as consecutive dispatches there and their re-reads hit that L2. The grid is padded to
// a multiple of 8 chunks; blocks of chunks past the end return.
__device__ inline void wgrad_block(int ntiles, int& tile, int& chunk) {
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    tile = idx % ntiles;
    chunk = (idx / ntiles) * 8 + xcd;
}

// Weight-gradient GEMMs: part[chunk][K][N] = sum over the chunk's rows of A(row, k) B(row, n), A from parts
// stacked along k, B from one or two row-shifted parts stacked along n, on 128 x 128 output tiles. A chunk
// is a run of rows_per_chunk rows of one window.
//
// With bf16 operands (rounded to nearest even, fp32 accumulation; 64-row steps, then 16-row groups,
// ascending): waves 0-1 stage the A tile, waves 2-3 the B tile: a thread loads 8 rows x 8 columns
// (one 16-byte load per row for bf16, two for fp32), transposes them in registers and writes 8
// columns of 8 rows as 16-byte words into LDS ([column][row], 144-byte columns: conflict-free
// writes and fragment reads). Two LDS buffers, one barrier per step; the next step's rows are
// loaded during the products. Wave (wk, wn) owns output rows 64 wk .. + 64 and columns 64 wn .. + 64.
// With a.cpart, the blocks of the first column tile also sum their A tile's columns over the chunk's
// rows (fp32 sums of the operand values as stored: fp32 rows before their rounding, bf16 rows
// exactly): each staging thread over its rows in order, then over the 8 threads of a column group.
constexpr int W2T = 128;                 // tile (k and n)
constexpr int W2R = 64;                  // rows per step
constexpr int W2LD = W2R * 2 + 16;       // bytes per LDS column
constexpr int W2OP = W2T * W2LD;         // bytes per operand tile
struct W2Operand {
    const uint16_t* p16;   // bf16 rows, or
    const float* p32;      // fp32 rows
    int64_t ld;
    int shift;             // row shift within the window (zero outside)
};

__device__ inline u32x4 w2_bf16x8(u32x4 lo, u32x4 hi) {  // 8 fp32 (raw bits) -> 8 bf16
    return __builtin_bit_cast(u32x4, bf16_pack8(__builtin_bit_cast(float4, lo), __builtin_bit_cast(float4, hi)));
}

// Eight rows of 8 bf16 columns -> 8 columns of 8 rows, as 16-byte words of the LDS tile.
__device__ inline void w2_store_columns(const u32x4 (&w)[8], uint8_t* dst) {
    // column c: rows (2q, 2q + 1) as one bf16 pair, q < 4
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        u32x4 o;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t lo = w[2 * q][c >> 1], hi = w[2 * q + 1][c >> 1];
            o[q] = (c & 1) ? ((lo >> 16) | (hi & 0xffff0000u)) : ((lo & 0xffffu) | (hi << 16));
        }
        *(u32x4*)(dst + c * W2LD) = o;
    }
}

__global__ __launch_bounds__(256) void gemm_wgrad_t128_kernel(WgradArgs a) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * 2 * W2OP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wk = wave & 1, wn = wave >> 1, h = lane >> 5, r = lane & 31;
    const int ntn = a.N / W2T, ntk = a.Ktot / W2T;
    int tile, chunk;
    wgrad_block(ntn * ntk, tile, chunk);
    const int64_t r0 = (int64_t)chunk * a.rows_per_chunk;
    if (r0 >= a.M) return;  // padding of the grid (uniform per block)
    const int k0 = (tile / ntn) * W2T, n0 = (tile % ntn) * W2T;
    // this thread's operand: waves 0-1 the A tile (columns k0 ..), waves 2-3 the B tile (n0 ..)
    W2Operand op;
    int col;
    const bool isA = wave < 2;
    if (isA) {
        int p = 0, kb = 0;
        while (kb + a.A[p].K <= k0) {
            kb += a.A[p].K;
            ++p;
        }
        op = W2Operand{a.A[p].p16, a.A[p].ptr, a.A[p].ld, a.A[p].shift};
        col = k0 - kb;
    } else {
        const int nb = a.N / a.nbparts, q = n0 / nb;
        op = W2Operand{a.B16, a.B, a.ldb, q ? a.bshift1 : a.bshift};
        col = n0 - q * nb;
    }
    const int t2 = tid & 127, rg = t2 & 7, cm = t2 >> 3;   // rows 8 rg .. + 8, columns 8 cm .. + 8
    col += 8 * cm;
    const bool csum = a.cpart != nullptr && isA && tile % ntn == 0;   // uniform per wave
    float cs[8] = {};
    const int tb = (int)(r0 % a.T);                        // the chunk's first time step and window
    const int64_t wrow0 = r0 - tb;
    const bool is16 = op.p16 != nullptr;
    // rows whose shifted source leaves the window read the unshifted row and are zeroed when staged
    auto load = [&](int step, u32x4 (&raw)[16]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int t = tb + step * W2R + 8 * rg + j;
            const bool ok = (unsigned)(t + op.shift) < (unsigned)a.T;
            const int64_t row = wrow0 + t + (ok ? op.shift : 0);
            if (is16) {
                raw[2 * j] = *(const u32x4*)(op.p16 + row * op.ld + col);
                raw[2 * j + 1] = u32x4{0, 0, 0, 0};
            } else {
                raw[2 * j] = *(const u32x4*)(op.p32 + row * op.ld + col);
                raw[2 * j + 1] = *(const u32x4*)(op.p32 + row * op.ld + col + 4);
            }
        }
    };
    auto stage = [&](int step, const u32x4 (&raw)[16], uint8_t* dst) __attribute__((always_inline)) {
        u32x4 w[8];  // row j: columns 8 cm .. + 8 in bf16
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int t = tb + step * W2R + 8 * rg + j;
            const bool ok = (unsigned)(t + op.shift) < (unsigned)a.T;
            const u32x4 v = is16 ? raw[2 * j] : w2_bf16x8(raw[2 * j], raw[2 * j + 1]);
            w[j] = ok ? v : u32x4{0, 0, 0, 0};
            if (csum && ok) {
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    cs[c] += is16 ? __uint_as_float((c & 1) ? (raw[2 * j][c >> 1] & 0xffff0000u) : (raw[2 * j][c >> 1] << 16))
                                  : __uint_as_float(raw[2 * j + (c >> 2)][c & 3]);
            }
        }
        w2_store_columns(w, dst + 8 * cm * W2LD + 16 * rg);
    };
    floatx16 acc[2][2] = {};
    u32x4 raw[16];
    const int nsteps = (int)(a.rows_per_chunk / W2R);
    load(0, raw);
    for (int s = 0; s < nsteps; ++s) {
        uint8_t* buf = lds + (s & 1) * 2 * W2OP;
        stage(s, raw, buf + (isA ? 0 : W2OP));
        __syncthreads();
        if (s + 1 < nsteps) load(s + 1, raw);   // in flight during the products
        const uint8_t* At = buf;
        const uint8_t* Bt = buf + W2OP;
#pragma unroll
        for (int s16 = 0; s16 < W2R / 16; ++s16) {
            bf16x8 av[2], bv[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                av[i] = *(const bf16x8*)(At + (64 * wk + 32 * i + r) * W2LD + 2 * (16 * s16 + 8 * h));
                bv[i] = *(const bf16x8*)(Bt + (64 * wn + 32 * i + r) * W2LD + 2 * (16 * s16 + 8 * h));
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    acc[i][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i], bv[c], acc[i][c], 0, 0, 0);
        }
    }
    float* out = a.part + (int64_t)chunk * a.Ktot * a.N;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int n = n0 + 64 * wn + 32 * c + r;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int k = k0 + 64 * wk + 32 * i + 8 * (e >> 2) + 4 * h + (e & 3);
                out[(int64_t)k * a.N + n] = acc[i][c][e];
            }
        }
    if (csum) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            cs[c] += __shfl_xor(cs[c], 1);
            cs[c] += __shfl_xor(cs[c], 2);
            cs[c] += __shfl_xor(cs[c], 4);
        }
        if (rg == 0) {
            float* o = a.cpart + (int64_t)chunk * a.Ktot + k0 + 8 * cm;
            *(float4*)o = make_float4(cs[0], cs[1], cs[2], cs[3]);
            *(float4*)(o + 4) = make_float4(cs[4], cs[5], cs[6], cs[7]);
        }
    }
}

// The 256 x 256 product of bf16 rows (the conv taps' gradient: A one part, B two) as one tile per block of eight
// waves: waves 0-3 stage A, waves 4-7 B, wave (wk, wn) owns output rows 128 wk .. + 128 and columns
// 64 wn .. + 64, everything else as above. What bounds the 128 x 128 tiles is the rows in flight between
// the caches and the CUs (64 KB per CU): four blocks of a chunk read every row twice. 524,288 rows: 167 us
// there, 126 us here with one block per CU; the bytes alone take 81 us at the rate of a copy.
constexpr int W3T = 256;
__global__ __launch_bounds__(512) void gemm_wgrad_t256_kernel(WgradArgs a) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * 2 * W3T * W2LD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wk = wave & 1, wn = wave >> 1, h = lane >> 5, r = lane & 31;
    const int chunk = blockIdx.x;
    const int64_t r0 = (int64_t)chunk * a.rows_per_chunk;
    const bool isA = wave < 4;
    const int t2 = tid & 255, rg = t2 & 7, cm = t2 >> 3;   // rows 8 rg .. + 8, columns 8 cm .. + 8
    const int second = !isA && cm >= 16;                   // B's second part: the same columns, shifted
    const uint16_t* src = isA ? a.A[0].p16 + 8 * cm : a.B16 + 8 * (cm & 15);
    const int64_t ld = isA ? a.A[0].ld : a.ldb;
    const int shift = isA ? 0 : second ? a.bshift1 : a.bshift;
    const bool csum = a.cpart != nullptr && isA;           // uniform per wave
    float cs[8] = {};
    const int tb = (int)(r0 % a.T);                        // the chunk's first time step and window
    const int64_t wrow0 = r0 - tb;
    u32x4 raw[8];
    auto load = [&](int step) __attribute__((always_inline)) {   // (rows outside the window read the unshifted row)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int t = tb + step * W2R + 8 * rg + j;
            raw[j] = *(const u32x4*)(src + (wrow0 + t + ((unsigned)(t + shift) < (unsigned)a.T ? shift : 0)) * ld);
        }
    };
    floatx16 acc[4][2] = {};
    const int nsteps = (int)(a.rows_per_chunk / W2R);
    load(0);
    for (int s = 0; s < nsteps; ++s) {
        uint8_t* At = lds + (s & 1) * 2 * W3T * W2LD;
        uint8_t* Bt = At + W3T * W2LD;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int t = tb + s * W2R + 8 * rg + j;
            if ((unsigned)(t + shift) >= (unsigned)a.T) raw[j] = u32x4{0, 0, 0, 0};
            if (csum) {
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    cs[c] += __uint_as_float((c & 1) ? (raw[j][c >> 1] & 0xffff0000u) : (raw[j][c >> 1] << 16));
            }
        }
        w2_store_columns(raw, (isA ? At : Bt) + 8 * cm * W2LD + 16 * rg);
        __syncthreads();
        if (s + 1 < nsteps) load(s + 1);   // in flight during the products
#pragma unroll
        for (int s16 = 0; s16 < W2R / 16; ++s16) {
            bf16x8 av[4], bv[2];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                av[i] = *(const bf16x8*)(At + (128 * wk + 32 * i + r) * W2LD + 2 * (16 * s16 + 8 * h));
#pragma unroll
            for (int c = 0; c < 2; ++c)
                bv[c] = *(const bf16x8*)(Bt + (64 * wn + 32 * c + r) * W2LD + 2 * (16 * s16 + 8 * h));
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    acc[i][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i], bv[c], acc[i][c], 0, 0, 0);
        }
    }
    float* out = a.part + (int64_t)chunk * W3T * W3T;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                out[(128 * wk + 32 * i + 8 * (e >> 2) + 4 * h + (e & 3)) * W3T + 64 * wn + 32 * c + r] = acc[i][c][e];
    if (csum) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            cs[c] += __shfl_xor(cs[c], 1);
            cs[c] += __shfl_xor(cs[c], 2);
            cs[c] += __shfl_xor(cs[c], 4);
        }
        if (rg == 0) {
            float* o = a.cpart + (int64_t)chunk * W3T + 8 * cm;
            *(float4*)o = make_float4(cs[0], cs[1], cs[2], cs[3]);
            *(float4*)(o + 4) = make_float4(cs[4], cs[5], cs[6], cs[7]);
        }
    }
}

// The same in fp32 (v_mfma_f32_32x32x2f32; rows ascending, two per step), for FP32 models: 32-row steps staged
// as they are ([row][column], a stride of 160 floats puts the two rows of a step in different banks), two
// LDS buffers, one barrier per step. The matrix cores bound it: 32,768 rows x 256 x 256 take 28 us at 154
// TFLOP/s and 46 us here. In 64 x 64 tiles with one chunk per window the 91 products of a backward over
// 8 windows of 4,096 took 14.5 ms (160 us each), the 61 of these tiles 2.2 ms.
constexpr int WFR = 32, WFLD = 160;
__global__ __launch_bounds__(256) void gemm_wgrad_f32_kernel(WgradArgs a) {
    __shared__ __attribute__((aligned(16))) float lds[2][2][WFR * WFLD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wk = wave & 1, wn = wave >> 1, h = lane >> 5, r = lane & 31;
    const int ntn = a.N / W2T, ntk = a.Ktot / W2T;
    int tile, chunk;
    wgrad_block(ntn * ntk, tile, chunk);
    const int64_t r0 = (int64_t)chunk * a.rows_per_chunk;
    if (r0 >= a.M) return;  // padding of the grid (uniform per block)
    const int k0 = (tile / ntn) * W2T, n0 = (tile % ntn) * W2T;
    int p = 0, kb = 0;
    while (kb + a.A[p].K <= k0) {
        kb += a.A[p].K;
        ++p;
    }
    const int nb = a.N / a.nbparts, q = n0 / nb;
    const int rr = tid >> 5, c4 = 4 * (tid & 31);   // staging: rows rr + 8 i, four columns of each operand
    const float* pa = a.A[p].ptr + k0 - kb + c4;
    const float* pb = a.B + n0 - q * nb + c4;
    const int64_t lda = a.A[p].ld, ldb = a.ldb;
    const int sa = a.A[p].shift, sb = q ? a.bshift1 : a.bshift;
    const bool csum = a.cpart != nullptr && tile % ntn == 0;   // uniform over the block
    floatx4 cs = {};
    const int tb = (int)(r0 % a.T);
    const int64_t wrow0 = r0 - tb;
    floatx4 ra[4], rb[4];
    auto load = [&](int step) __attribute__((always_inline)) {   // (rows outside the window read the unshifted row)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int t = tb + step * WFR + rr + 8 * i;
            ra[i] = *(const floatx4*)(pa + (wrow0 + t + ((unsigned)(t + sa) < (unsigned)a.T ? sa : 0)) * lda);
            rb[i] = *(const floatx4*)(pb + (wrow0 + t + ((unsigned)(t + sb) < (unsigned)a.T ? sb : 0)) * ldb);
        }
    };
    floatx16 acc[2][2] = {};
    const int nsteps = (int)(a.rows_per_chunk / WFR);
    const floatx4 zero = {};
    load(0);
    for (int s = 0; s < nsteps; ++s) {
        float* At = lds[s & 1][0];
        float* Bt = lds[s & 1][1];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int t = tb + s * WFR + rr + 8 * i;
            const floatx4 va = (unsigned)(t + sa) < (unsigned)a.T ? ra[i] : zero;
            *(floatx4*)&At[(rr + 8 * i) * WFLD + c4] = va;
            *(floatx4*)&Bt[(rr + 8 * i) * WFLD + c4] = (unsigned)(t + sb) < (unsigned)a.T ? rb[i] : zero;
            if (csum) cs += va;
        }
        __syncthreads();
        if (s + 1 < nsteps) load(s + 1);   // in flight during the products
#pragma unroll
        for (int r2 = 0; r2 < WFR; r2 += 2) {
            float av[2], bv[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                av[i] = At[(r2 + h) * WFLD + 64 * wk + 32 * i + r];
                bv[i] = Bt[(r2 + h) * WFLD + 64 * wn + 32 * i + r];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c) acc[i][c] = MFMA32(av[i], bv[c], acc[i][c]);
        }
    }
    float* out = a.part + (int64_t)chunk * a.Ktot * a.N;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int n = n0 + 64 * wn + 32 * c + r;
#pragma unroll
            for (int e = 0; e < 16; ++e)
                out[(int64_t)(k0 + 64 * wk + 32 * i + 8 * (e >> 2) + 4 * h + (e & 3)) * a.N + n] = acc[i][c][e];
        }
    if (csum) {   // the eight row groups' sums, in order
        __syncthreads();
        floatx4* red = (floatx4*)lds;
        red[tid] = cs;
        __syncthreads();
        if (tid < 32) {
            floatx4 t = red[tid];
            for (int k = 1; k < 8; ++k) t += red[32 * k + tid];
            *(floatx4*)(a.cpart + (int64_t)chunk * a.Ktot + k0 + c4) = t;
        }
    }
}

// dst[i * stride] += sum over chunks of part[chunk][i], i = k N + n, in two fixed-order stages:
// stage 1 adds the chunks of each of G consecutive groups (in order) into tmp[g][i], stage 2 adds
// the G group sums (in order) into dst. The result does not depend on scheduling.
__global__ __launch_bounds__(256) void reduce_groups_kernel(const float* part, int nchunks, int per, int64_t KN,
                                                            float* tmp) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= KN) return;
    const int c0 = blockIdx.y * per, c1 = min(c0 + per, nchunks);
    float s = 0.f;
    for (int c = c0; c < c1; ++c) s += part[(int64_t)c * KN + i];
    tmp[(int64_t)blockIdx.y * KN + i] = s;
}
__global__ __launch_bounds__(256) void reduce_parts_kernel(const float* part, int nchunks, int64_t KN, int N,
                                                           WgradDst d) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= KN) return;
    float s = 0.f;
    for (int c = 0; c < nchunks; ++c) s += part[(int64_t)c * KN + i];
    float* dst;
    if (d.taps) {
        const int64_t k = i / N;
        const int n = (int)(i - k * N), C = N / 2;
        dst = d.d0 + (k * C + n % C) * 2 + (n < C ? 1 : 0);
    } else {
        float* base = i < d.split ? d.d0 : d.d1;
        if (!base) return;  // (a null destination drops these sums)
        dst = i < d.split ? base + i * d.stride : base + (i - d.split) * d.stride;
    }
    *dst += s;
}

// Launch the reduction of nchunks partial sums of KN values each (part holds them; scratch for the
// group sums follows them within part_capacity floats).
static hipError_t reduce_parts(float* part, int64_t part_capacity, int nchunks, int64_t KN, int N,
                               const WgradDst& d, hipStream_t st) {
    // 16 groups: stage 1 keeps 16 x KN / 256 blocks busy, stage 2 sums 16 values per thread (with 64
    // groups, stage 2 ran at about 1 TB/s on its 64 sequential loads per thread)
    int G = nchunks >= 128 ? 16 : 1;
    while (G > 1 && (int64_t)(nchunks + G) * KN > part_capacity) G >>= 1;
    if (G > 1) {
        const int per = (nchunks + G - 1) / G;
        G = (nchunks + per - 1) / per;
        float* tmp = part + (int64_t)nchunks * KN;
        hipLaunchKernelGGL(reduce_groups_kernel, dim3((unsigned)((KN + 255) / 256), (unsigned)G), dim3(256), 0, st,
                           (const float*)part, nchunks, per, KN, tmp);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        part = tmp;
        nchunks = G;
    }
    hipLaunchKernelGGL(reduce_parts_kernel, dim3((unsigned)((KN + 255) / 256)), dim3(256), 0, st, (const float*)part,
                       nchunks, KN, N, d);
    return hipGetLastError();
}
static hipError_t reduce_parts(float* part, int64_t part_capacity, int nchunks, int64_t KN, float* dst,
                               int64_t stride, hipStream_t st) {
    return reduce_parts(part, part_capacity, nchunks, KN, (int)KN, WgradDst{dst, nullptr, KN, stride, false}, st);
}

// part[chunk] = sum over the chunk's rows of X[row ldx]: one column, one block per chunk, each thread its
// rows in order, then the threads pairwise (the bias of the logit: 524,288 rows in 4.5 us; 0.38 ms with one
// thread per chunk).
__global__ __launch_bounds__(256) void colsum1_kernel(const float* X, int64_t ldx, int64_t M, int64_t rows_per_chunk,
                                                      float* part) {
    __shared__ float red[256];
    const int64_t r0 = (int64_t)blockIdx.x * rows_per_chunk, r1 = min(r0 + rows_per_chunk, M);
    float s = 0.f;
#pragma unroll 8
    for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) s += X[r * ldx];
    red[threadIdx.x] = s;
    for (int w = 128; w > 0; w >>= 1) {
        __syncthreads();
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// part[chunk][n] = sum over the chunk's rows of f(X[row][n]) * w(row), f = identity or ReLU, for 16-byte
// aligned rows of N = 4 c columns (N <= 1024): one block per chunk, each thread a float4 of columns for every
// (256 / (N/4))-th row of the chunk, then the row groups added in LDS in a fixed order (the result does
// not depend on scheduling).
__global__ __launch_bounds__(256) void colsum4_kernel(const float* X, int64_t ldx, int64_t M, int N,
                                                      const float* w, int64_t wstride, int relu,
                                                      int64_t rows_per_chunk, float* part) {
    __shared__ float4 red[256];
    const int cpr = N >> 2;           // float4 columns per row
    const int groups = 256 / cpr;     // rows in flight per block
    const int tid = threadIdx.x, c4 = tid % cpr, g = tid / cpr;
    const int64_t r0 = (int64_t)blockIdx.x * rows_per_chunk;
    const int64_t r1 = min(r0 + rows_per_chunk, M);
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (g < groups) {
#pragma unroll 4
        for (int64_t r = r0 + g; r < r1; r += groups) {
            float4 v = *(const float4*)(X + r * ldx + 4 * c4);
            if (relu) { v.x = fmaxf(v.x, 0.f); v.y = fmaxf(v.y, 0.f); v.z = fmaxf(v.z, 0.f); v.w = fmaxf(v.w, 0.f); }
            if (w) { const float f = w[r * wstride]; v.x *= f; v.y *= f; v.z *= f; v.w *= f; }
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
    }
    red[tid] = s;
    __syncthreads();
    if (tid < cpr) {
        float4 t = red[tid];
        for (int k = 1; k < groups; ++k) {
            const float4 u = red[k * cpr + tid];
            t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
        }
        *(float4*)(part + (int64_t)blockIdx.x * N + 4 * tid) = t;
    }
}

// x0[row][c] = W_in[c] . u[row] + b_in[c]   (windows [B][T][2] interleaved)
__global__ __launch_bounds__(256) void input_proj_kernel(const float* u, int64_t M, const float* w_in,
                                                         const float* b_in, float* x0) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= M * kC) return;
    const int64_t row = i / kC;
    const int c = (int)(i % kC);
    x0[i] = b_in[c] + w_in[2 * c] * u[2 * row] + w_in[2 * c + 1] * u[2 * row + 1];
}

// Head backward, elementwise part: dh[row][j] = dz[row] * w2[j] * act'(h[row][j]);
// ah[row][j] = act(h[row][j]) (used for d w2).
__global__ __launch_bounds__(256) void head_bwd_elem_kernel(const float* h, const float* dz, int64_t M,
                                                            const float* w2, int mid_relu, float* dh, float* ah) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= M * kC) return;
    const int64_t row = i / kC;
    const int j = (int)(i % kC);
    const float hv = h[i];
    const bool on = !mid_relu || hv > 0.f;
    dh[i] = on ? dz[row] * w2[j] : 0.f;
    ah[i] = mid_relu ? fmaxf(hv, 0.f) : hv;
}

// logit[row] = w2 . act(h[row]) + b2
__global__ __launch_bounds__(256) void head_logit_kernel(const float* h, int64_t M, const float* w2,
                                                         const float* b2, int mid_relu, float* z) {
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row >= M) return;
    float s = 0.f;
    for (int j = 0; j < kC; ++j) {
        float v = h[row * kC + j];
        if (mid_relu) v = fmaxf(v, 0.f);
        s = fmaf(w2[j], v, s);
    }
    z[row] = s + b2[0];
}

// du[row][i] = sum_c dx0[row][c] W_in[c][i]
__global__ __launch_bounds__(256) void input_grad_kernel(const float* dx0, int64_t M, const float* w_in, float* du) {
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row >= M) return;
    float s0 = 0.f, s1 = 0.f;
    for (int c = 0; c < kC; ++c) {
        const float d = dx0[row * kC + c];
        s0 = fmaf(d, w_in[2 * c], s0);
        s1 = fmaf(d, w_in[2 * c + 1], s1);
    }
    du[2 * row] = s0;
    du[2 * row + 1] = s1;
}

// The same rounded to bf16, for the bf16 residual stream: four channels per thread, 8-byte stores (524,288 rows: a
// pass in fp32 and one to round it took 274 us).
__global__ __launch_bounds__(256) void input_proj_bf16_kernel(const float* u, int64_t M, const float* w_in, const float* b_in,
                                                              uint16_t* x0) {
    const int64_t i = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
    if (i >= M * kC) return;
    const int64_t row = i / kC;
    const int c = (int)(i % kC);
    const float u0 = u[2 * row], u1 = u[2 * row + 1];
    u32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = __float_as_uint(b_in[c + e] + w_in[2 * (c + e)] * u0 + w_in[2 * (c + e) + 1] * u1);
    *(u32x2*)(x0 + i) = bf16_pack4(v);
}
__global__ __launch_bounds__(256) void relu_copy_kernel(const float* x, int64_t n, float* y) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) y[i] = fmaxf(x[i], 0.f);
}

__global__ __launch_bounds__(256) void fill_kernel(float* p, int64_t n, float v) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

// ---- Adam with bias correction; per-block fp64 partial sums of g^2 for the global norm
__global__ __launch_bounds__(256) void adam_kernel(float* w, const float* g, float* m, float* v, int64_t n,
                                                   float lr, float b1, float b2, float eps, float c1, float c2,
                                                   double* norm_part) {
    __shared__ double red[4];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double sq = 0.0;
    if (i < n) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float mh = mi / c1, vh = vi / c2;
        w[i] -= lr * mh / (sqrtf(vh) + eps);
        sq = (double)gi * (double)gi;
    }
    for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sq;
    __syncthreads();
    if (threadIdx.x == 0) norm_part[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

__global__ __launch_bounds__(256) void norm_final_kernel(const double* part, int64_t n, double* out) {
    __shared__ double red[256];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sqrt(red[0]);
}

// BCE on logits: grad[i] = (sigmoid(z) - y) / n; loss partials in fp64
__global__ __launch_bounds__(256) void bce_kernel(const float* z, const float* y, int64_t n, float* grad,
                                                  double* part) {
    __shared__ double red[4];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double l = 0.0;
    if (i < n) {
        const double zz = z[i], yy = y[i];
        l = fmax(zz, 0.0) + log1p(exp(-fabs(zz))) - yy * zz;
        grad[i] = (float)((1.0 / (1.0 + exp(-zz)) - yy) / (double)n);
    }
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = l;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

__global__ __launch_bounds__(256) void mean_final_kernel(const double* part, int64_t nparts, int64_t n,
                                                         double* out) {
    __shared__ double red[256];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < nparts; i += 256) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0] / (double)n;
}

// ---------------------------------------------------------------- launchers
static inline unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

hipError_t gemm_rows(const GemmRowsArgs& a, hipStream_t st) {
    bool bf16 = a.bt != nullptr && (!a.mask || ((uintptr_t)a.mask & 15) == 0), any16 = false;
    int Ktot = 0;
    bool ok = a.N % BN == 0 && a.M % BR2 == 0 && a.nparts >= 1 && a.nparts <= 2;
    for (int p = 0; p < a.nparts; ++p) {
        Ktot += a.A[p].K;
        const APart& q = a.A[p];
        any16 = any16 || q.p16;
        bf16 = bf16 && q.K % BK == 0 && (!q.p16 || (q.ld % 8 == 0 && ((uintptr_t)q.p16 & 15) == 0));
        ok = ok && q.K % FK == 0 && (q.p16 || (q.ld % 4 == 0 && ((uintptr_t)q.ptr & 15) == 0));
    }
    // the epilogue moves 4 columns at a time
    ok = ok && (!a.C || (a.ldc % 4 == 0 && ((uintptr_t)a.C & 15) == 0)) && (!a.mask || a.ldm % 4 == 0) &&
         (!a.bias || ((uintptr_t)a.bias & 15) == 0);
    if (!ok || (!bf16 && (any16 || !a.btf))) return hipErrorInvalidValue;
    if (!a.C && !a.gpre && !a.gpre32) return hipErrorInvalidValue;
    if ((a.relu_a && bf16) || (a.c16 && (!a.C || a.gpre || a.gpre32 || ((uintptr_t)a.c16 & 7)))) return hipErrorInvalidValue;
    if ((a.gpre || a.gpre32) && (a.N != kC || a.bias || a.beta != 0.f || a.mask)) return hipErrorInvalidValue;
    if (a.gpre && (!bf16 || !a.g16 || !a.dpre16 || ((uintptr_t)a.gpre & 7))) return hipErrorInvalidValue;
    if (a.gpre32 && (!a.g32 || !a.dpre32 || (((uintptr_t)a.gpre32 | (uintptr_t)a.g32 | (uintptr_t)a.dpre32) & 15)))
        return hipErrorInvalidValue;
    const dim3 pgrid((unsigned)(((int64_t)a.N * Ktot + 255) / 256)), grid((unsigned)((a.M / BR2) * (a.N / BN)));
    if (bf16) hipLaunchKernelGGL(pack_bt_kernel, pgrid, dim3(256), 0, st, a, Ktot);
    else hipLaunchKernelGGL(pack_btf_kernel, pgrid, dim3(256), 0, st, a, Ktot);
    if (bf16) hipLaunchKernelGGL(gemm_rows_bf16_kernel, grid, dim3(256), 0, st, a, Ktot);
    else if (grid.x >= 512) {
        if (a.relu_a) hipLaunchKernelGGL((gemm_rows_f32_kernel<2, true>), grid, dim3(256), 0, st, a, Ktot);
        else hipLaunchKernelGGL((gemm_rows_f32_kernel<2, false>), grid, dim3(256), 0, st, a, Ktot);
    } else {
        const dim3 grid1(2 * grid.x);
        if (a.relu_a) hipLaunchKernelGGL((gemm_rows_f32_kernel<1, true>), grid1, dim3(256), 0, st, a, Ktot);
        else hipLaunchKernelGGL((gemm_rows_f32_kernel<1, false>), grid1, dim3(256), 0, st, a, Ktot);
    }
    return hipGetLastError();
}

// Rows per chunk: whole windows when they give a block for each of the chip's 512 slots (two per CU), else
// windows halved, down to 128 rows (two steps of the bf16 kernel). 8 windows of 4,096 rows have 8 chunks
// otherwise, 32 blocks or fewer; 128 windows the same 512 blocks for the conv taps, but 256 for skip and residual.
static int64_t wgrad_rows(int64_t M, int T, int64_t tiles, int64_t blocks) {
    int64_t rpc = T;
    while ((M / rpc) * tiles < blocks && rpc % 256 == 0) rpc /= 2;
    return rpc;
}

// Partial sums of `chunks` chunks, and the group sums that reduce_parts puts behind 128 or more.
static int64_t wgrad_floats(int64_t chunks, int64_t KN) { return (chunks + (chunks >= 128 ? 16 : 0)) * KN; }

// Rows per chunk of the 256 x 256 tile, 0 where it does not pay: enough chunks for three quarters of the CUs,
// long enough (16 steps) to be worth their partial sums of 256 KB each (128 windows of 4,096: 33 MB more, 4 us
// of reduction for the 41 us gained).
static int64_t wgrad_rows_t256(int64_t M, int T) {
    const int64_t rpc = wgrad_rows(M, T, 1, 192);
    return rpc >= 1024 && M / rpc >= 192 ? rpc : 0;
}

int64_t wgrad_part_floats(int64_t M, int T) {
    int64_t most = 0;
    for (int tiles : {1, 2, 4}) {   // 128 x 128, 256 x 128, 256 x 256
        int64_t rpc = wgrad_rows(M, T, tiles, 512);
        if (tiles == 4 && wgrad_rows_t256(M, T)) rpc = std::min(rpc, wgrad_rows_t256(M, T));
        most = std::max(most, wgrad_floats(M / rpc, (int64_t)tiles * W2T * W2T));
    }
    return most;
}

hipError_t gemm_wgrad(const WgradArgs& a0, const WgradDst& d, hipStream_t st, const WgradDst* cdst) {
    WgradArgs a = a0;
    if ((a.B16 || a.A[0].p16 || (a.nparts > 1 && a.A[1].p16)) && !a.bf16) return hipErrorInvalidValue;
    if (a.nbparts < 1 || a.nbparts > 2 || a.N % a.nbparts) return hipErrorInvalidValue;
    // whole tiles and steps, 16-byte rows
    bool ok = a.T % W2R == 0 && a.M % a.T == 0 && a.Ktot % W2T == 0 && (a.N / a.nbparts) % W2T == 0 && a.ldb % 8 == 0 &&
              ((uintptr_t)(a.B16 ? (const void*)a.B16 : a.B) & 15) == 0;
    for (int p = 0; p < a.nparts; ++p) {
        const APart& q = a.A[p];
        ok = ok && q.K % W2T == 0 && q.ld % 8 == 0 && ((uintptr_t)(q.p16 ? (const void*)q.p16 : q.ptr) & 15) == 0;
    }
    if (!ok || (a.cpart && (!cdst || a.A[0].shift != 0 || (a.nparts > 1 && a.A[1].shift != 0)))) return hipErrorInvalidValue;
    a.rows_per_chunk = wgrad_rows(a.M, a.T, (a.Ktot / W2T) * (a.N / W2T), 512);
    const int64_t r256 = wgrad_rows_t256(a.M, a.T);
    const bool t256 = r256 && a.bf16 && a.nparts == 1 && a.Ktot == W3T && a.N == W3T && a.nbparts == 2 && a.A[0].p16 &&
                      a.B16 && a.A[0].shift == 0;
    if (t256) a.rows_per_chunk = r256;
    // (where the workspace holds less than it might, fewer and longer chunks)
    const auto fits = [&](int64_t n) {
        return wgrad_floats(n, (int64_t)a.Ktot * a.N) <= a.part_capacity && (!a.cpart || wgrad_floats(n, a.Ktot) <= a.cpart_capacity);
    };
    while (a.rows_per_chunk < a.T && !fits(a.M / a.rows_per_chunk)) a.rows_per_chunk *= 2;
    const int nchunks = (int)(a.M / a.rows_per_chunk);
    if ((int64_t)nchunks * a.Ktot * a.N > a.part_capacity || (a.cpart && (int64_t)nchunks * a.Ktot > a.cpart_capacity))
        return hipErrorInvalidValue;
    const int64_t blocks = (int64_t)((nchunks + 7) / 8) * 8 * (a.Ktot / W2T) * (a.N / W2T);
    if (t256) hipLaunchKernelGGL(gemm_wgrad_t256_kernel, dim3((unsigned)nchunks), dim3(512), 0, st, a);
    else if (a.bf16) hipLaunchKernelGGL(gemm_wgrad_t128_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL(gemm_wgrad_f32_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = reduce_parts(a.part, a.part_capacity, nchunks, (int64_t)a.Ktot * a.N, a.N, d, st);
    if (e != hipSuccess || !cdst) return e;
    return a.cpart ? reduce_parts(a.cpart, a.cpart_capacity, nchunks, a.Ktot, a.Ktot, *cdst, st) : hipErrorInvalidValue;
}

hipError_t colsum(const float* X, int64_t ldx, int64_t M, int N, const float* w, int64_t wstride, int relu,
                  float* part, int64_t part_capacity, float* dst, int64_t dst_stride, hipStream_t st) {
    if (N < 1 || part_capacity < N) return hipErrorInvalidValue;
    const bool vec = N % 4 == 0 && N <= 1024 && ldx % 4 == 0 && ((uintptr_t)X & 15) == 0;
    if (!vec && (N != 1 || w || relu)) return hipErrorInvalidValue;
    // rows per chunk: enough chunks to fill the chip, partial sums within the buffer's capacity
    int64_t rpc = vec ? 512 : 4096;
    while (((M + rpc - 1) / rpc) * (int64_t)N > part_capacity) rpc *= 2;
    const int nchunks = (int)((M + rpc - 1) / rpc);
    if (vec)
        hipLaunchKernelGGL(colsum4_kernel, dim3(nchunks), dim3(256), 0, st, X, ldx, M, N, w, wstride, relu, rpc, part);
    else
        hipLaunchKernelGGL(colsum1_kernel, dim3(nchunks), dim3(256), 0, st, X, ldx, M, rpc, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return reduce_parts(part, part_capacity, nchunks, N, dst, dst_stride, st);
}

hipError_t launch_input_proj(const float* u, int64_t M, const float* w_in, const float* b_in, float* x0,
                             hipStream_t st) {
    hipLaunchKernelGGL(input_proj_kernel, dim3(nblk(M * kC)), dim3(256), 0, st, u, M, w_in, b_in, x0);
    return hipGetLastError();
}
hipError_t launch_head_bwd_elem(const float* h, const float* dz, int64_t M, const float* w2, int mid, float* dh,
                                float* ah, hipStream_t st) {
    hipLaunchKernelGGL(head_bwd_elem_kernel, dim3(nblk(M * kC)), dim3(256), 0, st, h, dz, M, w2, mid, dh, ah);
    return hipGetLastError();
}
hipError_t launch_head_logit(const float* h, int64_t M, const float* w2, const float* b2, int mid, float* z,
                             hipStream_t st) {
    hipLaunchKernelGGL(head_logit_kernel, dim3(nblk(M)), dim3(256), 0, st, h, M, w2, b2, mid, z);
    return hipGetLastError();
}
hipError_t launch_input_grad(const float* dx0, int64_t M, const float* w_in, float* du, hipStream_t st) {
    hipLaunchKernelGGL(input_grad_kernel, dim3(nblk(M)), dim3(256), 0, st, dx0, M, w_in, du);
    return hipGetLastError();
}
hipError_t launch_input_proj_bf16(const float* u, int64_t M, const float* w_in, const float* b_in, uint16_t* x0,
                                  hipStream_t st) {
    hipLaunchKernelGGL(input_proj_bf16_kernel, dim3(nblk(M * kC / 4)), dim3(256), 0, st, u, M, w_in, b_in, x0);
    return hipGetLastError();
}
hipError_t launch_relu_copy(const float* x, int64_t n, float* y, hipStream_t st) {
    hipLaunchKernelGGL(relu_copy_kernel, dim3(nblk(n)), dim3(256), 0, st, x, n, y);
    return hipGetLastError();
}
// dst[i] = src[idx[i]]: the two-branch member's gradient read back from its block-diagonal trunk's
__global__ void gather_kernel(const float* src, const int64_t* idx, int64_t n, float* dst) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) dst[i] = src[idx[i]];
}

hipError_t launch_gather(const float* src, const int64_t* idx, int64_t n, float* dst, hipStream_t st) {
    hipLaunchKernelGGL(gather_kernel, dim3(nblk(n)), dim3(256), 0, st, src, idx, n, dst);
    return hipGetLastError();
}

hipError_t launch_fill(float* p, int64_t n, float v, hipStream_t st) {
    hipLaunchKernelGGL(fill_kernel, dim3(nblk(n)), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}
hipError_t launch_adam(float* w, const float* g, float* m, float* v, int64_t n, float lr, float b1, float b2,
                       float eps, int64_t step, double* norm_part, double* norm_out, hipStream_t st) {
    const float c1 = (float)(1.0 - pow((double)b1, (double)step));
    const float c2 = (float)(1.0 - pow((double)b2, (double)step));
    const unsigned nb = nblk(n);
    hipLaunchKernelGGL(adam_kernel, dim3(nb), dim3(256), 0, st, w, g, m, v, n, lr, b1, b2, eps, c1, c2, norm_part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !norm_out) return e;
    hipLaunchKernelGGL(norm_final_kernel, dim3(1), dim3(256), 0, st, norm_part, (int64_t)nb, norm_out);
    return hipGetLastError();
}
hipError_t launch_bce(const float* z, const float* y, int64_t n, float* grad, double* part, double* loss,
                      hipStream_t st) {
    const unsigned nb = nblk(n);
    hipLaunchKernelGGL(bce_kernel, dim3(nb), dim3(256), 0, st, z, y, n, grad, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mean_final_kernel, dim3(1), dim3(256), 0, st, part, (int64_t)nb, n, loss);
    return hipGetLastError();
}

// ---------------------------------------------------------------- working-weight refresh on the device
// After an optimiser step the member's device image is rebuilt from the new fp32 master weights by
// one gather kernel, with the fragment orders of pack_member (pack.cpp) written out per element:
// blockIdx.y = layer (blockIdx.y == L: the input projection and the head, copied as fp32). BF16:
// each weight rounded to nearest even (the hardware conversion); FP32: copied.
namespace {
template <bool BF16>
__global__ void repack_kernel(const float* __restrict__ blob, uint8_t* __restrict__ img, const RepackLayer* tab, int L,
                              RepackFixed fx) {
    const int l = blockIdx.y;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (l == L) {   // fixed tensors: [w_in 256 | b_in 128 | h1w 16384 | h1b 128 | h2w 128 | h2b 1]
        const int64_t n_fix = 256 + 128 + 16384 + 128 + 128 + 1;
        for (int64_t e = t0; e < n_fix; e += step) {
            int64_t src, dst;
            if (e < 256) { src = fx.in_w + e; dst = fx.d_in_w + e; }
            else if (e < 384) { src = fx.in_b + e - 256; dst = fx.d_in_b + e - 256; }
            else if (e < 384 + 16384) { src = fx.h1w + e - 384; dst = fx.d_h1w + e - 384; }
            else if (e < 384 + 16384 + 128) { src = fx.h1b + e - 16768; dst = fx.d_h1b + e - 16768; }
            else if (e < 384 + 16384 + 256) { src = fx.h2w + e - 16896; dst = fx.d_h2w + e - 16896; }
            else { src = fx.h2b; dst = fx.d_h2b; }
            ((float*)img)[dst] = blob[src];
        }
        return;
    }
    const RepackLayer t = tab[l];
    const bool last = t.res_w < 0;
    const int nrs = last ? 128 : 256;
    const int64_t n_conv = 65536, n_rs = (int64_t)nrs * 128;
    const int64_t n_all = n_conv + n_rs + 256 + nrs;
    for (int64_t e = t0; e < n_all; e += step) {
        if (e < n_conv) {   // conv: K = 256 (tap 0 multiplies x[t - d]), N = 256
            int k, n;
            if (BF16) {
                const int i = e & 7, ln = (e >> 3) & 63, j = (e >> 9) & 15, cb = (int)(e >> 13);
                k = 16 * j + 8 * (ln >> 5) + i;
                n = 32 * cb + (ln & 31);
            } else {
                const int i = e & 3, ln = (e >> 2) & 63, j = (e >> 8) & 15, cb = (int)(e >> 12);
                k = 16 * j + 4 * (ln >> 4) + i;
                n = 16 * cb + (ln & 15);
            }
            const float w = blob[t.dil_w + ((int64_t)n * 128 + (k & 127)) * 2 + (k >> 7)];
            if (BF16) ((__bf16*)(img + t.wc))[e] = (__bf16)w;
            else ((float*)(img + t.wc))[e] = w;
        } else if (e < n_conv + n_rs) {   // res | skip: K = 128, N = 256 (last layer: skip only, N = 128)
            const int64_t f = e - n_conv;
            int k, n;
            if (BF16) {
                const int i = f & 7, ln = (f >> 3) & 63, j = (f >> 9) & 7, cb = (int)(f >> 12);
                k = 16 * j + 8 * (ln >> 5) + i;
                n = 32 * cb + (ln & 31);
            } else {
                const int i = f & 3, ln = (f >> 2) & 63, j = (f >> 8) & 15, cb = (int)(f >> 12);
                k = 8 * j + 4 * (ln >> 5) + i;
                n = 32 * cb + (ln & 31);
            }
            const float w = last ? blob[t.skip_w + (int64_t)n * 128 + k]
                          : n < 128 ? blob[t.res_w + (int64_t)n * 128 + k] : blob[t.skip_w + (int64_t)(n - 128) * 128 + k];
            if (BF16) ((__bf16*)(img + t.wrs))[f] = (__bf16)w;
            else ((float*)(img + t.wrs))[f] = w;
        } else if (e < n_conv + n_rs + 256) {   // conv bias
            const int c = (int)(e - n_conv - n_rs);
            ((float*)(img + t.bc))[c] = blob[t.dil_b + c];
        } else {   // res | skip bias
            const int c = (int)(e - n_conv - n_rs - 256);
            ((float*)(img + t.brs))[c] = last ? blob[t.skip_b + c] : c < 128 ? blob[t.res_b + c] : blob[t.skip_b + c - 128];
        }
    }
}

__global__ void scatter_kernel(const float* src, const int64_t* idx, int64_t n, float* dst) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) dst[idx[i]] = src[i];
}
}  // namespace

hipError_t launch_repack(bool bf16, const float* blob, uint8_t* img, const RepackLayer* tab, int L,
                         const RepackFixed& fx, hipStream_t st) {
    const dim3 grid(96, L + 1);
    if (bf16) hipLaunchKernelGGL(repack_kernel<true>, grid, dim3(256), 0, st, blob, img, tab, L, fx);
    else hipLaunchKernelGGL(repack_kernel<false>, grid, dim3(256), 0, st, blob, img, tab, L, fx);
    return hipGetLastError();
}

hipError_t launch_scatter(const float* src, const int64_t* idx, int64_t n, float* dst, hipStream_t st) {
    hipLaunchKernelGGL(scatter_kernel, dim3(nblk(n)), dim3(256), 0, st, src, idx, n, dst);
    return hipGetLastError();
}

}  // namespace gwd
