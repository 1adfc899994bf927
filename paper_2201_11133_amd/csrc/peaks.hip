// The paper's post-processing of model outputs ("AI ensemble construction", "Statistical
// Analysis", "Event Detection"): peak finding with a height threshold and a minimum width at half
// prominence (the semantics of SciPy's find_peaks), and all-member coincidence.
//
// Device steps over a float64 signal x[0, n):
//   1. one pass over x, a block per tile of 4096 samples: the bit of each sample that is the rising edge of
//      a qualifying peak (x[i-1] < x[i], the run of samples equal to x[i] ends below it before the last
//      sample, and x >= height), the tile's count, and the summaries of its blocks of 256 samples
//      (maximum, minimum, first and last index of the minimum), by which walks take whole blocks;
//   2. a scan of the counts, beside the summaries of 256 blocks each;
//   3. the ordered list of the peaks (the middle of each run);
//   4. one wave per peak walks to its bases and to the half-prominence crossings, 64 samples or 64 block
//      summaries at a time (float64), and marks the peaks whose width reaches the minimum;
//   5. a scan and an ordered list of those, which is all the host copies.
// Nothing waits for the host in between. Member of 900 s (3.7 M samples, 34,000 peaks above 0.9): the
// walks, one thread per peak before, bounded it (the wave waits for its longest walk): 644 us; now 44 us,
// and the passes over x together 66 us before, 39 us now.
#include <algorithm>
#include <mutex>
#include <new>
#include <vector>

#include "gwd_internal.h"

namespace gwd {

constexpr int PK_TILE = 4096;   // samples (or peaks) per tile of the ordered lists: one block
constexpr int PK_WORDS = PK_TILE / 64;
constexpr int PK_B1 = 256;                             // samples per block summary
constexpr int64_t PK_B2 = (int64_t)PK_B1 * PK_B1;      // and per second-level summary
constexpr int PK_WAVES = 8192;                         // resident waves of the walks
constexpr int PK_FIRST = 512;                          // peaks copied to the host with the count

struct PkSum {
    double mx, mn;
    int64_t first, last;
};
struct PkOut {
    int64_t peak;
    double width;
};
struct PkHead {        // followed by the kept peaks
    int64_t found;
    int64_t bad;       // NaN or Inf in the signal
};

__device__ inline PkSum pk_merge(PkSum a, PkSum b) {  // a covers lower indices than b
    PkSum r;
    r.mx = a.mx > b.mx ? a.mx : b.mx;
    if (a.mn < b.mn) { r.mn = a.mn; r.first = a.first; r.last = a.last; }
    else if (b.mn < a.mn) { r.mn = b.mn; r.first = b.first; r.last = b.last; }
    else { r.mn = a.mn; r.first = a.first; r.last = b.last; }
    return r;
}

// Minimum (MAX: maximum) over the wave, in every lane. Rotations within rows of 16 lanes, then the
// row and half swaps: register moves, where shuffles through LDS cost a round trip for each step.
template <bool MAX, class V>
__device__ inline double pk_pick(V lo, V hi) {
    const double a = __hiloint2double((int)hi[0], (int)lo[0]), b = __hiloint2double((int)hi[1], (int)lo[1]);
    return MAX ? (b > a ? b : a) : (b < a ? b : a);
}
template <bool MAX, int ROR>
__device__ inline double pk_rotate(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + ROR, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + ROR, 0xf, 0xf, false);
    const double w = __hiloint2double(hi, lo);
    return MAX ? (w > v ? w : v) : (w < v ? w : v);
}
template <bool MAX>
__device__ inline double wave_pick(double v) {
    v = pk_rotate<MAX, 1>(v);
    v = pk_rotate<MAX, 2>(v);
    v = pk_rotate<MAX, 4>(v);
    v = pk_rotate<MAX, 8>(v);
    unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    v = pk_pick<MAX>(__builtin_amdgcn_permlane16_swap(lo, lo, false, false), __builtin_amdgcn_permlane16_swap(hi, hi, false, false));
    lo = (unsigned)__double2loint(v);
    hi = (unsigned)__double2hiint(v);
    return pk_pick<MAX>(__builtin_amdgcn_permlane32_swap(lo, lo, false, false),
                        __builtin_amdgcn_permlane32_swap(hi, hi, false, false));
}
__device__ inline double wave_min(double v) { return wave_pick<false>(v); }
__device__ inline double wave_max(double v) { return wave_pick<true>(v); }

__device__ inline int64_t peak_of_edge(const double* x, int64_t n, int64_t i, double height) {
    if (!(x[i - 1] < x[i])) return -1;
    int64_t j = i + 1;
    while (j < n - 1 && x[j] == x[i]) ++j;
    if (!(x[j] < x[i])) return -1;
    const int64_t p = (i + j - 1) >> 1;
    return x[p] >= height ? p : -1;
}

// Step 1; also clears what step 4 marks (kmask: one bit per peak, kcount: kept peaks per tile of peaks).
__global__ __launch_bounds__(256) void pk_pass_kernel(const double* __restrict__ x, int64_t n, double height, uint64_t* mask,
                                                      int64_t* counts, PkSum* s1, PkHead* head, uint64_t* kmask,
                                                      int64_t* kcount, int64_t nkt) {
    __shared__ PkSum part[PK_TILE / PK_B1][4];
    __shared__ int cnt[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t tile = blockIdx.x, t0 = tile * PK_TILE;
    int c = 0;
    bool bad = false;
    double vals[PK_TILE / PK_B1];   // the tile's loads all in flight at once
#pragma unroll
    for (int r = 0; r < PK_TILE / PK_B1; ++r) vals[r] = x[min(t0 + r * PK_B1 + tid, n - 1)];
#pragma unroll
    for (int r = 0; r < PK_TILE / PK_B1; ++r) {
        const int64_t i = t0 + r * PK_B1 + tid;
        const double v = vals[r];
        bad = bad || !isfinite(v);
        const bool f = i >= 1 && i < n - 1 && v >= height && peak_of_edge(x, n, i, height) >= 0;
        const uint64_t m = __ballot(f);
        c += __popcll(m);
        const double mx = wave_max(i < n ? v : -INFINITY), mn = wave_min(i < n ? v : INFINITY);
        const uint64_t at = __ballot(i < n && v == mn);
        if (lane == 0) {
            mask[tile * PK_WORDS + r * 4 + wave] = m;
            part[r][wave] = PkSum{mx, mn, i + __ffsll((unsigned long long)at) - 1, i + 63 - __clzll((long long)at)};
        }
    }
    if (bad) head->bad = 1;   // (every writer stores the same value; cleared before this launch)
    if (lane == 0) cnt[wave] = c;
    __syncthreads();
    if (tid == 0) counts[tile] = cnt[0] + cnt[1] + cnt[2] + cnt[3];
    if (tid < PK_TILE / PK_B1 && t0 + tid * PK_B1 < n)
        s1[tile * (PK_TILE / PK_B1) + tid] = pk_merge(pk_merge(part[tid][0], part[tid][1]), pk_merge(part[tid][2], part[tid][3]));
    if (tile < nkt) {   // (at most half as many peaks as samples)
        if (tid < PK_WORDS) kmask[tile * PK_WORDS + tid] = 0;
        if (tid == 0) kcount[tile] = 0;
    }
}

__global__ void pk_clear_kernel(PkHead* head) {
    if (threadIdx.x == 0) *head = PkHead{0, 0};
}

// exclusive scan of counts[0, nt) in place, total in counts[nt]; one block of 256
__device__ void pk_scan(int64_t* counts, int64_t nt, int64_t (&part)[256]) {
    const int64_t per = (nt + 255) / 256;
    const int64_t a = std::min<int64_t>(threadIdx.x * per, nt), b = std::min<int64_t>(a + per, nt);
    int64_t s = 0;
    for (int64_t k = a; k < b; ++k) s += counts[k];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
        const int64_t v = (int)threadIdx.x >= o ? part[threadIdx.x - o] : 0;
        __syncthreads();
        part[threadIdx.x] += v;
        __syncthreads();
    }
    int64_t run = part[threadIdx.x] - s;
    if (threadIdx.x == 255) counts[nt] = part[255];
    for (int64_t k = a; k < b; ++k) {
        const int64_t v = counts[k];
        counts[k] = run;
        run += v;
    }
}

// Step 2: block 0 scans the counts, block 1 + g forms the second-level summary of s1[256 g, 256 (g + 1)).
__global__ __launch_bounds__(256) void pk_scan_kernel(int64_t* counts, int64_t nt, const PkSum* s1, int64_t n1, PkSum* s2) {
    __shared__ int64_t part[256];
    __shared__ PkSum red[4];
    if (blockIdx.x == 0) {
        pk_scan(counts, nt, part);
        return;
    }
    const int64_t k = (int64_t)(blockIdx.x - 1) * PK_B1 + threadIdx.x;
    PkSum v = k < n1 ? s1[k] : PkSum{-INFINITY, INFINITY, INT64_MAX, -1};
    for (int o = 1; o < 64; o <<= 1) {  // lane l merges l + o (lower lanes cover lower indices)
        const PkSum w{__shfl_down(v.mx, o), __shfl_down(v.mn, o), __shfl_down(v.first, o), __shfl_down(v.last, o)};
        if ((threadIdx.x & 63) + o < 64 && ((threadIdx.x & 63) & (2 * o - 1)) == 0) v = pk_merge(v, w);
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) s2[blockIdx.x - 1] = pk_merge(pk_merge(red[0], red[1]), pk_merge(red[2], red[3]));
}

// The set bits of tile `tile` of a mask, in order: put(index of the bit, its rank in the whole list).
template <class F>
__device__ inline void pk_each(const uint64_t* mask, const int64_t* offsets, int64_t tile, F put) {
    __shared__ int before[PK_WORDS];
    __shared__ uint64_t words[PK_WORDS];
    if (threadIdx.x < PK_WORDS) {   // one wave
        const uint64_t m = mask[tile * PK_WORDS + threadIdx.x];
        int s = __popcll(m);
        const int own = s;
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(s, o);
            if ((int)threadIdx.x >= o) s += v;
        }
        words[threadIdx.x] = m;
        before[threadIdx.x] = s - own;
    }
    __syncthreads();
    const int64_t base = offsets[tile];
    for (int k = threadIdx.x; k < PK_TILE; k += 256) {
        const uint64_t m = words[k >> 6];
        if ((m >> (k & 63)) & 1) put(tile * PK_TILE + k, base + before[k >> 6] + __popcll(m & ((1ull << (k & 63)) - 1)));
    }
    __syncthreads();
}

// Step 3
__global__ __launch_bounds__(256) void pk_list_kernel(const double* x, int64_t n, double height, const uint64_t* mask,
                                                      const int64_t* offsets, int64_t* cand) {
    pk_each(mask, offsets, blockIdx.x, [&](int64_t i, int64_t rank) { cand[rank] = peak_of_edge(x, n, i, height); });
}

// One direction of a peak's walks, by one wave: DIR -1 to lower indices, +1 to higher ones. `stop(i)` says
// whether sample i ends the walk, `stop_sum(s, b)` whether summary s of the samples [b, b + size) may hold
// such a sample, and `pass(value, index, steps)` takes what was passed: per lane the least value of the
// samples passed (+inf: none), its index nearest to the start and the lanes' order. From j on, samples go
// 64 at a time up to a block boundary, then block summaries, then second-level ones. Returns the index
// that ended the walk, or -1 / n.
template <int DIR, class Stop, class StopSum, class Pass>
__device__ inline int64_t pk_walk(const double* __restrict__ x, int64_t n, const PkSum* __restrict__ s1,
                                  const PkSum* __restrict__ s2, int64_t j, Stop stop, StopSum stop_sum, Pass pass) {
    const int lane = threadIdx.x & 63;
    int deny = 0;   // 2: the first-level summary of j's block may stop the walk, 1: the second-level one
    while (DIR < 0 ? j >= 0 : j < n) {
        const bool at1 = DIR < 0 ? (j & (PK_B1 - 1)) == PK_B1 - 1 || j == n - 1 : (j & (PK_B1 - 1)) == 0;
        const bool at2 = DIR < 0 ? (j & (PK_B2 - 1)) == PK_B2 - 1 || j == n - 1 : (j & (PK_B2 - 1)) == 0;
        if (at1 && deny < 2) {
            const bool two = at2 && deny < 1;
            const int64_t size = two ? PK_B2 : PK_B1, blk = j / size;
            // summaries up to the end of the signal, or of the second-level block
            const int64_t left = two ? (DIR < 0 ? blk + 1 : (n - 1) / size - blk + 1)
                                     : (DIR < 0 ? (blk & (PK_B1 - 1)) + 1
                                                : min((int64_t)PK_B1 - (blk & (PK_B1 - 1)), (n - 1) / size - blk + 1));
            const int cnt = (int)min(left, (int64_t)64);
            const int64_t b = blk + DIR * lane;
            PkSum s{0.0, 0.0, 0, 0};
            if (lane < cnt) s = (two ? s2 : s1)[b];
            const uint64_t m = __ballot(lane < cnt && stop_sum(s, b * size, size));
            const int cut = m ? __ffsll((unsigned long long)m) - 1 : cnt;
            pass(lane < cut ? s.mn : (double)INFINITY, DIR < 0 ? s.last : s.first);
            if (cut > 0) j = DIR < 0 ? (blk - cut + 1) * size - 1 : (blk + cut) * size;
            if (m) deny = two ? 1 : 2;          // go into that block one level down
            else if (cut > 0) deny = 0;
            continue;
        }
        const int64_t left = DIR < 0 ? (j & (PK_B1 - 1)) + 1 : min((int64_t)PK_B1 - (j & (PK_B1 - 1)), n - j);
        const int cnt = (int)min(left, (int64_t)64);
        const int64_t i = j + DIR * lane;
        const double v = lane < cnt ? x[i] : (double)INFINITY;
        const uint64_t m = __ballot(lane < cnt && stop(v, i));
        const int cut = m ? __ffsll((unsigned long long)m) - 1 : cnt;
        pass(lane < cut ? v : (double)INFINITY, i);
        j += DIR * cut;
        if (m) return j;
        if (left == cnt) deny = 0;              // the block is left behind
    }
    return j;
}

// The width of a peak whose walks leave the 64 samples next to it. A prominence walk ends at the first
// strictly higher sample, and the minimum nearest to the peak wins ties; a width walk ends at the first
// sample not above the level, or at the base.
__device__ inline double pk_long_width(const double* __restrict__ x, int64_t n, const PkSum* __restrict__ s1,
                                       const PkSum* __restrict__ s2, int64_t p, double xp) {
    auto higher = [&](double v, int64_t) { return v > xp; };
    auto higher_in = [&](const PkSum& s, int64_t, int64_t) { return s.mx > xp; };
    double low;
    int64_t base;
    auto lowest = [&](double v, int64_t at) {   // lanes in walking order: the first lane of the least value wins
        const double m = wave_min(v);
        if (m < low) {
            low = m;
            base = __shfl(at, __ffsll((unsigned long long)__ballot(v == m)) - 1);
        }
    };
    low = xp; base = p;
    pk_walk<-1>(x, n, s1, s2, p, higher, higher_in, lowest);
    const double lmin = low;
    const int64_t lb = base;
    low = xp; base = p;
    pk_walk<1>(x, n, s1, s2, p, higher, higher_in, lowest);
    const double rmin = low;
    const int64_t rb = base;
    const double prom = xp - (lmin > rmin ? lmin : rmin);
    const double level = xp - prom * 0.5;
    auto ignore = [](double, int64_t) {};
    int64_t i = pk_walk<-1>(x, n, s1, s2, p, [&](double v, int64_t at) { return at <= lb || !(level < v); },
                            [&](const PkSum& s, int64_t b, int64_t) { return b <= lb || !(level < s.mn); }, ignore);
    double left = (double)i;
    if (x[i] < level) left += (level - x[i]) / (x[i + 1] - x[i]);
    i = pk_walk<1>(x, n, s1, s2, p, [&](double v, int64_t at) { return at >= rb || !(level < v); },
                   [&](const PkSum& s, int64_t b, int64_t size) { return b + size > rb || !(level < s.mn); }, ignore);
    double right = (double)i;
    if (x[i] < level) right -= (level - x[i]) / (x[i - 1] - x[i]);
    return right - left;
}

// Step 4: prominence bases and the width at half prominence of each peak (float64, the order of the
// definition), one wave per peak.
__global__ __launch_bounds__(256) void pk_width_kernel(const double* __restrict__ x, int64_t n, const int64_t* __restrict__ cand,
                                                       const int64_t* total, const PkSum* __restrict__ s1,
                                                       const PkSum* __restrict__ s2, double min_width, double* width,
                                                       uint64_t* kmask, int64_t* kcount) {
    const int lane = threadIdx.x & 63;
    const int64_t k = *total, step = (int64_t)gridDim.x * 4;
    for (int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); c < k; c += step) {
        const int64_t p = cand[c];
        // the 64 samples on each side, lane 0 the peak itself: most peaks end all four walks there
        const double vl = x[max(p - lane, (int64_t)0)], vr = x[min(p + lane, n - 1)];
        const double xp = __shfl(vl, 0);
        const uint64_t hl = __ballot(p - lane < 0 || vl > xp), hr = __ballot(p + lane >= n || vr > xp);
        double w;
        if (hl && hr) {   // uniform over the wave
            const int cl = __ffsll((unsigned long long)hl) - 1, cr = __ffsll((unsigned long long)hr) - 1;
            const double lmin = wave_min(lane < cl ? vl : (double)INFINITY), rmin = wave_min(lane < cr ? vr : (double)INFINITY);
            const int bl = __ffsll((unsigned long long)__ballot(lane < cl && vl == lmin)) - 1;
            const int br = __ffsll((unsigned long long)__ballot(lane < cr && vr == rmin)) - 1;
            const double prom = xp - (lmin > rmin ? lmin : rmin);
            const double level = xp - prom * 0.5;
            const int il = __ffsll((unsigned long long)__ballot(lane >= bl || !(level < vl))) - 1;
            const int ir = __ffsll((unsigned long long)__ballot(lane >= br || !(level < vr))) - 1;
            const double xl = __shfl(vl, il), xl1 = __shfl(vl, max(il - 1, 0)), xr = __shfl(vr, ir), xr1 = __shfl(vr, max(ir - 1, 0));
            double left = (double)(p - il), right = (double)(p + ir);
            if (xl < level) left += (level - xl) / (xl1 - xl);
            if (xr < level) right -= (level - xr) / (xr1 - xr);
            w = right - left;
        } else {
            w = pk_long_width(x, n, s1, s2, p, xp);
        }
        if (lane == 0) {
            width[c] = w;
            if (w >= min_width) {
                atomicOr((unsigned long long*)&kmask[c >> 6], 1ull << (c & 63));
                atomicAdd((unsigned long long*)&kcount[c / PK_TILE], 1ull);
            }
        }
    }
}

// Step 5: one block scans the kept counts of the tiles in use; then their ordered list.
__global__ __launch_bounds__(256) void pk_kept_scan_kernel(const int64_t* total, int64_t* kcount, PkHead* head) {
    __shared__ int64_t part[256];
    const int64_t nkt = (*total + PK_TILE - 1) / PK_TILE;
    pk_scan(kcount, nkt, part);
    __syncthreads();
    if (threadIdx.x == 0) head->found = kcount[nkt];
}
__global__ __launch_bounds__(256) void pk_kept_kernel(const int64_t* total, const uint64_t* kmask, const int64_t* kcount,
                                                      const int64_t* cand, const double* width, PkOut* out) {
    const int64_t nkt = (*total + PK_TILE - 1) / PK_TILE;
    for (int64_t tile = blockIdx.x; tile < nkt; tile += gridDim.x)
        pk_each(kmask, kcount, tile, [&](int64_t c, int64_t rank) { out[rank] = PkOut{cand[c], width[c]}; });
}

__global__ __launch_bounds__(256) void prob64_kernel(const float* z, int64_t n, double* p) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step)
        p[i] = 1.0 / (1.0 + exp(-(double)z[i]));
}

// grow-only device workspace of the peak search, shared by all calls of the process
struct PeakWs {
    std::mutex mu;
    void* buf = nullptr;
    int64_t bytes = 0;
    int device = -1;
};
static PeakWs g_pk;

}  // namespace gwd

using namespace gwd;

gwd_status gwd_prob64(const float* z, int64_t n, double* p, void* hip_stream) {
    if (n < 0) { set_error("gwd_prob64: negative n"); return GWD_ERR_ARG; }
    if (n == 0) return GWD_OK;
    if (!z || !p || ((uintptr_t)z & 3) || ((uintptr_t)p & 7)) { set_error("gwd_prob64: NULL or misaligned pointer"); return GWD_ERR_ARG; }
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) { set_error("gwd_prob64: no HIP device"); return GWD_ERR_NO_DEVICE; }
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(prob64_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)hip_stream, z, n, p);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? GWD_OK : hip_fail(e, "prob64 kernel launch");
}

gwd_status gwd_find_peaks(const double* x, int64_t n, double height, double min_width, int64_t* peaks,
                          double* widths, int64_t capacity, int64_t* n_found, void* hip_stream) {
    if (!n_found) { set_error("gwd_find_peaks: n_found is NULL"); return GWD_ERR_ARG; }
    *n_found = 0;
    if (n < 0 || capacity < 0) { set_error("gwd_find_peaks: negative n or capacity"); return GWD_ERR_ARG; }
    if (capacity > 0 && (!peaks || !widths)) { set_error("gwd_find_peaks: NULL output"); return GWD_ERR_ARG; }
    if (std::isnan(height) || std::isnan(min_width)) { set_error("gwd_find_peaks: NaN height or width"); return GWD_ERR_ARG; }
    if (n < 3) return GWD_OK;
    if (!x || ((uintptr_t)x & 7)) { set_error("gwd_find_peaks: NULL or misaligned signal"); return GWD_ERR_ARG; }
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) { set_error("gwd_find_peaks: no HIP device"); return GWD_ERR_NO_DEVICE; }
    hipStream_t st = (hipStream_t)hip_stream;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    // workspace: head and kept peaks [kmax] | edge bits and counts per tile | peaks [kmax] | widths [kmax] |
    // block summaries | kept bits and counts per tile of peaks: 16 bytes per sample, or 8 without room for the
    // kept peaks where the device memory does not hold it (the host then takes them from all peaks and widths)
    const int64_t nt = (n + PK_TILE - 1) / PK_TILE;
    const int64_t kmax = n / 2 + 1, nkt = (kmax + PK_TILE - 1) / PK_TILE;
    const int64_t n1 = (n + PK_B1 - 1) / PK_B1, n2 = (n1 + PK_B1 - 1) / PK_B1;
    int64_t need = 0;
    auto take = [&](int64_t bytes) {
        const int64_t at = need;
        need += (bytes + 15) / 16 * 16;
        return at;
    };
    const int64_t off_out = take((int64_t)sizeof(PkHead) + PK_FIRST * (int64_t)sizeof(PkOut));
    const int64_t off_mask = take(nt * PK_WORDS * 8), off_cnt = take((nt + 1) * 8);
    const int64_t off_cand = take(kmax * 8), off_w = take(kmax * 8);
    const int64_t off_s1 = take(n1 * (int64_t)sizeof(PkSum)), off_s2 = take(n2 * (int64_t)sizeof(PkSum));
    const int64_t off_km = take(nkt * PK_WORDS * 8), off_kc = take((nkt + 1) * 8);
    const int64_t least = need, off_list = take((int64_t)sizeof(PkHead) + std::max<int64_t>(kmax, PK_FIRST) * (int64_t)sizeof(PkOut));
    std::lock_guard<std::mutex> lock(g_pk.mu);
    if (g_pk.bytes < need || g_pk.device != dev) {
        // grown only where there is room: a buffer that does without the list is not given up for a try in vain
        size_t free_b = 0, total_b = 0;
        const bool vain = g_pk.device == dev && g_pk.bytes >= least && hipMemGetInfo(&free_b, &total_b) == hipSuccess &&
                          (int64_t)free_b + g_pk.bytes < need;
        if (!vain) {
            if (g_pk.buf) {
                (void)hipStreamSynchronize(st);
                (void)hipFree(g_pk.buf);
                g_pk.buf = nullptr;
                g_pk.bytes = 0;
            }
            g_pk.device = dev;
            for (int64_t bytes : {need, least}) {
                e = hipMalloc(&g_pk.buf, bytes);
                if (e == hipSuccess) {
                    g_pk.bytes = bytes;
                    break;
                }
                g_pk.buf = nullptr;
                (void)hipGetLastError();   // (the launches after a second try check it)
            }
            if (e != hipSuccess) return hip_fail(e, "hipMalloc(peak workspace)");
        }
    }
    const bool list = g_pk.bytes >= need;
    char* b = (char*)g_pk.buf;
    PkHead* head = (PkHead*)(b + (list ? off_list : off_out));
    PkOut* out = (PkOut*)(head + 1);
    uint64_t *mask = (uint64_t*)(b + off_mask), *kmask = (uint64_t*)(b + off_km);
    int64_t *counts = (int64_t*)(b + off_cnt), *kcount = (int64_t*)(b + off_kc), *cand = (int64_t*)(b + off_cand);
    double* wd = (double*)(b + off_w);
    PkSum *s1 = (PkSum*)(b + off_s1), *s2 = (PkSum*)(b + off_s2);
    hipLaunchKernelGGL(pk_clear_kernel, dim3(1), dim3(64), 0, st, head);
    hipLaunchKernelGGL(pk_pass_kernel, dim3((unsigned)nt), dim3(256), 0, st, x, n, height, mask, counts, s1, head, kmask,
                       kcount, nkt);
    hipLaunchKernelGGL(pk_scan_kernel, dim3((unsigned)(1 + n2)), dim3(256), 0, st, counts, nt, s1, n1, s2);
    hipLaunchKernelGGL(pk_list_kernel, dim3((unsigned)nt), dim3(256), 0, st, x, n, height, mask, counts, cand);
    const unsigned wblocks = (unsigned)std::min<int64_t>(PK_WAVES / 4, (kmax + 3) / 4);
    hipLaunchKernelGGL(pk_width_kernel, dim3(wblocks), dim3(256), 0, st, x, n, cand, counts + nt, s1, s2, min_width, wd,
                       kmask, kcount);
    hipLaunchKernelGGL(pk_kept_scan_kernel, dim3(1), dim3(256), 0, st, counts + nt, kcount, head);
    if (list)
        hipLaunchKernelGGL(pk_kept_kernel, dim3((unsigned)std::min<int64_t>(nkt, 1024)), dim3(256), 0, st, counts + nt, kmask,
                           kcount, cand, wd, out);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "peak kernel launch");
    // the count and the first peaks in one copy, any others in a second one
    struct {
        PkHead head;
        PkOut out[PK_FIRST];
    } first;
    e = hipMemcpyAsync(&first, head, sizeof first, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e, "peak count copy");
    if (first.head.bad) { set_error("gwd_find_peaks: NaN or Inf in the signal"); return GWD_ERR_NONFINITE; }
    const int64_t found = first.head.found, ncopy = std::min(found, capacity);
    std::vector<PkOut> rest;
    std::vector<int64_t> all_p;
    std::vector<double> all_w;
    try {
        if (!list && ncopy > 0) {
            int64_t k = 0;
            e = hipMemcpyAsync(&k, counts + nt, sizeof k, hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipStreamSynchronize(st);
            if (e != hipSuccess) return hip_fail(e, "peak count copy");
            all_p.resize((size_t)k);
            all_w.resize((size_t)k);
            e = hipMemcpyAsync(all_p.data(), cand, k * sizeof(int64_t), hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipMemcpyAsync(all_w.data(), wd, k * sizeof(double), hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipStreamSynchronize(st);
            if (e != hipSuccess) return hip_fail(e, "peak copy");
        } else if (ncopy > PK_FIRST) {
            rest.resize((size_t)(ncopy - PK_FIRST));
            e = hipMemcpyAsync(rest.data(), out + PK_FIRST, rest.size() * sizeof(PkOut), hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipStreamSynchronize(st);
            if (e != hipSuccess) return hip_fail(e, "peak copy");
        }
    } catch (const std::bad_alloc&) {
        set_error("gwd_find_peaks: out of host memory");
        return GWD_ERR_ARG;
    }
    for (int64_t c = 0, i = 0; c < ncopy; ++c, ++i) {
        if (!list)
            while (!(all_w[(size_t)i] >= min_width)) ++i;   // (the device counted ncopy of them)
        const PkOut o = !list ? PkOut{all_p[(size_t)i], all_w[(size_t)i]} : c < PK_FIRST ? first.out[c] : rest[(size_t)(c - PK_FIRST)];
        peaks[c] = o.peak;
        widths[c] = o.width;
    }
    *n_found = found;
    if (found > capacity) { set_error("gwd_find_peaks: %lld peaks, capacity %lld", (long long)found, (long long)capacity); return GWD_ERR_CAPACITY; }
    return GWD_OK;
}

gwd_status gwd_coincidence(const int64_t* const* lists, const int64_t* counts, int32_t n_members, int64_t window,
                           int64_t* events, int64_t capacity, int64_t* n_events) {
    if (!n_events) { set_error("gwd_coincidence: n_events is NULL"); return GWD_ERR_ARG; }
    *n_events = 0;
    if (!lists || !counts || n_members < 1 || window < 0 || capacity < 0 || (capacity > 0 && !events)) {
        set_error("gwd_coincidence: bad argument");
        return GWD_ERR_ARG;
    }
    for (int m = 0; m < n_members; ++m)
        if (counts[m] < 0 || (counts[m] > 0 && !lists[m])) { set_error("gwd_coincidence: bad list %d", m); return GWD_ERR_ARG; }
    int64_t found = 0;
    for (int64_t a = 0; a < counts[0]; ++a) {
        const int64_t t = lists[0][a];
        bool ok = true;
        for (int m = 1; m < n_members && ok; ++m) {
            // the nearest peak of member m: the first at or after t - window
            const int64_t* q = lists[m];
            const int64_t* it = std::lower_bound(q, q + counts[m], t - window);
            ok = it != q + counts[m] && *it <= t + window;
        }
        if (ok) {
            if (found < capacity) events[found] = t;
            ++found;
        }
    }
    *n_events = found;
    if (found > capacity) { set_error("gwd_coincidence: %lld events, capacity %lld", (long long)found, (long long)capacity); return GWD_ERR_CAPACITY; }
    return GWD_OK;
}
