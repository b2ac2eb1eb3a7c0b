// som_update.hip -- gfx950 kernels of the batch-SOM update (Algorithm 2, steps 8-9;
// factorised box-blur update section), for binary rows.
//
// After a search has given every sample its best unit, the update
//   1. scatters the batch onto the E x E lattice: den[i] = samples at unit i and,
//      feature by feature, num[v][i] = samples at unit i holding feature v (integer
//      counts: exact and independent of the order they are taken in). Units that
//      hold many samples (on an untrained codebook a handful of units can take the
//      whole batch) are counted in LDS: their samples are sorted by unit and each
//      workgroup histograms a run of one unit's samples, then adds the non-zero
//      bins to global memory; the other units take one global atomic per feature.
//   2. converts both fields to fp32 and blurs them: three box passes along every
//      lattice row, then three along every lattice column, each a running window
//      sum over the clamped window (the first window summed in ascending order,
//      then per step the element entering added and the one leaving subtracted),
//      unnormalised -- the constant cancels in the quotient;
//   3. replaces every prototype by num / den (fp32 division), clamped to [0, 1] (a
//      mean of 0/1 inputs), leaving a unit unchanged where no sample lies in its
//      neighbourhood; an fp16 codebook receives the quotient rounded once to
//      binary16 at this final write. In exact arithmetic the blurred den is zero
//      exactly where no unit within 3r cells along both axes holds a sample, but
//      fp32 running sums past 2^24 can leave a residual there, so that support is
//      counted separately in whole numbers (k_support) and decides the rule.
// The blur's field is feature-major and held in LDS, a lattice or some of its lines at a
// time, so that it crosses memory once for the counts and the rows and once for the columns
// and the quotient; lattices whose lines are too long for that at a wide window keep their
// fields unit-major (cnt[i][v]; a lane owns one line and neighbouring lanes take
// neighbouring features) and run through memory. Every pass adds and subtracts in the order
// above in all forms, so the result is the same bits on every run and in each of them.
// There the quotient is fused with the one transpose, from the unit-major fields to the
// feature-major codebook. Features are processed in chunks, so the workspace holds three
// fields of chunk * M values rather than V * M.

#include <climits>

#include "../../include/som.h"
#include "som_internal.h"

namespace som {
namespace {

typedef unsigned long long u64;

// A unit with at least kHeavy samples is counted through LDS; kRunSamples sorted
// samples per workgroup there, and kLdsBins feature bins (128 KB) per LDS pass.
constexpr int32_t kHeavy = 1024;
constexpr int64_t kRunSamples = 8192;
constexpr int kLdsBins = 32768;

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }

// Clamped id range of sample s (relative to row_ptr[0]).
__device__ __forceinline__ void sample_ids(const int32_t *row_ptr, int64_t base, int64_t nnz, int64_t s, int64_t &rb,
                                           int64_t &re)
{
    rb = (int64_t)row_ptr[s] - base;
    re = (int64_t)row_ptr[s + 1] - base;
    rb = rb < 0 ? 0 : (rb > nnz ? nnz : rb);
    re = re < rb ? rb : (re > nnz ? nnz : re);
}

// Each wave takes a contiguous range of samples, 64 at a time; kScanBlocks blocks.
constexpr int64_t kScanBlocks = 2048;

__device__ __forceinline__ void wave_range(int64_t N, int64_t &w0, int64_t &w1)
{
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
    const int64_t w = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int64_t per = ((N + waves - 1) / waves + 63) / 64 * 64;
    w0 = w * per < N ? w * per : N;
    w1 = w0 + per < N ? w0 + per : N;
}

// Samples per unit. The lanes of a wave that share a unit add their count with one
// atomic, and a wave carries a unit's count over as long as consecutive samples keep
// it, so a unit that takes most of the batch does not serialise the grid on one
// address.
__global__ __launch_bounds__(256) void k_count_units(const int32_t *__restrict__ bmu, int64_t N, int64_t M,
                                                     int32_t *__restrict__ cnt)
{
    const int lane = lane_id();
    int64_t w0, w1;
    wave_range(N, w0, w1);
    int32_t pu = -1, pn = 0;  // the unit whose count is carried, and the count (wave-uniform)
    for (int64_t s0 = w0; s0 < w1; s0 += 64) {
        const int64_t s = s0 + lane;
        int32_t u = -1;
        if (s < w1) {
            u = bmu[s];
            if (u < 0 || u >= M) u = -1;
        }
        u64 todo = __ballot(u >= 0);
        while (todo) {
            const int leader = __builtin_ctzll(todo);
            const int32_t lu = __builtin_amdgcn_readlane(u, leader);
            const u64 same = __ballot(u == lu) & todo;
            if (lu == pu) {
                pn += (int32_t)__popcll(same);
            } else {
                if (pu >= 0 && lane == 0) atomicAdd(cnt + pu, pn);
                pu = lu;
                pn = (int32_t)__popcll(same);
            }
            todo &= ~same;
        }
    }
    if (pu >= 0 && lane == 0) atomicAdd(cnt + pu, pn);
}

// Samples per unit for maps of at most kLdsUnits units: a histogram in LDS per
// workgroup (1024 threads), then one global atomic per non-zero bin.
constexpr int kLdsUnits = 16384;

__global__ __launch_bounds__(1024) void k_count_units_lds(const int32_t *__restrict__ bmu, int64_t N, int64_t M,
                                                          int32_t *__restrict__ cnt)
{
    __shared__ uint32_t h[kLdsUnits];
    for (int64_t i = threadIdx.x; i < M; i += 1024) h[i] = 0u;
    __syncthreads();
    for (int64_t s = (int64_t)blockIdx.x * 1024 + threadIdx.x; s < N; s += (int64_t)gridDim.x * 1024) {
        const int32_t u = bmu[s];
        if (u >= 0 && u < M) atomicAdd(&h[u], 1u);
    }
    __syncthreads();
    for (int64_t i = threadIdx.x; i < M; i += 1024)
        if (h[i]) atomicAdd(cnt + i, (int32_t)h[i]);
}

// One workgroup: start[u] = number of samples of heavy units below u (heavy: at least
// kHeavy samples), start[M] = all samples of heavy units, start[M + 1] = number of
// heavy units; cursor = start; slot[u] = the heavy unit's rank among heavy units (-1
// for the others) and hunit[slot] = u. Each wave takes a contiguous stretch, 64 units a
// step, eight steps' counts loaded before any is used (one thread walking its stretch
// took 185 us at 65,536 units). Samples and heavy units are scanned as one packed word:
// both totals stay below 2^31.
constexpr int kScanSteps = 8;

__global__ __launch_bounds__(1024) void k_heavy_scan(const int32_t *__restrict__ cnt, int64_t M,
                                                     int32_t *__restrict__ start, int32_t *__restrict__ cursor,
                                                     int32_t *__restrict__ slot, int32_t *__restrict__ hunit)
{
    __shared__ u64 sum[16];
    const int lane = lane_id(), w = threadIdx.x >> 6;
    const int64_t steps = (M + 1023) / 1024;
    const int64_t u0 = w * steps * 64 + lane;
    auto packed = [&](int64_t k) -> u64 {
        const int64_t u = u0 + k * 64;
        const int32_t c = k < steps && u < M ? cnt[u] : 0;
        return c >= kHeavy ? ((u64)(uint32_t)c << 32) | 1ull : 0ull;
    };
    u64 total = 0;
    for (int64_t k0 = 0; k0 < steps; k0 += kScanSteps) {
        u64 x[kScanSteps];
#pragma unroll
        for (int k = 0; k < kScanSteps; ++k) x[k] = packed(k0 + k);
#pragma unroll
        for (int k = 0; k < kScanSteps; ++k) total += x[k];
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) total += __shfl_xor(total, d);
    if (lane == 0) sum[w] = total;
    __syncthreads();
    u64 run = 0;
    for (int q = 0; q < w; ++q) run += sum[q];
    if (threadIdx.x == 1023) {
        start[M] = (int32_t)((run + total) >> 32);
        start[M + 1] = (int32_t)((run + total) & 0xFFFFFFFFull);
    }
    for (int64_t k0 = 0; k0 < steps; k0 += kScanSteps) {
        u64 x[kScanSteps];
#pragma unroll
        for (int k = 0; k < kScanSteps; ++k) x[k] = packed(k0 + k);
#pragma unroll
        for (int k = 0; k < kScanSteps; ++k) {
            const int64_t u = u0 + (k0 + k) * 64;
            u64 before = run;
            if (__ballot(x[k] != 0)) {
                u64 inc = x[k];
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const u64 y = __shfl_up(inc, d);
                    if (lane >= d) inc += y;
                }
                before = run + inc - x[k];
                run += __shfl(inc, 63);
            }
            if (k0 + k < steps && u < M) {
                start[u] = cursor[u] = (int32_t)(before >> 32);
                const int32_t q = (int32_t)(before & 0xFFFFFFFFull);
                slot[u] = x[k] ? q : -1;
                if (x[k]) hunit[q] = (int32_t)u;
            }
        }
    }
}

// order[start[u] ...] = the samples of every heavy unit u, grouped by unit (in any
// order within a unit: the counts do not depend on it). A workgroup (1024 threads)
// takes a contiguous range of samples. With at most kLdsUnits heavy units it counts
// them per heavy unit in LDS, reserves each unit's positions with one global atomic,
// and hands them out from LDS in a second pass over the range. Otherwise each wave
// reserves, per 64 samples, one run of positions per distinct unit.
__global__ __launch_bounds__(1024) void k_heavy_scatter(const int32_t *__restrict__ bmu, int64_t N, int64_t M,
                                                        const int32_t *__restrict__ start,
                                                        const int32_t *__restrict__ slot,
                                                        const int32_t *__restrict__ hunit, int32_t *__restrict__ cursor,
                                                        int32_t *__restrict__ order)
{
    __shared__ int32_t h[kLdsUnits];
    const int64_t per = (N + gridDim.x - 1) / gridDim.x;
    const int64_t b0 = (int64_t)blockIdx.x * per < N ? (int64_t)blockIdx.x * per : N;
    const int64_t b1 = b0 + per < N ? b0 + per : N;
    const int32_t heavy = start[M + 1];
    auto slot_of = [&](int64_t s) {
        const int32_t u = bmu[s];
        return u >= 0 && u < M ? slot[u] : -1;
    };
    if (heavy <= kLdsUnits) {  // uniform
        for (int i = threadIdx.x; i < heavy; i += 1024) h[i] = 0;
        __syncthreads();
        for (int64_t s = b0 + threadIdx.x; s < b1; s += 1024) {
            const int32_t k = slot_of(s);
            if (k >= 0 && k < heavy) atomicAdd(&h[k], 1);
        }
        __syncthreads();
        for (int i = threadIdx.x; i < heavy; i += 1024)
            if (h[i]) h[i] = atomicAdd(cursor + hunit[i], h[i]);
        __syncthreads();
        for (int64_t s = b0 + threadIdx.x; s < b1; s += 1024) {
            const int32_t k = slot_of(s);
            if (k >= 0 && k < heavy) order[atomicAdd(&h[k], 1)] = (int32_t)s;
        }
        return;
    }
    const int lane = lane_id();
    const u64 below = (1ull << lane) - 1ull;
    const int64_t wb = b0 + (int64_t)(threadIdx.x >> 6) * 64;
    for (int64_t s0 = wb; s0 < b1; s0 += 1024) {
        const int64_t s = s0 + lane;
        int32_t u = -1;
        if (s < b1) {
            u = bmu[s];
            if (u < 0 || u >= M || slot[u] < 0) u = -1;
        }
        u64 todo = __ballot(u >= 0);
        while (todo) {
            const int leader = __builtin_ctzll(todo);
            const int32_t lu = __builtin_amdgcn_readlane(u, leader);
            const u64 same = __ballot(u == lu) & todo;
            int32_t at = 0;
            if (lane == leader) at = atomicAdd(cursor + lu, (int32_t)__popcll(same));
            at = __builtin_amdgcn_readlane(at, leader);
            if ((same >> lane) & 1ull) order[at + __popcll(same & below)] = (int32_t)s;
            todo &= ~same;
        }
    }
}

// Where unit u's count of feature v0 + w lies in a field: u * su + w * sw. Unit-major
// fields (su = features, sw = 1) serve k_blur3, feature-major ones (su = 1, sw = M) the
// kernels that hold a lattice or its lines in LDS.
struct Field {
    int64_t su, sw;
    __device__ int64_t at(int64_t u, int64_t w) const { return u * su + w * sw; }
};

// cnt[u][v - v0] += 1 for every id v in [v0, v1) of every sample whose unit is not heavy;
// the four lanes of a quad share a sample.
__global__ __launch_bounds__(256) void k_count_light(const int32_t *__restrict__ row_ptr,
                                                     const int32_t *__restrict__ col_idx, int64_t N, int64_t nnz,
                                                     const int32_t *__restrict__ bmu, int64_t M,
                                                     const int32_t *__restrict__ units, int32_t v0, int32_t v1,
                                                     int32_t *__restrict__ cnt, Field fd,
                                                     const uint32_t *__restrict__ flags)
{
    if (flags[0] & SOM_FLAG_ROW_PTR) return;  // invalid row pointers: no row is read
    const int64_t base = row_ptr[0];           // >= 0 once the row pointers passed the check
    const int sub = threadIdx.x & 3;
    for (int64_t s = (int64_t)blockIdx.x * 64 + (threadIdx.x >> 2); s < N; s += (int64_t)gridDim.x * 64) {
        const int32_t u = bmu[s];
        if (u < 0 || u >= M || units[u] >= kHeavy) continue;
        int64_t rb, re;
        sample_ids(row_ptr, base, nnz, s, rb, re);
        for (int64_t p = rb + sub; p < re; p += 16) {
            int32_t id[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) id[j] = p + 4 * j < re ? col_idx[base + p + 4 * j] : -1;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (id[j] >= v0 && id[j] < v1) atomicAdd(cnt + fd.at(u, id[j] - v0), 1);
        }
    }
}

// Heavy units: workgroup b takes the sorted positions [b * kRunSamples, ...) of
// order; each run of one unit's samples in that range is histogrammed in LDS, in
// passes of kLdsBins features, and the non-zero bins are added to cnt[u][.]. Sixteen waves,
// a quad of lanes per sample, one pass for up to 32,768 features (before: four waves, a
// lane per sample, 16,384 samples and features: 64 x 64 map, 1.6 M samples on eight units
// 932 -> 215 us).
__global__ __launch_bounds__(1024) void k_count_heavy(const int32_t *__restrict__ row_ptr,
                                                      const int32_t *__restrict__ col_idx, int64_t nnz,
                                                      const int32_t *__restrict__ bmu, int64_t M,
                                                      const int32_t *__restrict__ units,
                                                      const int32_t *__restrict__ start,
                                                      const int32_t *__restrict__ order, int32_t v0, int32_t v1,
                                                      int32_t *__restrict__ cnt, Field fd,
                                                      const uint32_t *__restrict__ flags)
{
    __shared__ uint32_t hist[kLdsBins];
    if (flags[0] & SOM_FLAG_ROW_PTR) return;  // uniform: invalid row pointers, no row is read
    const int64_t base = row_ptr[0];           // >= 0 once the row pointers passed the check
    const int64_t total = start[M];
    const int64_t p0 = (int64_t)blockIdx.x * kRunSamples;
    if (p0 >= total) return;  // uniform
    const int64_t p1 = p0 + kRunSamples < total ? p0 + kRunSamples : total;
    const int sub = threadIdx.x & 3;
    for (int64_t p = p0; p < p1;) {  // uniform: every thread reads the same run bounds
        const int32_t u = bmu[order[p]];
        int64_t re = p + 1;
        if (u >= 0 && u < M) {
            const int64_t end = (int64_t)start[u] + units[u];
            re = end < p1 ? end : p1;
            if (re <= p) re = p + 1;
        }
        if (u >= 0 && u < M) {
            for (int64_t h0 = v0; h0 < v1; h0 += kLdsBins) {
                const int hb = (int)((int64_t)v1 - h0 < kLdsBins ? (int64_t)v1 - h0 : kLdsBins);
                for (int b = threadIdx.x; b < hb; b += 1024) hist[b] = 0u;
                __syncthreads();
                for (int64_t q = p + (threadIdx.x >> 2); q < re; q += 256) {
                    int64_t rb, rend;
                    sample_ids(row_ptr, base, nnz, order[q], rb, rend);
                    for (int64_t k = rb + sub; k < rend; k += 16) {
                        int64_t id[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) id[j] = k + 4 * j < rend ? col_idx[base + k + 4 * j] : -1;
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (id[j] >= h0 && id[j] < h0 + hb) atomicAdd(&hist[id[j] - h0], 1u);
                    }
                }
                __syncthreads();
                for (int b = threadIdx.x; b < hb; b += 1024) {
                    const uint32_t c = hist[b];
                    if (c) atomicAdd(cnt + fd.at(u, h0 - v0 + b), (int32_t)c);
                }
                __syncthreads();
            }
        }
        p = re;
    }
}

// Three running-sum box passes of half-width r along lines of n values, `stride`
// apart, in one sweep of each line. Pass k+1 takes every value of pass k as pass k
// produces it -- that is the value entering pass k+1's window -- and reads the value
// leaving its window back from where pass k stored it (x holds pass 1's output, y
// pass 2's). Each pass is still exactly the oracle's sequence of fp32 operations: its
// first window summed in ascending order, then per step the entering value added and
// the leaving one subtracted. Per element that is four reads and three writes, where
// three separate passes take six reads and three writes.
// in holds the first pass's input as 32-bit words: integer counts (INT) or float
// bits. out receives the third pass as float bits and may be in itself: out[i] is
// written once pass 1 has gone past i + 2m (m = min(r, n - 1)), after its last read
// of in[i] at i + r + 1. The words are read and written through one type, so no
// access to in and out can be reordered across another.
// Fields are unit-major: element (r, c) of feature v is at (r * E + c) * f + v. Line
// l is feature v = l % f of the line k = l / f and starts at k * outer + v;
// neighbouring lanes take neighbouring features, so every step is one coalesced
// access per lane group. Row passes (along c): outer = E * f, stride = f; column
// passes (along r): outer = f, stride = E * f. The lines of different lanes are
// disjoint.
template <bool INT>
__global__ __launch_bounds__(256) void k_blur3(const uint32_t *in, float *x, float *y, uint32_t *out, int64_t lines,
                                               int64_t f, int64_t outer, int64_t n, int64_t stride, int64_t r)
{
    for (int64_t l = (int64_t)blockIdx.x * 256 + threadIdx.x; l < lines; l += (int64_t)gridDim.x * 256) {
        const int64_t off = (l / f) * outer + l % f;
        const uint32_t *src = in + off;
        float *px = x + off, *py = y + off;
        uint32_t *dst = out + off;
        auto input = [&](int64_t k) {
            const uint32_t u = src[k * stride];
            return INT ? (float)(int32_t)u : __uint_as_float(u);
        };
        const int64_t m = r < n - 1 ? r : n - 1;  // the first window is [0, m]
        float s1 = 0.0f, s2 = 0.0f;
        int64_t next1 = 0, next2 = 0;  // the next output index of passes 2 and 3
        // pass 3 receives pass 2's output j
        auto feed2 = [&](int64_t j, float v) {
            py[j * stride] = v;
            s2 += v;
            if (j >= m) {  // output i = j - m: its first window is complete, or v entered at i + r
                const int64_t i = j - m;
                if (i - r - 1 >= 0) s2 -= py[(i - r - 1) * stride];
                dst[i * stride] = __float_as_uint(s2);
                next2 = i + 1;
            }
        };
        // pass 2 receives pass 1's output j
        auto feed1 = [&](int64_t j, float v) {
            px[j * stride] = v;
            s1 += v;
            if (j >= m) {
                const int64_t i = j - m;
                if (i - r - 1 >= 0) s1 -= px[(i - r - 1) * stride];
                feed2(i, s1);
                next1 = i + 1;
            }
        };
        // pass 1
        float s0 = 0.0f;
        for (int64_t k = 0; k <= m; ++k) s0 += input(k);
        feed1(0, s0);
        for (int64_t i = 1; i < n; ++i) {
            if (i + r < n) s0 += input(i + r);
            if (i - r - 1 >= 0) s0 -= input(i - r - 1);
            feed1(i, s0);
        }
        // passes 2 and 3 past the last entering value: only leaving values remain
        for (int64_t i = next1; i < n; ++i) {
            if (i - r - 1 >= 0) s1 -= px[(i - r - 1) * stride];
            feed2(i, s1);
        }
        for (int64_t i = next2; i < n; ++i) {
            if (i - r - 1 >= 0) s2 -= py[(i - r - 1) * stride];
            dst[i * stride] = __float_as_uint(s2);
        }
    }
}

// ---- blur in LDS
//
// The same three passes per line with the line held in LDS, so the field crosses memory
// once per kernel instead of seven times per axis. A pass reads its input at one offset
// along the line and writes its output at another: half-width r, d = min(r, n - 1) + 1;
// either d slots lower (output i takes the slot of input i - d, the value that leaves the
// window at i and is not read again, so three passes need n + 3 d slots) or on the other of
// two stretches of n. The batches of line_pass read before they write, so both are safe.
//
// What bounds these kernels: instruction issue and LDS latency at one to three waves per
// SIMD (LDS holds no more lines); so a pass has no branch or select per step, and words
// find their LDS place by additions.

// Threads a workgroup: the passes take one per line, the words' way in and out takes all (a
// workgroup of one wave per 64 lines spent two thirds of its time there).
constexpr int kBlurThreads = 256;

// Steps lo ... hi - 1 in batches of 16, then 8, 4, 2, 1: body(first step, StaticInt<batch>).
template <int N>
struct StaticInt {
    static constexpr int value = N;
};

template <typename F>
__device__ __forceinline__ void in_batches(int lo, int hi, F &&body)
{
    int i = lo;
    for (; i + 16 <= hi; i += 16) body(i, StaticInt<16>{});
    const int rest = hi - i;
    if (rest <= 0) return;
    if (rest & 8) body(i, StaticInt<8>{}), i += 8;
    if (rest & 4) body(i, StaticInt<4>{}), i += 4;
    if (rest & 2) body(i, StaticInt<2>{}), i += 2;
    if (rest & 1) body(i, StaticInt<1>{});
}

// One running-sum pass over n values at x[k * step], results at y[k * step]: outputs whose
// window grows (a value enters, none leaves), slides, or shrinks -- or, for r >= n / 2,
// stands still in between -- each in batches that read all their values before they write.
// ENTER and LEAVE absent leave the sum as it is, as adding a zero would.
__device__ __forceinline__ void line_pass(const float *x, float *y, int n, int r, int step)
{
    const int m = r < n - 1 ? r : n - 1;  // the first window is [0, m]
    float s = 0.0f;
    in_batches(0, m + 1, [&](int k, auto b) {
        constexpr int B = decltype(b)::value;
        float v[B];
#pragma unroll
        for (int u = 0; u < B; ++u) v[u] = x[(k + u) * step];
#pragma unroll
        for (int u = 0; u < B; ++u) s += v[u];
    });
    auto run = [&](int lo, int hi, auto enter, auto leave) {
        in_batches(lo, hi, [&](int i, auto b) {
            constexpr int B = decltype(b)::value;
            constexpr bool ENTER = decltype(enter)::value != 0, LEAVE = decltype(leave)::value != 0;
            float in[B], out[B];
            const float *a = x + (i + r) * step, *z = x + (i - r - 1) * step;
            if constexpr (ENTER)
#pragma unroll
                for (int u = 0; u < B; ++u) in[u] = a[u * step];
            if constexpr (LEAVE)
#pragma unroll
                for (int u = 0; u < B; ++u) out[u] = z[u * step];
            float v[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                if constexpr (ENTER) s += in[u];
                if constexpr (LEAVE) s -= out[u];
                v[u] = s;
            }
            float *to = y + i * step;
#pragma unroll
            for (int u = 0; u < B; ++u) to[u * step] = v[u];
        });
    };
    const int last = n - 1 - m;  // outputs up to here take a value in; those past m lose one
    y[0] = s;
    run(1, (last < m ? last : m) + 1, StaticInt<1>{}, StaticInt<0>{});
    if (m < last)
        run(m + 1, last + 1, StaticInt<1>{}, StaticInt<1>{});
    else
        run(last + 1, m + 1, StaticInt<0>{}, StaticInt<0>{});
    run((m > last ? m : last) + 1, n, StaticInt<0>{}, StaticInt<1>{});
}

// The three passes of a line at a small half-width R, in one sweep with the windows in
// registers: each value of pass k is pass k + 1's entering value as soon as it is formed,
// and leaves its window 2R + 1 values later, from a register (the steps are unrolled by a
// multiple of 2R + 1, so that is always the same one). A value off the line is +0, which
// leaves a sum as it is, and so is a pass's output off the line (EDGE: the blocks of steps
// in which that can happen). read(t): value t of the line, t < n; write(i, v): result i, in
// order, after value i + 3R was read (or the line's last).
constexpr int kRegRadius = 8;

template <int R>
struct Passes3 {
    static constexpr int kWin = 2 * R + 1;
    static constexpr int kStep = kWin >= 9 ? kWin : (kWin == 7 ? 14 : (kWin == 5 ? 10 : 9));  // steps a block
    float x[kWin], a[kWin], b[kWin];
    float s1, s2, s3;

    template <bool EDGE, typename Read, typename Write>
    __device__ __forceinline__ void block(int t0, int n, const Read &read, const Write &write)
    {
        float v[kStep];
#pragma unroll
        for (int u = 0; u < kStep; ++u) v[u] = EDGE && t0 + u >= n ? 0.0f : read(t0 + u);
        float y[kStep];
#pragma unroll
        for (int u = 0; u < kStep; ++u) {
            constexpr int W = kWin;
            const int t = t0 + u;
            // slot u % W holds the value that entered 2R + 1 steps ago; passes 2 and 3 run R
            // and 2R steps behind, on slots of their own
            s1 += v[u];
            s1 -= x[u % W];
            x[u % W] = v[u];
            const float p = !EDGE || (t >= R && t - R < n) ? s1 : 0.0f;
            s2 += p;
            s2 -= a[u % W];
            a[u % W] = p;
            const float q = !EDGE || (t >= 2 * R && t - 2 * R < n) ? s2 : 0.0f;
            s3 += q;
            s3 -= b[u % W];
            b[u % W] = q;
            y[u] = s3;
        }
#pragma unroll
        for (int u = 0; u < kStep; ++u) {
            const int i = t0 + u - 3 * R;
            if (!EDGE || (i >= 0 && i < n)) write(i, y[u]);
        }
    }

    template <typename Read, typename Write>
    __device__ __forceinline__ void run(int n, const Read &read, const Write &write)
    {
#pragma unroll
        for (int u = 0; u < kWin; ++u) x[u] = a[u] = b[u] = 0.0f;
        s1 = s2 = s3 = 0.0f;
        for (int t0 = 0; t0 < n + 3 * R; t0 += kStep) {
            if (t0 >= 3 * R && t0 + kStep <= n)
                block<false>(t0, n, read, write);
            else
                block<true>(t0, n, read, write);
        }
    }
};

// The same between memory stretches of the line (step words apart); y may be x.
template <int R>
__device__ __forceinline__ void line_pass3(const float *x, float *y, int n, int step)
{
    Passes3<R> p;
    p.run(n, [&](int t) { return x[t * step]; }, [&](int i, float v) { y[i * step] = v; });
}

// Offsets of a line's three passes (rows and columns alike); see above.
struct LinePlan {
    int slots;    // per line
    int off[4];   // where the input of passes 1, 2 and 3 and the result start
};

inline LinePlan line_plan(int64_t n, int64_t r)
{
    const int d = (int)(r < n - 1 ? r : n - 1) + 1;
    if (3 * d <= n) return LinePlan{(int)n + 3 * d, {3 * d, 2 * d, d, 0}};
    return LinePlan{2 * (int)n, {0, (int)n, 0, (int)n}};
}

// num / den, clamped to [0, 1] (fp32; rounded once to binary16 for an fp16 codebook).
template <typename E>
__device__ __forceinline__ E quotient(float num, float den)
{
    return (E)fminf(fmaxf(num / den, 0.0f), 1.0f);
}

// The words of a lattice (rows of n) as a workgroup of T threads visits them, word t, t + T,
// ...: LDS places follow by additions from the one before. MANY: of several lattices one after
// the other, `words` places apart, with the unit each word belongs to.
template <bool MANY>
struct Walk {
    int c, at;          // column, place (row * pitch + column)
    int dc, dat, wrap;  // per step: columns and places on; a place more per row begun early
    int n;
    int r, dr, gap;     // MANY: row, rows on per step, places left out between lattices
    __device__ Walk(int t, int T, int n_, int pitch, int words) : n(n_)
    {
        c = t % n;
        at = t / n * pitch + c;
        dc = T % n;
        dat = T / n * pitch + dc;
        wrap = pitch - n;
        if constexpr (MANY) {
            gap = words - n * pitch;
            r = t / n % n;
            at += t / (n * n) * gap;
            dr = T / n % n;
            dat += T / (n * n) * gap;
        }
    }
    __device__ int unit() const { return r * n + c; }  // of the word next() is about to give
    __device__ int next()
    {
        const int place = at;
        c += dc;
        at += dat;
        const bool over = c >= n;
        c -= over ? n : 0;
        at += over ? wrap : 0;
        if constexpr (MANY) {
            r += dr + (over ? 1 : 0);
            const bool past = r >= n;  // once at most: dr < n
            r -= past ? n : 0;
            at += past ? gap : 0;
        }
        return place;
    }
};

// words words of src (integer counts) to LDS, LOADS per thread in flight; and back out of
// LDS: quotients by den (units without a positive den keep what they have) or, for DEN,
// the floats themselves.
template <int LOADS, bool MANY = false>
__device__ __forceinline__ void stage_in(const int32_t *src, float *lat, int words, int t, int T, int n, int pitch,
                                         int apart = 0)
{
    Walk<MANY> w(t, T, n, pitch, apart);
    for (int k0 = t; k0 < words; k0 += T * LOADS) {
        int32_t x[LOADS];
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            const int k = k0 + u * T;
            x[u] = src[k < words ? k : words - 1];
        }
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            const int at = w.next();
            if (k0 + u * T < words) lat[at] = (float)x[u];
        }
    }
}

template <typename E, bool DEN, int LOADS, bool MANY = false>
__device__ __forceinline__ void stage_out(E *W, const float *lat, const float *den, int words, int t, int T, int n,
                                          int pitch, int apart = 0)
{
    Walk<MANY> w(t, T, n, pitch, apart);
    for (int k0 = t; k0 < words; k0 += T * LOADS) {
        float d[LOADS], x[LOADS];
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            const int k = k0 + u * T;
            if constexpr (!DEN) d[u] = k < words ? den[MANY ? w.unit() : k] : 0.0f;
            const int at = w.next();
            x[u] = k < words ? lat[at] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            const int k = k0 + u * T;
            if constexpr (DEN) {
                if (k < words) W[k] = (E)x[u];
            } else {
                if (d[u] > 0.0f) W[k] = quotient<E>(x[u], d[u]);
            }
        }
    }
}

// Lattices that fit LDS: the whole update of `per` features a workgroup -- counts read once
// (coalesced), six passes, quotients written once. A thread owns one
// row, then one column, of one feature. Words of feature q: (k + R[s]) * pitch + c + C[s] at
// stage s (input of pass s + 1; s = 6 the result), pitch odd, so rows and columns are both
// read without bank conflicts.
struct LatticePlan {
    int per, pitch, words;  // features a workgroup, words a lattice row and a feature
    int R[7], C[7];
};

template <typename E, bool DEN, int R, bool MANY>
__global__ __launch_bounds__(kBlurThreads) void k_lattice(const int32_t *__restrict__ cnt, E *__restrict__ W,
                                                 const float *__restrict__ den, int n, int r, int64_t f, int64_t v0,
                                                 LatticePlan lp, const uint32_t *__restrict__ flags)
{
    extern __shared__ float lat[];
    if (flags[0] & SOM_FLAG_ROW_PTR) return;  // uniform: invalid row pointers leave the codebook as it is
    const int M = n * n;
    constexpr int threads = kBlurThreads;
    const int t = threadIdx.x;
    const int line = t % n, q = t / n;  // this thread's line and feature
    for (int64_t w0 = (int64_t)blockIdx.x * lp.per; w0 < f; w0 += (int64_t)gridDim.x * lp.per) {
        const int here = (int)(f - w0 < lp.per ? f - w0 : lp.per);
        float *first = lat + lp.R[0] * lp.pitch + lp.C[0], *last = lat + lp.R[6] * lp.pitch + lp.C[6];
        stage_in<MANY ? 8 : 16, MANY>(cnt + w0 * M, first, here * M, t, threads, n, lp.pitch, lp.words);
        __syncthreads();
        if (q < here) {
            float *a = lat + q * lp.words + line * lp.pitch;
            if constexpr (R > 0)
                line_pass3<R>(a, a, n, 1);
            else
                for (int s = 0; s < 3; ++s)
                    line_pass(a + lp.R[s] * lp.pitch + lp.C[s], a + lp.R[s + 1] * lp.pitch + lp.C[s + 1], n, r, 1);
        }
        __syncthreads();
        if (q < here) {
            float *a = lat + q * lp.words + line;
            if constexpr (R > 0)
                line_pass3<R>(a, a, n, lp.pitch);
            else
                for (int s = 3; s < 6; ++s)
                    line_pass(a + lp.R[s] * lp.pitch + lp.C[s], a + lp.R[s + 1] * lp.pitch + lp.C[s + 1], n, r, lp.pitch);
        }
        __syncthreads();
        stage_out<E, DEN, 8, MANY>(W + (v0 + w0) * M, last, den, here * M, t, threads, n, lp.pitch, lp.words);
        __syncthreads();
    }
}

// Larger lattices, rows: a workgroup takes `lines` consecutive rows of the
// field (rows of all features follow one another), three passes, and writes them where
// they were (or to out).
template <int R>
__global__ __launch_bounds__(kBlurThreads) void k_rows3(const int32_t *cnt, float *out, int n, int r, int64_t rows, int lines,
                                              int pitch, LinePlan lp)
{
    extern __shared__ float lat[];
    const int lane = threadIdx.x;
    for (int64_t g0 = (int64_t)blockIdx.x * lines; g0 < rows; g0 += (int64_t)gridDim.x * lines) {
        const int here = (int)(rows - g0 < lines ? rows - g0 : lines);
        stage_in<16>(cnt + g0 * n, lat + lp.off[0], here * n, lane, kBlurThreads, n, pitch);
        __syncthreads();
        if (lane < here) {
            float *a = lat + lane * pitch;
            if constexpr (R > 0)
                line_pass3<R>(a, a, n, 1);
            else
                for (int s = 0; s < 3; ++s) line_pass(a + lp.off[s], a + lp.off[s + 1], n, r, 1);
        }
        __syncthreads();
        stage_out<float, true, 8>(out + g0 * n, lat + lp.off[3], nullptr, here * n, lane, kBlurThreads, n, pitch);
        __syncthreads();
    }
}

// Larger lattices, columns: a workgroup takes `lines` neighbouring columns of
// one feature, three passes, and writes the quotients.
template <typename E, bool DEN>
__global__ __launch_bounds__(kBlurThreads) void k_cols3(const float *__restrict__ num, E *__restrict__ W,
                                              const float *__restrict__ den, int n, int r, int64_t f, int64_t v0,
                                              int lines, LinePlan lp, const uint32_t *__restrict__ flags)
{
    extern __shared__ float lat[];
    if (flags[0] & SOM_FLAG_ROW_PTR) return;  // uniform: invalid row pointers leave the codebook as it is
    const int lane = threadIdx.x;
    const int tiles = (n + lines - 1) / lines;
    const int col = lane % lines, first = lane / lines, per = kBlurThreads / lines;  // lattice rows at once
    const int64_t M = (int64_t)n * n;
    for (int64_t g = blockIdx.x; g < f * tiles; g += gridDim.x) {
        const int64_t w = g / tiles;
        const int c0 = (int)(g % tiles) * lines;
        const bool in = c0 + col < n;
        const float *src = num + w * M + (in ? c0 + col : n - 1);
        constexpr int kLoads = 16;
        for (int k0 = first; k0 < n; k0 += per * kLoads) {
            float x[kLoads];
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                const int k = k0 + u * per;
                x[u] = src[(k < n ? k : n - 1) * n];
            }
            float *to = lat + (k0 + lp.off[0]) * lines + col;
#pragma unroll
            for (int u = 0; u < kLoads; ++u)
                if (k0 + u * per < n) to[u * per * lines] = x[u];
        }
        __syncthreads();
        if (lane < lines && in)
            for (int s = 0; s < 3; ++s)
                line_pass(lat + lp.off[s] * lines + lane, lat + lp.off[s + 1] * lines + lane, n, r, lines);
        __syncthreads();
        E *out = W + (v0 + w) * M + c0 + col;
        const float *dp = den + c0 + col;
        constexpr int kStores = 8;
        if (in)
            for (int k0 = first; k0 < n; k0 += per * kStores) {
                float x[kStores], d[kStores];
                const float *from = lat + (k0 + lp.off[3]) * lines + col;
#pragma unroll
                for (int u = 0; u < kStores; ++u) {
                    const int k = k0 + u * per;
                    if constexpr (!DEN) d[u] = k < n ? dp[k * n] : 0.0f;
                    x[u] = k < n ? from[u * per * lines] : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < kStores; ++u) {
                    const int k = k0 + u * per;
                    if constexpr (DEN) {
                        if (k < n) out[k * n] = (E)x[u];
                    } else {
                        if (d[u] > 0.0f) out[k * n] = quotient<E>(x[u], d[u]);
                    }
                }
            }
        __syncthreads();
    }
}

// The same at a small half-width, straight from memory: a thread per column, the windows in
// registers, each value of the field read once.
template <typename E, bool DEN, int R>
__global__ __launch_bounds__(kBlurThreads) void k_cols3_small(const float *__restrict__ num, E *__restrict__ W,
                                                              const float *__restrict__ den, int n, int64_t f,
                                                              int64_t v0, const uint32_t *__restrict__ flags)
{
    if (flags[0] & SOM_FLAG_ROW_PTR) return;  // uniform: invalid row pointers leave the codebook as it is
    const int64_t M = (int64_t)n * n;
    for (int64_t l = (int64_t)blockIdx.x * kBlurThreads + threadIdx.x; l < f * n;
         l += (int64_t)gridDim.x * kBlurThreads) {
        const int64_t w = l / n;
        const int c = (int)(l - w * n);
        const float *src = num + w * M + c;
        E *out = W + (v0 + w) * M + c;
        const float *dp = den + c;
        Passes3<R> p;
        p.run(n, [&](int t) { return src[t * n]; },
              [&](int i, float v) {
                  if constexpr (DEN) {
                      out[i * n] = (E)v;
                  } else {
                      const float d = dp[i * n];
                      if (d > 0.0f) out[i * n] = quotient<E>(v, d);
                  }
              });
    }
}

// Occupied units counted over windows of half-width R along lattice lines: rows (in = the
// den counts, counted where > 0; out[r][c] = occupied units in row r within R of column c),
// then columns (in = the row counts, summed): a unit with none in reach gets den 0, which
// leaves its prototype as it is. Whole numbers, exact, so a window is the
// difference of two prefix sums: a workgroup per line, its prefix sums in LDS (a lane walking
// a whole line took 116 us at 256 x 256).
constexpr int kMaxEdge = 1024;
static_assert((int64_t)kMaxEdge * kMaxEdge >= SOM_MAX_NEURONS, "a lattice line fits the LDS prefix sums");

__global__ __launch_bounds__(256) void k_support(const int32_t *__restrict__ in, int32_t *__restrict__ out,
                                                 float *__restrict__ den, int64_t E, int64_t R, int rows)
{
    __shared__ int32_t pre[kMaxEdge + 1], part[256];
    const int t = threadIdx.x, n = (int)E;
    const int64_t first = rows ? (int64_t)blockIdx.x * E : blockIdx.x, step = rows ? 1 : E;
    const int per = (n + 255) / 256;
    int32_t x[kMaxEdge / 256];
    int32_t own = 0;
#pragma unroll
    for (int u = 0; u < kMaxEdge / 256; ++u) {
        const int j = t * per + u;
        const int32_t v = u < per && j < n ? in[first + j * step] : 0;
        x[u] = rows ? (v > 0 ? 1 : 0) : v;
        own += x[u];
    }
    part[t] = own;
    __syncthreads();
    for (int d = 1; d < 256; d <<= 1) {
        const int32_t a = t >= d ? part[t - d] : 0;
        __syncthreads();
        part[t] += a;
        __syncthreads();
    }
    int32_t run = part[t] - own;
#pragma unroll
    for (int u = 0; u < kMaxEdge / 256; ++u) {
        const int j = t * per + u;
        if (u < per && j < n) pre[j] = run;  // sum of the values before j
        run += x[u];
    }
    if (t == 255) pre[n] = part[255];
    __syncthreads();
    for (int i = t; i < n; i += 256) {
        const int64_t hi = i + R + 1 < n ? i + R + 1 : n, lo = i - R > 0 ? i - R : 0;
        const int32_t units = pre[hi] - pre[lo];
        if (rows) out[first + i * step] = units;
        else if (units <= 0) den[first + i * step] = 0.0f;
    }
}

// W[v0 + v][i] = num[i][v] / den[i], clamped to [0, 1], where den[i] > 0, unchanged
// elsewhere: the quotient fused with the transpose from unit-major to feature-major, in
// 64 (units) x 64 (features) tiles through LDS.
template <typename E>
__global__ __launch_bounds__(256) void k_quotient_t(E *__restrict__ W, const float *__restrict__ num,
                                                    const float *__restrict__ den, int64_t f, int64_t M, int64_t v0,
                                                    const uint32_t *__restrict__ flags)
{
    __shared__ float tile[64][65];
    if (flags[0] & SOM_FLAG_ROW_PTR) return;  // uniform: invalid row pointers leave the codebook as it is
    const int64_t it = (M + 63) / 64, vt = (f + 63) / 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;  // 64 x 4 threads
    for (int64_t t = blockIdx.x; t < it * vt; t += gridDim.x) {
        const int64_t i0 = (t / vt) * 64, w0 = (t % vt) * 64;
        for (int y = ty; y < 64; y += 4)
            if (i0 + y < M && w0 + tx < f) tile[y][tx] = num[(i0 + y) * f + w0 + tx];
        __syncthreads();
        if (i0 + tx < M) {
            const float d = den[i0 + tx];
            if (d > 0.0f)
                for (int y = ty; y < 64; y += 4)
                    if (w0 + y < f) W[(v0 + w0 + y) * M + i0 + tx] = quotient<E>(tile[tx][y], d);
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_zero_i32(int32_t *__restrict__ p, int64_t n)
{
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256) p[k] = 0;
}

unsigned grid_for(int64_t n)
{
    int64_t b = (n + 255) / 256;
    if (b < 1) b = 1;
    if (b > (1 << 20)) b = 1 << 20;
    return (unsigned)b;
}

// The blur of f unit-major lattices (E x E) of counts: three row passes, then three
// column passes, with a and b as the passes' scratch. Result in out (fp32), which
// may be the counts themselves.
void blur(const int32_t *cnt, float *a, float *b, float *out, int64_t f, int64_t E, int64_t r, hipStream_t st)
{
    const unsigned g = grid_for(f * E);
    const uint32_t *in = reinterpret_cast<const uint32_t *>(cnt);
    uint32_t *o = reinterpret_cast<uint32_t *>(out);
    hipLaunchKernelGGL(k_blur3<true>, dim3(g), dim3(256), 0, st, in, a, b, o, f * E, f, E * f, E, f, r);
    hipLaunchKernelGGL(k_blur3<false>, dim3(g), dim3(256), 0, st, o, a, b, o, f * E, f, f, E, E * f, r);
}

constexpr int kLdsBytes = 160 * 1024;  // of a compute unit

// Lattices of up to kManyEdge cells share workgroups, where half-widths past kManyRadius have no
// windows in registers (a line of 21 r cells is too long), while there are kSpreadFeatures
// features for each (36 x 36, 200 features: 50 us shared, 47 spread).
constexpr int kManyEdge = 48, kManyRadius = 2, kSpreadFeatures = 512;
static_assert(kManyEdge < 21 * (kManyRadius + 1), "see blur_plan");

// How the blur runs at edge E and half-width r: whole lattices in LDS, lines in LDS, or
// unit-major through memory. Measured per element of the field (fp32, blur and quotient,
// 2e8 elements; through memory it takes 13-15 ps at large chunks, more at small ones):
// - Windows in registers up to r = 8, unless the line is short for them (a line takes 3r
//   more steps, with selects): 64 x 64 r = 1 2.0 ps against 3.8, r = 3 3.9 and 3.9, r = 8 7.4
//   and 3.8; 32 x 32 r = 3 5.9 and 4.5; 128 x 128 r = 8 3.7 and 8.2.
// - Whole lattices where two workgroups fit a compute unit's LDS, or one does and the lines
//   would need a second half each (r > E / 4): 100 x 100 r = 12 5.3 ps, lines 6.0; 139 x 139
//   r = 69 7.8 and 10.2; but 160 x 160 r = 3 6.5 and 3.8, 128 x 128 r = 12 8.2 and 5.9.
// - Lines while two workgroups of 32 of them fit (of 16, with windows in registers or up to
//   450 cells): 256 x 256 r = 3 3.9 ps, r = 12 8.0, r = 64 11.2 (one workgroup of 64: 14.4);
//   512 x 512 r = 12 11.8; 1024 x 1024 r = 3 8.0. Past that sixteen lanes a wave are too few:
//   512 x 512 r = 128 18, 1024 x 1024 r = 12 20.
struct BlurPlan {
    bool lattice, lines, small;
    LatticePlan lp;
    LinePlan line;
    int row_lines, col_lines;  // lines a workgroup takes
    int row_pitch;
    bool feature_major() const { return lattice || lines; }
};

BlurPlan blur_plan(int64_t E, int64_t r)
{
    BlurPlan b = {};
    const int n = (int)E;
    const bool small = r <= kRegRadius && (n >= 88 || n >= 21 * r);  // windows in registers: blurred in place
    const int d = (int)(r < E - 1 ? r : E - 1) + 1;
    // whole lattice: as it is, d more slots per pass along both axes, or a second half beside
    // the first
    const int64_t shifted = (int64_t)(n + 3 * d) * ((n + 3 * d) | 1), halves = (int64_t)n * (2 * n + 1);
    LatticePlan &lp = b.lp;
    const bool shift = shifted < halves;
    const int64_t words = small ? (int64_t)n * (n | 1) : (shift ? shifted : halves);
    lp.words = (int)(words < (1 << 20) ? words : 1 << 20);
    lp.pitch = small ? n | 1 : (shift ? (n + 3 * d) | 1 : 2 * n + 1);
    for (int s = 0; s < 7 && !small; ++s) {
        lp.C[s] = shift ? (s < 3 ? (3 - s) * d : 0) : (s & 1) * n;
        lp.R[s] = shift ? (s < 3 ? 3 : 6 - s) * d : 0;
    }
    // Small lattices share a workgroup: its words are staged in one walk (lattice by lattice,
    // 2 x 2 cells and 60,000 features took 156 us, now 43; 16 x 16 210 -> 105), and it takes as
    // many lines as it has threads up to 20 cells, half as many up to 48 (32 x 32, r = 8: 248 and
    // 211 us), one lattice from there on (63 x 63, r = 15: two 288, one 240).
    lp.per = n <= kManyEdge ? kBlurThreads / (n <= 20 ? 1 : 2) / n : 1;
    const int64_t lds = (int64_t)lp.words * lp.per * 4;
    b.lattice = n <= kBlurThreads && (lds <= kLdsBytes / 2 || (lds <= kLdsBytes && 4 * r > n));
    b.line = small ? LinePlan{n, {0, 0, 0, 0}} : line_plan(E, r);
    b.row_pitch = b.line.slots | 1;
    auto fit = [&](int words) {
        int l = 64;
        while (l > 1 && (int64_t)l * words * 4 > kLdsBytes / 2) l /= 2;
        return l;
    };
    b.row_lines = fit(b.row_pitch);
    // small half-widths leave the passes short: twice the workgroups of half a wave's lines
    // overlap better (256 x 256, 18,000 features: 2.5 -> 1.9 ms)
    if (small && b.row_lines > 32) b.row_lines = 32;
    b.col_lines = fit(b.line.slots);
    b.small = small;
    b.lines = small || n <= 450 ? b.row_lines >= 16 : b.row_lines >= 32;
    return b;
}

// f(StaticInt<R>): the half-width whose windows are held in registers, 0 for none.
template <typename F>
auto with_radius(const BlurPlan &b, int64_t r, F &&f)
{
    static_assert(kRegRadius == 8, "the radii below");
    switch (b.small ? (int)r : 0) {
    case 1: return f(StaticInt<1>{});
    case 2: return f(StaticInt<2>{});
    case 3: return f(StaticInt<3>{});
    case 4: return f(StaticInt<4>{});
    case 5: return f(StaticInt<5>{});
    case 6: return f(StaticInt<6>{});
    case 7: return f(StaticInt<7>{});
    case 8: return f(StaticInt<8>{});
    default: return f(StaticInt<0>{});
    }
}

// Lets the kernels of blur_lds take a compute unit's LDS. The limit belongs to the process,
// so it is the same for every call: a smaller one would take away what another thread's
// launch of the same kernel is about to use.
template <typename T, bool DEN>
hipError_t allow_blur_lds(const BlurPlan &b, int64_t r)
{
    auto allow = [](auto kernel) {
        return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   kLdsBytes);
    };
    return with_radius(b, r, [&](auto radius) {
        constexpr int R = decltype(radius)::value;
        if (b.lattice) {
            if constexpr (R <= kManyRadius)
                if (b.lp.per > 1) {
                    const hipError_t e = allow(k_lattice<T, DEN, R, true>);
                    if (e != hipSuccess) return e;
                }
            return allow(k_lattice<T, DEN, R, false>);
        }
        hipError_t e = allow(k_rows3<R>);
        if constexpr (R == 0)
            if (e == hipSuccess) e = allow(k_cols3<T, DEN>);
        return e;
    });
}

// The blur of f feature-major lattices of counts and its quotients into W from feature v0
// on; DEN: W is a float field and takes the blurred counts. rows: the row passes'
// result (may be the counts' own memory).
template <typename T, bool DEN>
void blur_lds(const BlurPlan &b, const int32_t *cnt, float *rows, T *W, const float *den, int64_t f, int64_t E,
              int64_t r, int64_t v0, const uint32_t *flags, hipStream_t st)
{
    const int n = (int)E, rr = (int)(r < E ? r : E);
    auto grid = [](int64_t g) { return dim3((unsigned)(g < (1 << 20) ? g : 1 << 20)); };
    with_radius(b, r, [&](auto radius) {
        constexpr int R = decltype(radius)::value;
        const dim3 block(kBlurThreads);
        if (b.lattice) {
            // few features are better spread over the chip than sharing workgroups
            LatticePlan lp = b.lp;
            if (lp.per > f / kSpreadFeatures) lp.per = f / kSpreadFeatures > 1 ? (int)(f / kSpreadFeatures) : 1;
            const size_t lds = (size_t)lp.words * lp.per * 4;
            const dim3 wgs = grid((f + lp.per - 1) / lp.per);
            if constexpr (R <= kManyRadius)
                if (lp.per > 1) {
                    hipLaunchKernelGGL((k_lattice<T, DEN, R, true>), wgs, block, lds, st, cnt, W, den, n, rr, f, v0, lp,
                                       flags);
                    return;
                }
            hipLaunchKernelGGL((k_lattice<T, DEN, R, false>), wgs, block, lds, st, cnt, W, den, n, rr, f, v0, lp, flags);
            return;
        }
        const size_t row_lds = (size_t)b.row_lines * b.row_pitch * 4, col_lds = (size_t)b.col_lines * b.line.slots * 4;
        hipLaunchKernelGGL(k_rows3<R>, grid((f * E + b.row_lines - 1) / b.row_lines), block, row_lds, st, cnt, rows, n,
                           rr, f * E, b.row_lines, b.row_pitch, b.line);
        if constexpr (R > 0) {
            hipLaunchKernelGGL((k_cols3_small<T, DEN, R>), grid((f * E + kBlurThreads - 1) / kBlurThreads), block, 0, st,
                               rows, W, den, n, f, v0, flags);
        } else {
            hipLaunchKernelGGL((k_cols3<T, DEN>), grid(f * ((E + b.col_lines - 1) / b.col_lines)), block, col_lds, st,
                               rows, W, den, n, rr, f, v0, b.col_lines, b.line, flags);
        }
    });
}

}  // namespace

hipError_t launch_update(bool f16, void *W, int64_t V, int64_t E, const int32_t *row_ptr, const int32_t *col_idx,
                         int64_t N, int64_t nnz, const int32_t *bmu, int64_t radius, int64_t chunk,
                         const UpdateBuffers &ub, hipStream_t st)
{
    const int64_t M = E * E;
    const BlurPlan bp = blur_plan(E, radius);
    hipError_t e = hipSuccess;
    if (bp.feature_major()) {  // before anything is enqueued: an update that cannot run leaves the codebook as it is
        e = allow_blur_lds<float, true>(bp, radius);
        if (e == hipSuccess) e = f16 ? allow_blur_lds<_Float16, false>(bp, radius) : allow_blur_lds<float, false>(bp, radius);
        if (e != hipSuccess) return e;
    }
    // row pointers checked before any row is read: a batch that fails updates nothing
    e = launch_check_rows(row_ptr, N, nnz, ub.flags, st);
    if (e != hipSuccess) return e;
    // den: counts, blur, kept in ub.den_blur; the samples of heavy units sorted by unit
    const unsigned sg = (unsigned)((N + 255) / 256 < kScanBlocks ? (N + 255) / 256 + 1 : kScanBlocks);
    const unsigned lg = (unsigned)((N + 1023) / 1024 < 512 ? (N + 1023) / 1024 + 1 : 512);
    hipLaunchKernelGGL(k_zero_i32, dim3(grid_for(M)), dim3(256), 0, st, ub.den_cnt, M);
    if (M <= kLdsUnits)
        hipLaunchKernelGGL(k_count_units_lds, dim3(lg), dim3(1024), 0, st, bmu, N, M, ub.den_cnt);
    else
        hipLaunchKernelGGL(k_count_units, dim3(sg), dim3(256), 0, st, bmu, N, M, ub.den_cnt);
    hipLaunchKernelGGL(k_heavy_scan, dim3(1), dim3(1024), 0, st, ub.den_cnt, M, ub.start, ub.cursor, ub.slot,
                       ub.hunit);
    hipLaunchKernelGGL(k_heavy_scatter, dim3(lg), dim3(1024), 0, st, bmu, N, M, ub.start, ub.slot, ub.hunit, ub.cursor,
                       ub.order);
    if (bp.feature_major())
        blur_lds<float, true>(bp, ub.den_cnt, ub.den_a, ub.den_blur, nullptr, 1, E, radius, 0, ub.flags, st);
    else
        blur(ub.den_cnt, ub.den_a, ub.den_b, ub.den_blur, 1, E, radius, st);
    hipLaunchKernelGGL(k_support, dim3((unsigned)E), dim3(256), 0, st, ub.den_cnt, ub.sup_row, nullptr, E,
                       3 * radius, 1);
    hipLaunchKernelGGL(k_support, dim3((unsigned)E), dim3(256), 0, st, ub.sup_row, nullptr, ub.den_blur, E,
                       3 * radius, 0);
    const int64_t runs = (N + kRunSamples - 1) / kRunSamples;
    // The blur in LDS needs no scratch fields: the workspace's three fields, one after the
    // other, hold the counts of three chunks.
    const int64_t step = bp.feature_major() ? (chunk * 3 < V ? chunk * 3 : V) : chunk;
    for (int64_t v0 = 0; v0 < V; v0 += step) {
        const int64_t f = V - v0 < step ? V - v0 : step;
        const Field fd = bp.feature_major() ? Field{1, M} : Field{f, 1};
        hipLaunchKernelGGL(k_zero_i32, dim3(grid_for(f * M)), dim3(256), 0, st, ub.cnt, f * M);
        hipLaunchKernelGGL(k_count_light, dim3(grid_for(N * 4)), dim3(256), 0, st, row_ptr, col_idx, N, nnz, bmu, M,
                           ub.den_cnt, (int32_t)v0, (int32_t)(v0 + f), ub.cnt, fd, ub.flags);
        if (runs > 0)
            hipLaunchKernelGGL(k_count_heavy, dim3((unsigned)runs), dim3(1024), 0, st, row_ptr, col_idx, nnz, bmu, M,
                               ub.den_cnt, ub.start, ub.order, (int32_t)v0, (int32_t)(v0 + f), ub.cnt, fd, ub.flags);
        float *num = reinterpret_cast<float *>(ub.cnt);  // the blur's result replaces the counts
        if (bp.feature_major()) {
            if (f16)
                blur_lds<_Float16, false>(bp, ub.cnt, num, static_cast<_Float16 *>(W), ub.den_blur, f, E, radius, v0, ub.flags, st);
            else
                blur_lds<float, false>(bp, ub.cnt, num, static_cast<float *>(W), ub.den_blur, f, E, radius, v0, ub.flags, st);
            continue;
        }
        blur(ub.cnt, ub.a, ub.b, num, f, E, radius, st);
        const int64_t qt = ((M + 63) / 64) * ((f + 63) / 64);
        const unsigned qg = (unsigned)(qt < (1 << 20) ? qt : (1 << 20));
        if (f16)
            hipLaunchKernelGGL(k_quotient_t<_Float16>, dim3(qg), dim3(256), 0, st, static_cast<_Float16 *>(W), num,
                               ub.den_blur, f, M, v0, ub.flags);
        else
            hipLaunchKernelGGL(k_quotient_t<float>, dim3(qg), dim3(256), 0, st, static_cast<float *>(W), num,
                               ub.den_blur, f, M, v0, ub.flags);
    }
    return hipGetLastError();
}

}  // namespace som
