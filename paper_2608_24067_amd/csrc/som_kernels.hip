// som_kernels.hip -- gfx950 kernels of the sparse-binary BMU search other than the
// sweep (som_sweep.hip): the fp64 norms, the regrouping of the batch and the tile plan
// (Algorithm 2, step 5), and the finalize that reduces the sweep's per-strip keys.
//
// The plan (SpMM-tile kernel section) groups samples into tiles of TA consecutive
// rows and lists, per tile, the distinct feature ids of its rows in ascending order,
// each with a TA-bit mask of the rows holding it; the sweep (som_sweep.hip) streams
// those codebook rows once per tile and strip. Unless the caller keeps the sample
// order, the batch is first regrouped by each sample's least frequent feature (the
// post-submission section's lever of clustering samples so tiles share features).
// The finalize takes, per sample, the smallest of the sweep's per-strip keys and
// forms the winner's full squared distance from the dot product the sweep kept.

#include "som_device.h"

namespace som {
namespace {

// ----------------------------------------------------------------- norms

// n_i = sum_v W[v*M+i]^2: one thread per neuron, v ascending, fp64. The square of
// an fp32 (or fp16) value is exact in fp64, so fma(w, w, acc) equals acc + w*w.
// One wave per workgroup and NL rows in flight per wave: the sums are sequential, the
// loads are not. 32 rows read at 7 TB/s on a 256 x 256 map, where 128 cost 10%; a map of
// fewer than kNormWavesFew waves is bound by each lane's chain of batches and takes 128
// (130 x 130 map 785 -> 608 us).
constexpr int64_t kNormWavesFew = 512;

template <typename E, int NL>
__global__ __launch_bounds__(64) void k_norms(const E *__restrict__ W, int64_t V, int64_t M,
                                              double *__restrict__ norms)
{
    constexpr int kNormLoads = NL;
    const int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (i >= M) return;
    const E *p = W + i;
    double acc = 0.0;
    int64_t v = 0;
    for (; v + kNormLoads <= V; v += kNormLoads) {
        float w[kNormLoads];
#pragma unroll
        for (int u = 0; u < kNormLoads; ++u) w[u] = (float)__builtin_nontemporal_load(p + (v + u) * M);
#pragma unroll
        for (int u = 0; u < kNormLoads; ++u) {
            const double x = (double)w[u];
            acc = fma(x, x, acc);
        }
    }
    for (; v < V; ++v) {
        const double x = (double)(float)p[v * M];
        acc = fma(x, x, acc);
    }
    norms[i] = acc;
}

// The same for a map of no more waves than compute units, where each lane's chain of load
// batches was the time (64 x 64: 0.44 ms for 0.5 GB). Seven waves of a workgroup bring the
// rows of its 64 neurons, kNormDepth chunks of kNormRows rows each in flight, and leave
// their squares (exact in fp64) in LDS; the eighth adds them up in ascending v, one dependent
// fp64 addition per row, while the others fill the other half: V additions of about 10 ns
// are the bound. V = 30,000, fp32: 64 x 64 436 -> 328 us, 128 x 128 490 -> 343; fp16 549 -> 337.
constexpr int kNormProducers = 7, kNormRows = 16, kNormDepth = 3;
constexpr int kNormChunk = kNormProducers * kNormRows;
constexpr int64_t kNormFewBlocks = 256;

template <typename E>
__global__ __launch_bounds__(64 * (kNormProducers + 1)) void k_norms_few(const E *__restrict__ W, int64_t V, int64_t M,
                                                                         double *__restrict__ norms)
{
    __shared__ double sq[2][kNormChunk][64];
    const int lane = threadIdx.x & 63, w = wave_id();
    const int64_t i = (int64_t)blockIdx.x * 64 + lane;
    const int64_t chunks = (V + kNormChunk - 1) / kNormChunk;
    if (w == 0) {
        double acc = 0.0;
        for (int64_t c = 0; c < chunks; ++c) {
            __syncthreads();
            const double(*s)[64] = sq[c & 1];
            // a batch of squares is read while the one before it is added
            double x[2][kNormRows];
#pragma unroll
            for (int u = 0; u < kNormRows; ++u) x[0][u] = s[u][lane];
#pragma unroll
            for (int b = 0; b < kNormProducers; ++b) {
                if (b + 1 < kNormProducers)
#pragma unroll
                    for (int u = 0; u < kNormRows; ++u) x[(b + 1) & 1][u] = s[(b + 1) * kNormRows + u][lane];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < kNormRows; ++u) acc += x[b & 1][u];
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (i < M) norms[i] = acc;
        return;
    }
    const unsigned col = (unsigned)(i < M ? i : M - 1);  // beside a row's uniform address
    E x[kNormDepth][kNormRows];
    auto load = [&](int64_t c, E *to) {
        // rows past V read the last one (a branch here would make the waits below wait for
        // the newest loads) and add +0, which leaves a sum of squares as it is
        const int64_t v0 = c * kNormChunk + (w - 1) * kNormRows;
#pragma unroll
        for (int u = 0; u < kNormRows; ++u)
            to[u] = __builtin_nontemporal_load(W + (v0 + u < V ? v0 + u : V - 1) * M + col);
    };
#pragma unroll
    for (int d = 0; d < kNormDepth; ++d) load(d, x[d]);
    for (int64_t c0 = 0; c0 < chunks; c0 += kNormDepth) {
#pragma unroll
        for (int d = 0; d < kNormDepth; ++d) {
            const int64_t c = c0 + d;
            if (c >= chunks) break;  // uniform over the workgroup, as for the eighth wave
            double(*s)[64] = sq[c & 1] + (w - 1) * kNormRows;
#pragma unroll
            for (int u = 0; u < kNormRows; ++u) {
                const double q = (double)(float)x[d][u];
                s[u][lane] = q * q;
            }
            if ((c + 1) * kNormChunk > V)  // uniform
                for (int u = 0; u < kNormRows; ++u)
                    if (c * kNormChunk + (w - 1) * kNormRows + u >= V) s[u][lane] = 0.0;
            load(c + kNormDepth, x[d]);
            __syncthreads();
        }
    }
}

__global__ void k_clear_flags(uint32_t *flags) { flags[threadIdx.x] = 0u; }

// Row pointers checked before any kernel walks a row: non-decreasing and inside
// [row_ptr[0], row_ptr[0] + nnz], with row_ptr[0] >= 0. A batch that fails is flagged
// (SOM_FLAG_ROW_PTR) and every later kernel of the plan reads it as empty (rows_nnz),
// so row pointers that decrease cannot make rows overlap and multiply the work.
// The flags start from zero: cleared by k_clear_flags, or by k_check_few where one
// workgroup checks the whole batch.
// Rows one workgroup checks, eight per thread in one round trip (at 10,000 rows the search is
// 2 us slower so than with two launches).
constexpr int64_t kCheckFew = 8192;

__global__ __launch_bounds__(1024) void k_check_few(const int32_t *__restrict__ row_ptr, int64_t N, int64_t nnz,
                                                    uint32_t *__restrict__ flags)
{
    const int64_t base = row_ptr[0];
    bool bad = base < 0;
#pragma unroll
    for (int64_t k = 0; k < kCheckFew / 1024; ++k) {
        const int64_t s = k * 1024 + threadIdx.x;
        if (s < N) bad |= row_bad(row_ptr, base, nnz, s);
    }
    const int any = __syncthreads_or(bad);
    if (threadIdx.x < 64) flags[threadIdx.x] = threadIdx.x == 0 && any ? SOM_FLAG_ROW_PTR : 0u;
}

__global__ __launch_bounds__(256) void k_check_rows(const int32_t *__restrict__ row_ptr, int64_t N, int64_t nnz,
                                                    uint32_t *__restrict__ flags)
{
    const int64_t base = row_ptr[0];
    bool bad = base < 0;
    for (int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x; s < N; s += (int64_t)gridDim.x * 256)
        bad |= row_bad(row_ptr, base, nnz, s);
    if (__ballot(bad) != 0 && (threadIdx.x & 63) == 0) atomicOr(flags, SOM_FLAG_ROW_PTR);
}

// The ids a plan kernel may read: nnz, or none once the row pointers are flagged.
__device__ __forceinline__ int64_t rows_nnz(const uint32_t *flags, int64_t nnz)
{
    return (flags[0] & SOM_FLAG_ROW_PTR) ? 0 : nnz;
}

// ----------------------------------------------------------------- order

// Sample order. The post-submission section's tuning groups samples so that a
// tile's rows share features. Here the samples of a batch are bucketed by their
// least frequent feature in that batch: rows that share a rare feature land in
// the same or neighbouring tiles, which run close together in time, so a rare
// codebook row is re-read while still in L2. A sample's result does not depend on where it
// sits (its sum order is fixed by its own features), so the permutation never
// shows in the output. The permuted batch is written to the workspace as row offsets
// of its own and, per position, where that row's ids start in the caller's batch
// (both in pos, interleaved), from which the plan reads them; k_unpermute moves the results back
// to their samples.

constexpr int kLdsHistMax = 32768;          // features whose counts fit the LDS histogram
constexpr int64_t kFreqSample = 1ll << 25;  // ids counted: the ordering needs only a rough rarity rank

// The regrouping's counters: freq[V+1] and bucket[V+1] start at zero.
__global__ __launch_bounds__(256) void k_order_clear(uint32_t *__restrict__ freq, u64 *__restrict__ bucket, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        freq[i] = 0u;
        bucket[i] = 0ull;
    }
}

// freq[v] = occurrences of feature v among the batch's first kFreqSample ids (all of
// them for smaller batches; ids outside [0, V) skipped). Each workgroup counts a
// contiguous chunk in LDS (BINS >= V bins; global atomics for larger V), then adds its
// non-zero counts to the global histogram. The kernel waits on memory, not on the LDS
// atomics: sixteen waves a workgroup and eight ids per lane in flight (before: four waves,
// one id each; 2,000,000 rows 258 -> 48 us, 30,000 rows 93 -> 7 us).
constexpr int kFreqThreads = 1024;
constexpr int kFreqIds = 8;  // ids in flight per lane

template <int BINS>
__global__ __launch_bounds__(kFreqThreads) void k_freq(const int32_t *__restrict__ row_ptr,
                                                       const int32_t *__restrict__ col_idx, int64_t nnz, int32_t V,
                                                       uint32_t *__restrict__ freq)
{
    __shared__ uint32_t h[BINS];
    const int64_t base = csr_base(row_ptr, nnz);
    const bool lds = V <= BINS;
    if (lds)
        for (int v = threadIdx.x; v < V; v += kFreqThreads) h[v] = 0u;
    __syncthreads();
    const int64_t chunk = (nnz + gridDim.x - 1) / gridDim.x;
    const int64_t p0 = (int64_t)blockIdx.x * chunk;
    const int64_t p1 = p0 + chunk < nnz ? p0 + chunk : nnz;
    for (int64_t p = p0 + threadIdx.x; p < p1; p += kFreqThreads * kFreqIds) {
        int id[kFreqIds];
#pragma unroll
        for (int u = 0; u < kFreqIds; ++u) {
            const int64_t q = p + u * kFreqThreads;
            id[u] = q < p1 ? col_idx[base + q] : -1;
        }
#pragma unroll
        for (int u = 0; u < kFreqIds; ++u)
            if (id[u] >= 0 && id[u] < V) {
                if (lds) atomicAdd(&h[id[u]], 1u);
                else atomicAdd(&freq[id[u]], 1u);
            }
    }
    __syncthreads();
    if (lds)
        for (int v = threadIdx.x; v < V; v += kFreqThreads)
            if (h[v]) atomicAdd(&freq[v], h[v]);
}

// Clamped id range of row s (relative to row_ptr[0]); empty if row_ptr decreases.
__device__ __forceinline__ void row_range(const int32_t *row_ptr, int64_t base, int64_t nnz, int64_t s, int64_t &rb,
                                          int64_t &re, uint32_t &bad)
{
    const int64_t a = (int64_t)row_ptr[s] - base, b = (int64_t)row_ptr[s + 1] - base;
    if (b < a || a < 0 || b > nnz) bad |= SOM_FLAG_ROW_PTR;
    rb = clamp64(a, 0, nnz);
    re = b < a ? rb : clamp64(b, rb, nnz);
}

// skey[s] = the sample's least frequent valid feature (ties: the larger id), V if it
// has none; bucket[key] += (1 << 32) | row length: samples counted in the high
// half, ids in the low half of one 64-bit word. The word the atomic returns is the
// sample's rank in its bucket (samples and ids before it), kept in rank[s]: once the
// buckets' starts are known it gives the sample's place without a second atomic.
__global__ __launch_bounds__(256) void k_rarest(const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col_idx,
                                                int64_t N, int64_t nnz, int32_t V, const uint32_t *__restrict__ freq,
                                                int32_t *__restrict__ skey, u64 *__restrict__ bucket,
                                                u64 *__restrict__ rank,
                                                uint32_t *__restrict__ flags)
{
    // the four lanes of a quad share a row (lane q of the quad takes ids q, q + 4, ...)
    nnz = rows_nnz(flags, nnz);
    const int64_t base = csr_base(row_ptr, nnz);
    const int sub = threadIdx.x & 3;
    uint32_t bad = 0;
    for (int64_t s = (int64_t)blockIdx.x * 64 + (threadIdx.x >> 2); s < N; s += (int64_t)gridDim.x * 64) {
        int64_t rb, re;
        row_range(row_ptr, base, nnz, s, rb, re, bad);
        u64 best = kKeyNone;  // (frequency, V-1-id): smallest frequency, then largest id
        // three of the lane's ids, then their counts, per step: a row of up to 12 ids is one
        // round trip of dependent loads instead of three
        for (int64_t p = rb + sub; p < re; p += 12) {
            int id[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) id[j] = p + 4 * j < re ? col_idx[base + p + 4 * j] : -1;
            unsigned f[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) f[j] = id[j] >= 0 && id[j] < V ? freq[id[j]] : 0u;
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (id[j] >= 0 && id[j] < V) best = min_u64(best, ((u64)f[j] << 32) | (unsigned)(V - 1 - id[j]));
        }
        // the quad is active or idle as a whole (one row), so the swaps read its own lanes
        best = min_u64(best, dpp64<0xB1>(best));
        best = min_u64(best, dpp64<0x4E>(best));
        if (sub == 0) {
            const int key = best == kKeyNone ? V : (int)(V - 1 - (int)(unsigned)(best & 0xFFFFFFFFull));
            skey[s] = key;
            rank[s] = atomicAdd(&bucket[key], (1ull << 32) | (u64)(re - rb));
        }
    }
    if (bad) atomicOr(flags, bad);
}

// One workgroup: exclusive scan of the nb packed bucket counts into packed starting
// offsets (sample offset << 32 | id offset; both sums stay below 2^31, so the packed
// words add without a carry). *prp_end = total ids (capped at nnz). Each wave scans a
// contiguous stretch, four consecutive words per lane and step, the words of kScanSteps
// steps loaded before any is used: two round trips to memory for 32,768 buckets where one
// thread walking 30 words took 30 twice over (V = 30,000: 57 -> 13 us).
constexpr int kScanSteps = 8;

__global__ __launch_bounds__(1024) void k_bucket_scan(u64 *__restrict__ bucket, int64_t nb, int64_t nnz,
                                                      int32_t *__restrict__ prp_end)
{
    __shared__ u64 sum[16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t steps = (nb + 16 * 256 - 1) / (16 * 256);
    const int64_t b0 = w * steps * 256 + lane * 4;  // the lane's first word
    auto load = [&](int64_t at, u64 *x) {
        if (at + 4 <= nb) {  // two 16-byte loads
            const ulonglong2 *p = reinterpret_cast<const ulonglong2 *>(bucket + at);
            const ulonglong2 a = p[0], b = p[1];
            x[0] = a.x, x[1] = a.y, x[2] = b.x, x[3] = b.y;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = at + j < nb ? bucket[at + j] : 0ull;
        }
    };
    u64 total = 0;
    for (int64_t k0 = 0; k0 < steps; k0 += kScanSteps) {
        u64 x[kScanSteps][4];
#pragma unroll
        for (int k = 0; k < kScanSteps; ++k) {
            if (k0 + k < steps) load(b0 + (k0 + k) * 256, x[k]);
            else x[k][0] = x[k][1] = x[k][2] = x[k][3] = 0ull;
        }
#pragma unroll
        for (int k = 0; k < kScanSteps; ++k) total += (x[k][0] + x[k][1]) + (x[k][2] + x[k][3]);
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) total += __shfl_xor(total, d);
    if (lane == 0) sum[w] = total;
    __syncthreads();
    u64 run = 0;  // everything before the wave's current step
    for (int j = 0; j < w; ++j) run += sum[j];
    if (threadIdx.x == 1023) {
        const int64_t ids = (int64_t)((run + total) & 0xFFFFFFFFull);
        *prp_end = (int32_t)(ids < nnz ? ids : nnz);
    }
    for (int64_t k0 = 0; k0 < steps; k0 += kScanSteps) {
        u64 x[kScanSteps][4];
#pragma unroll
        for (int k = 0; k < kScanSteps; ++k) {
            if (k0 + k < steps) load(b0 + (k0 + k) * 256, x[k]);
            else x[k][0] = x[k][1] = x[k][2] = x[k][3] = 0ull;
        }
#pragma unroll
        for (int k = 0; k < kScanSteps; ++k) {
            if (k0 + k >= steps) break;
            const u64 own = (x[k][0] + x[k][1]) + (x[k][2] + x[k][3]);
            u64 inc = own;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const u64 y = __shfl_up(inc, d);
                if (lane >= d) inc += y;
            }
            u64 at = run + inc - own;
            const int64_t b = b0 + (k0 + k) * 256;
            if (b + 4 <= nb) {
                ulonglong2 *p = reinterpret_cast<ulonglong2 *>(bucket + b);
                const u64 a1 = at + x[k][0], a2 = a1 + x[k][1];
                p[0] = make_ulonglong2(at, a1);
                p[1] = make_ulonglong2(a2, a2 + x[k][2]);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (b + j < nb) bucket[b + j] = at;
                    at += x[k][j];
                }
            }
            run += __shfl(inc, 63);
        }
    }
}

// Sample s goes to its bucket's start plus its rank in the bucket (both packed as
// samples << 32 | ids; the id halves never carry): it sits at position inv[s] of the
// permuted batch, its ids at plan offsets pos[2 inv[s]] ..., and pos[2 inv[s] + 1] is where
// its row starts in the caller's col_idx (past row_ptr[0]). The rows themselves are
// not copied: the plan reads each position's ids from there. Positions past N and
// offsets past nnz (only reachable with invalid row pointers or a workspace the
// regrouping did not write) are dropped or clamped.
__global__ __launch_bounds__(256) void k_place(const int32_t *__restrict__ row_ptr, int64_t N, int64_t nnz,
                                               const int32_t *__restrict__ skey, const u64 *__restrict__ bucket,
                                               const u64 *__restrict__ rank, int64_t nb, int32_t *__restrict__ inv,
                                               int32_t *__restrict__ pos, const uint32_t *__restrict__ flags)
{
    nnz = rows_nnz(flags, nnz);
    const int64_t base = csr_base(row_ptr, nnz);
    for (int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x; s < N; s += (int64_t)gridDim.x * 256) {
        const u64 at = bucket[clamp64(skey[s], 0, nb - 1)] + rank[s];
        const int64_t ps = (int64_t)(at >> 32), pi = (int64_t)(at & 0xFFFFFFFFull);
        inv[s] = ps < N ? (int32_t)ps : -1;
        if (ps >= N) continue;
        // one 8-byte word per sample: a scattered write costs a whole memory burst either way
        reinterpret_cast<int2 *>(pos)[ps] =
            make_int2((int32_t)(pi < nnz ? pi : nnz), (int32_t)clamp64((int64_t)row_ptr[s] - base, 0, nnz));
    }
}

// ------------------------------------------------------------------ plan

constexpr int kPlanWaves = 4;
// ids staged in LDS per wave: 16 KiB a workgroup (2048 would halve the workgroups a CU
// holds, 5% slower on the 64x64 workload)
constexpr int kPlanStage = 1024;

// The TA-way merge of the sorted rows of one tile per TA lanes (lane sl of group grp walks
// its row's ids p ... pe - 1 through id_at; positions fit 32 bits: every offset lies in
// [0, nnz] and nnz < 2^31). Each step takes, per tile, the smallest current id over its TA
// lanes (the next element of the union, ascending), the ballot of the lanes holding it
// (its sample mask), and advances those lanes. Entries go to plan[lo ...], at most cap of
// them; ids outside [0, V) are skipped and flagged, and so are unsorted ones. Returns the
// union's size; every lane of the wave takes part (an empty row where it has none).
template <int TA, bool REAL, typename IdAt>
__device__ __forceinline__ int plan_merge(const IdAt &id_at, int p, int pe, int lo, int cap, int grp, int sl, int32_t V,
                                          const float *__restrict__ values, int64_t shift, uint2 *__restrict__ plan,
                                          float *__restrict__ vals, double &sq, uint32_t &bad)
{
    int cur = INT_MAX;
    float curv = 0.0f;
    int k = 0;
    // next valid id of this lane's row (INT_MAX once the row is done), with its value;
    // ids outside [0, V) (invalid input) are skipped on a path of their own
    auto fetch = [&]() {
        cur = INT_MAX;
        if (p >= pe) return;
        int id = id_at(p);
        if (id < 0 || id >= V) {
            for (;;) {
                bad |= SOM_FLAG_ID_RANGE;
                if (++p >= pe) return;
                id = id_at(p);
                if (id >= 0 && id < V) break;
            }
        }
        cur = id;
        if constexpr (REAL) {
            curv = values[shift + p];
            sq = fma((double)curv, (double)curv, sq);
        }
    };
    fetch();
    // Every step consumes at least one id of the group, so a tile takes at most as many
    // steps as its span holds ids; only lanes whose ranges overlap (row pointers that
    // decrease, flagged above) take more, and their surplus entries are dropped.
    // (Left by a break in its middle, the loop carries its exit condition to its end, four
    // scalar instructions a step: 500,000 rows 57 -> 51 us.)
    for (int m = group_min_i32<TA>(cur); __ballot(m != INT_MAX) != 0; m = group_min_i32<TA>(cur)) {
        const u64 bal = __ballot(m != INT_MAX && cur == m);
        const unsigned mask = (unsigned)((bal >> (grp * TA)) & (TA == 32 ? 0xFFFFFFFFull : ((1ull << TA) - 1)));
        if (m != INT_MAX) {
            if (k < cap) {
                if (sl == 0) plan[lo + k] = make_uint2((unsigned)m, plan_word<TA>(mask));
                if (REAL && cur == m) vals[(int64_t)(lo + k) * TA + sl] = curv;
            }
            ++k;
            if (cur == m) {
                ++p;
                fetch();
                if (cur != INT_MAX && cur <= m) bad |= SOM_FLAG_UNSORTED;
            }
        }
    }
    return k;
}

// A wave plans 64/TA consecutive tiles at once (TA = 2 ... 32): lane l works on row s = l % TA of
// tile l / TA, a TA-way merge of sorted lists per lane group (plan_merge). Tiles of 8 come
// here only when they hold many ids (k_plan_rank otherwise). Offsets are clamped to [row_ptr[0], row_ptr[0]+nnz)
// and to each tile's own range, ids outside [0, V) are skipped, and a tile never
// writes more entries than its own CSR span, so no input can drive an access out
// of bounds.
//
// Offsets are read os words apart: off[p * os]. Regrouped batch (psrc non-null, os = 2):
// off (the regrouped row offsets) places every tile's entries and gives each position's
// row length; the row's ids start at psrc[p * os] in the caller's col_idx (past
// src_ptr[0]), clamped to the batch. Otherwise off is the caller's row_ptr (os = 1) and
// positions are samples.
//
// Real-valued rows (REAL, values given): every union entry also gets the TA values of
// its samples (vals[entry*TA + s], written for the samples whose mask bit is set;
// the other slots are never read), and every row the fp64 sum of its squared
// values in its own order (xsq, by batch position), which is ||x||^2.
template <int TA, bool REAL>
__global__ __launch_bounds__(256) void k_plan(const int32_t *__restrict__ off, int os,
                                              const int32_t *__restrict__ src_ptr, const int32_t *__restrict__ psrc,
                                              const int32_t *__restrict__ col_idx,
                                              int64_t N, int64_t nnz, int32_t V, int64_t n_tiles,
                                              uint2 *__restrict__ plan, int2 *__restrict__ tiles,
                                              uint32_t *__restrict__ flags, const float *__restrict__ values,
                                              float *__restrict__ vals, double *__restrict__ xsq)
{
    constexpr int G = 64 / TA;  // tiles per wave
    __shared__ int32_t stage[kPlanWaves][kPlanStage];
    const int lane = threadIdx.x & 63;
    const int wv = wave_id();
    const int grp = lane / TA;
    const int sl = lane % TA;
    nnz = rows_nnz(flags, nnz);
    const int64_t base = csr_base(off, nnz);
    const int64_t sbase = psrc ? csr_base(src_ptr, nnz) : base;
    uint32_t bad = 0;

    for (int64_t tb = (int64_t)blockIdx.x * kPlanWaves * G; tb < n_tiles; tb += (int64_t)gridDim.x * kPlanWaves * G) {
        const int64_t tw = tb + (int64_t)wv * G;  // first tile of this wave
        const int64_t t = tw + grp;               // this lane's tile
        const bool live = t < n_tiles;
        // the wave's CSR span, for staging
        int64_t wlo = 0, whi = 0;
        if (tw < n_tiles) {
            const int64_t te = tw + G < n_tiles ? tw + G : n_tiles;
            wlo = clamp64((int64_t)off[tw * TA * os] - base, 0, nnz);
            whi = clamp64((int64_t)off[(te * TA < N ? te * TA : N) * os] - base, wlo, nnz);
        }
        int64_t lo = 0, hi = 0, b = 0, e = 0;
        int64_t src = 0;  // where the lane's ids start in col_idx (past its base)
        if (live) {
            const int64_t s0 = t * TA;
            const int64_t s1 = s0 + TA < N ? s0 + TA : N;
            lo = clamp64((int64_t)off[s0 * os] - base, wlo, whi);
            hi = clamp64((int64_t)off[s1 * os] - base, lo, whi);
            if (s0 + sl < N) {
                const int64_t rb = (int64_t)off[(s0 + sl) * os] - base;
                const int64_t re = (int64_t)off[(s0 + sl + 1) * os] - base;
                if (re < rb || rb < lo || re > hi) bad |= SOM_FLAG_ROW_PTR;
                b = clamp64(rb, lo, hi);
                e = clamp64(re, b, hi);
                src = b;
                if (psrc) {
                    // the caller's row at this position (its flags were set by the regrouping),
                    // never reaching past the batch
                    src = clamp64(psrc[(s0 + sl) * os], 0, nnz);
                    if (nnz - src < e - b) e = b + (nnz - src);
                }
            }
        }
        const bool staged = (whi - wlo) <= kPlanStage;  // wave-uniform
        if (staged) {
            if (psrc) {
                for (int64_t q = 0; q < e - b; ++q) stage[wv][b - wlo + q] = col_idx[sbase + src + q];
            } else {
                for (int64_t q = lane; q < whi - wlo; q += 64) stage[wv][q] = col_idx[base + wlo + q];
            }
        }
        __syncthreads();

        const int64_t shift = sbase + src - b;  // the lane's id q (b <= q < e) is col_idx[shift + q]
        const int pwlo = (int)wlo;
        const int cap = (int)(hi - lo);
        double sq = 0.0;
        int k;  // union entries found for this lane's tile (equal across its group)
        if (staged)
            k = plan_merge<TA, REAL>([&](int q) { return stage[wv][q - pwlo]; }, (int)b, (int)e, (int)lo, cap, grp, sl,
                                     V, values, shift, plan, vals, sq, bad);
        else
            k = plan_merge<TA, REAL>([&](int q) { return col_idx[shift + q]; }, (int)b, (int)e, (int)lo, cap, grp, sl,
                                     V, values, shift, plan, vals, sq, bad);
        if (live && sl == 0) tiles[t] = make_int2((int)lo, k < cap ? k : cap);
        if (REAL && live && t * TA + sl < N) xsq[t * TA + sl] = sq;
        __syncthreads();
    }
    if (bad) atomicOr(flags, bad);
}

// Tiles of 8, the same plan by ranks instead of a merge: a wave plans one tile, its lanes
// taking the tile's ids. An id's place among all ids of the tile is the sum over the eight
// rows of the row's ids below it -- eight binary searches in LDS, side by side -- and the
// searches also tell which rows hold it (its sample mask); its lowest holder stands for
// it, and counting the holders below a place gives the union's index. A merge takes a
// dependent step per union entry (about 90 a tile, 0.25 us each), the searches four or
// five, so a few tiles are planned in 7 us instead of 21 (33 rows).
// A tile with more than kRankIds ids, an id outside [0, V), or a row that is not strictly
// ascending takes plan_merge.
constexpr int kRankIds = 512;

// Orders a wave's LDS writes before the reads of its other lanes that follow.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <bool REAL>
__global__ __launch_bounds__(256) void k_plan_rank(const int32_t *__restrict__ off, int os,
                                                   const int32_t *__restrict__ src_ptr,
                                                   const int32_t *__restrict__ psrc,
                                                   const int32_t *__restrict__ col_idx, int64_t N, int64_t nnz,
                                                   int32_t V, int64_t n_tiles, uint2 *__restrict__ plan,
                                                   int2 *__restrict__ tiles, uint32_t *__restrict__ flags,
                                                   const float *__restrict__ values, float *__restrict__ vals,
                                                   double *__restrict__ xsq)
{
    constexpr int TA = 8;
    __shared__ int32_t s_id[kPlanWaves][kRankIds + 1];  // (an empty last row's place may be looked at)
    __shared__ uint32_t s_at[kPlanWaves][kRankIds];   // by place: mask | id's index << 8 (0: not the lowest holder)
    __shared__ float s_val[kPlanWaves][REAL ? kRankIds : 1];
    __shared__ uint16_t s_rep[kPlanWaves][REAL ? kRankIds : 1];  // by id: its lowest holder's place
    const int lane = threadIdx.x & 63;
    const int wv = wave_id();
    int32_t *id_l = s_id[wv];
    uint32_t *at_l = s_at[wv];
    nnz = rows_nnz(flags, nnz);
    const int64_t base = csr_base(off, nnz);
    const int64_t sbase = psrc ? csr_base(src_ptr, nnz) : base;
    uint32_t bad = 0;

    for (int64_t t = (int64_t)blockIdx.x * kPlanWaves + wv; t < n_tiles; t += (int64_t)gridDim.x * kPlanWaves) {
        // lane j < 8: row j's plan offsets [b, e) and where its ids start in col_idx (past its base)
        const int64_t s0 = t * TA, s1 = s0 + TA < N ? s0 + TA : N;
        const int rows = (int)(s1 - s0);
        int b = 0, e = 0, src = 0;
        if (lane < rows) {
            const int64_t rb = (int64_t)off[(s0 + lane) * os] - base;
            const int64_t re = (int64_t)off[(s0 + lane + 1) * os] - base;
            if (re < rb || rb < 0 || re > nnz) bad |= SOM_FLAG_ROW_PTR;
            b = (int)clamp64(rb, 0, nnz);
            e = (int)clamp64(re, b, nnz);
            src = b;
            if (psrc) {
                // the caller's row at this position, never reaching past the batch
                src = (int)clamp64(psrc[(s0 + lane) * os], 0, nnz);
                if (nnz - src < e - b) e = b + (int)(nnz - src);
            }
        }
        const int lo = __builtin_amdgcn_readfirstlane(b);
        const int hi = __builtin_amdgcn_readlane(e, rows - 1);
        if (lane >= rows && lane < TA) b = e = hi;
        int rs[TA], len[TA], sh[TA];  // wave-uniform: row starts past lo, lengths, col_idx shifts
        int longest = 0;
        bool plain = hi - lo <= kRankIds;  // the rows fill [lo, hi) one after the other
        int want = lo;
#pragma unroll
        for (int j = 0; j < TA; ++j) {
            const int bj = __builtin_amdgcn_readlane(b, j), ej = __builtin_amdgcn_readlane(e, j);
            plain = plain && bj == want;
            want = ej;
            rs[j] = bj - lo;
            len[j] = ej - bj;
            sh[j] = __builtin_amdgcn_readlane(src, j) - bj;
            longest = len[j] > longest ? len[j] : longest;
        }
        const int n = hi > lo ? hi - lo : 0;
        auto row_of = [&](int q, int &shift) {
            int r = 0;
            shift = sh[0];
#pragma unroll
            for (int j = 1; j < TA; ++j)
                if (q >= rs[j]) {
                    r = j;
                    shift = sh[j];
                }
            return r;
        };
        int k = 0;
        double sq = 0.0;
        if (plain) {
            // stage the ids, two per lane in flight, and check them
            bool wrong = false;
            for (int q0 = 0; q0 < n; q0 += 128) {
                int id[2];
                float v[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int q = q0 + u * 64 + lane;
                    int shift;
                    row_of(q, shift);
                    const int64_t at = sbase + lo + q + shift;
                    id[u] = q < n ? col_idx[at] : 0;
                    if constexpr (REAL) v[u] = q < n ? values[at] : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int q = q0 + u * 64 + lane;
                    if (q < n) {
                        id_l[q] = id[u];
                        wrong |= id[u] < 0 || id[u] >= V;
                        if constexpr (REAL) s_val[wv][q] = v[u];
                    }
                }
            }
            wave_sync();
            int top = 1;
            while (top * 2 <= longest) top *= 2;
            for (int q0 = 0; q0 < n; q0 += 64) {
                const int q = q0 + lane;
                int shift;
                const int r = row_of(q, shift);
                const int id = id_l[q < n ? q : n - 1];
                int pos[TA];
#pragma unroll
                for (int j = 0; j < TA; ++j) pos[j] = 0;
                for (int st = top; st > 0; st >>= 1) {
                    int x[TA];
#pragma unroll
                    for (int j = 0; j < TA; ++j) {
                        const int i = pos[j] + st;
                        x[j] = id_l[rs[j] + (i <= len[j] ? i - 1 : 0)];
                    }
#pragma unroll
                    for (int j = 0; j < TA; ++j)
                        if (pos[j] + st <= len[j] && x[j] < id) pos[j] += st;
                }
                int first = 0;
                unsigned mask = 0;
#pragma unroll
                for (int j = 0; j < TA; ++j) {
                    const int x = id_l[rs[j] + (pos[j] < len[j] ? pos[j] : 0)];
                    if (pos[j] < len[j] && x == id) mask |= 1u << j;
                    first += pos[j];
                }
                if (q < n) {
                    // a strictly ascending row holds its own id exactly where it stands
                    int own = 0;
#pragma unroll
                    for (int j = 0; j < TA; ++j)
                        if (j == r) own = rs[j] + pos[j];
                    wrong |= own != q;
                    const int below = __popc(mask & ((1u << r) - 1u));
                    const int place = first + below;
                    if (place < n) at_l[place] = below == 0 ? mask | ((unsigned)q << 8) : 0u;
                    if constexpr (REAL) s_rep[wv][q] = (uint16_t)first;
                }
            }
            wave_sync();
            plain = __ballot(wrong) == 0;
        }
        if (plain) {
            for (int q0 = 0; q0 < n; q0 += 64) {
                const int q = q0 + lane;
                const uint32_t a = q < n ? at_l[q] : 0u;
                const u64 heads = __ballot(a != 0u);
                const int u = k + __popcll(heads & ((1ull << lane) - 1ull));
                if (a != 0u) {
                    plan[lo + u] = make_uint2((unsigned)id_l[a >> 8], plan_word<TA>(a & 0xFFu));
                    if constexpr (REAL) at_l[q] = (uint32_t)u;
                }
                k += __popcll(heads);
            }
            if constexpr (REAL) {
                wave_sync();
                for (int q = lane; q < n; q += 64) {
                    int shift;
                    const int r = row_of(q, shift);
                    vals[(int64_t)(lo + (int)at_l[s_rep[wv][q]]) * TA + r] = s_val[wv][q];
                }
                if (lane < rows)
                    for (int q = b; q < e; ++q) {
                        const double x = (double)s_val[wv][q - lo];
                        sq = fma(x, x, sq);
                    }
            }
        } else {
            const int64_t shift = sbase + src - b;
            k = plan_merge<TA, REAL>([&](int q) { return col_idx[shift + q]; }, b, lane < TA ? e : b, lo, n, lane / TA,
                                     lane % TA, V, values, shift, plan, vals, sq, bad);
            k = __builtin_amdgcn_readfirstlane(k);
        }
        if (lane == 0) tiles[t] = make_int2(lo, k < n ? k : n);
        if (REAL && lane < rows) xsq[s0 + lane] = sq;
        wave_sync();  // the next tile's ids overwrite this one's
    }
    if (bad) atomicOr(flags, bad);
}

// -------------------------------------------------------------- finalize

// For each position k of the (possibly permuted) batch: smallest key over the strips; the winner's dot product comes from the sweep (the same fp32 sum of the
// row's weights in ascending feature order), so the full squared distance is
// (||w||^2 - 2*dot) + ||x||^2, with ||x||^2 = nnz for binary rows and xsq[k] from the
// plan for real-valued ones. Results are written by position (k_unpermute then moves
// them to their samples when the batch was regrouped): every write coalesced.
// Where a finalize kernel puts a position's result: the caller's arrays (positions are
// samples) or, for a regrouped batch, one staged record per position.
struct FinalOut {
    int32_t *bmu;
    double *dist;
    Staged *rec;  // non-null: staged
    __device__ void put(int64_t k, int32_t b, double d) const
    {
        if (rec) {
            rec[k] = Staged{d, b, 0};
        } else {
            bmu[k] = b;
            dist[k] = d;
        }
    }
};

// A finalize workgroup takes 64 positions (256 where one wave per 64 does); its waves share the strips (wave y takes strips
// y, y + waves, ...) and their results meet in LDS, so that a map of many strips does not
// put a chain of loads on one lane (1,024 x 1,024 map, 16,000 rows: 2,048 strips, 245 -> 48 us;
// two best on 256 x 256, 33 rows: 52 -> 8 us). A wave per eight strips, up to sixteen.
constexpr int kFinalizeBatch = 8;   // strips whose keys one lane loads at once
constexpr int kFinalize2Batch = 4;  // the same for the two-best search (four words per strip)
constexpr int kFinalizeWaves = 16;

inline int finalize_waves(int64_t n_strips)
{
    int64_t w = 1;
    while (w < kFinalizeWaves && w * kFinalizeBatch < n_strips) w *= 2;
    return (int)w;
}

// The batch's input flags: the plan's, or, for rows searched without a plan, each row's own
// (row pointers are judged for the batch, so every row's key tells), which the first
// workgroup gathers into the workspace's word.
struct FinalIn {
    const uint32_t *flags;
    const u64 *row_keys;  // non-null: no plan; the keys of strip 0
    uint32_t *gather;
    static __device__ unsigned flags_of(u64 key) { return (unsigned)((key & kKeyFlags) >> kKeyFlagShift); }
    __device__ int64_t rows(int64_t N, int64_t nnz) const
    {
        if (!row_keys) return rows_nnz(flags, nnz);
        if (blockIdx.x == 0 && threadIdx.y == 0 && threadIdx.x < 64) {
            unsigned f = 0;
#pragma unroll 8
            for (int64_t s = threadIdx.x; s < N; s += 64) f |= flags_of(row_keys[s]);
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) f |= (unsigned)__shfl_xor((int)f, d);
            gather[threadIdx.x] = threadIdx.x == 0 ? f : 0u;
        }
        return (flags_of(row_keys[0]) & SOM_FLAG_ROW_PTR) ? 0 : nnz;
    }
};

// Ids of position k's row (0 for a batch whose row pointers were flagged).
__device__ __forceinline__ double row_length(const int32_t *row_ptr, int rs, int64_t base, int64_t nnz, int64_t k)
{
    const int64_t rb = clamp64((int64_t)row_ptr[k * rs] - base, 0, nnz);
    return (double)(clamp64((int64_t)row_ptr[(k + 1) * rs] - base, rb, nnz) - rb);
}

__global__ __launch_bounds__(64 * kFinalizeWaves) void k_finalize(
    const double *__restrict__ norms, int64_t M, const int32_t *__restrict__ row_ptr, int rs, int64_t N, int64_t nnz,
    FinalIn in, const double *__restrict__ xsq, const u64 *__restrict__ keys,
    const float *__restrict__ dots, int64_t n_strips, int64_t pitch, FinalOut out)
{
    __shared__ u64 lk[kFinalizeWaves][64];
    __shared__ int ls[kFinalizeWaves][64];
    const int waves = (int)blockDim.y, y = (int)threadIdx.y;
    nnz = in.rows(N, nnz);
    const int64_t base = csr_base(row_ptr, nnz);
    for (int64_t k0 = (int64_t)blockIdx.x * blockDim.x; k0 < N; k0 += (int64_t)gridDim.x * blockDim.x) {  // uniform
        const int64_t k = k0 + threadIdx.x;
        u64 best = kKeyNone;
        int64_t gb = 0;
        if (k < N)
            for (int64_t g0 = y; g0 < n_strips; g0 += (int64_t)waves * kFinalizeBatch) {
                // a batch of strips' keys loaded before any is compared
                u64 kk[kFinalizeBatch];
#pragma unroll
                for (int j = 0; j < kFinalizeBatch; ++j)
                    kk[j] = g0 + j * waves < n_strips ? keys[(g0 + j * waves) * pitch + k] : kKeyNone;
                if (g0 == 0) kk[0] &= ~kKeyFlags;  // the flags that strip 0's key may carry
#pragma unroll
                for (int j = 0; j < kFinalizeBatch; ++j)
                    if (kk[j] < best) {
                        best = kk[j];
                        gb = g0 + j * waves;
                    }
            }
        if (waves > 1) {
            lk[y][threadIdx.x] = best;
            ls[y][threadIdx.x] = (int)gb;
            __syncthreads();
            if (y == 0)
                for (int j = 1; j < waves; ++j)
                    if (lk[j][threadIdx.x] < best) {
                        best = lk[j][threadIdx.x];
                        gb = ls[j][threadIdx.x];
                    }
        }
        if (y == 0 && k < N) {
            int64_t b = (int64_t)(best & kIndexMask);
            if (b >= M) b = M - 1;
            out.put(k, (int32_t)b, fma(-2.0, (double)dots[gb * pitch + k], norms[b]) +
                                       (xsq ? xsq[k] : row_length(row_ptr, rs, base, nnz, k)));
        }
        if (waves > 1) __syncthreads();
    }
}

// Two best units: the two smallest of the 2 * n_strips keys of each sample (each
// strip's two smallest), with their dot products from the sweep. Without a second
// unit (M == 1) bmu2 = -1 and dist2 = +inf.
struct TwoKeys {
    u64 k1, k2;
    float q1, q2;
    __device__ void offer(u64 key, float q)
    {
        if (key < k1) {
            k2 = k1;
            q2 = q1;
            k1 = key;
            q1 = q;
        } else if (key < k2) {
            k2 = key;
            q2 = q;
        }
    }
};

__global__ __launch_bounds__(64 * kFinalizeWaves) void k_finalize2(
    const double *__restrict__ norms, int64_t M, const int32_t *__restrict__ row_ptr, int rs, int64_t N, int64_t nnz,
    FinalIn in, const double *__restrict__ xsq, const u64 *__restrict__ keys,
    const float *__restrict__ dots, const u64 *__restrict__ keys2, const float *__restrict__ dots2, int64_t n_strips,
    int64_t pitch, FinalOut out, FinalOut out2)
{
    __shared__ TwoKeys lds[kFinalizeWaves][64];
    const int waves = (int)blockDim.y, y = (int)threadIdx.y;
    nnz = in.rows(N, nnz);
    const int64_t base = csr_base(row_ptr, nnz);
    for (int64_t k0 = (int64_t)blockIdx.x * blockDim.x; k0 < N; k0 += (int64_t)gridDim.x * blockDim.x) {  // uniform
        const int64_t k = k0 + threadIdx.x;
        TwoKeys t{kKeyNone, kKeyNone, 0.0f, 0.0f};
        if (k < N)
            for (int64_t g0 = y; g0 < n_strips; g0 += (int64_t)waves * kFinalize2Batch) {
                // a batch of strips' candidates loaded before any is offered
                u64 k1[kFinalize2Batch], k2[kFinalize2Batch];
                float d1[kFinalize2Batch], d2[kFinalize2Batch];
#pragma unroll
                for (int j = 0; j < kFinalize2Batch; ++j) {
                    const bool in = g0 + j * waves < n_strips;
                    const int64_t at = (g0 + j * waves) * pitch + k;
                    k1[j] = in ? keys[at] : kKeyNone;
                    d1[j] = in ? dots[at] : 0.0f;
                    k2[j] = in ? keys2[at] : kKeyNone;
                    d2[j] = in ? dots2[at] : 0.0f;
                }
                if (g0 == 0) k1[0] &= ~kKeyFlags;  // the flags that strip 0's key may carry
#pragma unroll
                for (int j = 0; j < kFinalize2Batch; ++j) {
                    t.offer(k1[j], d1[j]);
                    t.offer(k2[j], d2[j]);
                }
            }
        if (waves > 1) {
            lds[y][threadIdx.x] = t;
            __syncthreads();
            if (y == 0)
                for (int j = 1; j < waves; ++j) {
                    const TwoKeys o = lds[j][threadIdx.x];
                    t.offer(o.k1, o.q1);
                    t.offer(o.k2, o.q2);
                }
        }
        if (y == 0 && k < N) {
            const double len = xsq ? xsq[k] : row_length(row_ptr, rs, base, nnz, k);
            int64_t i1 = (int64_t)(t.k1 & kIndexMask);
            if (i1 >= M) i1 = M - 1;
            out.put(k, (int32_t)i1, fma(-2.0, (double)t.q1, norms[i1]) + len);
            if (t.k2 == kKeyNone) {
                out2.put(k, -1, __builtin_inf());
            } else {
                int64_t i2 = (int64_t)(t.k2 & kIndexMask);
                if (i2 >= M) i2 = M - 1;
                out2.put(k, (int32_t)i2, fma(-2.0, (double)t.q2, norms[i2]) + len);
            }
        }
        if (waves > 1) __syncthreads();
    }
}

// Results of a regrouped batch back to input order: sample s takes what position inv[s]
// got (bmu2/dist2 too when given). A sample never placed (inv[s] = -1, invalid row
// pointers only) is left untouched. Reads gather, writes run in sample order.
__global__ __launch_bounds__(256) void k_unpermute(const int32_t *__restrict__ inv, int64_t N,
                                                   const Staged *__restrict__ res, const Staged *__restrict__ res2,
                                                   int32_t *__restrict__ bmu,
                                                   double *__restrict__ dist, int32_t *__restrict__ bmu2,
                                                   double *__restrict__ dist2)
{
    for (int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x; s < N; s += (int64_t)gridDim.x * 256) {
        const int64_t k = inv[s];
        if (k < 0 || k >= N) continue;
        const Staged r = res[k];
        bmu[s] = r.b;
        dist[s] = r.d;
        if (bmu2) {
            const Staged r2 = res2[k];
            bmu2[s] = r2.b;
            dist2[s] = r2.d;
        }
    }
}

}  // namespace

// --------------------------------------------------------------- launchers

template <typename E>
static hipError_t norms_any(const E *W, int64_t V, int64_t M, double *norms, hipStream_t st)
{
    const int64_t blocks = (M + 63) / 64;
    // up to ten batches of 128 rows and a short rest are faster lane by lane: the pipeline's start
    // is not worth it (4,096 units, pipeline / lanes, us: 128 rows 7.2 / 6.4, 512 10.5 / 7.5, 1,024
    // 16.5 / 13.5; but 300 rows 8.2 / 9.1, 700 12.8 / 15.4, 30,000 rows 328 / 436), four batches of
    // fp16 rows on more than 8,192 units (16,384 units, 512 rows 11.3 / 9.4, 1,024 17.6 / 18.9)
    const bool batches = V >= 128 && V <= (sizeof(E) == 2 && blocks > 128 ? 512 + 27 : 1280) && V % 128 < 28;
    if (blocks <= kNormFewBlocks && !batches)
        hipLaunchKernelGGL(k_norms_few<E>, dim3((unsigned)blocks), dim3(64 * (kNormProducers + 1)), 0, st, W, V, M,
                           norms);
    else if (blocks < kNormWavesFew)
        hipLaunchKernelGGL((k_norms<E, 128>), dim3((unsigned)blocks), dim3(64), 0, st, W, V, M, norms);
    else
        hipLaunchKernelGGL((k_norms<E, 32>), dim3((unsigned)blocks), dim3(64), 0, st, W, V, M, norms);
    return hipGetLastError();
}

hipError_t launch_norms(const float *W, int64_t V, int64_t M, double *norms, hipStream_t st)
{
    return norms_any(W, V, M, norms, st);
}

hipError_t launch_norms_f16(const uint16_t *W, int64_t V, int64_t M, double *norms, hipStream_t st)
{
    return norms_any(reinterpret_cast<const _Float16 *>(W), V, M, norms, st);
}

hipError_t launch_check_rows(const int32_t *row_ptr, int64_t N, int64_t nnz, uint32_t *flags, hipStream_t st)
{
    if (N <= kCheckFew) {
        hipLaunchKernelGGL(k_check_few, dim3(1), dim3(1024), 0, st, row_ptr, N, nnz, flags);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_clear_flags, dim3(1), dim3(64), 0, st, flags);
    int64_t blocks = (N + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_check_rows, dim3((unsigned)blocks), dim3(256), 0, st, row_ptr, N, nnz, flags);
    return hipGetLastError();
}

// Whether tiles of 8 are planned by ranks: their mean leaves room below kRankIds, and they are
// few. The ranks take one wave and about 950 instructions a tile, the merge an eighth of a wave
// for a dependent step per union entry (about 90 at 12 ids a row), so the merge wins once its
// waves fill the chip, the sooner the shorter the rows; real-valued rows, whose merge also waits
// for each value, later. Plan by ranks / by the merge, us, by rows: 1.9 ids a row 12.0 / 11.8 at
// 60,000, 17.6 / 11.9 at 130,000; 3.6 ids 15.7 / 15.6 at 95,000; 11 ids 16.0 / 28.4 at 40,000, 29.4 /
// 29.0 at 110,000; 20 ids 48.6 / 54.0 at 130,000. Real-valued: 1.9 ids 14.0 / 13.1 at 60,000; 3.6 ids
// 21.9 / 21.3 at 110,000; 11 ids 41.0 / 44.4 at 130,000, 49.6 / 46.5 at 170,000; 20 ids 102 / 199 at
// 260,000. The merge reads a regrouped row lane by lane, the ranks read any row side by side
// (plan with regrouping: 11 ids 70.5 / 69.6 at 130,000; 3.7 ids 108.7 / 108.0 at 110,000;
// real-valued, 11 ids 102 / 109 at 200,000, 122 / 127 at 260,000).
static bool plan_by_ranks(int64_t N, int64_t nnz, int64_t nt, bool real, bool regrouped)
{
    if (nnz * 8 > N * (kRankIds / 2)) return false;
    if (regrouped) return nt <= (nnz < 5 * N ? 13312 : (real ? 32768 : 16384));
    if (nnz < 3 * N) return nt <= 6144;
    if (!real) return nt <= (nnz < 16 * N ? 13312 : 16384);
    return nt <= (nnz < 5 * N ? 13312 : (nnz < 16 * N ? 20480 : 32768));
}

hipError_t launch_plan(int ta, const int32_t *row_ptr, const int32_t *col_idx, const float *values, int64_t N,
                       int64_t nnz, int64_t V, const OrderBuffers *ob, uint2 *plan, int2 *tiles, float *vals,
                       double *xsq, uint32_t *flags, hipStream_t st)
{
    const int64_t nt = n_tiles(N, ta);
    const int64_t per_block = (int64_t)kPlanWaves * (64 / ta);
    int64_t blocks = (nt + per_block - 1) / per_block;
    if (blocks > (1 << 22)) blocks = 1 << 22;
    const dim3 grid((unsigned)blocks), block(256);
    const int32_t v = (int32_t)V;
    // a regrouped batch's offsets and sources are interleaved in ob->pos
    const int32_t *off = ob ? ob->pos : row_ptr;
    const int32_t *psrc = ob ? ob->pos + 1 : nullptr;
    const int os = ob ? 2 : 1;
    if (ta == 8 && plan_by_ranks(N, nnz, nt, xsq != nullptr, ob != nullptr)) {
        int64_t rb = (nt + kPlanWaves - 1) / kPlanWaves;
        if (rb > (1 << 22)) rb = 1 << 22;
        if (xsq)  // real-valued rows (values is null when the batch holds no id)
            hipLaunchKernelGGL(k_plan_rank<true>, dim3((unsigned)rb), block, 0, st, off, os, row_ptr, psrc, col_idx, N,
                               nnz, v, nt, plan, tiles, flags, values, vals, xsq);
        else
            hipLaunchKernelGGL(k_plan_rank<false>, dim3((unsigned)rb), block, 0, st, off, os, row_ptr, psrc, col_idx,
                               N, nnz, v, nt, plan, tiles, flags, nullptr, nullptr, nullptr);
        return hipGetLastError();
    }
    if (xsq) {  // real-valued rows: tiles of 8 only
        if (ta != 8) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_plan<8, true>), grid, block, 0, st, off, os, row_ptr, psrc, col_idx, N, nnz, v, nt,
                           plan, tiles, flags, values, vals, xsq);
        return hipGetLastError();
    }
    switch (ta) {
    case 8:
        hipLaunchKernelGGL((k_plan<8, false>), grid, block, 0, st, off, os, row_ptr, psrc, col_idx, N, nnz, v, nt,
                           plan, tiles, flags, nullptr, nullptr, nullptr);
        break;
    case 16:
        hipLaunchKernelGGL((k_plan<16, false>), grid, block, 0, st, off, os, row_ptr, psrc, col_idx, N, nnz, v, nt,
                           plan, tiles, flags, nullptr, nullptr, nullptr);
        break;
    case 32:
        hipLaunchKernelGGL((k_plan<32, false>), grid, block, 0, st, off, os, row_ptr, psrc, col_idx, N, nnz, v, nt,
                           plan, tiles, flags, nullptr, nullptr, nullptr);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_finalize(int ta, const double *norms, int64_t M, const int32_t *row_ptr, int64_t N, int64_t nnz,
                           const OrderBuffers *ob, const double *xsq, const SweepOut &o, int32_t *bmu, double *dist,
                           int32_t *bmu2, double *dist2, hipStream_t st)
{
    // rows without a plan fill strips of 512, each the first of two at tiles of 16 and 32
    const bool wide = o.direct && ta != 8;
    const int64_t ns = n_strips(M, wide ? 8 : ta), pitch = wide ? 2 * N : N;  // pitch: from a strip's keys to the next's
    const int waves = finalize_waves(ns);
    const dim3 block(waves > 1 ? 64 : 256, (unsigned)waves);
    int64_t blocks = (N + block.x - 1) / block.x;
    if (blocks > (1 << 22)) blocks = 1 << 22;
    // a regrouped batch is finalized by position into the workspace first, with its row
    // lengths from the interleaved offsets of its positions
    const FinalOut o1{bmu, dist, ob ? ob->res : nullptr}, o2{bmu2, dist2, ob ? ob->res2 : nullptr};
    const int32_t *rp = ob ? ob->pos : row_ptr;
    const int rs = ob ? 2 : 1;
    const FinalIn fin{o.flags, o.direct ? o.keys : nullptr, o.direct ? o.direct->flags : nullptr};
    if (bmu2)
        hipLaunchKernelGGL(k_finalize2, dim3((unsigned)blocks), block, 0, st, norms, M, rp, rs, N, nnz, fin, xsq,
                           o.keys, o.dots, o.keys2, o.dots2, ns, pitch, o1, o2);
    else
        hipLaunchKernelGGL(k_finalize, dim3((unsigned)blocks), block, 0, st, norms, M, rp, rs, N, nnz, fin, xsq,
                           o.keys, o.dots, ns, pitch, o1);
    if (ob) {
        int64_t ub = (N + 255) / 256;
        if (ub > (1 << 22)) ub = 1 << 22;
        hipLaunchKernelGGL(k_unpermute, dim3((unsigned)ub), dim3(256), 0, st, ob->inv, N, ob->res,
                           bmu2 ? ob->res2 : nullptr, bmu, dist, bmu2, dist2);
    }
    return hipGetLastError();
}

hipError_t launch_order(const int32_t *row_ptr, const int32_t *col_idx, int64_t N, int64_t nnz, int64_t V,
                        const OrderBuffers &ob, uint32_t *flags, hipStream_t st)
{
    const int64_t nb = V + 1;  // one bucket per feature, one for rows without a valid feature
    int64_t fb = (nb + 255) / 256;
    if (fb > 4096) fb = 4096;
    hipLaunchKernelGGL(k_order_clear, dim3((unsigned)fb), dim3(256), 0, st, ob.freq, ob.bucket, nb);
    // a workgroup per 16,384 ids (two rounds of its lanes' loads), up to the compute units:
    // the larger histogram fills a unit's LDS, and every workgroup adds its bins at the end
    const int64_t counted = nnz < kFreqSample ? nnz : kFreqSample;
    int64_t hb = (counted + 16383) / 16384;
    if (hb < 1) hb = 1;
    if (hb > 256) hb = 256;
    if (V <= 8192)
        hipLaunchKernelGGL(k_freq<8192>, dim3((unsigned)hb), dim3(kFreqThreads), 0, st, row_ptr, col_idx, counted,
                           (int32_t)V, ob.freq);
    else
        hipLaunchKernelGGL(k_freq<kLdsHistMax>, dim3((unsigned)hb), dim3(kFreqThreads), 0, st, row_ptr, col_idx,
                           counted, (int32_t)V, ob.freq);
    int64_t qb = (N + 63) / 64;  // a row per quad of lanes
    if (qb > (1 << 22)) qb = 1 << 22;
    hipLaunchKernelGGL(k_rarest, dim3((unsigned)qb), dim3(256), 0, st, row_ptr, col_idx, N, nnz, (int32_t)V, ob.freq,
                       ob.skey, ob.bucket, ob.rank, flags);
    hipLaunchKernelGGL(k_bucket_scan, dim3(1), dim3(1024), 0, st, ob.bucket, nb, nnz, ob.pos + 2 * N);
    int64_t pb = (N + 255) / 256;
    if (pb > (1 << 22)) pb = 1 << 22;
    hipLaunchKernelGGL(k_place, dim3((unsigned)pb), dim3(256), 0, st, row_ptr, N, nnz, ob.skey, ob.bucket, ob.rank, nb,
                       ob.inv, ob.pos, flags);
    return hipGetLastError();
}

}  // namespace som
