// som_rows.hip -- the search of a few rows (gfx950): no plan, each wave one row and one
// strip, read straight from the caller's batch.
//
// A search of a handful of rows is a chain of dependent kernels and of dependent loads
// inside them; the codebook rows it reads are few. The planned sweep needs four launches
// and, per tile of eight samples, a walk over about 85 union rows of which four to eight
// are in flight. Here a wave has the ids of its one row after two round trips and then
// its dozen codebook rows in one or two more, and the finalize follows: two launches.
// Without a union nothing is shared between rows, so this is for few of them (rows_direct).
//
// The result is the planned sweep's, bit for bit: the same fp32 sum in the row's order,
// the same two-stage ranking (an fp32 bound, then fp64 keys of the neurons within it; see
// k_sweep for the bound), one key and dot product per row and strip.
//
// The waves of strip 0 also leave a plan in the workspace, as a search with a plan would: a
// tile's entries are its rows' ids one row after the other, each held by its own sample
// alone. It is longer than a merged one where rows share features, and a sweep of it adds
// every sample's weights in the same order.

#include "som_device.h"

namespace som {
namespace {

// Neurons per lane: strips of 512. Tiles of 16 and 32 lay the workspace's keys out in strips of
// 256: a wave then fills the first of its two and leaves no key in the second.
constexpr int kNpl = 8;

template <typename E, int LD, bool TOP2, bool REAL>
__global__ __launch_bounds__(64) void k_rows(const E *__restrict__ W, const double *__restrict__ norms, int64_t M,
                                             int64_t N, int64_t V, int64_t nnz, const int32_t *__restrict__ row_ptr,
                                             const int32_t *__restrict__ col_idx, const float *__restrict__ values,
                                             u64 *__restrict__ keys, float *__restrict__ dots,
                                             u64 *__restrict__ keys2, float *__restrict__ dots2,
                                             double *__restrict__ xsq, int ta, uint2 *__restrict__ plan,
                                             int2 *__restrict__ tiles, float *__restrict__ vals)
{
    constexpr int G = group_elems<E, kNpl>();
    constexpr int U = sizeof(E) == 2 ? 16 : 8;  // codebook rows in flight: 64 registers
    typedef E vec __attribute__((ext_vector_type(G)));
    typedef vec any __attribute__((aligned(sizeof(E))));
    const int lane = threadIdx.x;
    const int Mi = (int)M;
    const int64_t strip = blockIdx.x, row = blockIdx.y;
    const int base = (int)strip * (64 * kNpl);
    // Element j's neuron as in k_sweep: groups of G, the last ones of a row read shifted back
    // to end with it and their elements before the group's own start not ranked.
    auto own = [&](int j) { return base + (j / G) * (64 * G) + lane * G; };
    auto group_at = [&](int j) { return LD == kLoadScalar ? own(j) : min(own(j), Mi - G); };
    auto neuron = [&](int j) { return group_at(j) + j % G; };
    auto ranked = [&](int j) { return neuron(j) >= own(j) && neuron(j) < Mi; };

    // the whole batch's row pointers, as k_check_rows would see them
    const int64_t first = row_ptr[0];
    bool bad = first < 0;
#pragma unroll 8
    for (int64_t s = lane; s < N; s += 64) bad |= row_bad(row_ptr, first, nnz, s);
    const bool flagged = __ballot(bad) != 0;
    const int64_t rb = flagged ? 0 : row_ptr[row], re = flagged ? 0 : row_ptr[row + 1];

    const int shift = ta == 8 ? 3 : (ta == 16 ? 4 : 5);  // 2^shift samples per tile
    const int slot = (int)row & ((1 << shift) - 1);

    double nrm[kNpl];
    float nf[kNpl], nmax_l = 0.0f;
#pragma unroll
    for (int j = 0; j < kNpl; ++j) {
        nrm[j] = ranked(j) ? norms[neuron(j)] : __builtin_inf();
        nf[j] = (float)nrm[j];
        if (ranked(j)) nmax_l = fmaxf(nmax_l, nf[j]);
    }
    float acc[kNpl];
#pragma unroll
    for (int j = 0; j < kNpl; ++j) acc[j] = 0.0f;
    double sq = 0.0;
    unsigned flag = flagged ? SOM_FLAG_ROW_PTR : 0u;
    int prev = -1;
    for (int64_t p0 = rb; p0 < re; p0 += 64) {  // uniform
        const int n = (int)(re - p0 < 64 ? re - p0 : 64);
        const int id = lane < n ? col_idx[p0 + lane] : -1;
        float x = 0.0f;
        if constexpr (REAL) x = lane < n ? values[p0 + lane] : 0.0f;
        const bool in = lane < n && id >= 0 && id < V;
        const u64 valid = __ballot(in);
        if (__ballot(lane < n && !in)) flag |= SOM_FLAG_ID_RANGE;
        // each valid id against the valid one before it
        const u64 below = valid & ((1ull << lane) - 1ull);
        const int left = __shfl(id, below ? 63 - __builtin_clzll(below) : 0);
        if (__ballot(in && id <= (below ? left : prev))) flag |= SOM_FLAG_UNSORTED;
        if (valid) prev = __builtin_amdgcn_readlane(id, 63 - __builtin_clzll(valid));
        for (int k = 0; k < n; k += U) {
            union {
                vec v[U][kNpl / G];
                E e[U][kNpl];
            } seg;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (k + u >= n) break;  // uniform
                const int i = __builtin_amdgcn_readlane(id, k + u);
                const E *r = W + (uint64_t)((valid >> (k + u)) & 1 ? (unsigned)i : 0u) * (uint64_t)(unsigned)Mi;
                if constexpr (LD == kLoadScalar) {
#pragma unroll
                    for (int j = 0; j < kNpl; ++j) seg.e[u][j] = r[min(neuron(j), Mi - 1)];
                } else {
#pragma unroll
                    for (int q = 0; q < kNpl / G; ++q)
                        seg.v[u][q] = *reinterpret_cast<const any *>(r + group_at(q * G));
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (k + u >= n) break;
                if (!((valid >> (k + u)) & 1)) continue;  // an id outside [0, V) is left out
                const float xv =
                    REAL ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), k + u)) : 1.0f;
                if constexpr (REAL) sq = fma((double)xv, (double)xv, sq);
#pragma unroll
                for (int j = 0; j < kNpl; ++j) {
                    const float w = (float)seg.e[u][j];
                    acc[j] = REAL ? fmaf(xv, w, acc[j]) : acc[j] + w;
                }
            }
        }
        // after the loads, which would wait for stores before them
        if (strip == 0 && lane < n) {
            const int64_t at = p0 + lane - first;
            plan[at] = make_uint2((unsigned)id, plan_word_one(1 << shift, slot, in));
            if constexpr (REAL) vals[(at << shift) + slot] = x;
        }
    }

    // stage 1: the fp32 bound that holds the neurons of the smallest key (two smallest keys)
    const float nmax = wave_max_f32(nmax_l);
    float da[kNpl], m1 = __builtin_inff(), m2 = __builtin_inff();
#pragma unroll
    for (int j = 0; j < kNpl; ++j) {
        da[j] = fmaf(-2.0f, acc[j], nf[j]);
        m2 = fminf(m2, fmaxf(m1, da[j]));
        m1 = fminf(m1, da[j]);
    }
    float thr;
    if constexpr (TOP2) {
        float w1, w2;
        wave_min2_f32(m1, m2, w1, w2);
        thr = w2 + 0x1p-20f * (nmax + fabsf(w1) + fabsf(w2) + 1.0f);
    } else {
        const float w1 = wave_min_f32(m1);
        thr = w1 + 0x1p-20f * (nmax + fabsf(w1) + 1.0f);
    }
    const bool every = !(fabsf(thr) <= __FLT_MAX__);
    // stage 2: their fp64 keys
    u64 k1 = kKeyNone, k2 = kKeyNone;
    float q1 = 0.0f, q2 = 0.0f;
#pragma unroll
    for (int j = 0; j < kNpl; ++j) {
        if (!ranked(j) || !(every || da[j] <= thr)) continue;
        const u64 key = rank_key(fma(-2.0, (double)acc[j], nrm[j]), (unsigned)neuron(j));
        if (key < k1) {
            k2 = k1;
            q2 = q1;
            k1 = key;
            q1 = acc[j];
        } else if (TOP2 && key < k2) {
            k2 = key;
            q2 = acc[j];
        }
    }
    auto owner_of = [&](u64 mine, u64 best) {
        const u64 h = __ballot(mine == best);
        return h ? __builtin_ctzll(h) : 0;
    };
    const u64 K1 = wave_min_u64(k1);
    const int o1 = owner_of(k1, K1);
    const float D1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q1), o1));
    const int64_t at = (shift == 3 ? strip : 2 * strip) * N + row;
    const bool second = shift != 3 && base + 32 * kNpl < Mi;  // the other strip of 256
    if (lane == 0) {
        keys[at] = strip == 0 ? (K1 & ~kKeyFlags) | (u64)flag << kKeyFlagShift : K1;
        dots[at] = D1;
        if (second) {
            keys[at + N] = kKeyNone;
            dots[at + N] = 0.0f;
        }
    }
    if constexpr (TOP2) {
        const u64 nxt = lane == o1 ? k2 : k1;  // keys are distinct: each holds its neuron
        const float nq = lane == o1 ? q2 : q1;
        const u64 K2 = wave_min_u64(nxt);
        const float D2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(nq), owner_of(nxt, K2)));
        if (lane == 0) {
            keys2[at] = K2;
            dots2[at] = D2;
            if (second) {
                keys2[at + N] = kKeyNone;
                dots2[at + N] = 0.0f;
            }
        }
    }
    if (strip == 0 && lane == 0) {
        if constexpr (REAL) xsq[row] = sq;
        if (slot == 0) {
            const int64_t end = row + (1 << shift) < N ? row + (1 << shift) : N;
            tiles[row >> shift] = flagged ? make_int2(0, 0) : make_int2((int)(rb - first), (int)(row_ptr[end] - rb));
        }
    }
}

template <typename E, bool TOP2, bool REAL>
hipError_t rows_any(const void *w, const double *norms, int64_t M, int64_t N, int64_t V, int64_t nnz,
                    const SweepOut &o, hipStream_t st)
{
    const E *W = static_cast<const E *>(w);
    const DirectRows &d = *o.direct;
    const dim3 grid((unsigned)n_strips(M, 8), (unsigned)N);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(64), 0, st, W, norms, M, N, V, nnz, d.row_ptr, d.col_idx, d.values,
                           o.keys, o.dots, o.keys2, o.dots2, d.xsq, d.ta, d.plan, d.tiles, d.vals);
    };
    if (M >= group_elems<E, kNpl>())
        launch(k_rows<E, kLoadAny, TOP2, REAL>);
    else
        launch(k_rows<E, kLoadScalar, TOP2, REAL>);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_rows(bool f16, bool top2, const void *W, const double *norms, int64_t M, int64_t N, int64_t V,
                       int64_t nnz, const SweepOut &o, hipStream_t st)
{
    const bool real = o.direct->xsq != nullptr;
    if (real && o.direct->ta != 8) return hipErrorInvalidValue;
    static_assert(neurons_per_lane(8) == kNpl && 2 * neurons_per_lane(16) == kNpl && 2 * neurons_per_lane(32) == kNpl,
                  "the strips that a wave fills");
    auto pick = [&](auto e) {
        typedef decltype(e) E;
        if (real)
            return top2 ? rows_any<E, true, true>(W, norms, M, N, V, nnz, o, st)
                        : rows_any<E, false, true>(W, norms, M, N, V, nnz, o, st);
        return top2 ? rows_any<E, true, false>(W, norms, M, N, V, nnz, o, st)
                    : rows_any<E, false, false>(W, norms, M, N, V, nnz, o, st);
    };
    return f16 ? pick(_Float16{}) : pick(float{});
}

}  // namespace som
