// som_internal.h -- shared between the C-ABI layer and the kernels of libsom.so.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "som.h"

namespace som {

// Tile sizes (samples per tile) the library is built for, and the default.
constexpr int kDefaultTileSamples = SOM_DEFAULT_TILE_SAMPLES;
inline bool valid_tile(int ta) { return ta == 8 || ta == 16 || ta == 32; }

// Neurons per lane of the sweep: 8 (two 16-byte loads per codebook row) for tiles of 8
// samples, 4 for larger tiles, so that the TA x NPL register accumulators stay at
// 64 or 128 VGPRs. One wave covers a strip of 64 * NPL neurons.
constexpr int neurons_per_lane(int ta) { return ta <= 8 ? 8 : 4; }
inline int64_t strip_neurons(int ta) { return 64 * neurons_per_lane(ta); }
inline int64_t n_strips(int64_t M, int ta) { return (M + strip_neurons(ta) - 1) / strip_neurons(ta); }
inline int64_t n_tiles(int64_t N, int ta) { return (N + ta - 1) / ta; }

// Sizes at which a search may read its rows without a plan (som_rows.hip). That saves two
// launches and the walk over tiles' unions, and reads a codebook row once per sample instead
// of once per tile: it wins while the rows times the units are few. Without / with the plan,
// us, fp32, 12 ids a row: 64 x 64 map 13.8 / 27 at one row, 15 / 36 at 512, 23 / 37 at 1,024,
// 44 / 44 at 2,048; 256 x 256 28 / 43 at 64, 88 / 101 at 256, 165 / 161 at 512; 512 x 512
// 61 / 86 at 33, 114 / 114 at 64 (fp16: 62 / 67); 16 x 16 map 14 / 33 at 2,048, 22 / 33 at
// 4,096; 32 x 32 19 / 36 at 2,048, 36 / 37 at 4,096.
inline bool few_rows(int64_t N, int64_t M, int ta)
{
    const int64_t pairs = N * M;
    return (N <= 256 && pairs <= (int64_t)1 << 24) ||
           (ta == 8 && ((N <= 1024 && pairs <= (int64_t)1 << 23) || (N <= 4096 && pairs <= (int64_t)3 << 20)));
}

// Whether it does at nnz ids in all. Longer rows keep to the line above while a launch is
// short of waves, since a plan's walk grows with the row too. Once it is not, the codebook
// rows that samples share are read by each of them, and the ids times the units are the work.
// Without / with the plan, us, by the rows and the ids of each (tests on Zipf rows, V = 30,000):
// - up to 2^15 units, fp32: 64 x 64, 1,024 rows of 1,000 889 / 3,100; 128 x 128, 512 of 4,000 9,384 /
//   12,670; 32 x 32, 3,000 of 15,000 10,743 / 21,973;
// - up to 2^17: 256 x 256, 64 of 4,000 7,344 / 7,868; 96 of 1,000 2,858 / 3,590; 256 of 200 1,473 /
//   1,487, of 400 3,020 / 2,750; fp16 64 of 4,000 3,518 / 6,821, 192 of 1,000 2,736 / 3,451;
// - above: 512 x 512, 16 of 1,000 2,464 / 2,886, of 4,000 9,863 / 8,582; 32 of 400 1,949 / 1,703; 64 of
//   100 908 / 797, of 1,000 9,863 / 6,198; fp16 64 of 200 925 / 972, of 400 1,847 / 1,722.
// Below 5 * 2^20 pairs the plan's launch has a quarter of the chip's waves. A single row
// shares nothing.
inline bool rows_direct(int64_t N, int64_t M, int64_t nnz, int ta, bool f16)
{
    if (!few_rows(N, M, ta)) return false;
    const bool thin = N * M <= (int64_t)5 << 20;
    int64_t most, times16 = 4;  // ids times units; so many times that with fp16 rows
    if (M <= 1 << 15) {
        most = (int64_t)1 << 36;
    } else if (M <= 1 << 17) {
        most = (int64_t)(thin ? 16 : 6) << 30;
        times16 = 2;
    } else {
        most = (int64_t)(thin ? 12 : 3) << 29;
    }
    return N == 1 || nnz * M <= (f16 ? times16 : 1) * most;
}

// Whether regrouping a batch by rarest features pays (its caller allowing it). Six kernels
// and the scattered reads they cause cost 35-45 us and 0.2 ns a row; the sweep then reads
// rare rows from L2 more often, 1% faster at 16,000 rows and 18-21% at 2,000,000 (fp32;
// 4-6% for fp16), where the strips do not fit there anyway, and far more where rows
// resemble each other. A batch's likeness is not known beforehand, so the line lies where
// independent rows lose at most a tenth and like ones do not yet gain more: from 9 * 2^28
// ids times units on, at 12 ids a row 49,000 rows on a 64 x 64 map. Whole searches, us, fp32,
// V = 30,000, regrouped / as given, for independent rows; for eight variants of each row (a tenth
// of the ids changed); for eight copies: 64 x 64 map 335 / 305, 216 / 277, 166 / 273 at 32,000 rows,
// 555 / 556, 376 / 530, 281 / 522 at 64,000; 128 x 128 635 / 606, 412 / 534, 288 / 509 at 16,000;
// 256 x 256 491 / 446, 326 / 369, 183 / 339 at 2,000, 801 / 758, 490 / 600, 297 / 561 at 4,000;
// 22 x 22 592 / 578, 462 / 576, 400 / 578 at 512,000. Longer rows gain as the product says (fp16
// 64 x 64, 30,000 rows of 200 ids 1,984 / 2,502). Maps of up to 256 units, half a strip, read too
// little per row (16 x 16, 2,000,000 rows 1,673 / 1,558, 1,534 / 1,555, 1,432 / 1,561).
// fp16 sweeps gain less (64 x 64, 64,000 rows 365 / 337, 320 / 334, 276 / 334); the plan and the
// finalize do not know the codebook's type. Nor do they know of a search that ran without a
// plan: its workspace holds the rows in the order given, so wherever one may (an fp16 one, the
// wider line) the phases regroup nothing.
inline bool regroup_pays(int64_t N, int64_t M, int64_t nnz, int ta)
{
    return M > 256 && nnz * M >= (int64_t)9 << 28 && !rows_direct(N, M, nnz, ta, true);
}

// Consecutive tiles per sweep workgroup. Longer groups let a wave keep its strip's
// norms over several tiles and keep the tiles in flight a compact stretch of the
// (regrouped) batch, but a strip must still span enough rounds of resident workgroups, or
// the chip works on two strips at once and their rows compete for L2.
// fp32: 8 tiles from 12,000 on, then one in 16,384, up to 32 (V = 20,000, ms by group size:
// 64 x 64, 31,250 tiles 1.48 at 4, 1.43 at 8 and 12, 1.50 at 32; 128 x 128, 15,000 tiles 2.86,
// 2.82, 2.87, 3.36; 256 x 256, 7,500 tiles 6.12, 6.22, 6.54, 8.52; 1024 x 1024, 62,500 tiles
// 784, 769, 812, 835; whole searches, V = 30,000, 64 x 64: 125,000 tiles 6.39 at 4, 6.32 at 8,
// 6.34 at 12, 6.39 at 24; 250,000 tiles 12.60, 12.44, 12.45, 12.48).
// fp16 rows are half as long, so two strips at once still fit and the tile's prologue and
// neighbourhood count for more: 8 tiles from 1,500 on, 12 from 6,000, 16 from 12,000, 24 from
// 20,000, 32 from 30,000 (256 x 256: 2,000 tiles 1.24 at 4, 1.20 at 8, 1.50 at 32; 7,500 tiles
// 4.23, 4.01, 3.92; 25,000 tiles 13.46, 12.62, 11.99; 1024 x 1024, 62,500 tiles 552, 520, 491).
// Tiles of 16 and 32 keep the line they were measured with.
//
// Those lines are for maps of many strips. All strips together must also give the chip
// enough workgroups: it holds 1,024 of them, and a last round that is half empty costs more
// than longer groups bring. So groups of tiles of 8 are shortened until there are kGroupRounds
// rounds (whole searches, us, by the lines above alone / bounded so: fp16 16 x 16, 12,000 rows
// 47 / 36, 100,000 rows 111 / 103; fp16 32 x 32, 50,000 rows 121 / 100; fp16 64 x 64, 250,000
// rows 1,183 / 1,161; fp32 32 x 32, 100,000 rows 260 / 244; elsewhere the same within 1%).
constexpr int64_t kResidentGroups = 1024;
constexpr int64_t kGroupRounds = 13, kGroupRoundsF16 = 8;

inline int64_t sweep_group_tiles(int64_t nt, int64_t strips, int ta, bool f16)
{
    int64_t g = nt / 16384 / 4 * 4;
    if (ta != 8) {
        if (g < 8 && nt >= 8 * 7500) g = 8;
        return g < 4 ? 4 : (g > 32 ? 32 : g);
    }
    if (f16)
        g = nt >= 30000 ? 32 : nt >= 20000 ? 24 : nt >= 12000 ? 16 : nt >= 6000 ? 12 : nt >= 1500 ? 8 : 4;
    else if (g < 8 && nt >= 12000)
        g = 8;
    const int64_t most = nt * strips / ((f16 ? kGroupRoundsF16 : kGroupRounds) * kResidentGroups) / 4 * 4;
    g = g < most ? g : most;
    return g < 4 ? 4 : (g > 32 ? 32 : g);
}

// One position's result of a regrouped batch, staged in the workspace: a whole 16-byte
// record, so the finalize writes full lines and the move back to input order reads one
// record per sample.
struct alignas(16) Staged {
    double d;
    int32_t b;
    int32_t pad;
};

// Workspace carve-up (offsets in bytes from the workspace base; every section 256-byte aligned).
// The order sections are empty when the caller keeps the given sample order.
struct Layout {
    size_t flags;   // uint32 [64]: input flags
    size_t plan;    // uint2 [nnz]: (feature id, sample mask) of every tile's union, tile t at its CSR offset
    size_t tiles;   // int2 [n_tiles]: (plan offset, union size) per tile
    size_t keys;    // uint64 [n_strips * N]: per-strip partial argmin keys, strip-major, by batch position
    size_t dots;    // float [n_strips * N]: fp32 dot product of the neuron each key names
    size_t freq;    // uint32 [V+1]: feature counts of the batch
    size_t bucket;  // uint64 [V+1]: per-bucket (samples << 32 | ids) counts, then offsets
    size_t skey;    // int32 [N]: each sample's bucket
    size_t rank;    // uint64 [N]: each sample's rank in its bucket (samples << 32 | ids before it)
    size_t inv;     // int32 [N]: each sample's position in the ordered batch (-1: never placed)
    size_t pos;     // int32 [2N+2]: per position p of the ordered batch, pos[2p] = its row offset and
                    // pos[2p+1] = where its ids start in the caller's col_idx; pos[2N] = all ids
    size_t res;     // Staged [N]: best unit and distance by position, before they go back to input order
    size_t keys2;   // uint64 [n_strips * N]: per-strip second-smallest keys (two-best search only)
    size_t dots2;   // float [n_strips * N]: their dot products (two-best search only)
    size_t res2;    // Staged [N]: second unit and distance by position (two-best search, ordered batch only)
    size_t vals;    // float [nnz * TA]: sample values of every plan entry (real-valued rows only)
    size_t xsq;     // double [N]: ||x||^2 by batch position (real-valued rows only)
    size_t total;
};

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// The two-best sections follow the single-best ones and the real-valued sections
// follow those, so each smaller layout is a prefix of the larger ones.
inline Layout layout_for(int64_t N, int64_t M, int64_t V, int64_t nnz, int ta, bool order, bool top2 = false,
                         bool real = false)
{
    Layout L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align256(bytes);
        return at;
    };
    L.flags = take(256);  // first, so that its place does not depend on the sizes or the config
    L.plan = take((size_t)nnz * 8);
    L.tiles = take((size_t)n_tiles(N, ta) * 8);
    L.keys = take((size_t)n_strips(M, ta) * (size_t)N * 8);
    L.dots = take((size_t)n_strips(M, ta) * (size_t)N * 4);
    const size_t o = order ? 1 : 0;
    L.freq = take(o * (size_t)(V + 1) * 4);
    L.bucket = take(o * (size_t)(V + 1) * 8);
    L.skey = take(o * (size_t)N * 4);
    L.rank = take(o * (size_t)N * 8);
    L.inv = take(o * (size_t)N * 4);
    L.pos = take(o * (size_t)(N + 1) * 8);
    L.res = take(o * (size_t)N * sizeof(Staged));
    const size_t t2 = top2 ? 1 : 0;
    L.keys2 = take(t2 * (size_t)n_strips(M, ta) * (size_t)N * 8);
    L.dots2 = take(t2 * (size_t)n_strips(M, ta) * (size_t)N * 4);
    L.res2 = take(t2 * o * (size_t)N * sizeof(Staged));
    const size_t r = real ? 1 : 0;
    L.vals = take(r * (size_t)nnz * (size_t)ta * 4);
    L.xsq = take(r * (size_t)N * 8);
    L.total = off;
    return L;
}

struct OrderBuffers {
    uint32_t *freq;
    unsigned long long *bucket, *rank;
    int32_t *skey, *inv, *pos;
    Staged *res, *res2;  // results by position (res2: two-best only)
};

// A few rows searched without a plan (som_rows.hip): the caller's batch, and what the
// sweep leaves besides the keys: ||x||^2, and the plan for a later phase call.
struct DirectRows {
    const int32_t *row_ptr, *col_idx;
    const float *values;
    int ta;           // samples per tile of the plan
    uint2 *plan;
    int2 *tiles;
    float *vals;      // real-valued rows only, as xsq (else null)
    double *xsq;
    uint32_t *flags;  // the workspace's input flags, which the finalize writes
};

// Where the sweep leaves its per-(sample, strip) results.
struct SweepOut {
    unsigned long long *keys;
    float *dots;
    unsigned long long *keys2;  // two-best only, else null
    float *dots2;
    const uint32_t *flags;  // the plan's input flags: a batch with bad row pointers has empty rows
    const DirectRows *direct;  // non-null: rows searched without a plan
};

// Records the calling thread's error text (som_last_error) and returns st.
som_status set_error(som_status st, const char *fmt, ...) __attribute__((format(printf, 2, 3)));

// Kernel launchers (som_kernels.hip). Each returns the launch's hipError_t.
hipError_t launch_norms(const float *W, int64_t V, int64_t M, double *norms, hipStream_t st);
// fp16 codebooks: W holds IEEE binary16 bit patterns.
hipError_t launch_norms_f16(const uint16_t *W, int64_t V, int64_t M, double *norms, hipStream_t st);
// Clears the flags, then sets SOM_FLAG_ROW_PTR if row_ptr decreases or leaves
// [row_ptr[0], row_ptr[0] + nnz]; the plan then reads the batch as empty.
hipError_t launch_check_rows(const int32_t *row_ptr, int64_t N, int64_t nnz, uint32_t *flags, hipStream_t st);
// values, vals, xsq: real-valued rows only (else null). row_ptr, col_idx, values: the caller's batch.
// ob non-null: the batch was regrouped: position p's row has plan offsets ob->pos[2p] ... and its
// ids start at ob->pos[2p + 1] in the caller's col_idx.
hipError_t launch_plan(int ta, const int32_t *row_ptr, const int32_t *col_idx, const float *values, int64_t N,
                       int64_t nnz, int64_t V, const OrderBuffers *ob, uint2 *plan, int2 *tiles, float *vals,
                       double *xsq, uint32_t *flags, hipStream_t st);
// f16: W holds binary16 values; top2: fill keys2/dots2 too; vals: real-valued rows (tile 8 only).
hipError_t launch_sweep(int ta, bool f16, bool top2, const void *W, const double *norms, int64_t M, int64_t N,
                        int64_t V, int64_t nnz, const uint2 *plan, const int2 *tiles, const float *vals,
                        const SweepOut &o, hipStream_t st);
// The sweep of rows without a plan (o.direct).
hipError_t launch_rows(bool f16, bool top2, const void *W, const double *norms, int64_t M, int64_t N, int64_t V,
                       int64_t nnz, const SweepOut &o, hipStream_t st);
// bmu2/dist2 non-null: the two best units. xsq: real-valued rows (else ||x||^2 = nnz of the row).
// ob non-null: the batch was regrouped (the row lengths come from ob->pos, not row_ptr); results
// are staged by position and then moved to their samples.
hipError_t launch_finalize(int ta, const double *norms, int64_t M, const int32_t *row_ptr, int64_t N, int64_t nnz,
                           const OrderBuffers *ob, const double *xsq, const SweepOut &o, int32_t *bmu, double *dist,
                           int32_t *bmu2, double *dist2, hipStream_t st);
hipError_t launch_order(const int32_t *row_ptr, const int32_t *col_idx, int64_t N, int64_t nnz, int64_t V,
                        const OrderBuffers &ob, uint32_t *flags, hipStream_t st);

// ----------------------------------------------------------------- update

// Workspace of the batch update (som_update.hip): the den field (counts, occupied units
// along the rows, and three float buffers, M each), the sort of heavy units' samples
// (start[M + 2], cursor[M], slot[M], hunit[M], order[N]) and three fields of chunk * M
// words, one after the other: the counts of a chunk of features and two float buffers where
// the blur runs through memory (cnt, a, b), the counts of three chunks, from cnt on through a
// and b, where it runs in LDS.
struct UpdateBuffers {
    uint32_t *flags;  // SOM_FLAG_ROW_PTR: the batch's row pointers are invalid, nothing is updated
    int32_t *den_cnt;
    int32_t *sup_row;      // occupied units in reach along the row
    float *den_a, *den_b;  // scratch of the den blur
    float *den_blur;       // the blurred den
    int32_t *start, *cursor, *slot, *hunit, *order;
    int32_t *cnt;
    float *a, *b;
};

struct UpdateLayout {
    size_t flags, den_cnt, sup_row, den_a, den_b, den_blur, start, cursor, slot, hunit, order, cnt, a, b, total;
};

inline UpdateLayout update_layout(int64_t M, int64_t N, int64_t chunk)
{
    UpdateLayout L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align256(bytes);
        return at;
    };
    L.flags = take(256);
    L.den_cnt = take((size_t)M * 4);
    L.sup_row = take((size_t)M * 4);
    L.den_a = take((size_t)M * 4);
    L.den_b = take((size_t)M * 4);
    L.den_blur = take((size_t)M * 4);
    L.start = take((size_t)(M + 2) * 4);
    L.cursor = take((size_t)M * 4);
    L.slot = take((size_t)M * 4);
    L.hunit = take((size_t)M * 4);
    L.order = take((size_t)N * 4);
    const size_t field = align256((size_t)chunk * (size_t)M * 4);
    L.cnt = take(3 * field);
    L.a = L.cnt + field;
    L.b = L.a + field;
    L.total = off;
    return L;
}

// f16: W holds binary16 values. radius >= 1; chunk >= 1 features per pass.
hipError_t launch_update(bool f16, void *W, int64_t V, int64_t E, const int32_t *row_ptr, const int32_t *col_idx,
                         int64_t N, int64_t nnz, const int32_t *bmu, int64_t radius, int64_t chunk,
                         const UpdateBuffers &ub, hipStream_t st);

}  // namespace som
