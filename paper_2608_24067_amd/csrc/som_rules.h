// som_rules.h -- the host's rules that choose a search's path and launch by its sizes.
#pragma once

#include <cstdint>

namespace som {

// Sizes at which a search may read its rows without a plan (som_rows.hip). That saves two
// launches and the walk over tiles' unions, and reads a codebook row once per sample instead
// of once per tile: it wins while the rows times the units are few. Without / with the plan,
// us, fp32, 12 ids a row: 64 x 64 map 12 / 19 at one row, 14 / 38 at 512, 23 / 41 at 1,024,
// 44 / 44 at 2,048; 256 x 256 29 / 44 at 64, 87 / 101 at 256, 165 / 161 at 512; 512 x 512
// 54 / 58 at 32, 113 / 108 at 64 (fp16 62 / 68); 1024 x 1024 56 / 64 at one row, 123 / 126 at 8,
// 169 / 150 at 16 (fp16 119 / 113); 16 x 16 map 15 / 35 at 2,000, 21 / 36 at 4,096; 32 x 32 26 / 39
// at 3,072, 36 / 37 at 4,096.
inline bool few_rows(int64_t N, int64_t M, int ta)
{
    const int64_t pairs = N * M;
    return (N <= 256 && pairs <= (int64_t)1 << 24) ||
           (ta == 8 && ((N <= 1024 && pairs <= (int64_t)1 << 23) || (N <= 4096 && pairs <= (int64_t)3 << 20)));
}

// Whether it does at nnz ids in all. Longer rows keep to the line above while a launch is
// short of waves, since a plan's walk grows with the row too. Once it is not, the codebook
// rows that samples share are read by each of them, and the ids times the units are the work.
// Without / with the plan, us, by the rows and the ids of each (Zipf rows, V = 30,000):
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
// resemble each other. Whether they do is not known beforehand, so the line lies where the
// kernels cost a search of independent rows a tenth at most: 9 * 2^28 ids times units, at 12
// ids a row 49,000 rows on a 64 x 64 map. Whole searches, us, fp32,
// V = 30,000, regrouped / as given, for independent rows; for eight variants of each row (a tenth
// of the ids changed); for eight copies: 64 x 64 map 335 / 305, 216 / 277, 166 / 273 at 32,000 rows,
// 555 / 556, 376 / 530, 281 / 522 at 64,000; 128 x 128 635 / 606, 412 / 534, 288 / 509 at 16,000;
// 256 x 256 491 / 446, 326 / 369, 183 / 339 at 2,000, 801 / 758, 490 / 600, 297 / 561 at 4,000;
// 22 x 22 592 / 578, 462 / 576, 400 / 578 at 512,000. Longer rows gain as the product says (fp16
// 64 x 64, 30,000 rows of 200 ids 1,984 / 2,502). Maps of up to 256 units, half a strip, read too
// little per row (16 x 16, 2,000,000 rows 1,673 / 1,558, 1,534 / 1,555, 1,432 / 1,561), unless the
// rows are long and many (16 x 16, 80,000 rows of 110 ids 689 / 625, ten copies of each 388 / 616;
// 5 x 5, fp16 712 / 638, 394 / 635; 20,000 rows 380 / 329).
// fp16 sweeps gain less (64 x 64, 64,000 rows 365 / 337, 320 / 334, 276 / 334); the plan and the
// finalize do not know the codebook's type. Nor do they know of a search that ran without a
// plan: its workspace holds the rows in the order given, so wherever one may (an fp16 one, the
// wider line) the phases regroup nothing.
inline bool regroup_pays(int64_t N, int64_t M, int64_t nnz, int ta)
{
    const bool work = M > 256 ? nnz * M >= (int64_t)9 << 28 : ta == 8 && nnz >= 48 * N && nnz >= (int64_t)5 << 20;
    return work && !rows_direct(N, M, nnz, ta, true);
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

}  // namespace som
