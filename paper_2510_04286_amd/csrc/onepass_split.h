// Where the one-pass expert backward (backward_expert_mfma.hip) runs, and how its hidden tiles are spread over wavefronts and passes.
// Plain C++, so that the choice can be checked on the host.
#pragma once

namespace slicemoe {

constexpr int kOnepassUnit = 32;   // stacked rows a block works on at a time

// Wavefronts per block, sixteen hidden units each: 12 of 168 registers, three per SIMD and one block per CU; at width 24 two blocks of 8, of
// 128 registers, or one of 16 where the hidden units are more than 128: a pass takes 256 of them (He 160 .. 256 in one pass instead
// of two).  Backward in us, 8 wavefronts / 16, 16 experts: He 192, 512 units 61.8 / 55.2, 4096 units 121 / 107; He 256, 128 units
// 48.9 / 47.6, 8192 units 201 / 197; He 768, 512 units 103 / 86, 8192 units 434 / 419; He 1536, 32 units 113 / 96.
constexpr int onepass_waves(int ds, int He) { return ds != 24 ? 12 : He <= 128 ? 8 : 16; }
constexpr int onepass_blocks_per_cu(int ds, int He) { return onepass_waves(ds, He) == 8 ? 2 : 1; }

// Passes over the rows: as many as the hidden tiles of 16 need, the tiles spread evenly, an even number in each pass (the last takes
// what is left).  He is a multiple of 32.
constexpr int onepass_passes(int ds, int He) { return (He / 16 + onepass_waves(ds, He) - 1) / onepass_waves(ds, He); }
constexpr int onepass_pass_tiles(int ds, int He) { return (He / 32 + onepass_passes(ds, He) - 1) / onepass_passes(ds, He) * 2; }

// Widths 24 and 48: always.  Backward of 32 to 8192 units, He 192 .. 3072, 4 and 16 experts, against the two kernels (one below He 288):
// width 48 1.06 to 1.76 times their speed, width 24 0.99 to 1.8.
// Width 96, for units of 32 rows: where one pass does (He <= 192: 1.09 to 1.5); in batches of up to a unit per CU where there are two to four
// passes -- with four only up to three quarters of that (seven eighths below 16 experts) where the row gradients' kernel is at its best: at most 32
// experts (its tiles of 256 rows are mostly full) and hidden tiles that it streams by three and more (rows_chunk, a divisor of their number); and where a block has so many units
// that starting the passes one after the other is little beside them -- the two kernels' groups of hidden tiles run side by side.
// Backward in us, two kernels / this one, 256 CUs, 16 experts unless stated:
//   He  384 (2 passes)   128 units 82.2 / 73.2, 256 units 89.7 / 84.4, 512 units 89.6 / 97.5, 2048 units 157.1 / 157.0, 3000 units 187 / 174
//   He  416 (3)          256 units 110.1 / 90.9; 4 experts 108.9 / 85.8, 64 143.5 / 128.4
//   He  480, 576         192 units 89.0 / 90.6 and 94.5 / 93.1, 256 units 88.4 / 96.1 and 96.7 / 100.8; He 576, 4 experts 94.4 / 94.6, 48 139.2 / 128.9;
//                        2600 units 203 / 213, 4096 units 283 / 265
//   He  608 (4; its 19 hidden tiles are streamed one by one) 256 units 134.1 / 107.9; 640 100.2 / 110.5, 704 122.1 / 113.9, 736 150.6 / 116.3
//   He  672, 768         128 units 102.6 / 98.2 and 110.4 / 102.3, 192 units 101.4 / 103.4 and 108.1 / 107.3, 256 units 101.8 / 112.2 and 107.3 / 117.5;
//                        4 experts 192 units 98.9 / 94.4 and 107.3 / 98.1, 224 units 99.6 / 100.5 and 107.6 / 106.0, 256 units 98.7 / 103.5 and 107.2 / 109.2;
//                        48 experts, 256 units 149.2 / 142.4 and 153.0 / 149.6; 3000 units 286 / 287, 4096 units 383 / 381
//   He 1536 (8)          1536 units 300 / 453, 8192 units 1208 / 1178
constexpr int rows_chunk(int He)   // hidden tiles that the row gradients' kernel streams at a time at width 96: 18 KB each in 140 KB
{
    for (int c = 7; c > 1; --c)
        if (He / 32 % c == 0) return c;
    return 1;
}
constexpr bool onepass_in_every_batch(int ds, int He) { return ds == 24 || ds == 48 || (ds == 96 && onepass_passes(ds, He) == 1); }
constexpr bool onepass_depends_on_batch(int ds, int He) { return ds == 96 && onepass_passes(ds, He) > 1; }
constexpr bool onepass_chosen(int ds, int He, int E, long long units, long long cus)
{
    if (!onepass_depends_on_batch(ds, He)) return onepass_in_every_batch(ds, He);
    const int passes = onepass_passes(ds, He);
    const bool early = passes == 4 && E <= 32 && rows_chunk(He) >= 3;
    return (passes <= 4 && units <= (early ? (E < 16 ? 7 * cus / 8 : 3 * cus / 4) : cus)) || units >= cus * (passes <= 2 ? 10 : 4 * passes);
}

}  // namespace slicemoe
