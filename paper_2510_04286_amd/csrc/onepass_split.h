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
// Width 96, for units of 32 rows: where one pass does (He <= 192: 1.09 to 1.5); in small batches, up to a unit per CU where there are two passes
// and up to three quarters of that where there are three or four (a block has two units, a position of the split goes to each expert's
// beginning); and where a block has so many that starting the passes one after the other is little beside them -- the two kernels' groups of
// hidden tiles run side by side.  Backward in us, two kernels / this one, 256 CUs, 16 experts unless stated:
//   He  384 (2 passes)   128 units 82.2 / 73.2, 256 units 89.7 / 84.4, 512 units 89.6 / 97.5, 2048 units 157.1 / 157.0, 3000 units 187 / 174
//   He  480 (3)          128 units 88.6 / 85.5, 192 units 89.0 / 90.6, 256 units 88.4 / 96.1, 2600 units 203 / 213, 4096 units 283 / 265
//   He  768 (4)          128 units 110.4 / 102.3, 192 units 108.4 / 109.9, 256 units 107.6 / 117.8, 3000 units 286 / 287, 4096 units 383 / 381
//           4 experts    128 units 106.9 / 94.3, 192 units 107.6 / 101.4, 256 units 108.0 / 108.9
//   He 1536 (8)          1536 units 300 / 453, 8192 units 1208 / 1178
constexpr bool onepass_in_every_batch(int ds, int He) { return ds == 24 || ds == 48 || (ds == 96 && onepass_passes(ds, He) == 1); }
constexpr bool onepass_depends_on_batch(int ds, int He) { return ds == 96 && onepass_passes(ds, He) > 1; }
constexpr bool onepass_chosen(int ds, int He, long long units, long long cus)
{
    const int passes = onepass_passes(ds, He);
    if (!onepass_depends_on_batch(ds, He)) return onepass_in_every_batch(ds, He);
    return passes == 2 ? units <= cus || units >= 10 * cus : (passes <= 4 && 4 * units <= 3 * cus) || units >= 4 * passes * cus;
}

}  // namespace slicemoe
