// Which wavefront of a block multiplies and stores which 32-wide output tiles of the fp32 expert kernel.  Plain C++, so that
// the map can be checked on the host: every (tile, part) has exactly one wavefront.
#pragma once

namespace slicemoe {

// With as many output tiles as wavefronts or more a wavefront takes tiles tile, tile + waves, ... whole (parts = 1).  With fewer,
// the hidden units of a tile are split into `parts` parts, one wavefront each; the wavefronts left over have no tile.
struct OutputRole {
    int tiles, waves;
    int parts;   // per tile
    int part;    // of this wavefront; parts or more: it has no tile
    int tile;    // its first tile
    constexpr bool has_tile(int o) const { return part < parts && tile + waves * o < tiles; }   // its o-th tile
};

constexpr OutputRole output_role(int tiles, int waves, int wave)
{
    return tiles >= waves ? OutputRole{tiles, waves, 1, 0, wave} : OutputRole{tiles, waves, waves / tiles, wave / tiles, wave % tiles};
}

}  // namespace slicemoe
