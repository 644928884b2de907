"""The map of output tiles to wavefronts of the fp32 expert kernel (csrc/output_role.h), compiled for the host: for every
number of tiles within the library's limits every part of every tile has exactly one wavefront."""
import os
import subprocess

SRC = r"""
#include <cstdio>
#include "output_role.h"
int main()
{
    const int waves = 8;
    for (int tiles = 1; tiles <= 64; ++tiles)
        for (int wave = 0; wave < waves; ++wave) {
            const slicemoe::OutputRole r = slicemoe::output_role(tiles, waves, wave);
            for (int o = 0; o < 8; ++o)
                if (r.has_tile(o)) std::printf("%d %d %d %d\n", tiles, r.parts, r.tile + waves * o, r.part);
        }
}
"""


def test_every_part_of_every_output_tile_has_one_wavefront(tmp_path):
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_04286_amd", "csrc")
    (tmp_path / "roles.cpp").write_text(SRC)
    exe = str(tmp_path / "roles")
    subprocess.check_call(["g++", "-std=c++17", "-I", csrc, str(tmp_path / "roles.cpp"), "-o", exe])
    rows = [tuple(map(int, l.split())) for l in subprocess.check_output([exe], text=True).splitlines()]
    for tiles in range(1, 65):
        mine = [r for r in rows if r[0] == tiles]
        (parts,) = {r[1] for r in mine}
        want = [(t, p) for t in range(tiles) for p in range(parts)]
        assert sorted((t, p) for _, _, t, p in mine) == want, f"{tiles} tiles"
