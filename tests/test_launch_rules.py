"""Launch constants of the library against what they have to cover, from the header's
values and counted out here. Runs on the CPU."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TEXT = open(os.path.join(ROOT, "paper_1310_5045_amd", "csrc", "ppf_internal.hpp")).read()


def const(name):
    v = re.search(r"constexpr \w+ %s = ([^;]+);" % name, TEXT).group(1)
    return eval(re.sub(r"k[A-Z]\w*", lambda m: str(const(m.group(0))), v))


def test_a_helper_wave_for_every_heavy_chunk():
    """With one launch for the segments and the heavy ones' tiles, no weights make more
    chunks of tiles than there are helper waves: the chunks that segments of every size
    have, for the size with the most chunks to a slot."""
    tile, coop, chunk = const("kSlotTile"), const("kCoopTiles"), const("kChunkTiles")
    slots = 64 * const("kHelpPerLane") * const("kSegItems")
    most = 0
    for start in range(4):  # a segment's first tile starts up to 3 slots early
        for size in range(1, 40 * tile):
            tiles = -(-(start + size) // tile)
            if tiles > coop:
                most = max(most, slots // size * -(-tiles // chunk))
    assert most <= const("kHelpWaves")
    assert most > const("kHelpWaves") // 2  # and not far more waves than can have work
