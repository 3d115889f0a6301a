"""Rules of the dispatch that need no GPU: workspace sizes (256 compute units without one)."""
import random

import pytest

import paper_2607_18081_amd as si

SCRATCH = si.api.NOALLOC_SCRATCH_BYTES


def rows_of_64_token_tiles(B, L, d):
    """Bytes of a row-word call with 64-token tiles: token bitmaps, union words, H at 4 bytes a
    (token, slot), and float32 partials of as many K chunks as fill 256 CUs with 256 columns."""
    words, up = (L + 31) // 32, (L + 63) // 64 * 64
    tiles = -(-d // 256) * (-(-B // 64))
    chunks = max(1, min(-(-256 // tiles), words, 64))
    return (B + 1) * words * 4 + B * up * 4 + chunks * B * (-(-d // 16)) * 64 + 4 * 256


@pytest.mark.parametrize("flags", [0, si.FLAG_FAST_H, si.FLAG_UNION, si.FLAG_EXACT_H])
def test_noalloc_takes_what_64_token_tiles_fit(flags):
    """si_selective_ffn_noalloc's 64 MiB hold every batch below 128 tokens whose 64-token tiles
    would fit, whatever tiles are taken."""
    shapes = [(127, 71117, 4264), (105, 99939, 2536), (124, 88838, 2168), (90, 151981, 1128),
              (85, 136154, 2536), (121, 82490, 2056), (101, 123247, 2096)]
    rng = random.Random(flags)
    while len(shapes) < 4000:
        B, d = rng.randint(2, 127), 8 * rng.randint(1, 1024)
        rest = SCRATCH * rng.uniform(0.7, 1.0) - B * d * 4 * rng.choice([1, 4, 8, 16])
        L = min(int(rest / (4.2 * B)), 524288, 2 ** 29 // d - 1)
        if L > 0:
            shapes.append((B, L, d))
    near = 0
    for B, L, d in shapes:
        if rows_of_64_token_tiles(B, L, d) <= SCRATCH:
            need = si.selective_ffn_workspace(B, B * 100, L, d, si.BF16, si.BF16, flags)
            assert need <= SCRATCH, (B, L, d)
            near += need > 0.8 * SCRATCH
    assert near > 100
