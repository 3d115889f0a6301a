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


@pytest.mark.parametrize("flags", [0, si.FLAG_EXACT_H])
def test_few_ids_take_the_tiles_of_their_number(flags):
    """From 128 tokens, ids for less than a third of the loaded slots: GEMM1's tile is that of a
    layer with as many slots as there are ids; the K chunks and the workspace never exceed those of
    a full list."""
    rng = random.Random(flags + 1)
    fewer = 0
    for _ in range(2000):
        B, d, L = rng.randint(128, 3000), 8 * rng.randint(8, 700), rng.randint(1000, 40000)
        nnz = rng.randint(0, (L - 1) // 3)
        few = si.selective_ffn_plan(B, nnz, L, d, flags=flags)
        full = si.selective_ffn_plan(B, B * L, L, d, flags=flags)
        if few[0] != 2:                                   # past the slot list's sizes
            continue
        assert few[1:3] == si.selective_ffn_plan(B, B * L, max(nnz, 1), d, flags=flags)[1:3]
        assert few[5] <= full[5]
        assert (si.selective_ffn_workspace(B, nnz, L, d, flags=flags) ==
                si.selective_ffn_workspace(B, B * L, L, d, flags=flags))
        fewer += few[1:5] != full[1:5]
        assert si.selective_ffn_plan(B, L // 3 + 1, L, d, flags=flags) == full
    assert fewer > 200


def test_few_slots_take_two_token_tiles():
    """65 to 127 tokens: with few slots one token tile would leave half of 256 CUs without a
    GEMM1 work-group."""
    for L, tokens in ((1, 64), (18, 64), (4096, 64), (4097, 128), (9677, 128)):
        for B in (65, 127):
            plan = si.selective_ffn_plan(B, B * L, L, 5120)
            assert (plan[0], plan[1], plan[3]) == (1, tokens, tokens), (B, L, plan)
    assert si.selective_ffn_plan(64, 64 * 18, 18, 5120)[1] == 64


GEMM1_TILES = {(256, 256), (256, 192), (256, 160), (128, 256), (128, 160)}


def test_value_checks_reach_every_tile():
    """The shapes whose values the GPU tests check take every tile of the pipelined GEMMs on 256
    CUs, so that a changed tile choice cannot leave one unchecked."""
    from tests.test_gpu_ffn import TILED_SHAPES, WORD_SHAPES
    from tests.test_gpu_select import ACT_SHAPES
    plan = lambda B, L, d, flags=0: si.selective_ffn_plan(B, B * L, L, d, flags=flags)
    one = [plan(B, L, d) for B, L, d, step in TILED_SHAPES]
    pair = [plan(B, L, d, si.FLAG_EXACT_H) for B, L, d, step in TILED_SHAPES]
    assert {p[0] for p in one + pair} == {2}
    assert {p[1:3] for p in one} == {p[1:3] for p in pair} == GEMM1_TILES
    assert {p[3:5] for p in one} == {(256, 256), (256, 128), (128, 128)}
    assert {p[3:5] for p in pair} == {(128, 256), (128, 128)}
    word = [plan(B, L, d) for B, L, d in WORD_SHAPES]
    assert {p[0] for p in word} == {1}
    assert {p[1:3] for p in word} == {(t, r) for t in (16, 32, 64, 128) for r in (64, 80, 96, 128)}
    assert {p[3:5] for p in word} == {(16, 128)} | {(t, c) for t in (32, 64, 128)
                                                    for c in (128, 256)}
    # (a batch in one token tile, and in two)
    assert {(p[1], -(-B // p[1])) for p, (B, _, _) in zip(word, WORD_SHAPES)} >= {(64, 1), (64, 2)}
    assert {si.activations_plan(T, L) for T, L, _ in ACT_SHAPES} == GEMM1_TILES
