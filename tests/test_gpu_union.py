"""The union path at the edges of its dispatch rules, against the definition in float64.

h travels as a hi + lo pair of 16-bit values below 128 tokens and with SI_FLAG_EXACT_H, held to
1e-4 as elsewhere; as one 16-bit value with SI_FLAG_FAST_H and by default from 128 tokens, where
rounding it to 8 (bf16) or 11 (half) significant bits leaves 2^-8 or 2^-11 of each product at
most, and of the sum where one product outweighs the others."""
import pytest
import torch

import paper_2607_18081_amd as si
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

BF16, F16 = torch.bfloat16, torch.float16
ONE_H = {BF16: 2.0 ** -8, F16: 2.0 ** -11}


def problem(B, L, d, dt=BF16, density=0.2, seed=0, pool=None):
    """A layer, activations and active sets (slots of `pool` only, when given; token 3 has none),
    with the float64 result."""
    g = torch.Generator(device="cuda").manual_seed(B + L + d + seed)
    r = lambda s, *sh: torch.empty(sh, device="cuda").normal_(0, s, generator=g).to(dt)
    gu, dn, x = r(d ** -0.5, L, 2, d), r(d ** -0.5, L, d), r(1.0, B, d)
    mask = torch.rand((B, L), device="cuda", generator=g) < density
    if pool is not None:
        inside = torch.zeros(L, dtype=torch.bool, device="cuda")
        inside[pool] = True
        mask &= inside
    mask[3] = False
    off = torch.zeros(B + 1, dtype=torch.int32, device="cuda")
    off[1:] = mask.sum(1).cumsum(0)
    idx = torch.arange(L, device="cuda").expand(B, -1)[mask].to(torch.int32)
    cols = mask.any(0).nonzero().flatten()                # (the union: no other slot adds to y)
    xx = x.double()
    h = torch.nn.functional.silu(xx @ gu[cols, 0].double().t()) * (xx @ gu[cols, 1].double().t())
    want = torch.where(mask[:, cols], h, 0.0) @ dn[cols].double()
    return x, off, idx, gu, dn, want


def call(x, off, idx, gu, dn, flags=0):
    """One call with a workspace full of NaN bits: nothing that it did not write may reach y."""
    et = 2 if x.dtype == F16 else 1
    need = si.selective_ffn_workspace(x.shape[0], idx.numel(), gu.shape[0], x.shape[1], et, et,
                                      flags)
    ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
    return si.selective_ffn(x, off, idx, gu, dn, flags=flags, workspace=ws)


def rel(got, want):
    return ((got - want).norm() / want.norm()).item()


@pytest.mark.parametrize("B,L,d", [
    # K chunks: 64 and as many as there are steps; 16, 8, 4 and 3 (at most 3 partials)
    (5, 6000, 8), (5, 600, 72), (16, 6000, 2048), (16, 3000, 4096), (7, 700, 8192),
    (6, 400, 10248),
    # (token, 16 columns) pairs up to the wave-a-pair form's last and past it
    (64, 6000, 2560), (64, 6000, 2568), (80, 3000, 2048), (81, 3000, 2048),
    # the same from 128 tokens
    (130, 4000, 128), (160, 3000, 1024), (161, 3000, 1024)])
@pytest.mark.parametrize("flags", [0, si.FLAG_EXACT_H])
def test_sums_of_the_k_chunks(B, L, d, flags):
    say(f"partials B={B} L={L} d={d} flags {flags}")
    p = problem(B, L, d)
    got = call(*p[:5], flags=flags)
    assert not got[3].any()
    err = rel(got, p[5])
    say(f"  {err:.2e}")
    assert err <= (ONE_H[BF16] if B >= 128 and not flags else 1e-4)
    assert torch.equal(got, call(*p[:5], flags=flags))


@pytest.mark.parametrize("B,d", [(5, 520), (17, 264), (33, 2568), (70, 2568), (100, 520)])
@pytest.mark.parametrize("dt", [BF16, F16])
def test_fast_h_is_one_value(B, d, dt):
    """SI_FLAG_FAST_H: h is its 16-bit rounding alone. With the pair, its low half (zero, or of
    the other sign) times an infinite down weight would make a NaN."""
    L, s, c = 700, 301, 7
    say(f"FAST_H B={B} d={d} {dt}")
    x, off, idx, gu, dn, _ = problem(B, L, d, dt)
    dn[s, c] = float("inf")
    k = 20                                                # every token has slot s
    idx = torch.cat([torch.randperm(L - 310, device="cuda")[:k - 1].add(310).sort().values if i
                     else torch.tensor([s], device="cuda") for b in range(B) for i in (0, 1)])
    off = torch.arange(0, (B + 1) * k, k, dtype=torch.int32, device="cuda")
    got = call(x, off, idx.to(torch.int32), gu, dn, si.FLAG_FAST_H)
    h = torch.nn.functional.silu(x.double() @ gu[s, 0].double()) * (x.double() @ gu[s, 1].double())
    assert torch.equal(got[:, c], h.sign().float() * float("inf"))
    got[:, c] = 0
    assert got.isfinite().all()


@pytest.mark.parametrize("B,L,d", [
    # the row-word GEMM2's token tiles of 16, 32, 64 and 128, with 128 and 256 columns
    (5, 3000, 520), (16, 900, 4104), (32, 3000, 520), (17, 3000, 2056), (64, 3000, 520),
    (33, 3000, 2568), (127, 5000, 520), (65, 5000, 2312)])
@pytest.mark.parametrize("dt", [BF16, F16])
def test_fast_h_tiles(B, L, d, dt):
    say(f"FAST_H tiles B={B} L={L} d={d} {dt}")
    p = problem(B, L, d, dt)
    got = call(*p[:5], flags=si.FLAG_FAST_H)
    assert not got[3].any()
    err = rel(got, p[5])
    say(f"  {err:.2e}")
    assert err <= ONE_H[dt]
    assert torch.equal(got, call(*p[:5], flags=si.FLAG_FAST_H))


@pytest.mark.parametrize("B,L,d", [
    # up to 4096 slots, with 128 and 256 columns of GEMM2; the least, one word, an odd last tile
    (65, 18, 4104), (100, 32, 520), (127, 1250, 2568), (66, 4096, 136), (127, 4095, 2312)])
@pytest.mark.parametrize("dt", [BF16, F16])
@pytest.mark.parametrize("flags", [0, si.FLAG_FAST_H])
def test_two_tiles_of_64_tokens(B, L, d, dt, flags):
    say(f"two 64-token tiles B={B} L={L} d={d} {dt} flags {flags}")
    p = problem(B, L, d, dt)
    got = call(*p[:5], flags=flags)
    assert not got[3].any()
    err = rel(got, p[5])
    say(f"  {err:.2e}")
    assert err <= (ONE_H[dt] if flags else 1e-4)
    assert torch.equal(got, call(*p[:5], flags=flags))


@pytest.mark.parametrize("B,L,d", [(128, 523800, 64), (130, 524288, 72), (260, 524000, 136)])
@pytest.mark.parametrize("flags", [0, si.FLAG_FAST_H])
def test_row_word_tiles_of_large_batches(B, L, d, flags):
    """More slots than the tiled path takes: the row-word GEMMs at one, two and three tiles of
    128 tokens."""
    say(f"row-word B={B} L={L} d={d} flags {flags}")
    p = problem(B, L, d, density=0.002)
    got = call(*p[:5], flags=flags)
    assert not got[3].any()
    err = rel(got, p[5])
    say(f"  {err:.2e}")
    assert err <= (ONE_H[BF16] if flags else 1e-4)
    assert torch.equal(got, call(*p[:5], flags=flags))


def sparse_pool(L, how):
    g = torch.Generator(device="cuda").manual_seed(L)
    if how == "none":
        return torch.zeros(0, dtype=torch.int64, device="cuda")
    if how == "ends":
        return torch.tensor([0, L - 1], device="cuda")
    if how == "run":
        return torch.arange(L // 3, L // 3 + 100, device="cuda")
    return torch.randperm(L, device="cuda", generator=g)[:60].sort().values


@pytest.mark.parametrize("B,L,d", [
    # token tiles of 16 to 128 and both column tiles; the last two have K chunks of several times
    # the 64 steps whose union words are held at a time
    (5, 7706, 520), (16, 30000, 2056), (32, 9000, 1032), (33, 9000, 2568), (64, 16000, 136),
    (100, 20000, 264), (127, 12000, 2312), (300, 524000, 520), (5, 48000, 11000)])
@pytest.mark.parametrize("how", ["none", "ends", "run", "spread"])
def test_sparse_unions(B, L, d, how):
    """Unions of few slots: tiles and K steps without any are passed over."""
    say(f"sparse union B={B} L={L} d={d} {how}")
    p = problem(B, L, d, density=0.5, pool=sparse_pool(L, how))
    for flags in (0, si.FLAG_FAST_H):
        got = call(*p[:5], flags=flags)
        if how == "none":
            assert not got.any()
            continue
        assert not got[3].any()
        err = rel(got, p[5])
        say(f"  flags {flags}: {err:.2e}")
        assert err <= (ONE_H[BF16] if flags else 1e-4)
        assert torch.equal(got, call(*p[:5], flags=flags))


def test_sparse_union_costs_its_rows():
    """Time follows the union's rows, not the loaded slots: 5 tokens without any active slot take
    under a third of the time of the same call with a fifth of the slots active (measured: a
    sixth; more than a half while every tile and step was run)."""
    B, L, d = 5, 131000, 1024
    full = problem(B, L, d)
    none = problem(B, L, d, pool=sparse_pool(L, "none"))
    time = []
    for p in (full, none):
        ws = torch.empty(si.selective_ffn_workspace(B, p[2].numel(), L, d), dtype=torch.uint8,
                         device="cuda")
        y = torch.empty((B, d), dtype=torch.float32, device="cuda")
        best = float("inf")
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            torch.cuda.synchronize()
            a.record()
            for _ in range(20):
                si.selective_ffn(*p[:5], y=y, workspace=ws)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) / 20)
        time.append(best)
    say(f"full {time[0] * 1e3:.1f} us, none {time[1] * 1e3:.1f} us")
    assert time[1] <= time[0] / 3


@pytest.mark.parametrize("B,L,d,n", [
    # tokens, slots, columns, ids in all: none, one, around a GEMM1 tile, as many as slots
    (128, 5000, 72, 0), (130, 5000, 264, 1), (200, 30000, 520, 63), (300, 9000, 2056, 81),
    (446, 28190, 2048, 1300), (700, 4000, 264, 1333),
    (700, 4000, 264, 4000), (600, 33000, 72, 500)])
@pytest.mark.parametrize("dt,flags", [(BF16, 0), (F16, si.FLAG_EXACT_H)])
def test_few_ids(B, L, d, n, dt, flags):
    """The slot-list path with its tiles chosen for the ids: each is some token's, spread over all
    the slots and the first and last among them."""
    say(f"few ids B={B} L={L} d={d} n={n} {dt} flags {flags}")
    x, _, _, gu, dn, _ = problem(B, L, d, dt, pool=sparse_pool(L, "none"))
    g = torch.Generator(device="cuda").manual_seed(n)
    slot = torch.randperm(L, device="cuda", generator=g)[:n]
    if n > 1:
        slot[:2] = torch.tensor([0, L - 1], device="cuda")
    slot = slot.unique()
    tok = torch.randint(0, B, slot.shape, device="cuda", generator=g).sort().values
    idx = slot[torch.randperm(len(slot), device="cuda", generator=g)]
    off = torch.zeros(B + 1, dtype=torch.int32, device="cuda")
    off[1:] = torch.bincount(tok, minlength=B).cumsum(0)
    got = call(x, off, idx.to(torch.int32), gu, dn, flags=flags)
    xx = x.double()[tok]                                  # a row an id
    h = torch.nn.functional.silu((xx * gu[idx, 0].double()).sum(1)) * \
        (xx * gu[idx, 1].double()).sum(1)
    want = torch.zeros((B, d), dtype=torch.float64, device="cuda")
    want.index_add_(0, tok, h[:, None] * dn[idx].double())
    assert not got[torch.bincount(tok, minlength=B) == 0].any()
    if n:
        err = rel(got, want)
        say(f"  {err:.2e}")
        assert err <= (1e-4 if flags else ONE_H[dt])
