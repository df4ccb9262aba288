"""The kernels a call can be sent to (heads shared or not, key blocks of a tile dealt to two sets of waves or not)
against each other, over the forms that each accepts."""
import threading

import pytest
import torch

from paper_2512_07011_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda"


def make(b, n, hq, hkv, d, layout, dtype, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    q, k, v = (torch.randn(b, n, h, d, generator=g, device=DEV).to(dtype) for h in (hq, hkv, hkv))
    if layout == "qkv":                                     # slices of one fused projection
        return torch.cat([q, k, v], dim=2).split([hq, hkv, hkv], dim=2)
    if layout == "bhnd":
        return tuple(t.transpose(1, 2).contiguous().transpose(1, 2) for t in (q, k, v))
    return q, k, v


def call(q, k, v, tau, bm, causal, dump=False, **kw):
    st = binding.alloc_stats(q, bm, 64, counts=True, skip_mask=True, block_max=dump, lse=True)
    st.lse.fill_(7.0)                                       # rows that do not exist keep it
    out = torch.full_like(q.contiguous(), 7.0)
    binding.bsfa_forward(q, k, v, tau, causal=causal, out=out, skip_stats=st, block_m=bm, **kw)
    torch.cuda.synchronize()
    return out, st.lse, st.counts, st.skip_mask


# (b, n, hq, hkv, d, bm, causal, layout): every tile shape with an even, an odd and no group of heads; lengths around
# tile and block edges, shares of the key blocks with no block, one block and an odd number of them
CASES = [
    (1, 1, 4, 2, 128, 128, True, "bnhd"), (1, 64, 4, 2, 128, 128, True, "bnhd"), (1, 65, 4, 2, 64, 128, True, "qkv"),
    (1, 127, 2, 2, 64, 64, True, "bnhd"), (2, 129, 4, 1, 128, 64, True, "bhnd"), (1, 193, 3, 1, 128, 64, True, "qkv"),
    (3, 1000, 8, 2, 128, 128, True, "qkv"), (1, 2047, 6, 2, 64, 64, True, "bnhd"), (2, 777, 4, 1, 64, 32, True, "bnhd"),
    (1, 449, 4, 2, 128, 128, True, "bnhd"), (1, 512, 4, 2, 128, 128, True, "bnhd"), (1, 257, 2, 1, 64, 128, True, "qkv"), (1, 513, 8, 4, 128, 64, True, "bnhd"),
    (1, 255, 3, 1, 128, 64, True, "bhnd"), (1, 193, 2, 2, 64, 64, True, "bnhd"), (1, 1217, 40, 8, 128, 128, True, "bnhd"), (1, 4100, 20, 4, 64, 64, True, "bnhd"),
    (1, 640, 4, 2, 128, 128, False, "bnhd"), (1, 320, 4, 2, 64, 64, False, "bhnd"), (2, 832, 6, 2, 128, 64, False, "bnhd"),
    (1, 960, 8, 2, 128, 32, False, "qkv"), (1, 512, 4, 1, 64, 32, False, "bnhd"), (1, 4096, 2, 1, 128, 128, False, "bnhd"),
]


@pytest.mark.parametrize("case", CASES)
def test_small_calls_agree_with_every_other_form(case):
    """One call by itself against (a) the same with the block maxima dumped (general stages only), bit for bit; (b) one
    head per workgroup, bit for bit; (c) the same element inside a batch large enough for the kernels that do not split
    a tile's key blocks: decisions bit for bit (the scores are the same sums in the same order), out and lse up to the
    rounding of P, of the row sums over rounded P, and of the result: 2^-9 relative each on either side, so 2^-7 of the
    largest |V| for out and 2^-8 for lse, bf16."""
    b, n, hq, hkv, d, bm, causal, layout = case
    q, k, v = make(b, n, hq, hkv, d, layout, torch.bfloat16, n)
    tau = binding.bsfa_calibrate(q, k, [0.5], causal=causal, block_m=bm)[0]
    tau = torch.where(tau.isfinite(), tau, torch.zeros_like(tau)).to(DEV)
    alone = call(q, k, v, tau, bm, causal)
    for other in (call(q, k, v, tau, bm, causal, dump=True), call(q, k, v, tau, bm, causal, single_head_groups=True)):
        for x, y in zip(alone, other):
            assert torch.equal(x, y)
    if n > 256:
        assert alone[2][..., 0].sum() > 0                   # something is skipped
    times = 1 + 150000 // (b * hq * n * (1 if causal else 2))    # (calls split tiles up to 98304 query rows over all heads)
    many = call(*(t.repeat(times, 1, 1, 1) for t in (q, k, v)), tau, bm, causal)
    for lo in (0, (times - 1) * b):
        out, lse, counts, mask = (x[lo:lo + b] for x in many)
        assert torch.equal(mask, alone[3]) and torch.equal(counts, alone[2])
        assert (out.float() - alone[0].float()).abs().max() <= 2.0 ** -7 * v.float().abs().max()
        assert (lse - alone[1]).abs().max() <= 2.0 ** -8


@pytest.mark.parametrize("b, n, hq, hkv, d, bm", [
    (4096, 1, 8, 2, 128, 128), (12, 300, 8, 2, 128, 128), (8, 1000, 8, 2, 64, 128), (9, 512, 8, 2, 128, 64), (9, 700, 8, 2, 64, 64),  # many tiles
    (9, 1536, 4, 2, 128, 128),                                                                                          # unevenly dealt to the XCDs
])
def test_short_prompts_are_not_split(b, n, hq, hkv, d, bm):
    """Calls whose tiles gain nothing from two sets of waves give the bits of one set: those of the same elements in a
    batch beyond the last line."""
    q, k, v = make(b, n, hq, hkv, d, "bnhd", torch.bfloat16, n)
    tau = torch.full((hq,), 2.5, device=DEV)
    times = 2 + 200000 // (b * hq * n)
    for x, y in zip(call(q, k, v, tau, bm, True), call(*(t.repeat(times, 1, 1, 1) for t in (q, k, v)), tau, bm, True)):
        assert torch.equal(x, y[:b]) and torch.equal(x, y[-b:])


@pytest.mark.parametrize("d, bm", [(128, 128), (64, 128), (128, 64), (64, 64)])
def test_split_tiles_with_lengths_and_thresholds_per_tile(d, bm):
    """Batch elements of different lengths (empty, one token, ends of tiles and blocks) and thresholds per query tile
    through the kernels that split a tile's key blocks, against one call per element at its own length."""
    n, hq, hkv = 700, 4, 2
    lengths = [0, 1, 63, 64, 129, 447, 640, 700]
    q, k, v = make(len(lengths), n, hq, hkv, d, "bnhd", torch.float16, d + bm)
    g = torch.Generator().manual_seed(bm)
    tau = (3.0 + torch.rand(hq, -(-n // bm), generator=g)).to(DEV)
    sl = torch.tensor(lengths, dtype=torch.int32, device=DEV)
    out, lse, counts, mask = call(q, k, v, tau, bm, True, seqlens=sl)
    for e, m in enumerate(lengths):
        assert (out[e, m:] == 7.0).all() and (lse[e, m:] == 7.0).all()
        if m == 0:
            assert (counts[e] == 0).all() and (mask[e] == 0).all()
            continue
        one = call(*(t[e:e + 1, :m] for t in (q, k, v)), tau, bm, True)
        assert torch.equal(out[e, :m], one[0][0]) and torch.equal(lse[e, :m], one[1][0]) and torch.equal(counts[e], one[2][0])
        tiles, words = one[3].shape[2:]
        assert torch.equal(mask[e, :, :tiles, :words], one[3][0]) and (mask[e, :, tiles:] == 0).all() and (mask[e, :, :tiles, words:] == 0).all()


SHARED_HEADS = [
    (32, 8, 2304, 128, 64, True, False, torch.bfloat16), (32, 8, 4160, 64, 64, True, False, torch.bfloat16),
    (32, 8, 2624, 64, 32, True, False, torch.bfloat16), (32, 8, 2112, 128, 32, True, False, torch.bfloat16),
    (16, 8, 4150, 128, 32, True, False, torch.float16), (16, 8, 6200, 64, 32, True, False, torch.bfloat16),
    (12, 6, 9800, 128, 128, True, False, torch.bfloat16), (16, 8, 8192, 128, 128, True, False, torch.float16),    # 924 and 1024 tiles
    (4, 2, 24640, 128, 128, True, False, torch.bfloat16),        # V from the workspace
    (32, 8, 4096, 128, 128, False, False, torch.bfloat16), (8, 4, 5120, 128, 128, False, False, torch.float16),   # V in place
    (4, 2, 65700, 128, 128, True, True, torch.bfloat16), (6, 3, 65610, 128, 128, True, True, torch.float16),      # fp8 scores
]


@pytest.mark.parametrize("hq, hkv, n, d, bm, causal, fp8, dtype", SHARED_HEADS)
def test_shared_heads_are_bit_identical(hq, hkv, n, d, bm, causal, fp8, dtype):
    """Two and four heads to a workgroup against one, fast stages and all, on problems large enough to be sent there
    (test_dispatch.py holds them to it)."""
    q, k, v = make(1, n, hq, hkv, d, "bnhd", dtype, n)
    kw = dict(qk_fp8=fp8)
    for tau in (binding.bsfa_calibrate(q, k, [0.6], causal=causal, block_m=bm, **kw)[0].to(DEV), torch.full((hq,), float("-inf"), device=DEV)):
        shared, single = (call(q, k, v, tau, bm, causal, single_head_groups=x, **kw) for x in (False, True))
        for x, y in zip(shared, single):
            assert torch.equal(x, y)
        assert (shared[2][..., 0].sum() > 0) == bool(tau.isfinite().all())


@pytest.mark.parametrize("b, hq, hkv, n", [(1, 6, 2, 11000), (2, 3, 3, 12300), (1, 1, 1, 98304)])
def test_two_workgroups_to_a_cu_change_nothing(b, hq, hkv, n):
    """Calls of head_dim 64 that keep the third workgroup off a CU against the same element in a batch that does not, bit
    for bit."""
    q, k, v = make(b, n, hq, hkv, 64, "bnhd", torch.bfloat16, n)
    tau = binding.bsfa_calibrate(q, k, [0.5])[0].to(DEV)
    few, many = call(q, k, v, tau, 128, True), call(*(t.repeat(2, 1, 1, 1) for t in (q, k, v)), tau, 128, True)
    for x, y in zip(few, many):
        assert torch.equal(x, y[:b]) and torch.equal(x, y[b:])


TURNED = [
    (1, 2100, 32, 8, 128, 128), (1, 2500, 28, 4, 128, 128), (1, 900, 40, 8, 128, 128), (11, 1000, 3, 3, 128, 128), (1, 4160, 28, 4, 128, 64), (4, 1000, 16, 8, 128, 32),
    (33, 700, 3, 3, 64, 64), (1, 3000, 28, 4, 64, 64), (2, 6000, 12, 4, 64, 64), (16, 130, 16, 8, 64, 64), (1, 1100, 64, 8, 64, 128), (1, 11000, 6, 2, 64, 128), (13, 420, 12, 4, 64, 32),
]


@pytest.mark.parametrize("b, n, hq, hkv, d, bm", TURNED)
def test_turned_places_change_nothing(b, n, hq, hkv, d, bm):
    """Calls whose workgroups fill the chip once or twice, with KV heads that fill the XCDs or do not, against the same call
    with lengths, whose work items are counted off in another way and never turned, bit for bit (test_dispatch.py holds them to
    it)."""
    q, k, v = make(b, n, hq, hkv, d, "bnhd", torch.bfloat16, n)
    tau = torch.full((hq,), 2.0, device=DEV)
    plain, counted = call(q, k, v, tau, bm, True), call(q, k, v, tau, bm, True, seqlens=torch.full((b,), n, dtype=torch.int32, device=DEV))
    for x, y in zip(plain, counted):
        assert torch.equal(x, y)


# tiles of 64 and 32 rows: two and four of them to a workgroup (a last one that lacks some, tiles that end in different
# blocks, with and without the mask), two and four shares of their key blocks
SMALL_TILES = [
    (1, 1090, 4, 2, 64, 32, True, "bnhd"), (1, 1217, 3, 1, 64, 64, True, "qkv"), (1, 1024, 2, 1, 64, 64, False, "bnhd"), (1, 1152, 3, 1, 64, 32, False, "bhnd"),
    (1, 1600, 3, 1, 128, 64, True, "bnhd"), (1, 2079, 5, 1, 128, 32, True, "bnhd"), (1, 1345, 28, 4, 128, 32, True, "qkv"), (1, 1473, 28, 4, 128, 64, True, "bnhd"),
    (1, 225, 3, 1, 128, 32, True, "bnhd"), (1, 193, 1, 1, 64, 32, True, "bnhd"), (1, 161, 5, 1, 64, 32, True, "bhnd"), (3, 129, 3, 3, 128, 64, True, "bnhd"),
    (2, 320, 3, 1, 128, 64, False, "bnhd"), (1, 576, 5, 5, 128, 32, False, "qkv"), (1, 1600, 12, 4, 64, 64, True, "bnhd"), (1, 1792, 28, 4, 64, 32, True, "bnhd"),
]


# tiles alone in a workgroup, in twos and in fours, and heads alone where a sequence is a single tile of 32 rows: the kernels
# of few or short sequences
FEW_TILES = [
    (12, 300, 6, 2, 128, 64, True, "qkv"), (30, 250, 3, 3, 128, 64, True, "bnhd"), (24, 250, 6, 2, 64, 64, True, "qkv"), (48, 192, 3, 1, 128, 64, False, "bnhd"),
    (2, 31, 4, 2, 128, 32, True, "bnhd"), (2, 32, 4, 2, 64, 32, True, "qkv"), (3, 1, 6, 3, 64, 32, True, "bnhd"), (2, 30, 8, 2, 64, 32, True, "bnhd"),
    (1, 100, 3, 1, 64, 32, True, "bnhd"), (2, 97, 5, 1, 64, 32, True, "qkv"), (3, 128, 3, 3, 64, 32, False, "bnhd"),
]


@pytest.mark.parametrize("case", FEW_TILES)
def test_few_tiles_agree_with_every_other_form(case):
    test_small_calls_agree_with_every_other_form(case)


@pytest.mark.parametrize("case", SMALL_TILES)
def test_small_tiles_agree_with_every_other_form(case):
    test_small_calls_agree_with_every_other_form(case)


IN_PLACE_ORDER = [
    (4, 2, 128, 128, 500, [500, 500, 0, 131, 64]), (3, 1, 128, 32, 450, [450, 33, 32]), (8, 8, 64, 32, 200, [0, 200, 64] * 8),
    (5, 5, 64, 128, 300, [300, 1, 256, 300, 255]), (2, 1, 128, 128, 260, [0, 0]),
]
COUNTED_OFF = [
    (6, 3, 64, 64, 700, [700, 0, 1, 63, 699, 128]), (16, 8, 128, 64, 640, [640, 17, 320, 321]),
    (24, 2, 128, 128, 500, [500, 500, 0, 131, 64]), (40, 1, 64, 128, 300, [300, 1, 256, 300, 255]), (64, 1, 128, 128, 260, [0, 0]), (32, 1, 128, 32, 450, [450, 33, 32]),
    (8, 4, 128, 128, 1300, [1300, 1299, 640, 5]), (12, 4, 64, 32, 500, [500, 33, 32, 257]), (8, 8, 64, 64, 330, [0, 330, 64, 65] * 4),
]


@pytest.mark.parametrize("hq, hkv, d, bm, n, lengths", IN_PLACE_ORDER + COUNTED_OFF)
def test_every_tile_of_elements_with_lengths_is_counted_off(hq, hkv, d, bm, n, lengths):
    """Work items of batches whose elements end early, counted off or in the order of their places, with pairs of element and KV
    head that fill the XCDs or do not, one and many to an XCD (more than 16 too): outputs, masks and counts of every element are those of a call of its own (out and lse up
    to rounding, where only one of the two splits its tiles; bounds as above), what lies beyond its end is untouched or empty."""
    q, k, v = make(len(lengths), n, hq, hkv, d, "bnhd", torch.bfloat16, n)
    tau = torch.full((hq,), 2.0, device=DEV)
    out, lse, counts, mask = call(q, k, v, tau, bm, True, seqlens=torch.tensor(lengths, dtype=torch.int32, device=DEV))
    for e, m in enumerate(lengths):
        assert (out[e, m:] == 7.0).all() and (lse[e, m:] == 7.0).all()
        if m == 0:
            assert (counts[e] == 0).all() and (mask[e] == 0).all()
            continue
        one = call(*(t[e:e + 1, :m] for t in (q, k, v)), tau, bm, True)
        tiles, words = one[3].shape[2:]
        assert torch.equal(counts[e], one[2][0]) and torch.equal(mask[e, :, :tiles, :words], one[3][0])
        assert (mask[e, :, tiles:] == 0).all() and (mask[e, :, :tiles, words:] == 0).all()
        assert (out[e, :m].float() - one[0][0].float()).abs().max() <= 2.0 ** -7 * v.float().abs().max()
        assert (lse[e, :m] - one[1][0]).abs().max() <= 2.0 ** -8


@pytest.mark.parametrize("hq, hkv, n", [(4, 2, 12700), (3, 1, 12416), (4, 2, 24641)])
def test_rewritten_v_with_lengths(hq, hkv, n):
    """Rewritten V with batch elements that end early, at block edges or are empty, and a workspace full of NaN: V in
    place gives the same bits, rows behind an end stay untouched, empty elements count nothing (the pass over V clears
    the counts)."""
    lengths = [0, 1, 64, 6321, n - 1, n]
    q, k, v = make(len(lengths), n, hq, hkv, 128, "bnhd", torch.bfloat16, n)
    tau = torch.full((hq,), 3.3, device=DEV)
    sl = torch.tensor(lengths, dtype=torch.int32, device=DEV)
    ws = torch.full((binding.forward_workspace_bytes(q, k),), 0xFF, dtype=torch.uint8, device=DEV)
    rewritten, in_place = (call(q, k, v, tau, 128, True, seqlens=sl, workspace=w) for w in (ws, None))
    for x, y in zip(rewritten, in_place):
        assert torch.equal(x, y)
    assert (ws != 0xFF).any()
    out, lse, counts, mask = rewritten
    assert (counts[0] == 0).all() and (counts[-1, :, 0] > 0).all()
    for e, m in enumerate(lengths):
        assert (out[e, m:] == 7.0).all() and (lse[e, m:] == 7.0).all() and out[e, :m].isfinite().all()


@pytest.mark.parametrize("hq, hkv, n, dtype", [(6, 2, 12500, torch.bfloat16), (3, 1, 24577, torch.float16), (4, 2, 24700, torch.bfloat16)])
def test_rewritten_v_is_bit_identical_to_v_in_place(hq, hkv, n, dtype):
    """Long enough for the pass over V (ragged, so the last tile repeats the last token), single heads and pairs."""
    q, k, v = make(1, n, hq, hkv, 128, "qkv", dtype, n)
    tau = binding.bsfa_calibrate(q, k, [0.5])[0].to(DEV)
    ws = torch.full((binding.forward_workspace_bytes(q, k),), 0xFF, dtype=torch.uint8, device=DEV)      # NaN everywhere
    for x, y in zip(call(q, k, v, tau, 128, True, workspace=ws), call(q, k, v, tau, 128, True, workspace=None)):
        assert torch.equal(x, y)
    assert (ws != 0xFF).any()


@pytest.mark.parametrize("b, n, n_levels, equal", [
    (1, 64, 3, False), (1, 640, 64, False), (3, 700, 8, True),          # nothing gateable; several rounds; all maxima equal
    (2, 8192, 9, False), (1, 11584, 7, False), (1, 11648, 9, False),     # 32768, 32761 and 33124 maxima a head
])
def test_order_statistics_on_both_selections(b, n, n_levels, equal):
    """bsfa_calibrate against a sort of the kernel's own block maxima, bit for bit, on dumps that one workgroup per head
    selects from and on those that go through separate passes."""
    q, k, _ = make(b, n, 2, 1, 64, "bnhd", torch.bfloat16, n)
    if equal:
        k = torch.zeros_like(k)
    fr = [l / max(1, n_levels - 1) for l in range(n_levels)]
    got = binding.bsfa_calibrate(q, k, fr, block_m=64)
    st = binding.alloc_stats(q, 64, 64, counts=False, block_max=True)
    binding.bsfa_forward(q, k, k, torch.full((2,), float("-inf"), device=DEV), skip_stats=st, block_m=64)
    for h in range(2):
        x = st.block_max[:, h].reshape(-1)
        x = torch.sort(x[~x.isnan()])[0].cpu()
        for l, f in enumerate(torch.tensor(fr).double().tolist()):
            r = int(f * len(x))
            want = float("-inf") if r == 0 else float("inf") if r >= len(x) else float(x[r])
            assert float(got[l, h]) == want, (h, f)


# (b, n, hq, hkv, d, bm): score kernels with a tile, two and four of them, with and without other heads, to a workgroup
SCORES = [
    (1, 589, 12, 4, 128, 64), (1, 300, 3, 3, 64, 64), (2, 65, 5, 1, 128, 64), (1, 1100, 28, 4, 128, 64), (1, 1700, 28, 4, 64, 64), (1, 193, 4, 2, 128, 64), (1, 200, 4, 2, 64, 64),
    (1, 450, 3, 1, 128, 32), (1, 290, 3, 1, 64, 32), (1, 161, 4, 2, 128, 32), (1, 161, 4, 2, 64, 32), (1, 450, 8, 2, 128, 32), (2, 225, 8, 2, 64, 32), (1, 700, 3, 1, 128, 128),
    (1, 700, 3, 1, 64, 128), (1, 8300, 32, 8, 128, 128),
]


@pytest.mark.parametrize("b, n, hq, hkv, d, bm", SCORES)
def test_every_score_kernel_gives_the_forward_kernels_maxima(b, n, hq, hkv, d, bm):
    """Order statistics of a calibration against a sort of the block maxima that a forward call dumps, bit for bit, without and
    with lengths (of which every element but the first is shorter)."""
    q, k, _ = make(b, n, hq, hkv, d, "bnhd", torch.float16, n)
    fr = [0.0, 0.125, 0.5, 0.75, 1.0]
    for lengths in (None, torch.tensor([n] + [max(1, n // 2 - 3)] * (b - 1), dtype=torch.int32, device=DEV)):
        got = binding.bsfa_calibrate(q, k, fr, block_m=bm, seqlens=lengths)
        st = binding.alloc_stats(q, bm, 64, counts=False, block_max=True)
        binding.bsfa_forward(q, k, k, torch.full((hq,), float("-inf"), device=DEV), skip_stats=st, block_m=bm, seqlens=lengths)
        for h in range(hq):
            x = st.block_max[:, h].reshape(-1)
            x = torch.sort(x[~x.isnan()])[0].cpu()
            for l, f in enumerate(fr):
                r = int(f * len(x))
                want = float("-inf") if r == 0 else float("inf") if r >= len(x) else float(x[r])
                assert float(got[l, h]) == want, (h, f)


def test_running_maximum_over_large_score_ranges():
    """Rows whose maximum grows with every block, only in the first one, and hardly at all, with scores of several
    hundred: finite, and equal to softmax in 64 bits (2e-2, the bound of every parity test; for lse the rounding of P
    and 32-bit scores)."""
    n, d = 1024, 128
    q, k, v = make(1, n, 1, 1, d, "bnhd", torch.bfloat16, 3)
    ramp = torch.linspace(0.2, 30.0, n, device=DEV)[None, :, None, None]
    for scale in (ramp, ramp.flip(1), torch.full_like(ramp, 1e-3)):
        ks = (k.float() * scale).to(torch.bfloat16)
        out, lse, _, _ = call(q, ks, v, torch.full((1,), float("-inf"), device=DEV), 128, True)
        s = (q[0, :, 0].double() @ ks[0, :, 0].double().t() / d ** 0.5).masked_fill(torch.ones(n, n, device=DEV).triu(1).bool(), float("-inf"))
        assert (out[0, :, 0].double() - s.softmax(-1) @ v[0, :, 0].double()).abs().max() <= 2e-2
        assert (lse[0, :, 0].double() - s.logsumexp(-1)).abs().max() <= 2.0 ** -8 + 1e-6 * s[s.isfinite()].abs().max()


@pytest.mark.parametrize("side_by_side", ["streams", "threads"])
def test_calls_that_overlap_do_not_share_scratch_memory(side_by_side):
    """Calls whose V goes through scratch memory of the binding's own, on two streams and from two threads on one stream,
    each side with its own V, against the same calls one after the other, bit for bit."""
    q, k, v = make(1, 16500, 8, 2, 128, "bnhd", torch.bfloat16, 1)
    vs = (v, v.flip(1).contiguous())
    tau = torch.full((8,), 3.0, device=DEV)
    want = [binding.bsfa_forward(q, k, x, tau) for x in vs]
    got = [[torch.empty_like(q) for _ in range(4)] for _ in vs]
    torch.cuda.synchronize()
    if side_by_side == "streams":
        streams = [torch.cuda.Stream() for _ in vs]
        for r in range(4):
            for x, o, s in zip(vs, got, streams):
                binding.bsfa_forward(q, k, x, tau, out=o[r], stream=s)
    else:
        def calls(x, o):
            for r in range(4):
                binding.bsfa_forward(q, k, x, tau, out=o[r])
        side = [threading.Thread(target=calls, args=a) for a in zip(vs, got)]
        for t in side:
            t.start()
        for t in side:
            t.join()
    torch.cuda.synchronize()
    for w, outs in zip(want, got):
        for o in outs:
            assert torch.equal(o, w)


def test_captured_call_keeps_its_scratch_memory():
    """A captured call with scratch memory, replayed between larger eager calls and tensors that take up whatever memory
    those have given back: every replay equals the eager result."""
    q, k, v = make(1, 1024, 4, 2, 128, "bnhd", torch.bfloat16, 2)
    big = make(1, 6000, 4, 2, 128, "bnhd", torch.bfloat16, 3)
    tau = torch.full((4,), 1.0, device=DEV)
    out = torch.empty_like(q)
    want = binding.bsfa_forward(q, k, v, tau, qk_fp8=True)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        binding.bsfa_forward(q, k, v, tau, out=out, qk_fp8=True)
    for r in range(3):
        want_big = binding.bsfa_forward(*big, tau, qk_fp8=True)
        others = [torch.full((s,), 0xFF, dtype=torch.uint8, device=DEV) for s in (1 << 20, 3 << 20, 9 << 20)]
        out.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), r
        assert torch.equal(binding.bsfa_forward(*big, tau, qk_fp8=True), want_big)
        assert all((o == 0xFF).all() for o in others)
