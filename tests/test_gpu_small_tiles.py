"""Options that meet adjacent query tiles in one workgroup (64- and 32-row tiles of an odd group of heads): the running-maximum
predicate, thresholds per query tile, lengths and the block maxima, with a last workgroup that lacks some of its tiles."""
import numpy as np
import pytest
import torch

from paper_2512_07011_amd import binding
from tests import parity
from tests.test_gpu_dispatch import call, make

pytestmark = pytest.mark.gpu
DEV = "cuda"

# (hq, hkv, head_dim, block_m), 576 tokens: 9 tiles of 64 rows, 18 of 32; the batch that puts them together in twos and fours
PREDICATE = [(3, 1, 128, 64), (3, 1, 64, 64), (3, 1, 128, 32), (5, 1, 64, 32)]
PREDICATE_TOKENS, PREDICATE_BATCH = 576, 64


@pytest.mark.parametrize("hq, hkv, d, bm", PREDICATE)
def test_running_max_predicate_on_small_tiles(oracle, hq, hkv, d, bm):
    """gate_mode = 1 against its step-by-step oracle form: statistics to 1e-4, decisions exactly (lambda is placed where no
    statistic of the oracle's own trajectory lies within 1e-3 of it), outputs within the usual tolerance; and the same element
    in a batch whose tiles share workgroups, bit for bit."""
    n = PREDICATE_TOKENS
    g = torch.Generator().manual_seed(d + bm)
    u = torch.nn.functional.normalize(torch.randn(d, generator=g), dim=0)
    q = 3.0 * u + 0.5 * torch.randn(1, n, hq, d, generator=g)
    k = torch.randn(1, n, hkv, d, generator=g)
    for blk, amp in ((0, 40.0), (2, 36.0), (5, 36.0), (3, 30.0), (6, 30.0)):     # a high maximum, blocks near it and not
        k[:, blk * 64:(blk + 1) * 64] += amp * u
    v = torch.randn(1, n, hkv, d, generator=g)
    qd, kd, vd = (t.to(torch.bfloat16).to(DEV) for t in (q, k, v))
    qf, kf, vf = (t.float().cpu().numpy() for t in (qd, kd, vd))
    lam = -2.0
    for _ in range(20):
        res = {(h, i): oracle.alg1_tile_running_max(qf, kf, vf, lam, 0, h, i, bm, 64) for h in range(hq) for i in range(n // bm)}
        if min(abs(float(s) - lam) for r in res.values() for s in r[3].values()) > 2e-3:
            break
        lam -= 0.0137
    else:
        pytest.fail("no clear lambda found")
    tau = torch.full((hq,), lam, device=DEV)

    def run(times):
        x = [t.repeat(times, 1, 1, 1) for t in (qd, kd, vd)]
        st = binding.alloc_stats(x[0], bm, 64, counts=True, skip_mask=True, block_max=True, lse=True)
        out = binding.bsfa_forward(*x, tau, skip_stats=st, block_m=bm, gate_mode=1)
        torch.cuda.synchronize()
        return out, st.lse, st.counts, st.skip_mask, st.block_max

    alone, many = run(1), run(PREDICATE_BATCH)
    for x, y in zip(alone, many):
        for e in (0, PREDICATE_BATCH - 1):
            assert torch.equal(x[0].nan_to_num(7.0), y[e].nan_to_num(7.0))
    o, lse, mask = alone[0].float().cpu().numpy()[0], alone[1].cpu().numpy()[0], parity.unpack_mask(alone[3].cpu().numpy(), n // 64)[0]
    bmx, n_skipped = alone[4].cpu().numpy()[0], 0
    for (h, i), (O, L, kept, stats) in res.items():
        skipped = [j for j in range(-(-(i + 1) * bm // 64)) if j not in kept]
        assert list(np.nonzero(mask[h, i])[0]) == skipped, (h, i)
        n_skipped += len(skipped)
        for j, s in stats.items():
            assert abs(bmx[h, i, j] - float(s)) < 1e-4
        assert np.isnan(bmx[h, i, len(stats):]).all()
        err = np.abs(o[i * bm:(i + 1) * bm, h] - O)
        assert err.max() <= parity.MAX_ABS and err.mean() <= parity.MEAN_ABS
        assert np.abs(lse[i * bm:(i + 1) * bm, h] - L).max() < 5e-3
    assert n_skipped > 10 and int(alone[2][0, :, 0].sum()) == n_skipped


LENGTHS = [2700, 2697, 2560, 1345, 1280, 65, 64, 33, 32, 31, 1, 0, 705, 130, 97, 2049]
WITH_LENGTHS = [(3, 1, 128, 64), (3, 1, 64, 64), (3, 1, 128, 32), (3, 1, 64, 32)]      # (hq, hkv, head_dim, block_m)


@pytest.mark.parametrize("hq, hkv, d, bm", WITH_LENGTHS)
def test_thresholds_per_tile_lengths_and_maxima_on_small_tiles(hq, hkv, d, bm):
    """Elements of different lengths with thresholds per query tile (fewer than the longest has tiles) and the block maxima
    against one call per element at its own length: decisions, maxima and counts bit for bit, out and lse up to rounding, as
    that call may split its tiles (bounds as for the forms of a call); tiles and rows beyond an end are empty or untouched."""
    n = LENGTHS[0]
    q, k, v = make(len(LENGTHS), n, hq, hkv, d, "bnhd", torch.bfloat16, d + bm)
    tau = (1.5 + torch.rand(hq, 2000 // bm, generator=torch.Generator().manual_seed(bm))).to(DEV)

    def run(q, k, v, lengths=None):
        st = binding.alloc_stats(q, bm, 64, counts=True, skip_mask=True, block_max=True, lse=True)
        st.lse.fill_(7.0)
        st.block_max.fill_(7.0)
        out = torch.full_like(q.contiguous(), 7.0)
        binding.bsfa_forward(q, k, v, tau, out=out, skip_stats=st, block_m=bm, seqlens=lengths)
        torch.cuda.synchronize()
        return out, st.lse, st.counts, st.skip_mask, st.block_max

    out, lse, counts, mask, bmx = run(q, k, v, torch.tensor(LENGTHS, dtype=torch.int32, device=DEV))
    fast = call(q, k, v, tau, bm, True, seqlens=torch.tensor(LENGTHS, dtype=torch.int32, device=DEV))
    for x, y in zip((out, lse, counts, mask), fast):                              # nobody asks for the maxima: the other stages
        assert torch.equal(x, y)
    assert counts[..., 0].sum() > 0
    for e, m in enumerate(LENGTHS):
        assert (out[e, m:] == 7.0).all() and (lse[e, m:] == 7.0).all()
        tiles, blocks = -(-m // bm), -(-m // 64)
        assert (mask[e, :, tiles:] == 0).all() and bmx[e, :, tiles:].isnan().all() and bmx[e, :, :, blocks:].isnan().all()
        if m == 0:
            assert (counts[e] == 0).all()
            continue
        one = run(*(t[e:e + 1, :m] for t in (q, k, v)))
        words = one[3].shape[3]
        assert torch.equal(counts[e], one[2][0]) and torch.equal(mask[e, :, :tiles, :words], one[3][0]) and (mask[e, :, :, words:] == 0).all()
        assert torch.equal(bmx[e, :, :tiles, :blocks].nan_to_num(9.0), one[4][0].nan_to_num(9.0))
        assert (out[e, :m].float() - one[0][0].float()).abs().max() <= 2.0 ** -7 * v.float().abs().max()
        assert (lse[e, :m] - one[1][0]).abs().max() <= 2.0 ** -8
