"""GPU parity of the offline recovery profile (block attention mass, recovery curves) and the
quality number it gives for pooled-score selection."""
import numpy as np
import pytest
import torch

import paper_2603_10353_amd as S
from oracle import shplb_oracle as orc
from workloads import bf16_bits_from_f32, make_custom, make_workload

from checks import MASS_ATOL, MASS_RTOL

pytestmark = pytest.mark.gpu


def _profile(wl, rows=None):
    from harness import DevicePass
    print("case", wl.name, "seqlens", np.diff(wl.cu_seqlens).tolist(), "heads", wl.n_q_heads, wl.n_kv_heads,
          "block", wl.block, flush=True)
    run = DevicePass(wl)
    run.mass_step()
    torch.cuda.synchronize()
    m_g = run.mass_host()
    m_o = orc.block_mass(wl.q, wl.k, wl.cu_seqlens, wl.block, rows=rows)
    for s in range(wl.n_seq):
        nb = m_o[s].shape[1]
        for h in range(wl.n_q_heads):
            for i in range(nb):
                if np.isnan(m_o[s][h, i, 0]):
                    continue
                np.testing.assert_allclose(m_g[s][h, i, :i + 1], m_o[s][h, i, :i + 1], rtol=MASS_RTOL, atol=MASS_ATOL)
                assert np.isnan(m_g[s][h, i, i + 1:]).all(), "entries above the diagonal must stay unwritten"
        tri = np.tril_indices(nb)
        rows_sum = np.where(np.tri(nb, dtype=bool), m_g[s], 0.0).sum(axis=2)
        np.testing.assert_allclose(rows_sum, 1.0, rtol=0, atol=2e-5)             # holds at any size
    return run, m_g, m_o


@pytest.mark.parametrize("block", [64, 128])
def test_block_mass_ragged_varlen_gqa(block):
    wl = make_custom([5 * block + 37, 1, block - 3, 2 * block, 3 * block + 1], 8, 2, block,
                     [2] * 8, seed=61, name="profile_b%d" % block)
    run, m_g, m_o = _profile(wl)
    c_o = orc.recovery_curves(m_o, wl.cu_seqlens, block)
    c_g = S.shplb_recovery_curves(run.p, run.mass_flat_host())
    np.testing.assert_allclose(c_g, c_o, rtol=2e-4, atol=1e-6)
    assert np.all(np.diff(c_g, axis=1) >= -1e-12) and np.allclose(c_g[:, -1], 1.0, atol=2e-5)


def test_block_mass_is_deterministic():
    from harness import DevicePass
    wl = make_workload(1, seqlens=[3000])
    run = DevicePass(wl)
    run.mass_step()
    torch.cuda.synchronize()
    a = run.mass_flat_host().copy()
    run.mass_step()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(a, run.mass_flat_host())


def test_profile_feeds_budget_shifting_and_rates_the_selection():
    # The whole offline-to-online chain on a scaled-down benchmark layer: profile -> recovery curves ->
    # max-min shifted budgets -> pooled-score selection -> how much attention weight that selection keeps,
    # against the best any selection of the same size could keep (the curve itself).
    from harness import DevicePass
    wl = make_workload(1, seqlens=[128 * 40])
    run, m_g, m_o = _profile(wl)
    curves = S.shplb_recovery_curves(run.p, run.mass_flat_host())
    nb, hq = 40, wl.n_q_heads
    budgets, moves = S.shplb_shift_budgets(curves, total=6 * hq, lower=2)
    bo, mo = orc.shift_budgets(curves, 6 * hq, 2)
    np.testing.assert_array_equal(budgets, bo)
    assert moves == mo and moves > 0
    equal_min = curves[:, 6].min()
    shifted_min = min(curves[h, budgets[h]] for h in range(hq))
    assert shifted_min >= equal_min                       # what the shifting is for
    wl.budgets = budgets.astype(np.int32)
    run2 = DevicePass(wl).run_all()
    kept = orc.selection_recovery(m_o, wl.cu_seqlens, wl.block, run2.sel_ptr_host, run2.sel_idx_host())
    best = np.array([curves[h, budgets[h]] for h in range(hq)])
    print("  budgets %s\n  kept by pooled-score selection %s\n  best possible %s" %
          (budgets.tolist(), np.round(kept, 3).tolist(), np.round(best, 3).tolist()), flush=True)
    assert np.all(kept <= best + 1e-4)
    # The quality number of the pooled-score estimator (the part of the oracle no paper figure pins):
    # on this synthetic layer it keeps 0.71 of the attention weight on average where the ideal choice
    # of the same size keeps 0.81; single heads fall as low as 0.55 of their ideal.
    assert kept.mean() >= 0.8 * best.mean() and np.all(kept >= 0.4 * best)


def test_block_mass_32k_layer_sampled_rows():
    # The 32K layer at full size: the profile of 24 seeded rows plus the last row of four heads (256 key
    # blocks each) against the oracle; every row of the whole profile must sum to one.
    wl = make_workload(1)
    nb, hq = wl.n_blocks[0], wl.n_q_heads
    rng = np.random.default_rng(11)
    rows = set(rng.choice(nb * hq, size=24, replace=False).tolist())
    rows |= {h * nb + nb - 1 for h in (0, 9, 18, 31)}
    _profile(wl, rows=sorted(rows))


@pytest.mark.parametrize("block,n_blocks,tail", [(64, 92, 64), (64, 93, 1), (64, 220, 64), (64, 221, 63), (64, 315, 5),
                                                 (128, 94, 127), (128, 221, 9)])
def test_block_mass_where_the_kept_sums_end(block, n_blocks, tail):
    # rows around the lengths up to which a query's block sums stay in LDS, in registers, and beyond
    T = (n_blocks - 1) * block + tail
    wl = make_custom([T], 2, 1, block, [2, 2], seed=n_blocks, name="mass_%d_blocks" % n_blocks)
    nb = wl.n_blocks[0]
    assert nb == n_blocks
    rows = sorted({h * nb + i for h in range(2) for i in (0, 1, 91, 92, 93, nb - 2, nb - 1) if i < nb})
    _profile(wl, rows=rows)


@pytest.mark.parametrize("block", [64, 128])
def test_block_mass_scores_far_above_those_of_the_first_keys(block):
    # exponents leave the range around the first tile's reference, in several steps, at odd and even blocks:
    # what is kept by then (in LDS and in registers) has to follow.  Scores reach some 100 nats; their fp32
    # rounding (2^-24 of sums of 128 products of that size) stays well inside MASS_RTOL.
    nb = 130
    T = nb * block - 3
    rng = np.random.default_rng(block)
    wl = make_custom([T], 2, 1, block, [2, 2], seed=5, name="mass_rising_%d" % block)
    k = rng.standard_normal((T, 1, 128)).astype(np.float32)
    k *= np.where(np.arange(T) < 64, 0.05, 1.0).astype(np.float32)[:, None, None]
    for b, f in ((37, 3.0), (100, 4.5), (127, 6.0)):
        k[b * block:(b + 1) * block] *= f
    wl.q = bf16_bits_from_f32(3 * rng.standard_normal((T, 2, 128)).astype(np.float32))
    wl.k = bf16_bits_from_f32(k)
    rows = sorted({h * nb + i for h in range(2) for i in (0, 36, 37, 38, 99, 100, 101, 127, 128, 129)})
    _profile(wl, rows=rows)


@pytest.mark.parametrize("block", [64, 128])
def test_block_mass_where_the_first_keys_weigh_nothing(block):
    # scores of -inf for all of the first tile and more: the reference exponent has to come from later keys.
    # (Query blocks of the first 70 tokens see no key with a weight: no numbers, in the oracle either.)
    from harness import DevicePass
    T = 5 * block + 9
    wl = make_custom([T], 2, 1, block, [2, 2], seed=8, name="mass_first_keys_%d" % block)
    rng = np.random.default_rng(8)
    q, k = rng.standard_normal((T, 2, 128)).astype(np.float32), rng.standard_normal((T, 1, 128)).astype(np.float32)
    q[:, :, 9] = 0.5 + np.abs(q[:, :, 9])
    k[:70, 0, 9] = -np.inf
    wl.q, wl.k = bf16_bits_from_f32(q), bf16_bits_from_f32(k)
    run = DevicePass(wl)
    run.mass_step()
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore"):
        want = orc.block_mass(wl.q, wl.k, wl.cu_seqlens, wl.block)[0]
    got, number = run.mass_host()[0], ~np.isnan(want)
    assert number[:, 2:].any(axis=2).all()
    np.testing.assert_allclose(got[number], want[number], rtol=MASS_RTOL, atol=MASS_ATOL)


@pytest.mark.parametrize("block,n_blocks,tail", [(64, 156, 64), (64, 158, 7), (128, 157, 128), (128, 156, 31)])
def test_block_mass_where_sums_move_to_registers(block, n_blocks, tail):
    # rows that keep all sums in LDS, that move 64 of them to registers once, and twice
    wl = make_custom([(n_blocks - 1) * block + tail], 2, 1, block, [2, 2], seed=700 + n_blocks, name="mass_banks_%d" % n_blocks)
    nb = wl.n_blocks[0]
    rows = sorted({h * nb + i for h in range(2) for i in (62, 63, 64, 91, 92, 127, 128, 154, 155, 156, nb - 2, nb - 1) if i < nb})
    _profile(wl, rows=rows)


# Key blocks 0 .. 219 of a long row are kept (64 each in two banks of registers, 92 in LDS), those behind them swept again.
@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("raises_at, wave", [(50, 0), (100, 1), (130, 2), (219, 0), (225, 0), (250, 3), (310, 1)])
def test_block_mass_reference_raised_in_long_rows(block, raises_at, wave):
    # Only the queries of one of the four waves of a workgroup see the raise: a token 46 nats above the first tile's
    # scores (2^66), where tokens of 43 nats (2^62) among the kept sums of every kind, and behind them, do not raise the
    # reference and have some 4% of the weight each.  The other waves' queries give all of these no weight, and their
    # sums may not follow.  Scores of up to 46 nats: fp32 rounding of 2^-24 of that, well inside MASS_RTOL.
    nb = 320
    T = nb * block - 3
    rng = np.random.default_rng(block + raises_at)
    wl = make_custom([T], 2, 1, block, [2, 2], seed=9, name="mass_raised_b%d_at%d_wave%d" % (block, raises_at, wave))
    q, k = rng.standard_normal((T, 2, 128)).astype(np.float32), rng.standard_normal((T, 1, 128)).astype(np.float32)
    q[:, :, 9] = np.where(np.arange(T) // 32 % 4 == wave, 4.0, -4.0)[:, None]
    k[:64] *= 0.05
    k[:, :, 9] = 0.0
    for b, height in [(x, 121.5) for x in (37, 101, 129, 200, 240)] + [(raises_at, 130.0)]:
        k[b * block + 7] = 0.0
        k[b * block + 7, :, 9] = height
    wl.q, wl.k = bf16_bits_from_f32(q), bf16_bits_from_f32(k)
    rows = sorted({h * nb + i for h in range(2) for i in (raises_at - 1, raises_at, raises_at + 1, 221, 230, nb - 2, nb - 1)})
    _profile(wl, rows=rows)


@pytest.mark.parametrize("head", [0, 1])
def test_block_mass_infinite_score_leaves_other_queries_alone(head):
    # One infinite key at block 240: the queries of every other block of one head, which share a workgroup with those of the
    # block behind them, have a score of +inf there and no numbers; the others' score is -inf.
    from harness import DevicePass
    block, nb = 64, 256
    T = nb * block
    wl = make_custom([T], 2, 1, block, [2, 2], seed=10, name="mass_infinite_key_%d" % head)
    rng = np.random.default_rng(10 + head)
    q, k = rng.standard_normal((T, 2, 128)).astype(np.float32), rng.standard_normal((T, 1, 128)).astype(np.float32)
    q[:, :, 9] = -1.0
    q[np.arange(T) // block % 2 == 0, head, 9] = 1.0
    k[:, 0, 9] = 0.0
    k[240 * block, 0, 9] = np.inf
    wl.q, wl.k = bf16_bits_from_f32(q), bf16_bits_from_f32(k)
    print("case", wl.name, flush=True)
    run = DevicePass(wl)
    run.mass_step()
    torch.cuda.synchronize()
    got = run.mass_host()[0]
    tri = np.tri(nb, dtype=bool)
    sums = np.where(tri, got, 0.0).sum(axis=2)
    lost = np.zeros((2, nb), bool)
    lost[head, 240::2] = True
    np.testing.assert_allclose(sums[~lost], 1.0, rtol=0, atol=2e-5)
    rows = sorted({h * nb + i for h in range(2) for i in (240, 241, 243, 249, nb - 2, nb - 1) if not lost[h, i]})
    want = orc.block_mass(wl.q, wl.k, wl.cu_seqlens, block, rows=rows)[0]
    number = ~np.isnan(want)
    np.testing.assert_allclose(got[number], want[number], rtol=MASS_RTOL, atol=MASS_ATOL)
