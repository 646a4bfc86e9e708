"""GPU parity of the token-granular recovery ratio (Section 2.4: the sum of a query's k largest
attention weights) against the oracle, through the C ABI."""
import time

import numpy as np
import pytest
import torch

import paper_2603_10353_amd as S
from oracle import shplb_oracle as orc
from workloads import bf16_bits_from_f32, make_custom, make_workload

from checks import TOKEN_RECOVERY_ATOL, TOKEN_RECOVERY_RTOL

pytestmark = pytest.mark.gpu


def _run(wl, budgets, softmax_scale=0.0):
    from harness import DevicePass
    print("case", wl.name, "seqlens", np.diff(wl.cu_seqlens).tolist(), "heads", wl.n_q_heads, wl.n_kv_heads,
          "block", wl.block, "budgets", list(budgets), flush=True)
    run = DevicePass(wl, softmax_scale=softmax_scale)
    run.token_recovery_step(budgets)
    torch.cuda.synchronize()
    return run, run.token_recovery.cpu().numpy()


@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("budgets", [[16], [1, 40], [3, 64, 65, 200], [1, 2, 8, 33, 128, 129, 500, 100000]])
def test_every_query_of_a_ragged_varlen_batch(block, budgets):
    wl = make_custom([5 * block + 37, 1, block - 3, 2 * block, 3 * block + 1], 8, 2, block,
                     [2] * 8, seed=71, name="token_recovery_b%d" % block)
    run, got = _run(wl, budgets)
    want = orc.token_recovery(wl.q, wl.k, wl.cu_seqlens, budgets)
    assert not np.isnan(got).any()
    np.testing.assert_allclose(got, want, rtol=TOKEN_RECOVERY_RTOL, atol=TOKEN_RECOVERY_ATOL)
    heads = S.shplb_token_recovery_heads(run.p, got)
    np.testing.assert_allclose(heads, orc.token_recovery_heads(want), rtol=TOKEN_RECOVERY_RTOL)
    assert (np.diff(heads, axis=1) >= -1e-7).all()                 # more keys never hold less


def test_equal_weights_are_ties_at_the_threshold():
    # all keys equal: every weight of a query ties with its k-th largest; the k best hold min(k, t+1)/(t+1)
    T, block = 700, 128
    rng = np.random.default_rng(4)
    wl = make_custom([T], 2, 1, block, [2, 2], seed=1, name="token_recovery_ties")
    wl.k = bf16_bits_from_f32(np.tile(rng.standard_normal((1, 1, 128)).astype(np.float32), (T, 1, 1)))
    budgets = [1, 100, 699]
    _, got = _run(wl, budgets)
    t = np.arange(T)
    for b, kk in enumerate(budgets):
        want = np.minimum(kk, t + 1) / (t + 1.0)
        np.testing.assert_allclose(got[b], np.tile(want, (2, 1)), rtol=TOKEN_RECOVERY_RTOL)


def test_one_dominant_key_and_a_custom_scale():
    # a sharp softmax (large scale): the best key alone holds nearly everything, log-weights span hundreds
    wl = make_custom([900], 4, 4, 128, [2] * 4, seed=9, name="token_recovery_sharp")
    budgets = [1, 2, 50]
    _, got = _run(wl, budgets, softmax_scale=1.5)
    want = orc.token_recovery(wl.q, wl.k, wl.cu_seqlens, budgets, softmax_scale=1.5)
    np.testing.assert_allclose(got, want, rtol=TOKEN_RECOVERY_RTOL, atol=TOKEN_RECOVERY_ATOL)
    assert np.median(got[0]) > 0.9


@pytest.mark.parametrize("shape", ["ties_beside_others", "all_scores_zero", "heavy_tailed", "rising_keys", "two_levels"])
@pytest.mark.parametrize("T", [768, 769, 2600])
def test_search_on_unfavourable_scores(shape, T):
    # rows on both sides of the length from which the search samples first; runs of equal scores longer than
    # the list of a bin, a tail far outside what a sample shows, keys above the query unlike those it sees
    rng = np.random.default_rng(T)
    wl = make_custom([T], 2, 1, 128, [2, 2], seed=3, name="token_recovery_" + shape)
    q, k = rng.standard_normal((T, 2, 128)).astype(np.float32), rng.standard_normal((T, 1, 128)).astype(np.float32)
    if shape == "ties_beside_others":
        k[rng.permutation(T)[:T // 2]] = k[0]
    elif shape == "all_scores_zero":
        q[:] = 0.0
    elif shape == "heavy_tailed":
        k *= np.exp(1.5 * rng.standard_normal((T, 1, 1))).astype(np.float32)
    elif shape == "rising_keys":
        k = 0.05 * k + np.linspace(-3, 12, T, dtype=np.float32)[:, None, None] * q.mean(axis=(0, 1))
        q += 40.0 * q.mean(axis=(0, 1))
    else:
        k[:] = np.where(rng.uniform(size=(T, 1, 1)) < 0.4, k[0], k[1])
    wl.q, wl.k = bf16_bits_from_f32(q), bf16_bits_from_f32(k)
    budgets = [1, 97, T // 2, T - 1]
    _, got = _run(wl, budgets)
    want = orc.token_recovery(wl.q, wl.k, wl.cu_seqlens, budgets)
    np.testing.assert_allclose(got, want, rtol=TOKEN_RECOVERY_RTOL, atol=TOKEN_RECOVERY_ATOL)


def test_sampled_keys_of_rows_far_apart():
    # 128K tokens whose K rows lie 256 KB apart: the first sample takes every 512th key, 64 of them span 8 GiB.
    # What lies between the rows is not K: were it read for K, a score would be infinite.
    from harness import to_dev_bf16
    T, stride = 131072, 131080
    wl = make_custom([T], 2, 1, 128, [2, 2], seed=17, name="token_recovery_wide_rows")
    q = to_dev_bf16(wl.q)
    room = torch.zeros((T, stride), dtype=torch.bfloat16, device="cuda:0")
    room[:, 128::128] = float("inf")
    room[:, :128] = to_dev_bf16(wl.k)[:, 0]
    p = S.Problem(wl.cu_seqlens, 2, 1, 128, kv_stride_t=stride, kv_stride_h=128)
    budgets = [2000]
    print("case", wl.name, "kv_stride_t", stride, "budgets", budgets, flush=True)
    out = torch.full((1, 2, T), float("nan"), dtype=torch.float32, device="cuda:0")
    S.shplb_token_recovery(p, q, room, budgets, out, torch.cuda.current_stream())
    torch.cuda.synchronize()
    _, want = _run(wl, budgets)
    np.testing.assert_array_equal(out.cpu().numpy()[0, :, :2000], 1.0)
    np.testing.assert_allclose(out.cpu().numpy(), want, rtol=TOKEN_RECOVERY_RTOL, atol=TOKEN_RECOVERY_ATOL)


@pytest.mark.parametrize("what", ["one_of_each", "later_nan", "most_without_weight", "far_below"])
@pytest.mark.parametrize("T", [700, 2600])
def test_infinite_scores(what, T):
    # Infinities in K: a key that a query does not see must not change its result, a score of -inf weighs nothing.
    # Every query whose reference is a number, rows that are sampled first (2600 tokens) and rows that are not.
    rng = np.random.default_rng(T)
    wl = make_custom([T], 2, 1, 128, [2, 2], seed=6, name="token_recovery_" + what)
    q, k = rng.standard_normal((T, 2, 128)).astype(np.float32), rng.standard_normal((T, 1, 128)).astype(np.float32)
    q[:, :, 9] = 0.5 + np.abs(q[:, :, 9])
    if what == "one_of_each":
        k[T // 2, 0, 3], k[T // 2 + 40, 0, 7], k[T // 3, 0, 9] = np.inf, -np.inf, -np.inf
    elif what == "later_nan":
        k[T - 70, 0, 3] = np.nan
    elif what == "most_without_weight":
        k[rng.permutation(T)[:2 * T // 3], 0, 9] = -np.inf       # more keys wanted than weigh anything
    else:
        # the same with finite scores, of at most 9000: fp32 rounds them by 5e-4, a weight by 5e-4 / sqrt(128) = 4e-5
        k[rng.permutation(T)[:2 * T // 3], 0, 9] = -3000
    wl.q, wl.k = bf16_bits_from_f32(q), bf16_bits_from_f32(k)
    budgets = [1, 40, T // 2, T - 1]
    _, got = _run(wl, budgets)
    with np.errstate(invalid="ignore"):
        want = orc.token_recovery(wl.q, wl.k, wl.cu_seqlens, budgets)
    number = ~np.isnan(want)
    assert number.mean() > 0.4
    np.testing.assert_allclose(got[number], want[number], rtol=TOKEN_RECOVERY_RTOL, atol=TOKEN_RECOVERY_ATOL)


@pytest.mark.parametrize("budgets", [[200], [100, 400], [3, 150, 151, 1200], [1, 20, 90, 300, 700, 1300, 2000, 2800]])
@pytest.mark.parametrize("seqlens, heads", [([3100, 1100], (28, 4)), ([900, 2, 2300, 130], (20, 4))])
def test_rows_of_a_batch_taken_out_of_their_order(seqlens, heads, budgets):
    # Enough workgroups for the second lap of compute units to start on rows of half the length, in batches of
    # unequal sequences, most of whose first workgroups have no row: every query is written, and those around
    # the rows of half the length, of the sequences' ends and some others agree with the oracle.
    hq, hkv = heads
    wl = make_custom(seqlens, hq, hkv, 128, [2] * hq, seed=sum(seqlens), name="token_recovery_laps")
    levels = -(-max(seqlens) // 128)
    per_level = len(seqlens) * hq
    assert levels * per_level >= 5 * 256 and (levels // 2) * per_level >= 256     # (256 compute units)
    _, got = _run(wl, budgets)
    assert not np.isnan(got).any()
    half = (levels - levels // 2) * 128                                           # behind the first row of half the length
    rng = np.random.default_rng(len(budgets))
    tokens = set(rng.integers(0, sum(seqlens), size=20).tolist())
    for s, n in enumerate(seqlens):
        tokens |= {int(wl.cu_seqlens[s]) + t for t in (0, half - 129, half - 128, half - 1, half, n - 1) if 0 <= t < n}
    tokens = sorted(tokens)
    want = orc.token_recovery(wl.q, wl.k, wl.cu_seqlens, budgets, tokens=tokens)
    np.testing.assert_allclose(got[:, :, tokens], want[:, :, tokens], rtol=TOKEN_RECOVERY_RTOL, atol=TOKEN_RECOVERY_ATOL)


def test_is_deterministic():
    wl = make_workload(1, seqlens=[3000])
    run, a = _run(wl, [256])
    run.token_recovery_step([256])
    torch.cuda.synchronize()
    np.testing.assert_array_equal(a, run.token_recovery.cpu().numpy())


def test_32k_layer_at_the_profiled_budget_on_sampled_queries():
    # The setting of Section 2.4: a 32K context, k = 4096 tokens, one figure per head.  Sampled queries
    # against the oracle (first and last query, both sides of the budget, random ones); every value in (0, 1].
    wl = make_workload(1)
    T = int(wl.cu_seqlens[-1])
    budgets = [4096]
    run, got = _run(wl, budgets)
    t0 = time.perf_counter()
    run.token_recovery_step(budgets)
    torch.cuda.synchronize()
    print("  32K, k = 4096: %.1f ms" % ((time.perf_counter() - t0) * 1e3), flush=True)
    assert not np.isnan(got).any() and (got > 0).all() and (got <= 1 + 1e-5).all()
    np.testing.assert_array_equal(got[0][:, :4096], 1.0)           # these queries see at most 4096 keys
    rng = np.random.default_rng(12)
    tokens = sorted({0, 4095, 4096, 4097, T - 1} | set(rng.integers(4096, T, size=40).tolist()))
    want = orc.token_recovery(wl.q, wl.k, wl.cu_seqlens, budgets, tokens=tokens)
    np.testing.assert_allclose(got[:, :, tokens], want[:, :, tokens], rtol=TOKEN_RECOVERY_RTOL, atol=TOKEN_RECOVERY_ATOL)
    heads = S.shplb_token_recovery_heads(run.p, got)
    print("  recovery per head at k = 4096:", np.round(heads[:, 0], 3), flush=True)
    assert heads.min() > 0.125 and heads.max() <= 1 + 1e-5        # a head recovers at least k/T by taking any k keys


def test_128k_layer_two_budgets_on_sampled_queries():
    # the longest context of the evaluation: 1024 key blocks per row, two budgets in one call
    wl = make_workload(2)
    T = int(wl.cu_seqlens[-1])
    budgets = [1024, 4096]
    run, got = _run(wl, budgets)
    assert not np.isnan(got).any() and (got > 0).all() and (got <= 1 + 1e-5).all()
    np.testing.assert_array_equal(got[0][:, :1024], 1.0)
    np.testing.assert_array_equal(got[1][:, :4096], 1.0)
    worst = float((got[0] - got[1]).max())
    print("  largest amount by which 1024 keys exceed 4096 keys: %.3g" % worst, flush=True)
    assert worst <= 2e-5                                           # more keys never hold less (fp32 sums of 4096 terms)
    rng = np.random.default_rng(13)
    tokens = sorted({1023, 1024, 4096, T - 1} | set(rng.integers(4096, T, size=20).tolist()))
    want = orc.token_recovery(wl.q, wl.k, wl.cu_seqlens, budgets, tokens=tokens)
    np.testing.assert_allclose(got[:, :, tokens], want[:, :, tokens], rtol=TOKEN_RECOVERY_RTOL, atol=TOKEN_RECOVERY_ATOL)
