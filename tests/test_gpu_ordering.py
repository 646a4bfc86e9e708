"""The ordering kernel where its cases change: more (sequence, head) pairs than one batch holds, fewer
K/V streams than dies (a stream is spread over several dies), and pieces of split rows in both layouts.
Every row must be dealt exactly once and the attention output match the oracle."""
import numpy as np
import pytest

from workloads import make_custom

from test_gpu_parity import _split_against_whole_rows, full_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seq, heads", [(64, (40, 8)), (1, (6, 1)), (1, (6, 3)), (1, (10, 5)), (2, (4, 2)), (7, (3, 1)), (9, (3, 1))])
def test_every_row_is_dealt_once(n_seq, heads):
    hq, hkv = heads
    rng = np.random.default_rng(100 * n_seq + hq)
    top = 90 if n_seq == 64 else 64 * 23
    seqlens = [int(x) for x in rng.integers(1, top, size=n_seq)]
    budgets = rng.choice([2, 3, 5, 999], size=n_seq * hq).tolist()
    wl = make_custom(seqlens, hq, hkv, 64, budgets, seed=400 + n_seq, name="order_%d_%d_%d" % (n_seq, hq, hkv))
    run = full_parity(wl)
    st = run.stats_host()
    assert st["n_items"].sum() == run.rows and st["cost_blocks"].sum() == run.sel_ptr_host[-1]


@pytest.mark.parametrize("heads", [(2, 1), (8, 8)])
def test_pieces_of_split_rows(heads):
    hq, hkv = heads
    wl = make_custom([64 * 140 + 21, 64 * 3], hq, hkv, 64, [999, 3] * hq, seed=62 + hq, name="order_split_%d" % hkv)
    _split_against_whole_rows(wl, 2048, 5 if hq == 2 else 3)


@pytest.mark.parametrize("n_blocks, budgets", [(1, [2, 2]), (64, [2, 3, 4, 5, 999, 7, 64, 33]), (65, [2, 3, 4, 5, 999, 7, 64, 33])])
def test_rows_shared_by_two_groups_of_waves(n_blocks, budgets):
    # 64-token rows of launches of up to two rows per compute unit (512) are worked on by two groups of
    # waves, each with every other selected block: rows of one block (a group with nothing), of odd and
    # even numbers, ragged tails; 520 rows go the other way.
    wl = make_custom([64 * n_blocks - 27], len(budgets), 1, 64, budgets, seed=500 + n_blocks, name="groups_%d" % n_blocks)
    full_parity(wl)
