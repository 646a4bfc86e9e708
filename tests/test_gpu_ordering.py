"""How the rows of an attention launch are dealt to its workgroups, where the cases change.  The ordering kernel:
more (sequence, head) pairs than one batch holds, fewer K/V streams than dies (a stream is spread over several
dies), rows without a block, and pieces of split rows in both layouts.  Launches of at most two 64-token or 128-token
rows per compute unit (four for 64-token rows of more than two) have no queues: runs of rows, or laps.
Every row must be dealt exactly once and the attention output match the oracle."""
import numpy as np
import pytest
import torch

import paper_2603_10353_amd as S
from oracle import shplb_oracle as orc
from workloads import make_custom, one_kv_head_per_query_head

from checks import compare_output
from harness import DevicePass, queues_of
from test_gpu_parity import _split_against_whole_rows, full_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seq, heads", [(64, (40, 8)), (1, (6, 1)), (1, (6, 3)), (1, (10, 5)), (2, (4, 2)), (7, (3, 1)), (9, (3, 1))])
def test_every_row_is_dealt_once(n_seq, heads):
    # the first shape through the sorting kernel (2560 pairs), the others without queues: up to 140 rows
    # in runs, 315 and 393 in laps
    hq, hkv = heads
    rng = np.random.default_rng(100 * n_seq + hq)
    top = 90 if n_seq == 64 else 64 * 23
    seqlens = [int(x) for x in rng.integers(1, top, size=n_seq)]
    budgets = rng.choice([2, 3, 5, 999], size=n_seq * hq).tolist()
    wl = make_custom(seqlens, hq, hkv, 64, budgets, seed=400 + n_seq, name="order_%d_%d_%d" % (n_seq, hq, hkv))
    run = full_parity(wl)
    st = run.stats_host()
    assert st["n_items"].sum() == run.rows and st["cost_blocks"].sum() == run.sel_ptr_host[-1]


@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("seqlens, heads", [
    ([230], (6, 1)), ([181], (6, 3)), ([109], (10, 5)), ([70, 67], (8, 4)), ([60, 17, 3, 41, 22, 30, 9], (6, 1)),
    ([30, 44, 7, 21, 50, 13, 36, 5, 19], (5, 1)), ([131], (8, 2)), ([40, 33, 67], (8, 2)), ([1, 260], (4, 4))])
def test_every_row_is_dealt_once_from_queues(block, seqlens, heads):
    # more rows than workgroups: 1, 3, 5, 4 x 2, 7, 9, 2, 6 and 8 K/V streams on eight dies, lengths that leave every
    # remainder over the dies of a stream, sequences of unequal length; short budgets keep the oracle quick
    hq, hkv = heads
    rng = np.random.default_rng(sum(seqlens) + hq + block)
    lens = [block * nb - int(rng.integers(0, block)) for nb in seqlens]
    budgets = rng.choice([2, 3, 5, 11], size=len(lens) * hq).tolist()
    wl = make_custom(lens, hq, hkv, block, budgets, seed=430 + len(lens), name="queues_%d_%d_%d" % (len(lens), hq, hkv))
    run = DevicePass(wl).run_all()
    assert run.rows > run.n_wg                       # (and so more than the launch has workgroups, of either kind)
    rows = sorted({0, run.rows - 1} | set(rng.integers(0, run.rows, size=120).tolist()))
    print("case", wl.name, "block", block, "rows", run.rows, "workgroups", run.n_wg, flush=True)
    out_o, lse_o = orc.sparse_attention(wl.q, wl.k, wl.v, wl.cu_seqlens, block, run.sel_ptr_host, run.sel_idx_host(), None, rows)
    compare_output(run.out_host(), out_o, run.lse_host(), lse_o)
    st = run.stats_host()
    assert st["n_items"].sum() == run.rows and st["cost_blocks"].sum() == run.sel_ptr_host[-1]
    # every row, by its denominators: those of whole causal rows are never zero, and the buffer was
    assert (run.lse != 0).all()


class QueueCase:
    """A launch whose queues are looked at: its rows, their dies, and all-zero inputs."""

    def __init__(self, block, seqlens, heads, kv_of, budget_choice):
        self.block, (hq, hkv) = block, heads
        self.rng = rng = np.random.default_rng(len(seqlens) + hq + block)
        self.lens = [block * nb - int(rng.integers(0, block)) for nb in seqlens]
        n_seq, self.nbs = len(self.lens), np.array(seqlens)
        budgets = rng.choice(budget_choice, size=n_seq * hq).astype(np.int32)
        self.p = S.Problem(np.concatenate([[0], np.cumsum(self.lens)]), hq, hkv, block, 128, kv_head_of=kv_of)
        self.n_wg = S.shplb_sched_num_workgroups(self.p)
        self.ptr = S.shplb_sel_row_ptr(self.p, budgets)
        self.kv_of = np.array(kv_of or [h // (hq // hkv) for h in range(hq)])
        self.what = np.array([(s, h, i) for s in range(n_seq) for h in range(hq) for i in range(self.nbs[s])])
        self.rows, n_streams = len(self.what), n_seq * hkv
        stream = self.what[:, 0] * hkv + self.kv_of[self.what[:, 1]]
        spread = 8 // n_streams if n_streams < 8 else 1
        self.die = stream % 8 if n_streams >= 8 else stream * spread + self.what[:, 2] % spread
        total = int(self.p.cu[-1])
        self.q = torch.zeros((total, hq, 128), dtype=torch.bfloat16, device="cuda:0")
        self.kv = torch.zeros((total, hkv, 128), dtype=torch.bfloat16, device="cuda:0")
        self.out = torch.zeros_like(self.q)

    def any_lists(self, long=None):
        """Rows of any number of blocks, the last of a head like the others: of all it sees, or 0 to 2 and, one in `long`, all."""
        n = np.array([int(self.rng.integers(0, i + 2)) for _, _, i in self.what])
        if long is not None:
            n = np.where(self.rng.integers(0, long, size=self.rows) == 0, self.what[:, 2] + 1, np.minimum(n, self.rng.integers(0, 3, size=self.rows)))
        return np.concatenate([[0], np.cumsum(n)]).astype(np.int64)

    def lists(self, sel, ascending=True):
        draw = lambda i, n: np.sort(self.rng.permutation(i + 1)[:n]) if ascending else self.rng.permutation(i + 1)[:n]
        return np.concatenate([draw(i, n) for (_, _, i), n in zip(self.what, np.diff(sel))] + [np.zeros(0)]).astype(np.int32)

    def launch(self, sel, idx, slots=0):
        args = (self.p, self.q, self.kv, self.kv, torch.from_numpy(sel).to("cuda:0"), torch.from_numpy(idx).to("cuda:0"), self.out, None, None)
        stream = torch.cuda.current_stream()
        size = S.shplb_split_workspace_bytes(self.p, slots) if slots else S.shplb_workspace_bytes(self.p)
        ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda:0")
        if slots:
            S.shplb_sparse_attn_prefill_split(*args, ws, slots, stream)
        else:
            S.shplb_sparse_attn_prefill(*args, ws, stream)
        torch.cuda.synchronize()
        return queues_of(ws, self.rows, slots)

    def rows_of(self, item):
        """Row of every item, by its sequence, head and query block."""
        at_token = np.concatenate([[0], np.cumsum(self.lens)])
        first_row = np.concatenate([[0], np.cumsum(self.nbs)]) * self.p.n_q_heads
        s_of = np.searchsorted(at_token, item[:, 8])
        assert (at_token[s_of] == item[:, 8]).all() and (at_token[s_of + 1] == item[:, 9]).all()
        assert (item[:, 10] < self.p.n_q_heads).all() and (item[:, 12] < self.nbs[s_of]).all() and (item[:, [10, 12]] >= 0).all()
        assert (item[:, 11] == self.kv_of[item[:, 10]]).all() and (item[:, 13] == self.nbs[s_of]).all()
        return first_row[s_of] + item[:, 10] * self.nbs[s_of] + item[:, 12]


def halved_rows(n, total, n_wg):
    """Which of rows of n blocks are worked on in halves: those of more than 1.2 times a workgroup's share, and 16 blocks, where the longest has 5/3 of
    it."""
    return (n > max(16, total * 6 // (n_wg * 5))) & (n.max() * 3 * n_wg >= total * 5)


def queues_of_whole_rows(block, seqlens, heads, kv_of, long=None):
    c = QueueCase(block, seqlens, heads, kv_of, [2, 3, 5, 11, 999] if long is None else [2, 3, 5])
    halves_seen = 0
    for by_budget, sel in ((True, c.ptr), (False, c.any_lists(long))):
        idx = c.lists(sel, ascending=False)
        print("case", block, seqlens[:4], heads, "rows", c.rows, "by budget", by_budget, flush=True)
        item, begin, halved = c.launch(sel, idx)
        assert c.rows > c.n_wg                                    # (so there are queues)
        assert begin.tolist() == np.concatenate([[0], np.cumsum(np.bincount(c.die, minlength=8))]).tolist()
        row = c.rows_of(item)
        assert (np.sort(row) == np.arange(c.rows)).all()
        assert (c.die[row] == np.repeat(np.arange(8), np.diff(begin))).all()
        n = np.diff(sel)[row]
        full = np.append(idx, 0)
        assert (item[:, 0] == 0).all() and (item[:, 1] == n).all() and (item[:, 2] == sel[row]).all() and (item[:, 3] == 0).all()
        assert (item[:, [4, 6, 7]] == -1).all() and (item[:, 5] == 1).all()
        assert (item[:, 14] == np.where(n > 0, full[sel[row]], 0)).all()
        assert (item[:, 15] == np.where(n > 0, full[sel[row] + np.minimum(1, np.maximum(n - 1, 0))], 0)).all()
        for x in range(8):
            assert (np.diff(n[begin[x]:begin[x + 1]]) <= 0).all()
        # which launches have halves at all is decided by the shapes: what the rows of any budgets select at least
        n_sh = len(seqlens) * heads[0]
        if block == 128 and c.rows <= 6 * c.n_wg and n_sh <= 2048 and halved_rows(np.array(seqlens), 2 * c.rows - n_sh, c.n_wg).any():
            assert halved.tolist() == np.bincount(c.die[halved_rows(np.diff(sel), int(sel[-1]), c.n_wg)], minlength=8).tolist()
            halves_seen += int(halved.sum())
    return halves_seen


@pytest.mark.parametrize("block, seqlens, heads, kv_of", [
    (128, [230], (6, 1), None), (128, [181], (6, 3), None), (64, [300], (10, 5), None), (128, [70, 67], (8, 4), None),
    (128, [33, 1, 64], (28, 4), None), (64, [97, 31, 32], (16, 8), None), (64, [17] * 64, (32, 8), None),
    (128, [90, 40], (8, 2), [0, 1, 1, 1, 1, 1, 1, 1]), (64, [131, 9], (24, 9), [x % 9 for x in range(24)])])
def test_queues_hold_every_row_by_cost(block, seqlens, heads, kv_of):
    # What the ordering kernel leaves in the workspace, where rows count their places for themselves (up to 2048
    # (sequence, head) pairs: the seventh shape): 1, 3, 5, 8, 12 .. 512 K/V streams on eight dies, heads of a stream and mapped ones, runs of 32 rows
    # that end inside a head; for rows of a budget and for rows of any number of blocks, none among them.  The long rows that
    # are worked on in halves are counted per queue, in ragged batches and with mapped heads too.
    halves = queues_of_whole_rows(block, seqlens, heads, kv_of)
    assert halves > 0 or block == 64


def test_rows_hardly_longer_than_the_share_stay_whole():
    # 1280 rows of up to 20 blocks, the share of a workgroup being 13 to 16: the longest rows stay whole, with others of 40 blocks they do not.
    for extra in (20, 40):
        c = QueueCase(128, [40], (32, 8), None, [2, 3, 4, 20])
        budgets = np.array([2, 3, 4, 20] * 7 + [20, 2, 2, extra], np.int32)
        sel = S.shplb_sel_row_ptr(c.p, budgets)
        n, share = np.diff(sel), sel[-1] / c.n_wg
        expect = halved_rows(n, int(sel[-1]), c.n_wg)
        print("share %.1f longest %d" % (share, n.max()), flush=True)
        assert (n > 1.2 * share).any() and expect.any() == (extra == 40)
        _, _, halved = c.launch(sel, c.lists(sel))
        assert halved.tolist() == np.bincount(c.die[expect], minlength=8).tolist()


def queues_of_pieces(block, seqlens, heads, kv_of, slots, long=None):
    # Every block of a row is in one of its pieces, in order; slots and counters are a split row's own and within what the workspace
    # holds; items lie by the cost of their rows, whose pieces are as many as split_length() makes of what they select.
    c = QueueCase(block, seqlens, heads, kv_of, [2, 3, 11, 999, 999] if long is None else [2] * 9 + [999])
    rows, share_wg = c.rows, c.n_wg // 2 if block == 128 and c.rows <= c.n_wg // 2 else c.n_wg
    cut_rows = 0
    for by_budget, sel in ((True, c.ptr), (False, c.any_lists(long))):
        idx = c.lists(sel)
        cost = int(sel[-1])
        cut = max(32 * 64 // block, -(-2 * cost // slots), -(-cost // (share_wg * 2)))
        wanted = np.clip(-(-np.diff(sel) // cut), 1, 64)              # pieces of a row
        print("case", block, seqlens[:4], heads, "rows", rows, "cut at", cut, "split rows", int((wanted > 1).sum()), "by budget", by_budget, flush=True)
        item, begin, _ = c.launch(sel, idx, slots)
        assert begin.tolist() == np.concatenate([[0], np.cumsum(np.bincount(c.die, weights=wanted, minlength=8))]).astype(int).tolist()
        item = item[:int(wanted.sum())]
        row = c.rows_of(item)
        assert (np.bincount(row, minlength=rows) == wanted).all()
        assert (c.die[row] == np.repeat(np.arange(8), np.diff(begin))).all()
        n_of = np.diff(sel)[row]
        for x in range(8):
            assert (np.diff(n_of[begin[x]:begin[x + 1]]) <= 0).all()
        whole = wanted[row] == 1
        assert (item[whole, 1] == n_of[whole]).all() and (item[whole, 2] == sel[row[whole]]).all()
        assert (item[whole][:, [4, 6, 7]] == -1).all() and (item[whole, 5] == 1).all()
        some = item[:, 1] > 0
        assert (item[some, 14] == idx[item[some, 2]]).all() and (item[some, 15] == idx[item[some, 2] + np.minimum(1, item[some, 1] - 1)]).all()
        used, counters = [], []
        for r in np.flatnonzero(wanted > 1):
            pieces = item[row == r]
            assert (pieces[:, 1] > 0).all() and int(pieces[:, 1].sum()) == sel[r + 1] - sel[r]
            assert (pieces[:, 2] == sel[r] + np.concatenate([[0], np.cumsum(pieces[:, 1])])[:-1]).all()
            assert (pieces[:, 5] == len(pieces)).all() and (pieces[:, 6] == pieces[0, 6]).all() and (pieces[:, 7] == pieces[0, 7]).all()
            assert (pieces[:, 4] == pieces[0, 6] + np.arange(len(pieces))).all()
            used += pieces[:, 4].tolist()
            counters.append(int(pieces[0, 7]))
        assert len(set(used)) == len(used) and len(set(counters)) == len(counters)
        assert not used or (min(used) >= 0 and max(used) < slots and min(counters) >= 0 and max(counters) <= slots // 2)
        cut_rows += len(counters)
    return cut_rows


@pytest.mark.parametrize("block, seqlens, heads, kv_of, slots", [
    (128, [230], (6, 1), None, 64), (128, [181], (6, 3), None, 2048), (64, [300], (10, 5), None, 512), (128, [70, 67], (8, 4), None, 2048),
    (128, [33, 1, 64], (28, 4), None, 2048), (64, [97, 31, 32], (16, 8), None, 3), (128, [17] * 64, (32, 8), None, 4096),
    (128, [90, 40], (8, 2), [0, 1, 1, 1, 1, 1, 1, 1], 2048), (64, [131, 9], (24, 9), [x % 9 for x in range(24)], 2048), (128, [40], (4, 4), None, 2048)])
def test_queues_hold_every_piece_of_cut_rows(block, seqlens, heads, kv_of, slots):
    # The same with pieces, for rows of a budget and for rows of any number of blocks.
    queues_of_pieces(block, seqlens, heads, kv_of, slots)


# Beyond 2048 (sequence, head) pairs or 65536 rows (16384 with pieces) a workgroup per die sorts its rows: eight streams and more, three and one
# (spread by query block), mapped heads, sequences of one block among long ones.  On the other side of the limits too: 2048 pairs, as many rows
# as are counted, on all dies and on one, and the most blocks of a sequence.
@pytest.mark.parametrize("block, seqlens, heads, kv_of, long", [
    (64, [150, 3, 140] + [1] * 61, (40, 8), None, 9), (128, [9], (2100, 3), None, 9), (128, [9], (2100, 1), None, 9),
    (64, [40, 3] + [2] * 62, (40, 9), [x % 9 for x in range(40)], 9), (64, [4096], (17, 1), None, 200), (64, [4096], (16, 1), None, 200),
    (64, [4000] + [1] * 7, (16, 1), None, 200), (64, [32], (2048, 8), None, 9)])
def test_queues_of_larger_launches(block, seqlens, heads, kv_of, long):
    queues_of_whole_rows(block, seqlens, heads, kv_of, long)


@pytest.mark.parametrize("block, seqlens, heads, kv_of, slots, long", [
    (64, [150, 3, 140] + [1] * 61, (40, 8), None, 2048, 50), (64, [33], (2052, 3), None, 65536, 300), (128, [2100], (8, 1), None, 2048, 50),
    (64, [90, 70] + [1] * 62, (40, 9), [x % 9 for x in range(40)], 300, 50), (128, [2048], (8, 1), None, 2048, 50), (64, [4096], (4, 1), None, 2048, 50)])
def test_queues_of_pieces_of_larger_launches(block, seqlens, heads, kv_of, slots, long):
    assert queues_of_pieces(block, seqlens, heads, kv_of, slots, long) > 0


@pytest.mark.parametrize("block, n_blocks, heads", [(128, 70, (8, 2)), (64, 140, (10, 5))])
def test_lists_that_follow_no_budget(block, n_blocks, heads):
    # Lists of a caller's own whose last row of a head is short and whose earlier ones are long, and the other way round: long rows
    # are in halves or cut, short ones whole, and the outputs are the oracle's.
    hq, hkv = heads
    wl = make_custom([block * n_blocks - 9], hq, hkv, block, [2] * hq, seed=910 + block, name="no_budget_%d" % block)
    rng = np.random.default_rng(911)
    run = DevicePass(wl)
    lists = []
    for h in range(hq):
        for i in range(n_blocks):
            long = i < n_blocks - 1 and i % 7 == 5 if h % 2 == 0 else i == n_blocks - 1
            lists.append(np.arange(i + 1) if long else np.union1d(rng.integers(0, i + 1, size=(i + h) % 5 // 2), [i]))
    ptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    idx = np.concatenate(lists).astype(np.int32)
    n = np.diff(ptr)
    rows = sorted(set(np.argsort(n)[-6:].tolist()) | set(rng.integers(0, run.rows, size=60).tolist()) | {n_blocks - 1, 2 * n_blocks - 1})
    out_o, lse_o = orc.sparse_attention(wl.q, wl.k, wl.v, wl.cu_seqlens, block, ptr, idx, None, rows)
    run.sel_ptr, run.sel_idx = torch.from_numpy(ptr).to("cuda:0"), torch.from_numpy(idx).to("cuda:0")
    cut = max(32 * 64 // block, -(-int(ptr[-1]) // (run.n_wg * 2)))
    wanted = np.clip(-(-n // cut), 1, 64)
    print("case", wl.name, "rows", run.rows, "blocks", int(ptr[-1]), "cut at", cut, "split rows", int((wanted > 1).sum()), flush=True)
    assert (wanted > 1).any() and wanted[n_blocks - 1] == 1
    for step, items in ((run.attn_step, run.rows), (lambda: run.attn_split_step(2048), int(wanted.sum()))):
        run.out.zero_()
        run.lse.zero_()
        step()
        torch.cuda.synchronize()
        st = run.stats_host()
        assert st["n_items"].sum() == items and st["cost_blocks"].sum() == ptr[-1]
        compare_output(run.out_host(), out_o, run.lse_host(), lse_o)
        assert (run.lse != 0).all()


@pytest.mark.parametrize("block, n_blocks, heads", [(128, 16, (32, 8)), (128, 17, (32, 8)), (64, 32, (40, 8)), (64, 33, (40, 8)), (128, 3, (8, 2))])
def test_rows_too_short_to_cut_through_the_splitting_entry_point(block, n_blocks, heads):
    # Up to 16 blocks of 128 tokens or 32 of 64 no row is cut: no queue, or the same as without splitting; beyond, as many
    # pieces as rows.  The same bits as from the entry point of whole rows (with 64-token rows shared by two groups of waves too).
    hq, hkv = heads
    wl = make_custom([block * n_blocks - 9], hq, hkv, block, [999] * (hq // 2) + [3] * (hq // 2), seed=700 + n_blocks, name="uncut_%d" % n_blocks)
    run = DevicePass(wl).run_all()
    out, lse = run.out.clone(), run.lse.clone()
    run.out.zero_()
    run.attn_split_step(64)
    torch.cuda.synchronize()
    st = run.stats_host()
    assert st["n_items"].sum() == run.rows and st["cost_blocks"].sum() == run.sel_ptr_host[-1]
    assert torch.equal(run.out.view(torch.int16), out.view(torch.int16)) and torch.equal(run.lse, lse)


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


@pytest.mark.parametrize("n_blocks, tail, heads", [(1, 5, (32, 8)), (2, 64, (8, 2)), (3, 1, (8, 2)), (5, 40, (8, 8)), (8, 63, (32, 8)), (9, 31, (8, 1)), (32, 64, (8, 8)), (250, 33, (1, 1))])
def test_64_token_rows_with_waves_that_copy(n_blocks, tail, heads):
    # Up to one row per compute unit: two waves copy three steps ahead.  Rows of one block up to many, odd and even, so that a
    # group has two, four, six and more tiles, none beyond them and none of its own; ragged tails; selections that begin with
    # another block than the sink, a single one and none.
    hq, hkv = heads
    T = 64 * (n_blocks - 1) + tail
    budgets = ([2, 3, 4, 5, 6, 7, 9, 999] * 4)[:hq] if hq > 1 else [999]
    wl = make_custom([T], hq, hkv, 64, budgets, seed=760 + n_blocks, name="copiers_%d" % n_blocks)
    rows = None if n_blocks <= 32 else [0, 1, 2, 3, 100, 248, 249]
    run = full_parity(wl, rows=rows)
    assert run.rows <= run.n_wg // 4
    pick = [lambda i: list(range(max(0, i - 2), i + 1)), lambda i: [i], lambda i: [] if i % 3 == 1 else [i // 2, i] if i else [0], lambda i: list(range(i + 1))]
    lists = [pick[h % 4](i) for h in range(hq) for i in range(n_blocks)]
    ptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    idx = np.concatenate([np.asarray(x, np.int32) for x in lists])
    run.attn_step(torch.from_numpy(ptr).to("cuda:0"), torch.from_numpy(idx).to("cuda:0"))
    torch.cuda.synchronize()
    at = [r for r in (range(len(lists)) if rows is None else rows) if len(lists[r])]
    out_o, lse_o = orc.sparse_attention(wl.q, wl.k, wl.v, wl.cu_seqlens, 64, ptr, idx, None, at)
    compare_output(run.out_host(), out_o, run.lse_host(), lse_o)


@pytest.mark.parametrize("n_blocks", [1, 5, 6])
def test_groups_of_waves_keep_infinite_values_apart(n_blocks):
    # The last block's first token has an infinite value in one dim: every query of that block sees it, and no
    # other dim or block may be touched by it.  A group of waves whose blocks ran out (rows of an odd number of
    # blocks) must not multiply it by zero.
    T = 64 * n_blocks
    wl = make_custom([T], 2, 1, 64, [999, 999], seed=520 + n_blocks, name="infinite_value_%d" % n_blocks)
    wl.v[T - 64, 0, 5], wl.v[T - 64, 0, 6] = 0x7f80, 0xff80            # bf16 infinities
    print("case", wl.name, flush=True)
    out = DevicePass(wl).run_all().out_host()
    assert (out[T - 64:, :, 5] == np.inf).all() and (out[T - 64:, :, 6] == -np.inf).all()
    rest = np.ones(out.shape, bool)
    rest[T - 64:, :, 5:7] = False
    assert np.isfinite(out[rest]).all()


@pytest.mark.parametrize("heads, block, n_blocks, budgets", [
    ((8, 2), 128, 64, [64, 2, 2, 2, 2, 26, 2, 2]), ((8, 2), 128, 62, [62, 62, 2, 2, 2, 2, 2, 2]),
    ((4, 2), 128, 128, [128, 4, 4, 4]), ((2, 1), 64, 256, [256, 8]), ((6, 1), 64, 170, [170, 170, 2, 2, 2, 2])])
def test_few_long_rows_are_spread_over_the_compute_units(heads, block, n_blocks, budgets):
    # Launches of one to four rows per compute unit, without queues: a dense head or two, and no compute unit may be
    # given much more than the longest row (the least possible).
    hq, hkv = heads
    wl = make_custom([block * n_blocks - 5], hq, hkv, block, budgets, seed=540 + n_blocks, name="spread_%d" % n_blocks)
    run = DevicePass(wl).run_all()
    heaviest = []
    for launch in range(3):                            # (the dispatcher has the last word: the best of three)
        run.attn_step()
        torch.cuda.synchronize()
        st = run.stats_host()
        assert run.rows <= run.n_wg and st["n_items"].sum() == run.rows and st["cost_blocks"].sum() == run.sel_ptr_host[-1]
        load = {}
        for r in st[st["n_items"] > 0]:
            cu = (int(r["xcc_id"]), int(r["cu_id"]))
            load[cu] = load.get(cu, 0) + int(r["cost_blocks"])
        heaviest.append(max(load.values()))
    print("case", wl.name, "rows", run.rows, "compute units", len(load), "heaviest", heaviest, flush=True)
    assert min(heaviest) <= 1.3 * n_blocks


def test_rows_without_a_block_do_not_end_a_workgroup():
    # Seven of eight heads select one block for one row and nothing for the others: their output stays as it
    # is, and the workgroups that are dealt such a row go on and help with the eighth head's.
    nb, block, window = 256, 128, 40
    wl = make_custom([block * nb], 8, 8, block, [2] * 8, seed=90, name="empty_rows")
    run = DevicePass(wl)
    lists = [list(range(max(0, i - window + 1), i + 1)) if h == 3 else [0] if i == 0 else [] for h in range(8) for i in range(nb)]
    ptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    idx = np.concatenate([np.asarray(x, np.int32) for x in lists])
    print("case", wl.name, flush=True)
    run.attn_step(torch.from_numpy(ptr).to("cuda:0"), torch.from_numpy(idx).to("cuda:0"))
    torch.cuda.synchronize()
    st = run.stats_host()
    assert st["n_items"].sum() == nb + 7 and st["cost_blocks"].sum() == len(idx)
    assert (st["n_items"] > 0).sum() >= 160                            # not the 64 of one die alone and seven more
    rows = [r for r in range(8 * nb) if len(lists[r]) and (r % nb < 3 or r % 37 == 0)]
    out_o, lse_o = orc.sparse_attention(wl.q, wl.k, wl.v, wl.cu_seqlens, block, ptr, idx, None, rows)
    compare_output(run.out_host(), out_o, run.lse_host(), lse_o)
    out = run.out.view(nb, block, 8, 128)
    assert not out[1:, :, [0, 1, 2, 4, 5, 6, 7]].any()


@pytest.mark.parametrize("block, nb", [(64, 9), (128, 5), (128, 9)])
def test_selections_that_do_not_begin_with_the_sink(block, nb):
    # Rows without queues start on block 0 before they know their selection: windows, single blocks (with two groups
    # of waves one has nothing), no block at all, and rows that do begin with it, one and two sequences.
    for lens in ([block * nb - 17], [block * nb - 17, block * 3 + 1]):
        wl = make_custom(lens, 4, 2, block, [2] * (4 * len(lens)), seed=100 + nb, name="no_sink_%d_%d" % (block, nb))
        run = DevicePass(wl)
        pick = [lambda i: list(range(max(0, i - 2), i + 1)), lambda i: [i], lambda i: [] if i % 3 == 1 else [i // 2, i] if i else [0],
                lambda i: list(range(0, i + 1))]
        lists = [pick[h](i) for n in lens for h in range(4) for i in range(-(-n // block))]
        ptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
        idx = np.concatenate([np.asarray(x, np.int32) for x in lists])
        print("case", wl.name, len(lens), flush=True)
        run.attn_step(torch.from_numpy(ptr).to("cuda:0"), torch.from_numpy(idx).to("cuda:0"))
        torch.cuda.synchronize()
        rows = [r for r in range(len(lists)) if len(lists[r])]
        out_o, lse_o = orc.sparse_attention(wl.q, wl.k, wl.v, wl.cu_seqlens, block, ptr, idx, None, rows)
        compare_output(run.out_host(), out_o, run.lse_host(), lse_o)


@pytest.mark.parametrize("n_blocks, budgets", [(6, [2, 3, 6, 5]), (7, [2, 3, 7, 5]), (32, [2, 3, 4, 5, 32, 7, 31, 20]), (33, [2, 3, 4, 5, 33, 7, 31, 20])])
def test_128_token_rows_shared_by_two_groups_of_waves(n_blocks, budgets):
    # Rows of launches of up to one per compute unit (256) are shared by two groups of waves half a step apart: few rows,
    # the last size of the rule and the first of the other, rows of one block, odd and even numbers, a ragged tail; and an
    # infinite value that every query of the last block sees, of a row of an odd number of blocks too.
    T = 128 * n_blocks - 45
    wl = make_custom([T], len(budgets), 1, 128, budgets, seed=560 + n_blocks, name="groups_128_%d" % n_blocks)
    full_parity(wl)
    last = 128 * (n_blocks - 1)
    wl.v[last, 0, 5], wl.v[last, 0, 6] = 0x7f80, 0xff80                # bf16 infinities
    out = DevicePass(wl).run_all().out_host()
    assert (out[last:, :, 5] == np.inf).all() and (out[last:, :, 6] == -np.inf).all()
    assert np.isfinite(np.delete(out[last:], [5, 6], axis=2)).all() and np.isfinite(out[:last]).all()


@pytest.mark.parametrize("n_blocks, tail, heads, times", [(1, 37, (8, 2), 64), (2, 128, (4, 2), 64), (7, 9, (32, 8), 2), (7, 9, (32, 8), 3),
                                                         (33, 64, (4, 1), 3), (64, 1, (4, 4), 3)])
def test_a_128_token_sequence_alone_and_in_a_larger_call(n_blocks, tail, heads, times):
    # The same bits in a launch of up to 256 rows, whose rows two groups of waves share, in one of up to 512 and in one with
    # queues; odd and even numbers of blocks, ragged tails.  Half of the queries of every 32 meet scores far above the earlier ones
    # (a later key's component 9), in one of two heads: references are raised for 16 queries at a time.
    hq, hkv = heads
    T = 128 * (n_blocks - 1) + tail
    budgets = np.random.default_rng(n_blocks).integers(2, n_blocks + 2, hq).tolist()
    one = make_custom([T], hq, hkv, 128, budgets, seed=600 + n_blocks, name="alone_%d" % n_blocks)
    sign = np.where(np.arange(T) % 32 < 16, 0x4000, 0xc000).astype(np.uint16)                  # 2 and -2
    one.q[:, ::2, 9] = sign[:, None]
    for j in range(1, n_blocks):
        one.k[128 * j, :, 9] = 0x4270 + 8 * j                                                  # from 60 on: 10.6 nats and more
    many = make_custom([T] * times, hq, hkv, 128, budgets, seed=1, name="together_%d" % n_blocks)
    for name in ("q", "k", "v"):
        setattr(many, name, np.tile(getattr(one, name), (times, 1, 1)))
    a, b = DevicePass(one).run_all(), DevicePass(many).run_all()
    print("case", one.name, "rows", a.rows, b.rows, flush=True)
    assert a.rows <= 256 < b.rows
    out_o, lse_o = orc.sparse_attention(one.q, one.k, one.v, one.cu_seqlens, 128, a.sel_ptr_host, a.sel_idx_host(), None, None)
    compare_output(a.out_host(), out_o, a.lse_host(), lse_o)
    for x in range(times):
        at = slice(x * T, (x + 1) * T)
        assert torch.equal(a.sel_idx, b.sel_idx[x * len(a.sel_idx):(x + 1) * len(a.sel_idx)])
        assert torch.equal(a.out.view(torch.int16), b.out[at].view(torch.int16)) and torch.equal(a.lse, b.lse[:, at])


@pytest.mark.parametrize("n_blocks, tail, heads, budgets", [(70, 128, (8, 2), [999] + [2] * 7), (70, 1, (8, 2), [2, 2, 999, 2, 2, 40, 2, 2]), (66, 64, (8, 8), [999, 3] * 4),
                                                           (65, 65, (8, 4), [2] * 7 + [50]), (520, 30, (1, 1), [999]), (131, 90, (4, 1), [2, 9, 999, 2])])
def test_long_rows_in_halves(n_blocks, tail, heads, budgets):
    # Launches of up to six 128-token rows a workgroup have rows of more than 1.2 times the average share worked on in halves of
    # 64 queries, where the longest has 5/3 of it: the same bits as whole rows, which they are among seven copies of the sequence; every row counted once; a last
    # block whose second half has no query, and references raised in one of the halves only (a later key's component 9).
    hq, hkv = heads
    T = 128 * (n_blocks - 1) + tail
    one = make_custom([T], hq, hkv, 128, budgets, seed=640 + n_blocks + tail, name="halves_%d_%d" % (n_blocks, tail))
    one.q[:, ::2, 9] = np.where(np.arange(T) % 128 < 64, 0x4000, 0xc000).astype(np.uint16)[:, None]     # 2 and -2
    one.k[128 * np.arange(1, n_blocks), :, 9] = (0x4200 + 2 * (np.arange(1, n_blocks) % 64)).astype(np.uint16)[:, None]   # from 32 on
    many = make_custom([T] * 7, hq, hkv, 128, budgets, seed=1, name="whole_%d" % n_blocks)
    for name in ("q", "k", "v"):
        setattr(many, name, np.tile(getattr(one, name), (7, 1, 1)))
    a, b = DevicePass(one).run_all(), DevicePass(many).run_all()
    n = np.diff(a.sel_ptr_host)
    above = max(16, n.sum() * 6 // (a.n_wg * 5))
    print("case", one.name, "rows", a.rows, b.rows, "in halves", int((n > above).sum()), flush=True)
    assert a.n_wg < a.rows <= 6 * a.n_wg < b.rows and halved_rows(n, int(n.sum()), a.n_wg).any()
    st = a.stats_host()
    assert st["n_items"].sum() == a.rows and st["cost_blocks"].sum() == n.sum()
    # Every workgroup that worked says when, and all start with the launch, those that begin with a second half too: at its end such a
    # half has taken more than half of an average share, about as much of the launch.  (Workgroups start within some microseconds.)
    worked = st["cost_blocks"] > 0
    assert (worked == (st["t_last"] > 0)).all() and (st["t_first"][worked] > 0).all() and (st["t_first"] < st["t_last"])[worked].all()
    late = (st["t_first"] - st["t_first"][worked].min())[worked].astype(np.float64) / (st["t_last"].max() - st["t_first"][worked].min())
    print("latest start %.3f of the launch" % late.max(), flush=True)
    assert late.max() < 0.3
    assert torch.equal(a.sel_idx, b.sel_idx[:len(a.sel_idx)])
    assert torch.equal(a.out.view(torch.int16), b.out[:T].view(torch.int16)) and torch.equal(a.lse, b.lse[:, :T])
    rows = np.flatnonzero(n > above)[[0, 1, -2, -1]].tolist() + [0, n_blocks - 1]
    out_o, lse_o = orc.sparse_attention(one.q, one.k, one.v, one.cu_seqlens, 128, a.sel_ptr_host, a.sel_idx_host(), None, rows)
    compare_output(a.out_host(), out_o, a.lse_host(), lse_o)


@pytest.mark.parametrize("lens, heads, kv_of", [([128 * 50 - 9, 128 * 20 - 100, 130], (8, 2), None), ([128 * 66 - 1, 300], (8, 2), [0, 1, 1, 1, 1, 1, 1, 1]),
                                                ([200, 128 * 40 - 64, 128 * 35 - 127], (9, 3), [2, 0, 0, 0, 1, 0, 2, 2, 0])])
def test_halves_of_batches_and_mapped_heads(lens, heads, kv_of):
    # Long rows in halves where the sequences are of unequal length or the heads have a map, for the lists of budgets, and for lists
    # of which every third row has no block (its output stays as it is).
    hq, hkv = heads
    wl = make_custom(lens, hq, hkv, 128, ([999] + [2] * (hq - 2) + [3]), seed=670 + len(lens) + hq, name="halves_batch")
    if kv_of:
        wl.kv_head_of = np.array(kv_of, np.int32)
    run = DevicePass(wl).run_all()
    plain = one_kv_head_per_query_head(wl) if kv_of else wl
    n = np.diff(run.sel_ptr_host)
    rng = np.random.default_rng(671)
    some = rng.permutation(run.rows)[:40].tolist()
    print("case", lens, heads, "rows", run.rows, "in halves", int(halved_rows(n, int(n.sum()), run.n_wg).sum()), flush=True)
    for empty in (False, True):
        keep = np.arange(run.rows) % 3 != 1 if empty else np.ones(run.rows, bool)
        idx = np.concatenate([run.sel_idx_host()[run.sel_ptr_host[r]:run.sel_ptr_host[r + 1]] for r in range(run.rows) if keep[r]])
        ptr = np.concatenate([[0], np.cumsum(n * keep)]).astype(np.int64)
        halved = np.flatnonzero(halved_rows(n * keep, int(ptr[-1]), run.n_wg))
        assert run.n_wg < run.rows <= 6 * run.n_wg and len(halved) > 4
        run.out.zero_()
        run.lse.zero_()
        run.attn_step(torch.from_numpy(ptr).to("cuda:0"), torch.from_numpy(idx).to("cuda:0"))
        torch.cuda.synchronize()
        st = run.stats_host()
        assert st["n_items"].sum() == keep.sum() and st["cost_blocks"].sum() == ptr[-1]
        rows = [r for r in set(some) | set(halved[[0, 1, -2, -1]].tolist()) if keep[r]]
        out_o, lse_o = orc.sparse_attention(plain.q, plain.k, plain.v, wl.cu_seqlens, 128, ptr, idx, None, rows)
        compare_output(run.out_host(), out_o, run.lse_host(), lse_o)
        written = np.zeros((hq, int(wl.cu_seqlens[-1])), bool)
        for r in np.flatnonzero(keep):
            s, h, i = orc.row_decode(wl.cu_seqlens, 128, hq, r)
            written[h, wl.cu_seqlens[s] + 128 * i:min(wl.cu_seqlens[s] + 128 * (i + 1), wl.cu_seqlens[s + 1])] = True
        assert ((run.lse.cpu().numpy() != 0) == written).all()
