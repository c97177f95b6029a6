"""The index half of a small batch on one workgroup, at the sizes where it can go wrong: the edges of a round of 1024
elements, the largest batch it takes on the caller's stream (8192 IDs) and ahead of time (12288, of a table of more than 65536 rows 10240), the first sizes it
leaves to the chain of launches, one list much shorter than the other, every row long, one radix pass and four.  The larger
cases run the chain.  Whole numbers: every output equals the oracle's."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2604_24073_amd as fs
from helpers import dev
from test_gpu_parity import class_order_from_oracle, zipf_ids

pytestmark = pytest.mark.gpu


@pytest.fixture
def ctx():
    # one per test: a context remembers ahead-of-time results by the address of their buffers
    c = fs.Context(max_ids=40_000, max_dim=4)
    yield c
    c.close()


def check_index_half(ctx, ids, nxt, rows, ahead):
    n0, n1 = len(ids), len(nxt)
    lay0, lay1, split = fs.alloc_layout(n0, "cuda"), fs.alloc_layout(n1, "cuda", sorted_ids=True), fs.alloc_split(n0, n1, "cuda")
    fs.fs_unique_ids(ctx, dev(ids), rows, out=lay0)
    d_nxt = dev(nxt)
    keep = [torch.zeros((k, 4), device="cuda") for k in (min(rows, 8), n0, n1)]
    args = fs.make_step_args(keep[0], torch.zeros(1, device="cuda"), 0.01, 1e-8, lay0, keep[1], d_nxt, None, lay1, split, None, keep[2])
    args.num_rows = rows                                     # the index half touches no table row
    if ahead:
        fs.fs_step_forward_ahead(ctx, args)
    else:
        fs.fs_step_forward(ctx, args)
    assert fs.fs_check_async(ctx) == fs.FS_OK
    want0, want1 = O.unique_ids(ids, rows), O.unique_ids(nxt, rows)
    for lay, want in ((lay0, want0), (lay1, want1)):
        for k in ("unique", "seg_offsets", "perm", "inverse"):
            assert np.array_equal(lay[k].cpu().numpy()[:len(want[k])], want[k]), k
        assert int(lay["n_unique"].item()) == len(want["unique"])
    assert np.array_equal(lay1["sorted_ids"].cpu().numpy(), np.sort(nxt))
    sp = O.collision_split(want0["unique"], want1["unique"])
    assert split["counts"].cpu().numpy().tolist() == [len(sp[k]) for k in ("co", "ex", "ex_next")]
    for k in ("co", "co_slot", "ex", "ex_slot", "ex_next", "ex_next_slot"):
        assert np.array_equal(split[k].cpu().numpy()[:len(sp[k])], sp[k]), k
    flag = split["co_flag_t1"].cpu().numpy()[:len(want1["unique"])]
    assert np.array_equal(flag, np.isin(want1["unique"], want0["unique"]).astype(np.uint8))
    cperm, cslot, cstart, class_pos = class_order_from_oracle(want0, sp)
    assert split["class_pos"].cpu().numpy().tolist() == [int(x) for x in class_pos]
    assert np.array_equal(split["cperm"].cpu().numpy()[:class_pos[1]], cperm)
    assert np.array_equal(split["cslot"].cpu().numpy()[:class_pos[1]], cslot)
    in_order = cstart >= 0
    assert np.array_equal(split["cstart"].cpu().numpy()[:len(cstart)][in_order], cstart[in_order])
    rec = split["short_rec"].cpu().numpy()[:24 * n0].reshape(2, n0, 12)
    seg = want0["seg_offsets"].astype(np.int64)
    for cls, name in enumerate(("co", "ex")):
        slots = sp[name + "_slot"]
        got, lens = rec[cls, :len(slots)], seg[slots + 1] - seg[slots]
        assert np.array_equal(got[:, 0:2].copy().view(np.int64).ravel(), sp[name])
        assert np.array_equal(got[:, 2], slots) and np.array_equal(got[:, 3], lens)
        for j in range(8):
            has = (lens <= fs.FS_SHORT_SEGMENT) & (lens > j)
            assert np.array_equal(got[has, 4 + j], want0["perm"][seg[slots[has]] + j])


@pytest.mark.parametrize("n0,n1,rows,ahead", [
    (1, 1, 1, False), (63, 65, 300, False), (1023, 1025, 500, False), (1025, 1023, 5000, True),
    (2048, 4097, 100_000, False), (8192, 8192, 300_000, False), (8193, 8192, 300_000, False), (8192, 40, 60, False),
    (40, 8192, 40_000_000, False), (16384, 16384, 64_000_000, True), (16384, 100, 1_000_000, True),
    (100, 16384, 1_000_000, True), (16384, 9000, 1700, True), (16385, 16384, 50_000, True),
    (12288, 12288, 64_000_000, True), (12288, 100, 1_000_000, True), (100, 12288, 1_000_000, True),
    (12288, 9000, 1700, True), (12289, 12288, 50_000, True), (12288, 12289, 50_000, True),
    (10240, 10240, 64_000_000, True), (10240, 100, 1_000_000, True), (100, 10240, 1_000_000, True),
    (10240, 9000, 70_000, True), (10241, 10240, 70_000, True), (10240, 10241, 65_537, True), (12288, 12288, 65_536, True)])
def test_index_half_of_a_small_batch(ctx, n0, n1, rows, ahead):
    rng = np.random.default_rng(n0 * 31 + n1)
    check_index_half(ctx, zipf_ids(rng, n0, rows, a=1.1), zipf_ids(rng, n1, rows, a=1.1), rows, ahead)


@pytest.mark.parametrize("n", [9 * 113, 9 * 1365, 16380])
def test_every_row_is_long(ctx, n):
    """As many long rows as a batch can have (nine occurrences each), half of them collision rows."""
    rng = np.random.default_rng(n)
    rows = n // 9
    check_index_half(ctx, rng.permutation(np.repeat(np.arange(rows), 9)), np.arange(0, rows, 2), rows, True)


@pytest.mark.parametrize("n0,n1", [(4096, 4096), (4097, 4096), (4096, 4097), (6144, 6144), (6145, 6144), (6144, 6145)])
def test_split_without_the_dedup_around_the_sizes_where_it_changes_over(ctx, n0, n1):
    rng = np.random.default_rng(n0 + n1)
    rows = 3000
    ids, nxt = zipf_ids(rng, n0, rows, a=1.1), zipf_ids(rng, n1, rows, a=1.1)
    lay0, lay1 = fs.fs_unique_ids(ctx, dev(ids), rows), fs.fs_unique_ids(ctx, dev(nxt), rows)
    want0 = O.unique_ids(ids, rows)
    sp = O.collision_split(want0["unique"], O.unique_ids(nxt, rows)["unique"])
    cperm, cslot, _, class_pos = class_order_from_oracle(want0, sp)
    alone = fs.fs_collision_split(ctx, lay0["unique"], lay0["n_unique"], lay1["unique"], lay1["n_unique"], n0, n1)
    split = fs.fs_collision_split_classes(ctx, lay0, lay1["unique"], lay1["n_unique"], n1)
    assert fs.fs_check_async(ctx) == fs.FS_OK
    for got in (alone, split):
        assert got["counts"].cpu().numpy().tolist() == [len(sp[k]) for k in ("co", "ex", "ex_next")]
        for k in ("co", "co_slot", "ex", "ex_slot", "ex_next", "ex_next_slot"):
            assert np.array_equal(got[k].cpu().numpy()[:len(sp[k])], sp[k]), k
    assert split["class_pos"].cpu().numpy().tolist() == [int(x) for x in class_pos]
    assert np.array_equal(split["cperm"].cpu().numpy()[:class_pos[1]], cperm)
    assert np.array_equal(split["cslot"].cpu().numpy()[:class_pos[1]], cslot)


GUARD = 1 << 17                 # more than the packed sums of any layout can reach


@pytest.mark.parametrize("n", [1024, 6144, 9000])
@pytest.mark.parametrize("what", ["overlapping rows", "short of the batch", "behind the start", "stale count", "no rows"])
def test_layout_that_does_not_fit_its_batch_writes_nothing_out_of_range(n, what):
    """Segment boundaries or a count left over from another batch: reported, and nothing is written past the class
    order, whose places the class passes then do not trust (one workgroup up to 6144 IDs, the chain of launches above)."""
    ctx = fs.Context(max_ids=16384, max_dim=4)
    u = 200
    seg = np.minimum(np.arange(n + 1) * 9, n).astype(np.int32)
    count = -(-n // 9)
    if what == "overlapping rows":                           # every other row spans nearly the whole batch
        seg[:u + 1] = np.where(np.arange(u + 1) % 2 == 1, n - 24, 0)
        count = u
    elif what == "short of the batch":
        count = u if u * 9 < n else 100
    elif what == "behind the start":
        seg[0] = 3
    elif what == "stale count":
        count = n
    else:
        count = 0
    lay = {"unique": dev(np.arange(n, dtype=np.int64)), "seg_offsets": dev(seg), "perm": dev(np.arange(n, dtype=np.int32)),
           "n_unique": dev(np.array([count], dtype=np.int64)), "n": n}
    u1 = dev(np.arange(0, n, 2, dtype=np.int64))
    split = fs.alloc_split(n, n, "cuda")
    guarded = ("cperm", "cslot", "cstart", "short_rec", "co", "co_slot", "ex", "ex_slot", "ex_next", "ex_next_slot")
    size = {k: split[k].numel() for k in guarded}
    for k in guarded:
        split[k] = torch.full((size[k] + GUARD,), -7, dtype=split[k].dtype, device="cuda")
    fs.fs_collision_split_classes(ctx, lay, u1, dev(np.array([u1.numel()], dtype=np.int64)), n, out=split)
    rc = fs.fs_check_async(ctx)
    assert rc == fs.FS_ERANGE and "internal" in ctx.last_error()
    for k in guarded:
        assert bool((split[k][size[k]:] == -7).all()), k
    first, end = split["class_pos"].cpu().tolist()
    if n <= 6144:
        assert (first, end) == (0, 0)
    ctx.close()


@pytest.mark.parametrize("n", [6144, 9000, 300_000])
@pytest.mark.parametrize("what", ["row without occurrences", "rows behind the batch", "every other row empty", "behind the start"])
def test_lists_are_whole_whatever_the_layout_and_a_misfit_is_reported(n, what):
    """The lists of the split follow from the two lists of rows alone: a layout that does not fit them leaves nothing of the
    call before in them, and is reported by one workgroup and by the chain of launches alike."""
    ctx = fs.Context(max_ids=n, max_dim=4)
    u = n // 9
    seg = (np.arange(n + 1, dtype=np.int64) * 9).clip(max=n)
    seg[u:] = n
    if what == "row without occurrences":
        seg[u // 2] = seg[u // 2 + 1]
    elif what == "rows behind the batch":
        seg[u - 40:u + 1] = n + 9 * np.arange(41)
    elif what == "every other row empty":
        seg[1:u:2] = seg[2:u + 1:2][:len(seg[1:u:2])]
    else:
        seg[0] = 3
    lay = {"unique": dev(np.arange(n, dtype=np.int64)), "seg_offsets": dev(seg.astype(np.int32)),
           "perm": dev(np.arange(n, dtype=np.int32)), "n_unique": dev(np.array([u], dtype=np.int64)), "n": n}
    u1 = np.arange(0, n, 3, dtype=np.int64)
    split = fs.alloc_split(n, n, "cuda")
    for k in ("co", "co_slot", "ex", "ex_slot", "ex_next", "ex_next_slot"):
        split[k].fill_(-7)
    fs.fs_collision_split_classes(ctx, lay, dev(u1), dev(np.array([u1.size], dtype=np.int64)), n, out=split)
    assert fs.fs_check_async(ctx) == fs.FS_ERANGE and "internal" in ctx.last_error()
    mine = np.arange(u)
    want = {"co": mine[mine % 3 == 0], "ex": mine[mine % 3 != 0], "ex_next": u1[u1 >= u]}
    assert split["counts"].cpu().tolist() == [want[k].size for k in ("co", "ex", "ex_next")]
    for k, rows in want.items():
        got = split[k].cpu().numpy()
        assert np.array_equal(got[:rows.size], rows) and (got[rows.size:] == -7).all(), k
        slots = split[k + "_slot"].cpu().numpy()[:rows.size]
        assert np.array_equal(slots, rows if k != "ex_next" else rows // 3), k
    ctx.close()
