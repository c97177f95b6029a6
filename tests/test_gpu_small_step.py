"""The self-contained step of a small batch (index half and update in one launch) against the same step with its index half
done ahead (the update in a launch of its own): the same bits in everything, for every width of a row, where the size of
the one workgroup changes, with hot rows and without, the two batches of different sizes; buffers that coincide; and
launches counted."""
import numpy as np
import pytest
import torch

import paper_2604_24073_amd as fs
from helpers import dev, table_to_dev
from test_gpu_one_stream import kernels_captured
from test_gpu_parity import rand_table, zipf_ids

pytestmark = pytest.mark.gpu


def make(ctx, rng, rows, dim, dtype, n_t, n_t1, a, reduced=False):
    ids = [dev(zipf_ids(rng, n, rows, a=a)) for n in (n_t, n_t1)]
    table, state = table_to_dev(rand_table(rng, rows, dim, dtype)), torch.zeros(rows, device="cuda")
    lay0, lay1 = fs.fs_unique_ids(ctx, ids[0], rows), fs.alloc_layout(n_t1, "cuda")
    split = fs.alloc_split(n_t, n_t1, "cuda")
    grads = dev(rng.standard_normal((n_t, dim)).astype(np.float32))
    emb = torch.zeros((n_t1, dim), dtype=table.dtype, device="cuda")
    red = torch.zeros((n_t, dim), device="cuda") if reduced else None
    args = fs.make_step_args(table, state, 0.01, 1e-8, lay0, grads, ids[1], None, lay1, split, red, emb)
    return args, {"table": table, "state": state, "emb": emb, "reduced": red}, lay0, lay1, split, (ids, grads)


SIZES = [(1, 1), (9, 300), (17, 16), (1000, 1024), (1025, 3), (3, 2049), (2048, 2000), (4097, 4096), (8192, 8191)]


@pytest.mark.parametrize("n_t,n_t1", SIZES)
@pytest.mark.parametrize("dim,dtype", [(4, "f32"), (8, "bf16"), (16, "f32"), (24, "bf16"), (64, "f32"), (100, "f32"), (128, "bf16"), (256, "f32")])
def test_same_bits_as_in_two_launches(n_t, n_t1, dim, dtype):
    rows = 700 if (n_t + dim) % 2 else 60_000
    a = 1.6 if n_t > 4000 else 1.1
    ctx = fs.Context(max_ids=max(n_t, n_t1), max_dim=dim)
    one = make(ctx, np.random.default_rng(n_t), rows, dim, dtype, n_t, n_t1, a, reduced=dim % 3 == 1)
    two = make(ctx, np.random.default_rng(n_t), rows, dim, dtype, n_t, n_t1, a, reduced=dim % 3 == 1)
    for _ in range(2):                                # the second time on counters and buffers that the first one left
        fs.fs_prioritized_step(ctx, one[0])
        assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
        fs.fs_step_forward_ahead(ctx, two[0])
        fs.fs_prioritized_step(ctx, two[0])
        assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
        for k, x in one[1].items():
            assert x is None or torch.equal(x.view(torch.uint8), two[1][k].view(torch.uint8)), k
        u = int(one[3]["n_unique"].item())
        assert u == int(two[3]["n_unique"].item())
        for k, m in (("unique", u), ("seg_offsets", u + 1), ("perm", n_t1), ("inverse", n_t1)):
            assert torch.equal(one[3][k][:m], two[3][k][:m]), k
        counts = one[4]["counts"].cpu().numpy()
        assert np.array_equal(counts, two[4]["counts"].cpu().numpy())
        for k, m in (("co", counts[0]), ("co_slot", counts[0]), ("ex", counts[1]), ("ex_slot", counts[1]), ("ex_next", counts[2]),
                     ("ex_next_slot", counts[2]), ("class_pos", 2)):
            assert torch.equal(one[4][k][:m], two[4][k][:m]), k
        for x, y in zip(class_order(one[4], n_t), class_order(two[4], n_t)):
            assert np.array_equal(x, y)
    ctx.close()


def class_order(split, n_t):
    """What is specified of the class order: the positions, the starts of the rows in it, the records (heads, and the
    occurrences of the rows with few)."""
    host = {k: split[k].cpu().numpy() for k in ("cperm", "cslot", "cstart", "class_pos", "counts", "short_rec")}
    end = host["class_pos"][1]
    cslot = host["cslot"][:end]
    rec = host["short_rec"].reshape(2, n_t, 12)
    rec = np.concatenate([rec[0, :host["counts"][0]], rec[1, :host["counts"][1]]])
    listed = (np.arange(8) < rec[:, 3:4]) & (rec[:, 3:4] <= fs.FS_SHORT_SEGMENT)
    return host["cperm"][:end], cslot, host["cstart"][np.unique(cslot)], rec[:, :4], np.where(listed, rec[:, 4:], -1)


def lay_over(what, over, args, kept, lay1, split, n_t, n_t1):
    """The output `what` of the index half in the memory of `over`, which the update or the lookup uses."""
    (ids, grads), offsets = kept[:2], kept[2]
    room = {"values": ids[1], "grads": grads, "offsets": offsets}[over].view(-1).view(torch.uint8)
    if what == "perm":                                # in the second half of the IDs
        lay1["perm"] = room[4 * n_t1:8 * n_t1].view(torch.int32)
        args.perm_t1 = lay1["perm"].data_ptr()
    elif what in ("unique", "sorted_ids"):
        lay1[what] = room[:8 * n_t1].view(torch.int64)
        setattr(args, "u_t1" if what == "unique" else "sorted_ids_t1", lay1[what].data_ptr())
    else:
        split[what] = room[:split[what].numel() * split[what].element_size()].view(split[what].dtype)
        setattr(args, "counts_dev" if what == "counts" else what, split[what].data_ptr())


@pytest.mark.parametrize("what,over", [("unique", "values"), ("sorted_ids", "values"), ("perm", "values"), ("ex", "values"),
                                       ("counts", "offsets"), ("short_rec", "grads"), ("ex_next", "grads")])
@pytest.mark.parametrize("n", [600, 3000, 8192])
def test_index_half_written_over_what_the_row_work_reads(what, over, n):
    """The index half of a call on one stream comes behind its row work, so that what it writes may lie where the update or
    the lookup has read: three launches then, and the results of a call whose buffers are all apart."""
    rows, dim = 50_000, 64
    ctx = fs.Context(max_ids=n, max_dim=dim)
    runs = []
    for coincide in (False, True):
        args, out, lay0, lay1, split, (ids, grads) = make(ctx, np.random.default_rng(n), rows, dim, "f32", n, n, 1.2)
        offsets = torch.arange(0, n + 1, n // 3, dtype=torch.int64, device="cuda")
        offsets[-1] = n
        args.offsets_t1, args.batch_t1 = offsets.data_ptr(), offsets.numel() - 1
        if what == "sorted_ids":
            lay1["sorted_ids"] = torch.empty(n, dtype=torch.int64, device="cuda")
            args.sorted_ids_t1 = lay1["sorted_ids"].data_ptr()
        if coincide:
            lay_over(what, over, args, (ids, grads, offsets), lay1, split, n, n)
        assert kernels_captured(lambda s: fs.fs_prioritized_step(ctx, args, stream=s)) == (3 if coincide else 2)
        fs.fs_prioritized_step(ctx, args)
        assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
        u = int(lay1["n_unique"].item())
        counts = split["counts"].cpu().numpy()
        out = {k: v.cpu() for k, v in out.items() if v is not None}
        out.update({k: lay1[k][:m].cpu() for k, m in (("unique", u), ("seg_offsets", u + 1), ("perm", n), ("sorted_ids", n)) if k in lay1})
        out.update({k: split[k][:m].cpu() for k, m in (("co", counts[0]), ("ex", counts[1]), ("ex_next", counts[2]))})
        out.update({str(i): torch.from_numpy(x) for i, x in enumerate(class_order(split, n))})
        runs.append(out)
    for k in runs[0]:
        assert torch.equal(runs[0][k], runs[1][k]), k
    ctx.close()


@pytest.mark.parametrize("n,launches", [(1, 2), (8192, 2), (8193, 7)])
def test_launches_of_a_step(n, launches):
    """Two up to 8192 IDs of either batch; beyond, update, lookup and five of the index half."""
    ctx = fs.Context(max_ids=n, max_dim=64)
    args, *keep = make(ctx, np.random.default_rng(1), 3_000_000, 64, "f32", n, n, 1.1)
    assert kernels_captured(lambda s: fs.fs_prioritized_step(ctx, args, stream=s)) == launches
    ctx.close()
