"""The self-contained step of a small batch (index half and update in one launch) against the same step with its index half
done ahead (the update in a launch of its own): the same bits in everything, for every width of a row, where the size of
the one workgroup changes, with hot rows and without, the two batches of different sizes; and launches counted."""
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
    ctx.close()


@pytest.mark.parametrize("n,launches", [(1, 2), (8192, 2), (8193, 7)])
def test_launches_of_a_step(n, launches):
    """Two up to 8192 IDs of either batch; beyond, update, lookup and five of the index half."""
    ctx = fs.Context(max_ids=n, max_dim=64)
    args, *keep = make(ctx, np.random.default_rng(1), 3_000_000, 64, "f32", n, n, 1.1)
    assert kernels_captured(lambda s: fs.fs_prioritized_step(ctx, args, stream=s)) == launches
    ctx.close()
