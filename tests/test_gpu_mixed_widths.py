"""Tables of different row widths in shared launches: every table's passes and lookup give the bits of a call of its own,
on one stream and on two, and the widths really share a launch."""
import numpy as np
import pytest
import torch

import paper_2604_24073_amd as fs
from helpers import dev, table_to_dev
from test_gpu_one_stream import kernels_captured
from test_gpu_parity import rand_table, zipf_ids

pytestmark = pytest.mark.gpu

# lanes of a row in the passes 2, 8, 8, 16, 16, 32, 64, 64 (narrow rows have launches of their own), in the lookups of
# bf16 rows half of that; edges of the widths among them
DIMS = (8, 24, 32, 40, 64, 96, 136, 256)


def prepare(ctx, rng, dims, dtype, n, two_part):
    args, keep = [], []
    for k, dim in enumerate(dims):
        rows = 3000 + 17 * k
        ids = [dev(zipf_ids(rng, n - 31 * k - b, rows, a=1.1)) for b in range(2)]
        table, state = table_to_dev(rand_table(rng, rows, dim, dtype)), torch.zeros(rows, device="cuda")
        lay0, lay1 = fs.fs_unique_ids(ctx, ids[0], rows), fs.alloc_layout(ids[1].numel(), "cuda", sorted_ids=not two_part)
        split = fs.alloc_split(ids[0].numel(), ids[1].numel(), "cuda")
        grads = dev(rng.standard_normal((ids[0].numel(), dim)).astype(np.float32))
        emb = torch.zeros((ids[1].numel(), dim), dtype=table.dtype, device="cuda")
        args.append(fs.make_step_args(table, state, 0.01, 1e-8, lay0, grads, ids[1], None, lay1, split, None, emb))
        keep.append((table, state, emb, ids, lay0, lay1, split, grads))
    for a in args:
        fs.fs_step_forward(ctx, a)
    return args, keep


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,two_part", [(700, False), (700, True), (40_000, False), (40_000, True)])
def test_a_table_does_not_notice_the_widths_beside_it(dtype, n, two_part):
    step = fs.fs_prioritized_step_two_part_multi if two_part else fs.fs_prioritized_step_pipelined_multi
    ctx = fs.Context(max_ids=n, max_dim=256)
    together, got = prepare(ctx, np.random.default_rng(5), DIMS, dtype, n, two_part)
    step(ctx, fs.step_args_array(together), None)
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    alone, want = prepare(ctx, np.random.default_rng(5), DIMS, dtype, n, two_part)
    for a in alone:
        step(ctx, fs.step_args_array([a]), None)
        fs.fs_two_part_forget(ctx)
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    view = torch.int32 if dtype == "f32" else torch.int16
    for dim, g, w in zip(DIMS, got, want):
        assert torch.equal(g[0].view(view), w[0].view(view)), dim
        assert torch.equal(g[1], w[1]) and torch.equal(g[2].view(view), w[2].view(view)), dim
    ctx.close()


@pytest.mark.parametrize("dims,launches", [((24, 64, 200, 256), 2), ((24, 64, 128, 200, 256), 3), ((4, 64, 128, 256), 3)])
def test_widths_share_launches(dims, launches):
    """On one stream: the passes of four tables a launch (rows of up to 16 columns a launch of their own), one lookup."""
    ctx = fs.Context(max_ids=4000, max_dim=256)
    args, keep = prepare(ctx, np.random.default_rng(6), dims, "f32", 4000, False)
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    record = fs.step_args_array(args)
    assert kernels_captured(lambda s: fs.fs_prioritized_step_pipelined_multi(ctx, record, None, stream=s)) == launches
    ctx.close()
