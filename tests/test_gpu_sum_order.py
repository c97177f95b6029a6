"""Sums of gradients of very different size: the self-contained step and the class passes add in fp64 in different fixed
orders, so their sums may differ by what fp64 addition leaves, and each of them gives the same bits on every run."""
import math

import numpy as np
import pytest
import torch

import paper_2604_24073_amd as fs
from helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [300, 3000, 60_000, 110_000])    # one chunk; chunks of 16, 32 and 64 positions
def test_sums_of_a_wide_range_stay_within_the_error_of_fp64_addition(n):
    rng = np.random.default_rng(n)
    rows, dim = 50, 4
    ids = np.where(rng.random(n) < 0.6, 7, rng.integers(0, rows, n)).astype(np.int64)
    grads = (rng.standard_normal((n, dim)) * 10.0 ** rng.integers(-3, 13, (n, dim))).astype(np.float32)
    ctx = fs.Context(max_ids=n, max_dim=dim)
    d_grads, d_ids = dev(grads), dev(ids)
    lay = fs.fs_unique_ids(ctx, d_ids, rows)
    split = fs.fs_collision_split_classes(ctx, lay, None, None, 0)
    u, seg, perm = (lay[k].cpu().numpy() for k in ("unique", "seg_offsets", "perm"))
    n_u = int(lay["n_unique"].item())

    def step():
        table, state = torch.zeros((rows, dim), device="cuda"), torch.zeros(rows, device="cuda")
        reduced = torch.zeros((n, dim), device="cuda")
        args = fs.make_step_args(table, state, 0.01, 1e-8, lay, d_grads, None, None, None, fs.alloc_split(n, 1, "cuda"),
                                 reduced, None)
        fs.fs_prioritized_step(ctx, args)
        assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
        return reduced[:n_u].cpu().numpy(), table.cpu().numpy(), state.cpu().numpy()

    def passes():
        table, state = torch.zeros((rows, dim), device="cuda"), torch.zeros(rows, device="cuda")
        reduced = torch.zeros((n, dim), device="cuda")
        for cls in (0, 1):
            fs.fs_reduce_update_class(ctx, cls, table, state, 0.01, 1e-8, d_grads, lay, split, reduced=reduced)
        assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
        return reduced[:n_u].cpu().numpy(), table.cpu().numpy(), state.cpu().numpy()

    for call in (step, passes):
        first, again = call(), call()
        for x, y in zip(first, again):
            assert x.tobytes() == y.tobytes(), call.__name__
        for k in range(n_u):
            g = grads[perm[seg[k]:seg[k + 1]]].astype(np.float64)
            for c in range(dim):
                exact = math.fsum(g[:, c])
                # (len - 1) additions in any order, each off by half an ulp of at most sum|g|; one rounding to fp32
                adding = (len(g) - 1) * 2.0 ** -53 * np.abs(g[:, c]).sum()
                bound = adding + 2.0 ** -24 * (abs(exact) + adding)
                assert abs(float(first[0][k, c]) - exact) <= bound, (call.__name__, int(u[k]), c)
    ctx.close()
