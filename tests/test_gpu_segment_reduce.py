"""The segment reduce as an operation of its own, on contexts that are just large enough, at the sizes where its chunks
change and for every width of a row; bit for bit (the gradients are multiples of 1/16, so every order of addition in fp64 is
exact), and again right behind itself, with and without the inverse map."""
import numpy as np
import pytest
import torch

import paper_2604_24073_amd as fs
from helpers import dev
from test_gpu_parity import zipf_ids

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rows,dim", [
    (1, 10, 4), (9, 1, 8), (63, 1, 64), (64, 3, 128), (65, 3, 256), (1000, 1, 20), (16_384, 40, 36), (65_535, 5, 4), (65_536, 5, 4),
    (65_535, 30_000, 16), (65_536, 30_000, 32), (131_071, 9, 12), (131_072, 9, 12), (131_071, 50_000, 64),
    (131_072, 50_000, 128), (200_001, 2, 8), (300_000, 100_000, 24), (90_000, 3_000_000, 144), (90_000, 900, 256)])
def test_sums(n, rows, dim):
    rng = np.random.default_rng(n + dim)
    ids = dev(zipf_ids(rng, n, rows, a=1.1))
    ctx = fs.Context(max_ids=n, max_dim=dim)
    lay = fs.fs_unique_ids(ctx, ids, rows)
    u = int(lay["n_unique"].item())
    grads = torch.randint(-64, 65, (n, dim), device="cuda", generator=torch.Generator("cuda").manual_seed(n)).float() / 16
    want = torch.zeros((u, dim), dtype=torch.float64).index_add_(0, lay["inverse"].cpu().long(), grads.cpu().double()).float()
    for inverse in (None, lay["inverse"], None):
        out = torch.full((n, dim), float("nan"), device="cuda")
        fs.fs_segment_reduce_grads(ctx, grads, lay["perm"], lay["seg_offsets"], lay["n_unique"], out=out, inverse=inverse)
        assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
        assert torch.equal(out[:u].cpu(), want) and bool(out[u:].isnan().all())
    ctx.close()


@pytest.mark.parametrize("special", [float("inf"), float("-inf"), float("nan")])
def test_special_values_stay_in_their_rows(special):
    rng = np.random.default_rng(3)
    n, rows, dim = 5000, 40, 64
    ids = zipf_ids(rng, n, rows, a=1.1)
    ctx = fs.Context(max_ids=n, max_dim=dim)
    lay = fs.fs_unique_ids(ctx, dev(ids), rows)
    u = int(lay["n_unique"].item())
    grads = torch.ones((n, dim), device="cuda")
    hit = int(ids[1234])
    grads[1234, 5] = special
    out = fs.fs_segment_reduce_grads(ctx, grads, lay["perm"], lay["seg_offsets"], lay["n_unique"])
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    bad = ~torch.isfinite(out[:u])
    slot = int((lay["unique"][:u] == hit).nonzero()[0])
    assert bad.sum() == 1 and bool(bad[slot, 5])
    ctx.close()


@pytest.mark.parametrize("n", [60_000, 200_000])
@pytest.mark.parametrize("calls", [1, 3, 1200])
def test_right_behind_a_call_whose_layout_does_not_fit(n, calls):
    """A call that leaves early where its layout makes no sense has counted some pieces of a cut segment in and others not:
    the next one on the context adds its own up all the same, with nothing asked in between, however often that happens."""
    dim = 8
    ctx = fs.Context(max_ids=n, max_dim=dim)
    lay = fs.fs_unique_ids(ctx, torch.arange(n, device="cuda", dtype=torch.int64) // (n // 3), 10)
    u = int(lay["n_unique"].item())
    grads = torch.randint(-64, 65, (n, dim), device="cuda", generator=torch.Generator("cuda").manual_seed(n)).float() / 16
    want = torch.zeros((u, dim), dtype=torch.float64).index_add_(0, lay["inverse"].cpu().long(), grads.cpu().double()).float()
    bad = lay["perm"].clone()
    bad[n // 2] = n                                  # one chunk in the middle of a long segment does not take part
    out = torch.empty((n, dim), device="cuda")
    for _ in range(calls):
        fs.fs_segment_reduce_grads(ctx, grads, bad, lay["seg_offsets"], lay["n_unique"], out=out)
    fs.fs_segment_reduce_grads(ctx, grads, lay["perm"], lay["seg_offsets"], lay["n_unique"], out=out)
    assert torch.equal(out[:u].cpu(), want)
    assert fs.fs_check_async(ctx) == fs.FS_ERANGE and "internal" in ctx.last_error()
    ctx.close()


def test_replayed_behind_a_call_whose_layout_does_not_fit():
    """The same with both calls recorded: eager and recorded calls between each other."""
    n, dim = 100_000, 8
    ctx = fs.Context(max_ids=n, max_dim=dim)
    lay = fs.fs_unique_ids(ctx, torch.arange(n, device="cuda", dtype=torch.int64) // (n // 3), 10)
    u = int(lay["n_unique"].item())
    grads = torch.randint(-64, 65, (n, dim), device="cuda", generator=torch.Generator("cuda").manual_seed(n)).float() / 16
    want = torch.zeros((u, dim), dtype=torch.float64).index_add_(0, lay["inverse"].cpu().long(), grads.cpu().double()).float()
    bad = lay["perm"].clone()
    bad[n // 2] = n
    out = torch.empty((n, dim), device="cuda")
    good = lambda: fs.fs_segment_reduce_grads(ctx, grads, lay["perm"], lay["seg_offsets"], lay["n_unique"], out=out)  # noqa: E731
    misfit = lambda: fs.fs_segment_reduce_grads(ctx, grads, bad, lay["seg_offsets"], lay["n_unique"], out=out)  # noqa: E731
    graphs = []
    torch.cuda.synchronize()
    for call in (good, misfit):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            call()
        graphs.append(g.replay)
    for first, then in ((misfit, graphs[0]), (graphs[1], good), (graphs[1], graphs[0]), (good, graphs[0]), (graphs[0], good)):
        for _ in range(2):
            first()
            then()
            assert torch.equal(out[:u].cpu(), want)
    fs.fs_check_async(ctx)
    ctx.close()
