"""The partitioners in every form of their sort (ranges of lengths that deal on the way, radix passes, one workgroup),
with lengths that many samples share, ranges beyond LDS and more ranks than samples: the oracle's partition."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2604_24073_amd as fs
from helpers import dev
from test_gpu_bucket_dedup import sample_places

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ranks", [1, 2, 7, 64, 10_001, 300_000])
@pytest.mark.parametrize("B,hi,what", [
    (8_193, 5000, "spread"), (20_000, 8192, "spread"), (20_000, 8192, "shared"), (100_000, 1 << 20, "unsampled"),
    (16_384, 600, "unsampled"), (20_000, 400, "spread"), (8_192, 5000, "spread"), (400_000, 2000, "shared")])
def test_partitions(B, hi, what, n_ranks):
    rng = np.random.default_rng(B + n_ranks)
    lengths = rng.integers(0, hi + 1, B)
    if what == "shared":                          # half the samples have one of three lengths
        lengths[rng.random(B) < 0.5] = rng.choice([0, 17, hi], int(B))[0]
        lengths[rng.random(B) < 0.2] = hi // 2
    if what == "unsampled":                       # the sample sees three lengths only: one range takes all others
        lengths[sample_places(B)] = rng.integers(0, 3, len(sample_places(B)))
    ctx = fs.Context(max_ids=B, max_dim=8)
    got_s, got_r = fs.fs_partition_fbs(ctx, dev(lengths), hi, n_ranks)
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    want_s, want_r = O.partition_fbs(lengths, n_ranks)
    assert np.array_equal(got_r.cpu().numpy(), want_r) and np.array_equal(got_s.cpu().numpy(), want_s)
    weights = (np.arange(hi + 1) * 3 + 1).astype(np.int64)
    got_s, got_r = fs.fs_partition_vbs(ctx, dev(lengths), dev(weights), n_ranks)
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    want_s, want_r = O.partition_vbs(lengths, weights, n_ranks)
    assert np.array_equal(got_r.cpu().numpy(), want_r) and np.array_equal(got_s.cpu().numpy(), want_s)
    ctx.close()
