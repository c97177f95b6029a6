"""Dedup by ranges at the sizes where the number of ranges, or who finds their cuts, changes; and jobs that share their
launches on either side of it."""
import numpy as np
import pytest

from test_gpu_bucket_dedup import check, check_chain, ctx, zipf_ids  # noqa: F401

import torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [24_576, 24_577, 49_152, 49_153, 98_304, 98_305, 196_608, 196_609, 393_216, 393_217])
@pytest.mark.parametrize("rows,a", [(2_000_000, 1.05), (300_000, 1.6)])
def test_sizes_where_the_cuts_change(ctx, n, rows, a):  # noqa: F811
    check(ctx, zipf_ids(np.random.default_rng(n), n, rows, a=a), rows, inverse=n % 2 == 0)


@pytest.mark.parametrize("sizes", [(49_152, 12_300, 30_000), (49_152, 49_153), (12_400, 400_000)])
def test_chains_on_either_side(sizes):
    check_chain(sizes, [400_000] * len(sizes))
