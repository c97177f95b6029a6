"""Dedup by ranges of keys: sizes around tiles (2048 IDs) and where the number of ranges changes, batches of one row,
of a few, of rows popular enough for ranges of their own, IDs at both ends of the table, a batch whose sample misses
where its IDs are (a range that does not fit LDS), batches of several jobs.  Whole numbers: equal to the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2604_24073_amd as fs
from helpers import dev
from test_gpu_parity import zipf_ids

pytestmark = pytest.mark.gpu

MAX_IDS = (1 << 20) + 5


@pytest.fixture(scope="module")
def ctx():
    c = fs.Context(max_ids=MAX_IDS, max_dim=4)
    yield c
    c.close()


def check(ctx, ids, rows, inverse=True):
    want = O.unique_ids(ids, rows)
    lay = fs.alloc_layout(len(ids), "cuda", inverse=inverse)
    got = fs.fs_unique_ids(ctx, dev(ids), rows, out=lay)
    assert fs.fs_check_async(ctx) == fs.FS_OK
    u = int(got["n_unique"].item())
    assert u == want["n_unique"]
    for k, m in (("unique", u), ("seg_offsets", u + 1), ("perm", len(ids))) + ((("inverse", len(ids)),) if inverse else ()):
        assert np.array_equal(got[k][:m].cpu().numpy(), want[k]), k


@pytest.mark.parametrize("n", [8193, 12287, 12288, 12289, 16384, 16385, 65535, 65537, 131073, 300_001, 393_217, 786_433, 1 << 20, (1 << 20) + 1])
@pytest.mark.parametrize("rows,a", [(3_000_000, 1.05), (50_000, 1.3)])
def test_sizes(ctx, n, rows, a):
    rng = np.random.default_rng(n)
    check(ctx, zipf_ids(rng, n, rows, a=a), rows, inverse=n % 2 == 1)


@pytest.mark.parametrize("n,rows", [(8193, 512), (8193, 513), (300_001, 500), (393_216, 1 << 18), (393_217, 1 << 18),
                                    (393_217, (1 << 18) + 1), (786_433, 600)])
def test_sizes_where_the_form_changes(ctx, n, rows):
    """One, two and three radix passes' worth of key bits, an operation of its own."""
    check(ctx, zipf_ids(np.random.default_rng(n + rows), n, rows, a=1.05), rows, inverse=n % 2 == 1)


@pytest.mark.parametrize("n", [9000, 200_000])
@pytest.mark.parametrize("what", ["one", "last", "two", "neighbours", "distinct", "descending", "periodic", "ends", "nines"])
def test_distributions(ctx, n, what):
    rng = np.random.default_rng(n + len(what))
    rows = 1 << 31
    ids = {"one": lambda: np.full(n, 42), "last": lambda: np.full(n, rows - 1), "two": lambda: rng.integers(0, 2, n) * 1000,
           "neighbours": lambda: rng.integers(0, 5, n) + rows - 5, "distinct": lambda: rng.permutation(n) * 7,
           "descending": lambda: np.arange(n)[::-1], "periodic": lambda: np.where(np.arange(n) % 64 == 0, 5, rng.integers(0, rows, n)),
           "ends": lambda: rng.choice([0, rows - 1], n), "nines": lambda: rng.permutation(np.arange(n) // 9 * 31)}[what]()
    check(ctx, ids.astype(np.int64), rows)


def sample_places(n):
    """Where the sample of a batch of n IDs is taken."""
    k = 0
    while (1 << k) < 1024 and (768 << k) < n:
        k += 1
    i = np.arange(4 << k, dtype=np.uint64)
    a, b = i * np.uint64(n) >> np.uint64(k + 2), (i + np.uint64(1)) * np.uint64(n) >> np.uint64(k + 2)
    h = i * np.uint64(0x9E3779B1) & np.uint64(0xFFFFFFFF)
    h ^= h >> np.uint64(15)
    h = h * np.uint64(0x85EBCA77) & np.uint64(0xFFFFFFFF)
    h ^= h >> np.uint64(13)
    return (a + (h * np.maximum(b - a, np.uint64(1)) >> np.uint64(32))).astype(np.int64)


@pytest.mark.parametrize("n,rows", [(16_384, 200), (16_384, 700), (30_001, 1 << 20), (100_000, 1 << 31)])
def test_a_range_beyond_lds(ctx, n, rows):
    """The sample sees the first few rows only; everything else falls into the last range."""
    rng = np.random.default_rng(n)
    ids = zipf_ids(rng, n, rows, a=1.1)
    ids[sample_places(n)] = rng.integers(0, 3, len(sample_places(n)))
    check(ctx, ids, rows)


def test_an_id_out_of_range_is_reported_and_leaves_the_other_rows_alone(ctx):
    rng = np.random.default_rng(5)
    n, rows = 20_000, 3_000
    ids = rng.integers(0, rows, n)
    bad = ids.copy()
    bad[[7, 9000, n - 1]] = [rows, 1 << 40 | 1 << 31, -1]
    got = fs.fs_unique_ids(ctx, dev(bad), rows)
    assert fs.fs_check_async(ctx) == fs.FS_ERANGE
    assert np.array_equal(np.sort(got["perm"][:n].cpu().numpy()), np.arange(n))
    check(ctx, ids, rows)


@pytest.mark.parametrize("sizes", [(20_000, 300_000), (70_000, 3, 9_000), (10_240, 5_000), (10_241, 10_240)])
def test_index_halves_of_different_sizes_in_one_chain(sizes):
    """Jobs that share their launches have ranges and tiles of their own number; what they write is the same as alone."""
    check_chain(sizes, [400_000] * len(sizes))


@pytest.mark.parametrize("sizes,rows,inverse", [
    ((400_000, 20_000), (1 << 18, 900), True),               # two passes' worth of bits, beyond one wave of ranges
    ((40_000, 4_097, 12_289), (512, 500, 2), False),         # radix, one pass
    ((4_096, 20_000, 4_097), (1 << 33, 1 << 40, 0), False),  # radix, 64-bit keys (0: table of unknown size)
    ((12_289, 4_097, 30_000), (700, 1 << 33, 400_000), True),     # one table that the ranges cannot take, two that they could
    (((1 << 20) + 1, 9_000), (400_000, 3_000), False)])           # one batch beyond them
def test_index_halves_of_every_form_in_one_chain(sizes, rows, inverse):
    check_chain(sizes, rows, inverse)


def check_chain(sizes, table_rows, inverse=True):
    rng = np.random.default_rng(sum(sizes))
    keep, args, lays = [], [], []
    c = fs.Context(max_ids=max(sizes), max_dim=4)
    for n, rows in zip(sizes, table_rows):
        most = rows if rows > 0 else 1 << 45
        ids, nxt = zipf_ids(rng, n, most, a=1.1), zipf_ids(rng, n, most, a=1.1)
        lay0, lay1 = fs.alloc_layout(n, "cuda"), fs.alloc_layout(n, "cuda", inverse=inverse, sorted_ids=True)
        split = fs.alloc_split(n, n, "cuda")
        fs.fs_unique_ids(c, dev(ids), rows, out=lay0)
        keep.append([torch.zeros((k, 4), device="cuda") for k in (8, n, n)] + [dev(nxt), split, lay0])
        a = fs.make_step_args(keep[-1][0], torch.zeros(1, device="cuda"), 0.01, 1e-8, lay0, keep[-1][1], keep[-1][3], None,
                              lay1, split, None, keep[-1][2])
        a.num_rows = rows                                     # the index half touches no table row
        args.append(a)
        lays.append((lay1, nxt, ids, split, rows))
    fs.fs_step_forward_ahead_batch(c, fs.step_args_array(args))
    assert fs.fs_check_async(c) == fs.FS_OK
    for lay, nxt, ids, split, rows in lays:
        want, sp = O.unique_ids(nxt, rows), O.collision_split(O.unique_ids(ids, rows)["unique"], O.unique_ids(nxt, rows)["unique"])
        for k in ("unique", "seg_offsets", "perm") + (("inverse",) if inverse else ()):
            assert np.array_equal(lay[k].cpu().numpy()[:len(want[k])], want[k]), k
        assert np.array_equal(lay["sorted_ids"].cpu().numpy()[:len(nxt)], np.sort(nxt))
        assert split["counts"].cpu().numpy().tolist() == [len(sp[k]) for k in ("co", "ex", "ex_next")]
    c.close()
