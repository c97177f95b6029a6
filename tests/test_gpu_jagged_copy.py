"""The copy behind the jagged shuffles at the sizes where it changes: ends of tiles and of groups of sixteen bytes, values
and outputs that lie at any multiple of the piece, inputs of less than sixteen bytes, more samples than a tile's window has
places for, more tiles than are written down ahead, samples taken twice; permutes side by side on streams of their own.  Byte
work: bit-exact."""
import numpy as np
import pytest
import torch

import paper_2604_24073_amd as fs

pytestmark = pytest.mark.gpu


def expected(values, offsets, order):
    parts = [values[offsets[p]:offsets[p + 1]] for p in order]
    lens = [len(p) for p in parts]
    return np.concatenate(parts) if parts else values[:0], np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)


def shifted(a, shift):
    """`a` on the GPU, `shift` 4-byte words behind an aligned address."""
    flat = torch.from_numpy(a.reshape(-1).view(np.int32))
    room = torch.zeros(flat.numel() + shift, dtype=torch.int32, device="cuda")
    room[shift:] = flat.cuda()
    return room[shift:]


def permute(ctx, values, offsets, order, words, shift_in=0, shift_out=0):
    """fs_jagged_indexed_permute on elements of `words` 32-bit words, through the C entry point (any address goes)."""
    want, want_offsets = expected(values, offsets, order)
    src, n = shifted(values, shift_in), len(want)
    out = torch.full((n * words + shift_out + 8,), -7, dtype=torch.int32, device="cuda")
    o = torch.from_numpy(offsets).cuda()
    sel = torch.from_numpy(np.asarray(order, np.int32)).cuda()
    out_offsets = torch.full((len(order) + 1,), -7, dtype=torch.int64, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    rc = fs.load_library().fs_jagged_indexed_permute(
        ctx.handle, src.data_ptr(), len(values), 4 * words, o.data_ptr(), len(offsets) - 1, sel.data_ptr(), len(order),
        out.data_ptr() + 4 * shift_out, n, out_offsets.data_ptr(), stream)
    assert rc == fs.FS_OK and fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    got = out.cpu().numpy()
    assert np.array_equal(out_offsets.cpu().numpy(), want_offsets)
    assert np.array_equal(got[shift_out:shift_out + n * words], want.reshape(-1).view(np.int32))
    assert (got[:shift_out] == -7).all() and (got[shift_out + n * words:] == -7).all()


def jagged(rng, lens, words):
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    return rng.integers(-2**31, 2**31 - 1, size=(int(offsets[-1]), words)).astype(np.int32), offsets


# 4-, 8- and 16-byte pieces, several to an element among them; samples of 0 to 2, 0 to 40 and about 700 pieces
@pytest.mark.parametrize("words", [1, 2, 3, 4, 6, 12])
@pytest.mark.parametrize("longest", [2, 40, 1500])
@pytest.mark.parametrize("samples", [700, 4096, 4097])
def test_tiles_and_groups(words, longest, samples):
    rng = np.random.default_rng(words * 100 + longest + samples)
    if samples > 700 and longest > 40:
        longest = 40
    values, offsets = jagged(rng, rng.integers(0, longest + 1, size=samples), words)
    ctx = fs.Context(max_ids=8192, max_dim=8)
    piece = 4 if words % 4 == 0 else 2 if words % 2 == 0 else 1           # words of a piece
    for shift_in, shift_out in ((0, 0), (piece, 0), (0, piece), (3 * piece, piece)):
        permute(ctx, values, offsets, rng.permutation(samples), words, shift_in, shift_out)
    ctx.close()


@pytest.mark.parametrize("words", [1, 2, 4])
@pytest.mark.parametrize("total", [1, 2, 3, 4, 5, 2047, 2048, 2049, 4095, 4096, 4097, 8191, 8192, 8193])
def test_outputs_of_about_a_tile_and_of_less_than_a_group(words, total):
    rng = np.random.default_rng(total)
    ctx = fs.Context(max_ids=64, max_dim=8)
    for lens in ([total], [0, total, 0], [1] * min(total, 5) + [max(total - 5, 0)], [max(total - 3, 0), 0, min(total, 3)]):
        values, offsets = jagged(rng, lens, words)
        permute(ctx, values, offsets, np.arange(len(lens))[::-1], words)
        permute(ctx, values, offsets, rng.integers(0, len(lens), size=2 * len(lens)), words)      # samples twice, or not at all
    ctx.close()


@pytest.mark.parametrize("words", [1, 2, 4])
@pytest.mark.parametrize("samples", [4000, 20_000])
def test_more_samples_in_a_tile_than_its_window_has_places_for(words, samples):
    """One element in five samples, and (16-byte pieces in tiles of 8192) one element a sample."""
    rng = np.random.default_rng(samples + words)
    values, offsets = jagged(rng, (rng.random(samples) < 0.2).astype(np.int64), words)
    ctx = fs.Context(max_ids=samples, max_dim=8)
    permute(ctx, values, offsets, rng.permutation(samples), words)
    values, offsets = jagged(rng, np.concatenate([np.ones(samples - 1, np.int64), [3 * 2**20 if words == 4 else 5]]), words)
    permute(ctx, values, offsets, np.arange(samples), words)
    ctx.close()


@pytest.mark.parametrize("words", [1, 2, 4])
def test_more_tiles_than_are_written_down_ahead(words):
    """Eight samples on a context for eight IDs: sixteen tiles are written down, the output has more."""
    rng = np.random.default_rng(words)
    values, offsets = jagged(rng, [5000, 0, 7000, 4096, 1, 9000, 6000, 4095], words)
    ctx = fs.Context(max_ids=8, max_dim=8)
    permute(ctx, values, offsets, [3, 1, 0, 7, 5, 6, 2, 4], words)
    permute(ctx, values, offsets, [0, 1, 4, 4, 1, 7, 0, 0], words)
    ctx.close()


@pytest.mark.parametrize("pieces", [3 * 2**20 - 1, 3 * 2**20, 3 * 2**20 + 5])
def test_sixteen_byte_pieces_around_the_size_where_the_tile_changes(pieces):
    rng = np.random.default_rng(pieces)
    lens = rng.multinomial(pieces, np.full(900, 1 / 900))
    values, offsets = jagged(rng, lens, 4)
    ctx = fs.Context(max_ids=4096, max_dim=8)
    permute(ctx, values, offsets, rng.permutation(900), 4)
    ctx.close()


@pytest.mark.parametrize("words", [1, 2, 4])
@pytest.mark.parametrize("samples", [40, 4096, 4097, 8192])
def test_permutes_of_a_list_on_two_streams_of_one_context(words, samples):
    """Up to 8192 samples of a caller's list nothing of the context is used: calls on two streams, one of them late, do not
    get in each other's way."""
    rng = np.random.default_rng(samples + words)
    ctx = fs.Context(max_ids=8192, max_dim=8)
    calls = []
    for k in range(24):
        values, offsets = jagged(rng, rng.integers(0, 2 * 40_000 // samples + 2, size=samples), words)
        order = rng.permutation(samples).astype(np.int32)
        calls.append((values, offsets, order, torch.from_numpy(values).cuda(), torch.from_numpy(offsets).cuda(),
                      torch.from_numpy(order).cuda()))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    slow = torch.randn(1024, 1024, device="cuda")
    torch.cuda.synchronize()
    got = []
    for k, (values, _, _, v, o, sel) in enumerate(calls):
        with torch.cuda.stream(streams[k % 2]):
            if k % 3 == 0:
                slow @ slow
            got.append(fs.fs_jagged_indexed_permute(ctx, v, o, sel, len(values)))
    torch.cuda.synchronize()
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    for (values, offsets, order, *_), (out, out_offsets) in zip(calls, got):
        want, want_offsets = expected(values, offsets, order)
        assert np.array_equal(out_offsets.cpu().numpy(), want_offsets)
        assert np.array_equal(out.cpu().numpy().reshape(want.shape), want)
    ctx.close()


@pytest.mark.parametrize("words", [1, 2, 4])
@pytest.mark.parametrize("tiles", [63, 64, 65, 66, 700])
@pytest.mark.parametrize("segments", [1, 40, 5000])
def test_samples_of_many_tiles(words, tiles, segments):
    """Samples with about as many tiles as one lane writes down, and with many more, among short ones: one in the one
    workgroup, one each in two neighbouring lanes, one behind the others; two launches for the offsets from 4097 samples on."""
    rng = np.random.default_rng(tiles)
    lens = rng.integers(0, 4, size=segments)
    lens[rng.permutation(segments)[:3]] = 2048 * tiles + rng.integers(-3, 4, size=min(3, segments))
    lens[segments // 2:segments // 2 + 2] = 2048 * tiles + 1
    lens[-1] = 2048 * tiles
    values, offsets = jagged(rng, lens, words)
    ctx = fs.Context(max_ids=8192, max_dim=8)
    v, o = torch.from_numpy(values).cuda(), torch.from_numpy(offsets).cuda()
    F = 4 if segments % 4 == 0 else 1
    out, out_offsets = fs.fs_jagged_keyed_transpose(ctx, v, o, F, segments // F)
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    want, want_offsets = expected(values, offsets, np.arange(segments).reshape(F, -1).T.reshape(-1))
    assert np.array_equal(out_offsets.cpu().numpy(), want_offsets)
    assert np.array_equal(out.cpu().numpy().reshape(want.shape), want)
    ctx.close()
