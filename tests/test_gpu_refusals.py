"""A step call that is refused leaves everything as it was: nothing enqueued, table and state untouched, results of
ahead-of-time calls still there for the call that is made instead."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2604_24073_amd as fs
from helpers import dev
from test_gpu_parity import zipf_ids

pytestmark = pytest.mark.gpu

ROWS, DIM = 5000, 32


class Step:
    """One iteration on buffers of its own; the lookahead layout has room for the ascending ID list."""

    def __init__(self, ctx, table, state, ids, nxt, seed=0, sorted_ids=True):
        rng = np.random.default_rng(seed)
        self.ids, self.nxt = dev(ids), dev(nxt)
        self.lay0 = fs.fs_unique_ids(ctx, self.ids, ROWS)
        self.lay1 = fs.alloc_layout(len(nxt), "cuda", sorted_ids=True)
        self.split = fs.alloc_split(len(ids), len(nxt), "cuda")
        self.grads = dev(rng.standard_normal((len(ids), DIM)).astype(np.float32))
        self.emb = torch.full((len(nxt), DIM), -3.0, device="cuda")
        self.args = self.record(table, state, sorted_ids)

    def record(self, table, state, sorted_ids):
        lay1 = dict(self.lay1) if sorted_ids else {k: v for k, v in self.lay1.items() if k != "sorted_ids"}
        return fs.make_step_args(table, state, 0.01, 1e-8, self.lay0, self.grads, self.nxt, None, lay1, self.split, None,
                                 self.emb)


def batches(n, count=3, seed=5):
    rng = np.random.default_rng(seed)
    return [zipf_ids(rng, n, ROWS, a=1.1) for _ in range(count)]


def raises(code, call, *args):
    with pytest.raises(fs.FreeScaleError) as e:
        call(*args)
    assert e.value.code == code


@pytest.mark.parametrize("n", [300, 90_000])                # index half behind the row work; on the side stream
@pytest.mark.parametrize("call", ["step", "forward", "ahead", "pipelined", "pipelined multi"])
def test_ascending_ids_of_a_batch_deduped_ahead_are_refused_before_anything_runs(n, call):
    ctx = fs.Context(max_ids=100_000, max_dim=DIM)
    torch.manual_seed(1)
    table, state = torch.randn((ROWS, DIM), device="cuda"), torch.rand(ROWS, device="cuda")
    before = (table.clone(), state.clone())
    a, b, c = batches(n)
    cur, nxt = Step(ctx, table, state, a, b, 1, sorted_ids=False), Step(ctx, table, state, b, c, 2)
    if call.startswith("pipelined"):
        fs.fs_step_forward(ctx, cur.args)
        subject = nxt
    else:
        subject = Step(ctx, table, state, a, b, 1)
    fs.fs_unique_ids_ahead(ctx, subject.nxt, ROWS, subject.lay1)
    if call == "step":
        raises(fs.FS_EINVAL, fs.fs_prioritized_step, ctx, subject.args)
    elif call == "forward":
        raises(fs.FS_EINVAL, fs.fs_step_forward, ctx, subject.args)
    elif call == "ahead":
        raises(fs.FS_EINVAL, fs.fs_step_forward_ahead, ctx, subject.args)
    elif call == "pipelined":
        raises(fs.FS_EINVAL, fs.fs_prioritized_step_pipelined, ctx, cur.args, nxt.args)
    else:
        raises(fs.FS_EINVAL, fs.fs_prioritized_step_pipelined_multi, ctx, fs.step_args_array([cur.args]),
               fs.step_args_array([nxt.args]))
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    assert torch.equal(table, before[0]) and torch.equal(state, before[1])
    assert bool((cur.emb == -3.0).all()) and bool((subject.emb == -3.0).all())
    # without the list the call goes through, once, on the dedup that was done ahead
    step = cur if call.startswith("pipelined") else subject
    subject.args = subject.record(table, state, False)
    if call == "step":
        fs.fs_prioritized_step(ctx, subject.args)
    elif call == "forward":
        fs.fs_step_forward(ctx, subject.args)
        fs.fs_prioritized_step_pipelined(ctx, subject.args, None)
    elif call == "ahead":
        fs.fs_step_forward_ahead(ctx, subject.args)
        fs.fs_prioritized_step_pipelined(ctx, subject.args, None)
    else:
        fs.fs_prioritized_step_pipelined(ctx, cur.args, subject.args)
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    want_t, want_s = before[0].clone(), before[1].clone()
    fresh = Step(ctx, want_t, want_s, a, b, 1)
    fs.fs_prioritized_step(ctx, fresh.args)
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    assert torch.equal(table, want_t) and torch.equal(state, want_s)
    assert torch.equal(step.emb, fresh.emb)
    ctx.close()


@pytest.mark.parametrize("call", ["step", "forward", "ahead", "pipelined"])
def test_batch_beyond_the_class_order_is_refused_before_anything_runs(call):
    n, dim = 7680 * 1024 + 1, 4                              # one occurrence more than the class order takes
    ctx = fs.Context(max_ids=n, max_dim=dim)
    table, state = torch.ones((ROWS, dim), device="cuda"), torch.ones(ROWS, device="cuda")
    ids = torch.arange(n, dtype=torch.int64, device="cuda") % ROWS
    lay = fs.fs_unique_ids(ctx, ids, ROWS)
    split = fs.alloc_split(n, 1, "cuda")
    args = fs.make_step_args(table, state, 0.01, 1e-8, lay, torch.ones((n, dim), device="cuda"), None, None, None, split,
                             None, None)
    if call == "step":
        raises(fs.FS_ERANGE, fs.fs_prioritized_step, ctx, args)
    elif call == "forward":
        raises(fs.FS_ERANGE, fs.fs_step_forward, ctx, args)
    elif call == "ahead":
        raises(fs.FS_ERANGE, fs.fs_step_forward_ahead, ctx, args)
    else:
        few = torch.arange(9, dtype=torch.int64, device="cuda")
        small = fs.make_step_args(table, state, 0.01, 1e-8, fs.fs_unique_ids(ctx, few, ROWS), torch.ones((9, dim), device="cuda"),
                                  None, None, None, fs.alloc_split(9, 1, "cuda"), None, None)
        fs.fs_step_forward(ctx, small)
        raises(fs.FS_ERANGE, fs.fs_prioritized_step_pipelined, ctx, small, args)
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    assert bool((table == 1.0).all()) and bool((state == 1.0).all())
    ctx.close()


def leave_a_host_error():
    """A runtime call of the caller's own that failed: the next launch check of the library finds its error."""
    assert ctypes.CDLL("libamdhip64.so").hipSetDevice(ctypes.c_int(9999)) != 0


@pytest.mark.parametrize("n", [300, 90_000])
def test_failed_steps_keep_what_was_done_ahead(n):
    """A step whose row work does not launch gives none of the ahead-of-time entries away: many times more failures than
    there are entries, and the last dedup is still found."""
    ctx = fs.Context(max_ids=100_000, max_dim=DIM)
    table, state = torch.zeros((ROWS, DIM), device="cuda"), torch.zeros(ROWS, device="cuda")
    a, b, _ = batches(n)
    step = Step(ctx, table, state, a, b, 1, sorted_ids=False)
    for _ in range(80):
        fs.fs_unique_ids_ahead(ctx, step.nxt, ROWS, step.lay1)
        leave_a_host_error()
        raises(fs.FS_EHIP, fs.fs_prioritized_step, ctx, step.args)
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    fs.fs_prioritized_step(ctx, step.args)
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    u = np.unique(b)
    assert int(step.lay1["n_unique"].item()) == len(u)
    assert np.array_equal(step.lay1["unique"][:len(u)].cpu().numpy(), u)
    assert torch.equal(step.emb, table[step.nxt])
    ctx.close()


def test_ahead_call_that_is_refused_leaves_no_entry_behind():
    """FS_STREAM_LAST_STEP before any pipelined call: refused, and the step that names the buffers dedups by itself
    instead of waiting for work that was never posted."""
    ctx = fs.Context(max_ids=1000, max_dim=DIM)
    table, state = torch.zeros((ROWS, DIM), device="cuda"), torch.zeros(ROWS, device="cuda")
    a, b, _ = batches(300)
    step = Step(ctx, table, state, a, b, 1)
    with pytest.raises(fs.FreeScaleError) as e:
        fs.fs_unique_ids_ahead(ctx, step.nxt, ROWS, step.lay1, stream=fs.FS_STREAM_LAST_STEP)
    assert e.value.code == fs.FS_EINVAL
    fs.fs_prioritized_step(ctx, step.args)
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    assert int(step.lay1["n_unique"].item()) == len(np.unique(b))
    ctx.close()
