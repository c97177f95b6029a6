"""The pipelined step keeps a call with little row work on one stream and runs a large one on two, and the
self-contained step does the same with its index half: iterations of both sizes in turn (so that every hand-over between
the two forms happens) give the bits of the building blocks issued one after another.  Also: contexts driven from one
stream share their side and index streams; a context that is called on a second stream, or captured, has its own."""
import ctypes
import threading

import numpy as np
import pytest
import torch

import paper_2604_24073_amd as fs
from paper_2604_24073_amd.schedule import new_hip_stream
from helpers import dev, table_to_host
from test_gpu_parity import rand_table, run_steps_gpu, zipf_ids
from test_gpu_pipeline import make_its, run_pipelined

pytestmark = pytest.mark.gpu

# longest sequence of 80 users: about 96 k IDs x 256 columns, 196 MB a call in fp32 and 147 MB with bf16 rows; and 5 MB
BIG, SMALL = 2400, 60
ONE_STREAM = 120 << 20          # most bytes of gradients and looked-up rows of a call on one stream


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_large_and_small_iterations_in_turn(dtype):
    rng = np.random.default_rng(7)
    rows, dim = 40_000, 256
    sizes = (BIG, BIG, BIG, SMALL, SMALL, BIG, BIG, BIG, SMALL, SMALL)
    its = [make_its(rng, rows, dim, 1, users=80, max_len=m)[0] for m in sizes]
    # with the index halves done ahead the bytes of a call decide: two on two streams in a row, so that the second one
    # finds exclusive rows fetched, and both ways between the forms (a small batch beside a large one: either)
    w = 4 if dtype == "f32" else 2
    two = [a.grads.nbytes + len(b.values) * dim * w > ONE_STREAM for a, b in zip(its, its[1:])]
    assert two[0] and two[1] and two[5] and two[6] and not two[3] and not two[8]
    table, state = rand_table(rng, rows, dim, dtype), np.zeros(rows, np.float32)
    ctx = fs.Context(max_ids=200_000, max_dim=dim)
    want_t, want_s, want = run_steps_gpu(ctx, table, state, its, 0.01, 1e-8, mode="fused_calls")
    view = torch.int16 if dtype == "bf16" else torch.int32
    got_t, got_s, got = run_steps_gpu(ctx, table, state, its, 0.01, 1e-8, mode="step")
    assert torch.equal(got_t.view(view), want_t.view(view)) and torch.equal(got_s, want_s)
    for ahead, sync_each, two_part in (("batch2_last_step", False, False), ("index", True, False), (False, False, False),
                                       ("index", False, True), (False, True, True), ("batch2_last_step", False, True),
                                       ("batch2", True, True)):
        got_t, got_s, got = run_pipelined(ctx, table, state, its, 0.01, 1e-8, ahead=ahead, sync_each=sync_each, two_part=two_part)
        what = f"ahead={ahead} sync_each={sync_each} two_part={two_part}"
        assert torch.equal(got_t.view(view), want_t.view(view)) and torch.equal(got_s, want_s), what
        for a, b in zip(got, want[1:]):
            assert a["reduced"].tobytes() == b["reduced"].tobytes(), what
            if "emb_next" in a:
                assert a["emb_next"].tobytes() == b["emb_next"].tobytes(), what
    ctx.close()


def test_contexts_share_their_streams_until_they_are_called_on_another():
    # both on the default stream (one set for the two), then each on a stream of its own from a thread of its own (a set
    # each, work still queued on the old one), then one of them alone
    rng = np.random.default_rng(8)
    rows, dim = 5000, 64
    its = [make_its(rng, rows, dim, 6, users=40, max_len=300) for _ in range(2)]
    table, state = rand_table(rng, rows, dim, "f32"), np.zeros(rows, np.float32)
    ctxs = [fs.Context(max_ids=20_000, max_dim=dim) for _ in range(2)]
    want = [run_pipelined(ctxs[k], table, state, its[k], 0.01, 1e-8, ahead="batch2_last_step") for k in range(2)]
    got, errors = [None, None], []

    def work(k):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                got[k] = run_pipelined(ctxs[k], table, state, its[k], 0.01, 1e-8, ahead="batch2_last_step", sync_each=False)
        except Exception as e:      # noqa: BLE001 - reported below, in the test's own thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for k in range(2):
        assert torch.equal(got[k][0], want[k][0]) and torch.equal(got[k][1], want[k][1])
    ctxs[0].close()                  # the other context still has its streams
    again = run_pipelined(ctxs[1], table, state, its[1], 0.01, 1e-8, ahead="index")
    assert table_to_host(again[0]).tobytes() == table_to_host(want[1][0]).tobytes()
    ctxs[1].close()


def test_contexts_on_one_stream_take_turns():
    """Two contexts stepped in turn on one stream that is not the default one, without a wait between the calls."""
    rng = np.random.default_rng(9)
    rows, dim = 5000, 64
    its = [make_its(rng, rows, dim, 5, users=40, max_len=300) for _ in range(2)]
    table, state = rand_table(rng, rows, dim, "f32"), np.zeros(rows, np.float32)
    ctxs = [fs.Context(max_ids=20_000, max_dim=dim) for _ in range(2)]
    want = [run_pipelined(ctxs[k], table, state, its[k], 0.01, 1e-8, ahead="index") for k in range(2)]
    got = [None, None]
    with torch.cuda.stream(torch.cuda.Stream()):
        fresh = [fs.Context(max_ids=20_000, max_dim=dim) for _ in range(2)]

        def inner(_):                # the other context's whole run between two steps of this one
            if got[1] is None:
                got[1] = run_pipelined(fresh[1], table, state, its[1], 0.01, 1e-8, ahead="batch2_last_step", sync_each=False)

        got[0] = run_pipelined(fresh[0], table, state, its[0], 0.01, 1e-8, ahead=False, sync_each=False, between=inner)
    for k in range(2):
        assert torch.equal(got[k][0], want[k][0]) and torch.equal(got[k][1], want[k][1])
    for c in ctxs + fresh:
        c.close()


@pytest.mark.parametrize("ahead", [False, "index_last_step", "batch2"])
def test_context_that_changes_its_stream_between_two_steps(ahead):
    """Consecutive pipelined calls on two streams in turn, ordered by the caller with events and nothing else: the work
    the context left on its side and index streams stays ordered before what follows on the new ones."""
    rng = np.random.default_rng(10)
    rows, dim = 30_000, 256
    its = make_its(rng, rows, dim, 6, users=80, max_len=1800)            # 147 MB a call: two streams
    table, state = rand_table(rng, rows, dim, "f32"), np.zeros(rows, np.float32)
    ctx = fs.Context(max_ids=100_000, max_dim=dim)
    want = run_pipelined(ctx, table, state, its, 0.01, 1e-8)
    ctx.close()
    ctx = fs.Context(max_ids=100_000, max_dim=dim)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    before = torch.cuda.current_stream()

    def switch(t):
        was = torch.cuda.current_stream()
        now = streams[t % 2]
        now.wait_stream(was)
        torch.cuda.set_stream(now)

    try:
        got = run_pipelined(ctx, table, state, its, 0.01, 1e-8, ahead=ahead, sync_each=False, between=switch)
    finally:
        torch.cuda.synchronize()
        torch.cuda.set_stream(before)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    ctx.close()


def test_captured_step_beside_another_context():
    """The self-contained step recorded into a graph by the caller, its index half on a side stream, while another context
    enqueues on its own streams: neither sees the other, and every replay gives the eager step's bits."""
    rng = np.random.default_rng(12)
    rows, dim, n = 20_000, 32, 90_000
    a, b = (zipf_ids(rng, n, rows, a=1.1) for _ in range(2))
    grads = dev(rng.standard_normal((n, dim)).astype(np.float32))
    start = rand_table(rng, rows, dim, "f32")

    def step_on(ctx, stream=None):
        table, state = dev(start), torch.zeros(rows, device="cuda")
        lay0, lay1 = fs.fs_unique_ids(ctx, dev(a), rows), fs.alloc_layout(n, "cuda")
        split, emb, nxt = fs.alloc_split(n, n, "cuda"), torch.zeros((n, dim), device="cuda"), dev(b)
        args = fs.make_step_args(table, state, 0.01, 1e-8, lay0, grads, nxt, None, lay1, split, None, emb)
        return args, (table, state, emb, lay1, split, lay0, nxt)

    ctx, other, ref = (fs.Context(max_ids=100_000, max_dim=dim) for _ in range(3))
    eager, out = step_on(ref)
    captured, got = step_on(ctx)
    beside, out2 = step_on(other)
    torch.cuda.synchronize()
    graph, stream, third = torch.cuda.CUDAGraph(), torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="relaxed"):
        fs.fs_prioritized_step(ctx, captured, stream=stream)
        fs.fs_step_forward(other, beside, stream=third)
    for _ in range(3):
        graph.replay()
        fs.fs_prioritized_step(ref, eager)
        torch.cuda.synchronize()
        for x, y in zip(got[:3], out[:3]):
            assert torch.equal(x, y)
        for k in ("co_slot", "counts"):
            m = int(out[4]["counts"][0].item()) if k == "co_slot" else 3
            assert torch.equal(got[4][k][:m], out[4][k][:m])
        u = int(out[3]["n_unique"].item())
        assert torch.equal(got[3]["unique"][:u], out[3]["unique"][:u])
    for c in (ctx, other, ref):
        assert fs.fs_check_async(c) == fs.FS_OK, c.last_error()
    assert torch.equal(out2[4]["counts"], out[4]["counts"])
    for c in (ctx, other, ref):
        c.close()


def kernels_captured(call):
    """Number of kernel nodes of what `call(stream)` enqueues (recorded, not run)."""
    hip = ctypes.CDLL("libamdhip64.so")
    stream = new_hip_stream()
    raw, graph = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p()
    assert hip.hipStreamBeginCapture(raw, ctypes.c_int(2)) == 0                    # relaxed
    call(stream)
    assert hip.hipStreamEndCapture(raw, ctypes.byref(graph)) == 0
    n = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    kernels = 0
    for node in nodes:
        kind = ctypes.c_int(-1)
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
        kernels += kind.value == 0                                                 # hipGraphNodeTypeKernel
    assert hip.hipGraphDestroy(graph) == 0
    return kernels


@pytest.mark.parametrize("n", [1, 2000, 49_152, 65_535, 65_536, 98_304, 131_071, 131_072, 600_000])
def test_tables_of_one_width_share_their_launches(n):
    """Eight equal tables as large as the context allows, on one stream: both passes of four tables a launch (the context
    has room for the pieces of all of them), and one lookup for the eight."""
    rows, dim = 500, 4
    ctx = fs.Context(max_ids=n, max_dim=dim)
    tables, keep = [], []
    for k in range(8):
        ids = (torch.arange(n, device="cuda") * (k + 1)) % rows
        nxt = torch.arange(min(n, 64), device="cuda")
        lay, lay1 = fs.fs_unique_ids(ctx, ids, rows), fs.alloc_layout(nxt.numel(), "cuda")
        split = fs.alloc_split(n, nxt.numel(), "cuda")
        table, state = torch.zeros((rows, dim), device="cuda"), torch.zeros(rows, device="cuda")
        grads, emb = torch.ones((n, dim), device="cuda"), torch.empty((nxt.numel(), dim), device="cuda")
        tables.append(fs.make_step_args(table, state, 0.01, 1e-8, lay, grads, nxt, None, lay1, split, None, emb))
        keep.append((ids, nxt, lay, lay1, split, table, state, grads, emb))
        fs.fs_step_forward(ctx, tables[-1])
    assert fs.fs_check_async(ctx) == fs.FS_OK, ctx.last_error()
    record = fs.step_args_array(tables)
    passes = kernels_captured(lambda s: fs.fs_prioritized_step_pipelined_multi(ctx, record, None, stream=s)) - 1
    assert passes == 2
    ctx.close()
