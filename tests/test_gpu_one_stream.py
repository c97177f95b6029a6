"""The pipelined step keeps a call with little row work on one stream and runs a large one on two, and the
self-contained step does the same with its index half: iterations of both sizes in turn (so that every hand-over between
the two forms happens) give the bits of the building blocks issued one after another.  Also: contexts of one GPU share
their side and index streams, also from two threads and after one of them is gone."""
import threading

import numpy as np
import pytest
import torch

import paper_2604_24073_amd as fs
from helpers import table_to_host
from test_gpu_parity import rand_table, run_steps_gpu
from test_gpu_pipeline import make_its, run_pipelined

pytestmark = pytest.mark.gpu

BIG, SMALL = 1800, 60           # longest sequence of 80 users: about 72 k IDs x 256 columns = 147 MB both ways, and 5 MB


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_large_and_small_iterations_in_turn(dtype):
    rng = np.random.default_rng(7)
    rows, dim = 40_000, 256
    its = [make_its(rng, rows, dim, 1, users=80, max_len=m)[0] for m in (BIG, BIG, SMALL, BIG, BIG, SMALL, SMALL)]
    table, state = rand_table(rng, rows, dim, dtype), np.zeros(rows, np.float32)
    ctx = fs.Context(max_ids=200_000, max_dim=dim)
    want_t, want_s, want = run_steps_gpu(ctx, table, state, its, 0.01, 1e-8, mode="fused_calls")
    view = torch.int16 if dtype == "bf16" else torch.int32
    got_t, got_s, got = run_steps_gpu(ctx, table, state, its, 0.01, 1e-8, mode="step")
    assert torch.equal(got_t.view(view), want_t.view(view)) and torch.equal(got_s, want_s)
    for ahead, sync_each, two_part in (("batch2_last_step", False, False), ("index", True, False), (False, False, False),
                                       ("index", False, True), (False, True, True)):
        got_t, got_s, got = run_pipelined(ctx, table, state, its, 0.01, 1e-8, ahead=ahead, sync_each=sync_each, two_part=two_part)
        what = f"ahead={ahead} sync_each={sync_each} two_part={two_part}"
        assert torch.equal(got_t.view(view), want_t.view(view)) and torch.equal(got_s, want_s), what
        for a, b in zip(got, want[1:]):
            assert a["reduced"].tobytes() == b["reduced"].tobytes(), what
            if "emb_next" in a:
                assert a["emb_next"].tobytes() == b["emb_next"].tobytes(), what
    ctx.close()


def test_contexts_share_their_streams():
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
