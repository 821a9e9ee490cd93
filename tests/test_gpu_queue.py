"""GPU tests of the persistent attention launch (the work queues in the
attention workspace) against the one-workgroup-per-item launch.

Both launches run the same device code per (query head, query block) on the
same values, so the bar is bit equality of O and lse.  A call takes the queues
only with many items for the GPU's size, more than most of the other GPU tests
have: the shapes here are past that line, and each test of a queued call checks
that the call wrote its counters.  The oracle parity of the attention itself is
covered by the other GPU tests."""

from __future__ import annotations

import sys

import numpy as np
import pytest

from synth import WORKLOADS, make_inputs
from tests import rbs_harness as H

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _setup(w, dense=False):
    import paper_2609_20971_amd as rbs
    inp = make_inputs(w)
    shape = rbs.make_shape(w.seq_len, w.n_q_heads, w.n_kv_heads, w.block_size)
    Q, K, V = (H.to_device(inp[x]) for x in ("q", "k", "v"))
    if dense:
        counts, indices = rbs.rbs_dense_indices(shape)
    else:
        st = rbs.rbs_block_stats(shape, K)
        counts, indices = rbs.rbs_select(shape, Q, st, w.tau_base, w.tau_rescue, w.n_sink, w.n_local, w.n_recent)
    return shape, Q, K, V, counts, indices


def _attend(shape, Q, K, V, counts, indices, workspace, stream=None):
    import torch
    import paper_2609_20971_amd as rbs
    lse = torch.full((shape.n_q_heads, shape.n_tokens), 7.0, dtype=torch.float32, device=Q.device)
    O = rbs.rbs_sparse_prefill(shape, Q, K, V, counts, indices, 0.0, lse=lse, stream=stream, workspace=workspace)
    return O, lse


def _past_the_line(B, n_q_heads):
    """Tokens of the smallest prompt (a few blocks more) whose attention takes the
    queues: more items than three times the workgroups the GPU holds at once
    (twice at B = 256)."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    line = {64: 3 * 4, 128: 3 * 2, 256: 2}[B] * cus
    return B * (line // n_q_heads + 3) - 5


def _stale_queues():
    import torch
    return torch.full((64,), -5, dtype=torch.int32, device="cuda")


def _assert_queued(ws):
    assert (ws != -5).all(), "the call did not take the queues"


def _assert_same(a, b, what):
    import torch
    torch.cuda.synchronize()
    assert torch.equal(a[0], b[0]), f"{what}: O differs"
    assert torch.equal(a[1], b[1]), f"{what}: lse differs"


@pytest.mark.parametrize("B", [64, 128, 256])
@pytest.mark.parametrize("dense", [False, True])
def test_queue_launch_equals_one_workgroup_per_item(B, dense):
    w = WORKLOADS["tiny-2k"].with_(name="queue", seq_len=_past_the_line(B, 16), n_q_heads=16, n_kv_heads=4,
                                   block_size=B, seed=31 + B)
    _say(f"[queue] B={B} dense={dense} N={w.seq_len} Hq=16 Hkv=4")
    shape, Q, K, V, counts, indices = _setup(w, dense)
    ws = _stale_queues()
    grid = _attend(shape, Q, K, V, counts, indices, None)
    queued = _attend(shape, Q, K, V, counts, indices, ws)
    _assert_same(grid, queued, f"B={B} dense={dense}")
    _assert_queued(ws)
    _assert_same(grid, _attend(shape, Q, K, V, counts, indices, "auto"), f"B={B} dense={dense}, the binding's workspace")


def test_a_call_of_few_items_with_a_workspace():
    # One query block of two heads: 2 work items, one workgroup each whatever the workspace.
    w = WORKLOADS["tiny-2k"].with_(name="queue-tiny", seq_len=100, n_q_heads=2, n_kv_heads=1, block_size=128)
    _say("[queue] 2 items")
    shape, Q, K, V, counts, indices = _setup(w)
    _assert_same(_attend(shape, Q, K, V, counts, indices, None), _attend(shape, Q, K, V, counts, indices, "auto"),
                 "2 items")


@pytest.mark.parametrize("B,extra", [(128, -1), (128, 0), (128, 1), (128, 7), (128, 9), (256, 0), (256, 1), (256, 7)])
def test_item_counts_around_the_resident_count(B, extra):
    """A call takes the queues once it has more than three times the items that
    the GPU holds workgroups (two per compute unit at B = 128), or twice (one per
    unit at B = 256).  Around that the queues hold unequal numbers of tickets, and
    each workgroup has to stop once all eight are empty."""
    import torch
    items = (3 * 2 if B == 128 else 2) * torch.cuda.get_device_properties(0).multi_processor_count + extra
    w = WORKLOADS["tiny-2k"].with_(name="queue-count", seq_len=B * items - 5, n_q_heads=1, n_kv_heads=1,
                                   block_size=B, needles_per_kv_head=0, seed=50)
    _say(f"[queue] {items} items")
    shape, Q, K, V, counts, indices = _setup(w)
    ws = _stale_queues()
    _assert_same(_attend(shape, Q, K, V, counts, indices, None), _attend(shape, Q, K, V, counts, indices, ws),
                 f"{items} items")
    if extra > 0:
        _assert_queued(ws)


@pytest.mark.parametrize("B", [64, 128, 256])
def test_queues_with_more_items_than_resident(B):
    """Every call that takes the queues, with more items than the line from which it
    does: equal to the one-workgroup-per-item launch, and replayed from a
    graph with eager calls on the same workspace between the replays."""
    import torch
    import paper_2609_20971_amd as rbs
    w = WORKLOADS["tiny-2k"].with_(name="queue-many", seq_len=12800, n_q_heads=16, n_kv_heads=2, block_size=B,
                                   seed=60 + B)
    _say(f"[queue] B={B} {16 * w.n_blocks} items")
    shape, Q, K, V, counts, indices = _setup(w)
    ws = _stale_queues()
    ref = _attend(shape, Q, K, V, counts, indices, None)
    _assert_same(ref, _attend(shape, Q, K, V, counts, indices, ws), "bf16")
    _assert_queued(ws)

    ws.fill_(-5)
    f8 = rbs.rbs_fp8_prepare(shape, Q, K, V)
    out8 = [rbs.rbs_sparse_prefill_fp8(shape, f8, counts, indices, workspace=x) for x in (None, ws)]
    torch.cuda.synchronize()
    assert torch.equal(out8[0], out8[1]), "fp8"
    _assert_queued(ws)
    ws.fill_(-5)

    batch = rbs.Batch([3901, 1899, 7000])
    bshape = rbs.varlen_shape(batch, 16, 2, B)
    bc, bi = rbs.rbs_dense_indices_varlen(bshape, batch)
    outb = [rbs.rbs_sparse_prefill_varlen(bshape, batch, Q, K, V, bc, bi, workspace=x) for x in (None, ws)]
    torch.cuda.synchronize()
    assert torch.equal(outb[0], outb[1]), "varlen"
    _assert_queued(ws)

    O, lse = torch.empty_like(Q), torch.empty_like(ref[1])
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        rbs.rbs_sparse_prefill(shape, Q, K, V, counts, indices, 0.0, O, lse=lse, workspace=ws)
    for rep in range(3):
        O.zero_()
        lse.fill_(7.0)
        g.replay()
        _assert_same((O, lse), ref, f"replay {rep}")
        _assert_same(_attend(shape, Q, K, V, counts, indices, ws), ref, f"eager call after replay {rep}")


@pytest.mark.parametrize("heads,blocks", [((8, 8), 239), ((16, 16), 121)])
def test_queues_of_launches_with_kv_heads_of_their_own_on_each_xcd(heads, blocks):
    """B = 64 and a whole number of KV heads per XCD: queued from 1900 items on,
    in the order that gives an XCD its own heads."""
    import torch
    w = WORKLOADS["tiny-2k"].with_(name="queue-own", seq_len=64 * blocks - 5, n_q_heads=heads[0], n_kv_heads=heads[1],
                                   block_size=64, needles_per_kv_head=0, seed=70)
    _say(f"[queue] {heads[0] * blocks} items, {heads[1]} KV heads")
    shape, Q, K, V, counts, indices = _setup(w)
    ws = _stale_queues()
    _assert_same(_attend(shape, Q, K, V, counts, indices, None), _attend(shape, Q, K, V, counts, indices, ws),
                 f"{heads}")
    _assert_queued(ws)


def test_caller_workspace_with_stale_contents_and_reuse():
    """A caller's workspace holding arbitrary values is reset by the call; the
    same workspace then serves a second, smaller problem that is queued too, with
    the counters the first call left, and a third of few items."""
    import torch
    ws = torch.randint(-2**31, 2**31 - 1, (64,), dtype=torch.int32, device="cuda")
    big = WORKLOADS["tiny-2k"].with_(name="queue-big", seq_len=_past_the_line(128, 16) + 1500, n_q_heads=16,
                                     n_kv_heads=2, block_size=128, seed=41)
    cases = [big, big.with_(name="queue-small", seq_len=_past_the_line(128, 16), seed=42),
             big.with_(name="queue-few", seq_len=700, seed=43)]
    runs = [(w, _setup(w)) for w in cases]
    refs = [_attend(*x, None) for _, x in runs]
    for fill in (None, -5, 2**31 - 1):  # first as the call before left it
        for (w, x), ref in zip(runs, refs):
            _say(f"[queue] caller workspace N={w.seq_len} fill={fill}")
            if fill is not None:
                ws.fill_(fill)
            _assert_same(ref, _attend(*x, ws), f"N={w.seq_len}")
            if w.seq_len > 700 and fill is not None:
                assert (ws != fill).all(), "the call did not take the queues"


def test_queue_on_a_side_stream():
    import torch
    w = WORKLOADS["tiny-2k"].with_(name="queue-stream", seq_len=_past_the_line(64, 16), n_q_heads=16, n_kv_heads=2,
                                   block_size=64, seed=43)
    _say("[queue] side stream")
    shape, Q, K, V, counts, indices = _setup(w)
    ws = _stale_queues()
    torch.cuda.synchronize()
    ref = _attend(shape, Q, K, V, counts, indices, None)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        got = _attend(shape, Q, K, V, counts, indices, ws, stream=s)
    s.synchronize()
    _assert_same(ref, got, "side stream")
    _assert_queued(ws)


@pytest.mark.parametrize("B,heads,seqs", [
    (64, (16, 2), [700, 6100, 64, 2049, 1, 4300]),      # by row (head groups of 8)
    (64, (12, 4), [700, 8100, 64, 3049, 1, 5300]),      # one sequence after another (past 3072 items)
    (128, (16, 4), [700, 6100, 64, 2049, 1, 4300]),     # by row
    (128, (64, 8), [700, 6100, 64, 2049, 1, 3400]),     # one after another (past 786432 tokens times heads)
    (256, (16, 4), [700, 6100, 64, 2049, 1, 4300]),     # by row
])
def test_queue_varlen_equals_one_workgroup_per_item(B, heads, seqs):
    import torch
    import paper_2609_20971_amd as rbs
    hq, hkv = heads
    _say(f"[queue] varlen B={B} heads={heads} seqs={seqs}")
    gen = torch.Generator(device="cuda").manual_seed(48)
    batch = rbs.Batch(seqs)
    shape = rbs.varlen_shape(batch, hq, hkv, B)
    Q, K, V = (torch.randn(h, batch.n_tokens, 128, generator=gen, device="cuda").to(torch.bfloat16)
               for h in (hq, hkv, hkv))
    st = rbs.rbs_block_stats_varlen(shape, batch, K)
    counts, indices = rbs.rbs_select_varlen(shape, batch, Q, st, 0.9, 0.95, 1, 2, 0)
    out, queues = [], _stale_queues()
    for ws in (None, queues):
        lse = torch.full((hq, batch.n_tokens), 7.0, dtype=torch.float32, device="cuda")
        O = rbs.rbs_sparse_prefill_varlen(shape, batch, Q, K, V, counts, indices, 0.0, lse=lse, workspace=ws)
        out.append((O, lse))
    _assert_same(out[0], out[1], f"varlen B={B}")
    _assert_queued(queues)


@pytest.mark.parametrize("B", [64, 128, 256])
def test_queue_fp8_equals_one_workgroup_per_item(B):
    import torch
    import paper_2609_20971_amd as rbs
    w = WORKLOADS["tiny-2k"].with_(name="queue-fp8", seq_len=_past_the_line(B, 16), n_q_heads=16, n_kv_heads=4,
                                   block_size=B, seed=44)
    _say(f"[queue] fp8 B={B} N={w.seq_len}")
    shape, Q, K, V, counts, indices = _setup(w)
    f8 = rbs.rbs_fp8_prepare(shape, Q, K, V)
    out, queues = [], _stale_queues()
    for ws in (None, queues):
        lse = torch.full((w.n_q_heads, w.seq_len), 7.0, dtype=torch.float32, device="cuda")
        O = rbs.rbs_sparse_prefill_fp8(shape, f8, counts, indices, lse=lse, workspace=ws)
        out.append((O, lse))
    _assert_same(out[0], out[1], "fp8")
    _assert_queued(queues)
    assert np.isfinite(out[1][1].cpu().numpy()).all()


@pytest.mark.parametrize("B", [64, 128, 256])
def test_queue_fused_equals_one_workgroup_per_item(B):
    import torch
    import paper_2609_20971_amd as rbs
    w = WORKLOADS["tiny-2k"].with_(name="queue-fused", seq_len=_past_the_line(B, 16), n_q_heads=16, n_kv_heads=4,
                                   block_size=B, seed=45 + B)
    _say(f"[queue] fused B={B} N={w.seq_len}")
    inp = make_inputs(w)
    shape = rbs.make_shape(w.seq_len, w.n_q_heads, w.n_kv_heads, w.block_size)
    Q, K, V = (H.to_device(inp[x]) for x in ("q", "k", "v"))
    st = rbs.rbs_block_stats(shape, K)
    out, queues = [], _stale_queues()
    for ws in (None, queues):
        lse = torch.full((w.n_q_heads, w.seq_len), 7.0, dtype=torch.float32, device="cuda")
        counts, indices = rbs.allocate_lists(shape)
        indices.fill_(-1)  # slots past a row's count are left as they are
        _, _, O = rbs.rbs_select_attend(shape, Q, K, V, st, w.tau_base, w.tau_rescue, w.n_sink, w.n_local, w.n_recent,
                                        counts=counts, indices=indices, lse=lse, workspace=ws)
        out.append((counts, indices, O, lse))
    torch.cuda.synchronize()
    for name, a, b in zip(("counts", "lists", "O", "lse"), *out):
        assert torch.equal(a, b), name
    _assert_queued(queues)


def test_persistent_attention_replays_from_a_graph():
    """The persistent launch captured in a graph (the queue reset is a kernel,
    not a memset): every replay equals the eager result, with eager calls on
    the same workspace between replays."""
    import torch
    import paper_2609_20971_amd as rbs
    w = WORKLOADS["tiny-2k"].with_(name="queue-graph", seq_len=_past_the_line(128, 16), n_q_heads=16, n_kv_heads=2,
                                   block_size=128, seed=47)
    _say("[queue] graph replays")
    shape, Q, K, V, counts, indices = _setup(w)
    ws = _stale_queues()
    ref = _attend(shape, Q, K, V, counts, indices, ws)
    torch.cuda.synchronize()
    _assert_queued(ws)
    O = torch.empty_like(Q)
    lse = torch.empty((w.n_q_heads, w.seq_len), dtype=torch.float32, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        rbs.rbs_sparse_prefill(shape, Q, K, V, counts, indices, 0.0, O, lse=lse, workspace=ws)
    for rep in range(3):
        O.zero_()
        lse.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(O, ref[0]), f"replay {rep}: O differs"
        assert torch.equal(lse, ref[1]), f"replay {rep}: lse differs"
        eager = _attend(shape, Q, K, V, counts, indices, ws)  # the same workspace, between replays
        _assert_same(eager, ref, f"eager call after replay {rep}")
