"""Graphs with bit rows of more nodes than the identity route takes: order 4
is counted by bit rows or, where the squared degrees say so, by the walks and
runs of graphs without them.  Each way against one that shares no code with
it, and what both owe the caller's stream."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hm():
    import torch
    import paper_2209_10241_amd as hm
    assert torch.cuda.is_available()
    return hm


def _hubs(n, hubs, degree, pairs, seed=0):
    """(members, offsets): `hubs` nodes of `degree` pairs each, other pairs, n 3-node and n / 4 4-node hyperedges."""
    rng = np.random.default_rng(seed + n + hubs)
    parts = [np.c_[np.full(degree, h), rng.choice(n, degree, replace=False)] for h in range(hubs)]
    parts += [rng.integers(0, n, (pairs, 2))]
    parts = [np.concatenate(parts), rng.integers(0, n, (n, 3)), rng.integers(0, n, (n // 4, 4))]
    parts = [np.sort(e, axis=1) for e in parts]
    parts = [e[(e[:, 1:] > e[:, :-1]).all(axis=1)] for e in parts]
    members = np.concatenate([e.ravel() for e in parts]).astype(np.uint32)
    offsets = np.r_[0, np.cumsum(np.concatenate([np.full(len(e), e.shape[1]) for e in parts]))].astype(np.uint64)
    return members, offsets


def _by_bit_rows(hm, g):
    """Order-4 counts by the entry point that always takes the bit rows."""
    import torch
    out = torch.empty(hm.hm_num_classes(4), dtype=torch.int64, device="cuda")
    assert hm.lib().count_exact_noalloc(g.handle, 4, ctypes.c_void_p(out.data_ptr()), None) == 0
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("one_pass", [True, False])
@pytest.mark.parametrize("n,hubs,degree,pairs,runs", [
    (8000, 5, 7900, 4000, True), (8000, 1, 7900, 10, True), (4097, 3, 4000, 0, True), (8000, 1, 1800, 4000, False),
    (2600, 1, 300, 2000, False)])
def test_few_hubs_decide_the_route(hm, n, hubs, degree, pairs, runs, one_pass):
    """A few hubs among few pairs outweigh the line between bit rows and runs
    (2^30 words) though the number of pairs alone lies far below it; in either
    kind of build, which sums the squared degrees."""
    members, offsets = _hubs(n, hubs, degree, pairs)
    keep = hm.hm_get_option(hm.HM_OPT_ONE_PASS_MAX_EDGES)
    hm.hm_set_option(hm.HM_OPT_ONE_PASS_MAX_EDGES, keep if one_pass else 0)
    try:
        g = hm.hm_graph_create(members, offsets, n)
    finally:
        hm.hm_set_option(hm.HM_OPT_ONE_PASS_MAX_EDGES, keep)
    with g:
        hm.hm_profile_enable(True)
        hm.hm_profile_reset()
        try:
            got = hm.count_exact(g, 4).cpu().numpy()
            names = hm.hm_profile_read()
        finally:
            hm.hm_profile_enable(False)
            hm.hm_profile_reset()
        assert ("k_walk" in names) == runs and ("k_exact4_bits" in names) != runs
        assert np.array_equal(got, _by_bit_rows(hm, g))


@pytest.mark.parametrize("n,hubs,degree,pairs", [(8000, 5, 7900, 4000), (2600, 0, 1, 120_000)])
def test_calls_do_not_wait(hm, n, hubs, degree, pairs):
    """Counts and samples of these graphs are enqueued on the stream, as the
    header says: behind work that keeps the stream busy they return before it
    ends, on a handle's first call too, and give what they give otherwise."""
    import torch
    members, offsets = _hubs(n, hubs, degree, pairs)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    torch.cuda._sleep(1_000_000)
    b.record()
    b.synchronize()
    cycles = int(1_000_000 * 400 / a.elapsed_time(b))   # about 0.4 s
    calls = [lambda g: hm.count_exact(g, 4)] + [lambda g: hm.count_sampled(g, 4, 0.05, 7)[1]] * 4
    with hm.hm_graph_create(members, offsets, n) as g:
        want = [f(g) for f in calls]   # (also leaves the memory that the calls need in the library's cache)
        torch.cuda.synchronize()
    with hm.hm_graph_create(members, offsets, n) as g:
        torch.cuda.synchronize()
        torch.cuda._sleep(cycles)
        after = torch.cuda.Event()
        after.record()
        got = [f(g) for f in calls]
        waited = after.query()
        torch.cuda.synchronize()
    assert not waited
    for w, x in zip(want, got):
        assert torch.equal(w, x)


def test_first_calls_refuse_a_capture(hm):
    """On a stream that is being captured, calls that would build a graph's
    indices are refused (a handle must not keep what was only recorded), leave
    the capture and the handle as they were, and work afterwards; graphs with
    bit rows are captured by them, whichever way they count otherwise, and
    replay."""
    import torch
    members, offsets = _hubs(3000, 3, 2500, 3000)
    keep = hm.hm_get_option(hm.HM_OPT_BITSET_MAX_NODES)
    hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 0)
    try:
        bare = hm.hm_graph_create(members, offsets, 3000)
    finally:
        hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, keep)
    with bare, hm.hm_graph_create(members, offsets, 3000) as g, hm.hm_graph_create(members, offsets, 3000) as ref:
        want = {k: hm.count_exact(ref, k).clone() for k in (3, 4)}
        sampled = [hm.count_sampled(ref, 4, 0.05, s)[1].clone() for s in (1, 2)]
        out = torch.zeros(hm.hm_num_classes(4), dtype=torch.int64, device="cuda")
        est, raw = torch.zeros(out.numel(), device="cuda"), torch.zeros_like(out)
        torch.cuda.synchronize()
        stream, graph, errors = torch.cuda.Stream(), torch.cuda.CUDAGraph(), []
        with torch.cuda.stream(stream):
            graph.capture_begin(capture_error_mode="thread_local")
            for call in (lambda: hm.count_exact(bare, 3, out=out), lambda: hm.count_exact(bare, 4, out=out),
                         lambda: hm.count_sampled(bare, 4, 0.05, 1, est=est, raw=raw)):
                try:
                    call()
                except hm.HMError as e:
                    errors.append(e.code)
            hm.count_exact(g, 4, out=out)
            for s in (1, 2):
                hm.count_sampled(g, 4, 0.05, s, est=est, raw=raw)
            graph.capture_end()
        assert errors == [hm.binding.HM_EDEVICE] * 3
        for _ in range(3):
            out.zero_()
            raw.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want[4]) and torch.equal(raw, sampled[1])
        del graph
        for k in (3, 4):
            assert torch.equal(hm.count_exact(bare, k), want[k])
            assert torch.equal(hm.count_exact(g, k), want[k])
        for s in (1, 2):
            assert torch.equal(hm.count_sampled(bare, 4, 0.05, s)[1], sampled[s - 1])


@pytest.mark.parametrize("n,hubs,degree,pairs", [(4000, 40, 3700, 8000), (3000, 3, 2900, 6000), (8000, 5, 7900, 4000)])
def test_walks_match_the_bit_rows(hm, n, hubs, degree, pairs):
    """The walks and runs (walks split into shares among them) against the
    bit rows: a graph without bit rows and one that turns to the walks against
    count_exact_noalloc, and samples of every stratum, on handles that have
    turned to the walks, against a handle's first call, which has not."""
    members, offsets = _hubs(n, hubs, degree, pairs)
    keep = hm.hm_get_option(hm.HM_OPT_BITSET_MAX_NODES)
    hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 0)
    try:
        bare = hm.hm_graph_create(members, offsets, n)
    finally:
        hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, keep)
    rng = np.random.default_rng(n)

    def profiled(call):
        hm.hm_profile_enable(True)
        hm.hm_profile_reset()
        try:
            return call().cpu().numpy(), hm.hm_profile_read()
        finally:
            hm.hm_profile_enable(False)
            hm.hm_profile_reset()

    with bare, hm.hm_graph_create(members, offsets, n) as turned:
        want = _by_bit_rows(hm, turned)
        got, names = profiled(lambda: hm.count_exact(turned, 4))
        assert "k_walk" in names and np.array_equal(got, want)
        assert np.array_equal(hm.count_exact(bare, 4).cpu().numpy(), want)
        for _ in range(4):   # enough words read for the later calls to turn
            hm.count_sampled(turned, 4, 0.2, 1)
        for size in (1, 40, 700):
            idx = {j: rng.integers(0, turned.stats()["n%d" % j], size) for j in (2, 3, 4)}
            with hm.hm_graph_create(members, offsets, n) as fresh:
                first = hm.count_sampled_indices(fresh, 4, idx)[1].cpu().numpy()
            assert np.array_equal(hm.count_sampled_indices(turned, 4, idx)[1].cpu().numpy(), first), size
            assert np.array_equal(hm.count_sampled_indices(bare, 4, idx)[1].cpu().numpy(), first), size


def test_enqueued_counts_share_their_temporaries(hm):
    """Counts by the walks enqueued one behind another, none of them waited
    for, take the temporaries of one: a hundred of them take no more of the
    device's free memory than two would, and count what one counts alone."""
    import torch
    members, offsets = _hubs(8000, 5, 7900, 4000)
    outs = [torch.zeros(hm.hm_num_classes(4), dtype=torch.int64, device="cuda") for _ in range(100)]
    with hm.hm_graph_create(members, offsets, 8000) as g:
        want = hm.count_exact(g, 4).clone()
        x = torch.ones(8192, 8192, device="cuda")
        y = x @ x
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        for _ in range(8):   # tens of milliseconds of work for the counts to pile up behind
            torch.mm(x, x, out=y)
        hm.count_exact(g, 4, out=outs[0])
        hm.count_exact(g, 4, out=outs[1])
        two = free - torch.cuda.mem_get_info()[0]
        for out in outs[2:]:
            hm.count_exact(g, 4, out=out)
        taken = free - torch.cuda.mem_get_info()[0]
        torch.cuda.synchronize()
        assert taken <= two + (8 << 20)   # (the runtime's own queues and events may grow)
        for out in outs:
            assert torch.equal(out, want)
