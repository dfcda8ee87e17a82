"""Exact counts through the C ABI on the GPU against the oracle (bit-exact int64)."""
import json
import os

import functools

import numpy as np
import pytest

import workloads as W
from oracle import core

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def hm():
    import torch
    import paper_2209_10241_amd as hm
    assert torch.cuda.is_available()
    return hm


def _gpu_counts(hm, h, k, bit_rows=True):
    """Counts through the C ABI; bit_rows=False forces the hash-probe kernels."""
    hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192 if bit_rows else 0)
    try:
        with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
            return hm.count_exact(g, k).cpu().numpy()
    finally:
        hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192)


def _golden(name, k):
    with open(os.path.join(ROOT, "tests", "golden", "workload_counts.json")) as f:
        for c in json.load(f)["cases"]:
            if c["workload"] == name and c["k"] == k:
                return np.array(c["counts"], dtype=np.int64)
    raise KeyError(name)


def test_ingest_strata_match_oracle(hm):
    h = W.random_small(3, 30, 300, {1: 0.05, 2: 0.5, 3: 0.3, 4: 0.1, 5: 0.05}, allow_dups=True)
    nh = core.normalise(h)
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        st = g.stats()
        assert (st["n2"], st["n3"], st["n4"]) == (nh.count(2), nh.count(3), nh.count(4))
        assert st["singletons"] == nh.n_dropped_singletons and st["duplicates"] == nh.n_duplicates
        for j in (2, 3, 4):
            assert np.array_equal(g.export(j).astype(np.int64), nh.edges(j))


@pytest.mark.parametrize("bit_rows", [True, False], ids=["bits", "hash"])
@pytest.mark.parametrize("seed", range(40))
def test_random_small_matches_oracle(hm, seed, bit_rows):
    mixes = [{2: 0.6, 3: 0.3, 4: 0.1}, {1: 0.05, 2: 0.45, 3: 0.3, 4: 0.15, 5: 0.05}, {2: 0.2, 3: 0.5, 4: 0.3},
             {2: 1.0}, {3: 0.5, 4: 0.5}]
    n = 12 + (seed * 7) % 60
    h = W.random_small(1000 + seed, n, 20 + (seed * 37) % 400, mixes[seed % len(mixes)], allow_dups=bool(seed % 3))
    for k in (3, 4):
        assert np.array_equal(_gpu_counts(hm, h, k, bit_rows), core.count_exact(h, k)), (seed, k)


def test_hand_examples(hm, golden_dir):
    with open(os.path.join(golden_dir, "hand_examples.json")) as f:
        examples = json.load(f)["examples"]
    for ex in examples:
        h = W.from_lists(ex["edges"], ex["n_nodes"])
        for k in (3, 4):
            for bit_rows in (True, False):
                assert np.array_equal(_gpu_counts(hm, h, k, bit_rows), core.count_exact(h, k)), ex["name"]


@pytest.mark.parametrize("bit_rows", [True, False], ids=["bits", "hash"])
def test_facetoface_order3_workload(hm, bit_rows):
    h = W.cfg0_facetoface_k3(0)
    assert np.array_equal(_gpu_counts(hm, h, 3, bit_rows), _golden("facetoface_N200_E2000", 3))


@pytest.mark.parametrize("bit_rows", [True, False], ids=["bits", "hash"])
def test_facetoface_order4_workload(hm, bit_rows):
    """The benchmark's workload: N=400, 30,000 hyperedges, k=4."""
    h = W.cfg1_facetoface_k4(0)
    assert np.array_equal(_gpu_counts(hm, h, 4, bit_rows), _golden("facetoface_N400_E30000", 4))


@pytest.mark.parametrize("bit_rows", [True, False], ids=["bits", "hash"])
def test_communication_scaled_workload(hm, bit_rows):
    """Heavy-tailed degrees (communication recipe at 0.4% of its size), stored oracle counts."""
    h = W.scaled_communication(0.004, 0)
    assert np.array_equal(_gpu_counts(hm, h, 4, bit_rows), _golden("communication_scaled_0.004", 4))


def _heavy_goldens():
    with open(os.path.join(ROOT, "tests", "golden", "workload_counts.json")) as f:
        names = [c["workload"] for c in json.load(f)["cases"]]
    out = []
    for name in names:
        for family, maker in (("communication", W.scaled_communication), ("coauthorship", W.scaled_coauthorship)):
            prefix = f"{family}_scaled_"
            if name.startswith(prefix) and name != "communication_scaled_0.004":
                out.append((name, maker, float(name[len(prefix):])))
    return out


@pytest.mark.parametrize("bit_rows", [True, False], ids=["bits", "hash"])
@pytest.mark.parametrize("name,maker,scale", _heavy_goldens(), ids=[c[0] for c in _heavy_goldens()])
def test_heavy_tailed_scaled_goldens(hm, name, maker, scale, bit_rows):
    """The heavy-tailed recipes at the largest fractions of their size whose
    oracle counts are stored (Algorithm 3 on every host core): both GPU paths
    bit-exact.  Graphs with more nodes than bit rows hold have one path."""
    h = maker(scale, 0)
    if bit_rows and h.n_nodes > 8192:
        pytest.skip(f"{h.n_nodes} nodes: more than adjacency bit rows hold, the hash path is the only one")
    assert np.array_equal(_gpu_counts(hm, h, 4, bit_rows), _golden(name, 4))


@pytest.fixture(scope="module")
def full_size():
    """The co-authorship (10^6 nodes, 2x10^6 draws) and communication (5x10^4
    nodes, 5x10^6 draws) workloads at full size, generated once."""
    out = {}
    for name, maker in (("coauthorship", W.cfg3_coauthorship), ("communication", W.cfg4_communication)):
        print(f"generating {name}", flush=True)
        out[name] = maker(0)
    return out


@pytest.mark.parametrize("name", ["coauthorship", "communication"])
def test_full_size_relabelling_and_census(hm, full_size, name):
    """At full size, where the oracle cannot run: (1) the exact counts do not
    change under a fixed node relabelling (Section 3: a motif is an
    isomorphism class), and (2) a census through the sampler - every
    hyperedge of size 2..4 drawn exactly once (Algorithm 4 with S_j = |E_j|)
    - gives raw counts countmax_m * n_m for every class and estimates equal to
    the exact counts.  The sampler enumerates each hyperedge's neighbourhood;
    the exact count uses graph identities and ownership rules: two
    independent routes to the same int64 vector."""
    h = full_size[name]
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        exact = hm.count_exact(g, 4).cpu().numpy()
        st = g.stats()
        samples = {j: np.arange(st[f"n{j}"]) for j in range(2, 5)}
        print(f"{name}: census of {sum(len(v) for v in samples.values())} hyperedges", flush=True)
        est, raw = hm.count_sampled_indices(g, 4, samples)
    countmax = np.array([hm.hm_class_info(4, c)[2] for c in range(len(exact))], dtype=np.int64)
    assert exact.sum() > 10**12
    assert np.array_equal(raw.cpu().numpy(), exact * countmax)
    assert np.array_equal(est.cpu().numpy(), exact.astype(np.float32))
    perm = np.random.default_rng(11).permutation(h.n_nodes)
    hp = W.Hypergraph(h.n_nodes, perm[h.members.astype(np.int64)].astype(np.uint32), h.offsets.copy())
    print(f"{name}: relabelled count", flush=True)
    assert np.array_equal(_gpu_counts(hm, hp, 4), exact)


@pytest.mark.parametrize("scale", [0.02, 0.05])
def test_sparse_path_agrees_with_bit_rows(hm, scale):
    """Larger heavy-tailed graphs: the counting formulas without bit rows and the
    bit-row enumeration are independent routes to the same int64 counts."""
    h = W.scaled_communication(scale, 1)
    for k in (3, 4):
        a = _gpu_counts(hm, h, k, True)
        b = _gpu_counts(hm, h, k, False)
        assert np.array_equal(a, b), (scale, k)
        assert a.sum() > 0


@pytest.mark.parametrize("bit_rows", [True, False], ids=["bits", "hash"])
def test_repeated_calls_on_one_graph(hm, bit_rows):
    """The counting scratch is left clear after every call: orders alternate on
    one graph and every call matches the oracle."""
    h = W.random_small(77, 50, 600, {2: 0.5, 3: 0.3, 4: 0.2}, allow_dups=True)
    want = {k: core.count_exact(h, k) for k in (3, 4)}
    hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192 if bit_rows else 0)
    try:
        with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
            for k in (4, 4, 3, 4, 3, 3, 4):
                assert np.array_equal(hm.count_exact(g, k).cpu().numpy(), want[k]), k
    finally:
        hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192)


def test_facetoface_order4_relabelled(hm):
    h = W.cfg1_facetoface_k4(0)
    perm = np.random.default_rng(5).permutation(h.n_nodes)
    hp = W.Hypergraph(h.n_nodes, perm[h.members.astype(np.int64)].astype(np.uint32), h.offsets.copy())
    assert np.array_equal(_gpu_counts(hm, hp, 4), _golden("facetoface_N400_E30000", 4))


@pytest.mark.parametrize("n_ids", [200_000, 1 << 22], ids=["ids_2e5", "ids_4M"])
@pytest.mark.parametrize("seed", range(3))
def test_large_node_ids(hm, seed, n_ids):
    """More nodes than the adjacency bit rows allow: pairs are probed in the hash set.
    At 2^22 ids three node ids no longer pack into 63 bits, so the 4-node
    hyperedges holding a 3-node one are found through the incidence lists
    instead of the 3-subset index."""
    base = W.random_small(2000 + seed, 60, 500, {2: 0.6, 3: 0.3, 4: 0.1})
    rng = np.random.default_rng(seed)
    ids = np.sort(rng.choice(n_ids, size=60, replace=False))
    h = W.Hypergraph(n_ids, ids[base.members.astype(np.int64)].astype(np.uint32), base.offsets.copy())
    for k in (3, 4):
        assert np.array_equal(_gpu_counts(hm, h, k), core.count_exact(h, k)), (seed, k)


def test_device_resident_input(hm):
    import torch
    h = W.random_small(77, 50, 400, {2: 0.5, 3: 0.3, 4: 0.2})
    m = torch.from_numpy(h.members.astype(np.int32)).cuda()
    o = torch.from_numpy(h.offsets.astype(np.int64)).cuda()
    with hm.hm_graph_create(m, o, h.n_nodes) as g:
        for k in (3, 4):
            assert np.array_equal(hm.count_exact(g, k).cpu().numpy(), core.count_exact(h, k))


def test_degenerate_inputs(hm):
    empty = W.Hypergraph(5, np.zeros(0, np.uint32), np.zeros(1, np.uint64))
    singles = W.from_lists([[0], [3], [4]], 5)
    big_only = W.from_lists([[0, 1, 2, 3, 4]], 5)
    for h in (empty, singles, big_only):
        for k in (3, 4):
            assert _gpu_counts(hm, h, k).sum() == 0


@pytest.mark.parametrize("edges,n", [([[0, 1], [2, 2]], 3), ([[0, 7]], 3)])
def test_invalid_inputs(hm, edges, n):
    h = W.from_lists(edges, n)
    with pytest.raises(hm.HMError) as e:
        hm.hm_graph_create(h.members, h.offsets, n)
    assert e.value.code == -1


def test_empty_hyperedge_is_rejected(hm):
    with pytest.raises(hm.HMError):
        hm.hm_graph_create(np.array([0, 1], np.uint32), np.array([0, 2, 2], np.uint64), 3)


@pytest.mark.parametrize("where", ["host", "device"])
@pytest.mark.parametrize("offsets", [[1, 3, 5], [0, 3, 2], [0, 2, 7]], ids=["start", "decrease", "beyond"])
def test_bad_offsets_are_rejected(hm, where, offsets):
    """Offsets must start at 0, not decrease and stay within the members."""
    import torch
    m = np.array([0, 1, 2, 3, 4], np.uint32)
    o = np.array(offsets, np.uint64)
    if where == "device":
        m = torch.from_numpy(m.astype(np.int32)).cuda()
        o = torch.from_numpy(o.astype(np.int64)).cuda()
    with pytest.raises(hm.HMError) as e:
        hm.hm_graph_create(m, o, 6)
    assert e.value.code == -1


def test_members_beyond_the_last_offset_are_ignored(hm):
    """Trailing entries of members that no hyperedge reaches do not count."""
    import torch
    h = W.random_small(78, 30, 200, {2: 0.5, 3: 0.3, 4: 0.2})
    tail = np.array([29, 29, 29], np.uint32)
    for dev in (False, True):
        m = np.concatenate([h.members.astype(np.uint32), tail])
        o = h.offsets.astype(np.uint64)
        if dev:
            m = torch.from_numpy(m.astype(np.int32)).cuda()
            o = torch.from_numpy(o.astype(np.int64)).cuda()
        with hm.hm_graph_create(m, o, h.n_nodes) as g:
            assert np.array_equal(hm.count_exact(g, 4).cpu().numpy(), core.count_exact(h, 4))


def test_many_graphs_created_and_destroyed_in_stream_order(hm):
    """Graphs destroyed without a device-wide wait: memory released in stream
    order is not reused before the work that reads it has run."""
    import torch
    hs = [W.random_small(90 + i, 40, 300, {2: 0.5, 3: 0.3, 4: 0.2}) for i in range(6)]
    want = [core.count_exact(h, 4) for h in hs]
    outs = []
    for _ in range(3):
        for h in hs:
            m = torch.from_numpy(h.members.astype(np.int32)).cuda()
            o = torch.from_numpy(h.offsets.astype(np.int64)).cuda()
            g = hm.hm_graph_create(m, o, h.n_nodes)
            outs.append(hm.count_exact(g, 4))
            g.close()
    torch.cuda.synchronize()
    for i, c in enumerate(outs):
        assert np.array_equal(c.cpu().numpy(), want[i % len(hs)]), i


@pytest.fixture(params=["one_pass", "two_pass"])
def build_mode(hm, request):
    """Graphs built in one pass (buffers sized by bounds) or in two (sized
    exactly after the counting pass)."""
    hm.hm_set_option(hm.HM_OPT_ONE_PASS_MAX_EDGES, (1 << 20) if request.param == "one_pass" else 0)
    yield request.param
    hm.hm_set_option(hm.HM_OPT_ONE_PASS_MAX_EDGES, 1 << 20)


@pytest.mark.parametrize("seed", range(6))
def test_build_modes_match_oracle(hm, build_mode, seed):
    h = W.random_small(500 + seed, 20 + 9 * seed, 100 + 90 * seed, {1: 0.05, 2: 0.5, 3: 0.3, 4: 0.1, 5: 0.05},
                       allow_dups=True)
    nh = core.normalise(h)
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        st = g.stats()
        assert (st["n2"], st["n3"], st["n4"]) == (nh.count(2), nh.count(3), nh.count(4))
        for j in (2, 3, 4):
            assert np.array_equal(g.export(j).astype(np.int64), nh.edges(j))
        for k in (3, 4):
            assert np.array_equal(hm.count_exact(g, k).cpu().numpy(), core.count_exact(h, k)), k
        est, _ = hm.count_sampled(g, 4, 0.5, 3)
        assert np.isfinite(est.cpu().numpy()).all()


@pytest.mark.parametrize("edges,n", [([[0, 1], [2, 2]], 3), ([[0, 7]], 3), ([[0, 1], [1, 2, 9]], 4)])
def test_build_modes_reject_invalid_input(hm, build_mode, edges, n):
    h = W.from_lists(edges, n)
    with pytest.raises(hm.HMError) as e:
        hm.hm_graph_create(h.members, h.offsets, n)
    assert e.value.code == -1
    # the library is still usable afterwards
    ok = W.random_small(7, 12, 40, {2: 0.6, 3: 0.4})
    with hm.hm_graph_create(ok.members, ok.offsets, ok.n_nodes) as g:
        assert np.array_equal(hm.count_exact(g, 4).cpu().numpy(), core.count_exact(ok, 4))


def test_one_pass_option_bounds(hm):
    with pytest.raises(hm.HMError):
        hm.hm_set_option(hm.HM_OPT_ONE_PASS_MAX_EDGES, (1 << 20) + 1)
    with pytest.raises(hm.HMError):
        hm.hm_set_option(hm.HM_OPT_ONE_PASS_MAX_EDGES, -1)
    assert hm.hm_get_option(hm.HM_OPT_ONE_PASS_MAX_EDGES) == 1 << 20


def test_wide_bit_rows(hm):
    """More than 64 words per bit row (N > 2048): the word loop of the pairs-only kernel."""
    base = W.random_small(3000, 80, 900, {2: 0.6, 3: 0.3, 4: 0.1})
    ids = np.sort(np.random.default_rng(9).choice(8000, size=80, replace=False))
    h = W.Hypergraph(8000, ids[base.members.astype(np.int64)].astype(np.uint32), base.offsets.copy())
    for k in (3, 4):
        assert np.array_equal(_gpu_counts(hm, h, k), core.count_exact(h, k)), k


def test_bit_row_option_bounds(hm):
    with pytest.raises(hm.HMError):
        hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8193)
    with pytest.raises(hm.HMError):
        hm.hm_set_option(99, 0)


def _hub_hypergraph(seed=11, n=150):
    """Hubs 0 and 1 with more than 64 pairwise neighbours each, the pair {0, 1}
    in 99 3-node hyperedges and {0, 2} in 38, and the 3-node hyperedge
    {0, 1, 2} inside 88 4-node hyperedges, over random background hyperedges:
    the exact step without bit rows meets lists both short enough to hold in
    LDS and too long to."""
    rng = np.random.default_rng(seed)
    E = set()

    def add(t):
        E.add(tuple(sorted(int(x) for x in t)))

    def count(k):
        return sum(1 for e in E if len(e) == k)

    for y in range(2, 91):
        add((0, y))
        add((1, y))
    while count(2) < 700:
        add(rng.choice(n, 2, replace=False))
    for y in range(2, 101):
        add((0, 1, y))
    for y in range(3, 41):
        add((0, 2, y))
    target = count(3) + 300
    while count(3) < target:
        add(rng.choice(n, 3, replace=False))
    for y in range(3, 91):
        add((0, 1, 2, y))
    target = count(4) + 200
    while count(4) < target:
        add(rng.choice(n, 4, replace=False))
    return W.from_lists([list(e) for e in sorted(E)], n)


@pytest.mark.parametrize("bit_rows", [True, False], ids=["bits", "hash"])
def test_hub_lists_match_oracle(hm, bit_rows):
    h = _hub_hypergraph()
    for k in (3, 4):
        assert np.array_equal(_gpu_counts(hm, h, k, bit_rows), core.count_exact(h, k)), k


@pytest.fixture
def hub_rows(hm):
    """Dense adjacency rows for every node with at least 2 pairwise
    neighbours, so that the bit-free kernels read rows instead of probing."""
    hm.hm_set_option(hm.HM_OPT_HUB_MIN_DEGREE, 2)
    try:
        yield
    finally:
        hm.hm_set_option(hm.HM_OPT_HUB_MIN_DEGREE, 256)


def test_hub_rows_match_oracle(hm, hub_rows):
    h = _hub_hypergraph()
    assert np.array_equal(_gpu_counts(hm, h, 4, bit_rows=False), core.count_exact(h, 4))
    h = W.scaled_communication(0.004, 0)
    assert np.array_equal(_gpu_counts(hm, h, 4, bit_rows=False), _golden("communication_scaled_0.004", 4))
    for seed in range(6):
        h = W.random_small(7100 + seed, 30 + 9 * seed, 200 + 60 * seed, {2: 0.5, 3: 0.35, 4: 0.15})
        assert np.array_equal(_gpu_counts(hm, h, 4, bit_rows=False), core.count_exact(h, 4)), seed


def test_hub_option_bounds(hm):
    with pytest.raises(hm.HMError):
        hm.hm_set_option(hm.HM_OPT_HUB_MIN_DEGREE, -1)
    with pytest.raises(hm.HMError):
        hm.hm_set_option(hm.HM_OPT_HUB_MIN_DEGREE, 1 << 32)
    assert hm.hm_get_option(hm.HM_OPT_HUB_MIN_DEGREE) == 256


def test_concurrent_threads_own_streams(hm):
    """Graphs built and counted from several host threads at once, each on its
    own stream, as the benchmark's throughput measurement runs them: every
    count equals the stored oracle counts, and an invalid input on one thread
    fails there alone with its own message."""
    import threading
    import torch
    dev = torch.device("cuda:0")
    h = W.cfg1_facetoface_k4(0)
    want = _golden("facetoface_N400_E30000", 4)
    members = torch.from_numpy(h.members.astype(np.int32)).to(dev)
    offsets = torch.from_numpy(h.offsets.astype(np.int64)).to(dev)
    bad = members.clone()
    bad[5] = h.n_nodes   # a node id out of range
    n_threads, per = 3, 12
    results, errors = {}, []

    def worker(t):
        try:
            torch.cuda.set_device(dev)
            st = torch.cuda.Stream()
            out = []
            for i in range(per):
                if t == 2 and i % 4 == 1:
                    with pytest.raises(hm.HMError, match="node id"):
                        hm.hm_graph_create(bad, offsets, h.n_nodes, stream=st)
                    continue
                with hm.hm_graph_create(members, offsets, h.n_nodes, stream=st) as g:
                    c = hm.count_exact(g, 4, stream=st)
                st.synchronize()
                out.append(c.cpu().numpy())
            results[t] = out
        except BaseException as e:
            errors.append(e)

    th = [threading.Thread(target=worker, args=(t,)) for t in range(n_threads)]
    for x in th:
        x.start()
    for x in th:
        x.join()
    assert not errors, errors[0]
    assert sorted(results) == list(range(n_threads))
    for t, out in results.items():
        assert len(out) == (per - 3 if t == 2 else per)
        for c in out:
            assert np.array_equal(c, want), t


@pytest.mark.parametrize("bit_rows", [True, False], ids=["bits", "hash"])
@pytest.mark.parametrize("tag_bits", [0, 1, -1, 32])
def test_duplicate_search_paths(hm, tag_bits, bit_rows):
    """The build's duplicate search.  With 0 tag bits every probe meets the
    first entry on its way, with 1 about half the meetings are of different
    hyperedges: the build finds them one launch later and repeats the search
    exactly.  -1 takes the exact search from the start, 32 is the default.
    Strata, singleton and duplicate counts and the order-4 counts equal the
    oracle's either way."""
    hm.hm_set_option(hm.HM_OPT_DEDUP_TAG_BITS, tag_bits)
    hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192 if bit_rows else 0)
    try:
        for seed in range(6):
            h = W.random_small(500 + seed, 40, 100 + 60 * seed, {1: 0.05, 2: 0.45, 3: 0.3, 4: 0.15, 5: 0.05},
                               allow_dups=True)
            nh = core.normalise(h)
            with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
                st = g.stats()
                assert (st["n2"], st["n3"], st["n4"]) == (nh.count(2), nh.count(3), nh.count(4)), seed
                assert st["singletons"] == nh.n_dropped_singletons and st["duplicates"] == nh.n_duplicates, seed
                for j in (2, 3, 4):
                    assert np.array_equal(g.export(j).astype(np.int64), nh.edges(j)), (seed, j)
                assert np.array_equal(hm.count_exact(g, 4).cpu().numpy(), core.count_exact(h, 4)), seed
    finally:
        hm.hm_set_option(hm.HM_OPT_DEDUP_TAG_BITS, 32)
        hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192)


def test_invalid_input_then_valid_same_size(hm):
    """A build that fails validation leaves its duplicate-search table
    unreturned to the all-ones state; the next build of the same size must
    not take it for a clean one.  Alternating invalid and valid builds of one
    size keeps giving the oracle's counts."""
    h = W.random_small(77, 50, 400, {2: 0.5, 3: 0.3, 4: 0.2}, allow_dups=True)
    want = core.count_exact(h, 4)
    bad = h.members.copy()
    bad[3] = h.n_nodes
    for _ in range(4):
        with pytest.raises(hm.HMError, match="node id"):
            hm.hm_graph_create(bad, h.offsets, h.n_nodes)
        with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
            assert np.array_equal(hm.count_exact(g, 4).cpu().numpy(), want)


def _device_graphs(hs):
    import torch
    dev = torch.device("cuda:0")
    return [(torch.from_numpy(h.members.astype(np.int32)).to(dev), torch.from_numpy(h.offsets.astype(np.int64)).to(dev),
             h.n_nodes) for h in hs]


@pytest.mark.parametrize("workers", [1, 3, 8])
def test_count_exact_many_matches_oracle(hm, workers):
    """Many hypergraphs in one call, shared among worker threads with a
    stream each: every row equals the oracle's counts of its hypergraph
    (different sizes, repeated hyperedges and singletons)."""
    hs = [W.random_small(900 + s, 10 + 9 * s, 40 + 50 * s, {1: 0.05, 2: 0.45, 3: 0.3, 4: 0.15, 5: 0.05},
                         allow_dups=True) for s in range(12)]
    # and the degenerate cases: no hyperedge, singletons only, one pair
    hs += [W.Hypergraph(7, np.zeros(0, np.uint32), np.zeros(1, np.uint64)),
           W.Hypergraph(5, np.array([0, 3, 4], np.uint32), np.array([0, 1, 2, 3], np.uint64)),
           W.Hypergraph(4, np.array([1, 2], np.uint32), np.array([0, 2], np.uint64))]
    graphs = _device_graphs(hs)
    for k in (3, 4):
        got = hm.count_exact_many(graphs, k, workers=workers).cpu().numpy()
        assert got.shape == (len(hs), hm.hm_num_classes(k))
        for g, h in enumerate(hs):
            assert np.array_equal(got[g], core.count_exact(h, k)), (k, g)


def test_count_exact_many_benchmark_workload(hm):
    """The benchmark's workload 24 times over in one call, three workers:
    every row equals the stored oracle counts."""
    h = W.cfg1_facetoface_k4(0)
    got = hm.count_exact_many(_device_graphs([h]) * 24, 4, workers=3).cpu().numpy()
    want = _golden("facetoface_N400_E30000", 4)
    for g in range(24):
        assert np.array_equal(got[g], want), g


@pytest.mark.parametrize("workers", [1, 3])
def test_count_exact_many_reports_the_failing_graph(hm, workers):
    """An invalid hypergraph among valid ones: the call fails with the
    hypergraph's index and its validation message, and the next call on valid
    input counts as before."""
    good = W.random_small(31, 30, 200, {2: 0.5, 3: 0.3, 4: 0.2}, allow_dups=True)
    bad_members = good.members.copy()
    bad_members[7] = good.n_nodes
    bad = W.Hypergraph(good.n_nodes, bad_members, good.offsets)
    graphs = _device_graphs([good, good, good, bad, good, good])
    with pytest.raises(hm.HMError, match="hypergraph 3: .*node id"):
        hm.count_exact_many(graphs, 4, workers=workers)
    got = hm.count_exact_many(_device_graphs([good] * 4), 4, workers=workers).cpu().numpy()
    for g in range(4):
        assert np.array_equal(got[g], core.count_exact(good, 4))


def test_count_exact_many_host_memory(hm):
    """count_exact_many with the hypergraphs in host memory (HM_MEM_HOST),
    called through the C ABI: each worker copies its graphs' arrays to the
    device on its own stream; every row equals the oracle's counts."""
    import ctypes
    import torch
    hs = [W.random_small(700 + s, 15 + 7 * s, 60 + 40 * s, {2: 0.5, 3: 0.3, 4: 0.2}, allow_dups=True)
          for s in range(9)]
    n = len(hs)
    C = hm.hm_num_classes(4)
    out = torch.empty((n, C), dtype=torch.int64, device="cuda")
    mp, op = (ctypes.c_void_p * n)(), (ctypes.c_void_p * n)()
    ne, nm, nn = (ctypes.c_uint64 * n)(), (ctypes.c_uint64 * n)(), (ctypes.c_uint32 * n)()
    for g, h in enumerate(hs):
        mp[g], op[g] = h.members.ctypes.data, h.offsets.ctypes.data
        ne[g], nm[g], nn[g] = h.n_edges, len(h.members), h.n_nodes
    st = torch.cuda.current_stream()
    rc = hm.lib().count_exact_many(n, mp, op, ne, nm, nn, hm.binding.HM_MEM_HOST, 4, ctypes.c_void_p(out.data_ptr()),
                                   4, ctypes.c_void_p(st.cuda_stream))
    assert rc == 0, hm.lib().hm_last_error().decode()
    got = out.cpu().numpy()
    for g, h in enumerate(hs):
        assert np.array_equal(got[g], core.count_exact(h, 4)), g


def test_count_exact_many_repeats_the_duplicate_search(hm):
    """With no tag bits every build's one-launch duplicate search meets
    different hyperedges and is repeated exactly, here inside the worker
    threads of count_exact_many: the rows still equal the oracle's counts."""
    hs = [W.random_small(610 + s, 25 + 5 * s, 150 + 40 * s, {1: 0.05, 2: 0.5, 3: 0.3, 4: 0.15}, allow_dups=True)
          for s in range(6)]
    hm.hm_set_option(hm.HM_OPT_DEDUP_TAG_BITS, 0)
    try:
        got = hm.count_exact_many(_device_graphs(hs), 4, workers=3).cpu().numpy()
    finally:
        hm.hm_set_option(hm.HM_OPT_DEDUP_TAG_BITS, 32)
    for g, h in enumerate(hs):
        assert np.array_equal(got[g], core.count_exact(h, 4)), g


def _hub_graph(n, hubs, hub_degree, ring, clique, seed):
    """Pairs only: a ring-like sparse part, `hubs` nodes of high degree, and a complete graph on `clique` nodes."""
    rng = np.random.default_rng(seed)
    parts = []
    if ring:
        v = np.arange(n)
        parts += [np.stack([v, (v + 1) % n], 1), np.stack([v, (v + 7) % n], 1)]
    for h in range(hubs):
        parts.append(np.stack([np.full(hub_degree, h), rng.choice(np.arange(hubs, n), hub_degree, replace=False)], 1))
    if hubs > 1:
        a, b = np.triu_indices(hubs, 1)
        parts.append(np.stack([a, b], 1))
    if clique:
        nodes = rng.choice(n, clique, replace=False)
        a, b = np.triu_indices(clique, 1)
        parts.append(np.stack([nodes[a], nodes[b]], 1))
    e = np.sort(np.concatenate(parts), axis=1)
    e = np.unique(e[e[:, 0] != e[:, 1]], axis=0)
    return e


def _pair_shape_counts(hm, e, n):
    """Non-induced copies of the pair shapes of order 3 and 4 (but 4-cliques), from sparse matrix products."""
    import scipy.sparse as sp
    A = sp.csr_matrix((np.ones(2 * len(e), np.int64), (np.r_[e[:, 0], e[:, 1]], np.r_[e[:, 1], e[:, 0]])), shape=(n, n))
    d = np.asarray(A.sum(1)).ravel()
    C = (A @ A).tocoo()
    off = C.row < C.col
    cyc2 = int((C.data[off] * (C.data[off] - 1) // 2).sum())
    T = (A @ A).multiply(A).tocoo()
    up = T.row < T.col
    t, a, b = T.data[up], T.row[up], T.col[up]
    tri = int(t.sum()) // 3
    du, dv = d[e[:, 0]], d[e[:, 1]]
    return {"tri": tri, "cyc": cyc2 // 2, "dia": int((t * (t - 1) // 2).sum()), "paw": int((t * (d[a] + d[b] - 4)).sum()) // 2,
            "p4": int(((du - 1) * (dv - 1)).sum()) - 3 * tri, "star": int((d * (d - 1) * (d - 2) // 6).sum())}


def test_walks_over_several_rank_ranges(hm):
    """More than 51,200 nodes of degree two and above, and hubs whose walks
    exceed the hash tables: the six pairs-only shapes against matrix products
    in int64 (order 3 too)."""
    n = 130_000
    e = _hub_graph(n, 4, 3000, True, 0, 5)
    want = _pair_shape_counts(hm, e, n)
    offsets = np.arange(0, 2 * len(e) + 1, 2, dtype=np.uint64)
    with hm.hm_graph_create(e.astype(np.uint32).ravel(), offsets, n) as g:
        got = hm.count_exact(g, 4).cpu().numpy()
        got3 = hm.count_exact(g, 3).cpu().numpy()
    cls = lambda *bits: hm.hm_pattern_class(4, sum(1 << b for b in bits))
    path, star, cycle = got[cls(0, 2, 7)], got[cls(0, 1, 4)], got[cls(0, 2, 7, 4)]
    paw, dia, k4 = got[cls(0, 1, 2, 4)], got[cls(0, 1, 2, 4, 5)], got[cls(0, 1, 2, 4, 5, 7)]
    assert dia + 6 * k4 == want["dia"]
    assert cycle + dia + 3 * k4 == want["cyc"]
    assert paw + 4 * dia + 12 * k4 == want["paw"]
    assert star + paw + 2 * dia + 4 * k4 == want["star"]
    assert path + 4 * cycle + 2 * paw + 6 * dia + 12 * k4 == want["p4"]
    assert got3[hm.hm_pattern_class(3, 7)] == want["tri"]
    assert k4 >= 1 and got.sum() == path + star + cycle + paw + dia + k4


@pytest.mark.parametrize("degree", [14, 15, 16, 17])
def test_paths_of_every_neighbour(hm, degree):
    """Nodes whose every neighbour is the hub's too, of degrees around the 15
    paths that a count of four bits holds, among more than 51,200 others:
    4-cycles against matrix products."""
    n, spokes, ends = 110_000, 3400, 300
    rng = np.random.default_rng(degree)
    x = 1 + np.arange(spokes)
    w = spokes + 1 + np.arange(ends)
    ring = np.arange(w[-1] + 1, n)
    pairs = [np.stack([np.zeros(spokes, int), x], 1), np.stack([ring[:-1], ring[1:]], 1), [[ring[0], ring[-1]]]]
    pairs += [np.stack([rng.choice(x, degree, replace=False), np.full(degree, v)], 1) for v in w]
    e = np.sort(np.concatenate(pairs), axis=1)
    want = _pair_shape_counts(hm, e, n)
    with hm.hm_graph_create(e.astype(np.uint32).ravel(), np.arange(0, 2 * len(e) + 1, 2, dtype=np.uint64), n) as g:
        got = hm.count_exact(g, 4).cpu().numpy()
        raw = hm.count_sampled_indices(g, 4, {2: np.arange(len(e))})[1].cpu().numpy()
    cls = lambda *bits: hm.hm_pattern_class(4, sum(1 << b for b in bits))
    assert want["tri"] == 0 and got[cls(0, 2, 7, 4)] == want["cyc"] > ends * degree * (degree - 1) // 2 - 1
    assert raw[cls(0, 2, 7, 4)] == 4 * want["cyc"]   # (each of its pairs finds a cycle)


@pytest.mark.parametrize("n,hubs,hub_degree,ring,clique", [
    (200, 0, 0, True, 0), (4000, 40, 3700, True, 0), (3000, 3, 2900, True, 0), (3000, 40, 700, True, 66), (1500, 0, 0, False, 24),
    (2000, 2, 500, True, 120), (2500, 0, 0, True, 700)])
def test_walks_match_bit_rows(hm, n, hubs, hub_degree, ring, clique):
    """Triangles, 4-cycles and 4-cliques without bit rows (hash tables of
    every size, counters by rank, walks split into shares, cliques of one word, of many and beyond the
    LDS matrix) against the bit-row path; and the per-pair statistics through
    samples of every kind of pair."""
    e = _hub_graph(n, hubs, hub_degree, ring, clique, n + clique)
    rng = np.random.default_rng(1)
    tri = np.sort(rng.choice(n, (300, 3)), axis=1)
    tri = tri[(tri[:, 0] < tri[:, 1]) & (tri[:, 1] < tri[:, 2])]
    members = np.r_[e.ravel(), tri.ravel()].astype(np.uint32)
    offsets = np.r_[np.arange(0, 2 * len(e), 2), 2 * len(e) + np.arange(0, 3 * len(tri) + 1, 3)].astype(np.uint64)
    got = {}
    for bits in (8192, 0):
        hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, bits)
        try:
            with hm.hm_graph_create(members, offsets, n) as g:
                idx = rng.integers(0, g.stats()["n2"], 200) if not got else idx
                raw = hm.count_sampled_indices(g, 4, {2: idx})[1].cpu().numpy()
                got[bits] = (hm.count_exact(g, 4).cpu().numpy(), hm.count_exact(g, 3).cpu().numpy(), raw)
        finally:
            hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192)
    for b, h in zip(got[8192], got[0]):
        assert np.array_equal(b, h)


@pytest.mark.parametrize("hub_min_degree", [0, 16, 2048])
@pytest.mark.parametrize("n,run,pairs", [(40, 12, 300), (1200, 700, 15000), (1200, 700, 300), (2500, 2, 4000)])
def test_triples_match_bit_rows(hm, n, run, pairs, hub_min_degree):
    """Sets around 3-node hyperedges without bit rows (pair runs of two entries
    up to more than a list that is searched, walked or looked up from the third
    node's lists, alone among many runs of one entry, with and without dense
    rows) against the bit-row path."""
    rng = np.random.default_rng(n + run + pairs)
    def distinct(k, m):
        s = np.sort(rng.choice(n, (m, k)), axis=1)
        return s[(s[:, 1:] > s[:, :-1]).all(axis=1)]
    third = np.sort(rng.choice(np.arange(3, n), run, replace=False))
    with_pair = lambda a, b, t: np.sort(np.c_[np.full(len(t), a), np.full(len(t), b), t], axis=1)
    e3 = np.r_[with_pair(0, 1, third), with_pair(0, 2, third[::2]), with_pair(1, int(third[0]), third[1::2]),
               with_pair(n - 1, int(third[-1]), np.setdiff1d(third[:-1:3], [n - 1])), distinct(3, 200)]
    e3 = e3[(e3[:, 0] < e3[:, 1]) & (e3[:, 1] < e3[:, 2])]
    e4 = np.r_[np.sort(np.c_[np.zeros(len(third) // 2, int), np.ones(len(third) // 2, int), third[:-1:2], third[1::2]], axis=1),
               distinct(4, 100)]
    # the whole of a few nodes, so that rows of every kind meet the runs
    hub = np.sort(np.array([(h, t) for h in (0, 1, 2, int(third[0])) for t in range(n) if t != h and rng.random() < 0.8]), axis=1)
    e2 = np.r_[distinct(2, pairs), hub]
    members = np.r_[e2.ravel(), e3.ravel(), e4.ravel()].astype(np.uint32)
    sizes = np.r_[np.full(len(e2), 2), np.full(len(e3), 3), np.full(len(e4), 4)]
    offsets = np.r_[0, np.cumsum(sizes)].astype(np.uint64)
    keep = hm.hm_get_option(hm.HM_OPT_HUB_MIN_DEGREE)
    got = {}
    try:
        hm.hm_set_option(hm.HM_OPT_HUB_MIN_DEGREE, hub_min_degree)
        for bits in (8192, 0):
            hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, bits)
            with hm.hm_graph_create(members, offsets, n) as g:
                got[bits] = hm.count_exact(g, 4).cpu().numpy()
    finally:
        hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192)
        hm.hm_set_option(hm.HM_OPT_HUB_MIN_DEGREE, keep)
    assert np.array_equal(got[8192], got[0])


@functools.lru_cache(maxsize=1)
def _large_input():
    """560,000 hyperedges of 1 to 100 nodes and two of 9,000 (one
    ascending, one not), some of them repeated in other orders; and what a set
    of sorted members keeps of them."""
    n, m = 20_000, 560_000
    rng = np.random.default_rng(5)
    size = np.minimum(1 + rng.geometric(0.5, m), 8)
    some = rng.choice(m, 4000, replace=False)
    size[some] = rng.integers(1, 101, some.size)
    size[[1234, 400_000]] = 9000
    # small hyperedges among 250 nodes (many alike), larger ones among as many
    # of 80 groups
    rows = {s: np.argsort(rng.random((k, 250)), axis=1)[:, :s] if s > 8 else rng.integers(0, 250 // s, (k, s)) * s + rng.permutation(s)
            for s, k in zip(*np.unique(size[size <= 100], return_counts=True))}
    edges = [None] * m
    for s, r in rows.items():
        r = r + (250 * rng.integers(0, 80, len(r))[:, None] if s > 3 else 0)
        for i, e in zip(np.nonzero(size == s)[0], r):
            edges[i] = e
    for i in (1234, 400_000):
        e = rng.permutation(n)[:9000]
        edges[i] = np.sort(e) if i == 1234 else e
    edges[300_000] = edges[1234][::-1]
    edges[500_000] = np.roll(edges[400_000], 77)
    for i in some[:500]:
        edges[(i * 7919) % m] = edges[i][::-1]
    offsets = np.r_[0, np.cumsum([len(e) for e in edges])].astype(np.uint64)
    members = np.concatenate(edges).astype(np.uint32)
    first, strata, singles, dups = set(), {2: [], 3: [], 4: []}, 0, 0
    for e in edges:
        if len(e) == 1:
            singles += 1
            continue
        t = tuple(sorted(e.tolist()))
        if t in first:
            dups += 1
            continue
        first.add(t)
        if len(t) <= 4:
            strata[len(t)].append(t)
    want = (singles, dups, len(first), sum(map(len, first)))
    return n, members, offsets, want, {j: np.array(x, dtype=np.uint32) for j, x in strata.items()}


@pytest.mark.parametrize("tag_bits", [32, 0, -1])
def test_large_build(hm, tag_bits):
    """The build of a large input without bit rows (tiles of hyperedges of every
    size class, and beyond the LDS staging); also with hashes cut so that
    different hyperedges meet, and by the exact search.  An invalid hyperedge
    far in is still named."""
    n, members, offsets, want, strata = _large_input()
    hm.hm_set_option(hm.HM_OPT_DEDUP_TAG_BITS, tag_bits)
    try:
        with hm.hm_graph_create(members, offsets, n) as g:
            st = g.stats()
            assert (st["singletons"], st["duplicates"], st["n_unique"], st["n_unique_members"]) == want
            for j in (2, 3, 4):
                assert np.array_equal(g.export(j), strata[j]), j
        members = members.copy()
        members[int(offsets[450_000])] = n
        with pytest.raises(hm.HMError, match="node id.*450000"):
            hm.hm_graph_create(members, offsets, n)
    finally:
        hm.hm_set_option(hm.HM_OPT_DEDUP_TAG_BITS, 32)


@pytest.mark.parametrize("n,pairs,hubs", [(2574, 100_000, 0), (2575, 40_000, 0), (2575, 60_000, 0), (2575, 60_000, 6),
                                          (2575, 100_000, 0), (8192, 30_000, 10)])
def test_count_beyond_identities_matches_noalloc(hm, n, pairs, hubs):
    """Graphs with bit rows on both sides of the identity route's end, of few
    pairs, of more with even degrees and with hubs, and of many: count_exact,
    by either way, against the count that always takes the bit rows, on a first
    call, a second one and after samples."""
    rng = np.random.default_rng(n + pairs + hubs)
    e2 = np.r_[rng.integers(0, n, (pairs, 2)), np.c_[np.arange(hubs * (n // 2)) % max(hubs, 1), rng.integers(1, n, hubs * (n // 2))]]
    e3 = np.r_[rng.integers(0, n, (n, 3)), np.c_[rng.integers(0, 12, (n, 2)), rng.integers(0, n, n)]]
    e4 = np.r_[rng.integers(0, n, (n // 2, 4)), np.c_[rng.integers(0, 12, (n // 4, 3)), rng.integers(0, n, n // 4)]]
    parts = [np.sort(e, axis=1) for e in (e2, e3, e4)]
    parts = [e[(e[:, 1:] > e[:, :-1]).all(axis=1)] for e in parts]
    members = np.concatenate([e.ravel() for e in parts]).astype(np.uint32)
    offsets = np.r_[0, np.cumsum(np.concatenate([np.full(len(e), e.shape[1]) for e in parts]))].astype(np.uint64)

    def by_bit_rows(g):
        import ctypes
        import torch
        out = torch.empty(hm.hm_num_classes(4), dtype=torch.int64, device="cuda")
        assert hm.lib().count_exact_noalloc(g.handle, 4, ctypes.c_void_p(out.data_ptr()), None) == 0
        torch.cuda.synchronize()
        return out.cpu().numpy()

    with hm.hm_graph_create(members, offsets, n) as g:
        want = by_bit_rows(g)
        first = hm.count_exact(g, 4).cpu().numpy()
        idx = {j: rng.integers(0, g.stats()["n%d" % j], 50) for j in (2, 3, 4)}
        raw = hm.count_sampled_indices(g, 4, idx)[1].cpu().numpy()
        second = hm.count_exact(g, 4).cpu().numpy()
        third = by_bit_rows(g)
        assert np.array_equal(raw, hm.count_sampled_indices(g, 4, idx)[1].cpu().numpy())
    for got in (first, second, third):
        assert np.array_equal(got, want)


@pytest.mark.parametrize("n,missing", [(34, 0.0), (67, 0.0), (90, 0.2)])
def test_dense_pairs_match_oracle(hm, n, missing):
    """Pairs with up to more common neighbours than a wavefront, or half of
    one, has lanes, beside 3- and 4-node hyperedges: one graph's count and the
    count of configuration copies (whose real counts take the same kernels)
    against the oracle."""
    rng = np.random.default_rng(n)
    a, b = np.triu_indices(n, 1)
    keep = rng.random(len(a)) >= missing
    parts = [np.c_[a, b][keep], rng.integers(0, n, (3 * n, 3)), rng.integers(0, n, (n, 4))]
    parts = [np.sort(e, axis=1) for e in parts]
    parts = [e[(e[:, 1:] > e[:, :-1]).all(axis=1)] for e in parts]
    members = np.concatenate([e.ravel() for e in parts]).astype(np.uint32)
    offsets = np.r_[0, np.cumsum(np.concatenate([np.full(len(e), e.shape[1]) for e in parts]))].astype(np.uint64)
    want = core.count_exact(W.Hypergraph(n, members, offsets), 4)
    with hm.hm_graph_create(members, offsets, n) as g:
        assert np.array_equal(hm.count_exact(g, 4).cpu().numpy(), want)
        nulls = hm.count_nulls_model(g, 4, 2, hm.HM_NULL_CONFIG, 1, 9)[1].cpu().numpy()
        m, o = hm.hm_null_export_model(g, hm.HM_NULL_CONFIG, 1, 9, 1)
        assert np.array_equal(nulls[1], core.count_exact(W.Hypergraph(n, m, o), 4))


def test_order4_node_range(hm):
    """A pairwise graph over more than 2^31 nodes is refused at order 4, exact
    and sampled."""
    import torch
    if torch.cuda.mem_get_info()[0] < 96 << 30:
        pytest.skip("needs 96 GiB of free device memory")
    n = 2**31 + 1
    members = np.array([0, 1, 1, n - 1, 0, 5, n - 1], dtype=np.uint32)
    offsets = np.array([0, 2, 4, 7], dtype=np.uint64)
    with hm.hm_graph_create(members, offsets, n) as g:
        for call in (lambda: hm.count_exact(g, 4), lambda: hm.count_sampled(g, 4, 1.0, 1)):
            with pytest.raises(hm.HMError, match="2\\^31") as e:
                call()
            assert e.value.code == hm.binding.HM_EUNSUPPORTED


@pytest.mark.parametrize("n,pairs,probes", [(2, 1, True), (10, 20, True), (3000, 150_000, True), (3000, 175_000, False),
                                            (300_000, 786_000, True), (300_000, 787_000, False)])
def test_order3_by_probes_and_walks(hm, n, pairs, probes):
    """Order 3 without bit rows on both sides of the lines between probes and
    walks (pairs, and pairs times degrees), and on a pair alone: the triangles
    and the paths against matrix products."""
    rng = np.random.default_rng(n)
    e = np.sort(rng.integers(0, n, (pairs + pairs // 3 + 40, 2)), axis=1)
    e = np.unique(e[e[:, 0] < e[:, 1]], axis=0)
    if n > 3000:   # closing some wedges of a hub
        e = np.unique(np.r_[np.c_[np.zeros(5000, int), 1 + np.arange(5000)], np.c_[1 + np.arange(4999), 2 + np.arange(4999)], e], axis=0)
    e = np.concatenate([e[:1] * 0 + [0, 1], e]) if n == 2 else e
    e = np.unique(e, axis=0)
    e = e[np.sort(rng.permutation(len(e))[:pairs])]
    d = np.bincount(e.ravel(), minlength=n)
    import scipy.sparse as sp
    A = sp.csr_matrix((np.ones(2 * len(e), np.int64), (np.r_[e[:, 0], e[:, 1]], np.r_[e[:, 1], e[:, 0]])), shape=(n, n))
    tri = int((A @ A).multiply(A).sum()) // 6
    hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 0)
    try:
        with hm.hm_graph_create(e.astype(np.uint32).ravel(), np.arange(0, 2 * len(e) + 1, 2, dtype=np.uint64), n) as g:
            hm.hm_profile_enable(True)
            hm.hm_profile_reset()
            got = hm.count_exact(g, 3).cpu().numpy()
            names = hm.hm_profile_read()
    finally:
        hm.hm_profile_enable(False)
        hm.hm_profile_reset()
        hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192)
    assert ("k_sp_pair_probes" in names) == probes and ("k_walk" in names) != probes
    assert got[hm.hm_pattern_class(3, 7)] == tri and got[hm.hm_pattern_class(3, 3)] == int((d * (d - 1) // 2).sum()) - 3 * tri
    assert n < 100 or tri > 0


@pytest.mark.parametrize("sizes", [(65, 511, 512), (513, 700, 1025), (2048, 2049, 6000), (6145, 70), (20_000, 513)])
def test_long_hyperedges_of_large_builds(hm, sizes):
    """Hyperedges of more than 64 nodes where graphs are built without bit
    rows, in LDS and beyond it: any order of a hyperedge's members is the same
    hyperedge, a changed member another one, and repeats and ids out of range
    are found wherever they stand.  A nearly ascending one is not much slower
    than an ascending one."""
    import time
    import torch
    n = 30_000
    rng = np.random.default_rng(sizes[0])
    edges, unique = [], 0
    for s in sizes:
        e = np.sort(rng.permutation(n - 1)[:s])
        swapped = e.copy()
        swapped[[s // 2, s // 2 + 1]] = swapped[[s // 2 + 1, s // 2]]
        other = e.copy()
        other[-1] = n - 1
        edges += [e, swapped, e[::-1], np.r_[e[-1], e[:-1]], np.r_[e[1:], e[0]], rng.permutation(e), other, rng.permutation(other)]
        unique += 2

    def build(edges):
        offsets = np.r_[0, np.cumsum([len(e) for e in edges])].astype(np.uint64)
        return hm.hm_graph_create(np.concatenate(edges).astype(np.uint32), offsets, n)

    for order in (range(len(edges)), rng.permutation(len(edges))):
        with build([edges[i] for i in order] + [np.array([0, 1])]) as g:
            st = g.stats()
            assert (st["n_unique"], st["duplicates"]) == (unique + 1, len(edges) - unique)
            assert st["n_unique_members"] == 2 * sum(sizes) + 2
    s = sizes[0]
    for at in (0, s // 2, s - 1):
        for value, message in ((edges[0][(at + 7) % s], "repeated"), (n, "node id")):
            bad = rng.permutation(edges[0])
            bad[at] = value if value == n else bad[(at + 7) % s]
            with pytest.raises(hm.HMError, match=message):
                build([edges[1], bad])
    took = {}
    for name, e in (("ascending", edges[0]), ("nearly", edges[1])):
        build([e, np.array([0, 1])])
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(3):
            build([e, np.array([0, 1])])
        torch.cuda.synchronize()
        took[name] = (time.perf_counter() - t) / 3
    assert took["nearly"] < took["ascending"] + 0.05, took


@pytest.mark.parametrize("leaves", [65_535, 65_536, 70_000])
def test_walks_beyond_every_table(hm, leaves):
    """Three hubs over the same tens of thousands of nodes of a ring of
    900,000: 4-cycle counts around the 65,535 paths that 16 bits hold, more
    ranks than one range of any table, more marked values than one window.
    Exact counts at orders 3 and 4 and the sampled pairs of a hub in closed
    form."""
    ring, hubs = 900_000, 3
    n = ring + hubs
    v = np.arange(ring)
    leaf = 12 * np.arange(leaves)
    chord = np.arange(850_000, 890_000, 5)   # (each closes one triangle with the ring)
    e = np.concatenate([np.stack([v, (v + 1) % ring], 1), np.stack([chord, chord + 2], 1)] +
                       [np.stack([leaf, np.full(leaves, ring + h)], 1) for h in range(hubs)])
    e = np.sort(e, axis=1)
    d = np.bincount(e.ravel(), minlength=n).astype(np.int64)
    du, dv = d[e[:, 0]], d[e[:, 1]]
    in_tri = np.zeros(len(e), bool)
    in_tri[chord] = in_tri[chord + 1] = in_tri[ring:ring + len(chord)] = True
    tri = len(chord)
    pairs = lambda x: x * (x - 1) // 2
    cyc = hubs * (hubs - 1) // 2 * pairs(leaves)
    paw = int((du + dv - 4)[in_tri].sum()) // 2
    star = int((d * (d - 1) * (d - 2) // 6).sum()) - paw
    path = int(((du - 1) * (dv - 1)).sum()) - 3 * tri - 4 * cyc - 2 * paw
    cls = lambda *bits: hm.hm_pattern_class(4, sum(1 << b for b in bits))
    want = np.zeros(hm.hm_num_classes(4), np.int64)
    want[cls(0, 2, 7)], want[cls(0, 1, 4)], want[cls(0, 2, 7, 4)], want[cls(0, 1, 2, 4)] = path, star, cyc, paw
    rng = np.random.default_rng(leaves)
    sample = ring + len(chord) + rng.integers(0, hubs * leaves, 200)   # pairs of a hub and a leaf
    one = np.zeros_like(want)
    one[cls(0, 2, 7, 4)] = (hubs - 1) * (leaves - 1)
    one[cls(0, 1, 4)] = pairs(leaves - 1) + pairs(hubs - 1 + 2)
    one[cls(0, 2, 7)] = 2 * (leaves - 1) + 2 + 2 * (leaves - 1)
    with hm.hm_graph_create(e.astype(np.uint32).ravel(), np.arange(0, 2 * len(e) + 1, 2, dtype=np.uint64), n) as g:
        got3 = hm.count_exact(g, 3).cpu().numpy()
        got4 = hm.count_exact(g, 4).cpu().numpy()
        raw = hm.count_sampled_indices(g, 4, {2: sample})[1].cpu().numpy()
    assert got3[hm.hm_pattern_class(3, 7)] == tri
    assert got3[hm.hm_pattern_class(3, 3)] == int(pairs(d).sum()) - 3 * tri
    assert np.array_equal(got4, want)
    assert np.array_equal(raw, 200 * one)
