"""Null model (stub matching) and z-scores through the C ABI against the oracle.

Both sides implement the same stub-matching procedure from the published
Philox4x64-10 generator, so the copies themselves must agree bit for bit, and
so must their exact counts."""
import json
import os

import numpy as np
import pytest

import workloads as W
from oracle import core, nulls

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def hm():
    import torch
    import paper_2209_10241_amd as hm
    assert torch.cuda.is_available()
    return hm


def _golden_cases():
    with open(os.path.join(ROOT, "tests", "golden", "workload_counts.json")) as f:
        return json.load(f)["cases"]


@pytest.mark.parametrize("seed", range(6))
def test_copies_match_oracle(hm, seed):
    h = W.random_small(5000 + seed, 30 + seed * 7, 150 + seed * 40, {1: 0.05, 2: 0.5, 3: 0.3, 4: 0.1, 6: 0.05},
                       allow_dups=bool(seed % 2))
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        for copy in (0, 1, 5):
            m, o = hm.hm_null_export(g, 77 + seed, copy)
            wm, wo = nulls.stub_matching(h, 77 + seed, copy)
            assert np.array_equal(o, wo)
            assert np.array_equal(m, wm), (seed, copy)
            nulls.check_null_invariants(h, m, o)


def test_facetoface_copies_match_oracle(hm):
    """Copies 0, 18 and 30 of seed 1 each hold stubs whose 64-bit keys share
    their high 32 bits (2, 4 and 3 such groups among the 86,051 stubs), so
    the device's ordering by (copy, high half) and then by the low half
    within such runs is checked against the oracle's order by the full key."""
    h = W.cfg1_facetoface_k4(0)
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        for copy in (0, 18, 30, 63):
            m, o = hm.hm_null_export(g, 1, copy)
            wm, wo = nulls.stub_matching(h, 1, copy)
            assert np.array_equal(o, wo) and np.array_equal(m, wm), copy


@pytest.mark.parametrize("k", [3, 4])
def test_counts_and_z_match_oracle(hm, k):
    h = W.random_small(5100 + k, 40, 260, {2: 0.5, 3: 0.3, 4: 0.15, 5: 0.05})
    R = 12
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        real, nl, z = hm.count_nulls(g, k, R, 4242)
        real, nl, z = real.cpu().numpy(), nl.cpu().numpy(), z.cpu().numpy()
    want_real = core.count_exact(h, k)
    want_nulls = np.array([core.count_exact(W.Hypergraph(h.n_nodes, *nulls.stub_matching(h, 4242, c)), k)
                           for c in range(R)])
    assert np.array_equal(real, want_real)
    assert np.array_equal(nl, want_nulls)
    want_z = nulls.zscores(want_real, want_nulls)
    finite = np.isfinite(want_z)
    assert np.array_equal(np.isfinite(z), finite)
    assert np.array_equal(np.sign(z[~finite]), np.sign(want_z[~finite]))
    np.testing.assert_allclose(z[finite], want_z[finite].astype(np.float32), rtol=2e-6, atol=1e-6)


def test_facetoface_64_copies(hm):
    """The batched null workload: 64 stub-matched copies of the face-to-face
    hypergraph counted at k = 4; copies 0, 1, 63 against stored oracle counts."""
    h = W.cfg1_facetoface_k4(0)
    cases = _golden_cases()
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        real, nl, z = hm.count_nulls(g, 4, 64, 1)
        real, nl, z = real.cpu().numpy(), nl.cpu().numpy(), z.cpu().numpy()
    exact = next(c for c in cases if c["workload"] == "facetoface_N400_E30000" and c["k"] == 4)
    assert np.array_equal(real, np.array(exact["counts"]))
    for c in cases:
        if c["workload"].endswith("/null"):
            assert np.array_equal(nl[c["copy"]], np.array(c["counts"])), c["copy"]
    # z is the z-score of the returned counts (property at full size)
    mu = nl.astype(np.float64).mean(axis=0)
    sd = nl.astype(np.float64).std(axis=0, ddof=1)
    ok = sd > 0
    np.testing.assert_allclose(z[ok], ((real[ok] - mu[ok]) / sd[ok]).astype(np.float32), rtol=1e-5, atol=1e-5)


def test_bad_arguments(hm):
    h = W.random_small(5200, 20, 60, {2: 0.6, 3: 0.4})
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        with pytest.raises(hm.HMError):
            hm.count_nulls(g, 4, 1, 0)
        with pytest.raises(hm.HMError):
            hm.count_nulls(g, 5, 4, 0)


def test_replay_new_seed_and_rebuild(hm):
    """The captured pipeline replays with a new seed; a different number of
    copies rebuilds it; both against the oracle."""
    h = W.random_small(5300, 35, 220, {2: 0.5, 3: 0.35, 4: 0.15})
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        for R, seed in ((6, 10), (6, 11), (9, 12), (6, 13)):
            _, nl, _ = hm.count_nulls(g, 4, R, seed)
            nl = nl.cpu().numpy()
            for c in (0, R - 1):
                want = core.count_exact(W.Hypergraph(h.n_nodes, *nulls.stub_matching(h, seed, c)), 4)
                assert np.array_equal(nl[c], want), (R, seed, c)
        sizes = hm.hm_null_tile_sizes(g)
        assert len(sizes) == 3 and min(sizes) >= 1


@pytest.mark.parametrize("bit_rows", [True, False], ids=["bits", "hash"])
def test_batched_paths_match_oracle(hm, bit_rows):
    h = W.random_small(5400, 45, 300, {2: 0.45, 3: 0.35, 4: 0.2})
    hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192 if bit_rows else 0)
    try:
        g = hm.hm_graph_create(h.members, h.offsets, h.n_nodes)
    finally:
        hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192)
    with g:
        for k in (3, 4):
            real, nl, _ = hm.count_nulls(g, k, 5, 99)
            assert np.array_equal(real.cpu().numpy(), core.count_exact(h, k))
            nl = nl.cpu().numpy()
            for c in range(5):
                want = core.count_exact(W.Hypergraph(h.n_nodes, *nulls.stub_matching(h, 99, c)), k)
                assert np.array_equal(nl[c], want), (k, c)


def test_empty_hypergraph(hm):
    h = W.from_lists([[0], [1]], 3)
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        real, nl, z = hm.count_nulls(g, 4, 3, 1)
        assert real.sum().item() == 0 and nl.sum().item() == 0 and float(z.abs().sum()) == 0.0


def _pairs(n_nodes, n_pairs, seed):
    """Hypergraph of n_pairs different pairs, in a random order."""
    rng = np.random.default_rng(seed)
    code = rng.choice(n_nodes * (n_nodes - 1) // 2, n_pairs, replace=False)
    b = ((1 + np.sqrt(1 + 8.0 * code)) / 2).astype(np.int64)
    b -= b * (b - 1) // 2 > code
    a = code - b * (b - 1) // 2
    return W.Hypergraph(n_nodes, np.c_[a, b].astype(np.uint32).ravel(),
                        np.arange(0, 2 * n_pairs + 1, 2).astype(np.uint64), name="pairs")


@pytest.mark.parametrize("n_pairs", [1, 2048, 2049, 2901, 5801, 371_200, 371_201])
def test_orders_match_oracle(hm, n_pairs):
    """Stub orders sorted by one workgroup, dealt to 2, 4 and 256 buckets, and
    by the radix sort."""
    h = _pairs(3000, n_pairs, n_pairs)
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        for copy in (0, 7):
            m, _ = hm.hm_null_export(g, 5, copy)
            assert np.array_equal(m, nulls.stub_matching(h, 5, copy)[0]), copy


@pytest.mark.parametrize("edges,sizes", [(2, (2,)), (3, (2, 3)), (4096, (2,)), (4097, (2,)), (2300, (2, 3, 4, 5)),
                                         (2400, (2, 3, 4, 5)), (6000, (2, 3))])
def test_config_rounds_match_oracle(hm, edges, sizes):
    """All rounds of a copy by one workgroup up to its largest numbers of
    hyperedges and members, and round by round beyond either."""
    from oracle import profiles
    h = W.random_small(edges, 2500, edges, {s: 1.0 for s in sizes})
    if sizes == (2,):
        h = _pairs(2500, edges, edges)
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        for sweeps, copy in ((1, 0), (3, 4)):
            m, _ = hm.hm_null_export_model(g, hm.HM_NULL_CONFIG, sweeps, 9, copy)
            assert np.array_equal(m, profiles.config_model(h, sweeps, 9, copy)[0]), (sweeps, copy)


@pytest.mark.parametrize("n,clique", [(33, 0), (500, 45), (900, 33), (1024, 40), (1025, 70)])
def test_half_wavefront_rows_match_hash(hm, n, clique):
    """Bit rows of up to 32 words, counted by halves of a wavefront, and the
    first beyond them: odd numbers of pairs and 3-node hyperedges, pairs with
    more common neighbours than a half has lanes; the hypergraph's counts and
    its copies' against the paths without bit rows."""
    rng = np.random.default_rng(n)
    rows = [tuple(p) for p in np.stack(np.triu_indices(clique, 1), 1)]
    for size, count in ((2, 3 * n), (3, 2 * n), (4, n // 2)):
        rows += [tuple(sorted(rng.choice(n // 2 if j % 2 else n, size, replace=False))) for j in range(count)]
    rows = sorted(set(rows))
    for size in (2, 3):
        if sum(len(r) == size for r in rows) % 2 == 0:
            rows.remove(next(r for r in rows if len(r) == size))
    members = np.concatenate([np.array(r, np.uint32) for r in rows])
    offsets = np.cumsum([0] + [len(r) for r in rows]).astype(np.uint64)
    got = {}
    for bits in (8192, 0):
        hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, bits)
        try:
            with hm.hm_graph_create(members, offsets, n) as g:
                real, nl, _ = hm.count_nulls(g, 4, 3, 2)
                got[bits] = (hm.count_exact(g, 4).cpu().numpy(), real.cpu().numpy(), nl.cpu().numpy())
        finally:
            hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192)
    assert np.array_equal(got[8192][0], got[8192][1])
    for b, h in zip(got[8192], got[0]):
        assert np.array_equal(b, h)


@pytest.mark.parametrize("k", [3, 4])
@pytest.mark.parametrize("n", [1, 2048, 2049, 2700])
def test_copy_rows_match_hash(hm, n, k):
    """Copies whose incidence lists one workgroup makes (bit rows of up to 2^17
    words), the first beyond, and rows that are read as lists as well, against
    the path without bit rows."""
    rng = np.random.default_rng(n)
    sizes = [j for j, m in ((1, 3), (2, 2001), (3, 1500), (4, 700), (6, 30)) for _ in range(m) if j <= n]
    rows = [np.sort(rng.choice(min(n, 400), j, replace=False)) for j in sizes]
    rows[-1] = np.sort(n - 1 - np.arange(len(rows[-1])))
    members = np.concatenate(rows).astype(np.uint32)
    offsets = np.cumsum([0] + sizes).astype(np.uint64)
    got = {}
    for bits in (8192, 0):
        hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, bits)
        try:
            with hm.hm_graph_create(members, offsets, n) as g:
                real, nl, _ = hm.count_nulls(g, k, 5, 3)
                got[bits] = (real.cpu().numpy(), nl.cpu().numpy())
        finally:
            hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192)
    for b, h in zip(got[8192], got[0]):
        assert np.array_equal(b, h)


@pytest.mark.parametrize("edges", [4, 60, 300, 700, 1500, 6000])
def test_repairs_of_every_size_match_oracle(hm, edges):
    """Repairs whose lists are sorted within a wavefront, by the workgroup in
    LDS and in device memory."""
    h = W.random_small(5400 + edges, 25, edges, {2: 0.5, 3: 0.3, 4: 0.15, 5: 0.05}, allow_dups=True)
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        for copy in (0, 3):
            m, o = hm.hm_null_export(g, 21, copy)
            wm, wo = nulls.stub_matching(h, 21, copy)
            assert np.array_equal(o, wo) and np.array_equal(m, wm), copy
