"""Order-5 sampled counting (Section 6.4: Algorithm 4 at order 5) through the
C ABI against the order-5 oracle: classes keyed by canonical pattern, raw
counts bit-exact, estimates exact to fp32, the census identity against brute
force, and unbiasedness over seeds."""
import numpy as np
import pytest

import workloads as W
from oracle import core, order5, philox, stats

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hm():
    import torch
    import paper_2209_10241_amd as hm
    assert torch.cuda.is_available()
    return hm


MIX = {2: 0.4, 3: 0.3, 4: 0.15, 5: 0.1, 6: 0.05}


def _as_dict(canon, vals):
    return {int(c): v for c, v in zip(canon.tolist(), vals.tolist())}


@pytest.mark.parametrize("bit_rows", [True, False], ids=["bits", "hash"])
@pytest.mark.parametrize("seed", range(6))
def test_census_matches_brute_force(hm, seed, bit_rows):
    """Every hyperedge of size 2..5 drawn once: raw = countmax x exact for
    every class (brute force over all 5-node sets), estimates = exact."""
    h = W.random_small(9500 + seed, 10 + seed * 2, 25 + 6 * seed, MIX, allow_dups=bool(seed % 2))
    nh = core.normalise(h)
    exact = order5.exact_brute(h)
    hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192 if bit_rows else 0)
    try:
        with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
            assert hm.hm_order5_sizes(g) == {j: nh.count(j) for j in (2, 3, 4, 5)}
            canon, raw, est = hm.count_sampled5_indices(g, {j: np.arange(nh.count(j)) for j in (2, 3, 4, 5)})
    finally:
        hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192)
    assert np.all(np.diff(canon.astype(np.int64)) > 0)
    assert set(_as_dict(canon, raw)) == set(exact)
    for c, r, e in zip(canon.tolist(), raw.tolist(), est.tolist()):
        assert r == order5.maxcard(c)[1] * exact[c]
        assert e == np.float32(exact[c])


@pytest.mark.parametrize("seed", range(4))
def test_draws_match_oracle(hm, seed):
    """count_sampled5 at a fraction: the same Philox draws, raw counts
    bit-exact, estimates the oracle's fp64 values rounded to fp32."""
    h = W.random_small(9600 + seed, 30 + 10 * seed, 150 + 40 * seed, MIX)
    nh = core.normalise(h)
    n = {j: nh.count(j) for j in (2, 3, 4, 5)}
    f = 0.3
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        canon, raw, est = hm.count_sampled5(g, f, 77 + seed)
    S = {j: int(np.ceil(f * n[j])) for j in n}
    samples = {j: philox.stratum_draws(77 + seed, j, n[j], S[j]) for j in n}
    want = order5.sampled_raw(h, samples)
    assert _as_dict(canon, raw) == want
    want_est = order5.scale(want, n, S)
    assert {c: v for c, v in _as_dict(canon, est).items()} == {c: float(np.float32(v)) for c, v in want_est.items()}


def test_sparse_larger_graph(hm):
    """A sparser, larger hypergraph (200 nodes, hyperedges of up to 8 nodes,
    repeats), every hyperedge of size 2..5 drawn once and some twice."""
    h = W.random_small(9650, 200, 260, {2: 0.5, 3: 0.25, 4: 0.1, 5: 0.1, 8: 0.05}, allow_dups=True)
    nh = core.normalise(h)
    rng = np.random.default_rng(3)
    samples = {j: np.concatenate([np.arange(nh.count(j)), rng.integers(0, nh.count(j), size=5)])
               for j in (2, 3, 4, 5)}
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        canon, raw, _ = hm.count_sampled5_indices(g, samples)
    assert _as_dict(canon, raw) == order5.sampled_raw(h, samples)


def test_unbiased_over_seeds(hm):
    """Section 5's estimator at order 5: the mean over 64 seeds of each
    class's estimate lies within 4.5 standard errors of the exact count."""
    h = W.random_small(9700, 14, 45, MIX)
    exact = order5.exact_brute(h)
    classes = sorted(exact)
    runs = []
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        for s in range(64):
            canon, _, est = hm.count_sampled5(g, 0.4, 1000 + s)
            d = _as_dict(canon, est)
            assert set(d) <= set(exact)
            runs.append([d.get(c, 0.0) for c in classes])
    z = stats.bias_z(np.array(runs), np.array([exact[c] for c in classes], dtype=np.float64))
    assert np.all(np.abs(z) < 4.5), np.abs(z).max()


@pytest.mark.parametrize("n_nodes,n_edges", [(5, 12), (31, 400), (32, 400), (33, 500), (64, 300), (65, 700), (130, 900),
                                            (1024, 1500), (1025, 1500)])
def test_dense_path_matches_general(hm, n_nodes, n_edges):
    """Hypergraphs of at most 1,024 nodes with bit rows take the bit-tensor
    path: the same classes, counts and estimates as the general path (taken
    without bit rows), around the edges of a bit row's words and of the rule;
    some hyperedges drawn twice."""
    h = W.random_small(9900 + n_nodes, n_nodes, n_edges, MIX, allow_dups=True)
    nh = core.normalise(h)
    rng = np.random.default_rng(n_nodes)
    samples = {j: rng.integers(0, nh.count(j), size=min(nh.count(j), 40) + 3) for j in (2, 3, 4, 5) if nh.count(j)}
    got = {}
    for bits in (8192, 0):
        hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, bits)
        try:
            with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
                got[bits] = hm.count_sampled5_indices(g, samples)
        finally:
            hm.hm_set_option(hm.HM_OPT_BITSET_MAX_NODES, 8192)
    for dense, general in zip(got[8192], got[0]):
        assert np.array_equal(dense, general)


def test_order5_errors(hm):
    h = W.random_small(9800, 12, 40, MIX)
    nh = core.normalise(h)
    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        with pytest.raises(hm.HMError):
            hm.count_sampled5(g, 0.0, 1)
        with pytest.raises(hm.HMError):
            hm.count_sampled5(g, 1.0, 1, capacity=1)
        with pytest.raises(hm.HMError):
            hm.count_sampled5_indices(g, {2: [nh.count(2)]})


@pytest.mark.parametrize("mix,few", [({2: 1.0}, {2: [3]}), ({2: 0.8, 3: 0.2}, {2: [0], 3: [1]}), ({4: 1.0}, {4: [0, 1]}),
                                     ({5: 0.9, 2: 0.1}, {5: [0], 2: [0]})])
def test_few_sets_leave_the_bit_tensors(hm, mix, few):
    """Samples of a hypergraph of a few hyperedges among many nodes take the
    general path, which needs no bit tensors; with the tensors there (after a
    call that pays for them) the same samples give the same classes."""
    h = W.random_small(9950 + len(mix), 1000, 60, mix)
    nh = core.normalise(h)
    many = {j: np.tile(np.arange(nh.count(j)), 400) for j in (2, 3, 4) if nh.count(j)}

    def route(g, samples):
        hm.hm_profile_enable(True)
        hm.hm_profile_reset()
        try:
            out = hm.count_sampled5_indices(g, samples)
            names = hm.hm_profile_read()
        finally:
            hm.hm_profile_enable(False)
            hm.hm_profile_reset()
        assert ("k_dense5" in names) != ("k_sampled5" in names)
        return "k_dense5" in names, out

    with hm.hm_graph_create(h.members, h.offsets, h.n_nodes) as g:
        dense, general = route(g, few)
        assert not dense
        pays, _ = route(g, many)
        dense, again = route(g, few)
        assert dense == pays
        for x, y in zip(general, again):
            assert np.array_equal(x, y)
    assert pays or 4 in mix or 5 in mix
