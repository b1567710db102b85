"""GPU parity of frequent subgraph mining (pg_fsm) against the CPU oracle:
supports from injective maps by definition on tiny graphs, edge-subset
enumeration with domain sets beyond.  Exact integers: the bar is equality."""
import hashlib

import numpy as np
import pytest
from scipy.sparse import csr_matrix

import oracle
from oracle import brute
from paper_1911_06969_amd import binding, synth
from tests.gpu_common import golden, gpu_or_skip, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return gpu_or_skip()


def gpu_fsm(g, max_edges, sigma, budget=None):
    with binding.Graph.from_csr(g) as G:
        if budget:
            G.set_memory_budget(budget)
        sup, nf = G.fsm(max_edges, sigma)
    assert nf == int((sup > 0).sum())
    return sup


@pytest.mark.parametrize("seed", range(12))
def test_against_injective_maps(torch, seed):
    rng = np.random.default_rng(400 + seed)
    L = int(rng.integers(1, 4))
    g = synth.gnp_small(int(rng.integers(5, 10)), float(rng.uniform(0.2, 0.7)), seed, n_labels=L)
    for sigma in (0, 1, 2, 3):
        for K in (1, 2, 3):
            want = brute.fsm(g, K, sigma)
            assert np.array_equal(gpu_fsm(g, K, sigma), want), (seed, sigma, K)


def test_single_label_edge_support(torch):
    g = synth.rmat(10, 4, seed=41)
    g = synth.CSR(g.row_ptr, g.col, np.zeros(g.n, np.int32), 1)
    sup = gpu_fsm(g, 1, 1)
    assert int(sup[0]) == int((g.degrees() > 0).sum())


@pytest.mark.parametrize("n,p,L,sigma", [(3000, 8 / 2999, 4, 50), (2000, 0.004, 3, 1), (4000, 0.003, 6, 20),
                                         (800, 0.02, 2, 400)])
def test_er_against_oracle(torch, n, p, L, sigma):
    g = synth.erdos_renyi(n, p, seed=42, n_labels=L)
    for K in (1, 2, 3):
        want = oracle.fsm(g, K, sigma)
        got = gpu_fsm(g, K, sigma)
        say("er", n, L, sigma, K, int((want > 0).sum()))
        assert np.array_equal(got, want)


def test_largest_label_alphabet(torch):
    """64 labels, the most a graph may carry: 11.5 million pattern slots
    for up to 3 edges, label ranks up to ~60 per class."""
    g = synth.erdos_renyi(3000, 0.004, seed=47, n_labels=64)
    for K in (1, 2, 3):
        for sigma in (1, 3):
            assert np.array_equal(gpu_fsm(g, K, sigma), oracle.fsm(g, K, sigma)), (K, sigma)


def test_power_law_labelled(torch):
    g = synth.rmat(11, 8, seed=43)
    g = synth.CSR(g.row_ptr, g.col, synth.random_labels(g.n, 5, 44), 5)
    for sigma in (10, 100):
        assert np.array_equal(gpu_fsm(g, 3, sigma), oracle.fsm(g, 3, sigma))


def test_bitmap_groups_under_small_budget(torch):
    g = synth.erdos_renyi(20000, 8 / 19999, seed=45, n_labels=8)
    want = oracle.fsm(g, 3, 5)
    assert np.array_equal(gpu_fsm(g, 3, 5, budget=8 << 20), want)


@pytest.mark.parametrize("n,L,sigma", [(30000, 6, 20), (5000, 3, 2)])
def test_bit_keys_and_atomic_bits_agree(torch, n, L, sigma):
    """Domain bits of three-edge patterns through sorted keys (the default)
    and through atomic ORs give the oracle's supports."""
    g = synth.erdos_renyi(n, 8 / (n - 1), seed=46, n_labels=L)
    want = oracle.fsm(g, 3, sigma)
    for keys in (1, 0):
        with binding.Graph.from_csr(g) as G:
            G.set_option(binding.PG_OPT_FSM_BIT_KEYS, keys)
            sup, nf = binding.pg_fsm(G.h, 3, sigma, g.n_labels)
        say("fsm bit keys", keys, n, L, sigma, nf)
        assert np.array_equal(sup, want)


def test_thresholds_and_antimonotone(torch):
    g = synth.erdos_renyi(3000, 0.003, seed=46, n_labels=3)
    allsup = gpu_fsm(g, 3, 0)
    none = gpu_fsm(g, 3, 10 ** 12)
    assert not none.any()
    mid = gpu_fsm(g, 3, 30)
    assert np.array_equal(mid, np.where(allsup >= 30, allsup, 0))


def test_rejects_unlabelled_and_bad_sizes(torch):
    g = synth.rmat(8, 4, seed=47)
    with binding.Graph.from_csr(g) as G:
        with pytest.raises(binding.PgError) as e:
            binding.pg_fsm(G.h, 3, 1, 4)
        assert e.value.code == binding.PG_EINVAL
    g.labels = np.zeros(g.n, np.int32)
    g.n_labels = 1
    with binding.Graph.from_csr(g) as G:
        with pytest.raises(binding.PgError) as e:
            binding.pg_fsm(G.h, 5, 1, 1)
        assert e.value.code == binding.PG_EUNSUPPORTED
    g.labels = (np.arange(g.n) % 33).astype(np.int32)
    g.n_labels = 33
    with binding.Graph.from_csr(g) as G:
        # four edges need at most 32 labels
        with pytest.raises(binding.PgError) as e:
            binding.pg_fsm(G.h, 4, 1, 33)
        assert e.value.code in (binding.PG_EUNSUPPORTED, binding.PG_EINVAL)


@pytest.mark.slow
def test_fsm_er_config(torch):
    """Labelled G(n, p), 500k vertices, average degree 8, 16 labels, sigma 1000,
    patterns of up to 3 edges."""
    g = synth.fsm_er()
    want = golden("full_configs.json")["fsm_er_500k"]["sigma1000"]
    sup = gpu_fsm(g, 3, 1000)
    say("fsm full", int((sup > 0).sum()))
    assert int((sup > 0).sum()) == want["n_frequent"]
    assert int(sup.sum()) == want["sum"]
    assert [int(sup[i]) for i in want["sample_index"]] == want["sample_support"]
    assert hashlib.sha256(sup.astype(np.uint64).tobytes()).hexdigest() == want["sha256"]


@pytest.mark.parametrize("seed", range(10))
def test_four_edges_against_injective_maps(torch, seed):
    """Patterns of four edges (5-path, 4-star, fork, 4-cycle, paw) on tiny
    graphs: supports by definition from injective maps."""
    rng = np.random.default_rng(900 + seed)
    L = int(rng.integers(1, 4))
    g = synth.gnp_small(int(rng.integers(5, 10)), float(rng.uniform(0.25, 0.7)), 50 + seed, n_labels=L)
    for sigma in (0, 1, 2, 3):
        want = brute.fsm(g, 4, sigma)
        say(f"fsm4 brute seed={seed} n={g.n} L={L} sigma={sigma}")
        assert np.array_equal(gpu_fsm(g, 4, sigma), want), (seed, sigma)


def test_four_edge_shapes_one_by_one(torch):
    """Each four-edge shape alone with distinct and with equal labels: its
    pattern's support is the smallest orbit's domain."""
    shapes = {
        "path5": [(0, 1), (1, 2), (2, 3), (3, 4)],
        "star4": [(0, 1), (0, 2), (0, 3), (0, 4)],
        "fork": [(0, 1), (0, 2), (0, 3), (3, 4)],
        "cycle4": [(0, 1), (1, 2), (2, 3), (3, 0)],
        "paw": [(0, 1), (0, 2), (0, 3), (2, 3)],
    }
    for name, edges in shapes.items():
        n = 1 + max(max(e) for e in edges)
        for labels in (np.zeros(n, np.int32), np.arange(n, dtype=np.int32) % 3):
            L = int(labels.max()) + 1
            g = synth.from_edges(n, edges)
            g = synth.CSR(g.row_ptr, g.col, labels, L)
            want = brute.fsm(g, 4, 1)
            assert np.array_equal(gpu_fsm(g, 4, 1), want), (name, labels)


@pytest.mark.parametrize("n,p,L,sigma", [(1500, 6 / 1499, 3, 40), (2500, 0.002, 4, 5), (500, 0.016, 2, 60)])
def test_four_edges_er_against_oracle(torch, n, p, L, sigma):
    g = synth.erdos_renyi(n, p, seed=61, n_labels=L)
    want = oracle.fsm(g, 4, sigma)
    say("fsm4 er", n, L, sigma, int((want > 0).sum()))
    assert np.array_equal(gpu_fsm(g, 4, sigma), want)


def test_four_edges_power_law_and_small_budget(torch):
    """A skewed graph (hub lists, many embeddings per pattern) and a budget
    that forces the level-4 domain bitmaps into several groups."""
    g = synth.rmat(8, 2, seed=62)
    g = synth.CSR(g.row_ptr, g.col, synth.random_labels(g.n, 3, 63), 3)
    want = oracle.fsm(g, 4, 20)
    assert np.array_equal(gpu_fsm(g, 4, 20), want)
    assert np.array_equal(gpu_fsm(g, 4, 20, budget=1 << 20), want)


@pytest.mark.parametrize("L", [1, 15, 16, 17, 29, 31, 32, 33, 64])
def test_domain_counting_label_widths(torch, L):
    """Up to three edges, label counts around the mask widths and the counters'
    places in LDS, on a graph with many triangles: the domain counts, for two
    edges the level pipeline too (a budget of 1 MiB leaves it no other), and
    the oracle."""
    g = synth.disjoint_union(synth.erdos_renyi(700, 0.012, seed=50 + L), synth.erdos_renyi(60, 0.3, seed=51 + L),
                             synth.complete(9), synth.star(140), synth.cycle(4), synth.path(4))
    g = synth.CSR(g.row_ptr, g.col, synth.random_labels(g.n, L, 52 + L), L)
    for K in (1, 2, 3):
        for sigma in (1, 4):
            want = oracle.fsm(g, K, sigma)
            assert np.array_equal(gpu_fsm(g, K, sigma), want), (K, sigma)
            if K < 3 and L < 20:
                assert np.array_equal(gpu_fsm(g, K, sigma, budget=1 << 20), want), (K, sigma)


@pytest.mark.parametrize("leaves", [1022, 1023, 1024, 2500])
def test_domain_counting_hubs(torch, leaves):
    """Vertices of about the degree from which a workgroup takes one together:
    two adjacent hubs sharing their leaves, some of which are joined."""
    n = leaves + 2
    rng = np.random.default_rng(leaves)
    edges = [(0, 1)] + [(h, v) for h in (0, 1) for v in range(2, n)]
    edges += [tuple(x) for x in rng.integers(2, n, (60, 2)) if x[0] != x[1]]
    g = synth.from_edges(n, edges)
    g = synth.CSR(g.row_ptr, g.col, synth.random_labels(n, 5, leaves), 5)
    if leaves > 2000:   # too many embeddings for levels in 1 MiB
        assert np.array_equal(gpu_fsm(g, 2, 3), oracle.fsm(g, 2, 3))
        return
    for K in (2, 3):
        assert np.array_equal(gpu_fsm(g, K, 3), gpu_fsm(g, K, 3, budget=1 << 20)), K


@pytest.mark.parametrize("L", [3, 40])
def test_thresholds_between_supports(torch, L):
    """Thresholds at, just below and just above supports that the graph's edges and
    wedges have, uneven labels on a skewed graph: what is filtered away on the way
    changes no reported support."""
    g = synth.rmat(9, 4, seed=71)
    lab = (np.random.default_rng(72).random(g.n) ** 3 * L).astype(np.int32)
    g = synth.CSR(g.row_ptr, g.col, lab, L)
    two = oracle.fsm(g, 2, 1)
    some = np.unique(two[two > 0])
    some = some[np.linspace(0, len(some) - 1, 7).astype(int)]
    full = oracle.fsm(g, 3, 1)
    for sigma in sorted({max(1, int(s) + d) for s in some for d in (-1, 0, 1)}):
        want = np.where(full >= sigma, full, 0).astype(full.dtype)
        assert np.array_equal(gpu_fsm(g, 3, sigma), want), sigma
    assert np.array_equal(gpu_fsm(g, 3, int(some[3])), oracle.fsm(g, 3, int(some[3])))


def test_filter_spares_the_walk(torch):
    """With no frequent wedge the paths of three edges are not walked."""
    g = synth.rmat(15, 8, seed=73)
    g = synth.CSR(g.row_ptr, g.col, synth.random_labels(g.n, 4, 74), 4)
    ms = []
    with binding.Graph.from_csr(g) as G:
        G.fsm(3, g.n)
        binding.pg_profile_enable(True)
        try:
            for sigma in (1, g.n):
                binding.pg_profile_reset()
                G.fsm(3, sigma)
                ms.append(binding.pg_profile_query("fsm_paths")[0])
        finally:
            binding.pg_profile_enable(False)
    say("paths, ms:", ms)
    assert 5 * ms[1] < ms[0]


def _supports_of_two_edges(g):
    """Supports of edges and wedges by definition, from the number of each vertex's
    neighbours of each label: {(a, b): s, (centre, a, b): s} with a <= b."""
    lab, src = g.labels, np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    used = [int(x) for x in np.unique(lab)]
    cnt = np.zeros((g.n, g.n_labels), np.int64)
    np.add.at(cnt, (src, lab[g.col]), 1)
    out = {}
    for a in used:
        for b in used:
            if a <= b:
                out[a, b] = min(int((cnt[lab == a, b] > 0).sum()), int((cnt[lab == b, a] > 0).sum()))
            for c in used:
                if a > b:
                    continue
                centres = int(((cnt[:, a] > 0) & (cnt[:, b] > (a == b)) & (lab == c)).sum())

                def leaves(x, y):   # of label x, next to a centre with another neighbour of label y
                    on = (lab[src] == x) & (lab[g.col] == c) & (cnt[g.col, y] > (x == y))
                    return int(np.unique(src[on]).size)

                out[c, a, b] = min(centres, leaves(a, b), leaves(b, a))
    return {k: v for k, v in out.items() if v > 0}


@pytest.mark.parametrize("L", [5, 40])
def test_long_lists(torch, L):
    """Vertices around the lengths from which a workgroup takes a list and takes it
    in several steps, with labels that occur once, twice and three times among the
    neighbours."""
    edges, labels, n = [], [], 0
    rng = np.random.default_rng(L)
    for i, d in enumerate((255, 256, 257, 1023, 1025, 8191, 8192, 8193, 20_000)):
        edges += [(n, n + 1 + j) for j in range(d)]
        lab = np.zeros(d + 1, np.int32)
        lab[rng.choice(np.arange(1, d + 1), 6, replace=False)] = [1, 2, 2, 3, 3, 3]
        lab[0] = i * 7 % L
        labels.append(lab)
        n += d + 1
    edges += [(1, 300), (2, 3), (5000, 20_000)]
    g = synth.from_edges(n, edges)
    g = synth.CSR(g.row_ptr, g.col, np.concatenate(labels), L)
    want = _supports_of_two_edges(g)
    for sigma in (1, 3):
        sup = gpu_fsm(g, 2, sigma)
        got = {tuple(binding.pg_fsm_pattern_key(int(i), 2, L)[1]): int(sup[i]) for i in np.nonzero(sup)[0]}
        assert got == {k: v for k, v in want.items() if v >= sigma}


def _hubs(n):
    return synth.from_edges(n + 4, [(h, v) for h in range(4) for v in range(4, n + 4)])


@pytest.mark.parametrize("g", [_hubs(20_000), synth.erdos_renyi(40_000, 20 / 40_000, seed=76)], ids=["hubs", "even"])
def test_infrequent_edges_spare_the_stars(torch, g):
    """With no frequent edge wedges and stars are not counted, a hub's or others'."""
    g = synth.CSR(g.row_ptr, g.col, synth.random_labels(g.n, 8, 75), 8)
    ms = []
    with binding.Graph.from_csr(g) as G:
        G.fsm(3, g.n)
        binding.pg_profile_enable(True)
        try:
            for sigma in (1, g.n):
                binding.pg_profile_reset()
                assert (G.fsm(3, sigma)[1] > 0) == (sigma == 1)
                ms.append(binding.pg_profile_query("fsm_stars")[0])
        finally:
            binding.pg_profile_enable(False)
    say("stars, ms:", ms)
    assert 5 * ms[1] < ms[0]


@pytest.mark.parametrize("leaves", [1023, 1100])
def test_hubs_under_any_label_count(torch, leaves):
    """The same labels out of 5, 32, 33 and 40: 32- and 64-bit masks, counters in LDS and
    in device memory, vertices that a workgroup takes together."""
    rng = np.random.default_rng(leaves)
    n = leaves + 2
    edges = [(0, 1)] + [(h, v) for h in (0, 1) for v in range(2, n)]
    edges += [tuple(x) for x in rng.integers(2, n, (90, 2)) if x[0] != x[1]]
    g = synth.from_edges(n, edges)
    lab = rng.integers(0, 5, n).astype(np.int32)
    for sigma in (1, 4, 60):
        rows = []
        for L in (5, 32, 33, 40):
            sup = gpu_fsm(synth.CSR(g.row_ptr, g.col, lab, L), 3, sigma)
            keys = [binding.pg_fsm_pattern_key(int(i), 3, L) for i in np.nonzero(sup)[0]]
            rows.append({(s, *l): int(x) for (s, l), x in zip(keys, sup[sup > 0])})
        assert len(rows[0]) > 0 and all(r == rows[0] for r in rows[1:]), sigma


@pytest.mark.parametrize("g", [synth.erdos_renyi(3_001, 8 / 3_000, seed=5), synth.rmat(12, 8, seed=2), synth.star(300),
                               synth.complete(66)], ids=["er", "rmat", "star", "complete"])
@pytest.mark.parametrize("max_edges", [1, 2, 3])
def test_recorded_embeddings(torch, g, max_edges):
    """The embeddings recorded with the kernel times: connected sets of up to so many
    edges, a triangle once (degrees around 64, from which a wave shares a list)."""
    a = csr_matrix((np.ones(g.nnz, np.int64), g.col, g.row_ptr), shape=(g.n, g.n))
    d = np.asarray(a.sum(axis=1)).ravel()
    u, v = a.nonzero()
    triangles = int((a @ a).multiply(a).sum()) // 6
    want = g.n_edges
    if max_edges >= 2:
        want += int((d * (d - 1) // 2).sum())
    if max_edges >= 3:
        want += int((d * (d - 1) * (d - 2) // 6).sum()) + int(((d[u] - 1) * (d[v] - 1)).sum()) // 2 - 2 * triangles
    labelled = synth.CSR(g.row_ptr, g.col, synth.random_labels(g.n, 4, 1), 4)
    with binding.Graph.from_csr(labelled) as G:
        binding.pg_profile_enable(True)
        try:
            binding.pg_profile_reset()
            G.fsm(max_edges, 1)
            got = binding.pg_profile_query("fsm_embeddings")[2]
        finally:
            binding.pg_profile_enable(False)
    say("embeddings", max_edges, want, got)
    assert int(round(got)) == want
