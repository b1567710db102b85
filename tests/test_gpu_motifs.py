"""GPU parity of motif counting (pg_count_motifs) against the CPU oracle
(brute force on tiny graphs, ESU and the closed form beyond).  Exact
integer counts: the bar is equality."""
from math import comb

import numpy as np
import pytest

import oracle
from oracle import brute, closed_form
from paper_1911_06969_amd import binding, synth
from tests.gpu_common import golden, gpu_or_skip, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return gpu_or_skip()


def gpu_motifs(g, k, budget=None):
    with binding.Graph.from_csr(g) as G:
        if budget:
            G.set_memory_budget(budget)
        return [int(x) for x in G.motifs(k)]


def test_every_graph_on_five_vertices(torch):
    for g in synth.all_graphs(5):
        for k in (3, 4):
            assert gpu_motifs(g, k) == [int(x) for x in brute.motif_counts(g, k)]


@pytest.mark.parametrize("seed", range(16))
def test_brute_force_small(torch, seed):
    rng = np.random.default_rng(300 + seed)
    g = synth.gnp_small(int(rng.integers(5, 13)), float(rng.uniform(0.1, 0.9)), seed)
    for k in (3, 4):
        assert gpu_motifs(g, k) == [int(x) for x in brute.motif_counts(g, k)]


def test_families(torch):
    assert gpu_motifs(synth.star(40), 4) == [0, comb(40, 3), 0, 0, 0, 0]
    assert gpu_motifs(synth.star(40), 3) == [comb(40, 2), 0]
    assert gpu_motifs(synth.cycle(50), 4) == [50, 0, 0, 0, 0, 0]
    assert gpu_motifs(synth.cycle(4), 4) == [0, 0, 1, 0, 0, 0]
    assert gpu_motifs(synth.path(30), 4) == [27, 0, 0, 0, 0, 0]
    assert gpu_motifs(synth.complete(12), 4) == [0, 0, 0, 0, 0, comb(12, 4)]
    assert gpu_motifs(synth.complete(12), 3) == [0, comb(12, 3)]
    a, b = 7, 9
    assert gpu_motifs(synth.complete_multipartite([a, b]), 4) == [
        0, a * comb(b, 3) + b * comb(a, 3), comb(a, 2) * comb(b, 2), 0, 0, 0]
    assert gpu_motifs(synth.empty(10), 4) == [0] * 6
    assert gpu_motifs(synth.empty(0), 3) == [0] * 2


def test_hub_lists_beyond_lds_stage(torch):
    """A star with 2000 leaves plus a dense core: adjacency lists longer than
    the LDS stage and common-neighbour lists longer than its LDS copy."""
    core = synth.complete(40)
    hub = synth.star(2000)
    g = synth.disjoint_union(core, hub, synth.erdos_renyi(1500, 0.05, seed=3))
    for k in (3, 4):
        want = closed_form.motif3(g) if k == 3 else closed_form.motif4(g)
        assert gpu_motifs(g, k) == [int(x) for x in want]


def test_dense_shared_neighbourhoods(torch):
    # degrees ~680 (> LDS stage), common-neighbour lists ~540 (> their LDS copy)
    g = synth.erdos_renyi(850, 0.8, seed=4)
    assert gpu_motifs(g, 4) == [int(x) for x in closed_form.motif4(g)]


@pytest.mark.parametrize("scale,ef,seed", [(9, 8, 1), (11, 8, 2), (12, 16, 3)])
def test_rmat_against_oracle(torch, scale, ef, seed):
    g = synth.rmat(scale, ef, seed=seed)
    for k in (3, 4):
        want = closed_form.motif3(g) if k == 3 else closed_form.motif4(g)
        say("rmat", scale, ef, k, list(want))
        assert gpu_motifs(g, k) == [int(x) for x in want]


def test_esu_on_rmat(torch):
    g = synth.rmat(9, 6, seed=8)
    for k in (3, 4):
        assert gpu_motifs(g, k) == [int(x) for x in oracle.motif_esu(g, k)]


def test_edge_blocking_same_counts(torch):
    g = synth.rmat(11, 8, seed=6)
    want = [int(x) for x in closed_form.motif4(g)]
    assert gpu_motifs(g, 4, budget=1 << 20) == want


def test_relabel_invariance(torch):
    g = synth.rmat(10, 8, seed=7)
    h = synth.relabel(g, np.random.default_rng(2).permutation(g.n))
    assert gpu_motifs(g, 4) == gpu_motifs(h, 4)


def test_reduce_example_triangles_and_wedge(torch):
    """Three embeddings reduce to {triangle: 2, wedge: 1} (section 3.1)."""
    g = synth.disjoint_union(synth.complete(3), synth.complete(3), synth.path(3))
    assert gpu_motifs(g, 3) == [1, 2]


def test_automorphism_example_counted_once(torch):
    """(3,5,4) and (2,5,4) both extend to {2,3,4,5} (section 3.2): the 4-set
    is counted once.  Graph: 5 adjacent to 2, 3 and 4; 4 adjacent to 3."""
    g = synth.from_edges(6, [(5, 2), (5, 3), (5, 4), (4, 3)])
    # {2,3,4,5}: edges 52 53 54 43 -> paw
    assert gpu_motifs(g, 4) == [0, 0, 0, 1, 0, 0]


def test_triangle_rmat_config(torch):
    g = synth.triangle_rmat()
    want = golden("full_configs.json")["triangle_rmat_s14"]
    assert gpu_motifs(g, 3) == want["motif3"]
    assert gpu_motifs(g, 4) == want["motif4"]


@pytest.mark.slow
def test_motif_rmat_config(torch):
    """R-MAT scale 18, edge factor 8: the motif workload at full size."""
    g = synth.motif_rmat()
    want = golden("full_configs.json")["motif_rmat_s18"]
    with binding.Graph.from_csr(g) as G:
        say("scale-18 k=3")
        assert [int(x) for x in G.motifs(3)] == want["motif3"]
        say("scale-18 k=4")
        assert [int(x) for x in G.motifs(4)] == want["motif4"]


def test_binary_search_connectivity_example(torch):
    """The connectivity check of section 5 (binary search figure): embedding
    {2, 5, 8} (here the path 2-5-8) and candidate 9, whose neighbour list
    holds 2 and 5 but not 8.  The 4-set {2, 5, 8, 9} is then a triangle
    2-5-9 with the pendant 8 (a paw), the only connected 4-set."""
    g = synth.from_edges(10, [(2, 5), (5, 8), (2, 9), (5, 9)])
    assert gpu_motifs(g, 4) == [0, 0, 0, 1, 0, 0]
    assert gpu_motifs(g, 4) == [int(x) for x in brute.motif_counts(g, 4)]
    assert gpu_motifs(g, 3) == [int(x) for x in brute.motif_counts(g, 3)]


@pytest.mark.parametrize("n_total", [60_000, 70_000, 200_000, 300_000, 600_000])
def test_map_kernel_sizes(torch, n_total):
    """4-motifs on graphs whose vertex count selects each size of the
    workgroup's two-bit vertex map (up to 2^16, 2^17, 2^18, 2^19 vertices)
    and one beyond it (per-wave kernel only): a hub of degree 3000, a dense
    random block and isolated vertices, against the closed form."""
    parts = [synth.star(3000), synth.erdos_renyi(700, 0.4, seed=11), synth.rmat(11, 8, seed=5)]
    used = sum(p.n for p in parts)
    g = synth.disjoint_union(*parts, synth.empty(n_total - used))
    assert g.n == n_total
    want = [int(x) for x in closed_form.motif4(g)]
    say("map sizes", n_total, want)
    assert gpu_motifs(g, 4) == want


def test_map_kernel_shared_hub_and_threshold(torch):
    """Entries just below and above the many-children threshold (255, 256
    and 257 leaves beyond a shared pair), a complete bipartite K_{2,300}
    (two hubs sharing every neighbour) and a budget small enough to cut the
    level-2 list into many chunks."""
    parts = [synth.complete_multipartite([2, 300])]
    for leaves in (255, 256, 257, 513):
        parts.append(synth.star(leaves))
    g = synth.disjoint_union(*parts, synth.erdos_renyi(700, 0.5, seed=9))
    want = [int(x) for x in closed_form.motif4(g)]
    a, b = 2, 300
    kab = [0, a * comb(b, 3) + b * comb(a, 3), comb(a, 2) * comb(b, 2), 0, 0, 0]
    assert [int(x) for x in closed_form.motif4(parts[0])] == kab
    assert gpu_motifs(g, 4) == want
    assert gpu_motifs(g, 4, budget=1 << 20) == want


@pytest.mark.parametrize("sizes", [range(42, 50), range(124, 134, 3), (300, 700)])
def test_table_kinds_dense(torch, sizes):
    """4-motifs of dense graphs around the limits between the tables of common
    neighbours (512 and 4,096 keys of a hash table, then an indexed table)."""
    g = synth.disjoint_union(*[synth.erdos_renyi(n, 0.5, seed=n) for n in sizes])
    want = [int(x) for x in closed_form.motif4(g)]
    assert gpu_motifs(g, 4) == want
    assert gpu_motifs(g, 3) == [int(x) for x in closed_form.motif3(g)]


@pytest.mark.parametrize("n,hub", [(3000, 2500), (70_000, 40_000), (500_000, 6000), (500_000, 60_000)])
def test_table_blocks_and_shared_hubs(torch, n, hub):
    """Two hubs of the same neighbours (more than 127 and more than 32,767
    common ones: each entry width), over a sparse graph whose names take one
    block of the indexed table or several, below and above the steps from
    which workgroups share a hub."""
    base = synth.erdos_renyi(n, 5.0 / n, seed=n + hub)
    rng = np.random.default_rng(hub)
    to = np.sort(rng.choice(n, hub, replace=False))
    edges = [base.edges()] + [np.stack([np.full(hub, n + i), to], axis=1) for i in (0, 1)]
    mid = to[rng.random(hub) < 200 / hub]
    edges += [np.stack([np.full(mid.shape[0], n + i), mid], axis=1) for i in (2, 3, 4)]
    g = synth.from_edges(n + 6, np.concatenate(edges))
    want = [int(x) for x in closed_form.motif4(g)]
    say("hubs", n, hub, want)
    assert gpu_motifs(g, 4) == want


@pytest.mark.slow
def test_more_than_2_31_edges(torch):
    """The complete bipartite graph of 2^24 + 1 and 128 vertices has 2^31 + 128
    edges: 3-motifs count it (as stars at either side), while the cliques' masks,
    whose edge numbers have 32 bits, still refuse it."""
    if torch.cuda.mem_get_info()[0] < 130 << 30:
        pytest.skip("needs 130 GB of device memory")
    a, b = (1 << 24) + 1, 128
    row_ptr = torch.cat([torch.arange(a, device="cuda") * b, a * b + torch.arange(b + 1, device="cuda") * a])
    col = torch.empty(2 * a * b, dtype=torch.int32, device="cuda")
    col[:a * b].view(a, b).copy_(torch.arange(a, a + b, dtype=torch.int32, device="cuda"))
    col[a * b:].view(b, a).copy_(torch.arange(a, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    say("bipartite graph made")
    with binding.Graph(row_ptr, col) as G:
        del col
        assert G.info() == (a + b, 2 * a * b, a)
        say("loaded")
        assert [int(x) for x in G.motifs(3)] == [a * (b * (b - 1) // 2) + b * (a * (a - 1) // 2), 0]
        with pytest.raises(binding.PgError) as e:
            G.cliques(3)
        assert e.value.code == binding.PG_EUNSUPPORTED
    del row_ptr
    torch.cuda.empty_cache()


def _closed_by_any_path(g):
    """3-motifs, which the size decides the way of, against the closed form and the
    triangles of the clique count."""
    with binding.Graph.from_csr(g) as G:
        got = [int(x) for x in G.motifs(3)]
        assert got == [int(x) for x in closed_form.motif3(g)]
        assert got[1] == G.cliques(3)


@pytest.mark.parametrize("hub", [1023, 1024, 1025])
def test_three_motifs_about_the_small_graphs_degree(torch, hub):
    edges = [(0, 1 + i) for i in range(hub)] + [(1 + i, 2 + i) for i in range(0, hub - 1, 2)]
    _closed_by_any_path(synth.from_edges(hub + 5, edges + [(hub + 2, hub + 4)]))


@pytest.mark.parametrize("n", [16_383, 16_384, 16_385])
def test_three_motifs_about_the_small_graphs_entries(torch, n):
    """16 entries a vertex: 2^18 at 16,384."""
    v = np.arange(n)
    edges = np.concatenate([np.stack([v, (v + s) % n], 1) for s in range(1, 9)])
    _closed_by_any_path(synth.from_edges(n, edges))


def test_three_motifs_of_small_graphs(torch):
    for g in [synth.empty(0), synth.empty(3), synth.complete(2), synth.complete(17), synth.complete(70),
              synth.rmat(9, 8, seed=5), synth.star(65), synth.cycle(3)]:
        _closed_by_any_path(g)


def test_a_small_graphs_first_call_builds_nothing(torch):
    """Three-motifs of a small graph take a block of device memory, not the DAG's and
    its plan's."""
    with binding.Graph.from_csr(synth.rmat(6, 4, seed=3)) as G:
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        G.motifs(3)
        assert torch.cuda.memory_stats()["allocation.all.allocated"] <= before + 1


def test_four_motifs_of_every_graph_on_five_vertices_by_either_way(torch):
    """As a batch of one graph, and beside enough other vertices by the walk over
    two-step paths: all 1,024 graphs, five vertices apart in one graph of 5,120, and
    the smallest and largest graph of a batch and one past it."""
    every = list(synth.all_graphs(5))
    want = np.stack([brute.motif_counts(g, 4) for g in every]).astype(np.int64)
    for i in range(0, 1024, 37):
        with binding.Graph.from_csr(every[i]) as G:
            assert [int(x) for x in G.motifs(4)] == want[i].tolist(), i
    with binding.Graph.from_csr(synth.disjoint_union(*every)) as G:
        assert [int(x) for x in G.motifs(4)] == want.sum(axis=0).tolist()


@pytest.mark.parametrize("n, p", [(1, 0.0), (2, 1.0), (63, 0.3), (64, 0.3), (65, 1.0), (511, 0.02), (512, 0.5), (512, 1.0),
                                  (513, 0.5), (700, 0.02)])
def test_four_motifs_about_the_largest_batch_graph(torch, n, p):
    g = synth.complete(n) if p == 1.0 else synth.erdos_renyi(n, p, seed=n)
    for extra in (0, 513):
        h = synth.disjoint_union(g, synth.empty(extra)) if extra else g
        with binding.Graph.from_csr(h) as G:
            assert [int(x) for x in G.motifs(4)] == [int(x) for x in closed_form.motif4(g)], extra


def test_a_batch_sized_graphs_first_call_builds_nothing(torch):
    """Its four-motifs take a block of device memory, not the renamed graph's, the DAG's
    and their plans'."""
    with binding.Graph.from_csr(synth.erdos_renyi(500, 0.3, seed=3)) as G:
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        G.motifs(4)
        assert torch.cuda.memory_stats()["allocation.all.allocated"] <= before + 1
