"""Every path of the planner's dispatch against the oracle, bit-exact, at the
sizes where the paths meet: rank groups per lane and wavefronts per start,
D^rem and the family records in LDS or in global memory, sums of shifts held
in registers or made again, one round of starts or several (a winner whose
wavefront has run another job since runs again), shapes of one family and of
many, patterns in one round of lanes or several."""
import struct

import numpy as np
import pytest
import torch

import oracle
import vpgen

pytestmark = pytest.mark.gpu

UNIT = 4096


@pytest.fixture(scope="module")
def vp():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2609_34340_amd as vp
    vp.lib()
    return vp


def sparse_demand(rng, N, per_row, scale):
    """About per_row destinations of every rank; a quarter of the entries near the lane caps' size."""
    D = rng.integers(1, scale + 1, (N, N)) * (rng.random((N, N)) < per_row / N)
    D *= np.where(rng.random((N, N)) < 0.25, 40, 1)
    np.fill_diagonal(D, 0)
    return (D * UNIT).astype(np.int64)


def check(vp, topo, D, **kw):
    """The whole schedule of up to 32 ranks; of more, where the oracle takes minutes for the thousands of activations
    a scattered demand needs, the first 24 (the capacity, which both report as exceeded)."""
    N = topo.n_ranks
    kw.setdefault("k_max", 64 * N if N <= 32 else 24)
    cat = vp.Catalog(topo)
    cat.upload()
    p = vp.plan_params(N, UNIT, **kw)
    out = vp.alloc_schedule(N, p.k_max, layout=True)
    st = vp.new_status()
    vp.plan(cat, torch.from_numpy(D).cuda(), p, status=st, out=out)
    torch.cuda.synchronize()
    o = oracle.Catalog(topo).plan(D, UNIT, check=False, **kw)
    print("N=%d K=%d %s" % (N, o["K"], kw), flush=True)
    assert vp.read_status(st) == o["status"] and o["status"] in (0, vp.CAPACITY)
    g = vp.schedule_to_host(out)
    assert g["K"] == o["K"] and g["tau"] == o["tau"]
    K = g["K"]
    for key in ("family", "dst", "inst", "bytes"):
        assert np.array_equal(g[key], o[key][:K]), key
    # the layout outputs, restated from the schedule
    sent, to, rows = np.zeros(N, np.int64), np.zeros((N, N), np.int64), np.arange(N)
    send_off, stream_off, recv_src = (out[k][:K].cpu().numpy() for k in ("send_off", "stream_off", "recv_src"))
    for k in range(K):
        assert np.array_equal(send_off[k], sent) and np.array_equal(stream_off[k], to[rows, g["dst"][k]]), k
        assert np.array_equal(recv_src[k][g["dst"][k]], rows), k
        sent += g["bytes"][k]
        to[rows, g["dst"][k]] += g["bytes"][k]


# groups per lane, wavefronts per start and where D^rem lies, on both sides of each line (G = rank groups)
SIZES = [
    vpgen.Topology(63, 1, 1, 2), vpgen.Topology(64, 1, 1, 2), vpgen.Topology(65, 1, 1, 2),   # G = 63, 64, 65
    vpgen.Topology(16), vpgen.Topology(17), vpgen.Topology(24), vpgen.Topology(25),          # G = 64 ... 100
    vpgen.Topology(32), vpgen.Topology(33), vpgen.Topology(65, 2, 2, 2),                     # G = 128, 132, 260
    vpgen.Topology(21, 1, 3, 3), vpgen.Topology(22, 1, 3, 3), vpgen.Topology(43, 1, 3, 3),   # triples: G = 63, 66, 129
    vpgen.Topology(32, 1, 2, 4), vpgen.Topology(33, 1, 2, 4), vpgen.Topology(65, 1, 2, 4),   # quads: G = 64, 66, 130
]


@pytest.mark.parametrize("topo", SIZES, ids=lambda t: "x".join(map(str, t.as_tuple()[:4])))
def test_sizes_of_the_runs(vp, topo):
    rng = np.random.default_rng(topo.n_ranks)
    check(vp, topo, sparse_demand(rng, topo.n_ranks, 1.5, 6))


# records in LDS and (with cross-socket peer to peer, from some size on) in global memory; several rounds of patterns
@pytest.mark.parametrize("nodes", [1, 2, 3, 8, 16, 20])
def test_large_catalogs(vp, nodes):
    topo = vpgen.Topology(nodes, flags=1)
    rng = np.random.default_rng(nodes)
    check(vp, topo, sparse_demand(rng, topo.n_ranks, min(2.0, topo.n_ranks / 2), 20))


# shifts of a NIC-lane set: two, four and eight per lane, one to sixteen lanes per set, and too many to hold
@pytest.mark.parametrize("topo", [vpgen.Topology(n) for n in (2, 3, 4, 5, 9, 10)] +
                         [vpgen.Topology(n, 1, 2, 2) for n in (6, 33, 34, 64)] +
                         [vpgen.Topology(n, 1, 1, 2) for n in (66, 120)] + [vpgen.Topology(66, 1, 2, 2)],
                         ids=lambda t: "x".join(map(str, t.as_tuple()[:4])))
def test_shift_layouts(vp, topo):
    rng = np.random.default_rng(1000 + topo.n_ranks)
    check(vp, topo, sparse_demand(rng, topo.n_ranks, 1.5, 6))


# starts: fewer than, as many as and more than the wavefronts; shapes of one family and of many
@pytest.mark.parametrize("topo", [vpgen.Topology(2), vpgen.Topology(1, 1, 2, 2, 2), vpgen.Topology(3, 1, 2, 2, 3),
                                  vpgen.Topology(2, 1, 2, 3), vpgen.Topology(33, 2, 2, 2)],
                         ids=lambda t: "x".join(map(str, t.as_tuple()[:5])))
@pytest.mark.parametrize("n_start", [1, 3, 4, 5, 8, 9, 16])
def test_rounds_of_starts(vp, topo, n_start):
    rng = np.random.default_rng(10 * topo.n_ranks + n_start)
    N = topo.n_ranks
    D = sparse_demand(rng, N, 3.0, 12)
    check(vp, topo, D, n_start=n_start, i_aa=[8, 0, 1, 2][n_start % 4], seed=n_start)


# more starts than run side by side, on every kernel that takes them in turn: groups per lane, wavefronts per start, D^rem
# in LDS and not
@pytest.mark.parametrize("topo", [vpgen.Topology(2), vpgen.Topology(17), vpgen.Topology(32), vpgen.Topology(33),
                                  vpgen.Topology(65), vpgen.Topology(2, 1, 3, 3), vpgen.Topology(21, 1, 3, 3),
                                  vpgen.Topology(22, 1, 3, 3), vpgen.Topology(43, 1, 3, 3), vpgen.Topology(86, 1, 3, 3),
                                  vpgen.Topology(2, 1, 2, 4), vpgen.Topology(32, 1, 2, 4), vpgen.Topology(33, 1, 2, 4),
                                  vpgen.Topology(65, 1, 2, 4)], ids=lambda t: "x".join(map(str, t.as_tuple()[:4])))
@pytest.mark.parametrize("n_start,i_aa", [(5, 8), (8, 0), (9, 8), (16, 2)])
def test_starts_in_turn(vp, topo, n_start, i_aa):
    rng = np.random.default_rng(topo.n_ranks + n_start)
    check(vp, topo, sparse_demand(rng, topo.n_ranks, 2.0, 8), n_start=n_start, i_aa=i_aa, seed=n_start)


def cut_catalog(vp, topo, begin, end):
    """The catalog of `topo` with its shift-0 part cut to the families begin ... end - 1 (vp_catalog_load takes any
    subset): magic and topology (48 bytes), family counts of both parts and lanes per node (12), one byte per lane,
    FNV-1a of it all."""
    p = vp.Catalog(topo).save()
    f0, f1, lanes = struct.unpack_from("<3i", p, 48)
    body = p[:48] + struct.pack("<3i", end - begin, f1, lanes) + p[60 + begin * lanes:60 + end * lanes] + \
        p[60 + f0 * lanes:-8]
    h = 0xcbf29ce484222325
    for x in body:
        h = (h ^ x) * 0x100000001b3 & 0xFFFFFFFFFFFFFFFF
    return vp.Catalog.load(body + struct.pack("<Q", h))


# A shape of 144 families (chunks of 64, 64 and 16) whose starts take two wavefronts each: the winner's chunk is not the
# last one, so its run is made again.  One start without draws, so that the families' numbers in the cut catalog do not
# matter, and the oracle's binding of the same shape of the whole catalog is the one to find.
@pytest.mark.parametrize("i_aa", [8, 0])
def test_winner_in_an_earlier_chunk(vp, i_aa):
    topo = vpgen.Topology(43, 1, 3, 2, 2)
    o = oracle.Catalog(topo)
    s = o.shapes()
    shape = int(np.argmax(s["fam_end"] - s["fam_begin"]))
    begin, end = int(s["fam_begin"][shape]), int(s["fam_end"][shape])
    assert end - begin == 144 and s["k"][shape] == 0
    cat = cut_catalog(vp, topo, begin, end)
    cat.upload()
    N, tab = o.N, cat.instances()
    rank = np.arange(N)
    node, switch, slot = rank // 6, rank // 2, rank // 2 % 3
    local = (node[:, None] == node[None]) & (switch[:, None] != switch[None])
    past_the_last = 0
    for seed in range(12):
        rng = np.random.default_rng(seed)
        D = (rng.integers(0, 200, (N, N)) * local * UNIT).astype(np.int64)
        cands, chosen = o.shape_candidates(D, UNIT, shape, k_target=8, n_start=1, i_aa=i_aa)
        past_the_last += chosen - begin < 128 and (chosen - begin) % 64 >= 16
        p = vp.plan_params(N, UNIT, k_target=8, n_start=1, i_aa=i_aa, k_max=4 * N)
        st = vp.new_status()
        out = vp.plan(cat, torch.from_numpy(D).cuda(), p, status=st)
        torch.cuda.synchronize()
        print("i_aa=%d seed=%d winner %d of 144" % (i_aa, seed, chosen - begin), flush=True)
        assert vp.read_status(st) == 0
        g = vp.schedule_to_host(out)
        best = next(c for c in cands if c["family"] == chosen)
        dst, nbytes, inst = np.zeros(N, np.int32), np.zeros(N, np.int64), np.zeros(N, np.int32)
        dst[best["src"]], nbytes[best["src"]] = best["dst"], best["x"]
        inst[best["src"]] = o.cluster_family(chosen)["id"]
        assert g["family"][0] == chosen - begin, seed
        assert np.array_equal(g["dst"][0], dst) and np.array_equal(g["bytes"][0], nbytes), seed
        assert np.array_equal(g["inst"][0], inst), seed
        # the whole schedule: every instance joins its lane's switches, and the demand is served exactly
        served = np.zeros_like(D)
        for k in range(g["K"]):
            assert np.array_equal(np.sort(g["dst"][k]), rank), (seed, k)
            assert np.array_equal(tab["src"][g["inst"][k]], slot), (seed, k)
            assert np.array_equal(tab["dst"][g["inst"][k]], slot[g["dst"][k]]), (seed, k)
            served[rank, g["dst"][k]] += g["bytes"][k]
        assert np.array_equal(served, D), seed
    assert past_the_last >= 4   # winners that the last, short chunk has no family for


# Shapes of many families, two wavefronts per start, with and without sweeps: every slot starts one run after another
# from the canonical binding, with no barrier of a half-step between them where there are no sweeps.
@pytest.mark.parametrize("topo", [vpgen.Topology(43, 1, 3, 2, 2), vpgen.Topology(66, 1, 2, 2, 2),
                                  vpgen.Topology(33, 1, 2, 3, 2)], ids=lambda t: "x".join(map(str, t.as_tuple()[:5])))
@pytest.mark.parametrize("n_start,i_aa", [(1, 0), (4, 0), (1, 8), (4, 1)])
def test_rounds_of_families(vp, topo, n_start, i_aa):
    N, n = topo.n_ranks, topo.n_ranks // topo.n_nodes
    rng = np.random.default_rng(N)
    node = np.arange(N) // n
    shift = (node[None] - node[:, None]) % topo.n_nodes
    D = (rng.integers(0, 200, (N, N)) * ((shift == 0) | (shift == 5)) * UNIT).astype(np.int64)
    np.fill_diagonal(D, 0)
    check(vp, topo, D, n_start=n_start, i_aa=i_aa, k_target=64, k_max=12)


# The quantum of a refused demand: of its true row and column sums, also where they do not fit the 32 bits (in units)
# that the sums of an accepted demand fit in.
@pytest.mark.parametrize("nodes", [1, 3, 33])
@pytest.mark.parametrize("unit,entries,k_target", [
    (16, {(0, 1): 1 << 40}, 16),                                      # 2^36 units
    (1, {(0, 1): 3 << 40, (2, 1): 1 << 41}, 1),                       # a column of 2^42 bytes and more
    (16, {(3, 1): 1 << 36, (3, 2): 1 << 35, (3, 5): 16}, 64),         # 2^32 units meet in a row
    (4096, {(7, 0): 1 << 50, (6, 0): 4096}, 1000),                    # an entry past 2^42
    (16, {(0, 1): 1 << 31, (2, 3): 1 << 31}, 4096)])                  # sums that fit, 2^28 units in all
def test_quantum_of_a_refused_demand(vp, nodes, unit, entries, k_target):
    topo = vpgen.Topology(nodes)
    N = topo.n_ranks
    D = np.zeros((N, N), np.int64)
    for (i, j), v in entries.items():
        D[N - 1 - i, N - 1 - j] = v
    cat = vp.Catalog(topo)
    cat.upload()
    st = vp.new_status()
    out = vp.plan(cat, torch.from_numpy(D).cuda(), vp.plan_params(N, unit, k_target=k_target), status=st)
    torch.cuda.synchronize()
    assert vp.read_status(st) == vp.UNSUPPORTED and int(out["K"]) == 0
    den = topo.pcie_bytes_per_ns * k_target
    assert int(out["tau"]) == -(-int(max(D.sum(0).max(), D.sum(1).max())) // den)


# Shifts that tie, at every number of them that the lanes of a set can share: demands of one unit, small caps
@pytest.mark.parametrize("topo", [vpgen.Topology(n) for n in (10, 13, 17, 18, 20, 22, 25, 27, 32)] +
                         [vpgen.Topology(66, 1, 2, 2, 2), vpgen.Topology(43, 1, 3, 3), vpgen.Topology(41, 1, 1, 2)],
                         ids=lambda t: "x".join(map(str, t.as_tuple()[:5])))
@pytest.mark.parametrize("per_row,seed", [(1, 0), (2, 0), (2, 1), (6, 0)])
def test_ties_between_shifts(vp, topo, per_row, seed):
    N = topo.n_ranks
    rng = np.random.default_rng(N + per_row + 1000 * seed)
    D = ((rng.random((N, N)) < per_row / N) * UNIT).astype(np.int64)
    np.fill_diagonal(D, 0)
    check(vp, topo, D, k_target=4 * N, k_max=120)
