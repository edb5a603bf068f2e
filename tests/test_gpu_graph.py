"""GPU parity: edge and triplet lists from the HIP library vs the oracle, bit-exact."""
import numpy as np
import pytest
import torch

import synth
from oracle import graph as ograph
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(lib):
    return lib.Context(0)


def _gpu_graph(lib, ctx, pos, gptr, cutoff, cap):
    dpos = H.to_dev(pos, torch.float32)
    dptr = H.to_dev(gptr, torch.int32)
    e, t = lib.build_graph(ctx, dpos, dptr, cutoff, cap)
    torch.cuda.synchronize()
    return e, t


def _check(lib, ctx, pos, gptr, cutoff, cap):
    ref = H.oracle_graph(pos, gptr, cutoff, cap)
    e, t = _gpu_graph(lib, ctx, pos, gptr, cutoff, cap)
    assert e["n_edges"] == len(ref["src"])
    assert t["n_triplets"] == len(ref["idx_kj"])
    assert np.array_equal(e["src"].cpu().numpy(), ref["src"])
    assert np.array_equal(e["dst"].cpu().numpy(), ref["dst"])
    assert np.array_equal(e["row_ptr"].cpu().numpy(), ref["row_ptr"])
    idx_kj, idx_ji = t["idx_kj"].cpu().numpy(), t["idx_ji"].cpu().numpy()
    assert np.array_equal(idx_kj, ref["idx_kj"])
    assert np.array_equal(idx_ji, ref["idx_ji"])
    assert np.array_equal(t["seg_ptr_ji"].cpu().numpy().astype(np.int64), ref["seg"])
    # kj-major view: a permutation of the triplets sorted by (idx_kj, idx_ji)
    perm = t["perm_kj"].cpu().numpy().astype(np.int64)
    assert np.array_equal(np.sort(perm), np.arange(len(perm)))
    key = idx_kj[perm].astype(np.int64) * (len(ref["src"]) + 1) + idx_ji[perm]
    assert np.all(np.diff(key) > 0)
    assert np.array_equal(t["idx_ji_kj"].cpu().numpy(), idx_ji[perm])
    seg_kj = np.zeros(len(ref["src"]) + 1, dtype=np.int64)
    np.add.at(seg_kj, idx_kj.astype(np.int64) + 1, 1)
    assert np.array_equal(t["seg_ptr_kj"].cpu().numpy().astype(np.int64), np.cumsum(seg_kj))
    # distances and unit vectors against fp64
    p = pos.astype(np.float64)
    vec = p[ref["dst"]] - p[ref["src"]]
    d = np.linalg.norm(vec, axis=1)
    if len(d):
        assert np.abs(e["dist"].cpu().numpy() - d).max() < 2e-6 * max(1.0, d.max())
        assert np.abs(e["unit"].cpu().numpy() - vec / d[:, None]).max() < 2e-6
    return ref


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_cfg1_graph(lib, ctx, seed):
    w = synth.get_workload("cfg1")
    pos, gptr = synth.make_positions(w, seed)
    _check(lib, ctx, pos, gptr, w.dims.cutoff, w.max_neighbors)


@pytest.mark.parametrize("cap", [0, 5, 12, 50])
def test_capped_multi_graph(lib, ctx, cap):
    pos, gptr = synth.slab_adsorbate_positions(3, 4, 3, 3, 7, seed=cap)
    ref = _check(lib, ctx, pos, gptr, 6.0, cap)
    assert len(ref["src"]) > 0


def test_cfg2_full_graph(lib, ctx):
    w = synth.get_workload("cfg2")
    pos, gptr = synth.make_positions(w, 0)
    ref = _check(lib, ctx, pos, gptr, w.dims.cutoff, w.max_neighbors)
    assert len(ref["idx_kj"]) > 1_000_000


def test_more_than_one_wave_of_sources_and_long_segments(lib, ctx):
    # 150 atoms in one structure, large cutoff: > 64 sources per target, > 64 triplets per edge
    pos, gptr = synth.cube_positions(150, 9.0, 0.9, seed=3)
    ref = _check(lib, ctx, pos, gptr, 7.5, 0)
    assert np.diff(ref["row_ptr"]).max() > 64
    ref = _check(lib, ctx, pos, gptr, 7.5, 70)
    assert np.diff(ref["row_ptr"]).max() == 70


def test_degenerate_inputs(lib, ctx):
    # no atoms
    e, t = _gpu_graph(lib, ctx, np.zeros((0, 3), np.float32), np.array([0], np.int32), 5.0, 0)
    assert e["n_edges"] == 0 and t["n_triplets"] == 0
    # one atom: no edges
    e, t = _gpu_graph(lib, ctx, np.zeros((1, 3), np.float32), np.array([0, 1], np.int32), 5.0, 0)
    assert e["n_edges"] == 0 and t["n_triplets"] == 0
    assert e["row_ptr"].cpu().tolist() == [0, 0]
    # two atoms in range: two edges, no triplet (k == i is excluded)
    pos = np.array([[0, 0, 0], [1, 0, 0]], np.float32)
    e, t = _gpu_graph(lib, ctx, pos, np.array([0, 2], np.int32), 5.0, 0)
    assert e["n_edges"] == 2 and t["n_triplets"] == 0
    assert t["seg_ptr_ji"].cpu().tolist() == [0, 0, 0] and t["seg_ptr_kj"].cpu().tolist() == [0, 0, 0]
    # two structures never connect; an empty structure in between is allowed
    pos = np.array([[0, 0, 0], [1, 0, 0], [0.5, 0, 0]], np.float32)
    e, t = _gpu_graph(lib, ctx, pos, np.array([0, 2, 2, 3], np.int32), 5.0, 0)
    assert e["n_edges"] == 2
    # three collinear atoms all in range: 6 edges, 6 triplets
    pos = np.array([[0, 0, 0], [1, 0, 0], [2, 0, 0]], np.float32)
    _check(lib, ctx, pos, np.array([0, 3], np.int32), 5.0, 0)


def test_error_codes(lib, ctx):
    import ctypes as C
    L = lib.load()
    pos = H.to_dev(np.zeros((4, 3), np.float32), torch.float32)
    gptr = H.to_dev(np.array([0, 4], np.int32), torch.int32)
    ws = torch.empty(4096, dtype=torch.uint8, device="cuda:0")
    n = C.c_int64()
    rc = L.gp_edges_count(ctx._h, C.c_void_p(pos.data_ptr()), C.c_void_p(gptr.data_ptr()), C.c_int64(4), C.c_int32(1),
                          C.c_float(-1.0), C.c_int32(0), C.c_void_p(ws.data_ptr()), C.c_size_t(4096), C.byref(n))
    assert rc == -1 and b"cutoff" in L.gp_last_error(ctx._h)
    rc = L.gp_edges_count(ctx._h, C.c_void_p(pos.data_ptr()), C.c_void_p(gptr.data_ptr()), C.c_int64(4), C.c_int32(1),
                          C.c_float(2.0), C.c_int32(0), C.c_void_p(ws.data_ptr()), C.c_size_t(8), C.byref(n))
    assert rc == -2
    rc = L.gp_edges_count(ctx._h, None, C.c_void_p(gptr.data_ptr()), C.c_int64(4), C.c_int32(1),
                          C.c_float(2.0), C.c_int32(0), C.c_void_p(ws.data_ptr()), C.c_size_t(4096), C.byref(n))
    assert rc == -1
    rc = L.gp_edges_count(ctx._h, C.c_void_p(pos.data_ptr()), C.c_void_p(gptr.data_ptr()), C.c_int64(-4), C.c_int32(1),
                          C.c_float(2.0), C.c_int32(0), C.c_void_p(ws.data_ptr()), C.c_size_t(4096), C.byref(n))
    assert rc == -1


@pytest.mark.parametrize("case", ["one shell of equal distances", "more candidates in range than the list holds", "cap of all but one"])
def test_cap_selection_edges(lib, ctx, case):
    # the kept neighbours end inside a run of equal squared distances / the selection recomputes distances / the cap is one
    # below the number in range
    if case == "one shell of equal distances":
        g = np.stack(np.meshgrid(*[np.arange(5.0)] * 3, indexing="ij"), -1).reshape(-1, 3).astype(np.float32)
        for cap in (3, 6, 10, 18):
            _check(lib, ctx, g, np.array([0, len(g)], np.int32), 2.3, cap)
    elif case == "more candidates in range than the list holds":
        pos, gptr = synth.cube_positions(530, 10.0, 0.5, seed=2)
        ref = _check(lib, ctx, pos, gptr, 30.0, 7)
        assert np.all(np.diff(ref["row_ptr"]) == 7)
    else:
        pos, gptr = synth.cube_positions(66, 8.0, 0.9, seed=4)
        ref = _check(lib, ctx, pos, gptr, 30.0, 64)
        assert np.all(np.diff(ref["row_ptr"]) == 64)


@pytest.mark.parametrize("n_struct,n", [(1, 3), (60, 5), (2900, 20)])   # below one chunk, a few chunks, over 1024 chunks of edges
def test_lists_of_complete_structures(lib, ctx, n_struct, n):
    # every atom of a structure sees every other one: all lists in closed form
    rng = np.random.default_rng(n)
    pos = rng.uniform(0, 3.0, (n_struct * n, 3)).astype(np.float32)
    e, t = _gpu_graph(lib, ctx, pos, (np.arange(n_struct + 1) * n).astype(np.int32), 50.0, 0)
    E = n_struct * n * (n - 1)
    assert e["n_edges"] == E and t["n_triplets"] == E * (n - 2)
    assert t["max_in_degree"] == n - 1 and t["max_out_degree"] == n - 1
    src, dst = e["src"].cpu().numpy().astype(np.int64), e["dst"].cpu().numpy().astype(np.int64)
    a = np.arange(n_struct * n, dtype=np.int64)
    edge_id = lambda s, d: d * (n - 1) + s % n - (s % n > d % n)     # in-edges of d in order of their source
    swap = edge_id(dst, src)
    assert np.array_equal(edge_id(src, dst), np.arange(E)) and np.array_equal(t["id_swap"].cpu().numpy(), swap)
    assert np.array_equal(t["out_list"].cpu().numpy(), np.lexsort((np.arange(E), src)))
    assert np.array_equal(t["out_ptr"].cpu().numpy(), np.concatenate([a, [len(a)]]) * (n - 1))
    seg = np.arange(E + 1) * (n - 2)
    assert np.array_equal(t["seg_ptr_ji"].cpu().numpy(), seg) and np.array_equal(t["seg_ptr_kj"].cpu().numpy(), seg)
    rows = src[:, None] * (n - 1) + np.arange(n - 1)                  # in-edges of the source, the opposite edge dropped
    kj = rows[rows != swap[:, None]]
    ji = np.repeat(np.arange(E), n - 2)
    assert np.array_equal(t["idx_kj"].cpu().numpy(), kj) and np.array_equal(t["idx_ji"].cpu().numpy(), ji)
    order = np.lexsort((ji, kj))
    assert np.array_equal(t["perm_kj"].cpu().numpy(), order) and np.array_equal(t["idx_ji_kj"].cpu().numpy(), ji[order])


@pytest.mark.parametrize("n,cutoff,cap", [(2, 5.0, 0), (66, 3.0, 0), (99, 20.0, 0), (131, 20.0, 0), (560, 30.0, 0), (140, 6.0, 20)])
def test_cosines_of_both_orders(lib, ctx, n, cutoff, cap):
    # lists shorter and longer than a chunk of either team size, several atoms per team, atoms whose out-list has no opposite edge
    from types import SimpleNamespace
    pos, gptr = synth.cube_positions(n, (n / 0.5) ** (1 / 3), 0.3, seed=n)
    e, t = _gpu_graph(lib, ctx, pos, gptr, cutoff, cap)
    dims = SimpleNamespace(**dict(vars(synth.get_workload("cfg4").dims), cutoff=cutoff, num_radial=2))
    b = lib.gp_basis_forward(ctx, dims, e, t)
    torch.cuda.synchronize()
    kj, ji, perm = (t[k].long() for k in ("idx_kj", "idx_ji", "perm_kj"))
    u = e["unit"].double()
    want = -(u[ji] * u[kj]).sum(1)
    # three products and two sums of numbers below one in fp32: within 5 half ulps of one
    assert t["n_triplets"] == 0 or (b["cos_alpha"].double() - want.clamp(-1, 1)).abs().max() < 3e-7
    assert torch.equal(b["cos_alpha_kj"], b["cos_alpha"][perm])
    # the fill of the index lists, checked against each other: every order lists every triplet once
    assert torch.equal(t["idx_ji_kj"].long(), ji[perm])
    key = kj[perm] * e["n_edges"] + t["idx_ji_kj"].long()
    assert bool((key[1:] > key[:-1]).all()) and torch.equal(e["dst"].long()[kj], e["src"].long()[ji])
    assert bool((e["src"].long()[kj] != e["dst"].long()[ji]).all())


def test_threads_count_on_one_context(lib, ctx):
    # the counts of a graph go through words that belong to the context: every thread gets its own graph's
    from concurrent.futures import ThreadPoolExecutor
    sizes = [20, 33, 47, 60]
    graphs = [tuple(H.to_dev(a, t) for a, t in zip(synth.cube_positions(n, 8.0, 0.5, seed=n), (torch.float32, torch.int32))) for n in sizes]

    def counts(k):
        e, t = lib.build_graph(ctx, *graphs[k % len(sizes)], 30.0, 0)     # every atom sees every other one
        return e["n_edges"], t["n_triplets"], t["max_in_degree"], t["max_out_degree"]

    with ThreadPoolExecutor(4) as pool:
        got = list(pool.map(counts, range(40)))
    torch.cuda.synchronize()
    for k, c in enumerate(got):
        n = sizes[k % len(sizes)]
        assert c == (n * (n - 1), n * (n - 1) * (n - 2), n - 1, n - 1)


def _cosines(lib, ctx, e, t):
    """Both orders as gp_basis_forward gives them, checked against the index arrays of t."""
    from types import SimpleNamespace
    dims = SimpleNamespace(**dict(vars(synth.get_workload("cfg4").dims), cutoff=50.0, num_radial=2))
    b = lib.gp_basis_forward(ctx, dims, e, t)
    torch.cuda.synchronize()
    kj, ji, perm = (t[k].long() for k in ("idx_kj", "idx_ji", "perm_kj"))
    u = e["unit"].double()
    assert b["cos_alpha"].shape == kj.shape and b["cos_alpha_kj"].shape == kj.shape
    # three products and two sums of numbers below one in fp32: within 5 half ulps of one
    assert (b["cos_alpha"].double() - (-(u[ji] * u[kj]).sum(1)).clamp(-1, 1)).abs().max() < 3e-7
    assert torch.equal(b["cos_alpha_kj"], b["cos_alpha"][perm])
    return b


def _without(t, drop, segments):
    """The triplets of t without those marked; segments: also the arrays that gp_basis_forward has no use for."""
    kj, ji = t["idx_kj"][~drop].long(), t["idx_ji"][~drop].long()
    E = t["n_edges"]
    perm = torch.argsort(kj * E + ji)
    out = dict(t, n_triplets=len(kj), idx_kj=kj.int(), idx_ji=ji.int(), perm_kj=perm.int())
    if segments:
        ptr = lambda i: torch.cat([torch.zeros(1, dtype=torch.int64, device=i.device), torch.cumsum(torch.bincount(i, minlength=E), 0)]).int()
        out.update(idx_ji_kj=ji[perm].int(), seg_ptr_ji=ptr(ji), seg_ptr_kj=ptr(kj))
    return out


@pytest.mark.parametrize("n,cap", [(140, 20), (131, 0)])   # short lists, long lists
def test_cosines_of_triplet_dicts_without_all_lists(lib, ctx, n, cap):
    # the lists by centre atom are optional members of a graph: without any of them the cosines follow from the index arrays
    pos, gptr = synth.cube_positions(n, (n / 0.5) ** (1 / 3), 0.3, seed=n)
    e, t = _gpu_graph(lib, ctx, pos, gptr, 20.0, cap)
    want = _cosines(lib, ctx, e, t)
    dicts = [(e, {k: v for k, v in t.items() if k not in gone}) for gone in (["out_list", "out_ptr", "row_ptr"], ["out_list"], ["id_swap"], ["seg_ptr_kj"])]
    dicts += [(e, dict(t, id_swap=None)), (e, dict(t, out_ptr=None)), ({k: v for k, v in e.items() if k != "dst"}, t)]
    for edges, trip in dicts:
        got = _cosines(lib, ctx, edges, trip)
        assert torch.equal(got["cos_alpha"], want["cos_alpha"]) and torch.equal(got["cos_alpha_kj"], want["cos_alpha_kj"])


@pytest.mark.parametrize("n,cap", [(140, 20), (131, 0)])   # short lists, long lists
@pytest.mark.parametrize("share", ["few", "third", "all but few", "one edge's"])
@pytest.mark.parametrize("segments", [False, True])
def test_cosines_after_triplets_were_taken_out(lib, ctx, n, cap, share, segments):
    # a dict whose triplets were filtered while the lists of the graph stayed: the index arrays count
    pos, gptr = synth.cube_positions(n, (n / 0.5) ** (1 / 3), 0.3, seed=n)
    e, t = _gpu_graph(lib, ctx, pos, gptr, 20.0, cap)
    T = t["n_triplets"]
    rnd = torch.as_tensor(np.random.default_rng(n).uniform(size=T)).to("cuda:0")
    drop = {"few": rnd < 30.0 / T, "third": rnd < 0.33, "all but few": rnd > 30.0 / T, "one edge's": t["idx_ji"] == e["n_edges"] // 2}[share]
    assert 0 < int(drop.sum()) < T
    _cosines(lib, ctx, e, _without(t, drop, segments))


@pytest.mark.parametrize("own", [True, False])   # the context on a stream of its own / on the default one while another is current
@pytest.mark.parametrize("with_kj", [True, False])
def test_graph_is_finished_on_a_stream_that_is_not_current(lib, own, with_kj):
    # the workspaces die with the calls, and a caller on the current stream reads the lists as soon as it has them
    other = torch.cuda.Stream()
    c = lib.Context(0, stream=other if own else None)
    pos, gptr = synth.cube_positions(300, (300 / 0.5) ** (1 / 3), 0.3, seed=5)
    dpos, dptr = H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32)
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.current_stream() if own else other):
        e = lib.gp_edges(c, dpos, dptr, 30.0)
        assert c.stream.query()
        t = lib.gp_triplets(c, e, with_kj=with_kj)
        assert c.stream.query()
        kj, ji = t["idx_kj"].clone(), t["idx_ji"].clone()   # on the current stream
    torch.cuda.synchronize()
    src, dst = e["src"].cpu().numpy().astype(np.int64), e["dst"].cpu().numpy().astype(np.int64)
    rows = src[:, None] * 299 + np.arange(299)              # every atom sees every other one
    back = dst * 1 + src * 299 - (dst > src)
    assert np.array_equal(kj.cpu().numpy(), rows[rows != back[:, None]])
    assert np.array_equal(ji.cpu().numpy(), np.repeat(np.arange(300 * 299), 298))


@pytest.mark.parametrize("n", [1000, 1300])   # below / above 2^31 triplets
def test_no_work_is_left_behind_by_a_count(lib, n):
    # gp_triplets_count returns with its stream idle, and so does every count that ends in an overflow: the workspace may go at once
    import ctypes as C
    from paper_2203_09697_amd.binding import GpError
    c = lib.Context(0, stream=torch.cuda.Stream())
    L = lib.load()
    pos = np.random.default_rng(6).uniform(0.0, 10.0, (n, 3))
    e = lib.gp_edges(c, H.to_dev(pos, torch.float32), H.to_dev(np.array([0, n]), torch.int32), 100.0)   # every atom sees every other one
    E, T = n * (n - 1), n * (n - 1) * (n - 2)
    assert e["n_edges"] == E
    nb, got = C.c_size_t(), C.c_int64()
    L.gp_triplets_workspace(C.c_int64(n), C.c_int64(E), C.byref(nb))
    ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda:0")
    torch.cuda.synchronize()
    rc = L.gp_triplets_count(c._h, *(C.c_void_p(e[k].data_ptr()) for k in ("src", "dst", "row_ptr")), C.c_int64(n), C.c_int64(E),
                             C.c_void_p(ws.data_ptr()), C.c_size_t(nb.value), C.byref(got))
    assert c.stream.query() and got.value == T and rc == (0 if T < 2 ** 31 else -3)
    if rc:
        with pytest.raises(GpError) as err:
            lib.gp_triplets(c, e)
        assert c.stream.query() and err.value.code == -3


def test_offsets_without_an_edge_list(lib, ctx):
    # gp_edges_fill with n_edges = 0 writes the offsets that the count left, and nothing else
    import ctypes as C
    L = lib.load()
    pos, gptr = synth.cube_positions(70, 6.0, 0.5, seed=7)
    want = lib.gp_edges(ctx, H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32), 3.0)
    dpos, dptr = H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32)
    nb, n = C.c_size_t(), C.c_int64()
    L.gp_edges_workspace(C.c_int64(70), C.byref(nb))
    ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda:0")
    row_ptr = torch.full((71,), -1, dtype=torch.int32, device="cuda:0")
    args = (ctx._h, C.c_void_p(dpos.data_ptr()), C.c_void_p(dptr.data_ptr()), C.c_int64(70), C.c_int32(1), C.c_float(3.0), C.c_int32(0),
            C.c_void_p(ws.data_ptr()), C.c_size_t(nb.value))
    ctx.check(L.gp_edges_count(*args, C.byref(n)))
    ctx.check(L.gp_edges_fill(*args, C.c_int64(0), None, None, C.c_void_p(row_ptr.data_ptr()), None, None))
    torch.cuda.synchronize()
    assert n.value == want["n_edges"] > 0 and torch.equal(row_ptr, want["row_ptr"])


# short lists with missing opposites / long lists with missing opposites / periodic ones, short and long
LIST_CASES = {"capped": dict(n=140, cutoff=6.0, cap=20), "capped, long": dict(n=420, cutoff=30.0, cap=150), "open, long": dict(n=131, cutoff=20.0, cap=0),
              "periodic, capped": dict(n=40, cutoff=5.0, cap=30, rep=(1, 1, 0)), "periodic, long": dict(n=60, cutoff=4.5, cap=0, rep=(1, 1, 1)),
              "no triplets": dict(n=2, cutoff=20.0, cap=0)}


def _list_case(lib, ctx, name):
    """edges of the case and its lists as the oracle gives them"""
    c = LIST_CASES[name]
    side = (c["n"] / 0.5) ** (1 / 3)
    pos, gptr = synth.cube_positions(c["n"], side, 0.3, seed=c["n"])
    if "rep" in c:
        cells = (side * np.array([[[1.0, 0.1, 0.0], [0.0, 1.0, -0.1], [0.0, 0.0, 1.0]]])).astype(np.float32)
        s, d, o, rp = ograph.edges_pbc(pos, gptr, cells, c["cutoff"], c["rep"], c["cap"])
        e = lib.gp_edges(ctx, H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32), c["cutoff"], c["cap"], H.to_dev(cells, torch.float32), c["rep"])
    else:
        o = None
        s, d, rp = ograph.edges(pos, gptr, c["cutoff"], c["cap"])
        e = lib.gp_edges(ctx, H.to_dev(pos, torch.float32), H.to_dev(gptr, torch.int32), c["cutoff"], c["cap"])
    kj, ji, seg = ograph.triplets(s, d, rp) if o is None else ograph.triplets(s, d, rp, o)
    swap = ograph.reverse_edges(s, d) if o is None else ograph.reverse_edges(s, d, o)
    order = np.lexsort((ji, kj))
    count = lambda i, n: np.concatenate([[0], np.cumsum(np.bincount(i, minlength=n))])
    want = dict(idx_kj=kj, idx_ji=ji, seg_ptr_ji=seg, perm_kj=order, idx_ji_kj=np.asarray(ji)[order], seg_ptr_kj=count(kj, len(s)),
                id_swap=swap, out_ptr=count(s, c["n"]), out_list=np.lexsort((np.arange(len(s)), s)))
    assert np.array_equal(e["src"].cpu().numpy(), s) and np.array_equal(e["dst"].cpu().numpy(), d)
    if "long" in name:
        assert len(kj) >= 128 * len(s)
    if "capped" in name:
        assert (np.asarray(swap) < 0).any() and (np.diff(want["out_ptr"]) != np.diff(rp)).any()
    return e, want


@pytest.mark.parametrize("name", list(LIST_CASES))
def test_lists_of_every_entry_point(lib, ctx, name):
    # gp_graph_lists_count/fill, gp_triplets_count/fill (with and without the kj-major order, twice on one workspace),
    # gp_reverse_edges, gp_edges_by_source and gp_csr_max_degree against the oracle
    import ctypes as C
    from paper_2203_09697_amd import binding as B
    L = lib.load()
    e, want = _list_case(lib, ctx, name)
    N, E, T = e["n_atoms"], e["n_edges"], len(want["idx_kj"])
    t = lib.gp_triplets(ctx, e)
    _cosines(lib, ctx, e, t) if T else None
    got = [t, lib.gp_triplets(ctx, e, with_kj=False), dict(id_swap=lib.gp_reverse_edges(ctx, e)),
           dict(zip(("out_ptr", "out_list"), lib.gp_edges_by_source(ctx, e)))]
    off = e.get("offset")
    nb, n = C.c_size_t(), C.c_int64()
    L.gp_triplets_workspace(C.c_int64(N), C.c_int64(E), C.byref(nb))
    ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda:0")
    args = (ctx._h, B._ptr(e["src"]), B._ptr(e["dst"])) + ((B._ptr(off),) if off is not None else ()) + (
        B._ptr(e["row_ptr"]), C.c_int64(N), C.c_int64(E), B._ptr(ws), C.c_size_t(nb.value))
    count, fill = (L.gp_triplets_count, L.gp_triplets_fill) if off is None else (L.gp_triplets_count_pbc, L.gp_triplets_fill_pbc)
    ctx.check(count(*args, C.byref(n)))
    assert n.value == T == t["n_triplets"]
    size = dict(idx_kj=T, idx_ji=T, seg_ptr_ji=E + 1, perm_kj=T, idx_ji_kj=T, seg_ptr_kj=E + 1)
    for kj in (True, False, True):
        a = {k: torch.full((v,), -7, dtype=torch.int32, device="cuda:0") for k, v in size.items()}
        if not kj:
            a.update(perm_kj=None, idx_ji_kj=None, seg_ptr_kj=None)
        ctx.check(fill(*args, C.c_int64(T), *(B._ptr(a[k]) for k in size)))
        got.append({k: v for k, v in a.items() if v is not None})
    torch.cuda.synchronize()
    for g in got:
        for k in want:
            if k in g:
                assert np.array_equal(g[k].cpu().numpy(), want[k]), k
    word, most = torch.empty(8, dtype=torch.uint8, device="cuda:0"), C.c_int32()
    for ptr, have in (("row_ptr", t["max_in_degree"]), ("out_ptr", t["max_out_degree"])):
        ctx.check(L.gp_csr_max_degree(ctx._h, B._ptr(t[ptr]), C.c_int64(N), B._ptr(word), C.c_size_t(8), C.byref(most)))
        assert most.value == have == int(t[ptr].diff().max())


@pytest.mark.parametrize("in_range", [511, 512, 513])
@pytest.mark.parametrize("cap", [1, 60])
def test_cap_at_the_length_of_the_candidate_list(lib, ctx, in_range, cap):
    # 512 candidates in range are selected from the list, one more makes the selection evaluate them again
    pos, gptr = synth.cube_positions(in_range + 1, 10.0, 0.5, seed=in_range)
    ref = _check(lib, ctx, pos, gptr, 30.0, cap)
    assert np.all(np.diff(ref["row_ptr"]) == cap)
