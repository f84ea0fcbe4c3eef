"""GPU parity: node sampling and radius graph against the oracle, bit for bit."""

import ctypes
import threading

import numpy as np
import pytest

import oracle
from oracle import radius_graph as org
from tests.helpers import announce, gpu_lib
from workloads import make_config

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return gpu_lib()


@pytest.mark.parametrize("M,s,seed", [(1, 1, 0), (10, 0, 3), (10, 10, 3), (37, 9, 2024), (4096, 1024, 4001),
                                      (65536, 8192, 4002), (1000003, 12345, 2 ** 64 - 5), (300000, 299999, 9)])
def test_sampling_bit_exact(env, M, s, seed):
    dm, lib, torch = env
    announce("sample", M, s, seed)
    got = lib.dsmp_sample_nodes(M, s, seed).cpu().numpy()
    assert np.array_equal(got, oracle.sampling.sample_nodes(M, s, seed))


@pytest.mark.parametrize("M", [2, 1023, 8191, 8192, 8193, 4 << 20, (8 << 20) - 3, (8 << 20) + 1])
def test_sampling_forms(env, M):
    """The one-workgroup, list and four-digit forms at their bounds, with few,
    half and nearly all candidates kept."""
    dm, lib, torch = env
    for s in sorted({1, M // 2, M - 1}):
        announce("sample form", M, s)
        got = lib.dsmp_sample_nodes(M, s, 1000 + s).cpu().numpy()
        assert np.array_equal(got, oracle.sampling.sample_nodes(M, s, 1000 + s)), s


@pytest.mark.parametrize("cols,offset", [(4, 0), (12, 0), (64, 0), (64, 1), (3, 0), (5, 2)])
def test_gather_rows_units(env, cols, offset):
    """16-byte and word units: row lengths, arrays off a 16-byte address, and
    indices out of range (zero rows)."""
    dm, lib, torch = env
    announce("gather", cols, offset)
    buf = torch.arange(offset + 50 * cols, dtype=torch.float32, device="cuda")
    src = buf[offset:].view(50, cols)
    idx = torch.tensor([49, -1, 0, 50, 7, 7], dtype=torch.int32, device="cuda")
    out = torch.full((offset + 6 * cols,), -1.0, device="cuda")[offset:].view(6, cols)
    lib.dsmp_gather_rows(src, idx, out=out)
    ok = (idx >= 0) & (idx < 50)
    want = torch.where(ok[:, None], src[idx.clamp(0, 49).long()], torch.zeros(1, device="cuda"))
    assert torch.equal(out, want)


@pytest.mark.parametrize("cols", [33, 64])
def test_gather_rows_in_several_steps(env, cols):
    """More units than the launch has threads, the last step part-filled."""
    dm, lib, torch = env
    announce("gather in steps", cols)
    src = torch.rand(1000, cols, device="cuda")
    idx = torch.randint(0, 1000, (70001,), device="cuda", dtype=torch.int32)
    assert torch.equal(lib.dsmp_gather_rows(src, idx), src[idx.long()])


def test_sampling_rejects_bad_sizes(env):
    dm, lib, torch = env
    with pytest.raises(dm.DsmpError) as ei:
        lib.dsmp_sample_nodes(5, 6, 0)
    assert ei.value.status == dm.INVALID_ARG


def _check_graph(lib, torch, pos, n_dst, r, cap=0, mode=0, seed=0, rows=None):
    dev = torch.device("cuda", 0)
    tpos = torch.from_numpy(np.ascontiguousarray(pos, np.float32)).to(dev)
    E = lib.dsmp_radius_graph_count(tpos, n_dst, r, cap, mode, seed)
    g = lib.dsmp_radius_graph_build(tpos, n_dst, r, cap, mode, seed, capacity=E)
    assert g.n_edges == E
    rp = g.row_ptr.cpu().numpy().astype(np.int64)
    col = g.col[:E].cpu().numpy()
    dst = g.dst[:E].cpu().numpy()
    if rows is None:
        rp_ref, col_ref = org.radius_graph(pos, n_dst, r, cap, mode, seed)
        assert np.array_equal(rp, rp_ref)
        assert np.array_equal(col, col_ref)
        assert np.array_equal(dst, org.dst_of_edges(rp_ref))
        cp_ref, ceid_ref = org.transpose(rp_ref, col_ref, pos.shape[0])
        assert np.array_equal(g.csc_ptr.cpu().numpy(), cp_ref)
        assert np.array_equal(g.csc_eid[:E].cpu().numpy(), ceid_ref)
    else:
        ref = org.rows_subset(pos, rows, n_dst, r, cap, mode, seed)
        for i, lst in zip(rows, ref):
            assert col[rp[i]:rp[i + 1]].tolist() == lst.tolist(), i
        assert np.all(np.diff(rp) >= 0) and rp[-1] == E
        assert np.array_equal(dst, np.repeat(np.arange(n_dst), np.diff(rp)))
        cp = g.csc_ptr.cpu().numpy().astype(np.int64)
        ceid = g.csc_eid[:E].cpu().numpy()
        assert cp[-1] == E and np.array_equal(np.bincount(col, minlength=pos.shape[0]), np.diff(cp))
        assert np.array_equal(col[ceid], np.repeat(np.arange(pos.shape[0]), np.diff(cp)))
        assert np.array_equal(np.sort(ceid), np.arange(E))
        for j in range(0, pos.shape[0], max(1, pos.shape[0] // 50)):
            assert np.all(np.diff(ceid[cp[j]:cp[j + 1]]) > 0)
    return g


def _rand(n, D, seed):
    return np.random.default_rng(seed).uniform(0, 1, (n, D)).astype(np.float32)


def _two_clusters(seed):
    """513 points within 0.002 of each other, and 514 more far away."""
    return np.concatenate([_rand(513, 3, seed) * 1e-3, _rand(514, 3, seed + 1) * 1e-3 + 10.0])


def _long_line(r=0.02, length=300.0, pairs=4000, seed=17):
    """Points along a line 15,000 cells long (one cell across) with pairs at
    the largest float32 distance that passes the radius test, the first point
    just past a cell bound, far from the origin, where the rounding of a cell
    coordinate is largest against the cell margin of 2^-10."""
    g = np.random.default_rng(seed)
    f32 = np.float32
    r2 = f32(r) * f32(r)
    c = r * (1.0 + 2.0 ** -10)
    k = g.integers(int(0.6 * length / c), int(length / c) - 2, pairs)
    x1 = ((k + g.uniform(0.9e-3, 1.5e-3, pairs)) * c).astype(f32)
    x2 = (x1 + f32(r)).astype(f32)
    for _ in range(8):   # the largest x2 with fl(fl(x2 - x1)^2) <= fl(r^2)
        d = (x2 - x1).astype(f32)
        over = (d * d).astype(f32) > r2
        x2 = np.where(over, np.nextafter(x2, f32(-np.inf)), x2)
    up = np.nextafter(x2, f32(np.inf))
    du = (up - x1).astype(f32)
    x2 = np.where((du * du).astype(f32) <= r2, up, x2)
    y = np.full(pairs, 5e-4, f32)
    pts = [np.array([[0.0, 0.0], [length, 1e-3]], f32),
           np.stack([x1, y], 1), np.stack([x2, y], 1),
           np.stack([g.uniform(0, length, 2000), g.uniform(0, 1e-3, 2000)], 1).astype(f32)]
    return np.concatenate(pts)


CASES = {
    "2d_uncapped": (lambda: _rand(3000, 2, 1), 2500, 0.03, 0, 0),
    "2d_knn5": (lambda: _rand(3000, 2, 2), 3000, 0.05, 5, 0),
    "2d_random5": (lambda: _rand(3000, 2, 3), 2800, 0.05, 5, 1),
    "3d_uncapped": (lambda: _rand(3000, 3, 4), 3000, 0.08, 0, 0),
    "3d_knn7": (lambda: _rand(3000, 3, 5), 2000, 0.12, 7, 0),
    "3d_random7": (lambda: _rand(3000, 3, 6), 3000, 0.12, 7, 1),
    "lattice64_ties_knn": (lambda: np.stack(np.meshgrid(np.linspace(0, 1, 64), np.linspace(0, 1, 64),
                                                        indexing="ij"), -1).reshape(-1, 2).astype(np.float32),
                           4096, 0.08, 12, 0),
    "lattice_uncapped": (lambda: np.stack(np.meshgrid(np.linspace(0, 1, 64), np.linspace(0, 1, 64),
                                                      indexing="ij"), -1).reshape(-1, 2).astype(np.float32),
                         4096, 0.08, 0, 0),
    "coincident_r0": (lambda: np.repeat(_rand(200, 2, 7), 3, axis=0), 600, 0.0, 0, 0),
    "empty_tiny_r": (lambda: _rand(2000, 3, 8), 2000, 1e-6, 0, 0),
    "complete_graph": (lambda: _rand(1500, 2, 9), 1500, 5.0, 0, 0),
    "complete_capped": (lambda: _rand(1500, 3, 10), 1500, 5.0, 100, 0),
    "clustered": (lambda: np.concatenate([_rand(1000, 2, 11) * 1e-3, _rand(1000, 2, 12)]), 2000, 0.01, 16, 0),
    "no_destinations": (lambda: _rand(100, 2, 13), 0, 0.1, 0, 0),
    "single_point": (lambda: _rand(1, 3, 14), 1, 0.1, 0, 0),
    "halo_far": (lambda: np.concatenate([_rand(500, 2, 15), _rand(500, 2, 16) + 5.0]), 500, 0.08, 0, 0),
    "long_line_15k_cells": (lambda: _long_line(), 10002, 0.02, 0, 0),
    # rows of 65..168 candidates capped at 40: the cap is selected in registers
    "dense_knn40": (lambda: _rand(4000, 3, 20), 4000, 0.2, 40, 0),
    # rows of 130..555 candidates, a cap above 64: both the register select
    # (up to 512 candidates) and the sort in shared memory (beyond)
    "dense_random80": (lambda: _rand(4000, 2, 21), 4000, 0.2, 80, 1),
    # two tight clusters: rows of exactly 512 and of 513 candidates
    "clusters_512_513_knn": (lambda: _two_clusters(22), 1027, 0.01, 30, 0),
    "clusters_512_513_random": (lambda: _two_clusters(24), 1027, 0.01, 30, 1),
    # capped graphs select each row in one pass: rows of 58..264 candidates
    # (the last few beyond what that pass holds), and a cap of exactly 64
    "dense_random48": (lambda: _rand(4000, 2, 25), 4000, 0.132, 48, 1),
    "dense_knn64": (lambda: _rand(4000, 3, 26), 4000, 0.2, 64, 0),
    # a cap of one (the select keeps the single smallest key), and a cap above
    # every row's size (no select; the fill pass, caps above 64)
    "3d_knn1": (lambda: _rand(3000, 3, 27), 3000, 0.12, 1, 0),
    "2d_random1": (lambda: _rand(3000, 2, 28), 3000, 0.05, 1, 1),
    "3d_cap200": (lambda: _rand(3000, 3, 29), 3000, 0.12, 200, 0),
    # the one-workgroup cell sort (up to 8,192 points): its largest size, with a
    # grid of more cells than its table; and one point more
    "sparse_8192_points": (lambda: _rand(8192, 2, 30), 8192, 0.004, 0, 0),
    "sparse_8193_points": (lambda: _rand(8193, 2, 31), 8193, 0.004, 0, 0),
    # more cells than points at one radius (12,996), in 2-D and, crowded in a corner, 3-D
    "8192_points_13k_cells": (lambda: _rand(8192, 2, 45), 8192, 0.00877, 0, 0),
    "8000_points_16k_cells_crowded": (lambda: np.concatenate([_rand(800, 3, 46), 0.2 * _rand(7200, 3, 47)]),
                                      8000, 0.0405, 24, 0),
    "8193_points_halo_random": (lambda: _rand(8193, 3, 32), 7000, 0.07, 6, 1),
    # the cap among shells of equal and nearly equal distances (a lattice), among
    # more equal distances than are ranked one per lane (coincident points, and
    # nearly coincident ones), and one edge short of the row
    "lattice3d_knn24": (lambda: np.stack(np.meshgrid(*[np.linspace(0, 1, 14)] * 3, indexing="ij"),
                                         -1).reshape(-1, 3).astype(np.float32), 2744, 0.2, 24, 0),
    "coincident_knn10": (lambda: np.repeat(_rand(20, 2, 35), 100, axis=0), 2000, 0.01, 10, 0),
    "coincident_random10": (lambda: np.repeat(_rand(20, 2, 36), 100, axis=0), 2000, 0.01, 10, 1),
    "near_coincident_knn40": (lambda: (np.repeat(_rand(10, 3, 37), 200, axis=0)
                                       + 1e-7 * _rand(2000, 3, 38)).astype(np.float32), 2000, 0.01, 40, 0),
    "complete_66_knn64": (lambda: _rand(66, 2, 39), 66, 5.0, 64, 0),
    # row counts scanned in one launch (up to 4,096 rows) and in two
    "2d_4096_rows": (lambda: _rand(4200, 2, 43), 4096, 0.03, 0, 0),
    "2d_4097_rows_knn": (lambda: _rand(4200, 2, 44), 4097, 0.05, 9, 0),
    "2d_16384_rows": (lambda: _rand(16384, 2, 33), 16384, 0.02, 0, 0),
    "2d_16385_rows_knn": (lambda: _rand(16500, 2, 34), 16385, 0.03, 9, 0),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_graph_bit_exact(env, name):
    dm, lib, torch = env
    mk, n_dst, r, cap, mode = CASES[name]
    announce("graph", name)
    _check_graph(lib, torch, mk(), n_dst, r, cap, mode, seed=123)


@pytest.mark.parametrize("r,cap", [(0.05, 0), (0.2, 0), (0.2, 80), (0.05, 5), (1e-6, 0)])
def test_graph_built_without_a_capacity(env, r, cap):
    """Without a capacity the arrays come with the graph's own size, also where
    it has more than 64 edges per destination."""
    dm, lib, torch = env
    announce("graph without capacity", r, cap)
    pos = _rand(1000, 2, 40)
    g = lib.dsmp_radius_graph_build(torch.from_numpy(pos).cuda(), 1000, r, cap)
    rp, col = org.radius_graph(pos, 1000, r, cap)
    E = int(rp[-1])
    assert g.n_edges == E and g.col.numel() == g.dst.numel() == g.csc_eid.numel() == max(E, 1)
    assert np.array_equal(g.row_ptr.cpu().numpy(), rp) and np.array_equal(g.col[:E].cpu().numpy(), col)
    assert np.array_equal(g.csc_eid[:E].cpu().numpy(), org.transpose(rp, col, 1000)[1])


@pytest.mark.parametrize("r,cap", [(0.05, 0), (0.2, 0), (0.2, 80), (0.6, 20), (0.05, 5), (1e-6, 0)])
def test_graph_built_without_a_capacity_counts_once_and_holds_its_edges(env, r, cap):
    """Few and many edges per destination, every row selected and some left to
    the fill: the arrays are as large as the graph, built by one pass over the
    candidates."""
    dm, lib, torch = env
    announce("graph without capacity, memory", r, cap)
    pos = torch.from_numpy(_rand(1000, 2, 41)).cuda()
    E = lib.dsmp_radius_graph_count(pos, 1000, r, cap)
    want = lib.dsmp_radius_graph_build(pos, 1000, r, cap, capacity=E)
    lib.dsmp_profile_enable(True)
    lib.dsmp_profile_reset()
    try:
        want2 = lib.dsmp_radius_graph_build(pos, 1000, r, cap, capacity=E, out=want)
        one = lib.dsmp_profile_read()["graph"][1]
        lib.dsmp_profile_reset()
        g = lib.dsmp_radius_graph_build(pos, 1000, r, cap)
        assert lib.dsmp_profile_read()["graph"][1] == 2 * one   # its two halves, each once
    finally:
        lib.dsmp_profile_enable(False)
    assert g.n_edges == want2.n_edges == E
    for a, b in ((g.row_ptr, want.row_ptr), (g.csc_ptr, want.csc_ptr)):
        assert torch.equal(a, b)
    for a, b in ((g.col, want.col), (g.dst, want.dst), (g.csc_eid, want.csc_eid)):
        assert torch.equal(a[:E], b[:E]) and a.untyped_storage().nbytes() == 4 * max(E, 1)


def test_graph_halves_check_their_arguments(env):
    """The second half of a build with too little room, and with counts that are
    not the first half's."""
    dm, lib, torch = env
    c, pos = ctypes, torch.from_numpy(_rand(1000, 2, 42)).cuda()
    want = lib.dsmp_radius_graph_build(pos, 1000, 0.05, 0)
    E = want.n_edges
    q, _ = lib._query(pos, 1000, 0.05, 0, dm.CAP_KNN, 0)
    ws = lib._graph_ws(q)
    args = (lib.h, c.byref(q), c.c_void_p(ws.data_ptr()), ws.numel())
    cg, row = want.c(), c.c_int32()
    assert lib.lib.dsmp_radius_graph_rows(*args, c.byref(cg), None) == dm.INVALID_ARG
    assert lib.lib.dsmp_radius_graph_rows(*args, c.byref(cg), c.byref(row)) == dm.OK
    assert cg.n_edges == E and row.value == int(torch.diff(want.row_ptr).max())
    assert lib.lib.dsmp_radius_graph_edges(*args, row, E - 1, c.byref(cg)) == dm.CAPACITY
    assert lib.lib.dsmp_radius_graph_edges(*args, 5000, E, c.byref(cg)) == dm.INVALID_ARG
    assert lib.lib.dsmp_radius_graph_edges(*args, -1, E, c.byref(cg)) == dm.INVALID_ARG
    cg.n_dst = 999
    assert lib.lib.dsmp_radius_graph_edges(*args, row, E, c.byref(cg)) == dm.INVALID_ARG


@pytest.mark.parametrize("cap", [0, 10])
def test_graph_capacity_error_reports_E(env, cap):
    dm, lib, torch = env
    pos = torch.from_numpy(_rand(1000, 2, 20)).cuda()
    E = lib.dsmp_radius_graph_count(pos, 1000, 0.05, cap)
    with pytest.raises(dm.DsmpError) as ei:
        lib.dsmp_radius_graph_build(pos, 1000, 0.05, cap, capacity=E - 1)
    assert ei.value.status == dm.CAPACITY


def test_graph_row_limit_is_unsupported(env):
    dm, lib, torch = env
    pos = torch.from_numpy(_rand(5000, 2, 21)).cuda()
    with pytest.raises(dm.DsmpError) as ei:
        lib.dsmp_radius_graph_count(pos, 5000, 10.0)
    assert ei.value.status == dm.UNSUPPORTED


def _sampled(k):
    w = make_config(k)
    pos, n_dst = [], w.n_dst
    for p in w.parts:
        idx = oracle.sampling.sample_nodes(p.pos.shape[0], p.s, p.seed)
        pos.append(p.pos[idx])
    return w, np.concatenate(pos)


@pytest.mark.parametrize("k", [1, 2, 3])
def test_graph_workload_full(env, k):
    dm, lib, torch = env
    announce("graph workload", k)
    w, pos = _sampled(k)
    _check_graph(lib, torch, pos, w.n_dst, w.r, w.cap, w.cap_mode)


@pytest.mark.parametrize("k", [4, 5])
def test_graph_workload_rows(env, k):
    dm, lib, torch = env
    announce("graph workload rows", k)
    w, pos = _sampled(k)
    rows = np.random.default_rng(k).choice(w.n_dst, 400, replace=False)
    rows = np.concatenate([rows, [0, w.n_dst - 1]])
    _check_graph(lib, torch, pos, w.n_dst, w.r, w.cap, w.cap_mode, rows=rows)


@pytest.mark.parametrize("n,n_dst,r,cap,mode", [(600, 500, 0.1, 0, 0), (600, 600, 0.1, 0, 0), (600, 500, 0.1, 6, 0),
                                                (600, 500, 0.1, 6, 1), (8300, 400, 0.05, 0, 0),
                                                (8300, 400, 0.05, 6, 0), (600, 500, 1e30, 30, 0)])
def test_graph_of_coordinates_that_are_not_finite(env, n, n_dst, r, cap, mode):
    """Both forms of the grid with infinite and NaN coordinates among the points:
    such points have no edges, the others theirs (a radius whose square
    overflows reaches the infinite ones too)."""
    dm, lib, torch = env
    announce("graph, infinite coordinates", n, n_dst, r, cap, mode)
    pos = _rand(n, 3, 60)
    pos[[3, n_dst - 1, n - 1], [0, 1, 2]] = np.inf
    pos[[7, n - 2]] = -np.inf
    pos[9, 1] = np.nan
    with np.errstate(invalid="ignore", over="ignore"):
        rp, col = org.radius_graph(pos, n_dst, r, cap, mode, 5, method="brute")
    g = lib.dsmp_radius_graph_build(torch.from_numpy(pos).cuda(), n_dst, r, cap, mode, 5, capacity=int(rp[-1]))
    assert np.array_equal(g.row_ptr.cpu().numpy(), rp) and np.array_equal(g.col.cpu().numpy()[:rp[-1]], col)
    assert np.array_equal(g.csc_eid.cpu().numpy()[:rp[-1]], org.transpose(rp, col, n)[1])


def test_graph_is_deterministic(env):
    dm, lib, torch = env
    pos = torch.from_numpy(_rand(20000, 3, 30)).cuda()
    a = lib.dsmp_radius_graph_build(pos, 20000, 0.05, 10)
    b = lib.dsmp_radius_graph_build(pos, 20000, 0.05, 10)
    for x, y in ((a.row_ptr, b.row_ptr), (a.col, b.col), (a.csc_eid, b.csc_eid)):
        assert torch.equal(x, y)


def test_two_threads_on_one_handle_get_their_own_totals(env):
    """Graph builds and sub-domain selections of two host threads through one
    handle, each with its own buffers and workspace (the library's C interface:
    the binding keeps one workspace per handle)."""
    dm, lib, torch = env
    announce("two threads, one handle")
    L, c = lib.lib, ctypes
    lib._bind()

    def graph_job(seed, n, r):
        pos = torch.from_numpy(_rand(n, 2, seed)).cuda()
        q, _ = lib._query(pos, n, r, 0, dm.CAP_KNN, 0)
        nb = c.c_size_t()
        assert L.dsmp_radius_graph_workspace(c.byref(q), c.byref(nb)) == dm.OK
        ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
        rp, _ = org.radius_graph(pos.cpu().numpy(), n, r)
        E = c.c_int64()

        def call():
            st = L.dsmp_radius_graph_count(lib.h, c.byref(q), c.c_void_p(ws.data_ptr()), ws.numel(), c.byref(E))
            return (st, E.value) == (dm.OK, int(rp[-1]))
        return call, pos

    def box_job(seed, n, hi):
        pos_np = _rand(n, 2, seed)
        pos = torch.from_numpy(pos_np).cuda()
        nb, a, b = c.c_size_t(), c.c_int64(), c.c_int64()
        assert L.dsmp_subdomain_workspace(n, c.byref(nb)) == dm.OK
        ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
        idx = torch.empty(n, dtype=torch.int32, device="cuda")
        lo_c, hi_c = (c.c_float * 2)(0.0, 0.0), (c.c_float * 2)(hi, hi)
        own = int((pos_np < np.float32(hi)).all(1).sum())

        def call():
            st = L.dsmp_subdomain_select(lib.h, c.c_void_p(pos.data_ptr()), n, 2, lo_c, hi_c, 0.0,
                                         c.c_void_p(idx.data_ptr()), c.c_void_p(ws.data_ptr()), ws.numel(),
                                         c.byref(a), c.byref(b))
            return (st, a.value, b.value) == (dm.OK, own, own)
        return call, pos

    jobs = [[graph_job(50, 1000, 0.05), box_job(51, 3000, 0.4)], [graph_job(52, 20000, 0.01), box_job(53, 12000, 0.7)]]
    torch.cuda.synchronize()
    wrong = [0, 0]

    def work(t):
        for _ in range(200):
            wrong[t] += sum(not call() for call, _ in jobs[t])

    threads = [threading.Thread(target=work, args=(t,)) for t in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert wrong == [0, 0]
