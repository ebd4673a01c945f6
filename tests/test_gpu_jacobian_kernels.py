"""The kernels of the Jacobian path's larger bases against the oracle, at the
sizes where they can go wrong: the radial pass (table and direct), the edge
Jacobian kernel of eight-edge chunks, the density step on the matrix cores."""
import numpy as np
import pytest

import oracle
from paper_2609_05709_amd import workloads
from tests.parity import TOL, gpu_run, jacobian_errors, row_errors

pytestmark = pytest.mark.gpu

MODES = [("float32", "mixed"), ("float32", "fp64"), ("float64", "mixed")]


def _check(wl, st, dtype, arith="mixed", centers=None):
    print(f"[kernels] {wl.name} {dtype} {arith}", flush=True)
    g = gpu_run(wl, st, dtype, centers=centers, arith=arith)
    idx = np.arange(st.n_atoms) if centers is None else np.asarray(centers)
    ref = oracle.OracleSOAP(wl.species, wl.r_cut, wl.n_max, wl.l_max, wl.sigma, wl.rbf).compute(
        st.pos64, st.Z, centers=idx, jacobian=True)
    ed = row_errors(g["desc"], ref["desc"]).max()
    ej = jacobian_errors(g, ref, st, wl.species, range(len(idx)), idx)
    print(f"[kernels] {wl.name} {dtype} {arith}: desc {ed:.2e} jac {ej:.2e}", flush=True)
    assert ed < TOL[dtype] and ej < TOL[dtype]


def _wl(species, rbf, n, l, r_cut=4.5, sigma=0.5):
    return workloads.Workload(f"s{len(species)}_{rbf}_n{n}l{l}", tuple(species), rbf, r_cut, sigma, n, l, True,
                              ("none",))


# (species, n, l): one and two matrix-core column tiles at their edges (S n = 15,
# 16, 18, 32, 33, 64), one degree, the last
# degree, odd and even degree counts, one radial function
BASES = [((1,), 1, 0), ((1,), 1, 1), ((1,), 15, 3), ((1, 8), 8, 4), ((1, 8), 9, 5), ((1, 8), 16, 2),
         ((1, 6, 8), 11, 6), ((1, 6, 7, 8), 16, 3), ((1, 8), 5, 14), ((1, 8), 12, 13)]


@pytest.mark.parametrize("dtype,arith", MODES)
@pytest.mark.parametrize("species,n,l", BASES)
def test_basis_edges(species, n, l, dtype, arith):
    """Rows from none to some tens of neighbours, so chunks of one to eight
    edges and species runs of every remainder."""
    st = workloads.random_small(40, 7 + n, 4.0, species=species, dmin=0.9)
    st.pos[-1] += np.float32(40.0)  # one atom without neighbours
    _check(_wl(species, "polynomial", n, l), st, dtype, arith)


@pytest.mark.parametrize("dtype,arith", MODES)
def test_long_rows(dtype, arith):
    """Rows longer than one row block of the edge Jacobian kernel (128 edges)
    and than one chunk per species of the density step (64)."""
    st = workloads.random_small(330, 5, 4.6, species=(1, 8), dmin=0.7)
    _check(_wl((1, 8), "polynomial", 8, 7, r_cut=5.0), st, dtype, arith, centers=[0, 11, 200, 329])


@pytest.mark.parametrize("dtype,arith,rbf,n,l,sigma",
                         [("float32", "fp64", "gto", 8, 8, 0.5),    # factors evaluated directly
                          ("float64", "mixed", "gto", 8, 12, 0.5),
                          ("float64", "mixed", "gto", 12, 6, 0.5),  # compensated
                          ("float32", "mixed", "gto", 9, 9, 0.02),  # too many intervals for a table
                          ("float32", "mixed", "gto", 9, 9, 0.5),   # from the table
                          ("float64", "mixed", "polynomial", 8, 8, 0.5),
                          ("float32", "mixed", "polynomial-laplace", 8, 8, 0.5)])
def test_coincident_neighbours_in_dense_rows(dtype, arith, rbf, n, l, sigma):
    """Atoms at one place in rows long enough for the density step on the matrix
    cores: a zero-length edge is an on-site term with a zero gradient, whichever
    evaluation the radial factors come from."""
    import torch
    from paper_2609_05709_amd.soap import Soap
    st = workloads.random_small(40, 3, 4.0, species=(1, 8), dmin=0.9)
    st.pos[7] = st.pos[3]
    st.pos[20] = st.pos[21]
    wl = _wl((1, 8), rbf, n, l, r_cut=6.0, sigma=sigma)
    sp = Soap(wl.species, wl.r_cut, n, l, sigma, rbf, dtype=dtype, arith=arith)
    sp.build_neighbors(torch.from_numpy(st.pos).to("cuda", torch.float64 if dtype == "float64" else torch.float32),
                       torch.from_numpy(st.Z).cuda())
    assert sp.get_option("jacobian_density_kernel") == 3
    sp.close()
    _check(wl, st, dtype, arith)


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("rbf,sigma", [("polynomial", 0.5), ("polynomial", 0.3), ("gto", 0.5),
                                       ("gto", 0.3), ("gto", 0.12), ("gto", 0.02),
                                       ("polynomial-laplace", 0.3)])
def test_radial_pass_distances(rbf, sigma, dtype):
    """Dimers over every distance: coincident, nearly so, at the table's
    interval boundaries and around them, up to the last value below the
    cutoff.  GTO in float32 has a table at sigma 0.3 and none at 0.12, and nothing has
    one at 0.02 (too many intervals; the oracle's Bessel functions end before the quadrature's would); the Laplace form
    never has one and starts where it is an expansion at all."""
    rc = 5.0
    h = float(np.exp2(np.floor(np.log2(sigma / (20.0 if dtype == "float64" else 16.0)))))  # an interval
    k = np.float32(h * np.floor(2.0 / h))
    last = float(np.nextafter(np.float32(rc), np.float32(0)))
    d = [0.5, 1.0, 2.345, k, np.nextafter(k, np.float32(0)), np.nextafter(k, np.float32(9)), rc - h / 2, last]
    if rbf != "polynomial-laplace":
        d += [0.0, 1e-3, 0.05, h, h / 3]
    pos, Z = [], []
    for k, r in enumerate(d):  # the x coordinates start at 0, so that r is the exact float32 distance
        pos += [[0.0, 20.0 * k, 0.0], [r, 20.0 * k, 0.0]]
        Z += [1, 8]
    st = workloads.Structure(np.array(pos, dtype=np.float32), np.array(Z, dtype=np.int32), 0.0, 0)
    _check(_wl((1, 8), rbf, 10 if rbf == "gto" else 6, 12 if rbf == "gto" else 5, r_cut=rc, sigma=sigma), st, dtype)


@pytest.mark.parametrize("dtype,arith", MODES)
@pytest.mark.parametrize("n,l", [(4, 12), (10, 10), (12, 6)])
def test_density_step_matrix_and_shared(n, l, dtype, arith):
    """The density step on the matrix cores (rows of eight and more edges per
    species) and the shared density kernel (djs_tile -1) on the same rows."""
    import torch
    from paper_2609_05709_amd.soap import Soap
    st = workloads.water_cluster(64, 0)
    tdt = torch.float64 if dtype == "float64" else torch.float32
    pos, Z = torch.from_numpy(st.pos).to("cuda", tdt), torch.from_numpy(st.Z).cuda()
    out = []
    for tile in (0, -1):
        sp = Soap((1, 8), 5.0, n, l, 0.5, "polynomial", dtype=dtype, arith=arith)
        sp.set_option("djs_tile", tile)
        sp.build_neighbors(pos, Z)
        assert sp.get_option("jacobian_density_kernel") == (3 if tile == 0 else 0)
        out.append([t.double() for t in sp.derivatives()])
        again = sp.derivatives()
        assert all(torch.equal(a.double(), b) for a, b in zip(again, out[-1]))
        sp.close()
    for a, b in zip(*out):
        scale = b.abs().flatten(1).max(1).values
        err = (a - b).abs().flatten(1).max(1).values
        assert torch.all(err <= TOL[dtype] * scale)


def _dimers(n_pairs, r_cut):
    """Pairs of atoms far apart, in random directions at distances over (0, r_cut)."""
    rng = np.random.default_rng(1)
    pos = np.zeros((2 * n_pairs, 3))
    pos[:, 1] = np.repeat(20.0 * np.arange(n_pairs), 2)
    v = rng.standard_normal((n_pairs, 3))
    pos[1::2] += v / np.linalg.norm(v, axis=1)[:, None] * rng.uniform(0.3, 0.98 * r_cut, n_pairs)[:, None]
    return workloads.Structure(pos.astype(np.float32), np.tile([1, 8], n_pairs).astype(np.int32), 0.0, 0)


@pytest.mark.parametrize("rbf,n,l,bound_c,bound_j", [("polynomial", 8, 6, 2.2e-15, 1.9e-15),
                                                     ("polynomial", 4, 3, 1.3e-15, 1.5e-15),
                                                     ("gto", 10, 4, None, 7.3e-16)])
def test_float64_table_keeps_the_direct_evaluations_bits(rbf, n, l, bound_c, bound_j):
    """Float64 dimers through the radial table: the root mean square errors of the
    coefficients (the polynomial's; GTO coefficients don't use the table) and of
    the center blocks are no larger than with every factor evaluated from its
    definition (the bounds: measured so, against the same oracle in long double)."""
    st = _dimers(400, 6.0)
    wl = _wl((1, 8), rbf, n, l, r_cut=6.0)
    print(f"[kernels] table {wl.name}", flush=True)
    g = gpu_run(wl, st, "float64", coefficients=True)
    ref = oracle.OracleSOAP(wl.species, wl.r_cut, n, l, wl.sigma, rbf).compute(
        st.pos64, st.Z, centers=np.arange(800), jacobian=True, coefficients=True)
    k, o = np.arange(800), np.tile([1, 0], 400)  # the neighbour's species
    c, cr = (a.reshape(800, 2, n, -1)[k, o] for a in (g["c"], ref["c"]))
    ec = np.abs(c - cr).max(-1) / np.abs(cr).max(-1)  # per center and radial index
    ej = []
    for i in range(800):
        b = [b for b in range(ref["blk_ptr"][i], ref["blk_ptr"][i + 1]) if ref["blk_j"][b] == i][0]
        ej.append(np.abs(g["jself"][i] - ref["jac"][b]).max() / np.abs(ref["jac"][b]).max())
    rc, rj = np.sqrt(np.mean(ec ** 2)), np.sqrt(np.mean(np.square(ej)))
    print(f"[kernels] table {wl.name}: coefficients {rc:.2e}, center blocks {rj:.2e}", flush=True)
    assert bound_c is None or rc < bound_c
    assert rj < bound_j


@pytest.mark.parametrize("n,l", [(8, 6), (10, 4)])
def test_float32_table_at_the_factors_zeros(n, l):
    """Mixed arithmetic: the factor is rounded to float32 once, so a dimer's
    coefficients, one factor times one harmonic, keep their digits also where a
    factor passes through zero.  Three roundings to float32 are 1.8e-7; the table
    adds up to 1e-7 of a value within 1e-4 of a zero."""
    st = _dimers(400, 6.0)
    wl = _wl((1, 8), "polynomial", n, l, r_cut=6.0)
    print(f"[kernels] zeros {wl.name}", flush=True)
    g = gpu_run(wl, st, "float32", jacobian=False, coefficients=True)
    ref = oracle.OracleSOAP(wl.species, wl.r_cut, n, l, wl.sigma, wl.rbf).compute(
        st.pos64, st.Z, centers=np.arange(800), coefficients=True)
    k, o = np.arange(800), np.tile([1, 0], 400)
    c, cr = (a.reshape(800, 2, n, -1)[k, o] for a in (g["c"], ref["c"]))
    e = np.abs(c - cr)[cr != 0] / np.abs(cr[cr != 0])
    print(f"[kernels] zeros {wl.name}: max {e.max():.2e}, rms {np.sqrt(np.mean(e ** 2)):.2e}", flush=True)
    assert e.max() < 2.8e-7


@pytest.mark.parametrize("n,l,tile", [(4, 5, 3), (5, 5, 3), (8, 3, 3), (3, 6, 3), (2, 2, 4), (8, 6, 2)])
def test_float64_tile_plan(n, l, tile):
    """The float64 edge Jacobian kernel takes the widest tile that keeps three
    workgroups per CU, not a narrower one for the sake of a fourth."""
    from paper_2609_05709_amd.soap import Soap
    sp = Soap((1, 8), 5.5, n, l, 0.5, "gto", dtype="float64")
    assert (sp.get_option("jacobian_kernel"), sp.get_option("jacobian_tile")) == (0, tile)
    sp.close()


def _table_context(arith):
    """A small polynomial structure with its neighbour rows, and the outputs of both arithmetics."""
    import torch
    from paper_2609_05709_amd.soap import Soap
    st = workloads.random_small(60, 4, 4.5, species=(1, 8), dmin=0.9)
    pos, Z = torch.from_numpy(st.pos).cuda(), torch.from_numpy(st.Z).cuda()
    ref = []
    for a in ("mixed", "fp64"):
        sp = Soap((1, 8), 5.0, 6, 5, 0.5, "polynomial", arith=a)
        sp.build_neighbors(pos, Z)
        ref.append([t.clone() for t in sp.derivatives()])
        sp.close()
    assert not torch.equal(ref[0][1], ref[1][1])
    sp = Soap((1, 8), 5.0, 6, 5, 0.5, "polynomial", arith=arith)
    sp.build_neighbors(pos, Z)
    return sp, ref


def test_options_leave_queued_calls_alone():
    """A call queued behind other work on its own stream keeps the arithmetic it
    was made with, and its radial table, when the option changes before it runs."""
    import torch
    sp, ref = _table_context("fp64")
    busy = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for k in range(3):  # both tables exist from the second pass on
        print(f"[kernels] queued calls {k}", flush=True)
        with torch.cuda.stream(side):
            for _ in range(10):
                busy = busy @ busy
                busy /= busy.norm()
            wide = [t.clone() for t in sp.derivatives()]
        sp.set_option("arith", 0)
        with torch.cuda.stream(side):
            mixed = [t.clone() for t in sp.derivatives()]
        sp.set_option("arith", 1)
        side.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(wide, ref[1]))
        assert all(torch.equal(a, b) for a, b in zip(mixed, ref[0]))
    sp.close()


def test_captured_calls_keep_their_table():
    """A graph captured over the allocation-free call gives the same outputs after
    the arithmetic was changed and calls in the other one ran."""
    import ctypes

    import torch
    sp, ref = _table_context("mixed")
    out = [torch.empty_like(t) for t in ref[0]]

    def call():
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert sp._L.soap_derivatives_batch_noalloc(sp._h, 0, sp.n_centers, *(t.data_ptr() for t in out), stream) == 0

    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for k in range(3):
        print(f"[kernels] replay {k}", flush=True)
        sp.set_option("arith", 1)
        wide = sp.derivatives()
        assert all(torch.equal(a, b) for a, b in zip(wide, ref[1]))
        for t in out:
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, ref[0]))
        sp.set_option("arith", 0)
    sp.close()


def test_noalloc_call_after_a_change_of_arithmetic():
    """One species and one radial function: in float64 arithmetic an edge's block
    cannot hold its factors.  Their buffer is there when the arithmetic changes
    after the neighbour build: the call can be captured, which an allocation would
    end with an error."""
    import ctypes

    import torch
    from paper_2609_05709_amd.soap import Soap
    st = workloads.random_small(50, 4, 4.0, species=(8,), dmin=0.9)
    pos, Z = torch.from_numpy(st.pos).cuda(), torch.from_numpy(st.Z).cuda()
    sp = Soap((8,), 5.0, 1, 4, 0.5, "polynomial", arith="fp64")
    sp.build_neighbors(pos, Z)
    ref = [t.clone() for t in sp.derivatives()]
    sp.close()
    sp = Soap((8,), 5.0, 1, 4, 0.5, "polynomial")
    sp.build_neighbors(pos, Z)
    sp.set_option("arith", 1)
    out = [torch.full_like(t, float("nan")) for t in ref]
    torch.cuda.synchronize()
    print("[kernels] capture after a change of arithmetic", flush=True)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        rc = sp._L.soap_derivatives_batch_noalloc(sp._h, 0, sp.n_centers, *(t.data_ptr() for t in out), stream)
    assert rc == 0
    graph.replay()
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(out, ref))
    sp.close()


def test_more_centers_than_one_launch_holds():
    """8.4 million centers at 512 threads each are more threads than a launch may
    have.  All but three of them are one isolated atom."""
    import torch
    from paper_2609_05709_amd.soap import Soap
    nc = 2 ** 32 // 512 + 3
    pos = torch.tensor([[0.0, 0, 0], [50, 0, 0], [51.1, 0.4, -0.3], [50.2, -0.9, 0.8]], device="cuda")
    Z = torch.tensor([8, 8, 1, 1], dtype=torch.int32, device="cuda")
    print("[kernels] many centers", flush=True)
    blocks = []
    for centers in (torch.arange(4, dtype=torch.int32), torch.zeros(nc, dtype=torch.int32)):
        centers[-3:] = torch.arange(1, 4, dtype=torch.int32)
        sp = Soap((1, 8), 4.0, 9, 0, 0.5, "polynomial")
        assert sp.build_neighbors(pos, Z, centers.cuda()) == 6
        desc, edge, own = sp.derivatives()
        assert sp.get_option("jacobian_kernel") == 1
        blocks.append([edge.clone(), desc[-4:].clone(), own[-4:].clone()])
        sp.close()
        del desc, edge, own
    torch.cuda.empty_cache()
    for a, b in zip(*blocks):
        assert a.abs().max() > 0 and torch.equal(a, b)


@pytest.mark.parametrize("rbf,n,l,arith", [("gto", 3, 2, "fp64"), ("gto", 5, 3, "fp64"), ("polynomial", 2, 4, "mixed"),
                                           ("polynomial", 7, 3, "mixed"), ("polynomial", 4, 2, "fp64"),
                                           ("polynomial-laplace", 3, 5, "mixed")])
def test_wave_tiles_of_small_bases(rbf, n, l, arith):
    """Small bases on 512 centers and more take the edge Jacobian kernel of wave
    tiles, on fewer the one of whole workgroups; a batch of the list takes its
    kernel, with the same bits."""
    import torch
    from paper_2609_05709_amd.soap import Soap
    wl = _wl((1, 8), rbf, n, l, r_cut=3.5)
    for atoms, kernel in ((511, 1), (512, 0)):
        st = workloads.random_small(atoms, 6, 8.5, species=(1, 8), dmin=0.8)
        sp = Soap(wl.species, wl.r_cut, n, l, wl.sigma, rbf, arith=arith)
        sp.build_neighbors(torch.from_numpy(st.pos).cuda(), torch.from_numpy(st.Z).cuda())
        assert sp.get_option("jacobian_kernel") == kernel
        row = sp.neighbors()[0].cpu().numpy()
        desc, edge, own = sp.derivatives()
        b = sp.derivatives_batch(100, 57, int(row[157] - row[100]))
        assert torch.equal(b[0], desc[100:157]) and torch.equal(b[1], edge[row[100]:row[157]])
        assert torch.equal(b[2], own[100:157])
        sp.close()
        _check(wl, workloads.Structure(st.pos, st.Z, 0.0, 0), "float32", arith, centers=None if atoms == 512 else [0, 3])


@pytest.mark.parametrize("n,l,dtype,arith,least", [(2, 2, "float32", "mixed", 384), (4, 4, "float32", "mixed", 384),
                                                   (6, 3, "float32", "mixed", 512), (2, 6, "float32", "mixed", 384),
                                                   (3, 4, "float32", "fp64", 512), (5, 3, "float64", "mixed", 512)])
def test_laplace_form_in_the_kernels(n, l, dtype, arith, least):
    """The Laplace form of small bases is evaluated in the density and edge
    Jacobian kernels from a number of centers on, by the radial pass below it;
    a batch of the list takes its kernels, with the same bits."""
    import torch
    from paper_2609_05709_amd.soap import Soap
    wl = _wl((1, 8), "polynomial-laplace", n, l, r_cut=3.5)
    tdt = torch.float64 if dtype == "float64" else torch.float32
    for atoms in (least - 1, least):
        st = workloads.random_small(atoms, 6, 8.5, species=(1, 8), dmin=0.8)
        sp = Soap(wl.species, wl.r_cut, n, l, wl.sigma, wl.rbf, dtype=dtype, arith=arith)
        sp.build_neighbors(torch.from_numpy(st.pos).to("cuda", tdt), torch.from_numpy(st.Z).cuda())
        assert (sp.get_option("jacobian_density_kernel") == 0) == (atoms == least)
        row = sp.neighbors()[0].cpu().numpy()
        desc, edge, own = sp.derivatives()
        b = sp.derivatives_batch(100, 57, int(row[157] - row[100]))
        assert torch.equal(b[0], desc[100:157]) and torch.equal(b[1], edge[row[100]:row[157]])
        assert torch.equal(b[2], own[100:157])
        sp.close()
        _check(wl, workloads.Structure(st.pos, st.Z, 0.0, 0), dtype, arith)


# S n (l_max + 1) below and from 240 on (float64 outputs 144), at S n >= 32, in float64 arithmetic
@pytest.mark.parametrize("rbf,n,l,dtype,arith,kernel",
                         [("polynomial", 10, 5, "float32", "mixed", 1), ("polynomial", 9, 5, "float32", "fp64", 1),
                          ("polynomial", 10, 5, "float32", "fp64", 2),
                          ("gto", 12, 4, "float32", "fp64", 2), ("polynomial-laplace", 8, 3, "float64", "mixed", 1),
                          ("gto", 12, 2, "float64", "mixed", 2), ("polynomial", 9, 6, "float64", "mixed", 2)])
def test_streamed_coefficients_of_several_species(rbf, n, l, dtype, arith, kernel):
    """Bases of many radial functions and species stream their coefficients to
    the output kernel on short rows, with the explicit choice left alone; not in the
    mixed arithmetic, whose scratch is float32."""
    import torch
    from paper_2609_05709_amd.soap import Soap
    wl = _wl((1, 6, 7, 8), rbf, n, l, r_cut=3.5)
    st = workloads.random_small(150, 6, 6.5, species=(1, 6, 7, 8), dmin=0.8)
    sp = Soap(wl.species, wl.r_cut, n, l, wl.sigma, rbf, dtype=dtype, arith=arith)
    sp.build_neighbors(torch.from_numpy(st.pos).to("cuda", sp.dtype), torch.from_numpy(st.Z).cuda())
    assert sp.get_option("jacobian_density_kernel") == kernel
    sp.set_option("djac_tile", 32)
    assert sp.get_option("jacobian_density_kernel") == 1
    sp.close()
    _check(wl, st, dtype, arith)


@pytest.mark.parametrize("species,rbf,n,l,arith,least,above",
                         [((1, 6, 7, 8), "gto", 5, 1, "fp64", 512, 0), ((1, 6, 7, 8), "gto", 4, 2, "fp64", 512, 0),
                          ((1, 6, 8), "polynomial", 9, 1, "mixed", 1024, 0), ((1, 6, 7, 8), "polynomial", 5, 4, "mixed", 1024, 0),
                          ((1, 6, 7, 8), "polynomial", 12, 2, "mixed", 1024, 0), ((1, 6, 8), "polynomial", 6, 5, "mixed", 1024, 1)])
def test_wave_tiles_of_several_species(species, rbf, n, l, arith, least, above):
    """With three species and more the edge Jacobian kernel of wave tiles takes
    more of the bases (above: the kernel from `least` centers on)."""
    import torch
    from paper_2609_05709_amd.soap import Soap
    wl = _wl(species, rbf, n, l, r_cut=3.0)
    for atoms, kernel in ((least - 1, 1), (least, above)):
        st = workloads.random_small(atoms, 6, 10.5, species=species, dmin=0.8)
        sp = Soap(wl.species, wl.r_cut, n, l, wl.sigma, rbf, arith=arith)
        sp.build_neighbors(torch.from_numpy(st.pos).cuda(), torch.from_numpy(st.Z).cuda())
        assert sp.get_option("jacobian_kernel") == kernel
        sp.close()
    _check(wl, st, "float32", arith)
