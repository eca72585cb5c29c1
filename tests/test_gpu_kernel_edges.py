"""Kernels and dispatch branches at the sizes where they can go wrong: block
remainders, the smallest surfaces and the first sizes past a branch, each
against the oracle or the path the oracle already pins."""
import time

import numpy as np
import pytest

import oracle
import pbgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_21713_amd as pb
    return pb.Context(0)


def rel2(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


# 64-triangle blocks: 20 triangles (one ragged block), 80 (two), 1280 (20 full
# blocks), 9680 (152 blocks: two groups of block slots, the second ragged)
@pytest.mark.parametrize("n", [1, 2, 8, 22])
@pytest.mark.parametrize("precision,bar", [(0, 1e-13), (1, 1e-6)])
def test_matrix_free_blocks_match_dense(ctx, n, precision, bar):
    """The same integrals as the stored operators in another order: FP64 to
    rounding (sums of up to 1e4 terms of one sign pattern, 1e-13 in the
    2-norm), FP32 evaluation to FP32 rounding of every term (1e-6)."""
    import paper_2511_21713_amd as pb
    prob = pbgen.make_problem(n=n, a=6.0, c=9.0, bump=n > 2, t=3.0, L=2, helix=0, partials=0, kappa=0.2, seed=(9, n),
                              center_charge=1.0)
    rng = np.random.default_rng(n)
    g = pb.Problem.from_inputs(ctx, prob, precision=precision)
    v = rng.standard_normal(g.n)
    phi = rng.standard_normal(g.n)
    dense = g.apply_jacobian(pb.LIN, phi, v)
    g.set_bem_mode(pb.BEM_MATRIX_FREE)
    mf = g.apply_jacobian(pb.LIN, phi, v)
    again = g.apply_jacobian(pb.LIN, phi, v)
    nn = g.n_nodes
    for lo, hi in ((nn, nn + g.n_m), (nn + g.n_m, g.n)):
        e = rel2(mf[lo:hi], dense[lo:hi])
        print(f"  n {n} precision {precision}: {e:.2e}", flush=True)
        assert e < bar
    assert np.array_equal(mf, again)
    g.close()


TIGHT = dict(tol_nl=1e-10, tol_gr=1e-11, tol_gr0=1e-11, tol_omega=1e-9, l_e=0.0, max_gmres=20000)


@pytest.fixture(scope="module")
def sphere(ctx):
    """1 458 unknowns: six Gram-Schmidt chunks, the last one ragged."""
    import paper_2511_21713_amd as pb
    prob = pbgen.make_config(0)
    o = oracle.Oracle.from_problem(prob)
    res, pl, pnl = o.solve(**TIGHT)
    return pb.Problem.from_inputs(ctx, prob), res, pl + pnl


# the first launch carries terms 0 and 1 of the preconditioner, the last term
# packs the apply's input: one, two and three terms and none; restarts: a
# cycle end after every step, inside a solve, and never
@pytest.mark.parametrize("opts", [dict(cheb_degree=1), dict(cheb_degree=2), dict(cheb_degree=3), dict(precond=0),
                                  dict(gmres_restart=7), dict(gmres_restart=33), dict(cheb_degree=2, gmres_restart=9),
                                  dict(hip_graph=0), dict(cheb_degree=64)])
def test_krylov_step_variants_reach_the_same_solution(sphere, opts):
    """Every preconditioner and restart length solves the same systems to
    1e-11, so the converged potentials agree to 1e-8 and the energies to 1e-9."""
    import torch
    g, ref, phi = sphere
    out = torch.zeros(2 * g.n, dtype=torch.float64, device="cuda:0")
    torch.cuda.synchronize()
    r = g.solve(phi_out=out, **{**TIGHT, **opts})
    u = out.cpu().numpy()
    e, d = abs(r["total"] - ref["total"]) / abs(ref["total"]), rel2(u[:g.n] + u[g.n:], phi)
    print(f"  {opts}: energy {e:.2e}, potential {d:.2e}, {r['gmres_iters_total']} steps", flush=True)
    assert e < 1e-9 and d < 1e-8
    again = g.solve(phi_out=out, **{**TIGHT, **opts})
    assert again["total"] == r["total"] and np.array_equal(out.cpu().numpy(), u)


# 256 x 96 = 24 576 rows is where a Gram-Schmidt chunk grows past one row per
# thread: unknowns just below and above (n = 13, 11 layers: 23 688; 12: 25 380);
# 2 048 FEM rows is where the preconditioner stage leaves its single workgroup
# (n = 4, 11 layers: 1 944; 12: 2 106); 7 layers (1 296): rows past one per thread
@pytest.mark.parametrize("n,layers", [(13, 11), (13, 12), (4, 11), (4, 12), (4, 7)])
@pytest.mark.parametrize("precision,tol", [(0, 1e-8), (1, 1e-5)])
def test_linear_solve_around_the_edges_of_its_kernels(ctx, n, layers, precision, tol):
    """A solve's own residual: the linear system's at the returned Phi_L is
    below the tolerance GMRES stopped at (mixed: the residual call takes the
    FP64 FEM values where GMRES took them in FP32, 6e-8 of a row)."""
    import torch
    import paper_2511_21713_amd as pb
    prob = pbgen.make_problem(n=n, a=8.0, c=10.0, bump=True, t=4.0, L=layers, helix=2, partials=20, kappa=0.125,
                              seed=(3, layers))
    g = pb.Problem.from_inputs(ctx, prob, precision=precision)
    out = torch.zeros(2 * g.n, dtype=torch.float64, device="cuda:0")
    torch.cuda.synchronize()
    r = g.solve(phi_out=out, tol_gr0=tol, tol_gr=tol)
    F = g.residual(pb.LIN, out[:g.n].contiguous())
    b = g.export_rhs()
    rel = float(torch.linalg.norm(F)) / np.linalg.norm(b)
    print(f"  unknowns {g.n} precision {precision}: {rel:.2e} after {r['gmres_lin']} steps", flush=True)
    assert rel < 1.1 * tol  # the estimate differs from the residual by rounding
    g.close()


# full rows beside the SpMV below 160 MiB a surface (FP64: n = 17 the last, 18
# the first past it; FP32: 21 and 22), the symmetric use above; n = 1: one
# ragged workgroup
@pytest.mark.parametrize("n,precision", [(1, 0), (1, 1), (6, 0), (6, 1), (17, 0), (18, 0), (21, 1), (22, 1)])
def test_dense_rows_of_either_form_match_the_stored_blocks(ctx, n, precision):
    """The surface rows of a product against numpy's with the exported blocks:
    FP64 sums of up to 1e4 terms, 1e-13 in the 2-norm, in both precisions (the
    export is what is stored)."""
    import paper_2511_21713_amd as pb
    prob = pbgen.make_problem(n=n, a=6.0, c=9.0, bump=n > 2, t=3.0, L=1, helix=0, partials=0, kappa=0.2, seed=(9, n),
                              center_charge=1.0)
    g = pb.Problem.from_inputs(ctx, prob, precision=precision)
    g.set_tile_shape(16, 16)
    rng = np.random.default_rng(n)
    v, phi = rng.standard_normal(g.n), rng.standard_normal(g.n)
    y = g.apply_jacobian(pb.LIN, phi, v)
    nn, nm = g.n_nodes, g.n_m
    for surf, ids, lo in ((0, np.unique(prob.tri_m), nn), (1, np.unique(prob.tri_s), nn + nm)):
        V, K = g.export_bem(surf)
        ref = K @ v[ids] + V @ v[lo:lo + ids.size]
        e = rel2(y[lo:lo + ids.size], ref)
        print(f"  n {n} precision {precision} surface {surf}: {e:.2e}", flush=True)
        assert e < 1e-13
    g.close()


# the centre of a meshed solute joins 12 (n = 1), 42 (2: a 43-entry row, so the
# element sums take one plane of LDS), 92 (3) and 252 (5) nodes: the last two
# are rows past 64 entries, kept outside their slice
@pytest.mark.parametrize("n", [1, 2, 3, 5])
def test_rows_of_many_neighbours_match_oracle(ctx, n):
    """Residual, Jacobian product (FP64, 1e-12 of the largest entry, the bar of
    the other products) and a tight solve with the relaxation search on meshes
    with one long row."""
    import paper_2511_21713_amd as pb
    prob = pbgen.make_problem(n=n, a=5.0, c=6.0, bump=False, t=3.0, L=2, helix=0, partials=0, kappa=0.2,
                              center_charge=2.0, solute_layers=1, seed=(4, n))
    o = oracle.Oracle.from_problem(prob)
    g = pb.Problem.from_inputs(ctx, prob)
    rng = np.random.default_rng(n)
    phi, v = rng.standard_normal(g.n), rng.standard_normal(g.n)
    for scheme in (pb.T3, pb.HS):
        for got, ref in ((g.residual(scheme, phi), o.residual(scheme, phi)),
                         (g.apply_jacobian(scheme, phi, v), o.apply_jacobian(scheme, phi, v))):
            e = np.abs(got - ref).max() / np.abs(ref).max()
            print(f"  n {n} scheme {scheme}: {e:.2e}", flush=True)
            assert e < 1e-12
    ref = o.solve(**TIGHT)[0]["total"]
    r = g.solve(**TIGHT)
    assert abs(r["total"] - ref) < 1e-10 * abs(ref)
    m = pb.Problem.from_inputs(ctx, prob, precision=pb.MIXED)
    assert abs(m.solve()["total"] - ref) < 1e-5 * abs(ref)
    m.close()
    g.close()


# 192 MiB of planes over the blocks' local vertices is where the assembly leaves
# its single tile launch: FP64 between n = 11 and 12, FP32 between 13 and 14;
# n = 1: two blocks, every vertex in both; n = 2: five
@pytest.mark.parametrize("n,precision", [(1, 0), (2, 1), (11, 0), (12, 0), (13, 1), (14, 1)])
def test_assembly_of_small_surfaces_matches_oracle_rows(ctx, n, precision):
    """Sampled rows of both stored operators against the oracle's, at the bars
    of the full-size rows; V' bitwise symmetric away from the touching pairs."""
    import paper_2511_21713_amd as pb
    prob = pbgen.make_problem(n=n, a=6.0, c=9.0, bump=n > 2, t=3.0, L=1, helix=0, partials=0, kappa=0.2, seed=(9, n),
                              center_charge=1.0)
    o = oracle.Oracle.from_problem(prob)
    g = pb.Problem.from_inputs(ctx, prob, precision=precision)
    g.set_tile_shape(16, 16)
    for surf in (0, 1):
        nv = o.n_m if surf == 0 else o.n_s
        rng = np.random.default_rng(n + surf)
        rows = np.unique(np.r_[0, nv - 1, rng.choice(nv, size=min(nv, 20), replace=False)])
        V, K = o.bem_rows(surf, rows)
        sV, sK = (-1.0, 1.0) if surf == 0 else (1.0, -1.0)
        x = rng.standard_normal(nv)
        Mx = o.surface_mass_apply(surf, x)[rows]
        Vp, Kp = g.export_bem_rows(surf, rows)
        eV = np.abs(Vp - sV * V).max() / np.abs(V).max()
        dK = np.abs(Kp @ x - (0.5 * Mx + sK * (K @ x))).max() / (np.abs(Kp) @ np.abs(x)).max()
        print(f"  n {n} precision {precision} surface {surf}: V {eV:.2e} K {dK:.2e}", flush=True)
        bar = 1e-12 if precision == 0 else 1e-6
        assert eV < bar and dK < bar
    g.close()


def test_server_without_room_for_assembly_planes(ctx):
    """A budget one byte short of the footprint: admitted, assembled without
    the planes, the same energy to rounding."""
    import paper_2511_21713_amd as pb
    prob = pbgen.make_problem(n=3, a=6.0, c=9.0, bump=True, t=3.0, L=1, helix=0, partials=0, kappa=0.2, seed=(9, 3),
                              center_charge=1.0)
    g = pb.Problem.from_inputs(ctx, prob)
    ref = g.solve(**TIGHT)["total"]
    g.close()
    g = pb.Problem.from_inputs(ctx, prob)
    srv = pb.Server(ctx, hbm_budget_bytes=sum(g.footprint(**TIGHT)) - 1, max_slots=1)
    t = srv.submit(g, **TIGHT)
    end = time.time() + 60
    r = srv.poll(t)
    while r is None and time.time() < end:
        time.sleep(0.005)
        r = srv.poll(t)
    srv.close()
    assert r is not None and r["status"] == 0
    assert abs(r["total"] - ref) < 1e-10 * abs(ref)
    g.close()


# 47 and 1 819 vertices: the last wavefront of the full rows holds one row;
# 3 453: past the full rows' 160 MiB, the symmetric use's last row
@pytest.mark.parametrize("nlon,nlat,precision", [(9, 6, 0), (9, 6, 1), (23, 80, 0), (23, 80, 1), (29, 120, 0)])
def test_dense_rows_of_an_odd_vertex_count(ctx, nlon, nlat, precision):
    """As test_dense_rows_of_either_form_match_the_stored_blocks, for the
    residual (FP64 FEM values) and the Newton-matrix product."""
    import paper_2511_21713_amd as pb
    from test_gpu_tiles import valence_problem
    prob = valence_problem(nlon, nlat=nlat)
    g = pb.Problem.from_inputs(ctx, prob, precision=precision)
    g.set_tile_shape(16, 16)
    assert g.n_m % 2 == 1
    rng = np.random.default_rng(nlon)
    v, phi = rng.standard_normal(g.n), rng.standard_normal(g.n)
    y = g.apply_jacobian(pb.LIN, phi, v)
    r = g.residual(pb.LIN, v) + g.export_rhs()
    nn, nm = g.n_nodes, g.n_m
    for surf, ids, lo in ((0, np.unique(prob.tri_m), nn), (1, np.unique(prob.tri_s), nn + nm)):
        V, K = g.export_bem(surf)
        ref = K @ v[ids] + V @ v[lo:lo + ids.size]
        for got in (y, r):
            e = rel2(got[lo:lo + ids.size], ref)
            print(f"  {ids.size} vertices precision {precision} surface {surf}: {e:.2e}", flush=True)
            assert e < 1e-13
    g.close()


@pytest.mark.parametrize("precision,bar", [(0, 1e-10), (1, 1e-5)])
def test_solve_on_an_odd_vertex_count(ctx, precision, bar):
    """The Krylov step's full rows on 47 vertices: a solve against the oracle's energy."""
    import paper_2511_21713_amd as pb
    from test_gpu_tiles import valence_problem
    prob = valence_problem(9, nlat=6)
    ref = oracle.Oracle.from_problem(prob).solve(**TIGHT)[0]["total"]
    g = pb.Problem.from_inputs(ctx, prob, precision=precision)
    r = g.solve(**(TIGHT if precision == 0 else {}))
    print(f"  precision {precision}: {abs(r['total'] - ref) / abs(ref):.2e}", flush=True)
    assert abs(r["total"] - ref) < bar * abs(ref)
    g.close()


@pytest.mark.parametrize("n,precision", [(14, 0), (16, 1)])
def test_full_rows_hold_nothing_of_the_symmetric_use(ctx, n, precision):
    """A surface applied by full rows holds neither the column partials nor
    the two-ring differences of the symmetric use: after a product, square
    tiles hold no more than rectangular ones do beyond their block tables."""
    import paper_2511_21713_amd as pb
    prob = pbgen.make_problem(n=n, a=6.0, c=9.0, bump=True, t=3.0, L=1, helix=0, partials=0, kappa=0.2, seed=(9, n),
                              center_charge=1.0)
    held = {}
    for shape in ((16, 16), (8, 16)):  # the second's tables hold the first's
        g = pb.Problem.from_inputs(ctx, prob, precision=precision)
        g.set_tile_shape(*shape)
        g.apply_jacobian(pb.LIN, np.zeros(g.n), np.ones(g.n))
        held[shape] = g.hbm()
        g.close()
    nv = np.unique(prob.tri_m).size
    print(f"  n {n} precision {precision}: {held}, partials {8 * (nv * (-(-nv // 64)) + nv)}", flush=True)
    assert held[(16, 16)] <= held[(8, 16)]
