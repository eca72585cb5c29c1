"""Kernels and dispatch branches at the sizes where they can go wrong: block
remainders, the smallest surfaces and the first sizes past a branch, each
against the oracle or the path the oracle already pins."""
import numpy as np
import pytest

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
