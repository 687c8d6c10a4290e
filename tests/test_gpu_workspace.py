"""Calls whose pieces outgrow the workspace that a first attempt gets: the results of the repeated attempt against the
oracle (chi, beta0, adjacency exact; volumes within 1e-5 relative, the bar of the other FP32 builds)."""
import numpy as np
import pytest

from paper_2403_18761_amd import synth
from tests.gpu_util import assert_parity, log, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle

    oracle.build(force=False)


@pytest.mark.parametrize("copies", [2, 24])
def test_slots_run_out_in_one_class(copies):
    """Equal spheres tie everywhere: each copy is a candidate of every tet (2 or 24 of them, one class of tets), several
    times the slots that the few sites suggest with 24."""
    import oracle

    base = synth.cube_random(N=16, n_sites=1, seed=5)
    prob = base.with_sites(*(np.repeat(a, copies) for a in (base.sx, base.sy, base.sz, base.sr)))
    log(f"case: {prob.n_tets} tets, {copies} copies of a sphere")
    g = run_gpu(prob)
    assert g["stats"]["n_candidates"] == copies * prob.n_tets
    assert_parity(g, oracle.rpd(prob, assemble=False), label=f"{copies} copies")


@pytest.mark.parametrize("N,n", [(8, 600), (8, 1660)])
@pytest.mark.parametrize("precision", [0, 1])
def test_dense_sites_of_equal_radius(N, n, precision):
    """Most chunks of pieces have several times the records of their own range."""
    import oracle

    prob = synth.cube_random(N=N, n_sites=n, seed=3, weights=False)
    log(f"case: {prob.n_tets} tets, {n} sites, precision {precision}")
    g = run_gpu(prob, precision=precision)
    assert_parity(g, oracle.rpd(prob, assemble=False), vol_rtol=1e-9 if precision else 1e-5, label=f"N{N} n{n}")
