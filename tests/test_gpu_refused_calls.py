"""Calls that the library refuses once its kernels have seen the input: the documented error, and the next call on the
same mesh (with the refused call's recycled buffers) as if nothing had happened."""
import numpy as np
import pytest

from paper_2403_18761_amd import synth
from tests.gpu_util import ELEMENT_ARRAYS, extract, log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _dev(a, dt=None):
    import torch

    return torch.as_tensor(np.ascontiguousarray(a), dtype=dt or torch.float32, device="cuda:0")


def _mesh(p):
    import torch

    from paper_2403_18761_amd import rpd

    return rpd.Mesh(_dev(p.vx), _dev(p.vy), _dev(p.vz), _dev(p.tv.reshape(-1), torch.int32))


def _candidates(p):
    """Per tet, the sites whose least value over it is at most the least over all sites of the largest value."""
    v = np.stack([p.vx, p.vy, p.vz], axis=1).astype(np.float64)
    c = np.stack([p.sx, p.sy, p.sz], axis=1).astype(np.float64)
    out = np.zeros(len(p.tv), np.int64)
    for t, tet in enumerate(p.tv):
        x = v[tet]
        d = ((x[:, None, :] - c[None]) ** 2).sum(axis=2) - ((x - x[0]) ** 2).sum(axis=1)[:, None]
        d -= p.sr.astype(np.float64)[None] ** 2
        out[t] = (d.min(axis=0) <= d.max(axis=0).min()).sum()
    return out


@pytest.mark.parametrize("N,n", [(4, 4000), (2, 1400)])
@pytest.mark.parametrize("precision", [0, 1])
def test_some_tets_over_the_candidate_limit(N, n, precision):
    """Tets over 1,020 candidates get no pieces, and glue to neighbours that do."""
    from paper_2403_18761_amd import rpd

    few = synth.cube_random(N=N, n_sites=40, seed=3)
    many = synth.cube_random(N=N, n_sites=n, seed=3)
    over = int((_candidates(many) > 1020).sum())
    assert 0 < over < many.n_tets
    log(f"case: {over} of {many.n_tets} tets over the candidate limit, precision {precision}")
    mesh = _mesh(few)
    sites = lambda p: tuple(_dev(a) for a in (p.sx, p.sy, p.sz, p.sr))
    before = extract(rpd.build([mesh], [sites(few)], precision=precision), 0)
    for _ in range(2):
        with pytest.raises(rpd.RPDError) as e:
            rpd.build([mesh], [sites(many)], precision=precision)
        assert e.value.code == -4
        after = extract(rpd.build([mesh], [sites(few)], precision=precision), 0)
        for k in ELEMENT_ARRAYS:
            np.testing.assert_array_equal(before[k], after[k], err_msg=k)


@pytest.mark.parametrize("bad", ["all_nan", "one_nan", "infinite", "off_grid"])
@pytest.mark.parametrize("n", [40, 600])
def test_invalid_sites(bad, n):
    """Sites the kernels must not search among: over 512 of them make groups of blocks share site lists."""
    from paper_2403_18761_amd import rpd

    p = synth.cube_random(N=4, n_sites=n, seed=4)
    log(f"case: invalid sites {bad}, {n}")
    mesh = _mesh(p)
    sites = [np.array(a) for a in (p.sx, p.sy, p.sz, p.sr)]
    before = extract(rpd.build([mesh], [tuple(_dev(a) for a in sites)]), 0)
    if bad == "all_nan":
        sites[0][:] = np.nan
    elif bad == "one_nan":
        sites[3][n // 2] = np.nan
    elif bad == "infinite":
        sites[1][0] = np.inf
    else:
        sites[2][-1] = 0.1
    for shapes in (1, 3):  # in a batch, beside valid shapes
        ok = tuple(_dev(a) for a in (p.sx, p.sy, p.sz, p.sr))
        with pytest.raises(rpd.RPDError) as e:
            rpd.build([mesh] * shapes, [ok] * (shapes - 1) + [tuple(_dev(a) for a in sites)])
        assert e.value.code == -1
        after = extract(rpd.build([mesh], [ok]), 0)
        for k in ELEMENT_ARRAYS:
            np.testing.assert_array_equal(before[k], after[k], err_msg=k)
