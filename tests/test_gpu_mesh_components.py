"""Connected components and simplex counts of prepared meshes whose tets fill one, several or a part of the windows
that the component search unites separately. Whole numbers: exact."""
import numpy as np
import pytest

from paper_2403_18761_amd import synth
from tests.gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _mesh(occ, N):
    from paper_2403_18761_amd import rpd

    p = synth.make_problem({"occ": occ}, N, np.zeros((1, 3)), np.ones(1))
    return p, rpd.Mesh(p.vx, p.vy, p.vz, p.tv.reshape(-1))


@pytest.mark.parametrize("N,length", [(4, 1), (16, 3), (64, 57), (256, 256)])
def test_components_over_windows(N, length):
    """Bars of voxels (6 tets each: 6 to 1536, a part of a window to one and a half) and full cubes (384 and 24576 tets):
    one component; two bars apart: refused as two components."""
    from paper_2403_18761_amd import rpd

    bar = np.zeros((N, N, N), bool)
    bar[1, 1, :length] = True
    log(f"case: components N {N} length {length}")
    for occ in (bar, np.ones((N, N, N), bool) if N in (4, 16) else bar):
        p, m = _mesh(occ, N)
        tv = np.sort(p.tv.reshape(-1, 4).astype(np.int64), axis=1)
        info = m.info()
        edges = np.unique(np.concatenate([tv[:, [a, b]] for a in range(4) for b in range(a + 1, 4)]), axis=0)
        faces = np.unique(np.concatenate([np.delete(tv, k, axis=1) for k in range(4)]), axis=0)
        verts = np.unique(tv)
        assert info["n_edges"] == len(edges) and info["n_faces"] == len(faces)
        assert info["euler"] == len(verts) - len(edges) + len(faces) - len(tv)
        assert info["components"] == 1
    two = bar.copy()
    two[3, 3, :length] = True
    with pytest.raises(rpd.RPDError, match="more than one connected component"):
        _mesh(two, N)
