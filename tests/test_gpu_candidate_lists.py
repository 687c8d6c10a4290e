"""A tet's candidates, and with them the bits of its pieces, depend on the tet and the sites alone: not on the sites that
its block's box is near (which decide how the list is reduced), nor on the clip budget as long as the list fits it. An
incremental round has to take back exactly the bits that an earlier round added with other sites around."""
import numpy as np
import pytest

from paper_2403_18761_amd import synth
from tests.gpu_util import ELEMENT_ARRAYS, extract, log

pytestmark = pytest.mark.gpu
UNIT = 2.0 ** -20


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _near_duplicates(seed, n_pairs, N=4):
    """A small cube in a corner of the domain, and pairs of spheres far from it that meet there: of a pair, the first
    loses to the second everywhere in the cube, by less than the FP32 rounding of either's power distance."""
    base = synth.cube_random(N=N, n_sites=1, seed=1)
    v = [(np.asarray(a, np.float64) + 1.0) / 64 - 1.0 for a in (base.vx, base.vy, base.vz)]
    lo, hi = v[0].min(), v[0].max()
    corners = np.array([[x, y, z] for x in (lo, hi) for y in (lo, hi) for z in (lo, hi)])
    rng = np.random.default_rng(seed)
    step = np.array([[x, y, z, r] for x in range(-2, 3) for y in range(-2, 3) for z in range(-2, 3)
                     for r in range(-3, 4)]) * UNIT
    pairs = []
    for _ in range(2000 * n_pairs):
        c = synth.quantize(rng.uniform(-0.2, 1.0, 3))
        p = lo + (hi - lo) * rng.uniform(0.4, 0.6, 3)
        if not 5.6 < ((c - p) ** 2).sum() < 9.0:
            continue
        r = synth.quantize(np.sqrt(((c - p) ** 2).sum() - 5.5))
        a = np.append(c, r)
        power = lambda s: ((corners - s[..., None, :3]) ** 2).sum(-1) - s[..., None, 3] ** 2
        worse = power(a + step) - power(a)  # FP64: exact on the grid
        ok = (worse.min(1) > 0) & (worse.max(1) < 1.5e-7) & (np.abs(step[:, :3]).sum(1) > 0)
        ok &= (np.abs((a + step)[:, :3]) <= 1).all(1)
        if ok.any():
            pairs.append((a + step[np.flatnonzero(ok)[0]], a))
        if len(pairs) == n_pairs:
            break
    s = np.array([q for pair in pairs for q in pair]).astype(np.float32)
    base.vx, base.vy, base.vz = (a.astype(np.float32) for a in v)
    return base.with_sites(*s.T)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("seed", [1, 2, 3, 4, 5, 6])
def test_same_bits_with_any_budget(seed, precision):
    import torch

    from paper_2403_18761_amd import rpd

    dev = lambda a, dt=torch.float32: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda:0")
    p = _near_duplicates(seed, 10)
    mesh = rpd.Mesh(dev(p.vx), dev(p.vy), dev(p.vz), dev(p.tv.reshape(-1), torch.int32))
    log(f"case: near duplicates {seed}, precision {precision}, {p.n_tets} tets")
    got = []
    for budget in (28, 16, 12):  # 20 sites: within the first budget in every block
        res = rpd.build([mesh], [tuple(dev(a) for a in (p.sx, p.sy, p.sz, p.sr))], precision=precision,
                        clip_budget=budget, flags=rpd.RPD_KEEP_PIECES)
        log(budget, res.stats())
        if res.stats()["n_deferred"] == 0:
            got.append((budget, extract(res, 0), res.pieces(0), res.stats()["n_candidates"]))
    assert len(got) > 1
    for budget, el, pc, n in got[1:]:
        assert n == got[0][3], f"budget {budget}: candidates"
        for k in ELEMENT_ARRAYS:
            np.testing.assert_array_equal(got[0][1][k], el[k], err_msg=f"budget {budget}: {k}")
        for x, y in zip(got[0][2], pc):
            np.testing.assert_array_equal(x, y, err_msg=f"budget {budget}: pieces")
