"""The culled paths of rpd_envelope_distance and rpd_shrink_spheres: forced on inputs that they would leave to brute force,
equal to it (the same inputs in parts below the rule's sizes; both paths evaluate an element or a triangle with the same
expressions), and not taken by themselves where they cannot leave out enough."""
import time

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


def _dev(a, dt=None):
    import torch

    return torch.as_tensor(np.ascontiguousarray(a), dtype=dt or torch.float32, device="cuda:0")


def _best(f):
    import torch

    best = np.inf
    for _ in range(8):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best * 1e6


def _long_elements(ns, g):
    """Cones and slabs as long as the model."""
    S = np.concatenate([g.uniform(-1, 1, (ns, 3)), g.uniform(0.01, 0.1, (ns, 1))], axis=1).astype(np.float32)
    k = np.arange(ns)
    return S, np.stack([k, (k + 1) % ns], 1).astype(np.int32), np.stack([k, (k + 1) % ns, (k + 5) % ns], 1).astype(np.int32)


@pytest.mark.parametrize("case", ["surface", "volume", "one_point", "line", "far_and_infinite", "most_not_finite"])
def test_forced_culling_of_elements(case):
    import torch

    from paper_2403_18761_amd import rpd

    g = np.random.default_rng(7)
    n = 50_000 + 33
    S, E, F = _long_elements(1400, g)  # 4,200 elements: just past the rule's sizes, the last run ragged
    F[::50, 2] = F[::50, 1]  # degenerate slabs
    q = synth.surface_samples(synth.torus_core(16, 64, 1), n, seed=3)
    if case == "volume":
        q = g.uniform(-1, 1, (n, 3)).astype(np.float32)
    elif case == "one_point":
        q[:] = q[0]
    elif case == "line":
        q[:, :2] = q[0, :2]
    elif case == "far_and_infinite":
        q[5] = 1e6
        q[6, 1] = np.inf
        q[7, 2] = np.nan
    elif case == "most_not_finite":
        q[np.arange(n) % 3 > 0] = np.nan
    log(f"case: forced culling, {case}")
    s, e, f, x = _dev(S), _dev(E, torch.int32), _dev(F, torch.int32), _dev(q)
    parts = [rpd.envelope_distance(s, e, f, x[k:k + 9000].contiguous()) for k in range(0, n, 9000)]
    want, who = (np.concatenate([p[c].cpu().numpy() for p in parts]) for c in (0, 1))
    dist, near = torch.empty(n, device="cuda:0"), torch.empty(n, dtype=torch.int32, device="cuda:0")
    rpd.envelope_distance_noalloc(s, e, f, x, dist, near)
    host = rpd.envelope_distance(S, E, F, q, flags=rpd.RPD_FORCE_CULLING)
    for d, w in (rpd.envelope_distance(s, e, f, x, flags=rpd.RPD_FORCE_CULLING), rpd.envelope_distance(s, e, f, x),
                 (dist, near), tuple(_dev(a, torch.float32 if k == 0 else torch.int32) for k, a in enumerate(host))):
        np.testing.assert_array_equal(d.cpu().numpy(), want)
        np.testing.assert_array_equal(w.cpu().numpy(), who)


@pytest.mark.parametrize("n,spread", [(100_000, 1.0), (200_000, 0.25)])
def test_elements_that_cannot_be_culled(n, spread):
    """Long elements, or all of them close together, and samples in the volume: 2 to 3 times the time of brute force."""
    import torch

    from paper_2403_18761_amd import rpd

    g = np.random.default_rng(1)
    S, E, F = _long_elements(800 if spread == 1 else 3000, g)
    S[:, :3] *= spread
    a = (_dev(S), _dev(E, torch.int32), _dev(F, torch.int32), _dev(g.uniform(-1, 1, (n, 3))))
    forced = _best(lambda: rpd.envelope_distance(*a, flags=rpd.RPD_FORCE_CULLING))
    chosen = _best(lambda: rpd.envelope_distance(*a))
    log(f"case: {n} samples, spread {spread}: forced {forced:.0f} us, chosen {chosen:.0f} us")
    assert 1.5 * chosen < forced


def _soup(g, nt, n):
    m = g.normal(size=(n, 3))
    return g.uniform(-1, 1, (nt, 3, 3)), g.uniform(-1, 1, (n, 3)), m / np.linalg.norm(m, axis=1, keepdims=True), None


def _strips(g, m, n):
    """A cylinder of m strips as long as itself, two triangles each, and pins on them."""
    th = np.linspace(0, 2 * np.pi, m + 1)
    p = np.stack([np.cos(th), np.sin(th), -2 + 0 * th], axis=1) * 0.5
    up = np.array([0, 0, 2.0])
    tri = np.concatenate([np.stack([p[:-1], p[1:], p[:-1] + up], 1), np.stack([p[1:], p[1:] + up, p[:-1] + up], 1)])
    own = g.integers(0, 2 * m, n)
    pin = (tri[own] * g.dirichlet([1, 1, 1], n)[:, :, None]).sum(axis=1)
    nrm = -pin * [1, 1, 0]
    return tri, pin, nrm / np.linalg.norm(nrm, axis=1, keepdims=True), own.astype(np.int32)


@pytest.mark.parametrize("shape", ["soup", "strips"])
def test_triangles_that_cannot_be_culled(shape):
    """Triangles as large as the model: 5 to 10 times the time of brute force."""
    import torch

    from paper_2403_18761_amd import rpd

    g = np.random.default_rng(2)
    tri, pin, nrm, own = _soup(g, 20_000, 4000) if shape == "soup" else _strips(g, 10_000, 5000)
    t, p, m = _dev(tri), _dev(pin), _dev(nrm)
    o = None if own is None else _dev(own, torch.int32)
    forced = _best(lambda: rpd.shrink_spheres(t, p, m, o, flags=rpd.RPD_FORCE_CULLING))
    chosen = _best(lambda: rpd.shrink_spheres(t, p, m, o))
    log(f"case: {shape}: forced {forced:.0f} us, chosen {chosen:.0f} us")
    assert 2 * chosen < forced
    if shape == "strips":  # (neighbouring strips are nearly coplanar: their terms are rounding, whatever the path)
        return
    a = rpd.shrink_spheres(t, p, m, o, flags=rpd.RPD_FORCE_CULLING).cpu().numpy()
    b = rpd.shrink_spheres(t, p, m, o).cpu().numpy()
    tol = 1e-5 + 1e-4 * np.abs(b[:, 3])
    fin = np.isfinite(b[:, 3])
    np.testing.assert_array_equal(np.isfinite(a[:, 3]), fin)
    assert np.all(np.abs(a[fin, 3] - b[fin, 3]) <= tol[fin])
