"""The sorted, culled paths of rpd_envelope_distance and rpd_shrink_spheres against their brute-force paths, which the
same inputs take when they come in small parts (each below the rule's sizes). Both paths evaluate an element or a
triangle with the same expressions and take a minimum, so they differ at most by the contraction of those expressions:
the bars are those of the comparisons with the FP64 oracle (1e-5 + 1e-5 |d|; 1e-5 + 1e-4 r)."""
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


def _same(got, want, tol):
    np.testing.assert_array_equal(np.isfinite(got), np.isfinite(want))
    fin = np.isfinite(want)
    assert np.all(np.abs(got[fin] - want[fin]) <= tol[fin]), float(np.abs(got[fin] - want[fin]).max())


@pytest.mark.parametrize("case", ["surface", "one_point", "line", "far_and_infinite"])
def test_envelope_sorted_matches_brute_force(case):
    import torch

    from paper_2403_18761_amd import rpd

    g = np.random.default_rng(7)
    ns, n = 1400, 50_000 + 33  # 4,200 elements: just past the rule, the last run ragged
    S = np.concatenate([g.uniform(-1, 1, (ns, 3)), g.uniform(0.01, 0.1, (ns, 1))], axis=1).astype(np.float32)
    E = np.stack([np.arange(ns), (np.arange(ns) + 1) % ns], axis=1).astype(np.int32)
    F = np.stack([np.arange(ns), (np.arange(ns) + 1) % ns, (np.arange(ns) + 5) % ns], axis=1).astype(np.int32)
    F[::50, 2] = F[::50, 1]  # degenerate slabs
    q = synth.surface_samples(synth.torus_core(16, 64, 1), n, seed=3)
    if case == "one_point":
        q[:] = q[0]
    elif case == "line":
        q[:, :2] = q[0, :2]
    elif case == "far_and_infinite":
        q[5] = 1e6
        q[6, 1] = np.inf
        q[7, 2] = np.nan
    log(f"case: sorted envelope {case}")
    s, e, f, x = _dev(S), _dev(E, torch.int32), _dev(F, torch.int32), _dev(q)
    d, near = (a.cpu().numpy() for a in rpd.envelope_distance(s, e, f, x))
    parts = [rpd.envelope_distance(s, e, f, x[k:k + 9000].contiguous()) for k in range(0, n, 9000)]
    want = np.concatenate([p[0].cpu().numpy() for p in parts])
    tie = np.concatenate([p[1].cpu().numpy() for p in parts])
    _same(d, want, 1e-5 + 1e-5 * np.abs(want))
    np.testing.assert_array_equal(near[d == want], tie[d == want])


@pytest.mark.parametrize("case", ["own", "no_own", "long", "short", "mixed", "not_finite", "degenerate"])
def test_shrink_sorted_matches_brute_force(case):
    import torch

    from paper_2403_18761_amd import rpd

    tri, n, cen, _, _ = synth.surface_pins(synth.torus_core(64, 64, 1))
    tri, n, cen = (np.array(a, np.float32) for a in (tri, n, cen))
    own = np.arange(len(tri), dtype=np.int32)
    keep = np.arange(0, len(cen), 4)[:3001]  # ragged runs
    n, cen, own = n[keep], cen[keep], own[keep]
    if case in ("long", "short"):
        n *= np.float32(1.7 if case == "long" else 0.6)
    elif case == "mixed":
        n[::2] *= np.float32(0.3)
        n[::3] *= np.float32(5)
    elif case == "not_finite":
        tri[7, 0, 0], tri[11, 1, 2], tri[len(tri) // 2, 2, 1], tri[13] = np.inf, -np.inf, np.nan, 1e25
    elif case == "degenerate":
        tri[::5, 1] = tri[::5, 0]
        tri[::7] = tri[0]
    assert len(cen) >= 2048 and len(cen) * len(tri) >= 40_000_000
    log(f"case: sorted shrinking {case}")
    t, p, m = _dev(tri), _dev(cen), _dev(n)
    o = None if case == "no_own" else _dev(own, torch.int32)
    part = lambda a, k: None if a is None else a[k:k + 1000].contiguous()
    got = rpd.shrink_spheres(t, p, m, o).cpu().numpy()
    want = np.concatenate([rpd.shrink_spheres(t, part(p, k), part(m, k), part(o, k)).cpu().numpy()
                           for k in range(0, len(cen), 1000)])
    tol = 1e-5 + 1e-4 * np.abs(want[:, 3])
    _same(got[:, 3], want[:, 3], tol)
    for c in range(3):  # centre = pin + r normal
        _same(got[:, c], want[:, c], tol * np.maximum(1, np.abs(n).max()))
