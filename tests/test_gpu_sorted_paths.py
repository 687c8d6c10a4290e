"""The sorted, culled path of rpd_envelope_distance against its brute-force path, which the same inputs take when they
come in small parts (each below the rule's sizes). Both paths evaluate an element with the same expressions and take a
minimum, so they differ at most by the contraction of those expressions: the bar is that of the comparison with the
FP64 oracle (1e-5 + 1e-5 |d|)."""
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
