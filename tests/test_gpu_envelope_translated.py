"""The sorted, culled distance path on a model far from the origin, where a bounding sphere's centre is rounded by as much
as its element is long: no element that holds a minimum may be passed over. Reference: the brute-force path, which the
same samples take in small parts and which evaluates an element with the same expressions."""
import numpy as np
import pytest

from tests.gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("offset", [0.0, 64.0, 4096.0, 1e6])
@pytest.mark.parametrize("seed", [1, 2])
def test_translated_model(offset, seed):
    import torch

    from paper_2403_18761_amd import rpd

    g = np.random.default_rng(seed)
    dev = lambda a, dt=torch.float32: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda:0")
    ulp = float(np.spacing(np.float32(max(offset, 1.0))))
    size = max(1.0, 2000 * ulp)  # of the model
    ns, n = 1400, 50_000 + 7
    a = g.uniform(0, size, (ns // 2, 3)) + offset
    b = a + g.integers(1, 4, (ns // 2, 3)) * ulp * np.where(g.random((ns // 2, 3)) < 0.5, -1, 1)  # a few ulps away
    r = size * g.uniform(0.01, 0.05, ns // 2)
    S = np.concatenate([np.concatenate([a, r[:, None]], 1), np.concatenate([b, r[:, None]], 1)]).astype(np.float32)
    k = np.arange(ns // 2)
    E = np.concatenate([np.stack([k, k + ns // 2], 1), np.stack([k, (k + 1) % (ns // 2)], 1)]).astype(np.int32)
    F = np.stack([k, k + ns // 2, (k + 1) % (ns // 2)], 1).astype(np.int32)
    F = np.concatenate([F] * 4)  # 4,200 elements and more: past the rule
    # samples beside the short cones, 256 and more at a place: neighbours with no extent of their own
    d = np.cross(b - a, g.normal(size=a.shape))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    q = ((a + b) / 2 + d * (r * g.uniform(1.0, 3.0, len(r)))[:, None])[g.integers(0, 190, n)].astype(np.float32)
    log(f"case: translated by {offset}, {ns + len(E) + len(F)} elements")
    s, e, f, x = dev(S), dev(E, torch.int32), dev(F, torch.int32), dev(q)
    assert n * (ns + len(E) + len(F)) >= 200_000_000
    d, near = (t.cpu().numpy() for t in rpd.envelope_distance(s, e, f, x, flags=rpd.RPD_FORCE_CULLING))
    parts = [rpd.envelope_distance(s, e, f, x[p:p + 9000].contiguous()) for p in range(0, n, 9000)]
    want = np.concatenate([p[0].cpu().numpy() for p in parts])
    tie = np.concatenate([p[1].cpu().numpy() for p in parts])
    log("further off:", int((d > want).sum()), "by at most", float((d - want).max()), "nearer:", int((d < want).sum()),
        "other elements:", int((near != tie).sum()))
    np.testing.assert_array_equal(d, want)
    np.testing.assert_array_equal(near, tie)
