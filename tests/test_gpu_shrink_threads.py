"""Sphere shrinking from several threads, each on a stream of its own: the workspaces come from one pool, and every
call's spheres are those of the same call alone, bit for bit."""
import threading

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


@pytest.mark.parametrize("device_arrays", [True, False])
@pytest.mark.parametrize("pins", [1000, 3001])  # brute force; sorted (15,384 triangles)
def test_threads_share_no_workspace(pins, device_arrays):
    import torch

    from paper_2403_18761_amd import rpd

    tri, n, cen, _, _ = synth.surface_pins(synth.torus_core(64, 64, 1))
    tri, n, cen = (np.array(a, np.float32) for a in (tri, n, cen))
    own = np.arange(len(tri), dtype=np.int32)
    dev = lambda a, dt=torch.float32: torch.as_tensor(a, dtype=dt, device="cuda:0") if device_arrays else a
    args = []
    for k in range(4):  # other pins for each thread, buffers of the same sizes
        at = np.random.default_rng(k).permutation(len(cen))[:pins]
        args.append((dev(tri), dev(cen[at]), dev(n[at]), dev(own[at], torch.int32)))
    host = lambda a: a.cpu().numpy() if device_arrays else a
    want = [host(rpd.shrink_spheres(*a)) for a in args]
    log(f"case: 4 threads, {pins} pins, device arrays {device_arrays}")
    streams = [torch.cuda.Stream() for _ in args]
    torch.cuda.synchronize()
    got = [[] for _ in args]

    def work(k):
        torch.cuda.set_device(0)
        with torch.cuda.stream(streams[k]):
            for _ in range(12):
                got[k].append(rpd.shrink_spheres(*args[k], stream=streams[k].cuda_stream))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(args))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for k in range(len(args)):
        assert len(got[k]) == 12
        for g in got[k]:
            np.testing.assert_array_equal(host(g), want[k])
