"""The room that a clipping pass gets (workspace.h, compiled for the host): what the first attempt of a build holds, against
the candidates and element records of dense sites counted with the oracle's pieces, and how it grows."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from paper_2403_18761_amd import synth

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("workspace") / "libworkspace.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC",
                           "-I" + os.path.join(ROOT, "paper_2403_18761_amd", "csrc"),
                           os.path.join(HERE, "workspace_host.cpp"), "-o", out])
    return C.CDLL(out)


def _room(lib, nt, ns, passes=1, slots12=0):
    out = (C.c_longlong * 4)()
    lib.host_pass_room(C.c_longlong(nt), C.c_longlong(ns), passes, slots12, out)
    return list(out)


def _grow(lib, room, asked):
    r = (C.c_longlong * 4)(*room)
    more = lib.host_grow(r, (C.c_longlong * 4)(*asked))
    return bool(more), list(r)


def _counts(p, tets):
    """Candidates that no other site beats at all four vertices, and element records (each from its smallest site), per
    tet of the sample."""
    import oracle

    v = np.stack([p.vx, p.vy, p.vz], axis=1).astype(np.float64)
    c = np.stack([p.sx, p.sy, p.sz], axis=1).astype(np.float64)
    r2 = p.sr.astype(np.float64) ** 2
    cand = 0
    for t in tets:
        y = v[p.tv[t]] - v[p.tv[t][0]]
        a = c - v[p.tv[t][0]]
        g = ((a * a).sum(axis=1) - r2)[:, None] - 2 * (a @ y.T)
        h = g[g.min(axis=1) <= g.max(axis=1).min()]
        cand += int((~(h[:, None, :] < h[None]).all(axis=2).any(axis=0)).sum())
    rec = 0
    for q in oracle.tet_pieces(p, tets)["pieces"]:
        i = q["i"]
        rec += sum(f[0] > i for f in q["face_terms"]) + sum(min(e[0], e[1]) > i for e in q["edge_terms"])
        rec += sum(min(w) > i for w in q["rpv"])
    return cand / len(tets), rec / len(tets)


@pytest.mark.parametrize("N,n,weights", [(8, 60, False), (8, 600, False), (8, 1660, False), (16, 500, False),
                                         (16, 4000, False), (16, 8000, False), (16, 8000, True), (16, 24000, False)])
def test_first_attempt_holds_dense_sites(lib, oracle_lib, N, n, weights):
    """Equal radii need most. A sample of 150 tets: its mean is within a few per cent of the mesh's."""
    p = synth.cube_random(N=N, n_sites=n, seed=3, weights=weights)
    tets = np.random.default_rng(1).choice(p.n_tets, 150, replace=False)
    cand, rec = _counts(p, tets)
    room = _room(lib, p.n_tets, n)
    print(f"{n / p.n_tets:.3f} sites per tet: {cand:.2f} candidates, {rec:.2f} records; room "
          f"{room[0] / p.n_tets:.2f}, {room[1] / p.n_tets:.2f}")
    assert room[0] >= 1.1 * cand * p.n_tets
    assert room[1] >= 1.1 * rec * p.n_tets
    two = _room(lib, p.n_tets, n, passes=2)
    assert two[0] >= 2 * room[0] - 64 and two[1] >= 2 * room[1] - 1


def test_growth(lib):
    room = _room(lib, 24576, 24)
    asked = [24 * 24576, 1000, 0, 0]
    more, g = _grow(lib, room, asked)
    assert more and g[0] >= asked[0] and g[0] < 2 * asked[0] and g[1] >= room[1] and g[2:] == room[2:]
    more, h = _grow(lib, g, [g[0], g[1], g[2], g[3]])  # nothing ran out
    assert not more and h == g
    for k in (1, 2, 3):
        asked = [10, 10, 10, 10]
        asked[k] = room[k] + 1
        more, g = _grow(lib, room, asked)
        assert more and g[k] >= asked[k] and all(g[q] == room[q] for q in range(4) if q != k)


@pytest.mark.parametrize("nt,ns", [(1, 1), (1, 2_000_000), (60_000_000, 2_000_000), (2_000_000_000, 2_000_000)])
def test_limits(lib, nt, ns):
    """Slots, two records a slot with the few of the last chunks, and the pool are numbered in 31 bits."""
    for passes in (1, 2):
        room = _room(lib, nt, ns, passes)
        for _ in range(4):
            assert room[0] % 64 == 0 and 0 < room[0] <= 800_000_000
            assert room[1] > 0 and 2 * room[0] + 768 + room[1] < 2 ** 31
            assert 0 < room[2] <= 2 ** 30 and 0 < room[3] <= 2 ** 20
            more, room = _grow(lib, room, [10 * r for r in room])
    assert not _grow(lib, room, [2 ** 40] * 4)[0] or _grow(lib, _grow(lib, room, [2 ** 40] * 4)[1], [2 ** 40] * 4)[0] is False
