"""Device neighbour list against the host list, element for element, over the
forms its binning and pre-test have to get right: batches of cells of their own
(skewed, thin, small against the cutoff), more atoms than one block scans,
cutoffs below the pre-test's range, coordinates far from the origin, graphs and
cubes that share a slot, and outputs untouched where the capacity is short."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
B = pytest.importorskip("paper_2510_23621_amd.binding")


@pytest.fixture(autouse=True, scope="module")
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _cells_batch(rng):
    cells = [np.diag([9.0, 4.0, 30.0]), np.array([[7.0, 0, 0], [5.0, 3.0, 0], [-4.0, 2.0, 6.0]]),
             np.eye(3) * 2.5, np.array([[0, 12.0, 0], [0, 0, 11.0], [13.0, 0, 0]])]
    counts = [60, 40, 3, 150]
    pos = np.concatenate([rng.uniform(-2, 3, (n, 3)) @ c for n, c in zip(counts, cells)])
    return pos, np.stack(cells), np.repeat(np.arange(4), counts).astype(np.int32)


def _inputs(name):
    rng = np.random.default_rng(21)
    if name == "cells of their own":
        pos, cells, g = _cells_batch(rng)
        return pos, 4.5, cells, g
    if name == "many atoms":
        return rng.uniform(0, 230, (70001, 3)), 5.0, None, None
    if name == "short cutoff":
        return rng.uniform(0, 6, (900, 3)), 0.6, np.eye(3)[None] * 6.0, None
    if name == "far away":
        return 3e8 + np.round(rng.uniform(0, 20, (400, 3)) * 64) / 64, 3.0, None, None
    if name == "many cells away":
        return rng.integers(-5, 6, (60, 3)) * 8.0 + rng.uniform(0, 8, (60, 3)), 5.0, np.eye(3)[None] * 8.0, None
    if name == "many small graphs":   # 1,566 cubes in 2,048 slots: many share one
        n = rng.integers(0, 5, 900)
        g = np.repeat(np.arange(900), n).astype(np.int32)
        return rng.uniform(0, 40, (len(g), 3)), 20.0, None, g
    if name == "cutoff beyond FP32":   # every pair, on both sides of the origin
        return rng.uniform(-30, 30, (50, 3)), 1e39, None, None
    if name == "on the cutoff":       # pairs at the cutoff exactly (left out) and one step inside
        x = np.arange(40) * 1.5
        return np.stack([x, np.zeros(40), np.zeros(40)], 1), 4.5, None, None
    raise AssertionError(name)


@pytest.mark.parametrize("name", ["cells of their own", "many atoms", "short cutoff", "far away", "many cells away",
                                  "many small graphs", "on the cutoff", "cutoff beyond FP32"])
def test_equals_host_list(name):
    pos, rc, cells, g = _inputs(name)
    G = 1 if g is None else int(g.max()) + 1
    off = None if g is None else np.searchsorted(g, np.arange(G + 1)).astype(np.int32)
    host = B.mace_neighbor_list(pos, rc, cells, g, G)
    dpos = torch.from_numpy(pos).cuda()
    for fn in (B.mace_neighbor_list_device, B.mace_neighbor_list_device_noalloc):
        if fn is B.mace_neighbor_list_device_noalloc and B.mace_neighbor_workspace_bytes(
                len(pos), rc, cells, off, G) > 80 << 20:
            continue
        dev = fn(dpos, rc, cells, off, G, max_edges=len(host[0]))
        torch.cuda.synchronize()
        print(f"[neighbors] {name}: {len(host[0])} edges", flush=True)
        assert len(host[0]) > 0
        for h, d in zip(host, dev):
            assert np.array_equal(h, d.cpu().numpy())


@pytest.mark.parametrize("n,graphs", [(0, 1000), (10, 500), (305, 305), (1024, 1024), (65536, 65536), (3000, 2000)])
def test_single_atoms_and_empty_graphs(n, graphs):
    """One atom or none in a graph, or (3000 in 2000) one and two."""
    rng = np.random.default_rng(n)
    g = np.sort(np.arange(n) % graphs).astype(np.int32)
    off = np.searchsorted(g, np.arange(graphs + 1)).astype(np.int32)
    pos = rng.uniform(0, 4, (n, 3))
    host = B.mace_neighbor_list(pos, 5.0, None, g, graphs)
    dpos = torch.from_numpy(pos).cuda()
    for fn in (B.mace_neighbor_list_device, B.mace_neighbor_list_device_noalloc):
        dev = fn(dpos, 5.0, None, off, graphs)
        torch.cuda.synchronize()
        print(f"[neighbors] {n} atoms in {graphs} graphs: {len(host[0])} edges", flush=True)
        assert (len(host[0]) > 0) == (n > graphs)
        for h, d in zip(host, dev):
            assert np.array_equal(h, d.cpu().numpy())


def test_short_capacity_leaves_outputs_alone():
    import ctypes
    pos, rc, cells, _ = _inputs("short cutoff")
    E = len(B.mace_neighbor_list(pos, rc, cells)[0])
    dpos = torch.from_numpy(pos).cuda()
    nbytes = B.mace_neighbor_workspace_bytes(len(pos), rc, cells)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    out = torch.full((5, E), -7, dtype=torch.int32, device="cuda")
    ne = ctypes.c_int64()
    cl = np.ascontiguousarray(cells)
    for cap, code in ((E - 1, -3), (E, 0)):
        got = B.lib().mace_neighbor_list_device(len(pos), dpos.data_ptr(), cl.ctypes.data, None, 1, rc, cap,
                                                out[0].data_ptr(), out[1].data_ptr(), out[2:].data_ptr(),
                                                ctypes.byref(ne), ws.data_ptr(), nbytes, None)
        torch.cuda.synchronize()
        assert got == code and ne.value == E
        assert bool((out == -7).all()) == (code != 0)
