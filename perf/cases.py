"""Performance cases of the library: what a user's program asks of it.

A molecular-dynamics or screening program builds a neighbour list, binds a
graph and a model once (`MaceGraph`), and then calls for energies, forces or
stress once per step with that handle.  The cases are those per-step calls
(energy only, energy + forces, energy + forces + stress; FP32, the 16-bit
linear arms and the BF16 radial layer) and the device neighbour list, over

* periodic water at 1 g/cm^3 from 96 to 36,864 atoms (cutoff 5 or 6 A), and
  batches of 1 to 512 molecules of 20 to 60 atoms with up to ten species;
* K = 32 to 128 channels, hidden features up to l = 0, 1 or 2, two or three
  interaction layers.

The FP64 debug precision is not among them: it exists to check the others.

`exact` is the same model in plain torch FP64, written from the model's
equations with dense couplings and a two-pass chunked backward.
"""
from __future__ import annotations

import itertools
import math
from functools import lru_cache

import numpy as np
import torch

from paper_2510_23621_amd import binding as B
from paper_2510_23621_amd.graph import MaceGraph

PREC = {"fp32": B.MACE_FP32, "bf16": B.MACE_BF16_LINEAR, "fp16": B.MACE_FP16_LINEAR, "bf16radial": B.MACE_BF16_RADIAL}
WEIGHT_SEED = 10   # of the first dozen the one whose atom energies cancel least in the totals
MEAN_DEGREE = {5.0: 52.5, 6.0: 90.7}   # mean neighbour count of water at the cutoff: the model's c_norm


def _model(kind, n, K, lmax, prec="fp32", call="forces", r_cut=5.0, layers=2, species=2):
    return {"kind": kind, "n": n, "K": K, "lmax": lmax, "prec": prec, "call": call, "r_cut": r_cut,
            "layers": layers, "species": species}


def _list(kind, n, r_cut):
    return {"kind": kind, "n": n, "call": "neighbours", "r_cut": r_cut}


def listed():
    return [
        # one molecule: interactive relaxation or a single-point request, all launches and latency
        dict(_model("molecules", 1, 128, 1, species=10), name="molecule1_k128_l1"),
        # a small, light model on a small box: the cheapest MD step
        dict(_model("water", 32, 32, 0), name="water96_k32_l0"),
        # the ordinary MD step of a medium box, and the same step with bfloat16 linears
        dict(_model("water", 512, 128, 1), name="water1536_k128_l1"),
        dict(_model("water", 512, 128, 1, "bf16"), name="water1536_k128_l1_bf16"),
        # constant-pressure MD: the stress every step
        dict(_model("water", 1536, 128, 1, call="stress"), name="water4608_k128_l1_stress"),
        # an odd-sized box, a width that is no power of two, l = 2, binary16 linears
        dict(_model("water", 1331, 96, 2, "fp16", r_cut=6.0), name="water3993_k96_l2_fp16"),
        # scoring a batch of independent molecules of ten species (training-set evaluation, screening)
        dict(_model("molecules", 512, 128, 1, species=10), name="molecules512_k128_l1"),
        # Monte Carlo or committee scoring of a large box: energies alone
        dict(_model("water", 4096, 128, 2, call="energy", r_cut=6.0), name="water12288_k128_l2_energy"),
        # the large MD step, in FP32 and in the fastest mode
        dict(_model("water", 12288, 128, 2, r_cut=6.0), name="water36864_k128_l2"),
        dict(_model("water", 12288, 128, 2, "bf16radial", r_cut=6.0), name="water36864_k128_l2_bf16radial"),
        # rebuilding the neighbour list between steps: a medium box, the large box
        dict(_list("water", 512, 5.0), name="neighbours_water1536"),
        dict(_list("water", 12288, 6.0), name="neighbours_water36864"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("water", "water", "water", "molecules"))
    r_cut = rng.choice((5.0, 6.0))
    if rng.random() < 0.15:
        return _list(kind, _log_int(rng, 32, 12288) if kind == "water" else _log_int(rng, 1, 512), r_cut)
    if kind == "molecules":
        return _model(kind, _log_int(rng, 1, 512), rng.choice((64, 96, 128, 128)), rng.choice((0, 1, 1, 2)),
                      rng.choice(("fp32", "fp32", "bf16")), rng.choice(("forces", "forces", "energy")), r_cut,
                      2, rng.choice((3, 4, 7, 10)))
    layers = rng.choice((2, 2, 2, 3))
    return _model(kind, _log_int(rng, 32, 12288 if layers == 2 else 4096), rng.choice((32, 64, 96, 128, 128, 128)),
                  rng.choice((0, 1, 1, 2, 2)), rng.choice(("fp32", "fp32", "fp32", "bf16", "fp16", "bf16radial")),
                  rng.choice(("forces", "forces", "forces", "energy", "stress")), r_cut, layers, 2)


# ----------------------------------------------------------------- inputs

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _rotations(rng, n):
    q = rng.standard_normal((n, 4))
    w, x, y, z = (q / np.linalg.norm(q, axis=1, keepdims=True)).T
    return np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                     2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                     2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)], -1).reshape(n, 3, 3)


def _water(n, rng):
    """O on a jittered cubic lattice at 1 g/cm^3, H at 0.96 A and 104.5 deg,
    orientations redrawn until atoms of different molecules are 1 A apart,
    thermal noise, wrapped into the box."""
    L = (n * 18.015 / 6.02214076e23 * 1e24) ** (1 / 3)
    m = math.ceil(n ** (1 / 3) - 1e-9)
    sites = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)
    oxy = (sites[rng.permutation(m ** 3)[:n]] + 0.5 + rng.uniform(-0.1, 0.1, (n, 3))) * (L / m)
    a = math.radians(104.5) / 2
    arms = 0.96 * np.array([[0, 0, 0], [math.sin(a), 0, math.cos(a)], [-math.sin(a), 0, math.cos(a)]])
    dev = _device()
    mols = torch.from_numpy(oxy[:, None] + arms @ _rotations(rng, n).transpose(0, 2, 1)).to(dev)
    todo = torch.arange(n, device=dev)
    for _ in range(60):
        bad = []
        for part in todo.split(512):   # closest approach to every other molecule, minimum image
            d = mols[part].reshape(-1, 1, 3) - mols.reshape(1, -1, 3)
            d -= L * torch.round(d / L)
            r2 = (d * d).sum(-1).reshape(len(part), 3, n, 3).amin((1, 3))
            r2.scatter_(1, part[:, None], 9.0)
            bad.append(part[r2.amin(1) < 1.0])
        todo = torch.cat(bad)   # a new close pair has a moved molecule in it: these are the ones to look at again
        if not len(todo):
            break
        move = todo[::2] if len(todo) > 8 else todo   # about one of each close pair
        i = move.cpu().numpy()
        mols[move] = torch.from_numpy(oxy[i][:, None] + arms @ _rotations(rng, len(i)).transpose(0, 2, 1)).to(dev)
    pos = np.mod(mols.reshape(-1, 3).cpu().numpy() + rng.normal(0.0, 0.05, (3 * n, 3)), L).astype(np.float32)
    species = np.tile(np.array([0, 1, 1], np.int32), n)
    return pos, species, np.diag([L, L, L])[None], np.array([0, 3 * n], np.int32)


def _molecule_sizes(n):
    return 20 + (np.arange(n) * 17) % 41


def _molecules(n, species, rng):
    """Clusters of 20 to 60 atoms, uniform in a sphere at 0.1 atoms/A^3, 0.9 A
    apart at least; molecule g stands 100 g A along x."""
    sizes = _molecule_sizes(n)
    rad = (3 * sizes / (4 * math.pi * 0.1)) ** (1 / 3)
    pos = np.full((n, 60, 3), 1e6)
    have = np.zeros(n, int)
    while (have < sizes).any():
        g = np.nonzero(have < sizes)[0]
        p = rng.uniform(-1, 1, (len(g), 3)) * rad[g, None]
        far = (np.square(pos[g] - p[:, None]).sum(-1).min(1) >= 0.81) & (np.square(p).sum(-1) <= rad[g] ** 2)
        pos[g[far], have[g[far]]] = p[far]
        have[g[far]] += 1
    out = np.concatenate([pos[g, :sizes[g]] + [100.0 * g, 0, 0] for g in range(n)]).astype(np.float32)
    return (out, rng.integers(0, species, len(out)).astype(np.int32), None,
            np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32))


def _system(case, seed):
    """positions [N, 3] float32, species, cells or None, first atom of each graph."""
    rng = np.random.default_rng([seed, 1])
    return _water(case["n"], rng) if case["kind"] == "water" else _molecules(case["n"], case.get("species", 10), rng)


def _list_system(case, seed):
    """One geometry per case, so that every list has the same length; the seed
    shuffles the order of the molecules (water) or of each molecule's atoms."""
    pos, _, cells, off = _system(case, 0)
    rng = np.random.default_rng([seed, 3])
    if case["kind"] == "water":
        order = (3 * rng.permutation(case["n"])[:, None] + np.arange(3)).ravel()
    else:
        order = np.lexsort((rng.random(len(pos)), np.repeat(np.arange(case["n"]), np.diff(off))))
    return pos[order], cells, off


def _atoms(case):
    return 3 * case["n"] if case["kind"] == "water" else int(_molecule_sizes(case["n"]).sum())


def _c_norm(case):
    return MEAN_DEGREE[case["r_cut"]] if case["kind"] == "water" else 22.0


def _in_ls(case, t):
    return [0] if t == 0 else list(range(case["lmax"] + 1))


def _out_ls(case, t):
    return [0] if t == case["layers"] - 1 else list(range(case["lmax"] + 1))


def _paths(case, t):
    return [(a, b, c) for a in _in_ls(case, t) for b in range(4) for c in range(4)
            if abs(a - b) <= c <= a + b and (a + b + c) % 2 == 0]


def _layout(case):
    """(name, shape, fan-in) of the weights, in the library's order."""
    S, K, T = case["species"], case["K"], case["layers"]
    lay = [("embed", (S, K), S)]
    for t in range(T):
        paths = _paths(case, t)
        lay += [(f"{t}.up.{l}", (K, K), K) for l in _in_ls(case, t)]
        lay += [(f"{t}.radial.{i}", s, s[0]) for i, s in enumerate([(8, 64), (64, 64), (64, 64), (64, len(paths) * K)])]
        lay += [(f"{t}.linear.{p}", (K, K), K * sum(q[2] == path[2] for q in paths)) for p, path in enumerate(paths)]
        lay += [(f"{t}.skip.{l}", (S, K, K), K) for l in (range(4) if t == 0 else _out_ls(case, t))]
        lay += [(f"{t}.symc.{L}.{nu}", (S, len(_trees(nu, L)), K), len(_trees(nu, L)))
                for L in _out_ls(case, t) for nu in (1, 2, 3)]
        lay += [(f"{t}.prod.{L}", (K, K), K) for L in _out_ls(case, t)]
        lay += [(f"{t}.readout", (K,), K)] if t < T - 1 else [(f"{t}.readout.0", (K, 16), K), (f"{t}.readout.1", (16,), 16)]
    return lay


def _weights(case):
    """One model per case: the seed changes the atoms it is evaluated on."""
    rng = np.random.default_rng(WEIGHT_SEED)
    return {n: (rng.standard_normal(s) / math.sqrt(f)).astype(np.float32) for n, s, f in _layout(case)}


def prepare(case, seed):
    dev = _device()
    if case["call"] == "neighbours":
        pos, cells, off = _list_system(case, seed)
        # a program keeps the capacity of its list's buffers with some room
        cap = int(1.15 * len(pos) * (MEAN_DEGREE[case["r_cut"]] if case["kind"] == "water" else 45)) + 64
        pos = torch.from_numpy(pos.astype(np.float64)).to(dev)
        return {"call": "neighbours", "pos": pos, "r_cut": case["r_cut"], "cells": cells, "off": off, "cap": cap}
    pos, species, cells, off = _system(case, seed)
    pos64 = torch.from_numpy(pos.astype(np.float64)).to(dev)
    snd, rcv, sh = B.mace_neighbor_list_device(pos64, case["r_cut"], cells, off, len(off) - 1)
    desc = B.make_desc(n_species=case["species"], K=case["K"], hidden_lmax=case["lmax"], r_cut=case["r_cut"],
                       c_norm=_c_norm(case), n_layers=case["layers"])
    blob = np.concatenate([w.ravel() for w in _weights(case).values()])
    graph = np.repeat(np.arange(len(off) - 1, dtype=np.int32), np.diff(off)) if len(off) > 2 else None
    g = MaceGraph(desc, blob, species, torch.stack([snd, rcv]), sh if cells is not None else None, cells, graph,
                  len(off) - 1, PREC[case["prec"]])
    return {"call": case["call"], "graph": g, "pos": torch.from_numpy(pos).to(dev)}


def run(state):
    if state["call"] == "neighbours":
        off = state["off"]
        return B.mace_neighbor_list_device(state["pos"], state["r_cut"], state["cells"], off, len(off) - 1, state["cap"])
    g = state["graph"]
    call = {"energy": g.energy, "forces": g.energy_forces, "stress": g.energy_forces_stress}[state["call"]]
    return call(state["pos"])


# ------------------------------------------------------- work and tolerance

def work(case):
    """Inputs read once, outputs written once; multiply-adds of the model's own
    formulas (first layer factorised over the species where that is less)."""
    N = _atoms(case)
    E = N * (MEAN_DEGREE[case["r_cut"]] - (3 if case["r_cut"] == 6.0 else 0) if case["kind"] == "water" else 22)
    if case["call"] == "neighbours":
        return {"bytes": 24 * N + 20 * E, "flops": 9 * E}
    K, S = case["K"], case["species"]
    fl = 0.0
    for t in range(case["layers"]):
        paths = _paths(case, t)
        mid = sum(2 * c + 1 for _, _, c in paths)
        nnz = sum(int((np.abs(_cg(*p)) > 0).sum()) for p in paths)
        fl += E * 2 * (8 * 64 + 2 * 64 * 64)
        per_edge = E * 2 * (64 * len(paths) * K + K * (nnz + mid))
        fl += min(per_edge, E * 2 * 64 * 16 + N * 2 * 16 * 64 * S * K) if t == 0 else per_edge
        fl += N * 2 * K * K * (mid + 16 * (t == 0) + sum((2 * l + 1) * (3 if t else 2) for l in _out_ls(case, t)))
        fl += N * K * 2 * sum(_tree_terms(L) for L in _out_ls(case, t))
    fl *= 1 if case["call"] == "energy" else 3
    n_w = sum(int(np.prod(s)) for _, s, _ in _layout(case))
    out = 4 * N + 8 * case["n"] + (0 if case["call"] == "energy" else 12 * N)
    return {"bytes": 4 * n_w + 16 * N + 20 * E + out, "flops": fl}


def tolerance(case):
    if case["call"] == "neighbours":
        return "exact"
    # against `exact`: FP32 up to 8e-7 of an output, the 16-bit modes 1e-3 to
    # 1e-2 (more only for the total energy, where atoms' energies cancel)
    return {"fp32": {"rel": 1e-5, "max": 1e-4}, "fp16": {"rel": 2e-3, "max": 0.02}}.get(case["prec"], {"rel": 1e-2, "max": 0.1})


# ------------------------------------- the model in FP64, plain torch

def _harmonics(u):
    """Real harmonics l <= 3 of unit vectors, component normalised, m = -l..l."""
    x, y, z = u.unbind(-1)
    one = torch.ones_like(x)
    s3, s5, s7 = math.sqrt(3), math.sqrt(5), math.sqrt(7)
    return torch.stack([
        one, s3 * y, s3 * z, s3 * x,
        s5 * s3 * x * y, s5 * s3 * y * z, s5 * (1.5 * z * z - 0.5), s5 * s3 * x * z, s5 * s3 / 2 * (x * x - y * y),
        s7 * math.sqrt(5 / 8) * y * (3 * x * x - y * y), s7 * math.sqrt(15) * x * y * z,
        s7 * math.sqrt(3 / 8) * y * (5 * z * z - 1), s7 * (2.5 * z ** 3 - 1.5 * z),
        s7 * math.sqrt(3 / 8) * x * (5 * z * z - 1), s7 * math.sqrt(15) / 2 * z * (x * x - y * y),
        s7 * math.sqrt(5 / 8) * x * (x * x - 3 * y * y)], -1)


def _wigner(l, R):
    """D with Y_l(R u) = D Y_l(u) on fixed points, for l up to 6 (l > 3 from products of lower ones)."""
    u = np.random.default_rng(5).standard_normal((400, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)

    def basis(v):
        Y = _harmonics(torch.from_numpy(v)).numpy()
        if l <= 3:
            return Y[:, l * l:(l + 1) ** 2]
        from_3 = (Y[:, 9:16, None] * Y[:, None, (l - 3) ** 2:(l - 2) ** 2]).reshape(len(v), -1)
        return from_3 @ _high(l)
    return np.linalg.lstsq(basis(u), basis(u @ R.T), rcond=None)[0].T


@lru_cache(maxsize=None)
def _high(l):
    """Coefficients [(7 (2l-5)), 2l+1] of harmonics of degree l > 3 as products of
    degree 3 and l - 3: the combinations of products orthogonal to lower degrees."""
    n_t, n_p = 16, 33   # exact quadrature on the sphere
    z, wz = np.polynomial.legendre.leggauss(n_t)
    phi = 2 * np.pi * np.arange(n_p) / n_p
    s = np.sqrt(1 - z * z)
    v = np.stack([np.outer(s, np.cos(phi)), np.outer(s, np.sin(phi)), np.outer(z, np.ones(n_p))], -1).reshape(-1, 3)
    w = np.repeat(wz, n_p) / (2 * n_p)
    Y = _harmonics(torch.from_numpy(v)).numpy()
    P = (Y[:, 9:16, None] * Y[:, None, (l - 3) ** 2:(l - 2) ** 2]).reshape(len(v), -1)
    low = [Y] + [(Y[:, 9:16, None] * Y[:, None, (k - 3) ** 2:(k - 2) ** 2]).reshape(len(v), -1) @ _high(k)
                 for k in range(4, l)]
    X = np.concatenate(low, 1).T @ (w[:, None] * P)
    null_low = np.linalg.svd(X)[2][np.linalg.matrix_rank(X, 1e-9):].T   # combinations without lower degrees
    ev, vec = np.linalg.eigh(null_low.T @ (P.T @ (w[:, None] * P)) @ null_low)
    assert (ev > 1e-9).sum() == 2 * l + 1
    return null_low @ (vec[:, -(2 * l + 1):] / np.sqrt(ev[-(2 * l + 1):]))


@lru_cache(maxsize=None)
def _cg(a, b, c):
    """The rotation-invariant tensor [2a+1, 2b+1, 2c+1], sum over (m1, m2) of
    squares 1 for each m3, first nonzero entry positive."""
    rng = np.random.default_rng(3)
    rows = []
    for R in _rotations(rng, 2):
        D = np.kron(np.kron(_wigner(a, R), _wigner(b, R)), _wigner(c, R))
        rows.append(D - np.eye(len(D)))
    t = np.linalg.svd(np.vstack(rows).T @ np.vstack(rows))[2][-1]
    t[np.abs(t) < 1e-10 * np.abs(t).max()] = 0
    t *= math.sqrt(2 * c + 1) / np.linalg.norm(t) * np.sign(t[np.nonzero(t)[0][0]])
    t = t.reshape(2 * a + 1, 2 * b + 1, 2 * c + 1)
    t[np.abs(t) < 1e-6] = 0   # couplings are far from zero or zero
    return t


@lru_cache(maxsize=None)
def _trees(nu, L):
    """Coupling trees of nu factors (l = 0..3, natural parity) into L that are
    linearly independent once symmetrised, with the scale to unit norm."""
    kept, ortho = [], []
    if nu == 1:
        cand = [(L,)]
    elif nu == 2:
        cand = [(a, b) for a in range(4) for b in range(a, 4) if abs(a - b) <= L <= a + b and (a + b + L) % 2 == 0]
    else:
        cand = [(a, b, c, k) for a in range(4) for b in range(a, 4) for c in range(b, 4) if (a + b + c + L) % 2 == 0
                for k in range(abs(a - b), a + b + 1) if abs(k - c) <= L <= k + c]
    for tree in cand:
        T = np.zeros((2 * L + 1,) + (16,) * nu)
        at = tuple(slice(l * l, (l + 1) ** 2) for l in tree[:nu])
        if nu == 1:
            T[(slice(None),) + at] = np.eye(2 * L + 1)
        elif nu == 2:
            T[(slice(None),) + at] = np.moveaxis(_cg(tree[0], tree[1], L), 2, 0)
        else:
            T[(slice(None),) + at] = np.einsum("abk,kcM->Mabc", _cg(tree[0], tree[1], tree[3]), _cg(tree[3], tree[2], L))
        perms = list(itertools.permutations(range(1, nu + 1)))
        T = sum(np.transpose(T, (0,) + p) for p in perms) / len(perms)
        v, norm = T.ravel().copy(), np.linalg.norm(T)
        for q in ortho:
            v -= (q @ v) * q
        if norm > 1e-9 and np.linalg.norm(v) > 1e-7 * norm:
            ortho.append(v / np.linalg.norm(v))
            kept.append((tree, 1 / norm))
    return kept


def _tree_terms(L):
    """Nonzero coupling entries over the trees into L."""
    n = 0
    for nu in (1, 2, 3):
        for tree, _ in _trees(nu, L):
            n += 2 * L + 1
            if nu == 2:
                n += int((np.abs(_cg(tree[0], tree[1], L)) > 0).sum())
            elif nu == 3:
                n += int((np.abs(_cg(tree[0], tree[1], tree[3])) > 0).sum() + (np.abs(_cg(tree[3], tree[2], L)) > 0).sum())
    return n


def _couple(x, y, C):
    """x [n, 2a+1, K], y [n, 2b+1, K] -> [n, 2c+1, K]."""
    n, K = x.shape[0], x.shape[2]
    xy = (x[:, :, None] * y[:, None]).reshape(n, -1, K)
    return torch.matmul(torch.from_numpy(C.reshape(-1, C.shape[2]).T.copy()).to(x), xy)


def _edges(case, pos, cells, off):
    """Every pair within the cutoff, every periodic image: (sender, receiver, shift vector)."""
    dev, rc2 = pos.device, case["r_cut"] ** 2
    got = []
    if cells is None:
        for a, b in zip(off[:-1].tolist(), off[1:].tolist()):
            d = pos[a:b][None] - pos[a:b][:, None]
            r2 = (d * d).sum(-1)
            i, j = torch.nonzero((r2 < rc2) & (r2 > 0), as_tuple=True)
            got.append((j + a, i + a, torch.zeros(len(i), 3, dtype=pos.dtype, device=dev)))
    else:
        L, N = float(cells[0, 0, 0]), len(pos)
        images = [torch.zeros(3)] if L > 2 * case["r_cut"] else [torch.tensor(s, dtype=torch.float64) for s in itertools.product((-1., 0., 1.), repeat=3)]
        for rows in torch.arange(N, device=dev).split(max(1, (1 << 25) // N)):
            d = pos[None] - pos[rows][:, None]
            for s in images:
                sh = (-L * torch.round(d / L) if len(images) == 1 else (L * s).to(d).expand_as(d))
                r2 = (d + sh).square().sum(-1)
                i, j = torch.nonzero((r2 < rc2) & (r2 > 0), as_tuple=True)
                got.append((j, rows[i], sh[i, j]))
    return [torch.cat(x) for x in zip(*got)]


def _edge_terms(case, W, t, up, vec, snd):
    """Messages of some edges, per path [e, 2c+1, K]."""
    r = vec.square().sum(-1).sqrt()
    Y = _harmonics(vec / r[:, None])
    x, p = r / case["r_cut"], 5
    env = 1 - (p + 1) * (p + 2) / 2 * x ** p + p * (p + 2) * x ** (p + 1) - p * (p + 1) / 2 * x ** (p + 2)
    n = torch.arange(1, 9, dtype=r.dtype, device=r.device)
    a = math.sqrt(2 / case["r_cut"]) * torch.sin(n * math.pi * x[:, None]) / r[:, None] * env[:, None]
    for i in range(3):
        a = torch.nn.functional.silu(a @ W[f"{t}.radial.{i}"])
    paths = _paths(case, t)
    R = (a @ W[f"{t}.radial.3"]).reshape(len(r), len(paths), case["K"])
    out = []
    for q, (lh, ly, lo) in enumerate(paths):
        C = torch.from_numpy(_cg(lh, ly, lo)).to(r)
        CY = torch.matmul(Y[:, ly * ly:(ly + 1) ** 2], C.permute(1, 2, 0).reshape(2 * ly + 1, -1))
        CY = CY.reshape(len(r), 2 * lo + 1, 2 * lh + 1)
        out.append(torch.bmm(CY, up[lh][snd]) * R[:, q, None])
    return out


def _node_terms(case, W, t, At, h, z):
    """Layer t after the neighbour sum: (next features per L, readout energy)."""
    paths = _paths(case, t)

    def by_species(x, Ws):
        return sum(torch.where((z == s)[:, None, None], x @ Ws[s], 0.0) for s in range(len(Ws)))
    A = [sum(At[q] @ W[f"{t}.linear.{q}"] for q, p in enumerate(paths) if p[2] == l) for l in range(4)]
    if t == 0:
        A = [by_species(A[l], W[f"0.skip.{l}"]) for l in range(4)]
    out, pair = {}, {}
    for L in _out_ls(case, t):
        acc = 0
        for nu in (1, 2, 3):
            for e, (tree, scale) in enumerate(_trees(nu, L)):
                if nu == 1:
                    term = A[L]
                elif nu == 2:
                    term = _couple(A[tree[0]], A[tree[1]], _cg(tree[0], tree[1], L))
                else:
                    key = (tree[0], tree[1], tree[3])
                    if key not in pair:
                        pair[key] = _couple(A[tree[0]], A[tree[1]], _cg(*key))
                    term = _couple(pair[key], A[tree[2]], _cg(tree[3], tree[2], L))
                acc = acc + scale * W[f"{t}.symc.{L}.{nu}"][z, e][:, None] * term
        out[L] = acc @ W[f"{t}.prod.{L}"]
        if t > 0:
            out[L] = out[L] + by_species(h[L], W[f"{t}.skip.{L}"])
    s = out[0][:, 0]
    if t < case["layers"] - 1:
        return out, s @ W[f"{t}.readout"]
    return out, torch.nn.functional.silu(s @ W[f"{t}.readout.0"]) @ W[f"{t}.readout.1"]


def exact(case, seed):
    if case["call"] == "neighbours":
        return None   # whole numbers
    dev = _device()
    p32, species, cells, off = _system(case, seed)
    pos = torch.from_numpy(p32.astype(np.float64)).to(dev)
    z = torch.from_numpy(species.astype(np.int64)).to(dev)
    W = {k: torch.from_numpy(w.astype(np.float64)).to(dev) for k, w in _weights(case).items()}
    snd, rcv, sh = _edges(case, pos, cells, off)
    vec = pos[snd] + sh - pos[rcv]
    N, E, K, T = len(pos), len(snd), case["K"], case["layers"]
    ec = torch.arange(E, device=dev).split(1 << 16)
    nc = torch.arange(N, device=dev).split(1 << 10)
    eps = torch.zeros(N, dtype=torch.float64, device=dev)
    hs, Ats = [{0: W["embed"][z][:, None]}], []
    with torch.no_grad():
        for t in range(T):
            up = {l: hs[t][l] @ W[f"{t}.up.{l}"] for l in _in_ls(case, t)}
            At = [torch.zeros(N, 2 * p[2] + 1, K, dtype=torch.float64, device=dev) for p in _paths(case, t)]
            for e in ec:
                for q, m in enumerate(_edge_terms(case, W, t, up, vec[e], snd[e])):
                    At[q].index_add_(0, rcv[e], m / _c_norm(case))
            new = [_node_terms(case, W, t, [a[i] for a in At], {l: v[i] for l, v in hs[t].items()}, z[i]) for i in nc]
            eps += torch.cat([x[1] for x in new])
            hs.append({l: torch.cat([x[0][l] for x in new]) for l in _out_ls(case, t)})
            Ats.append(At)
    graph = torch.from_numpy(np.repeat(np.arange(len(off) - 1), np.diff(off))).to(dev)
    Eg = torch.zeros(len(off) - 1, dtype=torch.float64, device=dev).index_add(0, graph, eps)
    # the total of one graph has a relative error of its own only where the
    # atoms' energies, of either sign with random weights, do not cancel in it
    Eg_out = Eg if len(Eg) > 1 or abs(float(Eg)) > 0.2 * float(eps.abs().sum()) else None
    if case["call"] == "energy":
        return eps, Eg_out
    g_vec = torch.zeros_like(vec)
    g_next = None
    for t in reversed(range(T)):
        gAt = [torch.zeros_like(a) for a in Ats[t]]
        gh = {l: torch.zeros_like(v) for l, v in hs[t].items()}
        for i in nc:
            a = [x[i].requires_grad_(True) for x in Ats[t]]
            h = {l: v[i].requires_grad_(True) for l, v in hs[t].items()}
            out, e_t = _node_terms(case, W, t, a, h, z[i])
            tot = e_t.sum()
            if g_next is not None:
                tot = tot + sum((out[l] * g_next[l][i]).sum() for l in out)
            got = torch.autograd.grad(tot, a + list(h.values()), allow_unused=True)
            for q in range(len(a)):
                if got[q] is not None:
                    gAt[q][i] = got[q]
            for l, v in zip(h, got[len(a):]):
                if v is not None:
                    gh[l][i] = v
        up = {l: (hs[t][l] @ W[f"{t}.up.{l}"]).requires_grad_(True) for l in _in_ls(case, t)}
        for e in ec:
            v = vec[e].requires_grad_(True)
            m = _edge_terms(case, W, t, up, v, snd[e])
            (sum((x * gAt[q][rcv[e]]).sum() for q, x in enumerate(m)) / _c_norm(case)).backward()
            g_vec[e] += v.grad
        g_next = {l: gh[l] + up[l].grad @ W[f"{t}.up.{l}"].T for l in up}
    F = torch.zeros_like(pos).index_add(0, rcv, g_vec).index_add(0, snd, -g_vec)
    if case["call"] == "forces":
        return eps, Eg_out, F
    vol = 1.0 if cells is None else abs(float(np.linalg.det(cells[0])))
    S = torch.zeros(len(off) - 1, 3, 3, dtype=torch.float64, device=dev)
    S.index_add_(0, graph[rcv], vec[:, :, None] * g_vec[:, None])
    return eps, Eg_out, F, S / vol
