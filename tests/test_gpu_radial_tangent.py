"""Forces through the forward-differentiated radial layers (da3/dr in the edge
prologue, dR/dr beside R in the edge products) against the FP64 oracle: sizes
of the radial basis and orders of its envelope at both input paddings, and
receivers of 1 to 33 edges (edge tiles of one, a full one, one over), one pair
just inside the cutoff, in both forms of the first layer."""
import numpy as np
import pytest
import torch

import synth
from synth.configs import model_params

pytestmark = pytest.mark.gpu

B = pytest.importorskip("paper_2510_23621_amd.binding")
from gpu_common import STRESS, STRESS_GAINS, assert_parity, lib_blob, oracle_blob, run_gpu, run_oracle  # noqa: E402


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _blobs():
    """Graphs of 2, 2, 16, 17, 18 and 34 atoms, every pair of a graph within
    5 A: 1, 15, 16, 17 and 33 edges per receiver; the second pair at 4.999 A."""
    rng = np.random.default_rng(8)
    pos, gid = [], []
    for g, n in enumerate((2, 2, 16, 17, 18, 34)):
        if g == 1:
            pts = np.array([[0, 0, 0], [4.999, 0, 0]])
        else:
            pts = np.empty((0, 3))
            while len(pts) < n:
                p = rng.uniform(-2.4, 2.4, 3)
                if p @ p < 2.4 ** 2 and (not len(pts) or np.linalg.norm(pts - p, axis=1).min() > 0.7):
                    pts = np.vstack([pts, p])
        pos.append(pts + [50.0 * g, 0, 0])
        gid += [g] * n
    pos = np.vstack(pos).astype(np.float32).astype(np.float64)
    return synth.System(pos, rng.integers(0, 3, len(pos)).astype(np.int32), None, np.array(gid, np.int32), 6)


@pytest.mark.parametrize("K,hl,nb,p,form", [(32, 0, 8, 5, "EDGE"), (64, 1, 5, 1, "EDGE"), (32, 2, 16, 3, "EDGE"),
                                            (128, 1, 9, 6, "FACTORED"), (96, 2, 1, 2, "FACTORED")])
def test_forces_match_oracle(K, hl, nb, p, form):
    params = model_params(4, K=K, hidden_lmax=hl, n_species=3, n_bessel=nb, envelope_p=p, **STRESS)
    sysm = _blobs()
    ref = run_oracle(params, sysm, oracle_blob(params, 9, STRESS_GAINS))
    for radial in (B.MACE_PRODUCTS_SPLIT_BF16, B.MACE_PRODUCTS_FP32):
        gpu = run_gpu(params, sysm, lib_blob(params, 9, STRESS_GAINS), l0_form=getattr(B, "MACE_L0_" + form),
                      radial=radial)
        assert_parity(gpu, ref, B.MACE_FP32, f"tangent K={K} hl={hl} nb={nb} p={p} {form} radial={radial}")


@pytest.mark.parametrize("nb", [8, 9])
def test_many_edges_match_oracle(nb):
    """The prologue's whole tiles with every layer in one block (over 131,072
    edges): copies of the graphs above, in place, against the oracle's one."""
    params = model_params(4, K=32, hidden_lmax=0, n_species=3, n_bessel=nb, **STRESS)
    one = _blobs()
    ref = run_oracle(params, one, oracle_blob(params, 9, STRESS_GAINS))
    M, n, G = 70, len(one.positions), one.n_graphs
    gid = (one.graph_of_atom[None] + G * np.arange(M, dtype=np.int32)[:, None]).ravel().astype(np.int32)
    sysm = synth.System(np.tile(one.positions, (M, 1)), np.tile(one.species, M), None, gid, M * G)
    blob = lib_blob(params, 9, STRESS_GAINS)
    gpu, energy = run_gpu(params, sysm, blob), run_gpu(params, sysm, blob, forces=False)
    assert gpu["n_edges"] > 131072
    for q in range(M):
        part = dict(eps=gpu["eps"][n * q:n * (q + 1)], energy=gpu["energy"][G * q:G * (q + 1)],
                    forces=gpu["forces"][n * q:n * (q + 1)])
        if q in (0, M // 2, M - 1):
            assert_parity(part, ref, B.MACE_FP32, f"copy {q} nb={nb}")
        assert np.allclose(energy["eps"][n * q:n * (q + 1)], part["eps"], rtol=1e-5, atol=1e-5 * np.abs(ref["eps"]).mean())
        assert np.linalg.norm(part["forces"] - ref["forces"]) <= 1e-5 * np.linalg.norm(ref["forces"])


@pytest.mark.parametrize("K,layers,form", [(128, 3, "EDGE"), (128, 8, "FACTORED"), (64, 5, "EDGE")])
def test_gradient_rows_of_many_layers_match_fp64(K, layers, form):
    """A layer's gradient rows take the hidden radial outputs of the layer above
    (both of them at K = 128), which the next call writes again: several calls.
    (Plain weights and a c_norm of the mean degree: each layer is cubic in its
    input, and eight of them with the gains of the other tests leave FP32.)"""
    params = model_params(4, K=K, hidden_lmax=1, n_layers=layers, n_species=3, c_norm=20.0)
    sysm, blob = _blobs(), lib_blob(params, 9)
    ref = run_gpu(params, sysm, blob, B.MACE_FP64)
    for radial in (B.MACE_PRODUCTS_SPLIT_BF16, B.MACE_PRODUCTS_FP32):
        outs = run_gpu(params, sysm, blob, l0_form=getattr(B, "MACE_L0_" + form), radial=radial, repeats=3)
        assert_parity(outs[0], ref, B.MACE_FP32, f"rows K={K} layers={layers} {form} radial={radial}")
        for o in outs[1:]:
            assert np.array_equal(o["forces"], outs[0]["forces"])
