"""The FP32 linears on split-BF16 products (launches of 256 blocks and more)
against the FP64 mode: every column split of a block (K = 32 to 128 and the
factorised first layer's contraction widths 64 S = 64 to 256 in both
directions), several species with partly filled tiles and quads, and launches
of few components that only large graphs send there. Which launches took them
is read from the library's launch counts."""
import numpy as np
import pytest
import torch

import synth
from synth.configs import model_params

pytestmark = pytest.mark.gpu

B = pytest.importorskip("paper_2510_23621_amd.binding")
from paper_2510_23621_amd.graph import MaceGraph  # noqa: E402
from gpu_common import STRESS, STRESS_GAINS, assert_parity, lib_blob, run_gpu  # noqa: E402


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _clusters(n, species):
    """n atoms in graphs of 5 (the last may be smaller), 0.7 to 3.5 A apart."""
    rng = np.random.default_rng(n)
    corners = np.array([[x, y, z] for x in (0, 1.5) for y in (0, 1.5) for z in (0, 1.5)])
    pos = np.vstack([corners[rng.choice(8, 5, replace=False)] + rng.uniform(-0.35, 0.35, (5, 3))
                     for _ in range((n + 4) // 5)])[:n].astype(np.float32).astype(np.float64)
    gid = (np.arange(n) // 5).astype(np.int32)
    return synth.System(pos, rng.integers(0, species, n).astype(np.int32), None, gid, int(gid[-1]) + 1)


def _linear_launches(params, sysm, blob, form, products):
    """(launches of the channel-mixing linears, those on split products) in one
    forces call."""
    snd, rcv, _ = B.mace_neighbor_list(sysm.positions, params["r_cut"], None, sysm.graph_of_atom, sysm.n_graphs)
    g = MaceGraph(B.make_desc(**params), blob, sysm.species, np.stack([snd, rcv]), None, None, sysm.graph_of_atom,
                  sysm.n_graphs, B.MACE_FP32)
    B.mace_layer0_form(g.handle, form)
    B.mace_fp32_products(g.handle, products)
    pos = torch.from_numpy(sysm.positions.astype(np.float32)).cuda()
    counts = []
    for name in ("linear_kernel", "linear_split_kernel"):
        B.mace_profile_select(g.handle, B.kernel_ids()[name])
        g.energy_forces(pos)
        counts.append(B.mace_profile_read(g.handle)[1])
    g.close()
    return counts


# n_split: of the ten launches of a forces call, those with 256 blocks or more:
# the 16 and more components of the first layer and of the mid arrays always
# (twice each way), the 1 to 9 of the hidden features in the largest graph
# (rh: the width of the last readout, after which the composed weights begin)
@pytest.mark.parametrize("K,hl,S,n,n_split,rh", [(32, 2, 1, 1025, 4, 16), (64, 1, 2, 1207, 4, 16),
                                                 (96, 1, 3, 1300, 4, 16), (128, 2, 4, 1100, 4, 16),
                                                 (128, 1, 5, 1331, 4, 16), (96, 2, 6, 1400, 4, 16),
                                                 (32, 1, 2, 4133, 8, 16), (64, 1, 3, 1100, 4, 5), (96, 2, 5, 1300, 4, 1)])
def test_split_linears_match_fp64(K, hl, S, n, n_split, rh):
    params = model_params(4, K=K, hidden_lmax=hl, n_species=S, readout_hidden=rh, **STRESS)
    sysm, blob = _clusters(n, S), lib_blob(params, 11, STRESS_GAINS)
    ref = run_gpu(params, sysm, blob, B.MACE_FP64)
    forms = (B.MACE_L0_FACTORED, B.MACE_L0_EDGE) if S <= 4 else (B.MACE_L0_EDGE,)
    for form in forms:
        err = []
        assert _linear_launches(params, sysm, blob, form, B.MACE_PRODUCTS_SPLIT_BF16) == [10, n_split]
        assert _linear_launches(params, sysm, blob, form, B.MACE_PRODUCTS_FP32) == [10, 0]
        for products in (B.MACE_PRODUCTS_SPLIT_BF16, B.MACE_PRODUCTS_FP32):
            gpu = run_gpu(params, sysm, blob, l0_form=form, radial=products)
            err.append(assert_parity(gpu, ref, B.MACE_FP32, f"K={K} hl={hl} S={S} n={n} rh={rh} form={form} products={products}"))
        # no less accurate than FP32 products: both are within a few roundoffs of
        # the exact result, and a dropped part (2^-16) would show as 100 times more
        assert err[0]["forces"] <= 2 * err[1]["forces"] + 1e-7
        assert err[0]["eps_l2"] <= 2 * err[1]["eps_l2"] + 1e-7


@pytest.mark.parametrize("power", [-90, -60, 0])
def test_split_linears_of_small_features_match_fp64(power):
    """Features of 2^power times their usual size (the embedding scaled): at
    2^-90, about 1e-27, the third parts are near 1e-32, in the normal range."""
    params = model_params(4, K=64, hidden_lmax=1, n_species=2, **STRESS)
    sysm, blob = _clusters(1207, 2), lib_blob(params, 11, STRESS_GAINS)
    assert B.mace_weight_layout(B.make_desc(**params))[0][0][:2] == ("embed", 2 * 64)
    blob[:2 * 64] *= np.float32(2.0 ** power)
    ref = run_gpu(params, sysm, blob, B.MACE_FP64)
    gpu = run_gpu(params, sysm, blob)
    assert_parity(gpu, ref, B.MACE_FP32, f"features times 2^{power}")
