"""The FP32 linears on split-BF16 products (launches of 256 blocks and more)
against the FP64 mode: every column split of a block (K = 32 to 128 and the
factorised first layer's contraction widths 64 S = 64 to 256 in both
directions), several species with partly filled tiles and quads, and launches
of few components that only large graphs send there."""
import numpy as np
import pytest
import torch

import synth
from synth.configs import model_params

pytestmark = pytest.mark.gpu

B = pytest.importorskip("paper_2510_23621_amd.binding")
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


@pytest.mark.parametrize("K,hl,S,n", [(32, 2, 1, 1025), (64, 1, 2, 1207), (96, 1, 3, 1300), (128, 2, 4, 1100),
                                      (128, 1, 5, 1331), (96, 2, 6, 1400), (32, 1, 2, 4133)])
def test_split_linears_match_fp64(K, hl, S, n):
    params = model_params(4, K=K, hidden_lmax=hl, n_species=S, **STRESS)
    sysm, blob = _clusters(n, S), lib_blob(params, 11, STRESS_GAINS)
    ref = run_gpu(params, sysm, blob, B.MACE_FP64)
    forms = (B.MACE_L0_FACTORED, B.MACE_L0_EDGE) if S <= 4 else (B.MACE_L0_EDGE,)
    for form in forms:
        err = []
        for products in (B.MACE_PRODUCTS_SPLIT_BF16, B.MACE_PRODUCTS_FP32):
            gpu = run_gpu(params, sysm, blob, l0_form=form, radial=products)
            err.append(assert_parity(gpu, ref, B.MACE_FP32, f"K={K} hl={hl} S={S} n={n} form={form} products={products}"))
        # no less accurate than FP32 products: both are within a few roundoffs of
        # the exact result, and a dropped part (2^-16) would show as 100 times more
        assert err[0]["forces"] <= 2 * err[1]["forces"] + 1e-7
        assert err[0]["eps_l2"] <= 2 * err[1]["eps_l2"] + 1e-7
