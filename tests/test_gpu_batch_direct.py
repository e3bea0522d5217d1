"""The grouped direct kernel of the uneven batch where it can go wrong: more
problems a launch than lanes look up at once (64), bonds off and on its tiles
and k blocks, halves of both layouts in one launch, all precisions, and the
split sum over the middle bond.  Gates of test_gpu_mps.py; single BF16 and two
BF16 terms by their products' rounding (2^-8 and 2^-16 a factor over the steps)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1905_01330_amd as tn
from paper_1905_01330_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def run(shapes, prec, gate, forced=-1):
    chains, refs = [], []
    for i, (n, chi) in enumerate(shapes):
        psi, _ = inputs.uneven_chain(i, n, chi, seed=77)
        psi = [s.astype(np.float32) for s in psi]
        refs.append(oracle.mps_inner([s.astype(np.float64) for s in psi], [s.astype(np.float64) for s in psi]))
        sites = [torch.tensor(s, device=DEV) for s in psi]
        chains.append((sites, sites))
    try:
        tn.tune_force_grouped_config(forced)
        got = tn.mps_inner_batched(chains, prec=prec)
        torch.cuda.synchronize()
    finally:
        tn.tune_force_grouped_config(-1)
    got = got.cpu().numpy()
    for i, (m, s) in enumerate(refs):
        rel = abs(got[i, 0] * np.exp(got[i, 1] - s) / m - 1)
        assert rel <= gate, (shapes[i], rel)


@pytest.mark.parametrize("prec", ["fp32", "split_bf16"])
def test_many_problems(prec):
    rng = np.random.default_rng(5)
    run([(int(rng.integers(2, 14)), int(rng.integers(1, 40))) for _ in range(150)], prec, 4e-5)


@pytest.mark.parametrize("forced", [-1, 1, 2])
@pytest.mark.parametrize("prec,gate", [("fp32", 4e-5), ("split_bf16", 4e-6), ("split_bf16_3p", 2e-3), ("bf16", 0.3)])
def test_bonds(prec, gate, forced):
    run([(18, chi) for chi in (31, 32, 33, 127, 128, 129, 160, 250)], prec, gate, forced)


def test_one_and_two_sites():
    run([(1, 1), (2, 2), (3, 2), (4, 4), (5, 3)], "fp32", 4e-5)
