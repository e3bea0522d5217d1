"""The direct contraction kernel (32 x 32 tiles, K cut over eight waves)
against the FP64 oracle where it can go wrong: tile remainders, every
remainder of the chunk of K, fewer chunks than waves, one more than a wave
keeps in flight, all pairs of layouts, several axes a group, permuted
outputs, and the problems it does not take.

Tolerances as in test_gpu_contract.py: the stated accuracy of each precision.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1905_01330_amd as tn

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
TOL = {"fp32": 1e-5, "split_bf16": 1e-6, "split_bf16_3p": 1e-4, "bf16": 2e-2}
TILE = 7   # the 32 x 32 configuration


def gpu(x):
    return torch.tensor(np.asarray(x, dtype=np.float32), device=DEV)


def check(got, a, b, pa, pb, tol, what):
    torch.cuda.synchronize()
    got = got.cpu().double().numpy()
    ref = oracle.tensordot(a, b, pa, pb)
    scale = oracle.tensordot(np.abs(a), np.abs(b), pa, pb)
    rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    assert rel <= tol, f"{what}: relative error {rel:.3e} > {tol:.1e}"
    assert (np.abs(got - ref) <= 4 * tol * scale + 1e-30).all(), what


def stored(x, inner):
    """x [rows, k] on the device with k unit-stride ("k"), the rows ("m"), or neither ("g")."""
    if inner == "k":
        return gpu(x)
    if inner == "m":
        return gpu(x.T.copy()).t()
    wide = gpu(np.zeros((x.shape[0], 2 * x.shape[1])))
    wide[:, ::2] = gpu(x)
    return wide[:, ::2]


@pytest.mark.parametrize("prec", list(TOL))
@pytest.mark.parametrize("layout", ["kk", "km", "mk", "mm", "gk", "mg", "gg"])
def test_edges_of_the_tile_and_of_k(prec, layout):
    rng = np.random.default_rng(91)
    ks = [2, 3, 7, 8, 9, 15, 16, 17, 31, 33, 64, 127, 130, 391, 513, 1030]
    shapes = [(32, 32), (2, 33), (31, 5), (65, 32), (33, 70)]
    for i, k in enumerate(ks):
        m, n = shapes[i % len(shapes)]
        a = rng.standard_normal((m, k)).astype(np.float32)
        b = rng.standard_normal((n, k)).astype(np.float32)
        got = tn.contract_between(stored(a, layout[0]), stored(b, layout[1]), [1], [1], prec=prec)
        if k > 1 and m * n > 256:
            assert tn.tune_last_choice() == TILE
        check(got, a, b, [1], [1], TOL[prec], f"{m}x{n}x{k}")


@pytest.mark.parametrize("prec", ["fp32", "split_bf16"])
@pytest.mark.parametrize("inner", [3, 4, 20])
def test_groups_of_several_axes(prec, inner):
    """Two contracted axes that do not merge (inner extents off and on the
    multiples of four), three free axes a side, the result written through
    permuted strides with either side contiguous; then three contracted
    axes, and four free ones, which the kernel does not take."""
    rng = np.random.default_rng(92)
    a = rng.standard_normal((5, 3, 6, 7, inner)).astype(np.float32)      # m m k m k
    b = rng.standard_normal((inner, 4, 6, 3, 5)).astype(np.float32)      # k n k n n
    out = torch.empty((5, 3, 7, 4, 3, 5), device=DEV)
    tn.contract_between(gpu(a), gpu(b), [2, 4], [2, 0], out=out, prec=prec)
    check(out, a, b, [2, 4], [2, 0], TOL[prec], "n contiguous")
    back = torch.empty(5 * 3 * 7 * 4 * 3 * 5, device=DEV)
    view = torch.as_strided(back, (5, 3, 7, 4, 3, 5), (1, 35, 5, 105 * 15, 105 * 5, 105))   # m axis 0 contiguous
    tn.contract_between(gpu(a), gpu(b), [2, 4], [2, 0], out=view, prec=prec)
    check(view, a, b, [2, 4], [2, 0], TOL[prec], "m contiguous")
    a = rng.standard_normal((9, 2, 5, 3, 4, inner)).astype(np.float32)
    b = rng.standard_normal((inner, 11, 2, 3, 4)).astype(np.float32)
    got = tn.contract_between(gpu(a), gpu(b), [1, 3, 5], [2, 3, 0], prec=prec)
    check(got, a, b, [1, 3, 5], [2, 3, 0], TOL[prec], "three contracted axes")
    a = rng.standard_normal((2, 3, 2, 5, 2, inner)).astype(np.float32)
    ga = gpu(a.transpose(3, 5, 0, 2, 4, 1).copy()).permute(2, 5, 3, 0, 4, 1)
    b = rng.standard_normal((40, inner)).astype(np.float32)
    check(tn.contract_between(ga, gpu(b), [5], [1], prec=prec), a, b, [5], [1], TOL[prec], "five free axes")


@pytest.mark.parametrize("prec", ["fp32", "split_bf16"])
@pytest.mark.parametrize("layout", ["kk", "km", "mk", "mm"])
@pytest.mark.parametrize("last,n,k", [(4, 36, 40), (4, 33, 37), (3, 5, 64), (8, 64, 33)])
def test_tiles_of_one_wave(last, n, k, layout, prec):
    """Four row axes that do not merge: the 32 x 32 tile then runs on one wave,
    with the gathers of the operands' layouts (k or the rows contiguous, whole
    and partial runs of four)."""
    rng = np.random.default_rng(last + n + k)
    a = rng.standard_normal((3, 2, 2, last, k)).astype(np.float32)
    b = rng.standard_normal((n, k)).astype(np.float32)
    if layout[0] == "k":     # memory (2, last, 3, 2, k)
        ga = gpu(a.transpose(1, 3, 0, 2, 4).copy()).permute(2, 0, 3, 1, 4)
    else:                    # memory (k, 2, 3, 2, last)
        ga = gpu(a.transpose(4, 2, 0, 1, 3).copy()).permute(2, 3, 1, 4, 0)
    gb = gpu(b) if layout[1] == "k" else gpu(b.T.copy()).t()
    tn.tune_force_config(TILE)
    try:
        got = tn.contract_between(ga, gb, [4], [1], prec=prec)
    finally:
        tn.tune_force_config(-1)
    check(got, a, b, [4], [1], TOL[prec], layout)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_infinities_stay_in_their_rows(bad):
    """A row past the end of a tile repeats the last one, and k past the end
    reads as zero: neither may carry an infinity or NaN elsewhere."""
    rng = np.random.default_rng(93)
    a = rng.standard_normal((34, 37)).astype(np.float32)
    b = rng.standard_normal((35, 37)).astype(np.float32)
    a[33, 36] = bad
    got = tn.contract_between(gpu(a), gpu(b), [1], [1]).cpu().double().numpy()
    with np.errstate(invalid="ignore"):
        ref = a.astype(np.float64) @ b.T.astype(np.float64)
    assert np.isfinite(got[:33]).all()
    assert np.array_equal(np.isnan(got[33]), np.isnan(ref[33]))
    assert np.array_equal(np.isposinf(got[33]), np.isposinf(ref[33]))
    assert np.allclose(got[:33], ref[:33], rtol=0, atol=1e-4)


@pytest.mark.parametrize("prec", ["fp32", "split_bf16"])
@pytest.mark.parametrize("bond", [1, 2, 3, 5, 7, 8])
def test_fused_operator_step(prec, bond):
    """Sweeps whose sites all run on the fused step (operator bonds with and
    without their own kernel, ragged outer extents, the ends' other bonds),
    both directions together and each alone."""
    rng = np.random.default_rng(94 + bond)
    dims = [1, 2, 4, 7, 13, 37, 33, 18, 9, 4, 2, 1]
    n = len(dims) - 1
    psi = [(rng.standard_normal((dims[k], 2, dims[k + 1])) / np.sqrt(dims[k] * 2)).astype(np.float32) for k in range(n)]
    w = [1] + [bond] * (n - 1) + [1]
    mpo = [(rng.standard_normal((w[k], w[k + 1], 2, 2)) / np.sqrt(2 * w[k])).astype(np.float32) for k in range(n)]
    gp, gm = [gpu(x) for x in psi], [gpu(x) for x in mpo]
    ls, rs, _, _ = oracle.env_sweep(psi, mpo)
    for left, right in [(True, True), (True, False), (False, True)]:
        got_l, got_r, _ = tn.mps_env_sweep(gp, gm, left=left, right=right, prec=prec)
        torch.cuda.synchronize()
        for got, ref in ([(got_l, ls)] if left else []) + ([(got_r, rs)] if right else []):
            for k in range(1, n):
                g = got[k].cpu().double().numpy()
                assert np.linalg.norm(g - ref[k]) <= TOL[prec] * np.linalg.norm(ref[k]), (left, right, k)


@pytest.mark.parametrize("prec", ["fp32", "split_bf16"])
@pytest.mark.parametrize("dims", [[1, 3, 33, 70, 21, 1], [1, 2, 4, 900, 4, 2, 1], [1, 5, 1100, 1150, 7, 1]])
def test_inner_product_in_shared_launches(prec, dims):
    """Steps small enough for both ends to share launches, chains of odd
    length (the last step has one end), bonds of psi and phi that differ, and
    steps too large for it in the middle of such a chain (the ends then run on
    their own streams and join again)."""
    rng = np.random.default_rng(len(dims) + dims[2])
    n = len(dims) - 1
    chains = []
    for q in (0, 1):
        dd = [1] + [x + q for x in dims[1:-1]] + [1]
        chains.append([(rng.standard_normal((dd[k], 3, dd[k + 1])) / np.sqrt(dd[k] * 3)).astype(np.float32)
                       for k in range(n)])
    psi, phi = chains
    m, s = tn.mps_inner([gpu(x) for x in psi], [gpu(x) for x in phi], prec=prec).cpu().numpy()
    ref = oracle.mps_inner(psi, phi)
    value = ref[0] * np.exp(ref[1])
    norms = [v[0] * np.exp(v[1]) for v in (oracle.mps_inner(psi, psi), oracle.mps_inner(phi, phi))]
    # relative to the Cauchy-Schwarz scale: the overlap of two random chains cancels
    assert abs(m * np.exp(s) - value) <= TOL[prec] * np.sqrt(norms[0] * norms[1])


def short_sums(side):
    """A chain whose site 1 contracts few terms that cancel (left: 11 with bond
    187 beside it, right: 2 beside 190), on one end of a long free extent."""
    rng = np.random.default_rng(12)
    if side == "left":
        a0 = np.zeros((1, 2, 11))
        a0[0, 0, 10] = 1
        a0[0, 1, :3] = 1   # L_1[a', a] = a0[0, a'] a0[1, a]
        a1 = rng.uniform(1, 2, (11, 2, 187))
        a1[0] = 2.0**24 * (2 * rng.integers(0, 4, (2, 187)) + 1)
        a1[2] = -a1[0]
        psi = [a0, a1, rng.standard_normal((187, 2, 1))]
        bonds = (1, 1)
    else:
        e = 2.0**-12
        k = rng.integers(1, 100, (190, 2))
        a1 = np.stack([1 + k * e, -(1 + (k + 1) * e)], axis=2)   # times (1 + e, 1): k e^2
        a2 = np.zeros((2, 2, 1))
        a2[0, 0] = 1
        a2[:, 1, 0] = 1 + e, 1
        psi = [rng.standard_normal((1, 2, 190)), a1, a2]
        bonds = (1, 8)
    psi = [x.astype(np.float32).astype(np.float64) for x in psi]
    up = np.array([[0.0, 1.0], [0.0, 0.0]])
    mpo = [np.zeros((1, bonds[0], 2, 2)), np.zeros((bonds[0], bonds[1], 2, 2)), np.zeros((bonds[1], 1, 2, 2))]
    mpo[0][0, 0], mpo[1][0, 0], mpo[2][0, 0] = (up, np.eye(2), np.eye(2)) if side == "left" else (np.eye(2), np.eye(2), up)
    return psi, mpo


@pytest.mark.parametrize("prec,gate", [("fp32", 2.0**-21), ("split_bf16_3p", 2.0**-14)])
@pytest.mark.parametrize("side", ["left", "right"])
def test_short_sums_of_a_sweep_are_exact(side, prec, gate):
    """A contraction of at most 32 terms with a free extent of at most 16 sums
    in FP64 from whole operands, in a sweep as anywhere else: what is left are
    the roundings of its result, the operator step and the second contraction
    (four of FP32; three terms of 2^-16 in two BF16 parts)."""
    psi, mpo = short_sums(side)
    left = side == "left"
    ls, rs, _, _ = oracle.env_sweep(psi, mpo)
    gl, gr, _ = tn.mps_env_sweep([torch.tensor(x, dtype=torch.float32, device=DEV) for x in psi],
                                 [torch.tensor(x, dtype=torch.float32, device=DEV) for x in mpo],
                                 left=left, right=not left, prec=prec)
    torch.cuda.synchronize()
    got, want = (gl[2], ls[2]) if left else (gr[1], rs[1])
    np.testing.assert_allclose(got.cpu().double().numpy(), want, rtol=gate)


@pytest.mark.parametrize("call", ["inner", "sweep"])
def test_last_choice_of_a_shared_launch(call):
    """Products that share a launch are seen by tune_last_choice as others are."""
    rng = np.random.default_rng(13)
    dims = [1, 40, 50, 60, 40, 1]
    psi = [gpu(rng.standard_normal((dims[k], 2, dims[k + 1])) / 10) for k in range(5)]
    mpo = [gpu(rng.standard_normal((1 if k == 0 else 3, 1 if k == 4 else 3, 2, 2))) for k in range(5)]
    big = gpu(rng.standard_normal((2048, 2048)))
    tn.contract_between(big, big, [1], [1])
    assert tn.tune_last_choice() != TILE
    if call == "inner":
        tn.mps_inner(psi, psi)
    else:
        tn.mps_env_sweep(psi, mpo, store=False)
    assert tn.tune_last_choice() == TILE
