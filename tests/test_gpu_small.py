"""Contractions with an operator (both small extents at most 16) at the edges of
the table kernel: K and N on and off its bounds, rows off the workgroup and past
one pass of the grid, strided operands and results, non-finite entries; and the
layout of such a step's result inside a network, feeding a contraction over the
streamed axis, over another one, or both.

Gates: the sums are formed in FP64 and stored in FP32, one rounding: 2^-23
relative to the sum of magnitudes; single BF16 rounds the factors first, the
reference rounds the same."""
import numpy as np
import pytest
import torch

import paper_1905_01330_amd as tn

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def rand(seed, *shape):
    g = torch.Generator(device="cpu").manual_seed(seed)
    return torch.randn(*shape, generator=g).to(DEV)


def check(a, b, ia, ib, out, prec="fp32"):
    tn.contract_between(a, b, ia, ib, out=out, prec=prec)
    torch.cuda.synchronize()
    x, y = (a.bfloat16(), b.bfloat16()) if prec == "bf16" else (a, b)
    ref = torch.tensordot(x.double(), y.double(), (ia, ib))
    mag = torch.tensordot(x.double().abs(), y.double().abs(), (ia, ib))
    assert ((out.double() - ref).abs() <= 2.0 ** -23 * mag + 1e-40).all()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("k", [1, 7, 8, 9, 16, 17])
@pytest.mark.parametrize("n", [1, 8, 9, 16])
def test_extents(k, n, prec):
    a, b = rand(k, k, 4099), rand(n, k, n)
    check(a, b, [0], [0], torch.empty(4099, n, device=DEV), prec)
    check(b, a, [0], [0], torch.empty(n, 4099, device=DEV), prec)


def test_axes_and_strides():
    a = rand(1, 3, 130, 2, 41).permute(1, 0, 3, 2)      # rows (130, 41), k (3, 2)
    w = rand(2, 5, 2, 3, 2).permute(1, 2, 3, 0)         # k at 1 and 0, columns (2, 5)
    out = torch.zeros(41, 5, 2, 130, 2, device=DEV)[..., 0].permute(3, 0, 2, 1)
    check(a, w, [1, 3], [1, 0], out)


def test_more_rows_than_one_pass():
    m = 65536 * 256 + 300
    a = torch.arange(2 * m, device=DEV, dtype=torch.int32).remainder_(1021).float().view(2, m)
    b = torch.tensor([[1.0, -2.0], [3.0, 0.5]], device=DEV)
    out = torch.empty(2, m, device=DEV)
    tn.contract_between(a, b, [0], [0], out=out.t())
    assert torch.equal(out[0], a[0] + 3 * a[1]) and torch.equal(out[1], -2 * a[0] + 0.5 * a[1])


def test_non_finite():
    a = rand(3, 6, 5000)
    a[0, 17], a[5, 40], a[2, 4999] = float("inf"), float("nan"), -float("inf")
    b = rand(4, 6, 6).abs() + 0.1
    out = torch.empty(5000, 6, device=DEV)
    tn.contract_between(a, b, [0], [0], out=out)
    ref = torch.tensordot(a, b, ([0], [0]))
    assert torch.equal(torch.isnan(out), torch.isnan(ref)) and torch.equal(torch.isinf(out), torch.isinf(ref))


@pytest.mark.parametrize("prec", ["fp32", "split_bf16"])
@pytest.mark.parametrize("case", ["streamed", "other", "both", "batchless chain"])
def test_layout_in_a_network(case, prec):
    """x [a, w, s, b] with an operator [w, v, t, s], then y over the axes named."""
    da, w, v, s, t, db = 67, 5, 3, 2, 2, 71
    x, op = rand(5, da, w, s, db), rand(6, w, v, t, s)
    first = rand(9, 33, da)      # makes x's part an intermediate
    nodes, labels = [first, x, op], [[-1, 1], [1, 2, 3, 4], [2, 5, 6, 3]]
    if case == "streamed":
        nodes.append(rand(7, 29, v, db))
        labels.append([-2, 5, 4])
        order, sub, opens = [1, 2, 3, 5, 4], "pa,awsb,wvts,qvb->pqt", [-3]
        labels[2][2] = -3
    elif case == "other":
        nodes.append(rand(7, t, v, 31))
        labels.append([6, 5, -2])
        labels[1][3] = -3
        order, sub = [1, 2, 3, 5, 6], "pa,awsb,wvts,tvq->pqb"
    elif case == "both":
        nodes.append(rand(7, db, t, 31))
        labels.append([4, 6, -2])
        labels[2][1] = -3
        order, sub = [1, 2, 3, 4, 6], "pa,awsb,wvts,btq->pqv"
    else:
        labels[1][3], labels[2][1], labels[2][2] = -2, -3, -4
        order, sub = [1, 2, 3], "pa,awsb,wvts->pbvt"
    got = tn.contract_network(nodes, labels, order=order, prec=prec)
    torch.cuda.synchronize()
    ref = torch.einsum(sub, *[z.double().cpu() for z in nodes])
    err = (got.double().cpu() - ref).norm() / ref.norm()
    assert err <= 1e-6, err
