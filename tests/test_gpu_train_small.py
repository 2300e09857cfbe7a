"""Training steps of small batches (at most 256 rows) on the GPU, at the sizes
where their tiles end: batches around 16, 32, 64 and 256 rows, widths that are
no multiple of a tile, of a slab of k or of a 16-byte load, and buffers that
are not 16-byte aligned.

* loss and gradient of a batch against the FP64 reference with the products'
  operands rounded to bfloat16 as the GPU rounds them;
* a step of kkm_mlp_train_fresh and of kkm_mlp_train against the same step made
  of kkm_gram, kkm_mlp_loss_grad and kkm_mlp_adam, bit for bit: the update and
  the kernel values are fused into other launches, the arithmetic is the same.
"""
import numpy as np
import pytest

import oracle
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu

# (B, d, h1, h2, out)
SIZES = [(1, 3, 5, 7, 2), (15, 33, 40, 36, 17), (16, 64, 32, 64, 32), (33, 77, 100, 65, 50),
         (64, 128, 512, 512, 256), (100, 516, 96, 640, 258), (255, 40, 64, 48, 300), (256, 100, 130, 520, 256),
         (257, 24, 64, 64, 33)]


@pytest.fixture(scope="module")
def kkm():
    import paper_2501_05587_amd as kkm
    kkm.lib()
    return kkm


def _case(B, d, h1, h2, out, steps=1):
    r = np.random.default_rng(B * 7 + d)
    th = []
    for rows, cols in ((h1, d), (h2, h1), (out, h2)):
        th += [r.uniform(-1, 1, rows * cols) / np.sqrt(cols), r.normal(0, 0.02, rows)]
    return np.concatenate(th).astype(np.float32), r.normal(0, 1, (B * steps, d)).astype(np.float32)


def _dev(a, offset=0):
    """On the GPU, `offset` floats past a 16-byte boundary."""
    import torch
    buf = torch.zeros(a.size + offset, dtype=torch.float32, device="cuda")
    buf[offset:] = torch.from_numpy(a.ravel()).cuda()
    return buf[offset:].view(a.shape)


@pytest.mark.parametrize("B,d,h1,h2,out", SIZES)
def test_loss_grad_edges(kkm, B, d, h1, h2, out):
    th, X = _case(B, d, h1, h2, out)
    K = oracle.kernel_matrix(X, oracle.GAUSS, 1.0 / d)
    print("loss_grad", B, d, h1, h2, out, flush=True)
    g, loss = kkm.kkm_mlp_loss_grad(_dev(th), _dev(X), _dev(K.astype(np.float32)), h1=h1, h2=h2, out=out)
    L, gr = omlp.loss_and_grad(th.astype(np.float64), X, K, d, h1, h2, out, bf16_operands=True)
    g = g.cpu().numpy().astype(np.float64)
    # An activation or error term next to a rounding midpoint may take the other
    # bfloat16 neighbour after FP32 accumulation: 2^-8 of one operand.  About one
    # in 2^13 does (FP32 error over bfloat16 spacing), so a block's norm moves by
    # 2^-8 sqrt(2^-13) = 4e-5 of itself where it has many terms, and by at most a
    # few spacings where it has few.
    tol = 1e-3 if B >= 15 else 2.0 ** -6
    at = 0
    for rows, cols in ((h1, d), (h2, h1), (out, h2)):
        for size in (rows * cols, rows):
            a, b = g[at:at + size], gr[at:at + size]
            assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b) + 1e-7, (rows, cols, size)
            at += size
    assert abs(float(loss[0]) - L) <= tol * L


@pytest.mark.parametrize("kernel,coef0,degree", [(0, 0.0, 1), (1, 1.0, 3), (2, 0.0, 1)])
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("B,d,h1,h2,out", SIZES)
def test_step_is_its_parts(kkm, B, d, h1, h2, out, offset, kernel, coef0, degree):
    import torch
    kernel = (kkm.GAUSS, kkm.POLY, kkm.LINEAR)[kernel]
    gamma = 1.0 / d if kernel == kkm.GAUSS else 0.01
    steps = 2
    th, X = _case(B, d, h1, h2, out, steps)
    net = dict(h1=h1, h2=h2, out=out)
    print("train step", B, d, h1, h2, out, offset, kernel, flush=True)
    Xd = _dev(X, offset)

    def fresh():
        return [_dev(th, offset), _dev(np.zeros_like(th), offset), _dev(np.zeros_like(th), offset)]

    want, losses = fresh(), []
    for s in range(steps):
        XB = Xd[s * B:(s + 1) * B]
        K, _ = kkm.kkm_gram(XB, kernel=kernel, gamma=gamma, coef0=coef0, degree=degree)[:2]
        KB = K[:B, :B].contiguous()
        g, loss = kkm.kkm_mlp_loss_grad(want[0], XB, KB, **net)
        losses.append(float(loss[0]))
        kkm.kkm_mlp_adam(*want, g, s + 1)

    got = fresh()
    tr = kkm.kkm_mlp_train_fresh(*got, Xd, B, kernel=kernel, gamma=gamma, coef0=coef0, degree=degree, **net)
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    np.testing.assert_array_equal(tr.cpu().numpy(), np.array(losses))

    got = fresh()
    Kall, _ = kkm.kkm_gram(Xd, kernel=kernel, gamma=gamma, coef0=coef0, degree=degree)[:2]
    idx = torch.arange(steps * B, dtype=torch.int32, device="cuda").view(steps, B)
    kkm.kkm_mlp_train(*got, Xd, Kall, idx, **net)
    for a, b in zip(got, want):
        assert torch.equal(a, b)
