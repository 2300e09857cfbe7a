"""The FP32 kernel matrix where its product is taken as six bfloat16 products
of three-part values: against 64 bits, in every shape and layout, and against
the FP32 kernel for the values that are left to it.

A workspace that holds only the row norms selects the FP32 kernel, which the
split must accept as before.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (n, d): the smallest sizes that take the split, one feature, a slab less and
# more than one, tiles that end inside a group of 16 rows
SIZES = [(2304, 65), (2311, 784), (3584, 1), (3600, 31), (3585, 33), (4100, 128)]


@pytest.fixture(scope="module")
def kkm():
    import paper_2501_05587_amd as kkm
    kkm.lib()
    return kkm


def _points(n, d, pad=0, offset=0):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n * 1000 + d)
    buf = torch.randn(n * (d + pad) + offset, generator=g, device="cuda")
    return buf[offset:].view(n, d + pad)[:, :d]


def _small_ws(n):
    import torch
    return torch.empty((4 * n + 255) // 256 * 256, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("pad,offset", [(0, 0), (3, 1)])
@pytest.mark.parametrize("n,d", SIZES)
def test_against_64_bits(kkm, n, d, pad, offset):
    X = _points(n, d, pad, offset)
    print("split", n, d, pad, offset, flush=True)
    assert kkm.gram_workspace_bytes(n, d, kkm.F32) > _small_ws(n).numel()
    K, diag = kkm.kkm_gram(X, kernel=kkm.LINEAR)
    Xd = X.double()
    # a slab of 32 features: 12 matrix instructions, each addition within 2^-23
    # (rounded either way); the slabs' sums within 2^-24 each; what the parts
    # leave out within 2^-24 of every product
    bound = (12 * 2.0 ** -23 + (-(-d // 32) + 1) * 2.0 ** -24) * (Xd.abs() @ Xd.abs().T)
    assert bool(((K.double() - Xd @ Xd.T).abs() <= bound).all())
    assert bool((K == K.T).all())
    assert bool((diag == K.diagonal()).all())


@pytest.mark.parametrize("kernel", ["GAUSS", "POLY", "LINEAR"])
@pytest.mark.parametrize("store", ["F32", "BF16"])
@pytest.mark.parametrize("n,d", SIZES)
def test_shapes_and_layouts_agree(kkm, n, d, store, kernel):
    import torch
    X = _points(n, d)
    a = dict(kernel=getattr(kkm, kernel), gamma=1.0 / d, coef0=1.0, degree=2, k_store=getattr(kkm, store))
    print("split shapes", n, d, store, kernel, flush=True)
    K, diag = kkm.kkm_gram(X, **a)
    F, fdiag = kkm.kkm_gram(X, shape=kkm.GRAM_FULL, **a)
    assert torch.equal(K, F) and torch.equal(diag, fdiag)
    P, pdiag = kkm.kkm_gram_packed(X, **a)
    assert torch.equal(diag, pdiag)
    at, ns, W = 0, -(-n // 1024), 1024
    for s in range(ns):
        rows, wide = min(W, n - s * W), (ns - s) * W
        B = P[at:at + rows * wide].view(rows, wide)[:, :n - s * W]
        assert torch.equal(B, K[s * W:s * W + rows, s * W:])
        at += rows * wide


@pytest.mark.parametrize("kernel", ["GAUSS", "POLY", "LINEAR"])
@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 2.0 ** 61, -3e38, "tiny row"])
def test_values_outside_the_split(kkm, value, full, kernel):
    import torch
    n, d = 2311, 70
    X = _points(n, d).clone()
    if value == "tiny row":
        X[n - 1] *= 2.0 ** -60
    else:
        X[n - 1, d - 1] = value
    a = dict(kernel=getattr(kkm, kernel), gamma=1.0 / d, coef0=1.0, degree=2,
             shape=kkm.GRAM_FULL if full else kkm.GRAM_TRIANGLE)
    print("split values", value, full, kernel, flush=True)
    K, diag = kkm.kkm_gram(X, **a)
    R, rdiag = kkm.kkm_gram(X, ws=_small_ws(n), **a)
    assert torch.equal(K.view(torch.int32) if K.is_contiguous() else K.contiguous().view(torch.int32),
                       R.contiguous().view(torch.int32))
    assert torch.equal(diag.view(torch.int32), rdiag.view(torch.int32))
    # and a row of zeros is within the range
    Z = _points(n, d).clone()
    Z[5] = 0
    K, _ = kkm.kkm_gram(Z, kernel=kkm.LINEAR)
    assert bool((K[5] == 0).all()) and bool((K[:, 5] == 0).all())


def test_batched_takes_a_workspace_without_it(kkm):
    """A batch's workspace of the size it had without the split is accepted; the
    problem below the split's sizes is the same bit for bit."""
    import torch
    X = [_points(2311, 96), _points(500, 20)]
    probs = [dict(X=x, k=5, kernel=kkm.GAUSS, gamma=1.0 / x.shape[1]) for x in X]
    g = np.random.default_rng(3)
    l0 = torch.from_numpy(g.integers(0, 5, 2811).astype(np.int32)).cuda()
    need = kkm.kkm_fit_batched_workspace_bytes(probs, kkm.F32, kkm.F32)
    groups = -(-2311 // 128) * 8
    # room for the split matrix and the flags, each begun on a multiple of 256
    small = need - groups * 3 * 3072 - 256
    r = kkm.kkm_fit_batched(probs, l0, kkm.F32, kkm.F32, max_iter=10)
    s = kkm.kkm_fit_batched(probs, l0, kkm.F32, kkm.F32, max_iter=10,
                            ws=torch.empty(small, dtype=torch.uint8, device="cuda"))
    assert torch.equal(r["labels"][2311:], s["labels"][2311:])
    assert r["objective"][1] == s["objective"][1]
    assert abs(r["objective"][0] - s["objective"][0]) <= 1e-5 * abs(s["objective"][0])


def _sparse(n, d, kind):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    X = torch.randn(n, d, generator=g, device="cuda")
    if kind == "one feature":
        Y = torch.zeros_like(X)
        Y[:, d // 2] = X[:, d // 2]
        return Y
    if kind == "three features":
        Y = torch.zeros_like(X)
        Y[:, ::d // 3] = X[:, ::d // 3]
        return Y
    if kind == "a fifth":
        return X * (torch.rand(n, d, generator=g, device="cuda") < 0.2)
    if kind == "a fifth, positive":
        return X.abs() * (torch.rand(n, d, generator=g, device="cuda") < 0.2)
    return X


@pytest.mark.parametrize("kind", ["one feature", "three features", "a fifth", "a fifth, positive", "dense"])
@pytest.mark.parametrize("d", [16, 65, 128, 784])
def test_no_further_off_than_the_fp32_kernel(kkm, d, kind):
    """Points too few for the split take the FP32 kernel: among the same points,
    the split's error is no larger, nor is a single product's (rounded once)."""
    n, few = 3600, 2200
    X = _sparse(n, d, kind)
    Xd = X.double()
    print("split error", d, kind, flush=True)
    K = kkm.kkm_gram(X, kernel=kkm.LINEAR)[0][:few, :few].double()
    R = kkm.kkm_gram(X[:few], kernel=kkm.LINEAR)[0].double()
    want = Xd[:few] @ Xd[:few].T
    # where both round every entry once, their few different last bits leave the
    # norm of some 10^6 errors the same within 1%
    assert float((K - want).norm()) <= 1.01 * float((R - want).norm())
    if kind == "one feature":
        # h h' exact, seven roundings of at most 2^-23 of the others' sum (below 2^-6),
        # l l' below 2^-33, and one rounding of the whole
        assert bool(((K - want).abs() <= (2.0 ** -24 + 7 * 2.0 ** -29 + 2.0 ** -33) * want.abs()).all())


@pytest.mark.parametrize("full", [False, True])
def test_a_small_value_beside_a_large_one(kkm, full):
    """Rows that meet only in a feature where one of them is tiny and the other
    large: the product keeps the tiny value's last bits."""
    import torch
    n, d = 2304, 70
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    X = torch.zeros(n, d, device="cuda")
    X[::2, 0] = (1 + torch.rand(n // 2, generator=g, device="cuda")) * 2.0 ** -115
    X[::2, 1] = 1.0
    X[1::2, 0] = (1 + torch.rand(n // 2, generator=g, device="cuda")) * 2.0 ** 49
    print("split small values", full, flush=True)
    K = kkm.kkm_gram(X, kernel=kkm.LINEAR, shape=kkm.GRAM_FULL if full else kkm.GRAM_TRIANGLE)[0][::2, 1::2].double()
    want = X[::2, :1].double() @ X[1::2, :1].double().T
    assert bool(((K - want).abs() <= 2.0 ** -24 * want).all())
