"""The FP32 kernel matrix where its product is taken as eight bfloat16 products
of three-part values: against 64 bits, in every shape and layout, and against
the FP32 kernel for the values that are left to it.

A workspace that holds only the row norms is accepted as before: the product
then splits the rows as it stages them.
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


@pytest.mark.parametrize("kernel", ["GAUSS", "POLY"])
@pytest.mark.parametrize("store", ["F32", "BF16"])
@pytest.mark.parametrize("n,d,pad,offset", [(2304, 65, 0, 0), (2311, 784, 0, 0), (3600, 31, 0, 0), (3585, 33, 3, 1),
                                            (3700, 64, 4, 0), (4100, 128, 0, 0), (3600, 15, 0, 0), (3600, 16, 0, 0)])
def test_the_workspace_does_not_change_k(kkm, n, d, pad, offset, store, kernel):
    """Rows split beforehand, in a workspace with room for them (16-byte aligned or
    not), or while they are staged: the same K bit for bit, in every shape."""
    import torch
    X = _points(n, d, pad, offset)
    a = dict(kernel=getattr(kkm, kernel), gamma=1.0 / d, coef0=1.0, degree=2, k_store=getattr(kkm, store))
    print("split workspaces", n, d, pad, store, kernel, flush=True)
    need = kkm.gram_workspace_bytes(n, d, kkm.F32)
    K, diag = kkm.kkm_gram(X, **a)
    for ws in (_small_ws(n), torch.empty(need + 4, dtype=torch.uint8, device="cuda")[4:],
               torch.empty(need - 1, dtype=torch.uint8, device="cuda")):
        R, rdiag = kkm.kkm_gram(X, ws=ws, **a)
        assert torch.equal(K, R) and torch.equal(diag, rdiag)
    R, rdiag = kkm.kkm_gram(X, ws=_small_ws(n), shape=kkm.GRAM_FULL, **a)
    assert torch.equal(K, R) and torch.equal(diag, rdiag)
    P, _ = kkm.kkm_gram_packed(X, **a)
    R, _ = kkm.kkm_gram_packed(X, ws=_small_ws(n), **a)
    wide = (-(-n // 1024)) * 1024
    assert torch.equal(P[:1024 * wide].view(1024, wide)[:, :n], R[:1024 * wide].view(1024, wide)[:, :n])


@pytest.mark.parametrize("small", [False, True])
@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 2.0 ** 51, 2.0 ** -46])
def test_only_the_tiles_of_marked_rows_leave_the_split(kkm, value, full, small):
    """A row outside the split's range: the tiles of its 128 rows are the FP32
    kernel's, the others are what they are without that row."""
    import torch
    n, d = 2311, 70
    X = _points(n, d)
    Y = X.clone()
    Y[n - 1, 3] = value
    a = dict(kernel=kkm.LINEAR, shape=kkm.GRAM_FULL if full else kkm.GRAM_TRIANGLE,
             ws=_small_ws(n) if small else None)
    print("split marked rows", value, full, small, flush=True)
    K = kkm.kkm_gram(Y, **a)[0].clone()
    last = (n - 1) // 128 * 128
    assert torch.equal(K[:last, :last], kkm.kkm_gram(X, **a)[0][:last, :last])
    R = kkm.kkm_gram(Y[1000:], kernel=kkm.LINEAR)[0].contiguous()  # too few for the split
    bits = lambda t: t.contiguous().view(torch.int32)
    assert torch.equal(bits(K[last:, 1000:n]), bits(R[last - 1000:n - 1000, :n - 1000]))
    assert torch.equal(bits(K[1000:n, last:n]), bits(R[:n - 1000, last - 1000:n - 1000]))


def test_batched_equals_the_single_runs(kkm):
    """Problems whose product is split, one of them with rows outside its range, and
    one too small for it, in one batch, with room for the split rows and without:
    the single runs' labels and objectives bit for bit."""
    import torch
    X = [_points(2311, 96), _points(3601, 20).clone(), _points(500, 20), _points(2400, 70)]
    X[1][77] *= 2.0 ** -60
    X[1][3000, 5] = 2.0 ** 55
    probs = [dict(X=x, k=5, kernel=kkm.POLY, gamma=2.0 ** -60, coef0=1.0, degree=2) for x in X]
    g = np.random.default_rng(3)
    ns = [x.shape[0] for x in X]
    l0 = torch.from_numpy(g.integers(0, 5, sum(ns)).astype(np.int32)).cuda()
    need = kkm.kkm_fit_batched_workspace_bytes(probs, kkm.F32, kkm.F32)
    room = 256 + sum(-(-n // 128) * 8 * (-(-x.shape[1] // 32)) * 3072 for n, x in zip(ns, X) if n >= 2304)
    print("split batch", flush=True)
    for ws in (None, torch.empty(need - room, dtype=torch.uint8, device="cuda")):
        r = kkm.kkm_fit_batched(probs, l0, kkm.F32, kkm.F32, max_iter=6, ws=ws)
        at = 0
        for b, (n, p) in enumerate(zip(ns, probs)):
            one = kkm.kkm_fit_ex(p["X"], 5, l0[at:at + n], kernel=kkm.POLY, gamma=2.0 ** -60, coef0=1.0, degree=2,
                                 max_iter=6)
            assert torch.equal(r["labels"][at:at + n], one["labels"]), b
            assert r["objective"][b] == one["objective"] and r["iters"][b] == one["iters"], b
            at += n


def test_fresh_training_with_the_smaller_workspace(kkm):
    """A large batch's kernel values are split: a workspace without room for the
    split rows gives the same step."""
    import torch
    B, d, net = 2304, 70, dict(h1=40, h2=36, out=20)
    X = _points(B, d)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    th = torch.randn(kkm.mlp_param_count(d, 40, 36, 20), generator=g, device="cuda") * 0.1
    need = kkm.lib().kkm_mlp_train_fresh_workspace_bytes(B, d, 40, 36, 20)
    out = []
    print("split training", flush=True)
    for size in (need, need - 256 - -(-B // 128) * 8 * 3 * 3072):
        p, m, v = th.clone(), torch.zeros_like(th), torch.zeros_like(th)
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        tr = kkm.kkm_mlp_train_fresh(p, m, v, X, B, kernel=kkm.GAUSS, gamma=1.0 / d, ws=ws, **net)
        out.append((p, m, v, tr))
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("kind", ["growing features", "shrinking features", "log-normal", "offset"])
@pytest.mark.parametrize("d", [16, 33, 65, 128, 784])
def test_features_of_different_sizes(kkm, d, kind):
    """The matrix unit sums eight products at a time, each cut off at 2^-24 of the
    largest one's power of two, and rounds their sums and the running sum to
    nearest (as measured on gfx950): the bound that follows, where the products
    of a sum differ by many powers of two."""
    import torch
    n = 3600
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    X = torch.randn(n, d, generator=g, device="cuda")
    if kind == "growing features":
        X = X * torch.exp2(torch.linspace(-12, 0, d, device="cuda"))
    elif kind == "shrinking features":
        X = X * torch.exp2(torch.linspace(0, -12, d, device="cuda"))
    elif kind == "log-normal":
        X = X * torch.exp2(4 * torch.randn(n, d, generator=g, device="cuda"))
    else:
        X = X + 10
    print("split sizes", d, kind, flush=True)
    K = kkm.kkm_gram(X, kernel=kkm.LINEAR)[0]
    Xd = X.double()
    # of a slab's h h': seven cut-offs and four roundings; per slab one addition
    # and, at 2^-6 of it, 28 roundings of the other products' sum; those products'
    # cut-offs (49 2^-6) and the joining of the two sums.  |h h'| <= 1.02 |x y|.
    slabs = -(-d // 32)
    bound = 1.02 * (11 + slabs * (1 + 28 / 64) + 49 / 64 + 1) * 2.0 ** -24 * (Xd.abs() @ Xd.abs().T)
    assert bool(((K.double() - Xd @ Xd.T).abs() <= bound).all())
