"""k-means++ and Lloyd on feature rows at the sizes where their tiles end (128
points, 32 or 64 clusters, 32 / 64 / 256 features), for rows that 16-byte loads
cannot read whole, and for both orders of the product's sums, against FP64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (n, f, k): the last two are large enough for the permuted order of features
SIZES = [(2, 1, 2), (64, 4, 1), (127, 31, 32), (128, 32, 33), (129, 33, 64), (257, 64, 65), (300, 65, 129),
         (1000, 257, 31), (513, 516, 7), (33000, 70, 32), (20000, 256, 60)]


@pytest.fixture(scope="module")
def kkm():
    import paper_2501_05587_amd as kkm
    kkm.lib()
    return kkm


def _features(n, f, k, pad):
    import torch
    r = np.random.default_rng(n + f + k)
    F = r.normal(0, 0.1, (n, f + pad)) + r.normal(0, 2, (k, f + pad))[r.integers(0, k, n)]
    return torch.from_numpy(F.astype(np.float32)).cuda()[:, :f]


def _nearest(F, C, norms, labels, f):
    """Labels match argmin |F_i - C_c|^2 except where FP32 cannot tell: a distance
    is ||F||^2 - 2 F.C + ||C||^2 with sums of f products, each within (f + 3)
    2^-24 of the sum of the products' sizes."""
    d = (F * F).sum(1)[:, None] - 2 * F @ C.T + norms
    size = (F * F).sum(1)[:, None] + 2 * np.abs(F) @ np.abs(C).T + norms
    err = (f + 3) * 2.0 ** -24 * size
    i = np.arange(F.shape[0])
    best = d.argmin(1)
    assert np.all(d[i, labels] - d[i, best] <= err[i, labels] + err[i, best])
    return np.maximum(d.min(1), 0).sum(), err.max(1).sum()


@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("n,f,k", SIZES)
def test_seeding_and_lloyd_step(kkm, n, f, k, pad):
    import torch
    F = _features(n, f, k, pad)
    u = np.random.default_rng(k).random(k)
    print("features", n, f, k, pad, flush=True)
    seeds, labels = kkm.kkm_feature_kmeanspp(F, k, u)[:2]
    X, seeds, lab = F.cpu().numpy().astype(np.float64), seeds.cpu().numpy(), labels.cpu().numpy()
    assert seeds[0] == int(u[0] * n) and ((0 <= seeds) & (seeds < n)).all()
    _nearest(X, X[seeds], (X[seeds] ** 2).sum(1), lab, f)
    # a seed is the first row whose running sum of squared distances passes its
    # share: the sums before and after it bracket the target, within the FP32
    # distances' error
    dmin = np.full(n, np.inf)
    for t in range(1, k):
        dmin = np.minimum(dmin, ((X - X[seeds[t - 1]]) ** 2).sum(1))
        run, total = np.cumsum(dmin), dmin.sum()
        slack = (f + 8) * 2.0 ** -23 * total
        if total > 0:
            assert run[seeds[t]] >= u[t] * total - slack
            assert run[seeds[t]] - dmin[seeds[t]] <= u[t] * total + slack
    out, it, changed, J = kkm.kkm_feature_lloyd(F, k, labels, max_iter=1, return_objective=True)
    cnt = np.bincount(lab, minlength=k)
    C = np.zeros((k, f))
    np.add.at(C, lab, X)
    C /= np.maximum(cnt, 1)[:, None]
    norms = np.where(cnt > 0, (C * C).sum(1), np.inf)
    new = out.cpu().numpy()
    # centroids are FP32 means: one more rounding of each sum of at most n rows
    want, err = _nearest(X, C, np.where(cnt > 0, norms, 1e30), new, f + n)
    assert changed[0] == (new != lab).sum() and it == 1
    assert abs(J - want) <= (f + n + 3) * 2.0 ** -24 * ((X * X).sum() + 2 * np.abs(X).sum() * np.abs(C).max()
                                                      + n * norms[cnt > 0].max())


@pytest.mark.parametrize("n,f,k,pad", [(98304, 5, 3, 0), (98305, 5, 3, 1), (98305, 4, 2, 0), (98560, 300, 2, 0),
                                       (300001, 3, 4, 0)])
def test_seeding_either_side_of_its_own_select(kkm, n, f, k, pad):
    """384 groups of 256 rows are the most that every workgroup selects from for
    itself; past them a launch selects."""
    test_seeding_and_lloyd_step(kkm, n, f, k, pad)


# (n, d, h1, h2, out): layers of fewer than 256 columns at the fewest rows that
# take the 64 x 64 tiles, columns and k around 32 and 64, rows past a whole tile
# and past the first 32768
@pytest.mark.parametrize("n,d,h1,h2,out,pad", [(4096, 33, 128, 130, 255, 0), (4099, 64, 129, 65, 200, 1),
                                               (8200, 96, 64, 65, 63, 0), (16384, 31, 1, 2, 3, 0), (32800, 7, 17, 16, 33, 1),
                                               (32768, 100, 255, 32, 64, 0)])
def test_narrow_layers_of_many_rows(kkm, n, d, h1, h2, out, pad):
    """The rows of a large call are those of small ones (other tiles, the same order
    of sums) bit for bit."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n + d)
    X = torch.randn(n, d + pad, generator=g, device="cuda")[:, :d]
    th = 0.1 * torch.randn(kkm.mlp_param_count(d, h1, h2, out), generator=g, device="cuda")
    net = dict(h1=h1, h2=h2, out=out)
    print("narrow layers", n, d, h1, h2, out, flush=True)
    F = kkm.kkm_mlp_forward(th, X, **net)
    for a in (0, 2000, n - 1001):
        assert torch.equal(F[a:a + 1001], kkm.kkm_mlp_forward(th, X[a:a + 1001], **net))
