"""A step on the strip-packed K against the step on the dense K at the sizes
where the packed step's pieces end: one point, one column past a strip, labels
missing from a strip, k of 1 and 128, more than sixteen strips to fold."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store", ["F32", "BF16"])
@pytest.mark.parametrize("n,k", [(1, 1), (63, 5), (1023, 128), (1025, 2), (2049, 1), (3000, 127), (4500, 65), (18500, 7)])
def test_packed_step_matches_dense(kkm, n, k, store):
    import torch
    r = np.random.default_rng(n + k)
    X = torch.from_numpy((r.normal(0, 0.3, (n, 8)) + 2 * r.integers(0, 3, (n, 1))).astype(np.float32)).cuda()
    lab = np.sort(r.integers(0, k, n)) if n % 2 else r.integers(0, k, n)  # sorted: a strip sees few labels
    lab = torch.from_numpy(lab.astype(np.int32)).cuda()
    a = dict(kernel=kkm.GAUSS, gamma=0.125, k_store=getattr(kkm, store))
    print("packed edges", n, k, store, flush=True)
    K, diag = kkm.kkm_gram(X, **a)
    P, pdiag = kkm.kkm_gram_packed(X, **a)
    out = []
    for step, M, d in ((kkm.kkm_iterate, K, diag), (kkm.kkm_iterate_packed, P, pdiag)):
        D, norms = torch.empty(n, k, device="cuda"), torch.empty(k, device="cuda")
        q = step(M, d, lab, k, D_out=D, ctilde_out=norms)
        out.append((q[0].cpu().numpy(), q[1].cpu().numpy(), D.cpu().numpy().astype(np.float64), norms.cpu().numpy()))
    (l0, c0, D0, n0), (l1, c1, D1, n1) = out
    # K's entries are at most 1.  A row's sum over a strip is added value by
    # value within a lane (16), then lane by lane (at most 64): 80 roundings of
    # 2^-24; everything else is compensated.  An average enters D twice, the norm
    # (an average of averages) once, and D is rounded three times.
    tol = (3 * 80 + 8) * 2.0 ** -24
    live = np.bincount(lab.cpu().numpy(), minlength=k) > 0
    assert np.abs(D0 - D1)[:, live].max() <= tol and np.abs(n0 - n1).max() <= tol
    assert np.isinf(D1[:, ~live]).all()
    i = np.arange(n)
    assert (np.abs(D0[i, l1] - D0[i, l0]) <= 2 * tol).all()
    assert c1.sum() == n and (c1 == np.bincount(l1, minlength=k)).all()


@pytest.fixture(scope="module")
def kkm():
    import paper_2501_05587_amd as kkm
    kkm.lib()
    return kkm
