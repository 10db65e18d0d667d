"""The network's gradient where the batch is split over workgroups: one
split and several, a ragged last split, ragged output tiles (-m gpu).

The gradient does not depend on the order of the batch's rows (reversing
them moves rows between splits; a row read twice or left out would show as
a change of about 1/batch), and the batch's gradient is the mean of the
gradients of its 256-row parts, each of which is one split (the parts hold
the same BF16 values: the 1/batch factor differs by a power of two).  Only
the order of the FP32 sums differs.  A sum of n <= 4096 terms rounds by about
sqrt(n) 2^-25 of a term, the sums themselves are about sqrt(n) terms or more
(they cancel like random signs), so the relative difference is about 2^-25
times a small factor; 1e-5 leaves two orders of magnitude.
"""
import numpy as np
import pytest

from oracle import mlp as OM

pytestmark = pytest.mark.gpu

SPLIT_REL = 1e-5


@pytest.fixture(scope="module")
def fm():
    from paper_2008_03518_amd import fastmdp
    return fastmdp


def _inputs(n_out, batch, seed):
    rng = np.random.default_rng(seed)
    p = OM.init_params(rng, n_out)
    for k in ("b1", "b2", "b3"):
        p[k] = rng.normal(0.0, 0.05, p[k].shape)
    return p, rng.uniform(0.0, 1.0, (batch, OM.N_FEAT)).astype(np.float32), rng.integers(0, n_out, batch).astype(np.int32)


# batches of one split (32, 480), of two (544) and four with a shorter last one (1056), of the most splits (4096)
@pytest.mark.parametrize("n_out,batch", [(81, 32), (360, 480), (65, 544), (360, 1056), (510, 4096)])
def test_gradient_does_not_depend_on_row_order(fm, n_out, batch):
    params, X, y = _inputs(n_out, batch, 70 + batch)
    net = fm.Mlp(n_out, max_batch=batch)
    net.set_params(params)
    g, loss = net.gradient(X, y)
    r, rloss = net.gradient(X[::-1].copy(), y[::-1].copy())
    assert abs(loss - rloss) <= SPLIT_REL * abs(loss)
    for k in g:
        rel = np.linalg.norm(g[k] - r[k]) / np.linalg.norm(g[k])
        print(f"[split grad] n_out {n_out} batch {batch} {k}: {rel:.2e} from the reversed batch's", flush=True)
        assert rel <= SPLIT_REL, k
    net.close()


@pytest.mark.parametrize("batch", [512, 4096])
def test_split_gradient_equals_mean_of_parts(fm, batch):
    params, X, y = _inputs(360, batch, 90 + batch)
    net = fm.Mlp(360, max_batch=batch)
    net.set_params(params)
    g, _ = net.gradient(X, y)
    parts = [net.gradient(X[i: i + 256], y[i: i + 256])[0] for i in range(0, batch, 256)]
    for k in g:
        mean = sum(p[k] for p in parts) / len(parts)
        rel = np.linalg.norm(g[k] - mean) / np.linalg.norm(mean)
        print(f"[split grad] batch {batch} {k}: {rel:.2e} from the mean of its parts", flush=True)
        assert rel <= SPLIT_REL, k
    net.close()
