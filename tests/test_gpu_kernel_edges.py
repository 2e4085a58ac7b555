"""Kernels at the sizes where their work split changes: remainders, first and last of a range."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import entries as oe
from oracle import hess as oh
from oracle import loglike as ol
from oracle import mlp as om
from oracle import pipeline as op

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    import paper_1904_00011_amd as P
    c = P.Context(0)
    yield c
    c.close()


# FP64 sums of at most 2^15 terms: 2^15 roundings of 2^-53 relative to the sum of magnitudes, which
# is within a factor 100 of the result here (4e-10); the oracle sums term by term.
@pytest.mark.parametrize("nbins", [1, 63, 1024, 10240, 10241, 30001])
@pytest.mark.parametrize("n", [1, 3])
def test_surrogate_loglike_bin_counts(ctx, n, nbins):
    r = np.random.default_rng(nbins + n)
    y = (r.normal(-9.0, 2.0, (n, nbins))).astype(np.float32)
    d = r.poisson(r.choice([0.0, 0.5, 40.0, 6000.0], nbins)).astype(np.int32)
    d[0] = 3
    out = torch.empty(n, dtype=torch.float64, device=DEV)
    ctx.surrogate_loglike(torch.from_numpy(y).to(DEV), torch.from_numpy(d).to(DEV), out)
    ctx.sync()
    for k in range(n):
        assert out[k].item() == pytest.approx(om.surrogate_loglike(y[k], d), rel=4e-10, abs=1e-9)
