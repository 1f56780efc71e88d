"""The result dicts of a batched solve, built field by field, against reading
each instance's hprqp_info: keys, order, values and Python types, and the
largest residual where some are NaN or infinite."""
import ctypes as C

import numpy as np
import pytest

from paper_2507_02470_amd import _native as N
from paper_2507_02470_amd import batch as B


@pytest.mark.parametrize("count", [1, 7, 300])
def test_info_dicts(count):
    infos = (N.hprqp_info * count)()
    rng = np.random.default_rng(count)
    special = [np.nan, np.inf, -np.inf, 0.0, -0.0, 1.0]
    for i, f in enumerate(infos):
        f.term, f.iters, f.restarts = i % 4, 2 ** 40 + i, i
        for k in ("sigma", "sigma0", "lambda_A", "lambda_Q", "pobj", "dobj", "R_last", "qwx_gap"):
            setattr(f, k, rng.standard_normal())
        f.eta_p, f.eta_d, f.eta_gap = (special[(i // d) % 6] for d in (1, 6, 36))
    want = [dict(term=N.TERM[f.term], iters=int(f.iters), restarts=int(f.restarts), sigma=f.sigma,
                 sigma0=f.sigma0, lambda_A=f.lambda_A, lambda_Q=f.lambda_Q, eta_p=f.eta_p, eta_d=f.eta_d,
                 eta_gap=f.eta_gap, pobj=f.pobj, dobj=f.dobj, R_last=f.R_last, qwx_gap=f.qwx_gap,
                 kkt=max(f.eta_p, f.eta_d, f.eta_gap)) for f in infos]
    got = B._info_dicts(np.frombuffer((C.c_char * C.sizeof(infos)).from_buffer(infos), dtype=B._INFO))
    assert len(got) == count
    for g, w in zip(got, want):
        assert list(g) == list(w)
        for k in w:
            assert type(g[k]) is type(w[k]) and (g[k] == w[k] or (g[k] != g[k] and w[k] != w[k])), k
