"""The population written out (marked gpu): every member against the oracle at
rows of every remainder, rows shorter and longer than a workgroup, more pairs than
one pass of the grid, and a destination that is only 4-byte aligned."""
import ctypes

import numpy as np
import pytest
import torch

from inputs import to_oracle
from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,N,R", [(1, 2, 1), (2, 5000, 2), (7, 66, 3), (255, 34, 2), (1023, 6, 1), (1025, 18, 2),
                                   (4097, 4, 5), (5, 40000, 1)])
@pytest.mark.parametrize("strategy", ["OPENAI_ES", "PGPE", "SEP_CMA"])
def test_population_matches_oracle(D, N, R, strategy):
    import paper_2212_04180_amd as P
    cfg = P.ESConfig(num_dims=D, popsize=N, num_runs=R, sigma=0.3, seed=9, problem=P.PROB_NONE,
                     strategy=getattr(P, "STRAT_" + strategy))
    es = P.ES(cfg)
    out = torch.full((R * N * D + 8,), -7.0, device="cuda")
    x = out[1:1 + R * N * D]  # 4-byte aligned
    es._check(P.lib().es_ask(es._h, ctypes.c_void_p(x.data_ptr())))
    got = out.cpu().numpy()
    assert got[0] == -7.0 and np.all(got[1 + R * N * D:] == -7.0)
    ref = O.OracleES(to_oracle(cfg)).ask()
    m = es.get_state()["m"].cpu().numpy()
    # the normals' bound (3e-7 |e| + 8e-7, |e| <= 5.77) times sigma, and the sum's rounding
    bound = 0.3 * 2.6e-6 + np.spacing(np.abs(ref) + np.abs(m)[:, None, :])
    assert np.all(np.abs(got[1:1 + R * N * D].reshape(R, N, D) - ref) <= bound)
