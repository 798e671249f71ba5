"""Evaluate and reduction in one launch (marked gpu): the fitness against the
oracle where a workgroup holds many pairs, one pair, or two passes of chunks,
and at both sides of the plan's lines."""
import numpy as np
import pytest
import torch

import stagecheck
from inputs import to_oracle
from oracle import oracle as O

pytestmark = pytest.mark.gpu


# (D, N, R, plan_eval_blocks) and the path (es_eval_path; 1: one launch) of each strategy.  512 chunks are the most
# that one launch takes (two passes, the largest partials in LDS), 513 too many; then both sides of the lines: 96 and
# 95 pairs, 6e6 pair-blocks (1.5e6 with a sigma a dim), workgroups half empty in many runs
SIZES = [((1, 2, 1, 0), (1, 1, 1)), ((2, 798, 1, 0), (1, 1, 1)), ((13, 130, 5, 1), (1, 1, 1)),
         ((1000, 256, 1, 0), (1, 1, 1)), ((2046, 18, 2, 1), (1, 1, 1)), ((2050, 10, 1, 1), (2, 2, 2)),
         ((4099, 18, 2, 1), (2, 2, 2)), ((4100, 10, 1, 1), (2, 2, 2)), ((2049, 66, 3, 2), (1, 1, 1)),
         ((30001, 200, 1, 0), (1, 1, 2)), ((10007, 514, 2, 0), (1, 1, 2)), ((20002, 192, 1, 0), (1, 1, 2)),
         ((20002, 190, 1, 0), (2, 2, 2)), ((11714, 1024, 1, 0), (1, 1, 2)), ((11718, 1024, 1, 0), (1, 2, 2)),
         ((46872, 1024, 1, 0), (1, 3, 2)), ((46876, 1024, 1, 0), (3, 3, 2)), ((2101, 512, 16, 0), (2, 2, 2))]


@pytest.mark.parametrize("size", range(len(SIZES)))
@pytest.mark.parametrize("strategy", ["OPENAI_ES", "PGPE", "SEP_CMA"])
@pytest.mark.parametrize("problem", ["SPHERE", "SHIFTED_SPHERE", "ROSENBROCK", "RASTRIGIN"])
def test_fitness_matches_oracle(size, strategy, problem):
    import paper_2212_04180_amd as P
    (D, N, R, bc), paths = SIZES[size]
    cfg = P.ESConfig(num_dims=D, popsize=N, num_runs=R, sigma=0.1, seed=5, init_lo=-2.0, init_hi=2.0,
                     problem=getattr(P, "PROB_" + problem), strategy=getattr(P, "STRAT_" + strategy), plan_eval_blocks=bc)
    assert P.eval_path(cfg)[0] == paths[("OPENAI_ES", "PGPE", "SEP_CMA").index(strategy)]
    es, ref = P.ES(cfg), O.OracleES(to_oracle(cfg))
    es.ask()
    f, fr, xs = es.eval().cpu().numpy(), ref.eval(), ref.ask()
    pdata = O.problem_data(to_oracle(cfg)) if problem == "SHIFTED_SPHERE" else None
    for r in range(R):
        for j in range(0, N, 256):
            bound = stagecheck._fitness_bound(cfg, xs[r][j:j + 256], np.float32(0.1), pdata)
            assert np.all(np.abs(f[r, j:j + 256].astype(np.float64) - fr[r, j:j + 256]) <= bound), (r, j)
    # a second evaluate of the same ask, and the other members' buffer untouched
    out = torch.full((R, N + 3), -5.0, device="cuda")
    flat = out.view(-1)[1:1 + R * N].view(R, N)
    es.eval(flat)
    got = out.view(-1).cpu().numpy()
    np.testing.assert_array_equal(got[1:1 + R * N].reshape(R, N), f)
    assert got[0] == -5.0 and np.all(got[1 + R * N:] == -5.0)
