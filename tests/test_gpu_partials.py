"""Partial sums of large evaluates (marked gpu): many runs or members do not
take more of them than the smaller runs' plan or the static scratch holds, so
the evaluates that es_eval_noalloc takes stay the same and a handle's memory
stays near its state's."""
import numpy as np
import pytest
import torch

import stagecheck
from inputs import to_oracle
from oracle import oracle as O

pytestmark = pytest.mark.gpu


# (D, N, R): 3.1e6, 3.3e6, 2.8e6 and 3.1e6 floats of partials by wave count; two launches, even and odd sums
@pytest.mark.parametrize("D,N,R", [(3696, 822, 268), (8200, 410, 186), (30000, 512, 30), (61993, 29590, 1)])
def test_noalloc_takes_many_runs(D, N, R):
    import paper_2212_04180_amd as P
    cfg = P.ESConfig(num_dims=D, popsize=N, num_runs=R, sigma=0.1, seed=5, init_lo=-2.0, init_hi=2.0,
                     problem=P.PROB_SPHERE)
    assert P.eval_path(cfg)[0] == 3
    es = P.ES(cfg)
    mean = es.get_state()["m"]
    es.ask()
    f_ref = es.eval()
    f = P.eval_noalloc(cfg, mean, torch.full((R,), 0.1, device="cuda"), 0)
    assert torch.equal(f, f_ref)
    # the last run's first member against the oracle's arithmetic
    m = mean[R - 1].cpu().numpy()
    x = (m + np.float32(0.1) * O.normals(cfg.seed + R - 1, O.DOM_NOISE, 0, 0, 0, D)).astype(np.float32)[None]
    bound = stagecheck._fitness_bound(cfg, x, np.float32(0.1), None)
    assert abs(float(f[R - 1, 0]) - float(np.sum(x.astype(np.float64) ** 2))) <= bound[0]


def test_handle_memory_of_many_members():
    # 45,472 dims x 4474 members x 136 runs: state of 25 MB an array, partials of at most 16 MB
    import paper_2212_04180_amd as P
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    es = P.ES(P.ESConfig(num_dims=45472, popsize=4474, num_runs=136, seed=5, problem=P.PROB_SPHERE))
    es.sync()
    assert free - torch.cuda.mem_get_info()[0] < 400 << 20


def test_one_launch_keeps_no_partials():
    # 20,003 dims x 2048 members in one launch: 10 MB of partial sums a handle if they were allocated
    import paper_2212_04180_amd as P
    cfg = P.ESConfig(num_dims=20003, popsize=2048, seed=5, problem=P.PROB_SPHERE)
    assert P.eval_path(cfg) == (1, 0)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    handles = [P.ES(cfg) for _ in range(8)]
    handles[-1].sync()
    assert free - torch.cuda.mem_get_info()[0] < 8 * 6 << 20
