"""The evaluate's kernels per configuration, from es_eval_path (CPU only: a host
rule).  The sizes of the GPU tests that name a kernel are checked against it there."""
import pytest

import paper_2212_04180_amd as P


def _path(D, N, R=1, bc=0, problem=P.PROB_SPHERE, **kw):
    return P.eval_path(P.ESConfig(num_dims=D, popsize=N, num_runs=R, problem=problem, plan_eval_blocks=bc, **kw))


@pytest.mark.parametrize("D,N,R,strategy,path", [
    (16, 32, 1, P.STRAT_OPENAI_ES, 1), (1000, 256, 1, P.STRAT_PGPE, 1), (100, 64, 1024, P.STRAT_SEP_CMA, 1),
    (131075, 130, 1, P.STRAT_OPENAI_ES, 3), (131075, 130, 1, P.STRAT_SNES, 3), (131075, 130, 1, P.STRAT_SEP_CMA, 2),
    (1_000_000, 2048, 1, P.STRAT_OPENAI_ES, 3), (2_000_000, 2, 1, P.STRAT_OPENAI_ES, 2)])
def test_kernel_of_a_configuration(D, N, R, strategy, path):
    got, partials = _path(D, N, R, strategy=strategy)
    assert got == path
    assert partials % (R * N) == 0 and (partials == 0) == (path == 1)


def test_other_problems_and_refused_configurations():
    assert P.eval_path(P.ESConfig(num_dims=8, popsize=4, problem=P.PROB_NONE)) == (0, 0)
    assert P.eval_path(P.ESConfig(num_dims=8, popsize=3)) == (0, 0)
    assert P.eval_path(P.ESConfig(num_dims=86544, popsize=64, problem=P.PROB_MLP,
                                  init=P.INIT_FANIN_NORMAL)) == (4, 0)
    assert P.lib().es_eval_path(None, None) == 0
