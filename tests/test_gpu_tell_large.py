"""The gradient of large populations over few Philox blocks (marked gpu): its many
splits are folded by slices side by side.  Sizes at the slices' edges: one block,
a second group of one block, slices that do not divide the splits, several runs."""
import pytest

import stagecheck

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,N,R", [(3, 8448, 1), (50, 16384, 1), (257, 9000, 3), (256, 8450, 2)])
@pytest.mark.parametrize("strategy,optimizer", [("OPENAI_ES", "ADAM"), ("OPENAI_ES", "CLIPUP"), ("PGPE", "CLIPUP"),
                                                ("SNES", "ADAM"), ("SEP_CMA", "ADAM")])
def test_many_splits_match_oracle(D, N, R, strategy, optimizer):
    import paper_2212_04180_amd as P
    cfg = P.ESConfig(num_dims=D, popsize=N, num_runs=R, sigma=0.2, lr=1.0 if strategy == "SNES" else 0.01, seed=21,
                     init_lo=-2.0, init_hi=2.0, problem=P.PROB_SPHERE, strategy=getattr(P, "STRAT_" + strategy),
                     optimizer=getattr(P, "OPT_" + optimizer), sigma_lr=0.2, flags=P.FLAG_KEEP_GRAD)
    print(cfg, flush=True)
    stagecheck.run(P, cfg, 2)
