"""The evaluate's kernels per configuration, from es_eval_path (CPU only: a host
rule).  The sizes of the GPU tests that name a kernel are checked against it there."""
import ctypes
import math
import random

import pytest
import torch

import paper_2212_04180_amd as P


def _path(D, N, R=1, bc=0, problem=P.PROB_SPHERE, **kw):
    return P.eval_path(P.ESConfig(num_dims=D, popsize=N, num_runs=R, problem=problem, plan_eval_blocks=bc, **kw))


@pytest.mark.parametrize("D,N,R,strategy,path", [
    (16, 32, 1, P.STRAT_OPENAI_ES, 1), (1000, 256, 1, P.STRAT_PGPE, 1), (100, 64, 1024, P.STRAT_SEP_CMA, 1),
    (131075, 130, 1, P.STRAT_OPENAI_ES, 3), (131075, 130, 1, P.STRAT_SNES, 3), (131075, 130, 1, P.STRAT_SEP_CMA, 2),
    (1_000_000, 2048, 1, P.STRAT_OPENAI_ES, 3), (2_000_000, 2, 1, P.STRAT_OPENAI_ES, 2),
    # one launch where it pays: many runs of full workgroups, but not of half-empty ones, of more than two passes
    # over the chunks, or of a third row a lane
    (1000, 256, 1000, P.STRAT_OPENAI_ES, 1), (2000, 512, 64, P.STRAT_SNES, 1), (4000, 512, 32, P.STRAT_OPENAI_ES, 2),
    (4000, 128, 128, P.STRAT_SEP_CMA, 2), (2100, 512, 8, P.STRAT_OPENAI_ES, 1), (2100, 512, 32, P.STRAT_OPENAI_ES, 2),
    (8192, 64, 1, P.STRAT_OPENAI_ES, 1), (9000, 64, 1, P.STRAT_OPENAI_ES, 2), (16384, 128, 1, P.STRAT_SEP_CMA, 2),
    (10007, 1024, 1, P.STRAT_PGPE, 1), (10007, 1024, 2, P.STRAT_PGPE, 2), (10007, 1024, 2, P.STRAT_OPENAI_ES, 1),
    (2100, 1000, 16, P.STRAT_OPENAI_ES, 3)])
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


@pytest.mark.parametrize("D,N,R", [(8200, 410, 186), (1100, 4096, 100), (500, 16384, 16), (3696, 822, 268), (2100, 4096, 64),
                                   (7157, 1776, 27), (1148, 1842, 213), (1_000_000, 2048, 1)])
@pytest.mark.parametrize("strategy", [P.STRAT_OPENAI_ES, P.STRAT_SEP_CMA])
def test_chunks_of_large_evaluates_fill_the_xcds(D, N, R, strategy):
    # chunk c runs on XCD c mod 8: the fullest one holds at most a quarter more than the mean
    path, partials = _path(D, N, R, strategy=strategy)
    chunks = partials // (R * N)
    assert path in (2, 3) and -(-chunks // 8) * 8 <= 1.25 * chunks, chunks


def test_partials_of_large_evaluates_are_bounded():
    # by the 24,576-wave plan of the smaller runs or the static scratch, whichever is larger
    rng = random.Random(5)
    for _ in range(20000):
        D, N, R = (int(math.exp(rng.uniform(0.0, math.log(hi)))) for hi in (4e9, 200000, 65535))
        N = 2 * max(1, N // 2)
        if R * D > 6e10 or R * N * D > 1e15:
            continue
        waves = -(-min(-(-N // 2 // 64) * 64, 1024) // 64) * -(-(N // 2) // 1024) * R
        nb = -(-D // 4)
        bc = max(4, -(-nb // max(1, -(-24576 // waves))))
        _, partials = _path(D, N, R, strategy=rng.choice((P.STRAT_OPENAI_ES, P.STRAT_PGPE, P.STRAT_SEP_CMA)))
        if (N // 2) * nb > 1 << 18:
            assert partials <= max(-(-nb // bc) * R * N, 1 << 22), (D, N, R)


@pytest.mark.parametrize("D,N,R,path", [(400, 66, 65535, 1), (4_000_000, 8_000_000, 1, 3)])
@pytest.mark.skipif(torch.cuda.is_available(), reason="made-up pointers: only where nothing could run on them")
def test_noalloc_is_held_to_two_launches(D, N, R, path):
    # refused before any device work where two launches would not fit the static scratch, whichever path runs
    cfg = P.ESConfig(num_dims=D, popsize=N, num_runs=R, problem=P.PROB_SPHERE)
    assert P.eval_path(cfg)[0] == path
    cs, p = cfg.cstruct(), ctypes.c_void_p(64)
    assert P.lib().es_eval_noalloc(ctypes.byref(cs), p, None, p, 0, p, None) == -1
    assert b"partial sums in two launches" in P.lib().es_last_error(None)
