"""The evaluate of large runs (even and odd sums of a pair) against the oracle
(marked gpu): every problem with a scalar and a per-dimension sigma, ragged
dimensions and populations, chunks that are not whole groups, and the lanes that
fall back to evaluating member by member."""
import numpy as np
import pytest
import torch

import stagecheck
from inputs import to_oracle
from oracle import oracle as O

pytestmark = pytest.mark.gpu


def _P():
    import paper_2212_04180_amd as P
    return P


def _cfg(problem, D, N, R=1, strategy="openai", bc=0, sigma=0.1, **kw):
    P = _P()
    return P.ESConfig(num_dims=D, popsize=N, num_runs=R, sigma=sigma, seed=5, init_lo=-2.0, init_hi=2.0,
                      problem=getattr(P, "PROB_" + problem.upper()),
                      strategy=P.STRAT_PGPE if strategy == "pgpe" else P.STRAT_OPENAI_ES, plan_eval_blocks=bc, **kw)


def _both(cfg, m=None, sig=None):
    es, ref = _P().ES(cfg), O.OracleES(to_oracle(cfg))
    if m is not None:
        z = torch.zeros(m.shape, device="cuda")
        es.set_state(torch.from_numpy(m).cuda(), z, z, 0)
        ref.set_state(m, np.zeros_like(m), np.zeros_like(m), 0, sig=sig)
    if sig is not None:
        es.set_strategy_state(torch.from_numpy(sig).cuda())
        ref.set_state(ref.m, ref.m1, ref.v, 0, sig=sig)
    es.ask()
    return es.eval().cpu().numpy(), ref.eval(), ref


# (D, N, R, plan_eval_blocks), the path (es_eval_path) with one sigma and with one a dim: 3 is the kernel of the even
# and odd sums (more than 2^18 pair-blocks a run and 2^16 wave-blocks, and no one-launch evaluate), the others are
# large runs on either side of it
SIZES = [((131075, 130, 1, 0), (3, 3)), ((131077, 94, 2, 0), (3, 3)), ((131075, 130, 1, 7), (3, 3)),
         ((262149, 66, 1, 3), (3, 3)), ((23501, 2048, 1, 700), (3, 3)), ((59302, 1026, 1, 0), (3, 3)),
         ((16389, 510, 1, 0), (1, 1)), ((33334, 1026, 1, 7), (3, 3)), ((131075, 128, 2, 0), (1, 3)),
         ((16400, 512, 2, 3), (2, 2)), ((20003, 2048, 1, 700), (1, 3))]


@pytest.mark.parametrize("strategy", ["openai", "pgpe"])
@pytest.mark.parametrize("problem", ["sphere", "shifted_sphere", "rosenbrock", "rastrigin"])
@pytest.mark.parametrize("size", range(len(SIZES)))
def test_large_evaluate_matches_oracle(size, problem, strategy):
    (D, N, R, bc), paths = SIZES[size]
    cfg = _cfg(problem, D, N, R, strategy, bc)
    assert _P().eval_path(cfg)[0] == paths[strategy == "pgpe"]
    sig = None
    if strategy == "pgpe":
        sig = np.random.default_rng(size).uniform(0.02, 0.2, (R, D)).astype(np.float32)
    print(problem, strategy, SIZES[size], flush=True)
    f, fr, ref = _both(cfg, sig=sig)
    pdata = O.problem_data(to_oracle(cfg)) if problem == "shifted_sphere" else None
    xs = ref.ask()
    for r in range(R):
        scale = sig[r] if sig is not None else np.float32(cfg.sigma)
        for j0 in range(0, N, 256):
            bound = stagecheck._fitness_bound(cfg, xs[r][j0:j0 + 256], scale, pdata)
            assert np.all(np.abs(f[r, j0:j0 + 256].astype(np.float64) - fr[r, j0:j0 + 256]) <= bound), (r, j0)


@pytest.mark.parametrize("D,N,path", [(16389, 512, 1), (131075, 130, 3)])
@pytest.mark.parametrize("problem", ["sphere", "shifted_sphere", "rosenbrock"])
def test_members_near_the_optimum_keep_their_digits(problem, D, N, path):
    # pair 3's + member sits on the optimum: its even and odd sums cancel
    cfg = _cfg(problem, D, N, sigma=0.5)
    assert _P().eval_path(cfg)[0] == path
    oc = to_oracle(cfg)
    eps = O.normals(cfg.seed, O.DOM_NOISE, 3, 0, 0, cfg.num_dims)
    opt = O.problem_data(oc) if problem == "shifted_sphere" else np.float32(1.0 if problem == "rosenbrock" else 0.0)
    m = (opt - np.float32(0.5) * eps).astype(np.float32)[None]
    f, fr, ref = _both(cfg, m)
    pdata = O.problem_data(oc) if problem == "shifted_sphere" else None
    bound = stagecheck._fitness_bound(cfg, ref.ask()[0], np.float32(0.5), pdata)
    assert np.all(np.abs(f[0].astype(np.float64) - fr[0]) <= bound)
    assert f[0, 3] <= fr[0, 3] + bound[3] and bound[3] < 1e-6 * f[0, 3 + N // 2]


@pytest.mark.parametrize("strategy", ["openai", "pgpe"])
@pytest.mark.parametrize("problem", ["sphere", "shifted_sphere", "rosenbrock", "rastrigin"])
@pytest.mark.parametrize("value", [1e19, 3e20, np.inf, np.nan])
@pytest.mark.parametrize("D,N,path", [(16389, 512, 1), (131075, 130, 3)])
def test_overflow_and_nan_as_member_by_member(value, problem, strategy, D, N, path):
    # one dim of the mean is huge or not a number: the same infinities and NaN as the oracle's members
    cfg = _cfg(problem, D, N, strategy=strategy)
    assert _P().eval_path(cfg)[0] == path
    m = np.random.default_rng(1).uniform(-2, 2, (1, D)).astype(np.float32)
    m[0, 9001] = value
    sig = np.full((1, D), 0.1, np.float32) if strategy == "pgpe" else None
    with np.errstate(over="ignore", invalid="ignore"):
        f, fr, _ = _both(cfg, m, sig)
        fr = fr.astype(np.float32)
    if problem == "rosenbrock" and np.isfinite(value):
        fr[:] = np.inf  # (1e19)^4 passes fp32's range in the kernel's terms, not in the oracle's
    np.testing.assert_array_equal(np.isnan(f), np.isnan(fr))
    ok = np.isfinite(fr)
    np.testing.assert_array_equal(f[~ok], fr[~ok])
    np.testing.assert_allclose(f[ok], fr[ok], rtol=1e-5)


def _exact(P, cfg, x, shift):
    """Fitness of the fp32 members x [N][D] in 64 bits."""
    f = torch.empty(len(x), dtype=torch.float64, device="cuda")
    for j in range(0, len(x), 64):
        y = x[j:j + 64].double()
        if cfg.problem == P.PROB_ROSENBROCK:
            f[j:j + 64] = (100 * (y[:, 1:] - y[:, :-1] ** 2) ** 2 + (1 - y[:, :-1]) ** 2).sum(1)
        else:
            f[j:j + 64] = ((y - shift) ** 2).sum(1)
    return f


@pytest.mark.parametrize("strategy", ["openai", "pgpe"])
@pytest.mark.parametrize("problem", ["sphere", "shifted_sphere", "rosenbrock"])
@pytest.mark.parametrize("where", ["near", "near and far", "one dim far", "far"])
def test_fitness_is_that_of_the_members_handed_out(where, problem, strategy):
    """Down to perturbations below the last place of the mean, f is f of the fp32 members.  4 x 2^-24 of f: its
    own rounding, the sums' (16 dims in fp32), what is left of the members', and the normals' squares by their
    radius instead of cosine and sine.  Where one dim holds the sum its 16 dims' roundings do not average: 16 x."""
    P = _P()
    for sigma in (1e-1, 1e-2, 3e-3, 1e-3, 1e-4, 1e-5, 1e-6, 1e-7):
        cfg = _cfg(problem, 131075, 130, 1, strategy, sigma=sigma)
        assert P.eval_path(cfg)[0] == 3
        es = P.ES(cfg)
        gen = torch.Generator("cuda").manual_seed(7)
        D = cfg.num_dims
        shift = es.problem_data() if problem == "shifted_sphere" else torch.zeros(D, device="cuda")
        off = torch.randn(1, D, generator=gen, device="cuda")
        scale = torch.full((1, D), sigma, device="cuda")
        if where == "near and far":
            scale[:, D // 3:] = 1.0
        elif where == "one dim far":
            scale[:, 70001] = 30.0
        elif where == "far":
            scale[:] = 1.0
        m = ((1.0 if problem == "rosenbrock" else shift) + scale * off).float().reshape(1, D)
        z = torch.zeros_like(m)
        es.set_state(m, z, z, 0)
        if strategy == "pgpe":
            es.set_strategy_state(sigma * (0.5 + torch.rand(1, D, generator=gen, device="cuda")))
        x = es.ask(materialize=True)[0]
        ref = _exact(P, cfg, x, shift.double())
        err = float(((es.eval()[0].double() - ref).abs() / ref).max())
        print(where, problem, strategy, sigma, f"{err:.2e}", flush=True)
        assert err <= (16 if where == "one dim far" else 4) * 2.0 ** -24, (sigma, err)
        es.close()
