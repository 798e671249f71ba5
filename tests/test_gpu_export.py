"""State read out by one launch (marked gpu): every array of a ragged, several-run
state equals the one read by itself, and nothing beyond the dense rows is written."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,R", [(1, 1), (1, 5), (3, 2), (4, 3), (7, 300), (1023, 4), (1026, 1), (70001, 3)])
def test_state_and_strategy_state_out(D, R):
    import paper_2212_04180_amd as P
    es = P.ES(P.ESConfig(num_dims=D, popsize=6, num_runs=R, seed=3, problem=P.PROB_SPHERE, strategy=P.STRAT_PGPE,
                         optimizer=P.OPT_CLIPUP))
    rng = np.random.default_rng(D)
    src = [torch.from_numpy(rng.normal(size=(R, D)).astype(np.float32)).cuda() for _ in range(5)]
    es.set_state(src[0], src[1], src[2], 7)
    es.set_strategy_state(src[3].abs(), src[4])
    L, h = P.lib(), es._h
    t = ctypes.c_int64()
    buf = torch.full((3, R * D + 8), -9.0, device="cuda")  # rows at 4-byte offsets 1, 2, 3
    at = [buf[k][1 + k:1 + k + R * D] for k in range(3)]
    es._check(L.es_get_state(h, *[ctypes.c_void_p(a.data_ptr()) for a in at], ctypes.byref(t)))
    got = buf.cpu().numpy()
    for k in range(3):
        np.testing.assert_array_equal(got[k, 1 + k:1 + k + R * D], src[k].cpu().numpy().ravel())
        assert np.all(got[k, :1 + k] == -9.0) and np.all(got[k, 1 + k + R * D:] == -9.0)
    alone = torch.empty(R, D, device="cuda")
    es._check(L.es_get_state(h, None, ctypes.c_void_p(alone.data_ptr()), None, ctypes.byref(t)))
    assert torch.equal(alone, src[1]) and t.value == 7
    sg, ve = es.strategy_state(velocity=True)
    assert torch.equal(sg, src[3].abs()) and torch.equal(ve, src[4])


def test_overlapping_destinations_keep_the_last_array():
    import paper_2212_04180_amd as P
    es = P.ES(P.ESConfig(num_dims=70001, popsize=6, seed=3, problem=P.PROB_SPHERE))
    src = [torch.full((1, 70001), v, device="cuda") for v in (1.0, 2.0, 3.0)]
    es.set_state(*src, 7)
    buf = torch.zeros(70001 + 5000, device="cuda")
    at = [ctypes.c_void_p(buf[k:].data_ptr()) for k in (0, 5000, 0)]
    es._check(P.lib().es_get_state(es._h, *at, None))
    got = buf.cpu().numpy()
    assert np.all(got[:70001] == 3.0) and np.all(got[70001:] == 2.0)


def test_destination_shorter_than_its_array_is_refused():
    # the runtime's copy refuses an array that runs past its destination's
    # allocation; so does the call with several destinations (the allocation's
    # page holds the array all the same)
    import paper_2212_04180_amd as P
    es = P.ES(P.ESConfig(num_dims=512, popsize=6, seed=3, problem=P.PROB_SPHERE))
    src = [torch.full((1, 512), v, device="cuda") for v in (1.0, 2.0, 3.0)]
    es.set_state(*src, 7)
    L = P.lib()
    L.hipMalloc.argtypes, L.hipFree.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t], [ctypes.c_void_p]
    short = ctypes.c_void_p()
    assert L.hipMalloc(ctypes.byref(short), 1024) == 0
    out = torch.zeros(2, 512, device="cuda")
    at = [ctypes.c_void_p(out[0].data_ptr()), short, ctypes.c_void_p(out[1].data_ptr())]
    assert L.es_get_state(es._h, None, short, None, None) == -3  # alone: the copy's own refusal
    L.hipGetLastError()
    assert L.es_get_state(es._h, *at, None) == -3
    assert b"copy out" in L.es_last_error(es._h)
    L.hipGetLastError()
    torch.cuda.synchronize()
    assert torch.all(out[0] == 1.0) and torch.all(out[1] == 0.0)
    st = es.get_state()
    assert all(torch.equal(st[k], x) for k, x in zip(("m", "m1", "v"), src))
    assert L.hipFree(short) == 0


@pytest.mark.parametrize("N,R", [(2, 1), (6, 1), (6, 3), (10, 2), (1030, 1), (70002, 1)])
def test_weights_and_ranks_out(N, R):
    # one row of N R words without padding: sizes of both remainders, each
    # array as it reads by itself, nothing written beyond it
    import paper_2212_04180_amd as P
    es = P.ES(P.ESConfig(num_dims=5, popsize=N, num_runs=R, seed=3, problem=P.PROB_NONE))
    es.ask()
    es.tell(torch.randn(R, N, device="cuda"))
    L, buf = P.lib(), torch.full((4, N * R + 3), -9, dtype=torch.int32, device="cuda")
    at = [ctypes.c_void_p(buf[k][1:].data_ptr()) for k in range(4)]
    es._check(L.es_get_shaped(es._h, at[0], at[1]))
    es._check(L.es_get_shaped(es._h, at[2], None))
    es._check(L.es_get_shaped(es._h, None, at[3]))
    got = buf.cpu().numpy()
    np.testing.assert_array_equal(got[0], got[2])
    np.testing.assert_array_equal(got[1], got[3])
    assert np.all(got[:, 0] == -9) and np.all(got[:, 1 + N * R:] == -9)
    for r in range(R):
        np.testing.assert_array_equal(np.sort(got[1, 1 + r * N:1 + (r + 1) * N]), np.arange(N))


def test_captured_readout_follows_the_state():
    # es_get_state and es_get_strategy_state in a graph: every replay reads the state of its time
    import paper_2212_04180_amd as P
    s = torch.cuda.Stream()
    es = P.ES(P.ESConfig(num_dims=1027, popsize=6, num_runs=3, seed=3, problem=P.PROB_SPHERE, strategy=P.STRAT_PGPE), stream=s)
    out = torch.zeros(4, 3, 1027, device="cuda")
    at = [ctypes.c_void_p(o.data_ptr()) for o in out]
    L = P.lib()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        es._check(L.es_get_state(es._h, *at[:3], None))
        es._check(L.es_get_strategy_state(es._h, at[3], None))
    for k in range(4):
        with torch.cuda.stream(s):
            src = [torch.randn(3, 1027, device="cuda") for _ in range(3)] + [torch.rand(3, 1027, device="cuda")]
            es.set_state(*src[:3], k)
            es.set_strategy_state(src[3])
            g.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, src):
            assert torch.equal(a, b), k
