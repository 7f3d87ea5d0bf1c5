"""The one-launch compression step at the edges of its range: lengths around every switch of its layout (one
block per node, several blocks that meet, more blocks than are resident at once), against the oracle bit for bit."""
import numpy as np
import pytest

from oracle import adacgd_oracle as O
from test_gpu_parity import _cuda, _eng, compare_step, make_vectors, until_near_tie

pytestmark = pytest.mark.gpu


DIMS = [(3, 1024), (3, 1025), (2, 4097), (2, 8193), (2, 16384), (2, 16385), (2, 20481), (3, 65535), (1, 65537), (1, 1 << 20)]


@pytest.mark.parametrize("n,d,kind", [(n, d, k) for n, d in DIMS for k in ("normal", "ties", "const", "denormal")]
                         + [(130, 18435, "normal")])
def test_one_launch_step_at_the_edges_of_its_layout(n, d, kind):
    check_steps(n, d, kind)


@pytest.mark.parametrize("n,d,kind", [(n, d, k) for n, d in [(2, 16385), (2, 20481), (3, 65535), (1, 65537), (1, 1 << 20)]
                                      for k in ("normal", "ties", "const", "sparse")] + [(130, 18435, "normal")])
def test_one_launch_step_where_blocks_do_not_wait_for_each_other(n, d, kind):
    """A node whose blocks were not all running at once is done by one of them; between other launches both ways may occur."""
    check_steps(n, d, kind, _eng().FLAG_NO_WAIT)


@pytest.mark.parametrize("n,d", [(3, 20000), (2, 16385)])
def test_compressed_start_and_differences_where_blocks_do_not_wait_for_each_other(n, d):
    E = _eng()
    rng = np.random.default_rng(d)
    v = [rng.standard_normal((n, d)).astype(np.float32) for _ in range(3)]
    x0 = _cuda(rng.standard_normal(d).astype(np.float32))
    base = dict(n=n, d=d, gamma=0.05, x0=x0, worker_levels=[(E.TOPK, d // 50), (E.QUANT, 4), (E.QUANT_BLOCK, (5, 128)), (E.TOPK, d // 10)],
                master_levels=[(E.QUANT_BLOCK, (4, 256))], zeta_worker=0.3, zeta_master=0.0, seed=9)
    for diff in (False, True):
        runs = []
        for flags in (0, E.FLAG_NO_WAIT):
            kw = dict(base, flags=flags | E.FLAG_ANY_LEVEL_ORDER)
            kw.update(dict(grad_mode=E.DIFF_EXTERNAL, init_mode=E.INIT_ZERO) if diff else
                      dict(grad_mode=E.GRAD_EXTERNAL, grad0=_cuda(v[2]), init_mode=E.INIT_COMPRESSED))
            eng = E.AdaCGD(**kw)
            for t in range(4):
                S = (v[t % 2].astype(np.float64) ** 2).sum(axis=1)
                eng.step(_cuda(v[t % 2]), *([_cuda(S * 0.9 * 4.0 ** -np.arange(n))] if diff else []))
            runs.append([eng.state(f) for f in (E.F_X, E.F_GI, E.F_GTILDE, E.F_G, E.F_LEVEL, E.F_MSG_IDX, E.F_MSG_VAL, E.F_QCODES, E.F_QSCALE,
                                                E.F_LEVEL_HIST)])
            eng.close()
        for a, b in zip(*runs):
            np.testing.assert_array_equal(a, b)


def test_many_contexts_side_by_side():
    """Ten contexts on streams of their own, each with launches whose blocks meet: more blocks that wait than the device holds
    at once.  Same results as one after the other."""
    import torch
    E = _eng()
    n, d, count = 8, 200001, 10
    rng = np.random.default_rng(3)
    g = [_cuda(rng.standard_normal((n, d)).astype(np.float32)) for _ in range(3)]
    x0 = _cuda(np.zeros(d, np.float32))
    torch.cuda.synchronize()
    out = []
    for side_by_side in (False, True):
        engs = [E.AdaCGD(n=n, d=d, gamma=0.05, worker_levels=[(E.TOPK, 50 + i), (E.QUANT, 4), (E.TOPK, d // 9)], zeta_worker=0.3,
                         master_levels=[(E.TOPK, d // 30)], zeta_master=0.0, grad_mode=E.GRAD_EXTERNAL, grad0=g[2], x0=x0, seed=i,
                         stream=torch.cuda.Stream().cuda_stream, flags=E.FLAG_ANY_LEVEL_ORDER | E.FLAG_RETAIN_EXT) for i in range(count)]
        torch.cuda.synchronize()
        for group in ([engs] if side_by_side else [[e] for e in engs]):
            for t in range(4):
                for e in group:
                    e.step(g[t % 2])
            torch.cuda.synchronize()
        out.append([[e.state(f) for f in (E.F_X, E.F_GI, E.F_G, E.F_LEVEL, E.F_LEVEL_HIST)] for e in engs])
        for e in engs:
            e.close()
    for a, b in zip(*out):
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("n,d", [(64, 512), (65, 512), (64, 513), (1, 512), (12, 1024), (9, 16384), (5, 16001), (33, 3001)])
def test_aggregation_inside_and_outside_the_workers_launch(n, d):
    check_steps(n, d, "sparse", quant=False)


@pytest.mark.parametrize("n,d", [(1, 300001), (2, 262147)])
def test_quantisers_over_many_blocks(n, d):
    check_steps(n, d, "normal", quant=True)


@pytest.mark.parametrize("no_wait", [False, True])
@pytest.mark.parametrize("what", [["inf"], ["nan"], ["inf", "nan", "-nan"], ["zeros"]])
def test_infinities_and_nan_between_blocks_that_meet(what, no_wait):
    """What the blocks of a node leave for each other may be infinite, not a number or zero: results are those of the general
    kernels, bit for bit (NaN where they are NaN)."""
    E = _eng()
    n, d = 3, 20483
    rng = np.random.default_rng(len(what))
    v = [rng.standard_normal((n, d)).astype(np.float32) for _ in range(2)]
    for a in v:
        for w in what:
            if w == "zeros":
                a[:2] = 0.0
            else:
                a[0, rng.integers(0, d, 5)] = {"inf": np.inf, "nan": np.nan, "-nan": -np.float32(np.nan)}[w]
                a[1, 4095] = -np.inf if w == "inf" else np.nan
    out = []
    for flags in (E.FLAG_TWO_PASS, E.FLAG_NO_WAIT if no_wait else 0):
        eng = E.AdaCGD(n=n, d=d, gamma=0.05, worker_levels=[(E.TOPK, 3), (E.QUANT, 4), (E.QUANT_BLOCK, (4, 256)), (E.TOPK, 900), (E.TOPK, d)],
                       zeta_worker=1.0, master_levels=[(E.TOPK, 100)], zeta_master=0.0, grad_mode=E.DIFF_EXTERNAL, init_mode=E.INIT_ZERO,
                       x0=_cuda(np.zeros(d, np.float32)), seed=3, flags=flags | E.FLAG_ANY_LEVEL_ORDER)
        for a, D in zip(v, (1e-3, 1e9)):
            eng.step(_cuda(a), _cuda(np.full(n, D)))
            out.append([eng.state(f) for f in (E.F_LEVEL, E.F_SQNORM, E.F_ERR, E.F_MSG_COUNT, E.F_MSG_IDX, E.F_MSG_VAL, E.F_GI, E.F_GTILDE, E.F_G, E.F_X)])
        eng.close()
    for a, b in zip(out[:2], out[2:]):
        for f, (x, y) in enumerate(zip(a, b)):
            if x.dtype == np.float64:
                np.testing.assert_allclose(x, y, rtol=1e-12, err_msg=str(f))
            else:
                np.testing.assert_array_equal(x, y, err_msg=str(f))


def check_steps(n, d, kind, flags=0, quant=None):
    E = _eng()
    rng = np.random.default_rng(d)
    topk = sorted({1, max(1, d // 1000), max(1, d // 300), max(1, d // 50), max(1, d // 9), max(1, d // 2)})   # more than four sizes
    if d > 100000:
        topk = topk[1:4]
    levels = [(O.TOPK, k) for k in topk] + [(O.TOPK, d)]
    quant = n < 100 and d < 100000 if quant is None else quant
    if quant:
        levels += [(O.QUANT, 3), (O.QUANT, 5), (O.QUANT_BLOCK, (4, 512)), (O.QUANT_BLOCK, (2, 64))]
    levels = sorted(levels, key=lambda l: (O.level_alpha(l, d), l[0], str(l[1])))
    kw = dict(n=n, d=d, gamma=0.05, worker_levels=levels, zeta_worker=0.3, master_levels=[(O.TOPK, max(1, d // 20))],
              zeta_master=0.0, seed=77)
    grads = [make_vectors(rng, n, d, kind) for _ in range(3)]
    x0 = rng.standard_normal(d).astype(np.float32)
    orc = O.AdaCGDOracle(**kw)
    orc.init(x0, grads[0], O.INIT_FULLGRAD)
    eng = E.AdaCGD(grad_mode=E.GRAD_EXTERNAL, x0=_cuda(x0), grad0=_cuda(grads[0]), flags=flags, **kw)
    with until_near_tie(("node", n, d, kind)):
        for t in (1, 2):
            g = (grads[t - 1] + grads[t] * np.float32(0.3)).astype(np.float32)
            res, rm = orc.step(grads=g)
            eng.step(_cuda(g))
            compare_step(eng, orc, res, rm, ("node", n, d, kind, t))
    eng.close()


@pytest.mark.parametrize("n,d,logistic", [(3, 20000, False), (12, 65000, False), (2, 5003, True), (3, 65000, True)])
def test_captured_steps_replay(n, d, logistic):
    """Two captured steps (they lead back to the buffers they began with) replayed any number of times between eager
    ones: what the blocks of a launch meet at is cleared around a captured launch."""
    import torch
    E = _eng()
    rng = np.random.default_rng(d)
    st = torch.cuda.Stream()
    kw = dict(n=n, d=d, gamma=0.05, worker_levels=[(E.TOPK, d // 100), (E.TOPK, d // 10)], zeta_worker=0.3,
              master_levels=[(E.TOPK, d // 20)], zeta_master=0.0, seed=5, x0=_cuda(rng.standard_normal(d).astype(np.float32)))
    if logistic:
        rows = 9
        kw.update(grad_mode=E.GRAD_LOGISTIC, A=_cuda(rng.standard_normal((n * rows, d)).astype(np.float32)), lam=0.1,
                  labels=_cuda(np.where(rng.random(n * rows) < 0.5, 1.0, -1.0).astype(np.float32)),
                  shard_offsets=np.arange(n + 1, dtype=np.int64) * rows)
        args = [(), ()]
    else:
        g = [_cuda(rng.standard_normal((n, d)).astype(np.float32)) for _ in range(3)]
        kw.update(grad_mode=E.GRAD_EXTERNAL, grad0=g[2], flags=E.FLAG_RETAIN_EXT)
        args = [(g[0],), (g[1],)]
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        eng, ref = E.AdaCGD(**kw), E.AdaCGD(**kw)
        both = lambda e: [e.step(*a) for a in args]
        both(eng)
        both(ref)
        graph = torch.cuda.CUDAGraph()
        st.synchronize()
        with torch.cuda.graph(graph, stream=st):
            both(eng)
        for replays in (1, 2, 1):
            for _ in range(replays):
                graph.replay()
                both(ref)
            both(eng)
            both(ref)
            eng.step(*args[0])
            eng.step(*args[1])
            both(ref)
            st.synchronize()
            for f in (E.F_X, E.F_GI, E.F_GTILDE, E.F_G):
                np.testing.assert_array_equal(eng.state(f), ref.state(f), err_msg=str((replays, f)))
    eng.close()
    ref.close()


@pytest.mark.parametrize("n,d,logistic,master", [(3, 900, False, True), (3, 5003, True, True), (2, 20000, False, True), (70, 20000, False, True),
                                                 (3, 900, True, False), (2, 20000, True, False), (2, 1100000, False, True)])
def test_captured_steps_without_a_step_before_them_and_with_a_state_set_between_replays(n, d, logistic, master):
    """Two steps captured right after init, and a state written between two replays: the iterate that a launch writes ahead
    is there at the first step too, and follows what is set."""
    import torch
    E = _eng()
    rng = np.random.default_rng(d + master)
    st = torch.cuda.Stream()
    kw = dict(n=n, d=d, gamma=0.05, worker_levels=[(E.TOPK, d // 100), (E.TOPK, d // 10)], zeta_worker=0.3,
              master_levels=[(E.TOPK, d // 20)] if master else [], zeta_master=0.0, seed=5,
              x0=_cuda(rng.standard_normal(d).astype(np.float32)))
    if logistic:
        rows = 9
        kw.update(grad_mode=E.GRAD_LOGISTIC, A=_cuda(rng.standard_normal((n * rows, d)).astype(np.float32)), lam=0.1,
                  labels=_cuda(np.where(rng.random(n * rows) < 0.5, 1.0, -1.0).astype(np.float32)),
                  shard_offsets=np.arange(n + 1, dtype=np.int64) * rows)
        args = [(), ()]
    else:
        g = [_cuda(rng.standard_normal((n, d)).astype(np.float32)) for _ in range(3)]
        kw.update(grad_mode=E.GRAD_EXTERNAL, grad0=g[2])
        args = [(g[0],), (g[1],)]
    torch.cuda.synchronize()
    same = lambda what: [np.testing.assert_array_equal(eng.state(f), ref.state(f), err_msg=str((what, f)))
                         for f in (E.F_X, E.F_GI, E.F_GTILDE) + ((E.F_G,) if master else ())]
    with torch.cuda.stream(st):
        eng, ref = E.AdaCGD(**kw), E.AdaCGD(**kw)
        both = lambda e: [e.step(*a) for a in args]
        graph = torch.cuda.CUDAGraph()
        st.synchronize()
        with torch.cuda.graph(graph, stream=st):
            both(eng)
        for turn in range(3):
            graph.replay()
            both(ref)
            same(("replay", turn))
        for f in (E.F_X, E.F_G if master else E.F_GTILDE):
            v = rng.standard_normal(d).astype(np.float32)
            for e in (eng, ref):
                e.set_state(f, v)
            graph.replay()
            both(ref)
            same(("set", f))
            both(eng)
            both(ref)
            same(("eager", f))
    eng.close()
    ref.close()
