"""The compression step of short vectors (short.hip) at the edges of its range: block sizes, remainders, as many and more workers
than its launch aggregates, ties and zeros that leave its histogram, levels and triggers on both sides; against the oracle bit
for bit, and against the general kernels where values are infinite or not numbers."""
import numpy as np
import pytest

from oracle import adacgd_oracle as O
from test_gpu_parity import _cuda, _eng, compare_step, make_vectors, until_near_tie

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,kind", [(n, d, k) for n, d in [(1, 1), (2, 2), (3, 63), (2, 64), (4, 65), (5, 127), (2, 128), (3, 129), (2, 255),
                                                             (64, 256), (65, 257), (20, 300), (3, 511), (33, 512), (70, 512)]
                                      for k in ("normal", "ties", "const", "denormal", "sparse")])
@pytest.mark.parametrize("master", ["none", "one", "many", "quant"])
def test_short_vectors(n, d, kind, master):
    E = _eng()
    rng = np.random.default_rng(d * 100 + n)
    sizes = sorted({1, max(1, d // 50), max(1, d // 9), max(1, d // 3), max(1, d // 2), d})
    some = sorted({max(1, d // 20), max(1, d // 4), d})
    ml = {"none": [], "one": [(O.TOPK, max(1, d // 20))], "many": [(O.TOPK, k) for k in some], "quant": [(O.QUANT, 4)]}[master]
    kw = dict(n=n, d=d, gamma=0.05, worker_levels=[(O.TOPK, k) for k in sizes], zeta_worker=0.3, master_levels=ml,
              zeta_master=0.4 if master == "many" else 0.0, seed=77)
    grads = [make_vectors(rng, n, d, kind) for _ in range(3)]
    x0 = rng.standard_normal(d).astype(np.float32)
    orc = O.AdaCGDOracle(**kw)
    orc.init(x0, grads[0], O.INIT_FULLGRAD)
    eng = E.AdaCGD(grad_mode=E.GRAD_EXTERNAL, x0=_cuda(x0), grad0=_cuda(grads[0]), **kw)
    with until_near_tie(("short", n, d, kind, master)):
        for t in (1, 2, 3):
            g = (grads[t - 1] + grads[t % 3] * np.float32(0.3)).astype(np.float32)
            res, rm = orc.step(grads=g)
            eng.step(_cuda(g))
            compare_step(eng, orc, res, rm, ("short", n, d, kind, master, t), check_master=bool(ml))
    eng.close()


@pytest.mark.parametrize("mode", ["overlap", "compressed", "diff"])
@pytest.mark.parametrize("n,d", [(3, 100), (20, 300), (65, 512)])
@pytest.mark.parametrize("what", ["normal", "inf", "nan", "wide"])
def test_short_vectors_against_the_general_kernels(n, d, what, mode):
    """The same results as the general kernels give, bit for bit, also where the largest key is infinite or not a number, where keys
    lie further below it than the histogram reaches, and in the other modes of a context."""
    E = _eng()
    rng = np.random.default_rng(n + d)
    v = [rng.standard_normal((n, d)).astype(np.float32) for _ in range(3)]
    for a in v:
        if what == "wide":
            a *= np.float32(2.0) ** rng.integers(-120, 20, (n, d)).astype(np.float32)
        elif what != "normal":
            a[0, rng.integers(0, d, 3)] = np.float32(what)
    out = []
    for flags in (E.FLAG_TWO_PASS, 0):
        kw = dict(grad_mode=E.DIFF_EXTERNAL, init_mode=E.INIT_ZERO) if mode == "diff" else dict(grad_mode=E.GRAD_EXTERNAL, grad0=_cuda(v[2]))
        if mode == "compressed":
            kw.update(init_mode=E.INIT_COMPRESSED)
        flags |= E.FLAG_ANY_LEVEL_ORDER | (E.FLAG_OVERLAP if mode == "overlap" else 0)
        eng = E.AdaCGD(n=n, d=d, gamma=0.05, worker_levels=[(E.TOPK, d // 9), (E.TOPK, 3), (E.TOPK, d // 2)], zeta_worker=0.5,
                       master_levels=[(E.TOPK, d // 4)], zeta_master=0.0, x0=_cuda(np.zeros(d, np.float32)), seed=3, flags=flags, **kw)
        for t, D in enumerate((1e-3, 1e9, 1e-3)):
            eng.step(_cuda(v[t]), *([_cuda(np.full(n, D))] if mode == "diff" else []))
            out.append([eng.state(f) for f in (E.F_LEVEL, E.F_SQNORM, E.F_ERR, E.F_MSG_COUNT, E.F_MSG_IDX, E.F_MSG_VAL, E.F_GI, E.F_GTILDE,
                                               E.F_G, E.F_X, E.F_LEVEL_HIST, E.F_M_MSG_IDX)])
        eng.close()
    for a, b in zip(out[:3], out[3:]):
        for f, (x, y) in enumerate(zip(a, b)):
            if x.dtype == np.float64:
                np.testing.assert_allclose(x, y, rtol=1e-12, err_msg=str(f))
            else:
                np.testing.assert_array_equal(x, y, err_msg=str(f))


@pytest.mark.parametrize("d", [1, 2047, 2048, 2049, 8192, 20483, 70001])
@pytest.mark.parametrize("mode", ["gradients", "diff", "compressed"])
@pytest.mark.parametrize("levels", ["identity", "quantiser", "rank"])
def test_level_sets_whose_only_sparsifier_is_the_identity(d, mode, levels):
    """No size below d: the general kernels look for no candidates, and the identity's message is the difference itself.  Against the
    oracle's definition: every coordinate sent, in order."""
    E = _eng()
    n = 3
    if levels == "rank":
        d = max(256, d // 16 * 16)
    rng = np.random.default_rng(d)
    v = [make_vectors(rng, n, d, "normal") for _ in range(3)]
    first = {"identity": [], "quantiser": [(E.QUANT, 4)], "rank": [(E.RANK, (1, 16))]}[levels]
    kw = dict(grad_mode=E.DIFF_EXTERNAL, init_mode=E.INIT_ZERO) if mode == "diff" else dict(grad_mode=E.GRAD_EXTERNAL, grad0=_cuda(v[2]))
    if mode == "compressed":
        kw.update(init_mode=E.INIT_COMPRESSED)
    eng = E.AdaCGD(n=n, d=d, gamma=0.05, worker_levels=first + [(E.TOPK, d)], zeta_worker=0.0, master_levels=[(E.TOPK, d)], zeta_master=0.0,
                   x0=_cuda(np.zeros(d, np.float32)), seed=3, flags=E.FLAG_TWO_PASS | E.FLAG_ANY_LEVEL_ORDER, **kw)
    h = np.zeros((n, d), np.float32) if mode == "diff" else v[2].copy()
    gt = (h.astype(np.float64).sum(axis=0) / n).astype(np.float32)
    for t in range(2):
        eng.step(_cuda(v[t]), *([_cuda(np.ones(n))] if mode == "diff" else []))
        msg = v[t] if mode == "diff" else v[t] - h
        h = h + msg
        gt = (gt.astype(np.float64) + msg.astype(np.float64).sum(axis=0) / n).astype(np.float32)
        assert eng.state(E.F_LEVEL).tolist() == [len(first) + 1] * n
        np.testing.assert_array_equal(eng.state(E.F_GI), h)
        np.testing.assert_array_equal(eng.state(E.F_GTILDE), gt)
        for idx, val in eng.messages():
            np.testing.assert_array_equal(idx, np.arange(d))
        np.testing.assert_array_equal(eng.state(E.F_MSG_VAL).reshape(n, d), msg)
        assert (eng.state(E.F_ERR)[:, -1] == 0).all()
    eng.close()


@pytest.mark.parametrize("d", [700, 2049, 20483, 70001])
@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("sizes", [True, False])
def test_the_identity_next_to_sizes_and_a_quantiser(d, general, sizes):
    """Level sets with the identity, a quantiser and (or not) sizes below d; every worker's difference is steered by its ||x - y||^2
    to another level, or to none, at every step."""
    E = _eng()
    wl = ([(O.TOPK, max(1, d // 50)), (O.TOPK, d // 4)] if sizes else []) + [(O.QUANT, 8), (O.TOPK, d)]
    m = len(wl)
    n = m + 1
    rng = np.random.default_rng(d + general)
    # (errors and squared norms lie within [1e-3 d, 10 d])
    tw = [(10.0 ** (-4 * (m - 1 - j)), 0.0) for j in range(m)]
    kw = dict(n=n, d=d, gamma=0.05, worker_levels=wl, zeta_worker=0.0, worker_triggers=tw, master_levels=[(O.TOPK, max(1, d // 30)), (O.TOPK, d)],
              zeta_master=0.0, master_triggers=[(0.0, 0.0), (0.0, 0.5)], seed=11)
    x0 = rng.standard_normal(d).astype(np.float32)
    orc = O.AdaCGDOracle(**kw)
    orc.init(x0, None, O.INIT_ZERO)
    eng = E.AdaCGD(grad_mode=E.DIFF_EXTERNAL, init_mode=E.INIT_ZERO, x0=_cuda(x0),
                   flags=E.FLAG_ANY_LEVEL_ORDER | (E.FLAG_TWO_PASS if general else 0), **kw)
    with until_near_tie(("identity", d, general, sizes)):
        for t in range(2 * n):
            want = [(i * (1 + t // n) + t) % n for i in range(n)]        # level of each worker
            v = make_vectors(rng, n, d, "normal")
            D = np.array([0.0 if k == m else 10.0 * d * 10.0 ** (4 * (m - 1 - k)) for k in want])
            res, rm = orc.step(diffs=v, D=D)
            assert [r.level for r in res] == want
            eng.step(_cuda(v), _cuda(D))
            compare_step(eng, orc, res, rm, ("identity", d, general, sizes, t))
    eng.close()
