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
    E = _eng()
    rng = np.random.default_rng(d)
    topk = sorted({1, max(1, d // 1000), max(1, d // 300), max(1, d // 50), max(1, d // 9), max(1, d // 2)})   # more than four sizes
    if d > 100000:
        topk = topk[1:4]
    levels = [(O.TOPK, k) for k in topk] + [(O.TOPK, d)]
    quant = n < 100 and d < 100000
    if quant:
        levels += [(O.QUANT, 3), (O.QUANT, 5), (O.QUANT_BLOCK, (4, 512)), (O.QUANT_BLOCK, (2, 64))]
    levels = sorted(levels, key=lambda l: (O.level_alpha(l, d), l[0], str(l[1])))
    kw = dict(n=n, d=d, gamma=0.05, worker_levels=levels, zeta_worker=0.3, master_levels=[(O.TOPK, max(1, d // 20))],
              zeta_master=0.0, seed=77)
    grads = [make_vectors(rng, n, d, kind) for _ in range(3)]
    x0 = rng.standard_normal(d).astype(np.float32)
    orc = O.AdaCGDOracle(**kw)
    orc.init(x0, grads[0], O.INIT_FULLGRAD)
    eng = E.AdaCGD(grad_mode=E.GRAD_EXTERNAL, x0=_cuda(x0), grad0=_cuda(grads[0]), **kw)
    with until_near_tie(("node", n, d, kind)):
        for t in (1, 2):
            g = (grads[t - 1] + grads[t] * np.float32(0.3)).astype(np.float32)
            res, rm = orc.step(grads=g)
            eng.step(_cuda(g))
            compare_step(eng, orc, res, rm, ("node", n, d, kind, t))
    eng.close()
