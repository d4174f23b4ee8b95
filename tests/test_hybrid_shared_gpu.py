"""The hybrid route with several V-tiles of a unit on one staged draft (d_k =
256, a stage that fills a CU's LDS): bit for bit the serial route where that
holds the draft, over one, two and four tiles per workgroup, tile counts that
do not divide, chains, stars and trees, and the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_16673_amd import binding as B
from paper_2607_16673_amd import inputs

from gpu_util import TOL, rel_err
from test_hybrid_gpu import _dev, _problem, _two_rounds

pytestmark = pytest.mark.gpu

# batch, heads, d_v, nodes, dtype, family: 16-column tiles on each side of one per CU (no sharing
# up to there) and of two
CASES = [(4, 4, 256, 64, inputs.F32, "gdn"), (5, 4, 256, 64, inputs.F32, "deltanet"),
         (20, 4, 48, 33, inputs.F32, "decay"), (33, 4, 80, 40, inputs.F32, "gdn"), (40, 8, 32, 48, inputs.F32, "gdn"),
         (17, 2, 256, 48, inputs.BF16, "gla"), (40, 1, 208, 50, inputs.F32, "gla"), (16, 8, 112, 41, inputs.BF16, "gla"),
         # pairs of tiles: an odd tile count, per-key gates just above one tile per CU
         (30, 4, 48, 33, inputs.F32, "decay"), (10, 2, 256, 48, inputs.BF16, "gla"), (15, 1, 288, 50, inputs.F32, "gla")]


@pytest.mark.parametrize("i", range(len(CASES)), ids=["B%d_H%d_dv%d_n%d_%s_%s" % c for c in CASES])
def test_shared_stage_is_the_serial_route(i):
    Bn, H, dv, n, dt, fam = CASES[i]
    r = np.random.default_rng(90 + i)

    def parents():
        rows = [inputs.random_tree(r, n, 8, 4) for _ in range(Bn)]
        rows[0] = inputs.chain(n)
        rows[1] = np.array([-1] + [0] * (n - 1), np.int32)                      # a star: leaf children only
        rows[2] = np.array([-1 if j < 3 else int(r.integers(0, j)) for j in range(n)], np.int32)  # a forest
        return rows

    cfg, r0, a0, b0, S0 = _problem(60 + i, Bn, H, 256, dv, n, parents(), dt, fam)
    _, r1, a1, b1, _ = _problem(80 + i, Bn, H, 256, dv, n, parents(), dt, fam)
    s_hy, res_hy = _two_rounds(cfg, r0, a0, b0, r1, a1, b1, S0, fam, "hybrid")
    s_ser, res_ser = _two_rounds(cfg, r0, a0, b0, r1, a1, b1, S0, fam, "serial")
    assert torch.equal(s_ser, s_hy)
    for (o_s, f_s), (o_h, f_h) in zip(res_ser, res_hy):
        assert torch.equal(o_s, o_h)
        assert torch.equal(f_s.u, f_h.u) and torch.equal(f_s.k, f_h.k)
        assert torch.equal(f_s.alpha, f_h.alpha) and torch.equal(f_s.parent, f_h.parent)
    m = slice(0, 3)
    ref, st = oracle.verify(S0[m], r0.q32[0][m], r0.k32[0][m], r0.v32[0][m], None if a0 is None else a0[m],
                            None if b0 is None else b0[m], r0.parent[m], family=fam)
    assert (st == 0).all()
    assert rel_err(res_hy[0][0][m].cpu().numpy(), ref) <= TOL[dt]
