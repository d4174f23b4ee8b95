"""The convolution's forms by launch size: 8, 16 or 64 lanes of a wave per
row, two to eight waves.  On both sides of each choice, over channel counts
ragged against every chunk width, node counts round the waves' row groups, all
kernel sizes and both activation types, fused with a pending path: the
first sequences against the fp64 oracle, the conv state exactly, and the
same sequences alone (the narrow form) bit for bit against the whole batch
(every channel's arithmetic is the same in all forms)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_16673_amd import binding as B
from paper_2607_16673_amd import inputs

from test_conv_gpu import check_outputs, random_draft, run_verify, to_np

pytestmark = pytest.mark.gpu

# batch, channels, nodes: batch x ceil(channels / 512) on each side of 32 and 256; narrow chunks on each
# side of one and three workgroups per CU above 32 nodes; whole chunks on each side of three
CASES = [(31, 504, 2), (32, 504, 3), (16, 1032, 33), (8, 2056, 64), (128, 1016, 5), (129, 520, 9), (257, 136, 8),
         (128, 1024, 17), (86, 1544, 16), (300, 8, 64),
         (40, 1032, 33), (85, 1032, 40), (300, 520, 6), (800, 16, 7)]


@pytest.mark.parametrize("i", range(len(CASES)), ids=["B%d_D%d_n%d" % c for c in CASES])
@pytest.mark.parametrize("dtype", [inputs.BF16, inputs.F32])
def test_conv_forms_agree(i, dtype):
    Bn, D, n = CASES[i]
    K = 1 + (i + (dtype == inputs.F32)) % 4
    r = np.random.default_rng(700 + i)
    prev, cur = random_draft(r, Bn, 5, D, dtype), random_draft(r, Bn, n, D, dtype)
    w = r.uniform(-0.5, 0.5, (D, K)).astype(np.float32)
    bias = r.standard_normal(D).astype(np.float32) if i % 2 else None
    C = inputs._to_dtype(r.standard_normal((Bn, K - 1, D)), dtype)[1].astype(np.float32)
    wg, bg = torch.from_numpy(w).cuda(), torch.from_numpy(bias).cuda() if bias is not None else None
    Cg = torch.from_numpy(C).cuda() if K > 1 else None
    st = torch.full((Bn,), 99, dtype=torch.int32, device="cuda")
    y = run_verify(Cg, cur, wg, bg, True, pending=(prev.x, prev.parent, prev.path, prev.length), status=st)
    torch.cuda.synchronize()
    assert int(st.abs().max()) == 0
    m = min(Bn, 3)
    C1, _ = oracle.conv_commit(C[:m] if K > 1 else np.zeros((m, 0, D)), prev.x32[:m], prev.parent_np[:m],
                               prev.path_np[:m], prev.length_np[:m])
    if K > 1:
        np.testing.assert_array_equal(Cg[:m].cpu().numpy().astype(np.float64), C1)
    ref, _ = oracle.conv_verify(C1, cur.x32[:m], w, bias, cur.parent_np[:m])
    check_outputs(to_np(y[:m]), ref, dtype)
    for b in (0, Bn // 2, Bn - 1):  # one sequence alone
        s = slice(b, b + 1)
        Cb = torch.from_numpy(C[s]).cuda() if K > 1 else None
        yb = torch.empty_like(y[s])
        B.sla_conv_verify(Cb, cur.x[s].contiguous(), wg, cur.parent[s].contiguous(), yb, bias=bg,
                          pending=(prev.x[s].contiguous(), prev.parent[s].contiguous(), prev.path[s].contiguous(),
                                   prev.length[s].contiguous()))
        assert torch.equal(yb, y[s])
        if K > 1:
            assert torch.equal(Cb, Cg[s])
