"""The tile kernel's block inverse, long accepted paths and launch regimes.

Chains, trees and forests whose root paths cross the 16-row blocks (the
diagonal blocks of T are inverted, the rest is substituted) and accepted
paths of 7 to 64 steps (staged eight at a time), at batch sizes on both
sides of a full round of workgroups and of the many-round regime, with one
and two V-tiles per workgroup.  The committed state equals the standalone
commit bit for bit, outputs and records agree with the fp64 oracle, and a
sequence alone gives the bits it gives in the batch (its arithmetic does not
depend on the regime)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_16673_amd import binding as B
from paper_2607_16673_amd import inputs

from gpu_util import TOL, act_tensor, rel_err

pytestmark = pytest.mark.gpu

# batch, heads, d_k, d_v, pending nodes, nodes, family, dtype
CASES = [(1, 2, 128, 128, 64, 48, "gdn", inputs.BF16), (2, 2, 64, 80, 9, 17, "deltanet", inputs.F32),
         (3, 1, 256, 48, 33, 32, "gdn", inputs.BF16), (1, 3, 128, 256, 17, 64, "gdn", inputs.BF16),
         (2, 1, 128, 64, 40, 33, "gla", inputs.BF16), (130, 8, 128, 128, 12, 16, "gdn", inputs.BF16),
         (70, 16, 128, 128, 24, 31, "gdn", inputs.BF16), (300, 16, 64, 64, 16, 15, "decay", inputs.F32),
         (66, 16, 128, 144, 10, 23, "gla", inputs.F32), (140, 16, 128, 256, 20, 40, "gdn", inputs.BF16),
         # fp32 with per-key gates, the state read behind the first barrier: d_k 256, and 32 node rows
         (24, 8, 256, 128, 12, 16, "gla", inputs.F32), (12, 6, 128, 96, 9, 23, "gla", inputs.F32),
         (30, 8, 64, 320, 20, 32, "gla", inputs.F32),
         # tiles of 48 columns: scalar gates (not at d_k 256 above 32 nodes), per-key gates above three or four tiles per CU
         (3, 2, 256, 80, 9, 24, "gdn", inputs.F32), (2, 2, 256, 80, 9, 40, "gdn", inputs.BF16),
         (129, 8, 64, 48, 10, 30, "gla", inputs.F32), (49, 8, 256, 96, 10, 15, "gla", inputs.BF16),
         (43, 8, 128, 144, 12, 17, "gla", inputs.BF16), (42, 8, 128, 144, 12, 17, "gla", inputs.BF16),
         (129, 8, 128, 16, 10, 9, "gla", inputs.F32),
         # pairs of 64-column tiles where one stage fills a CU and d_v holds no whole 128-column tile
         (18, 8, 128, 80, 20, 48, "gla", inputs.BF16), (17, 8, 128, 96, 12, 40, "gdn", inputs.F32),
         (17, 8, 256, 112, 20, 24, "gla", inputs.F32), (17, 8, 256, 80, 20, 48, "gdn", inputs.BF16),
         # eight column waves, just above one or two tiles per CU: one tile of 128 columns, pairs of them; with
         # per-key gates; in less than a round of workgroups
         (17, 8, 256, 128, 20, 48, "gdn", inputs.BF16), (17, 8, 128, 128, 20, 40, "gdn", inputs.F32),
         (9, 8, 256, 384, 20, 24, "gla", inputs.F32), (9, 8, 128, 384, 9, 33, "gla", inputs.F32),
         (9, 8, 256, 256, 20, 48, "gdn", inputs.BF16), (9, 8, 256, 256, 20, 24, "gdn", inputs.F32),
         (9, 8, 256, 256, 20, 24, "gla", inputs.BF16), (9, 8, 128, 256, 20, 40, "gla", inputs.BF16),
         (20, 8, 128, 256, 20, 40, "gdn", inputs.BF16), (17, 8, 64, 256, 20, 40, "deltanet", inputs.F32),
         (17, 8, 64, 256, 20, 33, "gla", inputs.BF16),
         # pairs of 64-column tiles, 33 to 64 nodes, two stages per CU
         (33, 8, 128, 128, 20, 40, "gdn", inputs.BF16), (33, 8, 64, 80, 20, 48, "decay", inputs.F32)]


def _parents(r, Bn, n):
    rows = []
    for b in range(Bn):
        if b % 3 == 0:
            rows.append(inputs.chain(n))
        elif b % 3 == 1:
            rows.append(np.array([int(r.integers(max(-1, j - 3), j)) if j else -1 for j in range(n)], np.int32))
        else:
            rows.append(inputs.random_tree(r, n, 7, 4))
    return np.stack(rows).astype(np.int32)


@pytest.mark.parametrize("i", range(len(CASES)), ids=["B%d_H%d_dk%d_dv%d_n%d-%d_%s_%s" % c for c in CASES])
def test_deep_paths_and_regimes(i):
    Bn, H, dk, dv, n0, n1, fam, dt = CASES[i]
    r = np.random.default_rng(40 + i)
    c0 = inputs.Config("tf0", 700 + i, Bn, H, dk, dv, n0, False, n0, 64, dt, 1)
    c1 = inputs.Config("tf1", 720 + i, Bn, H, dk, dv, n1, False, n1, 64, dt, 1)
    rnds = []
    for c in (c0, c1):
        rd = inputs.Round(parent=_parents(r, Bn, c.n_nodes), path=None, length=None)
        d = inputs.draw_layer(c, 0, 0)
        for key in ("q", "k", "v", "q32", "k32", "v32", "alpha", "beta"):
            getattr(rd, key).append(d[key])
        rnds.append((rd, *inputs.family_gates(c, rd, 0, fam, layer=0)))
    path, ln = np.full((Bn, n0), -1, np.int32), np.zeros(Bn, np.int32)
    for b in range(Bn):
        p = inputs.walk_to_root(rnds[0][0].parent[b], n0 - 1 if b % 2 == 0 else int(r.integers(0, n0)))
        path[b, :len(p)], ln[b] = p, len(p)
    S0 = inputs.draw_state(c0, 0)
    dev = lambda x: None if x is None else torch.from_numpy(np.ascontiguousarray(x)).cuda()
    tdt = torch.bfloat16 if dt == inputs.BF16 else torch.float32

    def verify(state, k, f, out, pend=None, st=None, s=slice(None)):
        rd, al, be = rnds[k]
        part = lambda x: None if x is None else x[s]
        B.sla_verify(state, act_tensor(rd.q[0][s], dt), act_tensor(rd.k[0][s], dt), act_tensor(rd.v[0][s], dt),
                     dev(part(al)), dev(part(be)), dev(rd.parent[s]), out, f, pending=pend, status=st, family=fam)

    def fac(n, m=Bn):
        return B.Factors.empty(m, n, H, dk, dv, tdt, family=fam)

    f0, f1, g1 = fac(n0), fac(n1), fac(n1)
    out0, out1, o1 = (torch.empty(Bn, n, H, dv, device="cuda") for n in (n0, n1, n1))
    fused, sep = dev(S0), dev(S0)
    verify(fused, 0, f0, out0)
    st = torch.full((Bn,), 99, dtype=torch.int32, device="cuda")
    pend = (f0, dev(path), dev(ln))
    verify(fused, 1, f1, out1, pend=pend, st=st)
    B.sla_commit(sep, f0, pend[1], pend[2], family=fam)
    verify(sep, 1, g1, o1)
    torch.cuda.synchronize()
    assert int(st.abs().max()) == 0
    assert torch.equal(fused, sep) and torch.equal(out1, o1) and torch.equal(f1.u, g1.u)
    for b in sorted({0, Bn // 2, Bn - 1}):
        s, h = slice(b, b + 1), b % H
        cut = lambda x: None if x is None else x[s, :, h:h + 1]
        (r0, a0, b0), (r1, a1, b1) = rnds
        S1, s1 = oracle.commit(S0[s, h:h + 1], cut(r0.k32[0]), cut(r0.v32[0]), cut(a0), cut(b0), r0.parent[s], path[s],
                               ln[s], family=fam)
        ref, s2 = oracle.verify(S1, cut(r1.q32[0]), cut(r1.k32[0]), cut(r1.v32[0]), cut(a1), cut(b1), r1.parent[s],
                                family=fam)
        assert s1[0] == 0 and s2[0] == 0
        assert rel_err(fused[b, h].cpu().numpy(), S1[0, 0]) <= TOL[dt]
        assert rel_err(out1[b, :, h].cpu().numpy(), ref[0, :, 0]) <= TOL[dt]
        # the sequence alone
        fb = B.Factors(f0.k[s].contiguous(), f0.u[s].contiguous(), f0.alpha[s].contiguous(), f0.parent[s].contiguous())
        alone, ob, gb = dev(S0[s]), torch.empty(1, n1, H, dv, device="cuda"), fac(n1, 1)
        verify(alone, 1, gb, ob, pend=(fb, dev(path[s]), dev(ln[s])), s=s)
        assert torch.equal(alone, fused[s]) and torch.equal(ob, out1[s]) and torch.equal(gb.u, f1.u[s])


@pytest.mark.parametrize("dk,n", [(64, 64), (128, 48), (256, 32)])
def test_fp32_corrected_values_hold_fp32(dk, n):
    """Corrected values of long fp32 chains against the step's definition in
    fp64: R = beta (v - gamma P) and the sum of R with its corrections (far
    smaller than R) round once each, at most 2^-24 of the value, so the
    2-norm stays within 2 x 2^-24 (summed product by product on top of R it
    was 1.1e-7 to 1.5e-7)."""
    Bn, H, dv = 3, 2, 64
    cfg = inputs.Config("tp", 790 + n, Bn, H, dk, dv, n, True, n, 1, inputs.F32, 1)
    rd = inputs.draw_round(cfg, 0, layers=[0])
    S0 = inputs.draw_state(cfg, 0)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    f = B.Factors.empty(Bn, n, H, dk, dv, torch.float32)
    B.sla_verify(dev(S0), *(act_tensor(x[0], inputs.F32) for x in (rd.q, rd.k, rd.v)), dev(rd.alpha[0]), dev(rd.beta[0]),
                 dev(rd.parent), torch.empty(Bn, n, H, dv, device="cuda"), f, topology="chain")
    S = torch.from_numpy(S0).double()  # [B][H][dk][dv]
    k, v, al, be = (torch.from_numpy(np.ascontiguousarray(x[0])).double() for x in (rd.k32, rd.v32, rd.alpha, rd.beta))
    want = torch.empty(Bn, n, H, dv, dtype=torch.float64)
    for j in range(n):
        S = S * al[:, j, :, None, None]
        want[:, j] = be[:, j, :, None] * (v[:, j] - (S * k[:, j, :, :, None]).sum(2))
        S = S + k[:, j, :, :, None] * want[:, j, :, None, :]
    err = float((f.u.cpu().double() - want).norm() / want.norm())
    print("dk %d n %d: corrected values %.2e from fp64" % (dk, n, err), flush=True)
    assert err <= 2 * 2.0 ** -24
