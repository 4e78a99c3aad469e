"""The repair of operand errors by several workgroups of an item (256 rows and columns each) against the oracle: a footprint that
crosses every slice, the symbols where the row of one error meets the column of another, several errors in one line."""
import numpy as np
import pytest

from paper_2508_04355_amd import gecc, inputs
from paper_2508_04355_amd.inputs import MAT_A, MAT_B, MAT_C

pytestmark = pytest.mark.gpu


def _faults(pattern, n, k, m):
    i, j, l = n - 1, m - 1, k // 2
    F = inputs.Fault
    return {"A": [F(MAT_A, i, l, 17.0)],
            "B+C": [F(MAT_B, l, j, -9.5), F(MAT_C, n // 2, m // 3, 55.0)],
            "A+B, one term": [F(MAT_A, i, l, 4.0), F(MAT_B, l, j, 6.0)],
            "two of A in one row": [F(MAT_A, i, l, 4.0), F(MAT_A, i, l + 1, -3.0)],
            "two of B in one column": [F(MAT_B, l, j, 5.0), F(MAT_B, l - 1, j, 2.5)],
            "2 x 2 crossing": [F(MAT_A, 0, l, 4.0), F(MAT_A, i, l - 1, -7.0), F(MAT_B, l, 0, 3.0), F(MAT_B, l - 1, j, 6.0)],
            "A in a row, B twice across it": [F(MAT_A, i, l, 4.0), F(MAT_B, l, j, 6.0), F(MAT_B, l + 1, j, -2.0)],
            "two in one column of A": [F(MAT_A, 0, l, 4.0), F(MAT_A, i, l, 7.3)]}[pattern]


@pytest.mark.parametrize("trans", [(0, 0), (1, 1)])
@pytest.mark.parametrize("dtype,shape,batch", [("f32", (257, 64, 256), 1), ("bf16", (256, 96, 513), 2), ("f32", (1030, 72, 300), 3),
                                               ("bf16", (64, 70, 1300), 1), ("f32", (257, 65, 260), 260),    # (one workgroup an item)
                                               ("f32", (2305, 24, 100), 130)])  # (three, where shorter lines would have one)
@pytest.mark.parametrize("pattern", ["A", "B+C", "A+B, one term", "two of A in one row", "two of B in one column", "2 x 2 crossing",
                                     "A in a row, B twice across it", "two in one column of A"])
def test_operand_errors_repaired_by_several_workgroups(pattern, dtype, shape, batch, trans):
    import gpu_harness as H
    n, k, m = shape
    rng = inputs.rng_for(98, n + m)
    law = ("normal", 1.0)
    faults = _faults(pattern, n, k, m)
    hit = batch - 1                                    # the last item has the errors
    A, B = [np.stack(x) for x in zip(*[inputs.operands(rng, n, k, m, law, law, dtype) for _ in range(batch)])]
    A2, B2 = A.copy(), B.copy()
    A2[hit], B2[hit], cf, eff = inputs.apply_operand_faults(A[hit], B[hit], faults, dtype)
    cfb = [(hit,) + c for c in cf]
    tau = gecc.noise_thresholds(n, k, m, 1.0, 1.0)
    g = H.run_gpu(A, B, A2, B2, cfb, tau, dtype, trans[0], trans[1])
    o = H.run_oracle(A[hit], B[hit], A2[hit], B2[hit], [(0,) + c for c in cf], tau)
    assert all(r.status == gecc.CLEAN for r in g.reports[:hit])
    last = H.GpuResult(reports=g.reports[hit:], C=g.C[hit:], A=g.A[hit:], B=g.B[hit:], A_par=g.A_par[hit:], B_par=g.B_par[hit:],
                       C_par=g.C_par[hit:], synd=g.synd)
    H.compare(last, o, 1e-5, what="%s, %s" % (pattern, shape))
    if pattern == "two in one column of A":
        assert o[0].status == gecc.UNCORRECTABLE
    else:
        assert o[0].status == gecc.CORRECTED
        assert [(e[0], e[1], e[2]) for e in last.reports[0].errors()] == [(e[0], e[1], e[2]) for e in eff]
    if batch < 4:                                       # the order in which the workgroups come does not show
        g2 = H.run_gpu(A, B, A2, B2, cfb, tau, dtype, trans[0], trans[1])
        assert np.array_equal(g.C, g2.C) and np.array_equal(g.A, g2.A) and np.array_equal(g.C_par, g2.C_par)


@pytest.mark.parametrize("trans", [(0, 0), (1, 1)])
@pytest.mark.parametrize("dtype,shape,batch", [("f32", (129, 130, 131), 1), ("f32", (300, 385, 127), 2), ("bf16", (129, 260, 257), 1),
                                               ("bf16", (260, 7, 64), 3), ("f32", (128, 64, 128), 255), ("f32", (128, 64, 128), 256)])
def test_audits_by_column_scans_of_either_width(dtype, shape, batch, trans):
    """The audit's column scans in vectors of 8 bytes (fewer than 256 workgroups of 16-byte ones) and of 16: errors in the first and
    the last column come back exactly where they are, with an encoding that the 16-byte scans or others have made."""
    import gpu_harness as H
    n, k, m = shape
    rng = inputs.rng_for(99, n + k + m)
    law = ("normal", 1.0)
    faults = [inputs.Fault(MAT_A, n - 1, k - 1, 17.0), inputs.Fault(MAT_B, 0, m - 1, -9.5)]
    hit = batch - 1
    A, B = [np.stack(x) for x in zip(*[inputs.operands(rng, n, k, m, law, law, dtype) for _ in range(batch)])]
    A2, B2 = A.copy(), B.copy()
    A2[hit], B2[hit], cf, eff = inputs.apply_operand_faults(A[hit], B[hit], faults, dtype)
    tau = gecc.noise_thresholds(n, k, m, 1.0, 1.0)
    g = H.run_gpu(A, B, A2, B2, [(hit,) + c for c in cf], tau, dtype, trans[0], trans[1])
    o = H.run_oracle(A[hit], B[hit], A2[hit], B2[hit], [(0,) + c for c in cf], tau)
    last = H.GpuResult(reports=g.reports[hit:], C=g.C[hit:], A=g.A[hit:], B=g.B[hit:], A_par=g.A_par[hit:], B_par=g.B_par[hit:],
                       C_par=g.C_par[hit:], synd=g.synd)
    H.compare(last, o, 1e-5, what="%s %s x %d, trans %s" % (dtype, shape, batch, trans))
    assert o[0].status == gecc.CORRECTED and [(e[0], e[1], e[2]) for e in last.reports[0].errors()] == [(e[0], e[1], e[2]) for e in eff]
