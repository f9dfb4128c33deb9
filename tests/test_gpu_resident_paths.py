"""Calls that run as one resident launch, told by the state array's address: a library-owned state swaps
its two arrays after an odd number of ordinary passes and keeps them in a resident call, which works
in place.  Each system's steps against the same sub-steps as separate calls (lsx_fibre_pass and
lsx_phase, ordinary launches): several sweeps of the workgroup over the rows (more than 256), bands
longer than the entries a lane loads together, BF16x3 bands of several chunks, and calls next to the
rules that are not resident."""
import numpy as np
import pytest

from paper_2103_14897_amd import lsx
from paper_2103_14897_amd import workloads as wl

pytestmark = pytest.mark.gpu

STRANG = [(1, 1, 1), (2, 0, 1), (1, 1, None)]
LIE = [(1, 0, 0), (2, 0, None)]
STRANG3 = [(1, 1, None), (2, 1, 1), (3, 0, 1), (2, 1, None), (1, 1, None)]
LIE3 = [(1, 0, None), (2, 0, 0), (3, 0, None)]


def blocks(*half):
    """Layers of one index each, |m_j| <= half[j] in any combination."""
    Rs = [np.array([[np.sqrt(2.0) / (h + 0.5)]]) for h in half]
    v = {(0,): 0.1, (1,): 0.6 + 0.2j, (-1,): 0.6 - 0.2j}
    nl = len(half)
    return lsx.System.blocks(Rs, [[j] for j in range(nl)], 1.0, [(j, j + 1) for j in range(nl)], [v] * nl)


def chain(Ec, v=1.0):
    return lsx.System.from_spec(wl.chain_system(Ec, v1=v, v2=0.7 * v))


# band_tol: None the default, < 0 dense products, 1e-4: above every off-diagonal entry (tau |v| = 2e-5),
# so that of a mixed path's blocks only the chunk of four columns at the diagonal is multiplied.
# start: the fewest of 1, 2 or 5 steps that are resident (a call of few passes is not where its entries
# are many), None: none is
@pytest.mark.parametrize("make,N,W,precision,band_tol,start", [
    (lambda: chain(150.0), 41, 1, "fp64", None, 1),                 # bodies of two passes in registers
    (lambda: chain(600.0), 155, 1, "fp64", None, 2),
    (lambda: chain(600.0), 155, 1, "mix_fp32", None, 2),
    (lambda: chain(600.0), 155, 300, "fp64", None, 5),              # two rounds of workgroups
    (lambda: chain(900.0), 229, 3, "fp64", None, 5),
    (lambda: chain(600.0), 155, 1100, "fp64", None, None),
    (lambda: chain(1000.0), 265, 1, "mix_fp32", None, None),        # more than 4096 entries
    (lambda: chain(1500.0), 389, 1, "fp64", None, None),
    (lambda: chain(1000.0, 0.01), 265, 1, "mix_fp32", 1e-4, 2),     # two sweeps, the second of 9 rows
    (lambda: chain(2000.0, 0.01), 513, 1, "mix_fp32", 1e-4, None),  # three
    (lambda: blocks(3, 3, 3), 343, 1, "fp64", None, 2),             # two sweeps, fibres of seven rows
    (lambda: blocks(3, 3, 3), 343, 1, "mix_fp32", None, 2),
    (lambda: blocks(3, 3, 3), 343, 3, "fp64", None, 2),
    (lambda: blocks(3, 3, 4), 441, 1, "mix_fp32", None, None),
    (lambda: blocks(20, 1), 123, 1, "mix_fp32", -1.0, 5),           # 44 and 16 columns: eleven k-steps
    (lambda: blocks(20, 0), 41, 2, "fp64", -1.0, 1),
    (lambda: blocks(16, 0), 33, 1, "mix_bf16x3", -1.0, 1),          # two chunks, the second of one column
    (lambda: blocks(20, 0), 41, 1, "mix_bf16x3", -1.0, 1),
    (lambda: blocks(20, 1), 123, 1, "mix_bf16x3", -1.0, None),
])
def test_resident_calls(make, N, W, precision, band_tol, start):
    S = make()
    print(f"[case] N={S.N} W={W} {precision} band_tol={band_tol} start={start}", flush=True)
    try:
        assert S.N == N
        strang, lie = (STRANG3, LIE3) if S.nlayers == 3 else (STRANG, LIE)
        for scheme, seq in (("strang", strang), ("lie", lie)):
            P = lsx.Plan(S, 2e-3, scheme, 0.6, precision, band_tol=band_tol)
            c = wl.random_state(S.N, W, seed=4)
            whole, parts = lsx.State(P, W), lsx.State(P, W)
            try:
                for n in (1, 2, 5):
                    for st in (whole, parts):
                        st.upload(c)
                    at = whole.device_ptr()
                    whole.step(n)
                    if scheme == "strang":  # 2 n + 1 passes, 4 n + 1 with three layers
                        assert (whole.device_ptr() == at) == (start is not None and n >= start)
                    for _ in range(n):
                        for layer, half, ph in seq:
                            parts.fibre_pass(layer, half)
                            if ph is not None:
                                parts.phase(ph)
                    a, b = whole.download(), parts.download()
                    err = (np.linalg.norm(a - b, axis=0) / np.linalg.norm(b, axis=0)).max()
                    # FP64 rounding of at most five passes a step over at most 51 terms; a mixed path's merged
                    # half steps are stored apart from the half steps, tau |V| 2^-24 a pass; entries left out
                    # of the bands are left out of the whole and of the half steps by the same blocks, and
                    # what two half steps lack against a whole one is of second order, (tau |v|)^2
                    tol = (1e-14 if precision == "fp64" else 2e-9) * 5 * n + ((2e-5) ** 2 * 5 * n if band_tol == 1e-4 else 0)
                    assert err < tol, (scheme, n, err)
            finally:
                whole.destroy()
                parts.destroy()
                P.destroy()
    finally:
        S.destroy()
