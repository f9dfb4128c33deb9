"""Fibre propagators against the oracle at the edges of the kernels that form them: layers whose
longest matrix is just below and above the 64 rows from which short fibres go through the blocked
eigensolver, fibres of one row up, beside multiples of 16 and 32, real and complex (embedded)
Hamiltonians, and the three stored formats.

Tolerances: FP64 as in the eigensolver's own test, 1e-13 up to t ||H|| = 10 and growing with it; the
mixed formats round the real and imaginary part of an off-diagonal entry of modulus below one to
2^-24, with the FP64 bar on the diagonal.
"""
import numpy as np
import pytest

from oracle import splitting
from paper_2103_14897_amd import lsx
from paper_2103_14897_amd import workloads as wl

pytestmark = pytest.mark.gpu

ASYM = {(1,): 0.6 + 0.45j, (-1,): 0.6 - 0.45j, (2,): 0.2 - 0.1j, (-2,): 0.2 + 0.1j}


@pytest.mark.parametrize("Ec,complex_pot,precision", [
    (6.6e3, False, "fp64"),      # longest 59 rows: scalar solver
    (8.0e3, False, "fp64"),      # longest 65: those above 32 rows blocked
    (8.0e3, False, "mix_fp32"),
    (8.0e3, False, "mix_bf16x3"),
    (1.5e3, True, "fp64"),       # embedded sizes up to 34 and 58: scalar
    (2.4e3, True, "mix_fp32"),   # up to 46 and 70: one layer of each kind
    (2.4e3, True, "mix_bf16x3"),
])
def test_propagators_at_the_edges(Ec, complex_pot, precision):
    spec = wl.chain_system(Ec, pot1=ASYM, pot2=ASYM) if complex_pot else wl.chain_system(Ec)
    tau = 1e-3
    S = lsx.System.from_spec(spec)
    O = splitting.Lifted.from_spec(spec)
    P = lsx.Plan(S, tau, "strang", 0.0, precision)
    try:
        plan = splitting.SplitPlan(O, 0.0)
        for layer in (1, 2):
            L = np.diff(S.fibres(layer)[0])
            print(f"[case] Ec={Ec} complex={complex_pot} {precision} layer {layer}: rows {L.min()} to {L.max()}", flush=True)
            ref = plan.propagators(layer, tau)
            for f in range(S.nfibres[layer]):
                H = O.fibre_hamiltonian(layer, O.fib[layer][f][1], 0.0)
                tol = 1e-13 * max(1.0, tau * np.abs(np.linalg.eigvalsh(H)).max() / 10.0)
                d = np.abs(P.propagator(layer, 0, f) - ref[f])
                assert np.diag(d).max() < tol, (layer, f, L[f])
                off = d - np.diag(np.diag(d))
                assert off.max() < tol + (0.0 if precision == "fp64" else 2.0 ** -24 * np.sqrt(2.0)), (layer, f, L[f])
    finally:
        P.destroy()
        S.destroy()
