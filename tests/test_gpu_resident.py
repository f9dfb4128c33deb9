"""Resident steps (small systems, every pass of a call in one launch): lsx_step against the same
sub-steps as separate calls of lsx_fibre_pass and lsx_phase, which launch the ordinary pass kernels.
Sizes around the rules (rows per workgroup sweep, entries a lane loads together, the two-pass body in
registers), every storage format, two and three layers, bodies of one to six passes, and a call
longer than one launch's span of passes."""
import numpy as np
import pytest

from paper_2103_14897_amd import lsx
from paper_2103_14897_amd import workloads as wl

pytestmark = pytest.mark.gpu

G1 = {"strang": [(1, 1, 1), (2, 0, 1), (1, 1, None)], "lie": [(1, 0, 0), (2, 0, None)], "lie_be": [(1, 0, 0), (2, 0, None)],
      "strang_cn": [(1, 1, 1), (2, 0, 1), (1, 1, None)],
      "yoshida4": [(1, 1, 0), (2, 0, 0), (1, 2, 1), (2, 2, 1), (1, 2, 0), (2, 0, 0), (1, 1, None)]}
G1_3 = {"strang": [(1, 1, None), (2, 1, 1), (3, 0, 1), (2, 1, None), (1, 1, None)], "lie": [(1, 0, None), (2, 0, 0), (3, 0, None)]}


def _relerr(a, b):
    return (np.linalg.norm(a - b, axis=0) / np.linalg.norm(b, axis=0)).max()


def _compare(S, scheme, kappa, precision, W, nsteps, seqs, seed=1):
    P = lsx.Plan(S, 2e-3, scheme, kappa, precision)
    c = wl.random_state(S.N, W, seed=seed)
    out = []
    try:
        for whole in (True, False):
            st = lsx.State(P, W)
            try:
                st.upload(c)
                if whole:
                    st.step(nsteps)
                else:
                    for _ in range(nsteps):
                        for layer, half, ph in seqs[scheme]:
                            st.fibre_pass(layer, half)
                            if ph is not None:
                                st.phase(ph)
                out.append(st.download())
            finally:
                st.destroy()
    finally:
        P.destroy()
    # FP64 rounding of at most 7 passes a step over fibres of at most 40 rows (the merged half steps
    # round apart too); the mixed formats' stored entries are the ones both multiply, but a merged
    # step's are not the half steps' product: their FP32 rounding, tau |V| 2^-24 per pass
    tol = (1e-14 if precision == "fp64" else 2e-9) * 7 * nsteps
    assert _relerr(out[0], out[1]) < tol


# N = 29, 53 (one sweep), 155, 247 (the pair rule's row limit), 389 and 775 (two and four sweeps)
@pytest.mark.parametrize("Ec", [100.0, 200.0, 600.0, 960.0, 1500.0, 3000.0])
@pytest.mark.parametrize("precision", ["fp64", "mix_fp32", "mix_bf16x3"])
def test_single_states_of_every_format(Ec, precision):
    S = lsx.System.from_spec(wl.chain_system(Ec))
    try:
        for scheme, kappa in (("strang", 0.0), ("strang", 0.6), ("lie", 0.3)):
            print(f"[case] resident chain N={S.N} {precision} {scheme} kappa={kappa}", flush=True)
            for nsteps in (1, 2, 5):
                _compare(S, scheme, kappa, precision, 1, nsteps, G1)
    finally:
        S.destroy()


@pytest.mark.parametrize("scheme", ["lie", "lie_be", "strang", "strang_cn", "yoshida4"])
@pytest.mark.parametrize("W", [2, 17, 300])
def test_columns_and_schemes(scheme, W):
    spec = wl.chain_system(300.0, pot1={(0,): 0.2, (1,): 0.5 + 0.2j, (-1,): 0.5 - 0.2j})
    S = lsx.System.from_spec(spec)
    try:
        print(f"[case] resident columns N={S.N} W={W} {scheme}", flush=True)
        for nsteps in (1, 2, 3, 4):
            _compare(S, scheme, 0.4, "fp64", W, nsteps, G1)
    finally:
        S.destroy()


def test_three_layers_and_wide_bands():
    for S in (lsx.System.layers(1, wl.chain_layers(60.0).As, 60.0, "ball", wl.chain_layers(60.0).pots),
              lsx.System.from_spec(wl.twisted_system(120.0))):
        try:
            for scheme in ("strang", "lie"):
                print(f"[case] resident layers={S.nlayers} N={S.N} {scheme}", flush=True)
                for nsteps in (1, 2, 5):
                    _compare(S, scheme, 0.5, "fp64", 3, nsteps, G1_3 if S.nlayers == 3 else G1)
        finally:
            S.destroy()


@pytest.mark.parametrize("Ec,precision", [(200.0, "fp64"), (200.0, "mix_bf16x3"), (500.0, "fp64")])
def test_calls_longer_than_one_launch(Ec, precision):
    """9000 steps (18001 passes, more than one launch's 16384) equal the same steps in two calls."""
    S = lsx.System.from_spec(wl.chain_system(Ec))
    P = lsx.Plan(S, 1e-3, "strang", 0.5, precision)
    try:
        print(f"[case] resident long call N={S.N} {precision}", flush=True)
        c = wl.random_state(S.N, 1, seed=2)
        out = []
        for parts in ((9000,), (8191, 809)):
            st = lsx.State(P, 1)
            try:
                st.upload(c)
                for n in parts:
                    st.step(n)
                out.append(st.download())
            finally:
                st.destroy()
        # one more F1(tau/2) F1(tau/2) pair instead of F1(tau); 18001 passes of FP64 rounding
        assert _relerr(out[0], out[1]) < (1e-11 if precision == "fp64" else 1e-8)
    finally:
        P.destroy()
        S.destroy()
