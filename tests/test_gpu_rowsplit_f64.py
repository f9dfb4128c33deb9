"""FP64 tile shapes of four waves at both sides of the rule that makes them row-split (enough
workgroups to fill the chip): passes and steps against the single-wave shape, single passes
against the oracle's flows, with ragged fibres, column counts around the column blocks, gathered and contiguous input,
and the increments of a sampler, which run the state's own tiles."""
import numpy as np
import pytest

from oracle import splitting
from paper_2103_14897_amd import lsx
from paper_2103_14897_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (system, W): row groups of four 16-row blocks times column blocks below and above 1024
CASES = [(wl.twisted_system(400.0), 20), (wl.twisted_system(900.0), 130), (wl.twisted_system(900.0), 99),
         (wl.chain_system(6.0e4, v1=1.0, v2=0.7), 130), (wl.chain_system(500.0, pot1={(1,): 0.4 + 0.3j, (-1,): 0.4 - 0.3j}), 33)]


@pytest.mark.parametrize("i", range(len(CASES)))
@pytest.mark.parametrize("nb", [1, 2])
def test_four_wave_shapes_match_the_oracle(i, nb):
    spec, W = CASES[i]
    print(f"[case] FP64 four-wave shapes: system {i} W={W} nb={nb}", flush=True)
    S = lsx.System.from_spec(spec)
    P = lsx.Plan(S, 2e-3, "strang", 0.5, "fp64")
    c = wl.random_state(S.N, W, seed=7 + i)
    out = {}
    try:
        for ks in (1, 4):
            st = lsx.State(P, W)
            try:
                for layer in (1, 2):
                    st.set_tuning(layer, nb, ks)
                    assert st.tuning(layer)[:2] == (nb, ks)
                st.upload(c)
                st.fibre_pass(1, 1, 1)
                first = st.download()
                st.step(3)
                out[ks] = (first, st.download())
            finally:
                st.destroy()
    finally:
        P.destroy()
        S.destroy()
    # the same products in another order: L <= 400 terms of unit roundoff, per pass
    for a, b in zip(out[1], out[4]):
        assert (np.linalg.norm(a - b, axis=0) <= 1e-13 * np.linalg.norm(a, axis=0)).all()
    if i in (0, 4):
        plan = splitting.SplitPlan(splitting.Lifted.from_spec(spec), 0.5)
        ref = plan.apply_fibres(c, 1, 1e-3)
        assert (np.linalg.norm(out[4][0] - ref, axis=0) <= 1e-12).all()


def test_sampler_increments_with_row_split_tiles():
    import torch

    spec, W = wl.twisted_system(900.0), 130
    S = lsx.System.from_spec(spec)
    P = lsx.Plan(S, 5e-3, "strang", 0.0, "fp64")
    c = wl.random_state(S.N, W, seed=3)
    got = []
    try:
        for ks in (1, 4):
            st = lsx.State(P, W)
            sm = None
            try:
                for layer in (1, 2):
                    st.set_tuning(layer, 1, ks)
                st.upload(c)
                sm = lsx.Sampler(st, 2, 2)
                b = torch.empty((W, S.nfibres[1]), dtype=torch.float64, device="cuda")
                sm.increments(1, 1, b)
                torch.cuda.synchronize()
                got.append(b.cpu().numpy())
            finally:
                if sm is not None:
                    sm.destroy()
                st.destroy()
    finally:
        P.destroy()
        S.destroy()
    assert np.allclose(got[0], got[1], rtol=1e-12, atol=1e-26)
