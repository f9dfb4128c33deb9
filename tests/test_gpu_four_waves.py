"""Which FP64 kernel a four-wave tile shape runs, and that kernel against the oracle.

Rule: with at least 1024 workgroups (groups of four 16-row blocks of every fibre times column blocks)
the four waves take consecutive row blocks, else they split the fibre length.  In the row split one
wave sums a whole row in order, as the single-wave shape does, from operands formed alike, so the two
agree bit for bit; four partial sums added at the end do not."""
import numpy as np
import pytest

from oracle import splitting
from paper_2103_14897_amd import lsx
from paper_2103_14897_amd import workloads as wl

pytestmark = pytest.mark.gpu

COMPLEX = {(1,): 0.4 + 0.3j, (-1,): 0.4 - 0.3j}


def workgroups(S, layer, W, nb):
    return int(((S.fibre_info(layer)[1] + 63) // 64).sum()) * ((W + 16 * nb - 1) // (16 * nb))


# the oracle's columns: the first, the last and those around the column blocks' ends
@pytest.mark.parametrize("spec,W,nb,split", [
    (wl.twisted_system(900.0), 99, 1, True),         # 1232 workgroups, ragged last column block
    (wl.twisted_system(900.0), 81, 1, True),         # 1056, one column in the last block
    (wl.twisted_system(900.0), 80, 1, False),        # 880
    (wl.twisted_system(1000.0), 175, 2, True),       # 1206, last pair of blocks one column short
    (wl.twisted_system(1000.0), 177, 2, True),       # 1206, last pair with 17 columns
    (wl.chain_system(6.0e4, pot1=COMPLEX), 130, 2, True),  # 1620 and 1455, fibres of 1 to 179 rows
    (wl.chain_system(3.0e4, pot1=COMPLEX), 17, 2, False),
])
def test_row_split_runs_above_the_rule(spec, W, nb, split):
    S = lsx.System.from_spec(spec)
    P = lsx.Plan(S, 2e-3, "strang", 0.5, "fp64")
    c = wl.random_state(S.N, W, seed=11)
    print(f"[case] FP64 four waves N={S.N} W={W} nb={nb}", flush=True)
    got = {}
    try:
        for layer in (1, 2):
            assert (workgroups(S, layer, W, nb) >= 1024) == split
        for ks in (1, 4):
            st = lsx.State(P, W)
            try:
                for layer in (1, 2):
                    st.set_tuning(layer, nb, ks)
                for layer, half in ((1, 1), (2, 0)):
                    st.upload(c)
                    st.fibre_pass(layer, half)
                    got[ks, layer] = st.download()
            finally:
                st.destroy()
    finally:
        P.destroy()
        S.destroy()
    cols = sorted({0, 15, 16, W // 2, W - 2, W - 1} & set(range(W)))
    plan = splitting.SplitPlan(splitting.Lifted.from_spec(spec), 0.5)
    for layer, t in ((1, 1e-3), (2, 2e-3)):
        same = np.array_equal(got[1, layer].view(np.float64), got[4, layer].view(np.float64))
        assert same == split
        ref = plan.apply_fibres(c[:, cols], layer, t)
        # unit columns; eigenvectors and sums of up to 179 terms at 1e-16 each
        assert (np.linalg.norm(got[4, layer][:, cols] - ref, axis=0) <= 1e-12).all()
        assert (np.linalg.norm(got[4, layer] - got[1, layer], axis=0) <= 1e-13).all()
