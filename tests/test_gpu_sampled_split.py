"""The FP32 sums of the mixed formats' sampled sub-steps of several wavepackets: with every fibre drawn
once by every wavepacket the weights are one and a sampled sub-step is the deterministic pass, so
lsx_ss_step equals lsx_step with the same tile shape (one column block, ks waves splitting the fibre
length, two groups of k-steps in flight) up to FP64 rounding.  A state whose pinned shape is a row
split takes two waves, and a state that timed its shapes the waves that the size of the pass gives.
Fibres of 7 to 61 rows: some waves without a k-step, and up to eight groups.  Layer 2 has no potential (its propagator is the identity at kappa = 1), so that the products of
layer 1 read the same state on both sides.

Tolerance: the two differ by the rounding of x + (P x - x), of the phase multiplied before or after it
is stored (2^-52 each, four operations) and of the weights, nf q p with |q nf - 1| <= 2^-51; 1e-13
bounds them by two orders.  Sums split otherwise differ by FP32 rounding, 2^-24 of the off-diagonal
part (tau |V| = 0.05 here): 1e-9.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2103_14897_amd import lsx  # noqa: E402
from paper_2103_14897_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu


def one_potential(spec):
    return lsx.System(spec.d, spec.A1, spec.A2, spec.Ec, spec.cutoff, spec.pot1, {})


@pytest.mark.parametrize("precision", ["mix_fp32", "mix_bf16x3"])
@pytest.mark.parametrize("which", ["chain", "twisted"])
@pytest.mark.parametrize("shape,ks", [((1, 1), 1), ((1, 2), 2), ((1, 4), 4), ((1, -2), 2), ((1, -4), 2)])
def test_sums_are_those_of_the_split_pass(which, shape, ks, precision):
    W = 19
    S = one_potential(wl.chain_system(4.0e3) if which == "chain" else wl.twisted_system(500.0))
    groups = 2 if precision == "mix_fp32" else 0
    print(f"[case] {which} N={S.N} nf={S.nfibres} shape={shape} {precision}", flush=True)
    P = lsx.Plan(S, 0.05, "lie", 1.0, precision)
    c = wl.random_state(S.N, W, seed=5)
    nf = S.nfibres
    sampled, whole = lsx.State(P, W), lsx.State(P, W)
    sm = lsx.Sampler(sampled, nf[1], nf[2], eps=0.1)
    try:
        for layer in (1, 2):
            sampled.set_tuning(layer, *shape, groups if shape[1] > 0 else 0)
            whole.set_tuning(layer, 1, ks, groups)
        u = np.zeros((1, 2, W, max(nf[1], nf[2])))
        for j in (1, 2):
            u[0, j - 1, :, :nf[j]] = (np.arange(nf[j]) + 0.5) / nf[j]
        for st in (sampled, whole):
            st.upload(c)
        sm.ss_step(torch.as_tensor(u).to("cuda:0"), 1)
        whole.step(1)
        a, b = sampled.download(), whole.download()
        err = (np.linalg.norm(a - b, axis=0) / np.linalg.norm(b, axis=0)).max()
        print(f"  rel diff {err:.2e}")
        assert err < 1e-13
    finally:
        sm.destroy()
        for o in (sampled, whole, P, S):
            o.destroy()


@pytest.mark.parametrize("Ec,W,precision,ks", [
    (500.0, 20, "mix_fp32", 4), (500.0, 20, "mix_bf16x3", 4), (1500.0, 20, "mix_fp32", 4), (1500.0, 40, "mix_fp32", 2),
    (1500.0, 40, "mix_bf16x3", 2), (2500.0, 96, "mix_fp32", 1), (1200.0, 64, "mix_fp32", 2),
    (4500.0, 40, "mix_fp32", 2)])
def test_tuned_states_repeat(Ec, W, precision, ks):
    """States that timed their own shapes, whatever they picked: the same split by the size of the pass
    (344 to 36909 tiles), so two states return the same bits."""
    S = one_potential(wl.twisted_system(Ec))
    P = lsx.Plan(S, 0.05, "lie", 1.0, precision)
    nf = S.nfibres
    c = wl.random_state(S.N, W, seed=6)
    u = np.broadcast_to((np.arange(nf[1]) + 0.5) / nf[1], (1, 2, W, nf[1])).copy()
    got = []
    whole = lsx.State(P, W)
    try:
        for _ in range(2):
            st = lsx.State(P, W)
            sm = lsx.Sampler(st, nf[1], 0, eps=0.1)
            try:
                tiles = int(((S.fibre_info(1)[1] + 15) // 16).sum()) * ((W + 15) // 16)
                print(f"[case] twisted N={S.N} W={W} {precision} tiles={tiles} pick={st.tuning(1)[:2]}", flush=True)
                # layer 2 (the identity) with one pinned shape
                st.set_tuning(2, 1, 2)
                st.upload(c)
                sm.ss_step(torch.as_tensor(u).to("cuda:0"), 1)
                got.append(st.download())
            finally:
                sm.destroy()
                st.destroy()
        assert np.array_equal(got[0].view(np.float64), got[1].view(np.float64))
        whole.set_tuning(1, 1, ks, 2 if precision == "mix_fp32" else 0)
        whole.set_tuning(2, 1, 2)
        whole.upload(c)
        whole.step(1)
        b = whole.download()
        err = (np.linalg.norm(got[0] - b, axis=0) / np.linalg.norm(b, axis=0)).max()
        print(f"  rel diff {err:.2e}")
        assert err < 1e-13
    finally:
        for o in (whole, P, S):
            o.destroy()
