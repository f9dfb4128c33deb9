"""The proposal network's forward and backward kernels for every kind of input count: 4 and 5 (compiled
in), fewer, other and the largest (read at run time), over a partial chunk of rows and over several
chunks per wave, whose inputs are loaded a chunk ahead.

Tolerances as for the network's other tests: FP32 rounding of 64-term sums, 1e-5 of the largest logit,
1e-4 of the gradient's norm.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import stochastic as sto  # noqa: E402
from paper_2103_14897_amd import lsx  # noqa: E402
from paper_2103_14897_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [17, 150001])
@pytest.mark.parametrize("nin", [1, 3, 4, 5, 8])
def test_mlp_input_counts(nin, M):
    print(f"[case] mlp nin={nin} M={M}", flush=True)
    rng = np.random.default_rng(nin)
    theta = (wl.mlp_init(nin, 64, seed=nin) + 0.1 * rng.standard_normal(64 * nin + 64 * 64 + 64 * 3 + 1)).astype(np.float32)
    X = rng.standard_normal((M, nin)).astype(np.float32)
    dz = rng.standard_normal(M).astype(np.float32)
    net = lsx.Mlp(nin)
    try:
        net.set(theta)
        Xd, dzd = torch.as_tensor(X).to("cuda:0"), torch.as_tensor(dz).to("cuda:0")
        z = torch.zeros(M, dtype=torch.float32, device="cuda:0")
        g = torch.zeros(net.nparams, dtype=torch.float32, device="cuda:0")
        net.forward(Xd, M, z)
        net.backward(Xd, M, dzd, g)
        t64, X64 = theta.astype(np.float64), X.astype(np.float64)
        zref = sto.mlp_forward(t64, X64)
        gref = sto.mlp_backward(t64, X64, dz.astype(np.float64))
        assert np.abs(z.cpu().numpy() - zref).max() < 1e-5 * max(1.0, np.abs(zref).max())
        assert np.linalg.norm(g.cpu().numpy() - gref) < 1e-4 * np.linalg.norm(gref)
    finally:
        net.destroy()
