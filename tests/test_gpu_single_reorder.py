"""A single state above the size from which its rows are put into the first pass's order by a launch
of their own (32768 rows), against the same wavepacket in a state of two, whose passes read through
the table.  Even and odd numbers of passes, library and caller arrays, every storage format.

Tolerance: both sides sum the same products of at most 300 terms in another order, 1e-13 a pass.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2103_14897_amd import lsx  # noqa: E402
from paper_2103_14897_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def system():
    S = lsx.System.from_spec(wl.twisted_system(1950.0))
    assert 32768 <= S.N < 40000
    yield S
    S.destroy()


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-13), ("mix_fp32", 1e-6), ("mix_bf16x3", 1e-6)])
@pytest.mark.parametrize("scheme,kappa,nsteps", [("strang", 0.0, 1), ("lie", 0.5, 2)])
@pytest.mark.parametrize("wrapped", [False, True])
def test_reordered_single_state(system, precision, tol, scheme, kappa, nsteps, wrapped):
    print(f"[case] single N={system.N} {precision} {scheme} wrapped={wrapped}", flush=True)
    P = lsx.Plan(system, 5e-3, scheme, kappa, precision)
    c = wl.random_state(system.N, 2, seed=7)
    pair = lsx.State(P, 2)
    mine = torch.as_tensor(np.ascontiguousarray(c[:, :1])).to("cuda:0")
    torch.cuda.synchronize()
    one = lsx.State(P, 1, dev_ptr=mine.data_ptr()) if wrapped else lsx.State(P, 1)
    try:
        pair.upload(c)
        if not wrapped:
            one.upload(c[:, :1])
        for _ in range(2):  # the second call starts from the canonical order again
            one.step(nsteps)
            pair.step(nsteps)
        torch.cuda.synchronize()
        got = mine.cpu().numpy()[:, 0] if wrapped else one.download()[:, 0]
        ref = pair.download()[:, 0]
        err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        print(f"  {err:.2e}")
        assert err < tol * 3 * 2 * nsteps
    finally:
        one.destroy()
        pair.destroy()
        P.destroy()
