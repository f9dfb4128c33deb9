"""A caller's captured graph of a single state's steps, replayed several times, where the library reorders
the state first (32768 rows or more, tiles of several fibres): a library-owned state keeps its array over a call of an even
number of passes, so every replay starts from the result of the one before.  Calls of an odd number
are replayed on a wrapped state, whose array never changes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2103_14897_amd import lsx  # noqa: E402
from paper_2103_14897_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu


# tiles of several fibres, which read a reordered state, and of single ones, which read through the table
@pytest.mark.parametrize("shape", [(8, -8), (1, -4)])
@pytest.mark.parametrize("owned,scheme,call", [
    (True, "lie", lambda st, s: st.step(2, s)),             # four passes
    (True, "strang", lambda st, s: st.fibre_pass(1, 0, 2, s)),
    (False, "lie", lambda st, s: st.step(2, s)),
    (False, "strang", lambda st, s: st.step(1, s)),         # three passes
])
def test_replays_follow_each_other(owned, scheme, call, shape):
    S = lsx.System.from_spec(wl.twisted_system(2000.0))
    assert S.N >= 32768
    print(f"[case] capture N={S.N} owned={owned} {scheme} shape={shape}", flush=True)
    P = lsx.Plan(S, 2e-3, scheme, 0.5, "fp64")
    c = torch.as_tensor(wl.random_state(S.N, 1, seed=8)).to("cuda:0").reshape(S.N, 1).contiguous()
    d = c.clone()
    st = lsx.State(P, 1, dev_ptr=None if owned else d.data_ptr())
    e = c.clone()
    ref = lsx.State(P, 1, dev_ptr=e.data_ptr())
    try:
        for x in (st, ref):
            for layer in (1, 2):
                x.set_tuning(layer, *shape)
            x.set_store_mode(0)
            x.upload(c.cpu().numpy())
        torch.cuda.synchronize()
        at = st.device_ptr()
        s = torch.cuda.Stream()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            call(st, s)
        assert st.device_ptr() == at
        for k in range(4):
            g.replay()
            torch.cuda.synchronize()
            call(ref, None)
            mass = st.observables(lsx.OBS_MASS)["mass"]  # eager work between the replays
            a, b = st.download(), ref.download()
            assert np.array_equal(a, b), k
            assert abs(mass[0] - 1.0) < 1e-12
        del g
    finally:
        for o in (st, ref, P, S):
            o.destroy()
