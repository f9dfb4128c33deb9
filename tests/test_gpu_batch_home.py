"""Batched steps after a member state swapped its two arrays and an allocation failed: the batch keeps
the table of its copies home (results of an odd number of passes), so the failed call reports
LSX_E_OOM and the next one gives the members' own steps."""
import numpy as np
import pytest

from paper_2103_14897_amd import lsx
from paper_2103_14897_amd import workloads as wl

pytestmark = pytest.mark.gpu


def test_failed_allocation_after_a_swap(monkeypatch):
    specs = [(wl.chain_system(700.0), 5), (wl.chain_system(1100.0), 17), (wl.twisted_system(200.0), 16)]
    items, alone = [], []
    for k, (spec, W) in enumerate(specs):
        S = lsx.System.from_spec(spec)
        P = lsx.Plan(S, 1e-3, "strang", 0.0, "mix_fp32")
        c = wl.random_state(S.N, W, seed=k)
        for out in (items, alone):
            st = lsx.State(P, W)
            st.upload(c)
            out.append((S, P, st))
    print(f"[case] batch of N={[S.N for S, _, _ in items]}, allocation failing after a swap", flush=True)
    B = lsx.Batch([st for _, _, st in items])
    try:
        B.step(1)  # three passes: copied home
        before = [st.device_ptr() for _, _, st in items]
        items[1][2].step(2)  # five passes on one member alone: its arrays swap roles
        assert items[1][2].device_ptr() != before[1]
        live = lsx.live_buffers()
        # the first allocation of the call, before anything is launched
        monkeypatch.setenv("LSX_TEST_FAIL_ALLOC", "1")
        with pytest.raises(lsx.LsxError) as e:
            B.step(1)
        assert e.value.code == lsx.LSX_E_OOM
        monkeypatch.delenv("LSX_TEST_FAIL_ALLOC")
        assert lsx.live_buffers() <= live  # argument tables given back, nothing held twice
        B.step(1)
        B.step(2)
        for k, (_, _, st) in enumerate(alone):
            for n in ([1, 2] if k == 1 else [1]) + [1, 2]:
                st.step(n)
        for (S, _, a), (_, _, b) in zip(items, alone):
            x, y = a.download(), b.download()
            # FP32 rounding of products summed in another tile shape, tau |V| 2^-24 a pass, 16 passes
            assert (np.linalg.norm(x - y, axis=0) / np.linalg.norm(y, axis=0)).max() < 16 * 1e-3 * 2.0 ** -24 * 16
    finally:
        B.destroy()
        for out in (items, alone):
            for _, _, st in out:
                st.destroy()
        for S, P, _ in items:
            P.destroy()
            S.destroy()
