"""Semi-implicit and random batch steps on both row orders of the kernel: wavepacket counts whose rows
fill whole lines (slabs of the canonical order, parts for large states) and ragged ones (parts), each
column against the same column stepped in a narrow state (slabs), bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2103_14897_amd import lsx  # noqa: E402
from paper_2103_14897_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def twisted():
    S = lsx.System.from_spec(wl.twisted_system(2000.0))  # 36937 rows
    P = lsx.Plan(S, 5e-3, "lie", 1.0, "fp64")
    yield S, P
    P.destroy()
    S.destroy()


# parts: 9, 13, 31, 63 and, by its 151 MB, 256; slabs: 17 and 33 (few lanes), 48 and 248
@pytest.mark.parametrize("W", [9, 13, 17, 31, 33, 48, 63, 248, 256])
def test_wide_states_equal_narrow_ones(twisted, W, monkeypatch):
    monkeypatch.setenv("LSX_AUTOTUNE", "0")
    compare(*twisted, W, (7, 11))


# few rows, whose column blocks are on workgroups of their own: one block, all at once, and more blocks (38
# and 13) than workgroups a row group has (32 and 8)
@pytest.mark.parametrize("Ec,W", [(300.0, 7), (300.0, 100), (300.0, 300), (3000.0, 100)])
def test_small_systems(Ec, W):
    S = lsx.System.from_spec(wl.chain_system(Ec))
    P = lsx.Plan(S, 5e-3, "lie", 1.0, "fp64")
    try:
        compare(S, P, W, (3, 5))
    finally:
        P.destroy()
        S.destroy()


def compare(S, P, W, p):
    print(f"[case] semi-implicit N={S.N} W={W}", flush=True)
    cols = sorted({0, 7, 8, W // 2, W - 2, W - 1} & set(range(W)))
    g = torch.Generator(device="cuda").manual_seed(W)
    c = torch.view_as_complex(torch.randn((S.N, W, 2), dtype=torch.float64, device="cuda", generator=g))
    d = c[:, cols].contiguous()
    u = torch.as_tensor(wl.uniforms((1, 2, W, max(p)), seed=1), device="cuda")
    wide, narrow = lsx.State(P, W, dev_ptr=c.data_ptr()), lsx.State(P, len(cols), dev_ptr=d.data_ptr())
    sw, sn = lsx.Sampler(wide, *p), lsx.Sampler(narrow, *p)
    try:
        for st in (wide, narrow):
            st.si_step(3)
        sw.rb_step(u, 1)
        sn.rb_step(u[:, :, cols].contiguous(), 1)
        torch.cuda.synchronize()
        assert torch.equal(torch.view_as_real(c[:, cols]), torch.view_as_real(d))
        assert bool(torch.isfinite(torch.view_as_real(d)).all())
    finally:
        for o in (sw, sn, wide, narrow):
            o.destroy()
