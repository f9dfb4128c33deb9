"""Mass and energy reductions through the C-ABI at the edges of their sweeps: row counts around the
workgroup's rows and the slab split, column counts around the column block, stencils whose term
count does and does not fill a load group, a potential with an entry at index zero.  Each column's
values against the oracle-independent definition in NumPy, and the same bits whichever of the two
is asked for."""
import numpy as np
import pytest

from paper_2103_14897_amd import lsx
from paper_2103_14897_amd import workloads as wl

pytestmark = pytest.mark.gpu

SYSTEMS = {
    "one_row": (wl.chain_system(1.0), None),
    "chain": (wl.chain_system(2000.0), None),
    "chain_v0": (wl.chain_system(700.0, pot1={(0,): 0.3, (1,): 0.5 + 0.2j, (-1,): 0.5 - 0.2j, (3,): 0.1, (-3,): 0.1},
                                 pot2={(2,): 0.4j, (-2,): -0.4j}), None),
    "free": (wl.chain_system(700.0, pot1={}, pot2={}), None),
    "twisted": (wl.twisted_system(900.0), None),
    "trilayer": (wl.chain_layers(900.0), "layers"),
    "example3": (wl.example3_system(60.0), "blocks"),
}


def _energy(S, pots, owns, Rs, c):
    """sum |K|^2/2 |c|^2 + Re conj(c) V c with V by its definition (eq. 3.6), row by row."""
    mn = S.index()
    where = {tuple(r): i for i, r in enumerate(mn.tolist())}
    K = sum(mn[:, o:o + R.shape[1]] @ R.T for o, R in Rs)
    out = 0.5 * ((K ** 2).sum(axis=1)[:, None] * np.abs(c) ** 2).sum(axis=0)
    for pot, (o, e) in zip(pots, owns):
        for p, v in pot.items():
            shifted = mn.copy()
            shifted[:, o:e] -= np.asarray(p)
            j = np.array([where.get(tuple(r), -1) for r in shifted.tolist()])
            out += (c.conj() * np.where(j[:, None] >= 0, complex(v) * c[j], 0.0)).real.sum(axis=0)
    return out


@pytest.mark.parametrize("name", list(SYSTEMS))
def test_mass_and_energy_match_their_definition(name):
    spec, kind = SYSTEMS[name]
    if kind == "blocks":
        S = lsx.System.blocks(spec.Rs, spec.groups, spec.Ec, spec.layers, spec.pots)
        off = np.concatenate([[0], np.cumsum([R.shape[1] for R in spec.Rs])])
        Rs, pots = [(off[b], R) for b, R in enumerate(spec.Rs)], spec.pots
        owns = [(off[a], off[b]) for a, b in spec.layers]
    else:
        As = spec.As if kind else [spec.A1, spec.A2]
        d = spec.d
        S = lsx.System.layers(d, As, spec.Ec, spec.cutoff, spec.pots) if kind else lsx.System.from_spec(spec)
        pots = spec.pots if kind else [spec.pot1, spec.pot2]
        Rs = [(j * d, 2.0 * np.pi * np.linalg.inv(A).T) for j, A in enumerate(As)]
        owns = [(j * d, (j + 1) * d) for j in range(len(As))]
    P = lsx.Plan(S, 1e-3, "strang", 0.0, "fp64")
    try:
        for W in (1, 2, 7, 8, 9, 33):
            print(f"[case] observables {name} N={S.N} W={W}", flush=True)
            c = wl.random_state(S.N, W, seed=W) * 1.5
            st = lsx.State(P, W)
            try:
                st.upload(c)
                both = st.observables(lsx.OBS_MASS | lsx.OBS_ENERGY)
                assert np.array_equal(both["mass"], st.observables(lsx.OBS_MASS)["mass"])
                assert np.array_equal(both["energy"], st.observables(lsx.OBS_ENERGY)["energy"])
            finally:
                st.destroy()
            # sums of N terms in a fixed tree: 1e-13 of the sum of their magnitudes
            assert np.allclose(both["mass"], (np.abs(c) ** 2).sum(axis=0), rtol=1e-13, atol=0)
            scale = 2.25 * (spec.Ec * 2.0 * len(pots) + sum(abs(complex(v)) for p in pots for v in p.values()))
            assert np.abs(both["energy"] - _energy(S, pots, owns, Rs, c)).max() <= 1e-13 * scale
    finally:
        P.destroy()
        S.destroy()
