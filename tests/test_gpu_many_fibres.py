"""A layer of more distinct fibres than a grid's second dimension holds: 66049 fibres of 65 rows, every
one with its own kinetic share, go through the block rounds of the eigensolver together.  The
propagators of the first and the last, and of those around number 65535, against a dense exponential."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2103_14897_amd import lsx  # noqa: E402

pytestmark = pytest.mark.gpu


def test_more_matrices_than_65535():
    tau, v, half = 0.5, 0.3, (32, 128, 128)
    r = np.array([np.sqrt(2.0) / (h + 0.5) for h in half])  # |r m|^2 / 2 <= 1 for |m| <= half
    S = lsx.System.blocks([np.array([[x]]) for x in r], [[0], [1], [2]], 1.0, [(0, 1), (1, 2), (2, 3)],
                          [{(1,): v, (-1,): v}, {}, {}])
    print(f"[case] N={S.N} fibres {S.nfibres}", flush=True)
    assert S.nfibres[1] == 257 * 257 > 65535
    P = None
    try:
        P = lsx.Plan(S, tau, "lie", 0.0, "fp64")
        mn = S.index()
        ptr, rows = S.fibres(1)
        for f in (0, 1, 32768, 65534, 65535, 65536, 65537, S.nfibres[1] - 1):
            own = mn[rows[ptr[f]:ptr[f + 1]]]
            assert len(own) == 65 and np.array_equal(np.diff(own[:, 0]), np.ones(64))
            K = own @ r
            H = np.diag(K * K / 6.0) + v * (np.eye(65, k=1) + np.eye(65, k=-1))
            lam, V = np.linalg.eigh(H)
            ref = (V * np.exp(-1j * tau * lam)) @ V.T
            err = np.abs(P.propagator(1, 0, f) - ref).max()
            # eigenvectors and values to a few hundred roundings of norms of order one
            assert err < 1e-12, (f, err)
    finally:
        if P is not None:
            P.destroy()
        S.destroy()
