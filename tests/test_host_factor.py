"""The host factorisation at the edges of its tiles (no GPU)."""
import numpy as np
import pytest
import scipy.sparse as sp

import scgen

P = pytest.importorskip("paper_2509_21037_amd")


@pytest.mark.parametrize("kind,elems", [("heat", (1, 1)), ("heat", (5, 4)), ("heat", (13, 9)), ("heat", (3, 4, 3)),
                                        ("elasticity", (2, 2, 1)), ("elasticity", (4, 3, 4)), ("tri", 17)])
@pytest.mark.parametrize("leaf", [4, 23, 200])
def test_factor_at_tile_edges(kind, elems, leaf):
    """Supernodes of every width and row count that a few cuts of small meshes
    give (one column, remainders of the 16 x 8 tiles and of the 32-column
    blocks, rows in runs and scattered): L L^T is the permuted matrix up to the
    rounding of a backward stable factorisation (n eps, entry by entry), in the
    triangle that is read (the generator's K is symmetric up to rounding)."""
    s = scgen.simplex_subdomain(2, elems, 5) if kind == "tri" else scgen.box_subdomain(kind, elems, 0.25, 5)
    K = sp.csr_matrix((s.val, s.col, s.rowptr), shape=(s.n, s.n)).toarray()
    r = P.host_analyze(s, want_L=True, leaf_nodes=leaf)
    L = np.tril(r["L"])
    A = K[np.ix_(r["perm"], r["perm"])]
    bound = (s.n + 2) * np.finfo(float).eps * (np.abs(L) @ np.abs(L).T)
    assert (np.tril(np.abs(L @ L.T - A)) <= 2 * bound).all()
