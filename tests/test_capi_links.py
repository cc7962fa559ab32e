"""Argument checks of the calls that take several links (no GPU needed: they
are made before anything is enqueued)."""
import ctypes as ct

import pytest


@pytest.mark.parametrize("n, bad, code", [(0, None, "LSDF_E_SHAPE"), (17, None, "LSDF_E_SHAPE"),
                                          (2, "nt", "LSDF_E_SHAPE"), (2, "verts", "LSDF_E_INVALID_ARG"),
                                          (2, "comp", "LSDF_E_SHAPE"), (2, "dtype", "LSDF_E_UNSUPPORTED")])
def test_links_arguments(n, bad, code):
    from paper_2309_12543_amd import lsdf as B
    lib = B.load_library()
    k = 17
    ptr, comp = ct.c_void_p(4096), (ct.c_int32 * 2)(0, 11 if bad == "comp" else 12)
    ptrs = (ct.c_void_p * k)(*[4096] * k)
    verts = (ct.c_void_p * k)(4096, None if bad == "verts" else 4096)
    nv, nt = (ct.c_int32 * k)(*[8] * k), (ct.c_int32 * k)(12, 0 if bad == "nt" else 12)
    comps, ncomp = (ct.c_void_p * k)(None, ct.addressof(comp)), (ct.c_int32 * k)(0, 1)
    grids = (B.lsdf_grid * k)()
    for g in grids:
        for a in range(3):
            g.lo[a], g.hi[a], g.n[a] = 0.0, 1.0, 4
    if bad == "dtype":
        grids[1].dtype = 7
    want = getattr(B, code)
    assert lib.lsdf_build_link_sdfs(n, verts, nv, ptrs, nt, comps, ncomp, grids, ptr, None) == want
    assert lib.lsdf_sdf_labels_links(n, verts, nv, ptrs, nt, comps, ncomp, grids, ptr, ptrs, 5, ptrs, None) == want


@pytest.mark.parametrize("order", ["C", "F", "list"])
def test_dh_rows_hold_the_table(order):
    import numpy as np
    from paper_2309_12543_amd import lsdf as B
    table = np.random.default_rng(3).uniform(-2, 2, size=(5, 4))
    given = table.tolist() if order == "list" else np.array(table, order=order)
    rows, dof = B._dh_rows(given)
    assert dof == 5
    for r, want in zip(rows, table.astype(np.float32)):
        assert [r.a, r.alpha, r.d, r.theta_offset] == want.tolist()
