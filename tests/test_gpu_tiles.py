"""Tiles of bundles that are no power of two, and the split kernels of small solves.

One rhs per lane (any bundle size; where the site's lanes do not divide a wave,
the last lanes idle) must give the bits of the n-rhs-per-lane tile, because the
sums over slots run in the same order.  The split form (four lanes per site and
rhs, the built-in choice for launches that do not fill the chip) adds the
directions in another order: a solve on it has to reach the true residual.
"""
import numpy as np
import pytest

import oracle
from paper_1411_4439_amd import workload as W
from tests.gpu_util import dev, gpu_lib, host, rel_l2_per_rhs

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _reset_tuning():
    yield
    gpu_lib().hisq_set_tuning(0)


@pytest.mark.parametrize("n,nr", [(3, 1), (5, 1), (6, 1), (6, 2), (7, 1)])
@pytest.mark.parametrize("L", [(6, 4, 6, 4), (8, 8, 8, 4)])  # ragged last tile; whole tiles, XCD order
def test_lanes_that_do_not_fill_a_wave(L, n, nr):
    H = gpu_lib()
    U, N = W.make_links(L, 0.3, 811)
    links = H.Links(L, dev(U), dev(N))
    v = W.make_sources(L, n, 812)
    want = oracle.dslash_eo(L, U, N, v, 1)
    for prec, nk, tol in ((H.PREC_F64, H.NAIK_FULL, 1e-13), (H.PREC_F32, H.NAIK_R14, 1e-6)):
        for layout in (H.LAYOUT_SITE, H.LAYOUT_COLOUR):
            f = dev(v if layout == H.LAYOUT_SITE else np.ascontiguousarray(v.transpose(1, 0, 2)))
            f = f if prec == H.PREC_F64 else f.to(dev(v[:1].astype(np.complex64)).dtype)
            got = []
            for tile in ((n, 64, 0), (nr, 64, 0), (nr, 128, 1), (nr, 256, 3)):
                H.hisq_set_tuning(1, *tile)
                got.append(host(H.dslash(links, 1, f, prec, nk, layout=layout)))
            for g in got[1:]:
                assert np.array_equal(g, got[0])
            g = got[0] if layout == H.LAYOUT_SITE else got[0].transpose(1, 0, 2)
            assert rel_l2_per_rhs(g.astype(np.complex128), want) <= tol


@pytest.mark.parametrize("n", [1, 2, 3, 5, 6, 7, 8])
@pytest.mark.parametrize("L", [(4, 4, 4, 4), (6, 4, 6, 4)])
def test_small_solves_on_the_split_kernels(L, n):
    H = gpu_lib()
    m = 0.1
    U, N = W.make_links(L, 0.3, 821)
    links = H.Links(L, dev(U), dev(N), r13=True, r9=True)
    b = W.make_sources(L, n, 822)
    H.hisq_set_tuning(2)
    for mode, nk in ((H.MODE_FP64, H.NAIK_FULL), (H.MODE_MIXED, H.NAIK_FULL), (H.MODE_MIXED, H.NAIK_R14),
                     (H.MODE_MIXED, H.NAIK_R13), (H.MODE_MIXED, H.NAIK_R9)):
        x, st, info = H.solve(links, m, dev(b), mode=mode, naik=nk)
        assert st == H.HISQ_OK and info["rhs_per_thread"] == 1
        assert oracle.residual(L, U, N, m, b, host(x)).max() <= 1e-10
        y, _, _ = H.solve(links, m, dev(b), mode=mode, naik=nk)
        assert np.array_equal(host(x), host(y))


def test_forced_one_rhs_per_lane_solve():
    """A 7-rhs mixed solve with 7 lanes per site in every kernel, reductions included."""
    H = gpu_lib()
    L, m, n = (8, 6, 4, 10), 0.1, 7
    U, N = W.make_links(L, 0.3, 831)
    links = H.Links(L, dev(U), dev(N))
    b = W.make_sources(L, n, 832)
    H.hisq_set_tuning(1, 1, 64, 0)
    for mode, nk in ((H.MODE_FP64, H.NAIK_FULL), (H.MODE_MIXED, H.NAIK_R14)):
        x, st, info = H.solve(links, m, dev(b), mode=mode, naik=nk)
        assert st == H.HISQ_OK and info["rhs_per_thread"] == 1
        assert oracle.residual(L, U, N, m, b, host(x)).max() <= 1e-10


@pytest.mark.parametrize("L", [(6, 4, 6, 4), (12, 12, 4, 4), (10, 8, 8, 4)])
@pytest.mark.parametrize("n", [1, 3, 5, 8])
def test_staged_rows_in_both_field_orders(L, n):
    """Staged x-rows on site-major fields, and tiles whose last wave is not full
    (L0/2 * lanes * rows no multiple of 64), give the bits of the unstaged tile of
    the same rhs per lane."""
    H = gpu_lib()
    U, N = W.make_links(L, 0.3, 841)
    links = H.Links(L, dev(U), dev(N))
    v = W.make_sources(L, n, 842)
    want = oracle.dslash_eo(L, U, N, v, 0)
    for prec, nk, tol in ((H.PREC_F64, H.NAIK_FULL, 1e-13), (H.PREC_F32, H.NAIK_R14, 1e-6)):
        for layout in (H.LAYOUT_SITE, H.LAYOUT_COLOUR):
            f = dev(v if layout == H.LAYOUT_SITE else np.ascontiguousarray(v.transpose(1, 0, 2)))
            f = f if prec == H.PREC_F64 else f.to(dev(v[:1].astype(np.complex64)).dtype)
            for nr in {n, 1}:
                H.hisq_set_tuning(1, nr, 64, 0, 0)
                plain = host(H.dslash(links, 0, f, prec, nk, layout=layout))
                g = plain if layout == H.LAYOUT_SITE else plain.transpose(1, 0, 2)
                assert rel_l2_per_rhs(g.astype(np.complex128), want) <= tol
                for rows, order in ((1, 0), (2, 1), (4, 2), (4, 3)):
                    H.hisq_set_tuning(1, nr, 64, order, rows)
                    assert np.array_equal(host(H.dslash(links, 0, f, prec, nk, layout=layout)), plain), (nr, rows)
