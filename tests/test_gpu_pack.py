"""Packing of links that are not finite: what each storage refuses, and what it lets through."""
import numpy as np
import pytest

from paper_1411_4439_amd import workload as W
from tests.gpu_util import dev, gpu_lib, host

pytestmark = pytest.mark.gpu

L = (6, 4, 6, 4)  # 576 sites: the last packing work-group is ragged


def _bad_links(value, where):
    U, N = W.make_links(L, 0.3, 851)
    N = N.copy()
    if where == "all":
        N[...] = value
    else:
        N[2, 575 if where == "last" else 17, 1, 2] = value
    return U, N


@pytest.mark.parametrize("value", [np.nan, -np.nan, complex(0, np.nan), np.inf])
@pytest.mark.parametrize("where", ["one", "last", "all"])
def test_r9_refuses_links_that_are_not_finite(value, where):
    """r9 stores scale * exp(iH): a NaN or infinite Naik link has no such form, and
    a buffer left valid would hold finite matrices for it."""
    H = gpu_lib()
    U, N = _bad_links(value, where)
    buf = H.empty_bytes(H.hisq_links_bytes(L, H.PREC_F32, H.NAIK_R9))
    with pytest.raises(H.HisqError) as e:
        H.hisq_pack_links(L, dev(U), dev(N), H.PREC_F32, H.NAIK_R9, buf)
    assert e.value.code == H.HISQ_EPACK
    v = dev(W.make_sources(L, 2, 852).astype(np.complex64))
    with pytest.raises(H.HisqError) as e:
        H.hisq_dslash(L, 1, 2, H.PREC_F32, H.NAIK_R9, H.LAYOUT_SITE, buf, v, v.clone())
    assert e.value.code == H.HISQ_EINVAL


@pytest.mark.parametrize("naik", ["full", "r14", "r13"])
def test_other_storages_keep_a_nan(naik):
    """The forms that store the elements of rows 0 and 1 take a NaN link and return NaN
    at the sites that it reaches, nowhere else."""
    H = gpu_lib()
    nk = {"full": H.NAIK_FULL, "r14": H.NAIK_R14, "r13": H.NAIK_R13}[naik]
    U, N = _bad_links(np.nan, "one")
    buf = H.empty_bytes(H.hisq_links_bytes(L, H.PREC_F32, nk))
    H.hisq_pack_links(L, dev(U), dev(N), H.PREC_F32, nk, buf)
    v = dev(W.make_sources(L, 2, 852).astype(np.complex64))
    sites = 0
    for parity in (0, 1):
        out = v.clone()
        H.hisq_dslash(L, parity, 2, H.PREC_F32, nk, H.LAYOUT_SITE, buf, v, out)
        sites += np.isnan(host(out)).any(axis=(1, 2)).sum()
    assert sites == 2  # the link's root and the site three hops on
