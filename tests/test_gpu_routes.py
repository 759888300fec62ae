"""Branches of the launch rules at their edges: tile orders with lanes that do not fill a
wave, staged tiles with a part-filled last wave, poll blocks as repeated smaller graphs,
and a batch whose problems end one after another."""
import numpy as np
import pytest

import oracle
from paper_1411_4439_amd import workload as W
from tests.gpu_util import dev, gpu_lib, host

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _reset_tuning():
    yield
    gpu_lib().hisq_set_tuning(0)


def _setup(H, L, n, seed=901, **k):
    U, N = W.make_links(L, 0.3, seed)
    return U, N, H.Links(L, dev(U), dev(N), **k), W.make_sources(L, n, seed + 1)


# lattices whose x-y planes and time slices hold whole tiles of one wave: 12, 9, 21, 10
# and 21 sites
@pytest.mark.parametrize("L,n,nr", [((12, 8, 8, 4), 5, 1), ((18, 4, 8, 4), 7, 1), ((14, 6, 8, 4), 3, 1),
                                    ((10, 4, 8, 4), 6, 1), ((14, 6, 8, 4), 6, 2)])
def test_xcd_orders_with_lanes_that_do_not_fill_a_wave(L, n, nr):
    H = gpu_lib()
    U, N, links, b = _setup(H, L, n)
    for prec, nk in ((H.PREC_F64, H.NAIK_FULL), (H.PREC_F32, H.NAIK_R14)):
        v = b if prec == H.PREC_F64 else b.astype(np.complex64)
        for layout in (H.LAYOUT_SITE, H.LAYOUT_COLOUR):
            f = dev(v if layout == H.LAYOUT_SITE else np.ascontiguousarray(v.transpose(1, 0, 2)))
            H.hisq_set_tuning(1, n, 64, 0)
            want = host(H.dslash(links, 1, f, prec, nk, layout=layout))
            for order in (0, 1, 2, 3):
                H.hisq_set_tuning(1, nr, 64, order)
                assert np.array_equal(host(H.dslash(links, 1, f, prec, nk, layout=layout)), want), order
    for mode, nk in ((H.MODE_FP64, H.NAIK_FULL), (H.MODE_MIXED, H.NAIK_R14)):
        for order in (2, 3):
            H.hisq_set_tuning(1, nr, 64, order)
            x, st, info = H.solve(links, 0.2, dev(b), mode=mode, naik=nk)
            assert st == H.HISQ_OK
            assert (info["rhs_per_thread"], info["tile_order"], info["eo_tile_order"]) == (nr, order, order)
            assert oracle.residual(L, U, N, 0.2, b, host(x)).max() <= 1e-10


@pytest.mark.parametrize("n", [1, 2, 4, 8])
@pytest.mark.parametrize("L", [(4, 4, 4, 4), (8, 8, 8, 4)])
def test_staged_tiles_with_a_part_filled_last_wave(L, n):
    """Every staged tile of the plain Dslash that does not fill its waves, in both field
    orders: the bits of the unstaged tile."""
    H = gpu_lib()
    U, N, links, b = _setup(H, L, n, r13=True, r9=True)
    ran = 0
    for prec, nk in ((H.PREC_F64, H.NAIK_FULL), (H.PREC_F32, H.NAIK_FULL), (H.PREC_F32, H.NAIK_R14),
                     (H.PREC_F32, H.NAIK_R13), (H.PREC_F32, H.NAIK_R9)):
        v = b if prec == H.PREC_F64 else b.astype(np.complex64)
        for layout in (H.LAYOUT_SITE, H.LAYOUT_COLOUR):
            f = dev(v if layout == H.LAYOUT_SITE else np.ascontiguousarray(v.transpose(1, 0, 2)))
            for nr in (d for d in (1, 2, 4, 8) if n % d == 0):
                H.hisq_set_tuning(1, nr, 64, 1, 0)
                want = host(H.dslash(links, 0, f, prec, nk, layout=layout))
                for rows in (d for d in range(1, 9) if L[1] % d == 0):
                    used = rows * (L[0] // 2) * (n // nr)
                    if used % 64 == 0 or used > 512:
                        continue
                    H.hisq_set_tuning(1, nr, 64, 1, rows)
                    assert np.array_equal(host(H.dslash(links, 0, f, prec, nk, layout=layout)), want), (nr, rows)
                    ran += 1
    assert ran > 0


@pytest.mark.parametrize("poll", [8, 16, 17, 18, 26, 32, 64])
def test_poll_blocks_as_repeated_graphs(poll):
    """Blocks of up to 16 iterations and those without a divisor of 8 to 16 (17) are one
    graph, the others a smaller one several times; none changes a bit against launches
    without a graph, or the number of polls."""
    H = gpu_lib()
    L, n = (8, 6, 4, 10), 3
    U, N, links, b = _setup(H, L, n)
    H.hisq_set_tuning(2)
    for mode, nk in ((H.MODE_FP64, H.NAIK_FULL), (H.MODE_MIXED, H.NAIK_R14)):
        got = []
        for graph in (0, 1):
            x, st, info = H.solve(links, 0.05, dev(b), mode=mode, naik=nk, poll_every=poll, use_graph=graph)
            assert st == H.HISQ_OK
            got.append((host(x), info["iters"], info["polls"], info["reliable_updates"]))
        assert np.array_equal(got[0][0], got[1][0]) and got[0][1:] == got[1][1:]
        assert oracle.residual(L, U, N, 0.05, b, got[1][0]).max() <= 1e-10


def test_split_kernels_run_in_small_solves():
    """The built-in choice of a small solve adds the directions in another order than one
    rhs per lane does: other bits, the same solution."""
    H = gpu_lib()
    L = (6, 4, 6, 4)
    U, N, links, b = _setup(H, L, 5)
    H.hisq_set_tuning(2)
    x, st, _ = H.solve(links, 0.1, dev(b))
    H.hisq_set_tuning(1, 1, 128, 0)
    y, _, _ = H.solve(links, 0.1, dev(b))
    assert st == H.HISQ_OK and not np.array_equal(host(x), host(y))
    assert np.abs(host(x) - host(y)).max() <= 1e-9 * np.abs(host(y)).max()


# the problem that runs last: on split kernels, on one rhs per lane, and too large to
# leave the batched kernels
@pytest.mark.parametrize("last,n", [((6, 4, 6, 4), 3), ((8, 8, 8, 8), 5), ((16, 16, 8, 8), 5)])
@pytest.mark.parametrize("mode", ["fp64", "mixed"])
@pytest.mark.parametrize("poll", [4, 18])
def test_batch_whose_problems_end_one_after_another(last, n, mode, poll):
    H = gpu_lib()
    import torch
    md, nk = (H.MODE_FP64, H.NAIK_FULL) if mode == "fp64" else (H.MODE_MIXED, H.NAIK_R14)
    shapes = [((8, 8, 8, 4), 2, 1.0), (last, n, 0.05), ((4, 4, 6, 4), 8, 0.3)]
    made = [_setup(H, L, k, 921 + 10 * j) for j, (L, k, _) in enumerate(shapes)]
    res = []
    for graph in (0, 1):
        probs, xs, keep = [], [], []
        for (L, k, m), (U, N, links, b) in zip(shapes, made):
            bd = dev(b)
            x = torch.empty_like(bd)
            keep.append(bd)
            xs.append(x)
            probs.append(H.Problem(H.geom(L), m, k, links.f64.data_ptr(), links.f32r14.data_ptr(), bd.data_ptr(),
                                   x.data_ptr()))
        p = H.hisq_default_params(mode=md, naik=nk, poll_every=poll, use_graph=graph)
        ws = H.empty_bytes(H.hisq_batched_workspace_bytes(probs, md))
        H.hisq_set_tuning(2)
        st, infos = H.hisq_cg_solve_batched(probs, p, ws)
        assert st == H.HISQ_OK
        res.append(([host(x) for x in xs], [list(i.iters) for i in infos], infos[0].polls))
        its = [i.total_iters for i in infos]
        assert its[0] + poll < its[2] and its[2] + poll < its[1], its  # each leaves in a poll of its own
    assert all(np.array_equal(a, c) for a, c in zip(res[0][0], res[1][0])) and res[0][1:] == res[1][1:]
    for (L, _, m), (U, N, _, b), x in zip(shapes, made, res[1][0]):
        assert oracle.residual(L, U, N, m, b, x).max() <= 1e-10
