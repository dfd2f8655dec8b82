"""The kernels that finish a call (metric, status), diagnose and project states, at
the edges of their tiles: 4 points per thread, 64 threads per wavefront, up to 4096
(finalize) or 2048 (diagnostics) interior points per tile, 16 rows, modes and points
per turn of the projection."""
import numpy as np
import pytest

import oracle as O
from paper_1706_07413_amd import adscl
from test_gpu_parity import FIELDS, adot_scale, assert_close, gpu_state

pytestmark = pytest.mark.gpu

# N - 2 interior points: one thread's remainder, a wavefront and one more, a tile of
# either kernel and one thread more, several tiles
EDGES = [17, 19, 21, 257, 259, 261, 2049, 2051, 2053, 4095, 4097, 4111, 8195 + 16]


@pytest.mark.parametrize("gauge", [O.GAUGE_BOUNDARY, O.GAUGE_ORIGIN])
@pytest.mark.parametrize("alone", [False, True])
def test_metric_and_diagnostics_at_tile_edges(gauge, alone):
    """`alone`: each grid in a context of its own (the block is sized for it),
    else all in one batch (sized for the largest)."""
    rng = np.random.default_rng(5)
    state = []
    for N in EDGES:
        x = np.linspace(0.0, np.pi / 2, N)
        Phi, Pi = O.init_gaussian(N, 2.0, 0.3)
        state.append((0.4 * np.sin(2.0 * x) ** 3 * np.cos(x) ** 2 * rng.uniform(0.5, 1.0), Pi))
    groups = [[i] for i in range(len(EDGES))] if alone else [list(range(len(EDGES)))]
    for grp in groups:
        print("tile edges", [EDGES[i] for i in grp], gauge, flush=True)
        b = adscl.Batch([EDGES[i] for i in grp], gauge=gauge, a_collapse=0.0)
        b.init(np.concatenate([state[i][0] for i in grp]), np.concatenate([state[i][1] for i in grp]))
        g, d, st = gpu_state(b), b.constraints(), b.status()
        b.close()
        o = 0
        for k, i in enumerate(grp):
            N = EDGES[i]
            Phi, Pi = state[i][0].copy(), state[i][1].copy()
            Phi[0] = Phi[-1] = Pi[-1] = 0.0
            ref = O.constraints(Phi, Pi, gauge=gauge)
            for f, r in zip(FIELDS, (Phi, Pi, ref["A"], ref["delta"], ref["m"])):
                assert_close(g[f][o:o + N], r, "N=%d %s" % (N, f))
            assert abs(st["minA"][k] - min(1.0, ref["A"].min())) <= 1e-12
            # the residuals of the same metric, on the scale of the terms they are differences of
            A, dl, m = (g[f][o:o + N] for f in ("A", "delta", "m"))
            x = O.grid(N)[0][1:-1]
            sc, q = np.sin(x) * np.cos(x), (Phi ** 2 + Pi ** 2)[1:-1]
            RA, Rd = O.residuals(Phi, Pi, A, dl)
            scale_A = np.max(np.abs((1 + 2 * np.sin(x) ** 2) / sc * (1 - A[1:-1]))) + np.max(sc * A[1:-1] * q)
            assert abs(d[k, 0] - np.abs(RA).max()) <= 1e-11 * scale_A, N
            assert abs(d[k, 1] - np.abs(Rd).max()) <= 1e-11 * np.max(sc * q), N
            Ad, Rt = O.adot_residual(Phi, Pi, gauge=gauge)
            assert abs(d[k, 2] - np.abs(Rt[1:-1]).max()) <= 1e-11 * adot_scale(Phi, Pi, A, dl, Ad), N
            assert d[k, 3] == m[-1]
            assert abs(d[k, 4] - O.mass_paper(Phi, Pi, A)) <= 1e-12 * d[k, 4]
            o += N


@pytest.mark.parametrize("N,rows,J", [(17, 1, 1), (257, 15, 16), (255, 16, 15), (259, 17, 17), (271, 33, 31),
                                      (273, 2, 33), (1025, 3, 128), (4097, 1, 16)])
def test_projection_at_tile_edges(N, rows, J):
    rng = np.random.default_rng(7)
    c = rng.uniform(-1.0, 1.0, size=(rows, min(J, 5)))
    eps = rng.uniform(0.05, 0.1, size=rows)
    print("projection", N, rows, J, flush=True)
    b = adscl.Batch([N] * rows, n_modes=J, a_collapse=0.0)
    b.init_modes(eps, c)
    b.step(6, 1e9)
    g = gpu_state(b)
    E, P, F = b.spectrum(J)
    b.close()
    for r in range(rows):
        s = slice(r * N, (r + 1) * N)
        Eo, Po, Fo = O.spectrum(g["Phi"][s], g["Pi"][s], g["A"][s], J)
        assert_close(P[r], Po, "Pihat row %d" % r)
        assert_close(F[r], Fo, "Phihat row %d" % r)
        assert_close(E[r], Eo, "E row %d" % r)


@pytest.mark.parametrize("gauge", [O.GAUGE_BOUNDARY, O.GAUGE_ORIGIN])
def test_a_grid_is_finished_alike_alone_and_beside_larger_ones(gauge):
    """The block is sized for the batch's largest grid: the sums of a smaller one
    must not depend on it, bit for bit."""
    N, big = 129, [129, 2049, 4097]
    Phi, Pi = O.init_gaussian(N, 3.0, 0.2)
    got = []
    for grids in ([N], big[:2], big):
        b = adscl.Batch(grids, gauge=gauge, a_collapse=0.0)
        rest = np.zeros(sum(grids[1:]))
        b.init(np.concatenate([Phi, rest]), np.concatenate([Pi, rest]))
        g, m = gpu_state(b), b.status()["minA"][0]
        b.close()
        got.append([g[f][:N] for f in FIELDS] + [m])
    for other in got[1:]:
        for f, x, y in zip(FIELDS + ("minA",), got[0], other):
            assert np.array_equal(x, y), f
